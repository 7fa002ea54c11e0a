// The slots of pinned memory that COCG's step counts come through, on the host
// alone: the runtime's calls are stand-ins here.  Prints "ok" or what is wrong.
#include "step_flag.hpp"

#include <cstdio>
#include <cstdlib>
#include <thread>

static bool g_no_memory = false;
static hipError_t g_sync = hipSuccess, g_query = hipErrorNotReady;
static std::atomic<int> g_copies{0}, g_queries{0};

extern "C" {
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    if (g_no_memory) return hipErrorOutOfMemory;
    *p = std::aligned_alloc(64, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    ++g_copies;
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return g_sync; }
hipError_t hipStreamQuery(hipStream_t) {
    ++g_queries;
    return g_query;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
}
namespace chaff {
void set_error(const std::string&) {}
chaff_status fail(chaff_status st, const std::string&) { return st; }
}  // namespace chaff
using namespace chaff;

static void check(bool ok, const char* what) {
    if (ok) return;
    std::printf("wrong: %s\n", what);
    std::exit(1);
}
static int free_slots() {
    std::vector<int> got;
    int s;
    while (g_flag_page.take(s)) got.push_back(s);
    for (int k : got) g_flag_page.give(k);
    return (int)got.size();
}
static void publish(StepFlag& f, uint32_t seq, uint32_t n) {
    __atomic_store_n(f.p, (uint64_t)seq << 32 | n, __ATOMIC_RELEASE);
}

int main(int argc, char**) {
    const int32_t counter = 41;
    int32_t n = 0;
    if (argc > 1) {   // no pinned memory: the count is copied
        g_no_memory = true;
        StepFlag f(nullptr);
        f.take();
        check(!f.p, "no slot without memory");
        check(f.wait(&counter, n) == CHAFF_OK && n == 41 && g_copies == 1, "the count is copied");
        std::puts("ok");
        return 0;
    }
    check(free_slots() == 64, "64 slots");
    {   // the solve's own sequence number alone counts
        StepFlag f(nullptr);
        f.take();
        check(f.p && free_slots() == 63, "a slot is taken");
        check(*f.p == 0, "and cleared");
        publish(f, 7, 3);
        f.seq = 8;
        check(!f.read(n), "an earlier step's count");
        std::thread late([&] {
            std::this_thread::sleep_for(std::chrono::milliseconds(60));
            publish(f, 8, 5);
        });
        check(f.wait(&counter, n) == CHAFF_OK && n == 5, "the count of the step");
        late.join();
        check(g_queries >= 1 && g_queries <= 4, "the stream is asked every 20 ms");
        f.seq = 9;
        g_query = hipSuccess;   // the stream is done and no count came
        check(f.wait(&counter, n) == CHAFF_EHIP, "a step without its count");
        g_query = hipErrorUnknown;
        check(f.wait(&counter, n) == CHAFF_EHIP, "a stream that failed");
    }   // left without give(), as a solve that returns early
    check(free_slots() == 64, "an early return gives its slot back");
    for (int i = 0; i < 200; ++i) {
        StepFlag f(nullptr);
        f.take();
        check(f.p, "200 early returns leave slots");
    }
    {
        StepFlag f(nullptr);
        f.take();
        f.give();
        check(!f.p && free_slots() == 64, "given back once");
    }
    {   // none left: the count is copied
        std::vector<int> got(64);
        for (int& s : got) check(g_flag_page.take(s), "64 taken");
        StepFlag f(nullptr);
        f.take();
        g_copies = 0;
        check(!f.p && f.wait(&counter, n) == CHAFF_OK && n == 41 && g_copies == 1, "the 65th solve copies");
        for (int s : got) g_flag_page.give(s);
    }
    {   // threads never share a slot
        std::atomic<int> owner[64] = {};
        std::atomic<bool> shared{false};
        auto work = [&] {
            for (int i = 0; i < 20000; ++i) {
                StepFlag f(nullptr);
                f.take();
                if (!f.p) continue;
                const int s = f.slot;
                if (owner[s].fetch_add(1) != 0) shared = true;
                owner[s].fetch_sub(1);
            }
        };
        std::vector<std::thread> t;
        for (int i = 0; i < 4; ++i) t.emplace_back(work);
        for (auto& x : t) x.join();
        check(!shared && free_slots() == 64, "a slot for one solve at a time");
    }
    {   // a stream that does not drain keeps its slot
        g_sync = hipErrorUnknown;
        StepFlag f(nullptr);
        f.take();
    }
    g_sync = hipSuccess;
    check(free_slots() == 63, "a failed stream keeps its slot");
    std::puts("ok");
    return 0;
}
