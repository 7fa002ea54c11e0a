// Small solves: one workgroup takes one system (cloud, incidence) from its
// excitation to its currents in a single launch.
//
// The lockstep solver (krylov_impl.hpp) spends six launches and a look at pinned
// memory on a COCG step (30 us whatever the system's size), twice that and a host
// synchronisation on a GMRES step (100 us and more), and 0.3 ms on a solve beside
// them; a cloud of a few thousand sparsely coupled wires needs 10 to 40 us of
// arithmetic and L2 latency per step on one CU.  Here the vectors of a system
// sit in L2, its threads take one row each, and barriers of one workgroup stand
// in for the launches: nothing returns to the host until the residual of every
// system is below the tolerance or the launch has run its share of steps
// (LAUNCH_STEPS; the next launch then goes on where this one stopped).
//
// The recurrences, targets and restarts are those of the lockstep solver
// (GMRES with classical Gram-Schmidt applied twice; COCG restarted at each FP64
// residual); sums run in another fixed order.  In complex64 the wires without
// neighbours are solved beforehand (k_lone) and leave the iteration, as there;
// where the block inverses do not solve them, they stay in it.
//
// Included by small7.hip and small19.hip (CHAFF_KNB unknowns per wire, namespace
// CHAFF_KNS).
#include "common.hpp"
#include "lone.hpp"
#include "prof.hpp"

#include <algorithm>
#include <chrono>

namespace chaff {
namespace CHAFF_KNS {

namespace small {

constexpr int NB = CHAFF_KNB, NSEG = NB + 1, NB2 = NB * NB;
constexpr int TH = NB <= 8 ? 1024 : 512;    // threads of a workgroup (128 and 256 registers)
constexpr int NW = TH / 64;                 // its waves
constexpr int MAX_WIRES = 4096;             // wires of one cloud (16-bit indices in LDS)
constexpr int MAX_CLOUDS = 32;              // cloud offsets travel with the launch
constexpr int MAX_M = 200;                  // restart lengths chaff_solve accepts
// Krylov steps of a system per launch: a solve that does not converge (restart
// lengths up to 10^6, 1,000 cycles) is then a row of short launches with the host
// between them, as the lockstep solver's is.  A step takes 20 us and more, a
// further launch with its read back about 30 us.
constexpr int LAUNCH_STEPS = 512;
constexpr double PI_S = 3.14159265358979323846;
constexpr int64_t MAX_SYSTEMS = 256;         // one workgroup per CU
constexpr int64_t MAX_BYTES = 5 << 18;        // of the blocks that a product reads (1.25 MiB)

struct Out {             // what a system tells the host
    double rel;          // FP64 relative residual, +inf after a breakdown
    int32_t cycles, ok;  // refinement cycles run; 1 converged, 0 not, -1 broken down, 2 goes on in another launch
};

// What a system carries over the end of a launch's share into the next; its
// vectors lie in the workspace.
struct Resume {
    double bn, lone2, scale, target, ckpt;
    c128 rho;
    int32_t k, cycles;       // COCG cycle under way: r^T z of its last step, steps taken; cycles run
    int32_t all, in_cycle;   // every wire is iterated on; the launch ended inside a cycle
};

template <typename C>
struct Args {
    const Wire* wires;
    const int32_t* perm;
    const int64_t* row_ptr;
    const int32_t* col_idx;
    const C *Z, *P;
    const double *k_hat, *e_hat;
    double k, tol, inner_tol;
    int64_t s;
    int n_clouds, m, max_cycles, use_x0, method, nvec;
    int32_t off[MAX_CLOUDS + 1];   // wires before each cloud
    c128* X;                       // caller's rows
    c128 *b, *x, *r;               // per system [wires * NB]
    C* V;                          // per system [nvec][wires * NB]
    c128* H;                       // per system [m][m + 1], column by column
    double* lone_e2;               // [wires][s] squared residual of a wire solved by k_lone
    int take_lone;                 // k_lone ran
    Resume* resume;                // per system
    Out* out;
    int32_t* steps;                // per system [max_cycles]
};

struct Shared {
    uint16_t list[MAX_WIRES];      // coupled wires of the cloud
    uint16_t where[MAX_WIRES];     // their place in the list
    c128 h[MAX_M + 1], h2[MAX_M + 1], g[MAX_M + 1], sn[MAX_M];
    double cs[MAX_M];
    c128 red[NW][2];
    c128 dots[NW];
    int32_t cnt[NW];
    double val[4];
    int32_t flag;
};

// A value that every thread holds and that lives across the cycles.  In complex64
// it goes to scalar registers (2,000 wires x 10 COCG steps 230 us, 237 with the
// spilled registers of the vector form); complex128's loops fill the scalar ones
// themselves (43 wires x 7 steps 69 us, 73 so).
template <typename C>
__device__ __forceinline__ double held(double v) {
    if (sizeof(C) == sizeof(c128)) return v;
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

__device__ __forceinline__ double wave_add(double v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
// sums over the workgroup, the same value in every thread, fixed order
__device__ __forceinline__ void block_add(Shared& S, c128& a, c128& b) {
    a.re = wave_add(a.re);
    a.im = wave_add(a.im);
    b.re = wave_add(b.re);
    b.im = wave_add(b.im);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        S.red[w][0] = a;
        S.red[w][1] = b;
    }
    __syncthreads();
    a = b = c128{0, 0};
    for (int k = 0; k < NW; ++k) {
        a = cadd(a, S.red[k][0]);
        b = cadd(b, S.red[k][1]);
    }
}
__device__ __forceinline__ double block_add(Shared& S, double v) {
    c128 a = {v, 0}, b = {0, 0};
    block_add(S, a, b);
    return a.re;
}

// A[q][.] v over one row of a stored block
template <typename R, typename C, typename V>
__device__ __forceinline__ void row_dot(cplx<R>& acc, const C* __restrict__ a, const V* v) {
    C av[NB];
    V vv[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        av[k] = a[k];
        vv[k] = v[k];
    }
#pragma unroll
    for (int k = 0; k < NB; ++k) cfma(acc, ccast<cplx<R>>(av[k]), ccast<cplx<R>>(vv[k]));
}

// One system: its cloud's wires, its vectors and the rows that are iterated on.
template <typename C>
struct System {
    using R = typename real_of<C>::type;
    const Args<C>& A;
    Shared& S;
    int w0, n, nc, rows;   // first wire, wires, coupled wires, their rows
    int64_t row0;          // of the whole cloud set
    c128 *b, *x, *r;
    C* V;
    int64_t vs;            // stride of the Krylov vectors
    int64_t rhs;

    __device__ __forceinline__ int wire(int ci) const { return S.list[ci]; }
    __device__ __forceinline__ C* vec(int i) const { return V + (int64_t)i * vs; }

    // y = P v over the coupled rows
    __device__ void precond(const C* v, C* y) const {
        for (int t = threadIdx.x; t < rows; t += TH) {
            const int ci = t / NB, q = t - ci * NB;
            cplx<R> a = {0, 0};
            row_dot<R>(a, A.P + ((int64_t)(w0 + wire(ci)) * NB + q) * NB, v + ci * NB);
            y[t] = a;
        }
        __syncthreads();
    }
    // sum over the row's blocks of Z v, v indexed by coupled wire (compact) or by wire of the cloud
    template <typename T, typename VT>
    __device__ __forceinline__ cplx<T> z_row(int i, int q, const VT* v, bool compact) const {
        cplx<T> a = {0, 0};
        const int64_t e1 = A.row_ptr[w0 + i + 1];
        for (int64_t e = A.row_ptr[w0 + i]; e < e1; ++e) {
            const int j = A.col_idx[e] - w0;
            row_dot<T>(a, A.Z + e * NB2 + q * NB, v + (int64_t)(compact ? S.where[j] : j) * NB);
        }
        return a;
    }
    __device__ void product(const C* v, C* y) const {
        for (int t = threadIdx.x; t < rows; t += TH) {
            const int ci = t / NB;
            y[t] = z_row<R>(wire(ci), t - ci * NB, v, true);
        }
        __syncthreads();
    }
    // r = b - Z x (FP64) on the coupled rows; its squared norm
    __device__ double residual(bool zero_x) const {
        double s2 = 0.0;
        for (int t = threadIdx.x; t < rows; t += TH) {
            const int ci = t / NB, q = t - ci * NB, i = wire(ci);
            c128 v = b[i * NB + q];
            if (!zero_x) v = csub(v, z_row<double>(i, q, x, false));
            r[i * NB + q] = v;
            s2 += v.re * v.re + v.im * v.im;
        }
        return block_add(S, s2);
    }

    // the coupled wires in order; nc of them
    __device__ void list_coupled(bool all) {
        int base = 0;
        for (int i0 = 0; i0 < n; i0 += TH) {
            const int i = i0 + threadIdx.x;
            const bool on = i < n && (all || A.row_ptr[w0 + i + 1] - A.row_ptr[w0 + i] > 1);
            const uint64_t m = __ballot(on);
            const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
            __syncthreads();
            if (lane == 0) S.cnt[w] = __popcll(m);
            __syncthreads();
            int ci = base + __popcll(m & ((1ull << lane) - 1)), tot = 0;
            for (int k = 0; k < NW; ++k) {
                if (k < w) ci += S.cnt[k];
                tot += S.cnt[k];
            }
            if (i < n) S.where[i] = on ? (uint16_t)ci : (uint16_t)0xffff;
            if (on) S.list[ci] = (uint16_t)i;
            base += tot;
        }
        nc = base;
        rows = nc * NB;
        __syncthreads();
    }

    // the incidence's drive of a wire: amplitude (the rooftops differ by their phase
    // alone), phase step of half the wire's rooftops
    __device__ __forceinline__ double drive(const Wire& w, double& beta, double& ph0) const {
        const double* kh = A.k_hat + 3 * rhs;
        const double* eh = A.e_hat + 3 * rhs;
        const double tp = w.tx * eh[0] + w.ty * eh[1] + w.tz * eh[2];
        beta = A.k * (kh[0] * w.tx + kh[1] * w.ty + kh[2] * w.tz);
        ph0 = A.k * (kh[0] * w.cx + kh[1] * w.cy + kh[2] * w.cz);
        const double D = w.len / NSEG;
        const double h = 0.5 * beta * D;
        const double sc = fabs(h) < 1e-4 ? 1.0 - h * h / 6.0 : sin(h) / h;
        return tp * D * sc * sc;
    }
    // u (eq. 4) on the coupled rows
    __device__ void excite() const {
        for (int t = threadIdx.x; t < rows; t += TH) {
            const int ci = t / NB, q = t - ci * NB, i = wire(ci);
            const Wire w = A.wires[w0 + i];
            double beta, ph0, sn, cs;
            const double env = drive(w, beta, ph0);
            sincos(ph0 + beta * (-0.5 * w.len + (q + 1) * (w.len / NSEG)), &sn, &cs);
            b[i * NB + q] = c128{env * cs, -env * sn};
        }
        __syncthreads();
    }
    // ||u||^2 over the whole cloud, and the squared residual that k_lone left
    __device__ void norms(double& u2, double& lone2) const {
        c128 a = {0, 0}, none = {0, 0};
        for (int i = threadIdx.x; i < n; i += TH) {
            double beta, ph0;
            const double env = drive(A.wires[w0 + i], beta, ph0);
            a.re += NB * (env * env);
            if (S.where[i] == 0xffff) a.im += A.lone_e2[(int64_t)(w0 + i) * A.s + rhs];
        }
        block_add(S, a, none);
        u2 = a.re;
        lone2 = a.im;
    }
};

// One restarted GMRES(m) cycle from r (squared norm rn2); returns its steps.
template <typename C>
__device__ int gmres_cycle(System<C>& Y, double rn, double target, c128* H) {
    using R = typename real_of<C>::type;
    Shared& S = Y.S;
    const int m = Y.A.m, rows = Y.rows, w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    C* W = Y.vec(m + 1);
    C* T = Y.vec(m + 2);
    for (int t = threadIdx.x; t < rows; t += TH) {
        const int ci = t / NB, q = t - ci * NB;
        Y.vec(0)[t] = ccast<C>(cscale(Y.r[Y.wire(ci) * NB + q], 1.0 / rn));
    }
    if (threadIdx.x == 0) S.g[0] = c128{1, 0};
    __syncthreads();
    int j = 0, used = 0;
    for (; j < m; ++j) {
        Y.precond(Y.vec(j), T);
        Y.product(T, W);
        const int nv = j + 1;
        double n2 = 0.0;
        for (int pass = 0; pass < 2; ++pass) {   // classical Gram-Schmidt, twice
            c128* h = pass ? S.h2 : S.h;
            const int G = nv >= NW ? 1 : NW / nv;   // waves per vector
            for (int i0 = 0; i0 < nv; i0 += NW) {
                const int i = i0 + (G == 1 ? w : w / G), part = G == 1 ? 0 : w % G;
                c128 a = {0, 0};
                if (i < nv) {
                    const C* v = Y.vec(i);
#pragma unroll 4
                    for (int t = part * 64 + lane; t < rows; t += 64 * G) cfma_conj(a, ccast<c128>(v[t]), ccast<c128>(W[t]));
                }
                a.re = wave_add(a.re);
                a.im = wave_add(a.im);
                if (lane == 0) S.dots[w] = a;
                __syncthreads();
                if ((int)threadIdx.x < NW && i0 + (int)threadIdx.x < nv && (int)threadIdx.x * G < NW) {
                    c128 t = {0, 0};
                    for (int k = 0; k < G; ++k) t = cadd(t, S.dots[threadIdx.x * G + k]);
                    h[i0 + threadIdx.x] = t;
                }
                __syncthreads();
            }
            n2 = 0.0;
            for (int t = threadIdx.x; t < rows; t += TH) {
                cplx<R> v = W[t];
#pragma unroll 4
                for (int i = 0; i < nv; ++i) {
                    const cplx<R> a = Y.vec(i)[t];
                    cfma(v, cmk<R>(-a.re, -a.im), ccast<cplx<R>>(h[i]));
                }
                W[t] = v;
                n2 += (double)v.re * v.re + (double)v.im * v.im;
            }
            if (pass == 0) __syncthreads();
        }
        const double beta = sqrt(fmax(block_add(S, n2), 0.0));
        if (threadIdx.x == 0) {   // column j of H, the earlier rotations, the new one
            c128* Hj = H + (int64_t)j * (m + 1);
            c128 prev = cadd(S.h[0], S.h2[0]);
            for (int i = 0; i < j; ++i) {
                const c128 next = cadd(S.h[i + 1], S.h2[i + 1]);
                Hj[i] = cadd(cscale(prev, S.cs[i]), cmul(S.sn[i], next));
                prev = csub(cscale(next, S.cs[i]), cmul(c128{S.sn[i].re, -S.sn[i].im}, prev));
            }
            const double aa = sqrt(prev.re * prev.re + prev.im * prev.im);
            double cj;
            c128 sj, rr;
            if (beta == 0.0) {
                cj = 1.0; sj = c128{0, 0}; rr = prev;
            } else if (aa == 0.0) {
                cj = 0.0; sj = c128{1, 0}; rr = c128{beta, 0};
            } else {
                const double tn = sqrt(aa * aa + beta * beta);
                const c128 ph = {prev.re / aa, prev.im / aa};
                cj = aa / tn;
                sj = cscale(ph, beta / tn);
                rr = cscale(ph, tn);
            }
            S.cs[j] = cj;
            S.sn[j] = sj;
            Hj[j] = rr;
            const c128 gj = S.g[j];
            S.g[j] = cscale(gj, cj);
            S.g[j + 1] = cmul(c128{-sj.re, sj.im}, gj);
            const double est = sqrt(S.g[j + 1].re * S.g[j + 1].re + S.g[j + 1].im * S.g[j + 1].im);
            const double hscale = sqrt(aa * aa + beta * beta);
            const bool breakdown = !(beta > 1e-14 * hscale) || !isfinite(beta);
            S.val[0] = breakdown ? 0.0 : 1.0 / beta;
            S.flag = est <= target || breakdown || j + 1 >= m;
        }
        __syncthreads();
        used = j + 1;
        if (S.flag) break;
        const R f = (R)S.val[0];
        C* vn = Y.vec(j + 1);
        for (int t = threadIdx.x; t < rows; t += TH) vn[t] = cscale(W[t], f);
        __syncthreads();
    }
    // y = R^-1 g, scaled by the cycle's residual norm: one wave, column by column
    if (w == 0) {
        for (int i = used - 1; i >= 0; --i) {
            const c128* Hi = H + (int64_t)i * (m + 1);
            const c128 d = Hi[i];
            const double dd = d.re * d.re + d.im * d.im;
            const c128 y = dd > 0 ? cmul(S.g[i], c128{d.re / dd, -d.im / dd}) : c128{0, 0};
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            for (int l = lane; l < i; l += 64) S.g[l] = csub(S.g[l], cmul(Hi[l], y));
            if (lane == 0) S.h[i] = cscale(y, rn);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < rows; t += TH) {   // T = V y
        cplx<R> a = {0, 0};
#pragma unroll 4
        for (int i = 0; i < used; ++i) cfma(a, Y.vec(i)[t], ccast<cplx<R>>(S.h[i]));
        T[t] = a;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < rows; t += TH) {   // x += P T
        const int ci = t / NB, q = t - ci * NB, i = Y.wire(ci);
        c128 a = {0, 0};
        row_dot<double>(a, Y.A.P + ((int64_t)(Y.w0 + i) * NB + q) * NB, T + ci * NB);
        Y.x[i * NB + q] = cadd(Y.x[i * NB + q], a);
    }
    __syncthreads();
    return used;
}

// One COCG cycle: r in units of scale, ended below the checkpoint or after m
// steps; S.flag says whether x_c holds a correction.  Returns its steps, or -1
// where left, the launch's remaining steps, ran out first: called again, it goes
// on from pause.
template <typename C>
__device__ int cocg_cycle(System<C>& Y, double scale, double target, double ckpt, int k0, int left, Resume* pause) {
    using R = typename real_of<C>::type;
    Shared& S = Y.S;
    const int rows = Y.rows;
    C *rv = Y.vec(0), *p = Y.vec(1), *q = Y.vec(2), *xc = Y.vec(3);
    if (threadIdx.x == 0) S.flag = k0;   // every step so far added to x_c
    if (k0 == 0)
        for (int t = threadIdx.x; t < rows; t += TH) {
            const int ci = t / NB;
            rv[t] = ccast<C>(cscale(Y.r[Y.wire(ci) * NB + t - ci * NB], 1.0 / scale));
        }
    __syncthreads();
    c128 rho = {0, 0}, alpha = {0, 0};
    if (k0 > 0) rho = pause->rho;
    int steps;
    for (int k = k0;; ++k) {
        steps = k;
        if (k - k0 >= left) {
            if (threadIdx.x == 0) {
                pause->rho = rho;
                pause->k = k;
            }
            steps = -1;
            break;
        }
        // r -= alpha q was applied; z = P r (in q until p takes it), rho' = r^T z, ||r||^2
        c128 rz = {0, 0}, rr = {0, 0};
        for (int t = threadIdx.x; t < rows; t += TH) {
            const int ci = t / NB;
            cplx<R> z = {0, 0};
            row_dot<R>(z, Y.A.P + ((int64_t)(Y.w0 + Y.wire(ci)) * NB + t - ci * NB) * NB, rv + ci * NB);
            q[t] = z;
            const C v = rv[t];
            cfma(rz, ccast<c128>(v), ccast<c128>(z));
            rr.re += (double)v.re * v.re + (double)v.im * v.im;
        }
        block_add(S, rz, rr);
        const double rn = sqrt(fmax(rr.re, 0.0));
        const double dd = rho.re * rho.re + rho.im * rho.im;
        if (!(rn > target) || !isfinite(rn) || !(rn > ckpt) || k == Y.A.m) break;
        const c128 beta = k > 0 && dd > 0.0 ? cmul(rz, c128{rho.re / dd, -rho.im / dd}) : c128{0, 0};
        rho = rz;
        const cplx<R> bt = ccast<cplx<R>>(beta);
        for (int t = threadIdx.x; t < rows; t += TH) {   // p = z + beta p
            cplx<R> z = q[t];
            if (k > 0) cfma(z, bt, p[t]);
            p[t] = z;
        }
        __syncthreads();
        steps = k + 1;
        c128 sg = {0, 0}, none = {0, 0};
        for (int t = threadIdx.x; t < rows; t += TH) {
            const int ci = t / NB;
            const cplx<R> v = Y.template z_row<R>(Y.wire(ci), t - ci * NB, p, true);
            q[t] = v;
            cfma(sg, ccast<c128>(p[t]), ccast<c128>(v));
        }
        block_add(S, sg, none);
        const double sd = sg.re * sg.re + sg.im * sg.im;
        if (!(sd > 0.0) || !isfinite(sd)) break;   // the recurrence broke down: restart from the FP64 residual
        alpha = cmul(rho, c128{sg.re / sd, -sg.im / sd});
        const cplx<R> al = ccast<cplx<R>>(alpha), na = {-al.re, -al.im};
        for (int t = threadIdx.x; t < rows; t += TH) {
            cplx<R> v = rv[t], xv = k > 0 ? xc[t] : cplx<R>{0, 0};
            cfma(v, na, q[t]);
            rv[t] = v;
            cfma(xv, al, p[t]);
            xc[t] = xv;
        }
        __syncthreads();
        if (threadIdx.x == 0) S.flag = k + 1;   // xc holds something
    }
    __syncthreads();
    return steps;
}

// The wires without neighbours of every cloud and incidence, one lane each.
template <typename C>
__global__ __launch_bounds__(64) void k_lone(Args<C> A, int64_t n) {
    __shared__ c128 lv[NB][64];
    const int lane = threadIdx.x;
    const int64_t t = (int64_t)blockIdx.x * 64 + lane;
    const int64_t i = t / A.s, r = t - i * A.s;
    if (i >= n || A.row_ptr[i + 1] - A.row_ptr[i] > 1) return;   // no barrier below
    const double kv[3] = {A.k_hat[3 * r], A.k_hat[3 * r + 1], A.k_hat[3 * r + 2]};
    const double ev[3] = {A.e_hat[3 * r], A.e_hat[3 * r + 1], A.e_hat[3 * r + 2]};
    c128 x[NB];
    double w2, e2;
    lone_wire<NB>(A.wires[i], A.Z + A.row_ptr[i] * NB2, A.P + i * NB2, kv, ev, A.k / PI_H, 0.01 * A.tol, lv, lane, x,
                   w2, e2);
    const int64_t o = (int64_t)A.perm[i] * NB * A.s + r;
#pragma unroll
    for (int q = 0; q < NB; ++q) A.X[o + q * A.s] = x[q];
    A.lone_e2[i * A.s + r] = e2;
}

// AGAIN: a further launch of the same solve
template <typename C, bool AGAIN>
__global__ __launch_bounds__(TH) void k_solve_small(Args<C> A) {
    __shared__ Shared S;
    const int cl = (int)(blockIdx.x % A.n_clouds);
    const int64_t rhs = blockIdx.x / A.n_clouds;
    const int64_t sys = (int64_t)cl * A.s + rhs;
    const int w0 = A.off[cl], n = A.off[cl + 1] - w0;
    const int64_t at = ((int64_t)w0 * A.s + rhs * n) * NB;   // this system's part of the vectors
    System<C> Y{A, S, w0, n, 0, 0, 0, A.b + at, A.x + at, A.r + at, A.V + at * A.nvec, (int64_t)n * NB, rhs};
    c128* H = A.H + sys * (int64_t)A.m * (A.m + 1);
    if (n == 0) {
        if (threadIdx.x == 0) A.out[sys] = Out{0.0, 0, 1};
        return;
    }
    Resume* const pause = A.resume + sys;
    double bn, lone2 = 0.0, scale = 0.0, target = 0.0, ckpt = 0.0;
    int cycles = 0, k0 = 0;
    bool all = !A.take_lone, in_cycle = false;
    if (AGAIN) {
        if (A.out[sys].ok != 2) return;   // this system is done
        bn = held<C>(pause->bn);
        lone2 = held<C>(pause->lone2);
        scale = held<C>(pause->scale);
        target = held<C>(pause->target);
        ckpt = held<C>(pause->ckpt);
        cycles = pause->cycles;
        all = pause->all != 0;
        in_cycle = pause->in_cycle != 0;
        k0 = in_cycle ? pause->k : 0;
        Y.list_coupled(all);
    } else {
        Y.list_coupled(all);
        double b2;
        Y.norms(b2, lone2);
        if (Y.nc < n && !(lone2 <= 0.01 * A.tol * A.tol * b2)) {   // the block inverses do not solve them
            Y.list_coupled(true);
            all = true;
            lone2 = 0.0;
        }
        bn = held<C>(sqrt(b2));
        lone2 = held<C>(lone2);
        Y.excite();
        // initial guess on the rows that are iterated on
        for (int t = threadIdx.x; t < Y.rows; t += TH) {
            const int ci = t / NB, q = t - ci * NB, i = Y.wire(ci);
            c128 v = {0, 0};
            if (A.use_x0 == 1) v = A.X[((int64_t)A.perm[w0 + i] * NB + q) * A.s + rhs];
            if (A.use_x0 == 2) row_dot<double>(v, A.P + ((int64_t)(w0 + i) * NB + q) * NB, Y.b + i * NB);
            Y.x[i * NB + q] = v;
        }
        __syncthreads();
    }
    double rel = 0.0;
    int ok = 0, left = LAUNCH_STEPS;   // a cycle counts as one more, for its residual
    for (;;) {
        if (left <= 0) {
            ok = 2;
            break;
        }
        double rn = 0.0;
        if (!in_cycle) {
            const double r2 = held<C>(Y.residual(cycles == 0 && A.use_x0 == 0));
            rn = held<C>(sqrt(fmax(r2, 0.0)));
            rel = bn > 0 ? sqrt(r2 + lone2) / bn : 0.0;
            if (!isfinite(r2)) {
                rel = INFINITY;
                ok = -1;
                break;
            }
            if (!(rel > A.tol)) {
                ok = 1;
                break;
            }
            if (cycles >= A.max_cycles) break;
            --left;
        }
        int steps;
        if (A.method == CHAFF_GMRES) {
            const double need = A.tol * bn / rn;
            const double goal = sizeof(C) == sizeof(c64) ? fmax(A.inner_tol, fmin(need, 1.0) * 0.5) : fmin(need * 0.5, 1.0);
            steps = gmres_cycle<C>(Y, rn, goal, H);
        } else {
            if (!in_cycle) {
                if (scale <= 0.0) scale = rn > 0 ? rn : 1.0;
                target = held<C>(0.5 * A.tol * bn / scale);
                ckpt = held<C>(fmax(target, A.inner_tol * rn / scale));
                k0 = 0;
            }
            steps = cocg_cycle<C>(Y, scale, target, ckpt, k0, left, pause);
            in_cycle = steps < 0;
            if (in_cycle) {
                left = 0;
                continue;
            }
            left += k0;
            if (S.flag) {   // a correction was formed
                const C* xc = Y.vec(3);
                for (int t = threadIdx.x; t < Y.rows; t += TH) {
                    const int ci = t / NB, a = Y.wire(ci) * NB + t - ci * NB;
                    const c128 v = ccast<c128>(xc[t]);
                    Y.x[a] = c128{Y.x[a].re + scale * v.re, Y.x[a].im + scale * v.im};
                }
            }
            __syncthreads();
        }
        left -= steps;
        if (threadIdx.x == 0) A.steps[sys * A.max_cycles + cycles] = steps;
        ++cycles;
    }
    if (threadIdx.x == 0) A.out[sys] = Out{rel, cycles, ok};
    if (ok == 2) {
        if (threadIdx.x == 0) {   // (rho and k: by the cycle that stopped)
            pause->bn = bn;
            pause->lone2 = lone2;
            pause->scale = scale;
            pause->target = target;
            pause->ckpt = ckpt;
            pause->cycles = cycles;
            pause->all = all;
            pause->in_cycle = in_cycle;
        }
        return;
    }
    // a system that broke down has no solution: an excitation that is not finite would leave its guess
    for (int t = threadIdx.x; t < Y.rows; t += TH) {
        const int ci = t / NB, q = t - ci * NB, i = Y.wire(ci);
        A.X[((int64_t)A.perm[w0 + i] * NB + q) * A.s + rhs] = ok < 0 ? c128{NAN, NAN} : Y.x[i * NB + q];
    }
}

// complex128 keeps one recurrence over every wire (its iterate at the tolerance is
// then the lockstep solver's to rounding); a caller's guess is left as it is given
inline bool takes_lone(const Cloud* c, const chaff_solve_opts* o) {
    return o->prec == CHAFF_C64 && o->use_x0 != 1 && 2 * c->n_pairs < c->n;
}

// vectors of a system beside b, x and r: GMRES m + 1 basis vectors, W and T; COCG r, p, q, x_c
inline int vectors(const chaff_solve_opts* o) { return o->method == CHAFF_GMRES ? o->restart + 3 : 4; }

template <typename C>
static size_t carve(void* ws, size_t cap, const Cloud* c, const chaff_solve_opts* o, int64_t s, Args<C>& a) {
    Carve cv(ws, cap);
    const int64_t rows = c->n * NB, nsys = (int64_t)c->n_clouds * s;
    const int m = o->method == CHAFF_GMRES ? o->restart : 0;
    a.nvec = vectors(o);
    a.b = cv.take<c128>(rows * s);
    a.x = cv.take<c128>(rows * s);
    a.r = cv.take<c128>(rows * s);
    a.V = cv.take<C>((size_t)a.nvec * rows * s);
    a.H = cv.take<c128>((size_t)nsys * m * (m + 1));
    a.lone_e2 = cv.take<double>((size_t)c->n * s);
    a.resume = cv.take<Resume>(nsys);
    a.out = cv.take<Out>(nsys);
    a.steps = cv.take<int32_t>((size_t)nsys * o->max_cycles);
    return cv.off + 256;
}

}  // namespace small

// Whether a call goes through one launch: blocks of at most MAX_BYTES (one CU
// streams too slowly from there on) and an estimate of its step's time on the CU
// that the largest cloud takes, in us, against the lockstep solver's.
//   A step here takes 5 us, 21 per MB of blocks, per iterated row 3.2e-3 (complex64,
// 7 unknowns; in complex128 1.6 times as much, with 19 unknowns another 1.65), and
// in GMRES 0.5e-3 per row and basis vector that a full cycle holds.  COCG, measured /
// estimated: complex64 0.11 MB on 1,050 rows 11.0 / 10.7, 0.74 MB on 7,000 rows 46 / 43,
// 1.27 MB on 399 rows 37 / 33; complex128 0.43 MB on 2,100 rows 25 / 25, 0.86 MB on
// 4,200 rows 44 / 44; 19 unknowns, 1.06 MB on 6,650 rows 61 / 62.  GMRES(30), complex64,
// 7,000 rows 121 / 148; GMRES(200), complex128, 2,100 rows 276 / 230, 7,000 rows 941 / 760.
//   Lockstep COCG: 30 us a step (19 unknowns 40) and 0.3 ms a solve; the line is where a
// solve of ten steps takes as long either way.  Whole solves, here / lockstep, ms:
// estimate 38 (complex128, 600 sparse wires, 8 steps) 0.39 / 0.60; 44 (600 in a box,
// 12 steps) 0.67 / 0.74; 47 (complex64, 1,200, 18 steps) 0.80 / 0.87; 59 (complex128,
// 1,000 sparse, 9 steps) 0.64 / 0.63; 64 (900 in a box, 17 steps) 1.26 / 0.89.  A
// solve of hundreds of steps would be faster in lockstep from an estimate of 30 on
// (at 44: 12.3 / 8.9), but no call says beforehand how many it will take.
//   Lockstep GMRES: 80 us a step and 1.75 per basis vector.  A full cycle may cost
// 1.3 times that: the cycles that end early, as most do, then gain.  Ratio of the
// estimates against whole solves, here / lockstep, ms: 0.55 (GMRES(200), 300 wires,
// complex128, 1,070 steps) 295 / 466; 0.8 (GMRES(30), 600 wires in a box, 10 steps)
// 0.68 / 1.04; 1.2 (1,200, complex64, 18 steps) 1.08 / 1.81; 1.2 (900, complex128, 15 steps)
// 1.55 / 1.62; 1.5 (GMRES(60), 1,000 wires, complex128, 1,380 steps) 399 / 255; 1.8
// (GMRES(200), the same) 1,130 / 562.
//   A system takes a CU; 256 of them take 1.3 times as long as 32, lockstep 1.5 to 2.5.
bool small_solve(const Cloud* c, const chaff_solve_opts* o, int64_t s) {
    if (o->precond != CHAFF_PRECOND_BLOCK || (o->method != CHAFF_GMRES && o->method != CHAFF_COCG)) return false;
    if (o->spmm_variant >= 0) return false;   // the caller asks for a product kernel
    if (c->n_clouds > small::MAX_CLOUDS || o->max_cycles > 1000) return false;
    const int64_t nsys = (int64_t)c->n_clouds * s;
    if (nsys > small::MAX_SYSTEMS) return false;
    int64_t largest = 0;
    for (int k = 0; k < c->n_clouds; ++k) largest = std::max(largest, c->cloud_off[k + 1] - c->cloud_off[k]);
    if (largest > small::MAX_WIRES) return false;
    // wires that are iterated on and blocks that a product reads: of the coupled wires (at most) or of all
    const bool single = o->prec == CHAFF_C64;
    const int64_t coupled = small::takes_lone(c, o) ? std::min<int64_t>(c->n, 2 * c->n_pairs) : c->n;
    const int64_t bytes = (2 * c->n_pairs + coupled) * small::NB2 * (single ? 8 : 16);
    if (bytes > small::MAX_BYTES) return false;
    const double share = (double)largest / (double)std::max<int64_t>(c->n, 1);
    const double rows = (double)(std::min(largest, coupled) * small::NB);
    const double step = 5.0 + 21e-6 * share * (double)bytes +
                        3.2e-3 * (single ? 1.0 : 1.6) * (small::NB > 8 ? 1.65 : 1.0) * rows;
    if (o->method == CHAFF_COCG) return step <= (small::NB > 8 ? 70.0 : 60.0);
    return step + 0.5e-3 * rows * o->restart <= 1.3 * (80.0 + 1.75 * o->restart);
}

size_t small_workspace_bytes(const Cloud* c, const chaff_solve_opts* o, int64_t s) {
    if (o->prec == CHAFF_C64) {
        small::Args<c64> a{};
        return small::carve<c64>(nullptr, 0, c, o, s, a);
    }
    small::Args<c128> a{};
    return small::carve<c128>(nullptr, 0, c, o, s, a);
}

template <typename C>
static chaff_status solve_small_impl(Cloud* c, const chaff_solve_opts* o, const void* Z, const void* Pinv,
                                     const double* k_hat, const double* e_hat, int64_t s, void* X, void* ws,
                                     size_t ws_bytes, chaff_solve_stats* stats, double* rel_res, hipStream_t st) {
    const auto t0 = std::chrono::steady_clock::now();
    small::Args<C> a{};
    if (small::carve<C>(ws, ws_bytes, c, o, s, a) > ws_bytes) return fail(CHAFF_EWORKSPACE, "solve workspace too small");
    a.wires = c->wires;
    a.perm = c->perm;
    a.row_ptr = c->row_ptr;
    a.col_idx = c->col_idx;
    a.Z = static_cast<const C*>(Z);
    a.P = static_cast<const C*>(Pinv);
    a.k_hat = k_hat;
    a.e_hat = e_hat;
    a.k = 2.0 * small::PI_S / c->wavelength;
    a.tol = o->tol;
    a.inner_tol = o->inner_tol;
    a.s = s;
    a.n_clouds = c->n_clouds;
    a.m = o->restart;
    a.max_cycles = o->max_cycles;
    a.use_x0 = o->use_x0;
    a.method = o->method;
    for (int k = 0; k <= c->n_clouds; ++k) a.off[k] = (int32_t)c->cloud_off[k];
    a.X = static_cast<c128*>(X);
    const int64_t nsys = (int64_t)c->n_clouds * s;
    a.take_lone = small::takes_lone(c, o) ? 1 : 0;
    // the systems' answers and steps lie one after the other: one copy
    const size_t head = (const char*)a.steps - (const char*)a.out;
    std::vector<char> back(head + (size_t)nsys * o->max_cycles * sizeof(int32_t));
    const small::Out* out = reinterpret_cast<const small::Out*>(back.data());
    const int32_t* steps = reinterpret_cast<const int32_t*>(back.data() + head);
    for (bool again = false, more = true; more; again = true) {   // a launch per LAUNCH_STEPS steps of the slowest system
        {
            ProfScope ps("solve_small", st);
            if (a.take_lone && !again)
                hipLaunchKernelGGL(small::k_lone<C>, dim3((unsigned)((c->n * s + 63) / 64)), dim3(64), 0, st, a, c->n);
            if (again)
                hipLaunchKernelGGL((small::k_solve_small<C, true>), dim3((unsigned)nsys), dim3(small::TH), 0, st, a);
            else
                hipLaunchKernelGGL((small::k_solve_small<C, false>), dim3((unsigned)nsys), dim3(small::TH), 0, st, a);
        }
        CHAFF_LAUNCH_CHECK();
        CHAFF_HIP(hipMemcpyAsync(back.data(), a.out, back.size(), hipMemcpyDeviceToHost, st));
        CHAFF_HIP(hipStreamSynchronize(st));
        more = false;
        for (int64_t i = 0; i < nsys; ++i) more = more || out[i].ok == 2;
    }
    int cycles = 0, iters = 0;
    double worst = 0.0;
    bool all = true, broken = false;
    for (int64_t i = 0; i < nsys; ++i) {
        cycles = std::max(cycles, out[i].cycles);
        worst = std::max(worst, out[i].rel);
        all = all && out[i].ok == 1;
        broken = broken || out[i].ok < 0;
        if (rel_res) rel_res[i] = out[i].rel;
    }
    for (int k = 0; k < cycles; ++k) {   // as in lockstep: a cycle lasts as long as its longest system
        int most = 0;
        for (int64_t i = 0; i < nsys; ++i)
            if (k < out[i].cycles) most = std::max(most, steps[i * o->max_cycles + k]);
        iters += most;
    }
    if (stats) {
        stats->cycles = cycles;
        stats->iterations = iters;
        stats->max_rel_residual = worst;
        stats->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    }
    if (!all)
        return fail(CHAFF_ENOCONV, (broken ? "breakdown (non-finite solution) after " : "no convergence after ") +
                                       std::to_string(cycles) + " cycles; max relative residual " +
                                       std::to_string(worst));
    return CHAFF_OK;
}

chaff_status solve_small(Cloud* c, const chaff_solve_opts* o, const void* Z, const void* Pinv, const double* k_hat,
                         const double* e_hat, int64_t s, void* X, void* ws, size_t ws_bytes, chaff_solve_stats* stats,
                         double* rel_res, hipStream_t st) {
    if (o->prec == CHAFF_C64)
        return solve_small_impl<c64>(c, o, Z, Pinv, k_hat, e_hat, s, X, ws, ws_bytes, stats, rel_res, st);
    return solve_small_impl<c128>(c, o, Z, Pinv, k_hat, e_hat, s, X, ws, ws_bytes, stats, rel_res, st);
}

}  // namespace CHAFF_KNS
}  // namespace chaff
