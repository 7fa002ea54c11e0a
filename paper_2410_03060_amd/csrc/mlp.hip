// Learned initial guess for the Krylov solve: per-(wire, incidence) features,
// a 192-128-128-128-14 SiLU network on BF16 matrix cores with FP32
// accumulation (forward, backward, Adam), and the maps between solved
// currents and network outputs.  Not part of the paper's method: the solver
// still drives the true residual of the S-NFC system (eq. 9) to the same
// tolerance, so the guess can only change how many iterations that takes.
//
// Products use v_mfma_f32_16x16x32_bf16: a wave multiplies a 16 x 32 BF16
// tile of A (rows = samples) by a 32 x 16 tile of B into a 16 x 16 FP32
// accumulator.  Each lane supplies 8 consecutive k of one row of A and of
// one column of B (A and B stored k-contiguous), and receives 4 consecutive
// rows of one output column.  The operands of the weight gradients are written
// transposed, so no product reads strided memory.
#include <algorithm>

#include "common.hpp"
#include "phase.hpp"
#include "precond.hpp"
#include "prof.hpp"

namespace chaff {
namespace {

constexpr int KNB = 16, FOWN = 16, FNB = 11, NF = FOWN + KNB * FNB, NH = 128, NO = 14;
constexpr int OW1 = 0, OB1 = OW1 + NF * NH, OW2 = OB1 + NH, OB2 = OW2 + NH * NH, OW3 = OB2 + NH,
              OB3 = OW3 + NH * NH, OW4 = OB3 + NH, OB4 = OW4 + NH * NO, NPARAM = OB4 + NO;
static_assert(NF == CHAFF_MLP_NFEAT && NH == CHAFF_MLP_HIDDEN && NO == CHAFF_MLP_NOUT, "header sizes");
static_assert(NPARAM == CHAFF_MLP_NPARAM, "parameter count");
constexpr int NOP = 16;          // output columns padded to one MFMA tile
constexpr int DYLD = 32;         // row stride of dL/dy (K of the first backward product)
constexpr int ROWS_WG = 128;     // rows per workgroup in the row-parallel products
constexpr int SPLIT_ROWS = 512;  // rows per partial sum of the weight gradients
constexpr double X_SCALE = 0.5;  // network outputs are current departures / 0.5
constexpr int NB_W = 7;          // rooftop unknowns per wire (8 segments)

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f) {  // nearest even on the FP32 pattern
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
// the same rounding (nearest even) by the hardware conversion, for activations
__device__ __forceinline__ uint16_t f2bf_hw(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
// FP64 -> FP32 -> BF16, each to nearest even.  The empty statement keeps the FP32
// value: left to itself the compiler joins the two roundings into one, which
// resolves the ties of the second otherwise.
__device__ __forceinline__ uint16_t d2bf(double x) {
    float f = (float)x;
    asm("" : "+v"(f));
    return f2bf_hw(f);
}

__device__ __forceinline__ bf16x8 ld8(const uint16_t* p) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p));
}
__device__ __forceinline__ bf16x8 zero8() { return __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0)); }

// logistic function with the hardware exponential and reciprocal (about 1 ulp each;
// the result is rounded to BF16 or enters a BF16 product)
__device__ __forceinline__ float sigmoidf(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

__device__ __forceinline__ float wave_sum(float v) {  // fixed butterfly order
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// ------------------------------------------------------------------ parameters -> BF16 operands
// Wt_l [n_out_pad][n_in]  (B operand of the forward product)
// Wn_l [n_in][n_out_pad'] (B operand of the backward data product), l = 2..4
struct Packed {
    uint16_t *wt1, *wt2, *wt3, *wt4, *wn2, *wn3, *wn4;
};

__global__ void k_pack(const float* __restrict__ th, Packed pk) {
    const int which = blockIdx.y;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // (dst, offset of W, n_in, n_out, transposed?, padded width)
    uint16_t* dst;
    int off, nin, nout, pad;
    bool tr;
    switch (which) {
        case 0: dst = pk.wt1; off = OW1; nin = NF; nout = NH; tr = true; pad = NH; break;
        case 1: dst = pk.wt2; off = OW2; nin = NH; nout = NH; tr = true; pad = NH; break;
        case 2: dst = pk.wt3; off = OW3; nin = NH; nout = NH; tr = true; pad = NH; break;
        case 3: dst = pk.wt4; off = OW4; nin = NH; nout = NO; tr = true; pad = NOP; break;
        case 4: dst = pk.wn2; off = OW2; nin = NH; nout = NH; tr = false; pad = NH; break;
        case 5: dst = pk.wn3; off = OW3; nin = NH; nout = NH; tr = false; pad = NH; break;
        default: dst = pk.wn4; off = OW4; nin = NH; nout = NO; tr = false; pad = DYLD; break;
    }
    if (t >= (int64_t)nin * pad) return;
    int i, o;
    if (tr) { o = (int)(t / nin); i = (int)(t % nin); }
    else { i = (int)(t / pad); o = (int)(t % pad); }
    dst[t] = o < nout ? f2bf(th[off + i * nout + o]) : (uint16_t)0;
}

// ------------------------------------------------------------------ fused inference
// All four layers in one persistent kernel: each workgroup copies the BF16
// weights into LDS once (rows padded by 8 elements so that the 16 rows a
// ds_read_b128 touches fall in distinct banks), then every wave walks its own
// 16-row tiles: layer 1 reads the features from HBM, the hidden activations
// stay in the wave's LDS tile, and only the 14 outputs are written.  Weight
// traffic is 116 KB per workgroup instead of per tile.
//   Bound: the SiLU of the hidden layers (one exponential and one reciprocal at
// quarter rate each: 384 per row, 94 us of vector issue for 800,000 rows against
// 38 us of MFMAs), so two waves per SIMD are wanted, whose products and SiLUs
// overlap: eight waves of 16 rows are what the LDS holds beside the weights.
// 305 us for 800,000 rows, 216 so
constexpr int FWD_WAVES = 8;
constexpr int FLD1 = NF + 8, FLDH = NH + 8;   // padded LDS row strides (BF16)
constexpr int FUSED_LDS = (NH * FLD1 + 2 * NH * FLDH + NOP * FLDH + FWD_WAVES * 16 * FLDH) * 2;
static_assert(FUSED_LDS <= 160 * 1024, "the weights and the activation tiles share one CU's LDS");

__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__global__ __launch_bounds__(64 * FWD_WAVES) void k_fwd_fused(const uint16_t* __restrict__ feat, int64_t M,
                                                   const float* __restrict__ th, Packed pk, float* __restrict__ Y) {
    extern __shared__ uint16_t lds[];
    uint16_t* w1 = lds;                      // [128][FLD1]
    uint16_t* w2 = w1 + NH * FLD1;           // [128][FLDH]
    uint16_t* w3 = w2 + NH * FLDH;           // [128][FLDH]
    uint16_t* w4 = w3 + NH * FLDH;           // [16][FLDH]
    uint16_t* act = w4 + NOP * FLDH;         // [waves][16][FLDH]
    // weights -> LDS (16-byte chunks)
    for (int t = threadIdx.x; t < NH * (NF / 8); t += 64 * FWD_WAVES) {
        const int r = t / (NF / 8), c = (t % (NF / 8)) * 8;
        *reinterpret_cast<uint4*>(w1 + r * FLD1 + c) = *reinterpret_cast<const uint4*>(pk.wt1 + r * NF + c);
    }
    for (int t = threadIdx.x; t < NH * (NH / 8); t += 64 * FWD_WAVES) {
        const int r = t / (NH / 8), c = (t % (NH / 8)) * 8;
        *reinterpret_cast<uint4*>(w2 + r * FLDH + c) = *reinterpret_cast<const uint4*>(pk.wt2 + r * NH + c);
        *reinterpret_cast<uint4*>(w3 + r * FLDH + c) = *reinterpret_cast<const uint4*>(pk.wt3 + r * NH + c);
    }
    for (int t = threadIdx.x; t < NOP * (NH / 8); t += 64 * FWD_WAVES) {
        const int r = t / (NH / 8), c = (t % (NH / 8)) * 8;
        *reinterpret_cast<uint4*>(w4 + r * FLDH + c) = *reinterpret_cast<const uint4*>(pk.wt4 + r * NH + c);
    }
    __syncthreads();
    // The weights are the A operand (rows = output features) and the activations
    // the B operand (columns = sample rows): a lane then holds 4 consecutive
    // output features of one sample, written to the LDS tile as one 8-byte store.
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint16_t* my = act + w * 16 * FLDH;
    const int l16 = lane & 15, g4 = (lane >> 4) * 4, kb = (lane >> 4) * 8;
    const int64_t n_tiles = (M + 15) / 16;
    constexpr int KS1 = NF / 32, MT = NH / 16;
    auto load_tile = [&](int64_t tile, bf16x8 (&fa)[KS1]) {
        const int64_t m = tile * 16 + l16;
#pragma unroll
        for (int ks = 0; ks < KS1; ++ks) fa[ks] = m < M ? ld8(feat + m * NF + ks * 32 + kb) : zero8();
    };
    // bias + SiLU of acc -> BF16 activation tile
    auto to_tile = [&](const f32x4 (&acc)[MT], const float* bias) {
        wave_lds_sync();
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int f0 = 16 * i + g4;
            const float4 b = *reinterpret_cast<const float4*>(bias + f0);
            const float bb[4] = {b.x, b.y, b.z, b.w};
            uint16_t h[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float z = acc[i][r] + bb[r];
                h[r] = f2bf_hw(z * sigmoidf(z));
            }
            *reinterpret_cast<uint2*>(my + l16 * FLDH + f0) =
                make_uint2(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16));
        }
        wave_lds_sync();
    };
    const int64_t t_step = (int64_t)gridDim.x * FWD_WAVES;
    int64_t tile = (int64_t)blockIdx.x * FWD_WAVES + w;
    bf16x8 fa[KS1];
    if (tile < n_tiles) load_tile(tile, fa);
    for (; tile < n_tiles; tile += t_step) {
        bf16x8 fnext[KS1];
        if (tile + t_step < n_tiles) load_tile(tile + t_step, fnext);
        f32x4 acc[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS1; ++ks)   // layer 1
#pragma unroll
            for (int i = 0; i < MT; ++i)
                acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(w1 + (16 * i + l16) * FLD1 + ks * 32 + kb), fa[ks],
                                                                 acc[i], 0, 0, 0);
#pragma unroll
        for (int layer = 0; layer < 2; ++layer) {   // layers 2 and 3
            to_tile(acc, th + (layer == 0 ? OB1 : OB2));
            const uint16_t* wl = layer == 0 ? w2 : w3;
#pragma unroll
            for (int i = 0; i < MT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < NH; k += 32) {
                const bf16x8 b = ld8(my + l16 * FLDH + k + kb);
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(wl + (16 * i + l16) * FLDH + k + kb), b, acc[i],
                                                                     0, 0, 0);
            }
        }
        to_tile(acc, th + OB3);
        f32x4 out = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < NH; k += 32)   // output layer (14 of 16 rows of W4^T used)
            out = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(w4 + l16 * FLDH + k + kb), ld8(my + l16 * FLDH + k + kb),
                                                          out, 0, 0, 0);
        const int64_t m = tile * 16 + l16;
        if (m < M) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int f = g4 + r;
                if (f < NO) Y[m * NO + f] = out[r] + th[OB4 + f];
            }
        }
#pragma unroll
        for (int ks = 0; ks < KS1; ++ks) fa[ks] = fnext[ks];
    }
}

// ------------------------------------------------------------------ training
// One step is four launches: the BF16 operands (k_pack), forward and backward
// of every row (k_train_rows), the partial weight and bias gradients
// (k_train_wgrad), their sum and Adam (k_reduce).
//   Rows: a workgroup takes 16 MT rows through all four layers and back.  Wave w
// owns 32 of the 128 columns of every hidden layer; pre-activations stay in its
// registers for the backward pass, activations and layer gradients pass through
// LDS, and only the transposed operands of the weight gradients are written.
//   Bound: latency at training batches (seven dependent layer products with
// weights from L2), so the rows are spread as thinly as 512 workgroups allow:
// the layers as separate launches of 32 rows per wave left 4,096 rows on 32 of
// the 256 CUs and took 17 launches: 210 us a step, now 31 us (rows 18, weight
// gradients 11, sum and Adam 4 us).
struct RowsArgs {
    const uint16_t* feat;   // [*][192] BF16, row m at idx[m]
    const int64_t* idx;     // optional row gather of feat and T
    const float* T;         // [*][14] targets
    int64_t M, Mpad;
    Packed pk;
    const float* th;
    uint16_t *fT, *aT1, *aT2, *aT3;           // [features or units][Mpad] BF16
    uint16_t *dYT, *dZT3, *dZT2, *dZT1;       // [units][Mpad] BF16 (dYT: 16 rows)
    float* loss_part;       // [workgroups] sums of (y - t)^2
};

constexpr int FLDY = DYLD + 8;   // padded LDS row stride of dL/dy

template <int MT>
__global__ __launch_bounds__(256) void k_train_rows(RowsArgs g) {
    constexpr int NTW = NH / 64;   // 16-column tiles per wave
    __shared__ __align__(16) uint16_t act[2][16 * MT * FLDH];
    __shared__ __align__(16) uint16_t dy[16 * MT * FLDY];
    __shared__ float sq_s[4];
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int l16 = lane & 15, rq = (lane >> 4) * 4, kb = (lane >> 4) * 8;
    const int64_t m0 = (int64_t)blockIdx.x * (16 * MT);
    f32x4 z[3][MT][NTW];

    // acc += A B^T over K, A [16 MT][lda] in LDS, B the rows n of a packed operand [*][K]
    auto product = [&](const uint16_t* A, int lda, const uint16_t* Bn, int K, f32x4 (&acc)[MT][NTW]) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NTW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < K; k += 32) {
            bf16x8 a[MT], b[NTW];
#pragma unroll
            for (int j = 0; j < NTW; ++j) b[j] = ld8(Bn + (int64_t)(16 * (NTW * w + j) + l16) * K + k + kb);
#pragma unroll
            for (int i = 0; i < MT; ++i) a[i] = ld8(A + (16 * i + l16) * lda + k + kb);
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NTW; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    };
    // four consecutive rows of column n: into the LDS tile (or nullptr) and the transposed operand
    auto put = [&](uint16_t* tile, uint16_t* T, int i, int n, const uint16_t (&h)[4]) {
        if (tile)
#pragma unroll
            for (int r = 0; r < 4; ++r) tile[(16 * i + rq + r) * FLDH + n] = h[r];
        *reinterpret_cast<uint2*>(T + (int64_t)n * g.Mpad + m0 + 16 * i + rq) =
            make_uint2(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16));
    };
    // z += bias, SiLU(z) to the tile and the transposed operand
    auto activate = [&](f32x4 (&zz)[MT][NTW], const float* bias, uint16_t* tile, uint16_t* T) {
#pragma unroll
        for (int j = 0; j < NTW; ++j) {
            const int n = 16 * (NTW * w + j) + l16;
            const float b = bias[n];
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                uint16_t h[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float v = zz[i][j][r] + b;
                    zz[i][j][r] = v;
                    h[r] = f2bf_hw(v * sigmoidf(v));
                }
                put(tile, T, i, n, h);
            }
        }
        __syncthreads();
    };
    // dZ = (product) SiLU'(z), to the tile and the transposed operand
    auto back = [&](const f32x4 (&acc)[MT][NTW], const f32x4 (&zz)[MT][NTW], uint16_t* tile, uint16_t* T) {
#pragma unroll
        for (int j = 0; j < NTW; ++j)
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                uint16_t h[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float v = zz[i][j][r], sg = sigmoidf(v);
                    h[r] = f2bf_hw(acc[i][j][r] * (sg * (1.0f + v * (1.0f - sg))));
                }
                put(tile, T, i, 16 * (NTW * w + j) + l16, h);
            }
    };

    {   // layer 1: the features come from HBM; wave w also writes k-steps w, w + 4 of their transpose
        const uint16_t* src[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int64_t m = m0 + 16 * i + l16;
            src[i] = m < g.M ? g.feat + (g.idx ? g.idx[m] : m) * NF : nullptr;
#pragma unroll
            for (int j = 0; j < NTW; ++j) z[0][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int ks = 0; ks < NF / 32; ++ks) {
            bf16x8 a[MT], b[NTW];
#pragma unroll
            for (int i = 0; i < MT; ++i) a[i] = src[i] ? ld8(src[i] + ks * 32 + kb) : zero8();
#pragma unroll
            for (int j = 0; j < NTW; ++j) b[j] = ld8(g.pk.wt1 + (16 * (NTW * w + j) + l16) * NF + ks * 32 + kb);
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NTW; ++j)
                    z[0][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], z[0][i][j], 0, 0, 0);
            if ((ks & 3) == w)
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const __bf16 f = a[i][e];
                        g.fT[(int64_t)(ks * 32 + kb + e) * g.Mpad + m0 + 16 * i + l16] = __builtin_bit_cast(uint16_t, f);
                    }
        }
    }
    activate(z[0], g.th + OB1, act[0], g.aT1);
    product(act[0], FLDH, g.pk.wt2, NH, z[1]);
    activate(z[1], g.th + OB2, act[1], g.aT2);
    product(act[1], FLDH, g.pk.wt3, NH, z[2]);
    activate(z[2], g.th + OB3, act[0], g.aT3);
    // output layer: 14 of 16 columns, one 16-row tile per wave; dL/dy = 2 (y - t)
    float sq = 0.f;
    for (int i = w; i < MT; i += 4) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < NH; k += 32)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(act[0] + (16 * i + l16) * FLDH + k + kb),
                                                          ld8(g.pk.wt4 + l16 * NH + k + kb), acc, 0, 0, 0);
        const float b = l16 < NO ? g.th[OB4 + l16] : 0.f;
        uint16_t h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t m = m0 + 16 * i + rq + r;
            float d = 0.f;
            if (m < g.M && l16 < NO) d = (acc[r] + b) - g.T[(g.idx ? g.idx[m] : m) * NO + l16];
            sq += d * d;
            h[r] = f2bf_hw(2.0f * d);
            dy[(16 * i + rq + r) * FLDY + l16] = h[r];
            dy[(16 * i + rq + r) * FLDY + NOP + l16] = 0;
        }
        *reinterpret_cast<uint2*>(g.dYT + (int64_t)l16 * g.Mpad + m0 + 16 * i + rq) =
            make_uint2(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16));
    }
    sq = wave_sum(sq);
    if (lane == 0) sq_s[w] = sq;
    __syncthreads();
    if (threadIdx.x == 0) g.loss_part[blockIdx.x] = (sq_s[0] + sq_s[1]) + (sq_s[2] + sq_s[3]);
    f32x4 acc[MT][NTW];
    product(dy, FLDY, g.pk.wn4, DYLD, acc);
    back(acc, z[2], act[1], g.dZT3);
    __syncthreads();
    product(act[1], FLDH, g.pk.wn3, NH, acc);
    back(acc, z[1], act[0], g.dZT2);
    __syncthreads();
    product(act[0], FLDH, g.pk.wn2, NH, acc);
    back(acc, z[0], nullptr, g.dZT1);
}

// Partial gradients over one split of SPLIT_ROWS rows, one wave per unit:
// part[s][w_off + i*n_out + o] = sum_m aT[i][m] dZT[o][m] for a 16 x 64 tile of
// a layer's weights (16 x 14 of the last), or one bias part[s][off] = sum_m dZT[o][m].
constexpr int WG_L1 = NF / 16 * (NH / 64), WG_L = NH / 16 * (NH / 64), WG_L4 = NH / 16;
constexpr int WG_TILES = WG_L1 + 2 * WG_L + WG_L4, WG_UNITS = WG_TILES + NO + 3 * NH;
// splits per launch: the threads of a launch are counted in 32 bits, and 145,258
// splits (74 million rows) have more
constexpr int64_t WG_LAUNCH = 65536;

template <int NT>
__device__ __forceinline__ void wgrad_tile(const uint16_t* __restrict__ aT, const uint16_t* __restrict__ dZT,
                                           int64_t Mpad, int i0, int o0, int n_out, int64_t s, float* __restrict__ dst) {
    const int lane = threadIdx.x & 63;
    const int kb = (lane >> 4) * 8;
    const uint16_t* ap = aT + (int64_t)(i0 + (lane & 15)) * Mpad + s * SPLIT_ROWS + kb;
    const uint16_t* bp[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) bp[j] = dZT + (int64_t)(o0 + 16 * j + (lane & 15)) * Mpad + s * SPLIT_ROWS + kb;
    f32x4 acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int k = 0; k < SPLIT_ROWS; k += 32) {
        const bf16x8 a = ld8(ap + k);
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, ld8(bp[j] + k), acc[j], 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int o = o0 + 16 * j + (lane & 15);
        if (o >= n_out) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) dst[(int64_t)(i0 + (lane >> 4) * 4 + r) * n_out + o] = acc[j][r];
    }
}

__global__ __launch_bounds__(64) void k_train_wgrad(RowsArgs g, int64_t split0, float* __restrict__ part) {
    const int64_t s = split0 + blockIdx.x / WG_UNITS;
    int u = (int)(blockIdx.x % WG_UNITS);
    float* dst = part + s * NPARAM;
    if (u < WG_L1) {
        wgrad_tile<4>(g.fT, g.dZT1, g.Mpad, u / 2 * 16, u % 2 * 64, NH, s, dst + OW1);
    } else if (u < WG_L1 + WG_L) {
        u -= WG_L1;
        wgrad_tile<4>(g.aT1, g.dZT2, g.Mpad, u / 2 * 16, u % 2 * 64, NH, s, dst + OW2);
    } else if (u < WG_L1 + 2 * WG_L) {
        u -= WG_L1 + WG_L;
        wgrad_tile<4>(g.aT2, g.dZT3, g.Mpad, u / 2 * 16, u % 2 * 64, NH, s, dst + OW3);
    } else if (u < WG_TILES) {
        wgrad_tile<1>(g.aT3, g.dYT, g.Mpad, (u - WG_L1 - 2 * WG_L) * 16, 0, NO, s, dst + OW4);
    } else {
        u -= WG_TILES;   // 0..13: b4, then b3, b2, b1 (128 each)
        const uint16_t* row;
        int off;
        if (u < NO) { row = g.dYT + (int64_t)u * g.Mpad; off = OB4 + u; }
        else if (u < NO + NH) { row = g.dZT3 + (int64_t)(u - NO) * g.Mpad; off = OB3 + (u - NO); }
        else if (u < NO + 2 * NH) { row = g.dZT2 + (int64_t)(u - NO - NH) * g.Mpad; off = OB2 + (u - NO - NH); }
        else { row = g.dZT1 + (int64_t)(u - NO - 2 * NH) * g.Mpad; off = OB1 + (u - NO - 2 * NH); }
        row += s * SPLIT_ROWS;
        float v = 0.f;
#pragma unroll
        for (int k = 0; k < SPLIT_ROWS; k += 64) v += bf2f(row[k + threadIdx.x]);
        v = wave_sum(v);
        if (threadIdx.x == 0) dst[off] = v;
    }
}

__device__ __forceinline__ void adam_one(float& th, float& m, float& v, float gj, float lr, float b1, float b2,
                                         float eps, float bc1, float bc2) {
    const float mj = b1 * m + (1.0f - b1) * gj;
    const float vj = b2 * v + (1.0f - b2) * gj * gj;
    m = mj;
    v = vj;
    th -= lr * (mj / bc1) / (sqrtf(vj / bc2) + eps);
}

struct AdamArgs {
    float *th, *m, *v;   // th nullptr: the gradient alone
    float lr, b1, b2, eps, bc1, bc2;
};

// grad = scale * sum over splits (fixed order), then Adam on it; the last block also reduces the loss.
__global__ __launch_bounds__(256) void k_reduce(const float* __restrict__ part, int64_t nsplit, float scale,
                                                float* __restrict__ grad, const float* __restrict__ loss_part,
                                                int64_t nloss, float* __restrict__ loss, AdamArgs a) {
    if (blockIdx.x == gridDim.x - 1) {
        if (threadIdx.x < 64 && loss) {   // one wave, fixed order
            double acc = 0.0;
            for (int64_t i = threadIdx.x; i < nloss; i += 64) acc += loss_part[i];
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
            if (threadIdx.x == 0) *loss = (float)(acc * (double)scale);
        }
        return;
    }
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= NPARAM) return;
    float acc = 0.f;
#pragma unroll 8
    for (int64_t s = 0; s < nsplit; ++s) acc += part[s * NPARAM + j];
    const float gj = acc * scale;
    grad[j] = gj;
    if (a.th) adam_one(a.th[j], a.m[j], a.v[j], gj, a.lr, a.b1, a.b2, a.eps, a.bc1, a.bc2);
}

__global__ void k_adam(float* __restrict__ th, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, float lr, float b1, float b2, float eps, float bc1, float bc2) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= NPARAM) return;
    adam_one(th[j], m[j], v[j], g[j], lr, b1, b2, eps, bc1, bc2);
}

// ------------------------------------------------------------------ features
// FP64 squared centroid distance ((dx*dx + dy*dy) + dz*dz), every operation
// rounded on its own, as in the near-set test.
__device__ __forceinline__ double dist2(const Wire& a, const Wire& b) {
#pragma clang fp contract(off)
    const double dx = b.cx - a.cx, dy = b.cy - a.cy, dz = b.cz - a.cz;
    const double xx = dx * dx, yy = dy * dy, zz = dz * dz;
    double s = xx + yy;
    s = s + zz;
    return s;
}

__device__ __forceinline__ double sinc_d(double x) {
    if (fabs(x) < 1e-4) return 1.0 - x * x / 6.0;
    return sin(x) / x;
}

constexpr int FW_CAND = 256;   // near-set rows up to this length are ranked in parallel
constexpr int FW_ROWS = 8;     // rows formed at a time

// One wave per wire p (caller order) and the rows p*R + r of it that fall in
// the requested range.  The 16 nearest neighbours are chosen once per wire:
// every lane ranks its candidates by counting the candidates with a smaller
// (squared distance, caller index) key (rows longer than FW_CAND fall back to
// repeated minimum search), and the neighbours' geometry is staged in LDS.
// The features that do not depend on the incidence are formed once per wire.
// The rows are formed FW_ROWS at a time in LDS, one lane per (row, neighbour) and
// then per (row, own rooftop), and stored with 16-byte writes.
//   Bound: FP64 arithmetic and the store of 384 bytes a row.  Two rows per pass
// (24 of 32 lanes each), the library's sincos and 2-byte stores straight to HBM
// took 373 us for 800,000 rows, 219 so.
__global__ __launch_bounds__(64) void k_features(const Wire* __restrict__ wires, const int32_t* __restrict__ perm,
                                                 const int32_t* __restrict__ iperm,
                                                 const int64_t* __restrict__ row_ptr,
                                                 const int32_t* __restrict__ col_idx, int64_t R, int64_t row0,
                                                 int64_t n_rows, const double* __restrict__ k_hat,
                                                 const double* __restrict__ e_hat, double kp, double lam, double d_c,
                                                 uint16_t* __restrict__ feat) {
#pragma clang fp contract(off)
    // the candidates while the neighbours are chosen, then the staged rows
    __shared__ __align__(16) unsigned char buf[FW_CAND * 16];
    static_assert(FW_ROWS * NF * 2 <= FW_CAND * 16, "the rows fit the candidates' space");
    double* cd2 = reinterpret_cast<double*>(buf);
    int32_t* cid = reinterpret_cast<int32_t*>(buf + FW_CAND * 8);
    int32_t* cint = cid + FW_CAND;
    uint16_t* st = reinterpret_cast<uint16_t*>(buf);   // [FW_ROWS][192]
    __shared__ int32_t slot[KNB];
    __shared__ double sg[KNB][6];   // d.x, d.y, d.z, t'.x, t'.y, t'.z
    __shared__ uint16_t fixed[KNB][4];   // |d|/d_c, length feature, Re, Im exp(-j k |d|)
    const int lane = threadIdx.x;
    const int64_t p = row0 / R + blockIdx.x;
    const int64_t rb = p * R > row0 ? p * R : row0;
    const int64_t re = (p + 1) * R < row0 + n_rows ? (p + 1) * R : row0 + n_rows;
    if (rb >= re) return;   // uniform over the (single-wave) block
    const int32_t ip = iperm[p];
    const Wire w = wires[ip];
    const int64_t e0 = row_ptr[ip], e1 = row_ptr[ip + 1];
    const int64_t ne = e1 - e0;   // includes the diagonal
    const int64_t cnt = ne - 1;
    if (lane < KNB) slot[lane] = -1;
    // geometry of the neighbour in slot j and its incidence-independent features
    auto set_slot = [&](int j, const Wire& v, double d2) {
        sg[j][0] = v.cx - w.cx;
        sg[j][1] = v.cy - w.cy;
        sg[j][2] = v.cz - w.cz;
        sg[j][3] = v.tx;
        sg[j][4] = v.ty;
        sg[j][5] = v.tz;
        double sn, cs;
        sincospi_any(kp * sqrt(d2), sn, cs);
        fixed[j][0] = d2bf(sqrt(d2) / d_c);
        fixed[j][1] = d2bf(10.0 * (v.len / lam - 0.5));
        fixed[j][2] = d2bf(cs);
        fixed[j][3] = d2bf(-sn);
    };
    if (ne <= 64) {   // one candidate per lane, kept in its registers until its rank is known
        Wire v = w;
        double d2 = 0.0;
        int32_t id = 0, c = ip;
        if (lane < ne) {
            c = col_idx[e0 + lane];
            id = perm[c];
            v = wires[c];
            if (c != ip) d2 = dist2(w, v);
            cd2[lane] = c == ip ? INFINITY : d2;   // the wire itself comes before nobody
            cid[lane] = id;
        }
        __syncthreads();
        int rank = 0;
        for (int u = 0; u < (int)ne; ++u) {
            const double du = cd2[u];
            rank += (du < d2 || (du == d2 && cid[u] < id)) ? 1 : 0;
        }
        if (lane < ne && c != ip && rank < KNB) {
            slot[rank] = c;
            set_slot(rank, v, d2);
        }
    } else {
        if (ne <= FW_CAND) {
            for (int64_t t = lane; t < ne; t += 64) {
                const int32_t c = col_idx[e0 + t];
                cint[t] = c;
                cid[t] = perm[c];
                cd2[t] = c == ip ? 0.0 : dist2(w, wires[c]);
            }
            __syncthreads();
            for (int64_t t = lane; t < ne; t += 64) {
                if (cint[t] == ip) continue;
                const double d2 = cd2[t];
                const int32_t id = cid[t];
                int rank = 0;
                for (int64_t u = 0; u < ne; ++u) {
                    if (cint[u] == ip) continue;
                    const double du = cd2[u];
                    rank += (du < d2 || (du == d2 && cid[u] < id)) ? 1 : 0;
                }
                if (rank < KNB) slot[rank] = cint[t];
            }
        } else {   // long row: repeated minimum search (the same on every lane)
            double pd2 = -1.0;
            int32_t pid = -1;
            for (int j = 0; j < KNB; ++j) {
                double bd2 = INFINITY;
                int32_t bid = INT32_MAX, bint = -1;
                for (int64_t e = e0; e < e1; ++e) {
                    const int32_t c = col_idx[e];
                    if (c == ip) continue;
                    const double d2 = dist2(w, wires[c]);
                    const int32_t id = perm[c];
                    const bool after = d2 > pd2 || (d2 == pd2 && id > pid);
                    const bool before = d2 < bd2 || (d2 == bd2 && id < bid);
                    if (after && before) { bd2 = d2; bid = id; bint = c; }
                }
                if (bint < 0) break;
                if (lane == 0) slot[j] = bint;
                pd2 = bd2;
                pid = bid;
            }
        }
        __syncthreads();
        if (lane < KNB && slot[lane] >= 0) {
            const Wire v = wires[slot[lane]];
            set_slot(lane, v, dist2(w, v));
        }
    }
    __syncthreads();
    const double D = w.len / 8.0;
    for (int64_t row0s = rb; row0s < re; row0s += FW_ROWS) {
        const int nr = (int)(re - row0s < FW_ROWS ? re - row0s : FW_ROWS);
        for (int t = lane; t < KNB * nr; t += 64) {   // neighbour slots
            const int m = t % KNB, rl = t / KNB;
            uint16_t* f = st + rl * NF + FOWN + FNB * m;
            if (slot[m] < 0) {
#pragma unroll
                for (int g = 0; g < FNB; ++g) f[g] = 0;
                continue;
            }
            const int64_t r = row0s + rl - p * R;
            const double kx = k_hat[3 * r], ky = k_hat[3 * r + 1], kz = k_hat[3 * r + 2];
            const double ex = e_hat[3 * r], ey = e_hat[3 * r + 1], ez = e_hat[3 * r + 2];
            const double sp = (w.tx * ex + w.ty * ey + w.tz * ez) >= 0.0 ? 1.0 : -1.0;
            const double tx = sp * w.tx, ty = sp * w.ty, tz = sp * w.tz;
            const double dx = sg[m][0], dy = sg[m][1], dz = sg[m][2];
            double sn, cs;
            sincospi_any(kp * (kx * dx + ky * dy + kz * dz), sn, cs);
            const double vtx = sg[m][3], vty = sg[m][4], vtz = sg[m][5];
            const double sv = (vtx * ex + vty * ey + vtz * ez) >= 0.0 ? 1.0 : -1.0;
            const double ux = sv * vtx, uy = sv * vty, uz = sv * vtz;
            const double ue = ux * ex + uy * ey + uz * ez;
            f[0] = fixed[m][0];
            f[1] = d2bf((tx * dx + ty * dy + tz * dz) / d_c);
            f[2] = d2bf((ux * dx + uy * dy + uz * dz) / d_c);
            f[3] = d2bf(tx * ux + ty * uy + tz * uz);
            f[4] = d2bf(ue * cs);
            f[5] = d2bf(-ue * sn);
            f[6] = fixed[m][1];
            f[7] = d2bf(kx * ux + ky * uy + kz * uz);
            f[8] = fixed[m][2];
            f[9] = fixed[m][3];
            f[10] = d2bf(1.0);
        }
        for (int t = lane; t < 8 * nr; t += 64) {   // own rooftops (7 a row) and the two scalars
            const int q = t % 8, rl = t / 8;
            uint16_t* out = st + rl * NF;
            if (q == 7) {
                out[0] = d2bf(10.0 * (w.len / lam - 0.5));
                out[1] = d2bf((double)cnt / 16.0);
                continue;
            }
            const int64_t r = row0s + rl - p * R;
            const double kx = k_hat[3 * r], ky = k_hat[3 * r + 1], kz = k_hat[3 * r + 2];
            const double te0 = w.tx * e_hat[3 * r] + w.ty * e_hat[3 * r + 1] + w.tz * e_hat[3 * r + 2];
            const double sp = te0 >= 0.0 ? 1.0 : -1.0;
            const double te = sp * te0;
            const double beta = kp * (sp * (kx * w.tx + ky * w.ty + kz * w.tz));   // half turns per metre
            double sn, cs;
            sincospi_any(beta * (-0.5 * w.len + (q + 1) * D), sn, cs);
            const double env = sinc_d(PI_H * beta * D / 2.0);
            const double a = te * (env * env);
            out[2 + 2 * q] = d2bf(a * cs);
            out[3 + 2 * q] = d2bf(-a * sn);
        }
        __syncthreads();
        uint4* dst = reinterpret_cast<uint4*>(feat + (row0s - row0) * NF);   // the rows are consecutive, 384 bytes each
        for (int t = lane; t < nr * (NF / 8); t += 64) dst[t] = reinterpret_cast<const uint4*>(st)[t];
        __syncthreads();
    }
}

// ------------------------------------------------------------------ currents <-> outputs
// Isolated response of wire w: b = Pinv_p u_p exp(+j k k_hat.c_p), raw rooftop
// order, FP64 accumulation over the stored inverse self block; kp = 2/lambda.
// The rooftops' phases are walked outwards from the wire's centre by one complex
// product each, the segment's phase and its sinc come from one half angle.
template <typename CZ>
__device__ __forceinline__ void isolated_response(const Wire& w, const CZ* __restrict__ P, const double* kh,
                                                  const double* eh, double kp, c128 (&b)[7]) {
    const double te = w.tx * eh[0] + w.ty * eh[1] + w.tz * eh[2];
    const double D = w.len / 8.0;
    const double bd = kp * (kh[0] * w.tx + kh[1] * w.ty + kh[2] * w.tz) * D;   // phase of a segment, half turns
    double sh, ch;
    sincospi_any(0.5 * bd, sh, ch);
    const double h = PI_H * 0.5 * bd;
    const double sc = fabs(h) < 1e-4 ? 1.0 - h * h / 6.0 : sh / h;
    const double env = te * D * (sc * sc);
    const c128 fwd = {fma(-2.0 * sh, sh, 1.0), -2.0 * sh * ch}, bwd = {fwd.re, -fwd.im};
    c128 u[7];
    u[3] = c128{env, 0.0};
#pragma unroll
    for (int m = 1; m <= 3; ++m) {
        u[3 + m] = cmul(u[2 + m], fwd);
        u[3 - m] = cmul(u[4 - m], bwd);
    }
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        c128 a{0.0, 0.0};
#pragma unroll
        for (int j = 0; j < 7; ++j) cfma(a, ccast<c128>(P[i * 7 + j]), u[j]);
        b[i] = a;
    }
}

template <typename CZ>
__global__ void k_targets(const Wire* __restrict__ wires, const int32_t* __restrict__ iperm, const CZ* __restrict__ Pinv,
                          int64_t n, int64_t R, const double* __restrict__ k_hat, const double* __restrict__ e_hat,
                          double kp, const c128* __restrict__ X, float* __restrict__ Y) {
    const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (row >= n * R) return;
    const int64_t p = row / R, r = row - p * R;
    const int32_t ip = iperm[p];
    const Wire w = wires[ip];
    const double* kh = k_hat + 3 * r;
    const double* eh = e_hat + 3 * r;
    const bool flip = (w.tx * eh[0] + w.ty * eh[1] + w.tz * eh[2]) < 0.0;
    c128 b[7];
    isolated_response(w, Pinv + (int64_t)ip * 49, kh, eh, kp, b);
    double sn, cs;
    sincospi_any(kp * (kh[0] * w.cx + kh[1] * w.cy + kh[2] * w.cz), sn, cs);
    const double sc = (flip ? -1.0 : 1.0) / X_SCALE;
#pragma unroll
    for (int q = 0; q < 7; ++q) {
        const int qr = flip ? 6 - q : q;
        const c128 x = X[(p * 7 + qr) * R + r];
        const double dr = (x.re * cs - x.im * sn) - b[qr].re;
        const double di = (x.re * sn + x.im * cs) - b[qr].im;
        Y[row * NO + 2 * q] = (float)(sc * dr);
        Y[row * NO + 2 * q + 1] = (float)(sc * di);
    }
}

template <typename CZ>
__global__ void k_assemble(const Wire* __restrict__ wires, const int32_t* __restrict__ iperm,
                           const CZ* __restrict__ Pinv, int64_t R, int64_t row0, int64_t n_rows,
                           const double* __restrict__ k_hat, const double* __restrict__ e_hat, double kp,
                           const float* __restrict__ Y, c128* __restrict__ X) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_rows) return;
    const int64_t row = row0 + t;
    const int64_t p = row / R, r = row - p * R;
    const int32_t ip = iperm[p];
    const Wire w = wires[ip];
    const double* kh = k_hat + 3 * r;
    const double* eh = e_hat + 3 * r;
    const bool flip = (w.tx * eh[0] + w.ty * eh[1] + w.tz * eh[2]) < 0.0;
    c128 b[7];
    isolated_response(w, Pinv + (int64_t)ip * 49, kh, eh, kp, b);
    double sn, cs;
    sincospi_any(kp * (kh[0] * w.cx + kh[1] * w.cy + kh[2] * w.cz), sn, cs);
    const double sc = (flip ? -1.0 : 1.0) * X_SCALE;
#pragma unroll
    for (int q = 0; q < 7; ++q) {
        const int qr = flip ? 6 - q : q;
        const double dr = b[qr].re + sc * Y[t * NO + 2 * q];
        const double di = b[qr].im + sc * Y[t * NO + 2 * q + 1];
        // x = (b + d) exp(-j phase)
        X[(p * 7 + qr) * R + r] = c128{dr * cs + di * sn, di * cs - dr * sn};
    }
}

// ------------------------------------------------------------------ host side
// ------------------------------------------------------------------ learned neighbourhood inverse
// The same network as a block preconditioner: sample (wire i, slot s,
// column c) of a neighbourhood-inverse buffer predicts column c of the raw
// row block W_i[i, q] (q = N(i)[s]) in the canonical frames of i and q, from
// the neighbourhood's geometry alone; the predicted rows are symmetrised like
// the computed ones.  Canonical tangent tau = sigma t, sigma = +1 when the
// first nonzero of (t_z, t_y, t_x) is positive; S = sigma P maps rooftop
// coefficients to the canonical frame (P reverses the rooftops for sigma = -1).
// Rows: (i size + s) 7 + c, internal wire order i.
constexpr int NBF_HEAD = 24, NBF_MEM = 15;   // features: head, then 15 per neighbourhood member
constexpr double NBH_TARGET_SCALE = 0.05;    // targets: departures from the block-Jacobi blocks, times this

__device__ __forceinline__ double canon_sign(const Wire& w) {
    return (w.tz > 0.0 || (w.tz == 0.0 && (w.ty > 0.0 || (w.ty == 0.0 && w.tx > 0.0)))) ? 1.0 : -1.0;
}

// |d|/d_c, tau_x.d/d_c, tau_y.d/d_c, tau_x.tau_y, Re, Im exp(-j k |d|) with d = c_y - c_x
__device__ __forceinline__ void pair_feats(const Wire& x, double sx, const Wire& y, double sy, double k, double dc,
                                           double (&f)[6]) {
#pragma clang fp contract(off)
    const double dx = y.cx - x.cx, dy = y.cy - x.cy, dz = y.cz - x.cz;
    const double xx = dx * dx, yy = dy * dy, zz = dz * dz;
    double s2 = xx + yy;
    s2 = s2 + zz;
    const double dist = sqrt(s2);
    const double xd = sx * ((x.tx * dx + x.ty * dy) + x.tz * dz);
    const double yd = sy * ((y.tx * dx + y.ty * dy) + y.tz * dz);
    const double tt = sx * sy * ((x.tx * y.tx + x.ty * y.ty) + x.tz * y.tz);
    const double ph = k * dist;
    f[0] = dist / dc;
    f[1] = xd / dc;
    f[2] = yd / dc;
    f[3] = tt;
    f[4] = cos(ph);
    f[5] = -sin(ph);
}

// One wave per (wire, slot): lanes 0..m-1 form the 15 features of one member
// each, lane 63 the head; the 192-entry row is staged in LDS and written for
// the 7 columns (one-hot c patched in) with coalesced stores.
__global__ __launch_bounds__(256) void k_nbhd_feat(const Wire* __restrict__ wires, const int32_t* __restrict__ nbt,
                                                   int size, int64_t n, int64_t row0, int64_t n_rows, double k,
                                                   double lam, double dc, uint16_t* __restrict__ feat) {
#pragma clang fp contract(off)
    __shared__ uint16_t fs[4][NF];
    const int w = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
    const int64_t g = row0 / NB_W + (int64_t)blockIdx.x * 4 + w;   // rows 7 g .. 7 g + 6
    const int64_t i = g / size;
    const int s = (int)(g - i * size);
    if (i >= n || NB_W * g >= row0 + n_rows) return;   // wave-uniform
    for (int f = lane; f < NF; f += 64) fs[w][f] = 0;
    int32_t mem[8];
    int m = 0;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        mem[t] = t < size ? nbt[i * size + t] : -1;
        m += mem[t] >= 0 ? 1 : 0;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const bool live = s < m;
    if (live) {
        const Wire wp = wires[i];
        const int32_t q = mem[s];
        const Wire wq = wires[q];
        const double sp = canon_sign(wp), sq = canon_sign(wq);
        double f6[6];
        if (lane < m) {
            int32_t wt = mem[0];
#pragma unroll
            for (int t = 1; t < 8; ++t)
                if (t == lane) wt = mem[t];
            const Wire ww = wires[wt];
            const double sw = canon_sign(ww);
            uint16_t* o = &fs[w][NBF_HEAD + NBF_MEM * lane];
            o[0] = d2bf(1.0);
            o[1] = d2bf(10.0 * (ww.len / lam - 0.5));
            pair_feats(wp, sp, ww, sw, k, dc, f6);
#pragma unroll
            for (int j = 0; j < 6; ++j) o[2 + j] = d2bf(f6[j]);
            pair_feats(wq, sq, ww, sw, k, dc, f6);
#pragma unroll
            for (int j = 0; j < 6; ++j) o[8 + j] = d2bf(f6[j]);
            const double dx = ww.cx - wq.cx, dy = ww.cy - wq.cy, dz = ww.cz - wq.cz;
            const double xx = dx * dx, yy = dy * dy, zz = dz * dz;
            double s2 = xx + yy;
            s2 = s2 + zz;
            o[14] = d2bf((wt == q || s2 <= dc * dc) ? 1.0 : 0.0);
        }
        if (lane == 63) {
            uint16_t* o = fs[w];
            o[7 + s] = d2bf(1.0);
            o[15] = d2bf(10.0 * (wp.len / lam - 0.5));
            o[16] = d2bf(10.0 * (wq.len / lam - 0.5));
            pair_feats(wp, sp, wq, sq, k, dc, f6);
#pragma unroll
            for (int j = 0; j < 6; ++j) o[17 + j] = d2bf(f6[j]);
            o[23] = d2bf(m / 8.0);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint16_t one = d2bf(1.0);
    for (int c = 0; c < NB_W; ++c) {
        const int64_t row = NB_W * g + c;
        if (row < row0 || row >= row0 + n_rows) continue;
        uint16_t* out = feat + (row - row0) * NF;
        for (int f = lane; f < NF; f += 64) out[f] = (live && f == c) ? one : fs[w][f];
    }
}

__device__ __forceinline__ int64_t block_pos(const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                             int64_t i, int32_t q) {
    int64_t p = -1;
    for (int64_t e = row_ptr[i]; e < row_ptr[i + 1]; ++e)
        if (col_idx[e] == q) p = e;
    return p;
}

// Targets of every row from a buffer of raw rows: y[2r], y[2r+1] = scale *
// (S_i (W - delta_iq Pinv_i) S_q)[r][c], the departure from the block-diagonal
// preconditioner (Pinv the inverse self blocks of the fill).
template <typename CZ>
__global__ void k_nbhd_targets(const Wire* __restrict__ wires, const int32_t* __restrict__ nbt, int size, int64_t n,
                               const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                               const CZ* __restrict__ Mv, const CZ* __restrict__ Pinv, float* __restrict__ Y) {
    const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (row >= n * size * NB_W) return;
    const int64_t g = row / NB_W;
    const int c = (int)(row - g * NB_W);
    const int64_t i = g / size;
    const int s = (int)(g - i * size);
    float* y = Y + row * NO;
    const int32_t q = nbt[i * size + s];
    if (q < 0) {
#pragma unroll
        for (int r = 0; r < NO; ++r) y[r] = 0.f;
        return;
    }
    const int64_t pos = block_pos(row_ptr, col_idx, i, q);
    const double sp = canon_sign(wires[i]), sq = canon_sign(wires[q]);
    const int cq = sq > 0 ? c : NB_W - 1 - c;
    const double f = sp * sq * NBH_TARGET_SCALE;
#pragma unroll
    for (int r = 0; r < NB_W; ++r) {
        const int rp = sp > 0 ? r : NB_W - 1 - r;
        const CZ v = Mv[pos * NB_W * NB_W + rp * NB_W + cq];
        double re = (double)v.re, im = (double)v.im;
        if (q == i) {
            const CZ b = Pinv[i * NB_W * NB_W + rp * NB_W + cq];
            re -= (double)b.re;
            im -= (double)b.im;
        }
        y[2 * r] = (float)(f * re);
        y[2 * r + 1] = (float)(f * im);
    }
}

// Raw rows from network outputs (rows [row0, row0 + n_rows)): the inverse map of k_nbhd_targets.
template <typename CZ>
__global__ void k_nbhd_assemble(const Wire* __restrict__ wires, const int32_t* __restrict__ nbt, int size,
                                const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx, int64_t row0,
                                int64_t n_rows, const float* __restrict__ Y, const CZ* __restrict__ Pinv,
                                CZ* __restrict__ Mv) {
    using R = typename real_of<CZ>::type;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_rows) return;
    const int64_t row = row0 + t;
    const int64_t g = row / NB_W;
    const int c = (int)(row - g * NB_W);
    const int64_t i = g / size;
    const int s = (int)(g - i * size);
    const int32_t q = nbt[i * size + s];
    if (q < 0) return;
    const int64_t pos = block_pos(row_ptr, col_idx, i, q);
    const double sp = canon_sign(wires[i]), sq = canon_sign(wires[q]);
    const int cq = sq > 0 ? c : NB_W - 1 - c;
    const double f = sp * sq / NBH_TARGET_SCALE;
    const float* y = Y + t * NO;
#pragma unroll
    for (int r = 0; r < NB_W; ++r) {
        const int rp = sp > 0 ? r : NB_W - 1 - r;
        double re = f * (double)y[2 * r], im = f * (double)y[2 * r + 1];
        if (q == i) {
            const CZ b = Pinv[i * NB_W * NB_W + rp * NB_W + cq];
            re += (double)b.re;
            im += (double)b.im;
        }
        Mv[pos * NB_W * NB_W + rp * NB_W + cq] = CZ{(R)re, (R)im};
    }
}

inline unsigned nblk(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }
inline int64_t pad_rows(int64_t m, int64_t a) { return (m + a - 1) / a * a; }

struct TrainBufs {
    Packed pk;
    uint16_t *fT, *aT1, *aT2, *aT3, *dYT, *dZT3, *dZT2, *dZT1;
    float *part, *loss_part, *grad;
};

void carve_packed(Carve& cv, Packed& pk) {
    pk.wt1 = cv.take<uint16_t>(NH * NF);
    pk.wt2 = cv.take<uint16_t>(NH * NH);
    pk.wt3 = cv.take<uint16_t>(NH * NH);
    pk.wt4 = cv.take<uint16_t>(NOP * NH);
    pk.wn2 = cv.take<uint16_t>(NH * NH);
    pk.wn3 = cv.take<uint16_t>(NH * NH);
    pk.wn4 = cv.take<uint16_t>(NH * DYLD);
}

TrainBufs carve_train(Carve& cv, int64_t Mpad) {
    TrainBufs b{};
    carve_packed(cv, b.pk);
    b.fT = cv.take<uint16_t>(NF * Mpad);
    b.aT1 = cv.take<uint16_t>(NH * Mpad);
    b.aT2 = cv.take<uint16_t>(NH * Mpad);
    b.aT3 = cv.take<uint16_t>(NH * Mpad);
    b.dYT = cv.take<uint16_t>(NOP * Mpad);
    b.dZT3 = cv.take<uint16_t>(NH * Mpad);
    b.dZT2 = cv.take<uint16_t>(NH * Mpad);
    b.dZT1 = cv.take<uint16_t>(NH * Mpad);
    b.part = cv.take<float>((size_t)(Mpad / SPLIT_ROWS) * NPARAM);
    b.loss_part = cv.take<float>(Mpad / 16);
    b.grad = cv.take<float>(NPARAM);
    return b;
}

struct FwdBufs {
    Packed pk;
    float* Y;
};

FwdBufs carve_fwd(Carve& cv, int64_t Mpad, bool with_y) {
    FwdBufs b{};
    carve_packed(cv, b.pk);
    b.Y = with_y ? cv.take<float>(Mpad * NO) : nullptr;
    return b;
}

chaff_status launch_pack(const float* theta, const Packed& pk, hipStream_t st) {
    hipLaunchKernelGGL(k_pack, dim3(nblk(NF * NH, 256), 7), dim3(256), 0, st, theta, pk);
    CHAFF_LAUNCH_CHECK();
    return CHAFF_OK;
}

double layer_flops(int64_t m, int k, int n) { return 2.0 * (double)m * k * n; }

// Fused inference over rows [0, M): one persistent workgroup per CU.
chaff_status forward_fused(const float* theta, const Packed& pk, const uint16_t* feat, int64_t M, float* Y,
                           hipStream_t st) {
    static const bool attr = [] {
        return hipFuncSetAttribute((const void*)k_fwd_fused, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   FUSED_LDS) == hipSuccess;
    }();
    if (!attr) return fail(CHAFF_EHIP, "cannot reserve LDS for the fused forward kernel");
    const int64_t tiles = (M + 15) / 16;
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(256, (tiles + FWD_WAVES - 1) / FWD_WAVES));
    ProfScope ps("mlp_forward", st, layer_flops(M, NF, NH) + 2 * layer_flops(M, NH, NH) + layer_flops(M, NH, NO), true);
    hipLaunchKernelGGL(k_fwd_fused, dim3(grid), dim3(64 * FWD_WAVES), FUSED_LDS, st, feat, M, theta, pk, Y);
    CHAFF_LAUNCH_CHECK();
    return CHAFF_OK;
}

}  // namespace

// ---------------------------------------------------------------- entry points (called from abi.cpp)

size_t mlp_workspace_bytes(int64_t rows, int32_t train) {
    Carve cv(nullptr, 0);
    if (train) carve_train(cv, pad_rows(rows, SPLIT_ROWS));
    else carve_fwd(cv, pad_rows(rows, ROWS_WG), false);
    return cv.off + 256;
}

chaff_status mlp_forward(const float* theta, const uint16_t* feat, int64_t M, float* Y, void* ws, size_t ws_bytes,
                         hipStream_t st) {
    Carve cv(ws, ws_bytes);
    FwdBufs b = carve_fwd(cv, pad_rows(M, ROWS_WG), false);
    if (!cv.ok()) return fail(CHAFF_EWORKSPACE, "mlp workspace too small");
    chaff_status s = launch_pack(theta, b.pk, st);
    if (s != CHAFF_OK) return s;
    return forward_fused(theta, b.pk, feat, M, Y, st);
}

// Gradient, loss and (with ad.th) the Adam step; see k_train_rows.
static chaff_status train_pass(const float* theta, const uint16_t* feat, const float* T, const int64_t* idx, int64_t M,
                               float* grad, float* loss, const AdamArgs& ad, void* ws, size_t ws_bytes,
                               hipStream_t st) {
    const int64_t Mpad = pad_rows(M, SPLIT_ROWS);
    Carve cv(ws, ws_bytes);
    TrainBufs b = carve_train(cv, Mpad);
    if (!cv.ok()) return fail(CHAFF_EWORKSPACE, "mlp workspace too small");
    if (!grad) grad = b.grad;
    chaff_status s = launch_pack(theta, b.pk, st);
    if (s != CHAFF_OK) return s;
    const int64_t nsplit = Mpad / SPLIT_ROWS;
    ProfScope ps("mlp_grad", st, 3.0 * (layer_flops(M, NF, NH) + 2 * layer_flops(M, NH, NH) + layer_flops(M, NH, NO)),
                 true);
    RowsArgs g{feat, idx, T, M, Mpad, b.pk, theta, b.fT, b.aT1, b.aT2, b.aT3, b.dYT, b.dZT3, b.dZT2, b.dZT1, b.loss_part};
    // 64 rows per workgroup re-read the weights a quarter as often, 16 spread the
    // rows over four times as many CUs: the larger tile once two workgroups per CU remain.
    // Steps of 4,096 / 16,384 / 32,768 / 262,144 rows: 16 rows 51 / 86 / 135 / 1,084 us,
    // 32 rows 55 / 80 / 122 / 892 us, 64 rows 60 / 80 / 120 / 842 us.
    const int mt = Mpad / 64 >= 512 ? 4 : Mpad / 32 >= 512 ? 2 : 1;
    const unsigned rows_grid = (unsigned)(Mpad / (16 * mt));
    switch (mt) {
        case 4: hipLaunchKernelGGL(k_train_rows<4>, dim3(rows_grid), dim3(256), 0, st, g); break;
        case 2: hipLaunchKernelGGL(k_train_rows<2>, dim3(rows_grid), dim3(256), 0, st, g); break;
        default: hipLaunchKernelGGL(k_train_rows<1>, dim3(rows_grid), dim3(256), 0, st, g); break;
    }
    CHAFF_LAUNCH_CHECK();
    for (int64_t s0 = 0; s0 < nsplit; s0 += WG_LAUNCH) {
        hipLaunchKernelGGL(k_train_wgrad, dim3((unsigned)(WG_UNITS * std::min(WG_LAUNCH, nsplit - s0))), dim3(64), 0, st, g,
                           s0, b.part);
        CHAFF_LAUNCH_CHECK();
    }
    const float scale = (float)(1.0 / ((double)M * NO));
    hipLaunchKernelGGL(k_reduce, dim3(nblk(NPARAM, 256) + 1), dim3(256), 0, st, (const float*)b.part, nsplit, scale,
                       grad, (const float*)b.loss_part, (int64_t)rows_grid, loss, ad);
    CHAFF_LAUNCH_CHECK();
    return CHAFF_OK;
}

chaff_status mlp_grad(const float* theta, const uint16_t* feat, const float* T, const int64_t* idx, int64_t M,
                      float* grad, float* loss, void* ws, size_t ws_bytes, hipStream_t st) {
    return train_pass(theta, feat, T, idx, M, grad, loss, AdamArgs{}, ws, ws_bytes, st);
}

static void bias_corrections(int32_t t, float b1, float b2, float& bc1, float& bc2) {
    bc1 = (float)(1.0 - std::pow((double)b1, (double)t));
    bc2 = (float)(1.0 - std::pow((double)b2, (double)t));
}

chaff_status mlp_adam(float* theta, float* m, float* v, const float* grad, int32_t t, float lr, float b1, float b2,
                      float eps, hipStream_t st) {
    float bc1, bc2;
    bias_corrections(t, b1, b2, bc1, bc2);
    ProfScope ps("mlp_adam", st, 4.0 * 7 * NPARAM);
    hipLaunchKernelGGL(k_adam, dim3(nblk(NPARAM, 256)), dim3(256), 0, st, theta, m, v, grad, lr, b1, b2, eps,
                       bc1, bc2);
    CHAFF_LAUNCH_CHECK();
    return CHAFF_OK;
}

chaff_status mlp_train_step(float* theta, float* m, float* v, int32_t t, float lr, float b1, float b2, float eps,
                            const uint16_t* feat, const float* T, const int64_t* idx, int64_t M, float* loss, void* ws,
                            size_t ws_bytes, hipStream_t st) {
    AdamArgs ad{theta, m, v, lr, b1, b2, eps, 0.f, 0.f};
    bias_corrections(t, b1, b2, ad.bc1, ad.bc2);
    return train_pass(theta, feat, T, idx, M, nullptr, loss, ad, ws, ws_bytes, st);
}

chaff_status mlp_features(Cloud* c, const double* k_hat, const double* e_hat, int64_t R, int64_t row0, int64_t n_rows,
                          uint16_t* feat, hipStream_t st) {
    if (n_rows == 0) return CHAFF_OK;
    ProfScope ps("mlp_features", st, (double)n_rows * NF * 2.0);
    const int64_t n_wires = (row0 + n_rows - 1) / R - row0 / R + 1;
    hipLaunchKernelGGL(k_features, dim3((unsigned)n_wires), dim3(64), 0, st, (const Wire*)c->wires,
                       (const int32_t*)c->perm, (const int32_t*)c->iperm, (const int64_t*)c->row_ptr,
                       (const int32_t*)c->col_idx, R, row0, n_rows, k_hat, e_hat, 2.0 / c->wavelength, c->wavelength,
                       c->d_c, feat);
    CHAFF_LAUNCH_CHECK();
    return CHAFF_OK;
}

chaff_status mlp_targets(Cloud* c, chaff_prec prec, const void* Pinv, const double* k_hat, const double* e_hat,
                         int64_t R, const void* X, float* Y, hipStream_t st) {
    const double kp = 2.0 / c->wavelength;
    ProfScope ps("mlp_targets", st, (double)c->n * R * (7 * 16 + NO * 4));
    if (prec == CHAFF_C64)
        hipLaunchKernelGGL(k_targets<c64>, dim3(nblk(c->n * R, 256)), dim3(256), 0, st, (const Wire*)c->wires,
                           (const int32_t*)c->iperm, (const c64*)Pinv, c->n, R, k_hat, e_hat, kp, (const c128*)X, Y);
    else
        hipLaunchKernelGGL(k_targets<c128>, dim3(nblk(c->n * R, 256)), dim3(256), 0, st, (const Wire*)c->wires,
                           (const int32_t*)c->iperm, (const c128*)Pinv, c->n, R, k_hat, e_hat, kp, (const c128*)X, Y);
    CHAFF_LAUNCH_CHECK();
    return CHAFF_OK;
}

constexpr int64_t GUESS_CHUNK = 1 << 18;  // rows per features/forward pass

size_t mlp_guess_workspace_bytes(const Cloud* c, int64_t R) {
    const int64_t rows = std::min<int64_t>(c->n * R, GUESS_CHUNK);
    Carve cv(nullptr, 0);
    carve_fwd(cv, pad_rows(rows, ROWS_WG), true);
    cv.take<uint16_t>((size_t)pad_rows(rows, ROWS_WG) * NF);
    return cv.off + 256;
}

chaff_status mlp_guess(Cloud* c, chaff_prec prec, const void* Pinv, const float* theta, const double* k_hat,
                       const double* e_hat, int64_t R, void* X, void* ws, size_t ws_bytes, hipStream_t st) {
    const int64_t total = c->n * R;
    const int64_t chunk = std::min<int64_t>(total, GUESS_CHUNK);
    Carve cv(ws, ws_bytes);
    FwdBufs b = carve_fwd(cv, pad_rows(chunk, ROWS_WG), true);
    uint16_t* feat = cv.take<uint16_t>((size_t)pad_rows(chunk, ROWS_WG) * NF);
    if (!cv.ok()) return fail(CHAFF_EWORKSPACE, "mlp guess workspace too small");
    chaff_status s = launch_pack(theta, b.pk, st);
    if (s != CHAFF_OK) return s;
    const double kp = 2.0 / c->wavelength;
    for (int64_t r0 = 0; r0 < total; r0 += chunk) {
        const int64_t nr = std::min(chunk, total - r0);
        s = mlp_features(c, k_hat, e_hat, R, r0, nr, feat, st);
        if (s != CHAFF_OK) return s;
        s = forward_fused(theta, b.pk, feat, nr, b.Y, st);
        if (s != CHAFF_OK) return s;
        ProfScope ps("mlp_assemble", st, (double)nr * (NO * 4 + 7 * 16) + (double)nr / R * 49 * (prec == CHAFF_C64 ? 8 : 16));
        if (prec == CHAFF_C64)
            hipLaunchKernelGGL(k_assemble<c64>, dim3(nblk(nr, 256)), dim3(256), 0, st, (const Wire*)c->wires,
                               (const int32_t*)c->iperm, (const c64*)Pinv, R, r0, nr, k_hat, e_hat, kp,
                               (const float*)b.Y, (c128*)X);
        else
            hipLaunchKernelGGL(k_assemble<c128>, dim3(nblk(nr, 256)), dim3(256), 0, st, (const Wire*)c->wires,
                               (const int32_t*)c->iperm, (const c128*)Pinv, R, r0, nr, k_hat, e_hat, kp,
                               (const float*)b.Y, (c128*)X);
        CHAFF_LAUNCH_CHECK();
    }
    return CHAFF_OK;
}

// ---------------------------------------------------------------- learned neighbourhood inverse (host)

constexpr int64_t NBH_MLP_CHUNK = 7 * (1 << 15);   // rows per features/forward pass (whole wire slots)

chaff_status nbhd_mlp_features_n(Cloud* c, int size, const void* M, int64_t row0, int64_t n_rows, uint16_t* feat,
                                 hipStream_t st) {
    if (n_rows == 0 || c->n == 0) return CHAFF_OK;
    const int32_t* nbt = reinterpret_cast<const int32_t*>(static_cast<const char*>(M) + NBH_HEADER);
    const double k = 2.0 * 3.14159265358979323846 / c->wavelength;
    const int64_t g0 = row0 / NB_W, g1 = (row0 + n_rows - 1) / NB_W;
    ProfScope ps("nbhd_mlp_features", st, (double)n_rows * NF * 2.0);
    hipLaunchKernelGGL(k_nbhd_feat, dim3(nblk(g1 - g0 + 1, 4)), dim3(256), 0, st, (const Wire*)c->wires, nbt, size,
                       c->n, row0, n_rows, k, c->wavelength, c->d_c, feat);
    CHAFF_LAUNCH_CHECK();
    return CHAFF_OK;
}

chaff_status nbhd_mlp_features(Cloud* c, const void* M, int64_t row0, int64_t n_rows, uint16_t* feat, hipStream_t st) {
    NbhdHeader h{};
    chaff_status s = nbhd_header(c, M, &h, st);
    if (s != CHAFF_OK) return s;
    if (row0 + n_rows > c->n * h.size * NB_W)
        return fail(CHAFF_EINVAL, "rows beyond the buffer's N * size * 7 samples");
    return nbhd_mlp_features_n(c, h.size, M, row0, n_rows, feat, st);
}

chaff_status nbhd_mlp_targets(Cloud* c, chaff_prec prec, const void* M, const void* Pinv, float* Y, hipStream_t st) {
    NbhdHeader h{};
    chaff_status s = nbhd_header(c, M, &h, st);
    if (s != CHAFF_OK) return s;
    if (!h.raw || h.prec != (int32_t)prec)
        return fail(CHAFF_EINVAL, "targets need a buffer of raw rows (chaff_nbhd_raw_rows) of the same precision");
    const int64_t rows = c->n * h.size * NB_W;
    if (rows == 0) return CHAFF_OK;
    const int32_t* nbt = reinterpret_cast<const int32_t*>(static_cast<const char*>(M) + NBH_HEADER);
    const char* vals = static_cast<const char*>(M) + nbhd_blocks_offset(c->n, h.size);
    if (prec == CHAFF_C64)
        hipLaunchKernelGGL(k_nbhd_targets<c64>, dim3(nblk(rows, 256)), dim3(256), 0, st, (const Wire*)c->wires, nbt,
                           h.size, c->n, (const int64_t*)c->row_ptr, (const int32_t*)c->col_idx, (const c64*)vals,
                           (const c64*)Pinv, Y);
    else
        hipLaunchKernelGGL(k_nbhd_targets<c128>, dim3(nblk(rows, 256)), dim3(256), 0, st, (const Wire*)c->wires, nbt,
                           h.size, c->n, (const int64_t*)c->row_ptr, (const int32_t*)c->col_idx, (const c128*)vals,
                           (const c128*)Pinv, Y);
    CHAFF_LAUNCH_CHECK();
    return CHAFF_OK;
}

size_t nbhd_mlp_workspace_bytes(const Cloud* c, int size) {
    const int64_t rows = std::max<int64_t>(1, std::min<int64_t>(c->n * size * NB_W, NBH_MLP_CHUNK));
    Carve cv(nullptr, 0);
    carve_fwd(cv, pad_rows(rows, ROWS_WG), true);
    cv.take<uint16_t>((size_t)pad_rows(rows, ROWS_WG) * NF);
    return cv.off + 256;
}

chaff_status nbhd_mlp_precond(Cloud* c, chaff_prec prec, int size, const float* theta, const void* Pinv, void* M,
                              void* ws, size_t ws_bytes, hipStream_t st) {
    chaff_status s = nbhd_begin(c, prec, size, false, M, st);
    if (s != CHAFF_OK || c->n == 0) return s;
    const int64_t total = c->n * size * NB_W;
    const int64_t chunk = std::min<int64_t>(total, NBH_MLP_CHUNK);
    Carve cv(ws, ws_bytes);
    FwdBufs b = carve_fwd(cv, pad_rows(chunk, ROWS_WG), true);
    uint16_t* feat = cv.take<uint16_t>((size_t)pad_rows(chunk, ROWS_WG) * NF);
    if (!cv.ok()) return fail(CHAFF_EWORKSPACE, "learned preconditioner workspace too small");
    s = launch_pack(theta, b.pk, st);
    if (s != CHAFF_OK) return s;
    const int32_t* nbt = reinterpret_cast<const int32_t*>(static_cast<const char*>(M) + NBH_HEADER);
    char* vals = static_cast<char*>(M) + nbhd_blocks_offset(c->n, size);
    for (int64_t r0 = 0; r0 < total; r0 += chunk) {
        const int64_t nr = std::min(chunk, total - r0);
        s = nbhd_mlp_features_n(c, size, M, r0, nr, feat, st);
        if (s != CHAFF_OK) return s;
        s = forward_fused(theta, b.pk, feat, nr, b.Y, st);
        if (s != CHAFF_OK) return s;
        ProfScope ps("nbhd_mlp_assemble", st, (double)nr * (NO * 4 + 7 * (prec == CHAFF_C64 ? 8 : 16)));
        if (prec == CHAFF_C64)
            hipLaunchKernelGGL(k_nbhd_assemble<c64>, dim3(nblk(nr, 256)), dim3(256), 0, st, (const Wire*)c->wires, nbt,
                               size, (const int64_t*)c->row_ptr, (const int32_t*)c->col_idx, r0, nr,
                               (const float*)b.Y, (const c64*)Pinv, (c64*)vals);
        else
            hipLaunchKernelGGL(k_nbhd_assemble<c128>, dim3(nblk(nr, 256)), dim3(256), 0, st, (const Wire*)c->wires,
                               nbt, size, (const int64_t*)c->row_ptr, (const int32_t*)c->col_idx, r0, nr,
                               (const float*)b.Y, (const c128*)Pinv, (c128*)vals);
        CHAFF_LAUNCH_CHECK();
    }
    s = nbhd_symmetrise(c, prec, vals, st);
    if (s != CHAFF_OK) return s;
    CHAFF_HIP(hipStreamSynchronize(st));
    return CHAFF_OK;
}

}  // namespace chaff
