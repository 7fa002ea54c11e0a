// Wires without neighbours: a wire whose block row is its self block alone is a
// system of its own, solved in FP64 by sweeps with its inverse self block.
// Shared by the lockstep solver (krylov_impl.hpp) and the single-launch small
// solves (krylov_small.hpp); NB = rooftop unknowns per wire.
#pragma once

#include "phase.hpp"

namespace chaff {

// a^T v over one row of a stored block, FP64, four independent chains
template <int NB, typename CZ>
__device__ __forceinline__ c128 row_times(const CZ* __restrict__ row, const c128 (&v)[NB]) {
    double r0 = 0.0, r1 = 0.0, i0 = 0.0, i1 = 0.0;
#pragma unroll
    for (int m = 0; m < NB; ++m) {
        const c128 a = ccast<c128>(row[m]);
        r0 = fma(a.re, v[m].re, r0);
        r1 = fma(a.im, v[m].im, r1);
        i0 = fma(a.re, v[m].im, i0);
        i1 = fma(a.im, v[m].re, i1);
    }
    return c128{r0 - r1, i0 + i1};
}

// u of one wire and incidence (eq. 4): its first entry and the factor from one
// rooftop to the next (kp = k / pi; the half step's sine serves both the envelope
// and the factor)
template <int NB>
__device__ __forceinline__ void lone_excitation(const Wire& w, const double (&kv)[3], const double (&ev)[3], double kp,
                                                c128& first, c128& step) {
    const double tp = w.tx * ev[0] + w.ty * ev[1] + w.tz * ev[2];
    const double D = w.len / (NB + 1);
    const double bd = kp * (kv[0] * w.tx + kv[1] * w.ty + kv[2] * w.tz) * D;   // phase of a segment
    const double ph0 = kp * (kv[0] * w.cx + kv[1] * w.cy + kv[2] * w.cz);
    double sn, cs;
    sincospi_any(0.5 * bd, sn, cs);
    const double h = PI_H * (0.5 * bd);
    const double sc = fabs(h) < 1e-4 ? 1.0 - h * h / 6.0 : sn / h;
    const double env = tp * D * sc * sc;
    step = c128{cs * cs - sn * sn, -2.0 * sn * cs};
    sincospi_any(ph0 - (double)(NB / 2) * bd, sn, cs);
    first = c128{env * cs, -env * sn};
}

// One wire and incidence (kv propagation, ev polarisation): x = P u, then at most
// four sweeps of r = u - Z x, x += P r until ||r|| <= thr ||u||.  w2 = ||u||^2,
// e2 = ||r||^2 of the x returned.  u (eq. 4) is formed where it is needed, each
// rooftop's phase from the last by one complex product.  lv: the lane's own column
// of LDS; one vector at a time is held in registers and the rows of a product are
// walked by a rolled loop through it (with every product unrolled, NB^2 terms
// each, the 19-unknown form ran out of registers and instruction cache).
template <int NB, typename CZ>
__device__ __forceinline__ void lone_wire(const Wire& w, const CZ* __restrict__ zb, const CZ* __restrict__ pb,
                                          const double (&kv)[3], const double (&ev)[3], double kp, double thr,
                                          c128 (*lv)[64], int lane, c128 (&x)[NB], double& w2, double& e2) {
    c128 first, step;   // u_0 and the phase step of one rooftop
    lone_excitation<NB>(w, kv, ev, kp, first, step);
    w2 = 0.0;
    x[0] = first;
#pragma unroll
    for (int q = 1; q < NB; ++q) x[q] = cmul(x[q - 1], step);
#pragma unroll
    for (int q = 0; q < NB; ++q) w2 += x[q].re * x[q].re + x[q].im * x[q].im;
#pragma unroll 1
    for (int q = 0; q < NB; ++q) lv[q][lane] = row_times<NB>(pb + q * NB, x);
#pragma unroll 1
    for (int sweep = 0;; ++sweep) {
#pragma unroll
        for (int q = 0; q < NB; ++q) x[q] = lv[q][lane];
        e2 = 0.0;
        c128 uq = first;
#pragma unroll 1
        for (int q = 0; q < NB; ++q) {   // r = u - Z x, over x in LDS
            const c128 rq = csub(uq, row_times<NB>(zb + q * NB, x));
            e2 += rq.re * rq.re + rq.im * rq.im;
            lv[q][lane] = rq;
            uq = cmul(uq, step);
        }
        if (!(e2 > thr * thr * w2) || sweep == 4) break;
        c128 rv[NB];
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            rv[q] = lv[q][lane];
            lv[q][lane] = x[q];
        }
#pragma unroll 1
        for (int q = 0; q < NB; ++q) lv[q][lane] = cadd(lv[q][lane], row_times<NB>(pb + q * NB, rv));
    }
}

}  // namespace chaff
