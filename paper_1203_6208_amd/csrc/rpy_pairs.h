// rpy_pairs.h -- the real-space pair terms without erfc and exp: with the
// smooth part S = Omega_A - M1 (the piece the reciprocal sum carries; even
// and entire in x = alpha r), every image within r_c contributes
//   r >= 2a : M1 = Omega_A(r) - S(x^2)          (eq. M1)
//   r <  2a : M1 + M* = Omega_B(r) - S(x^2)     (eq. cor5)
// so one polynomial in r^2 per coefficient serves every image, and the only
// special function left is 1/sqrt(r^2).  Near r_c a block is the small difference of two terms
// of order a/r: its entries are accurate to the rounding of those (1e-17 of the largest
// entries of D), not to their own size as with erfc.
#pragma once

#include "rpy_internal.h"

namespace rpy {

// Coefficients of S1, S2 as polynomials in z = 2 r^2 / r_c^2 - 1, highest
// power first, interleaved (S1_n, S2_n); read through the constant address
// space so that uniform loads go to scalar registers and straight into the
// multiply-adds.
typedef const __attribute__((address_space(4))) double *SmoothCoef;

__device__ inline SmoothCoef smooth_ptr(const double *p) { return (SmoothCoef)p; }

// (c1, w) of R images at squared distances r2, all within r_c: the block is
// c1 I + w d d^T.  At r2 = 0 (coincident beads) w multiplies a zero vector.
template <int R, int NP>
__device__ inline void smooth_images(const double (&r2)[R], const PairConst &p, SmoothCoef coef,
                                     double (&c1)[R], double (&w)[R])
{
    constexpr int CH = 6, NC = (NP + CH - 1) / CH;   // terms per chunk, chunks
    const double zs = 2.0 / p.rc2;
    double z[R], s1[R], s2[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        z[q] = fma(r2[q], zs, -1.0);
        s1[q] = s2[q] = 0.0;
    }
    // The coefficients of a chunk are loaded while the previous chunk is
    // used; the empty asm ties each load to that chunk's start, since all
    // of them at once do not fit the scalar registers.  Scalar loads return
    // out of order, so a wait is always for all of them: the asm also takes
    // the current chunk, whose wait then comes before the next chunk's loads.
    double cur[2 * CH], nxt[2 * CH];
#pragma unroll
    for (int q = 0; q < R; ++q) __asm__ volatile("" : "+s"(coef), "+v"(z[q]));
#pragma unroll
    for (int i = 0; i < 2 * CH; ++i) cur[i] = coef[i];
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        if (k + 1 < NC) {
            __asm__ volatile("" : "+s"(coef), "+s"(cur[0]), "+s"(cur[2 * CH - 1]));
#pragma unroll
            for (int q = 0; q < R; ++q)
                __asm__ volatile("" : "+s"(coef), "+v"(s1[q]), "+v"(s2[q]));
#pragma unroll
            for (int i = 0; i < 2 * CH; ++i)
                if (CH * (k + 1) + i / 2 < NP) nxt[i] = coef[2 * CH * (k + 1) + i];
        }
#pragma unroll
        for (int n = 0; n < CH; ++n) {
            if (CH * k + n >= NP) break;
#pragma unroll
            for (int q = 0; q < R; ++q) {
                s1[q] = k + n ? fma(s1[q], z[q], cur[2 * n]) : cur[0];
                s2[q] = k + n ? fma(s2[q], z[q], cur[2 * n + 1]) : cur[1];
            }
        }
#pragma unroll
        for (int i = 0; i < 2 * CH; ++i) cur[i] = nxt[i];
    }
    const double ia = 1.0 / p.a;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const double ir = rsqrt(r2[q] > 0.0 ? r2[q] : 1.0);
        const double ar = p.a * ir, ar2 = ar * ar;
        const double xa = r2[q] * ir * ia;   // r / a
        const bool ov = r2[q] < p.a2x4;
        const double o1 = ov ? fma(-0.28125, xa, 1.0) : ar * fma(0.5, ar2, 0.75);
        const double o2 = ov ? 0.09375 * xa : ar * fma(-1.5, ar2, 0.75);
        c1[q] = o1 - s1[q];
        w[q] = (o2 - s2[q]) * (ir * ir);
    }
}

// Rows of one stored tile for one wave.  The beads of the row tile (nI valid)
// are at sI, those of the column tile (nJ valid) at sJ, 3 doubles each; the
// wave's 64 lanes cover 64 / TBB rows of TBB columns, and it takes
// ngroups groups of G x (64 / TBB) rows from row0.  Per group:
//   - every lane's nearest image, G rows at a time (the coefficient loads are
//     shared and the G x 2 Horner chains hide each other's latency);
//   - the images beyond the nearest one: with max(r_c, 2a) < L only those
//     with some components moved by one box length towards zero can be within
//     reach -- single components (codes 1, 2, 4) while the reach is below
//     L / sqrt 2 (NF = 3), any of the 7 combinations above (NF = 7) -- and
//     none of them is below 2a (4a < L).  The lanes' candidates are tested on
//     their exact squared distance, queued per wave in LDS (ballot + prefix
//     count) and evaluated 64 at a time: at alpha L = 6, M = 3.5 about 5 of
//     64 pairs have one.
// Two rows per group: with one the build of N = 4000 beads takes 134 us, with
// two 97, with four 105 (registers).
// store(bi, bj, b) receives the rows bi[q] of a group and the 6 entries of
// each pair (zero for padding).
constexpr int PAIR_GROUP = 2;
constexpr int PAIR_CAND = 4;   // candidates per row queued at a time
template <int NF, int G = PAIR_GROUP> constexpr int pair_queue()
{
    return G * 64 * (NF < PAIR_CAND ? NF : PAIR_CAND);
}
template <int NF> constexpr int pair_code(int f) { return NF == 3 ? 1 << f : f + 1; }

__device__ inline void pair_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Components 0..2 summed over the wave: lane l receives component l & 3 (0 in
// lane 3).
__device__ inline double wave_sum3(double a0, double a1, double a2, int lane)
{
    const bool b0 = lane & 1, b1 = lane & 2;
    const double r0 = (b0 ? a1 : a0) + __shfl_xor(b0 ? a0 : a1, 1);
    const double r1 = (b0 ? 0.0 : a2) + __shfl_xor(b0 ? a2 : 0.0, 1);
    double r = (b1 ? r1 : r0) + __shfl_xor(b1 ? r0 : r1, 2);
#pragma unroll
    for (int o = 4; o <= 32; o <<= 1) r += __shfl_xor(r, o);
    return r;
}

// Lanes below this one that are set in a wave mask.
__device__ inline int lanes_below(unsigned long long m)
{
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
}

template <int TBB, int NP, int NF, int G = PAIR_GROUP, typename Store>
__device__ inline void build_rows(const PairConst &p, SmoothCoef coef, const double *sI,
                                  const double *sJ, int nI, int nJ, bool diag, int lane, int row0,
                                  int ngroups, double *qa, double *qb, Store store)
{
    constexpr int RS = 64 / TBB;   // rows per wave step
    const int bj = lane % TBB, sub = lane / TBB;
    const double xj = sJ[3 * bj], yj = sJ[3 * bj + 1], zj = sJ[3 * bj + 2];
    const bool okj = bj < nJ;
    for (int g = 0; g < ngroups; ++g) {
        double d[G][3], e[G][3], r2[G];   // nearest image; its components moved one box length
        int rows[G];
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int bi = rows[q] = row0 + (g * G + q) * RS + sub;
            const double d0[3] = {sI[3 * bi] - xj, sI[3 * bi + 1] - yj, sI[3 * bi + 2] - zj};
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const double n = -rint(d0[a] * p.invL);
                d[q][a] = d0[a] + n * p.L;
                e[q][a] = d0[a] + (n - copysign(1.0, d[q][a])) * p.L;
            }
            r2[q] = d[q][0] * d[q][0] + d[q][1] * d[q][1] + d[q][2] * d[q][2];
        }
        double c1[G], w[G], bb[G][6];
        smooth_images<G, NP>(r2, p, coef, c1, w);
#pragma unroll
        for (int q = 0; q < G; ++q) {
            double(&b)[6] = bb[q];
            const bool live = okj && rows[q] < nI, self = diag && rows[q] == bj;
            const bool in = live && !self && (r2[q] <= p.rc2 || r2[q] < p.a2x4);
            const double a = in ? c1[q] : live && self ? p.self_coeff : 0.0, v = in ? w[q] : 0.0;
            const double vx = v * d[q][0], vy = v * d[q][1];
            b[0] = fma(vx, d[q][0], a);
            b[1] = vx * d[q][1];
            b[2] = vx * d[q][2];
            b[3] = fma(vy, d[q][1], a);
            b[4] = vy * d[q][2];
            b[5] = fma(v * d[q][2], d[q][2], a);
        }
#pragma unroll
        for (int f0 = 0; f0 < NF; f0 += PAIR_CAND) {
            unsigned hit = 0;   // bit q PAIR_CAND + f: candidate f0 + f of row q contributes
            int qn = 0;         // queued candidates (wave-uniform)
#pragma unroll
            for (int q = 0; q < G; ++q) {
                const bool live = okj && rows[q] < nI && !(diag && rows[q] == bj);
#pragma unroll
                for (int f = 0; f < PAIR_CAND && f0 + f < NF; ++f) {
                    const int code = pair_code<NF>(f0 + f);
                    const double fx = code & 1 ? e[q][0] : d[q][0],
                                 fy = code & 2 ? e[q][1] : d[q][1],
                                 fz = code & 4 ? e[q][2] : d[q][2];
                    const double f2 = fx * fx + fy * fy + fz * fz;
                    const bool in = live && f2 <= p.rc2;
                    const unsigned long long m = __ballot(in);
                    if (in) qa[qn + lanes_below(m)] = f2;
                    qn += __popcll(m);
                    hit |= in ? 1u << (q * PAIR_CAND + f) : 0u;
                }
            }
            pair_wave_sync();
            for (int s = lane; s < qn; s += 64) {
                const double f2[1] = {qa[s]};
                double fc[1], fw[1];
                smooth_images<1, NP>(f2, p, coef, fc, fw);
                qa[s] = fc[0];
                qb[s] = fw[0];
            }
            pair_wave_sync();
            int base = 0;
#pragma unroll
            for (int q = 0; q < G; ++q)
#pragma unroll
                for (int f = 0; f < PAIR_CAND && f0 + f < NF; ++f) {
                    const bool has = hit & (1u << (q * PAIR_CAND + f));
                    const unsigned long long m = __ballot(has);
                    if (m == 0) continue;   // wave-uniform
                    const int code = pair_code<NF>(f0 + f);
                    double(&b)[6] = bb[q];
                    if (has) {
                        const int s = base + lanes_below(m);
                        const double fc = qa[s], fw = qb[s];
                        const double fx = code & 1 ? e[q][0] : d[q][0],
                                     fy = code & 2 ? e[q][1] : d[q][1],
                                     fz = code & 4 ? e[q][2] : d[q][2];
                        const double ux = fw * fx, uy = fw * fy;
                        b[0] += fma(ux, fx, fc);
                        b[1] += ux * fy;
                        b[2] += ux * fz;
                        b[3] += fma(uy, fy, fc);
                        b[4] += uy * fz;
                        b[5] += fma(fw * fz, fz, fc);
                    }
                    base += __popcll(m);
                }
            pair_wave_sync();   // the queue is rewritten
        }
        store(rows, bj, bb);
    }
}

}  // namespace rpy
