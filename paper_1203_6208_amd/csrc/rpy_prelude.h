// rpy_prelude.h -- per-thread parts of what a step needs before its tensor, shared by
// the launches of their own and by the one that does them all (rpy_step.hip).
#pragma once
#include "rpy_internal.h"

namespace rpy {

// Workgroup b (256 threads) of wrap_groups: 256 beads of entry e = axis (nmax + 1) + j, the
// phase e^{i 2 pi j s} (s = r/L
// wrapped) by bead (etab) and bead-contiguous (axt); with j = 0 the wrapped position
// rt = L (r/L - floor(r/L)).  A non-finite coordinate raises flags[0] and is
// replaced by 0 so that every later kernel still runs on finite data.
__device__ inline void wrap_entry(const WrapArgs &a, int b)
{
    const int nm1 = a.nmax + 1, nb = (a.N - 1) / 256 + 1, e = b / nb;
    const int nu = 256 * (b - e * nb) + threadIdx.x, i = e / nm1, j = e - i * nm1;
    if (nu >= a.N) return;
    double r = a.pos[3 * (size_t)nu + i];
    if (!isfinite(r)) {
        if (j == 0) atomicOr(a.flags, 1);
        r = 0.0;
    }
    double s = r / a.L;
    s = s - floor(s);
    if (j == 0) a.rt[3 * (size_t)nu + i] = a.L * s;
    double sn, cs;
    sincospi(2.0 * j * s, &sn, &cs);
    const double2 p = make_double2(cs, sn);
    a.etab[((size_t)3 * nu + i) * nm1 + j] = p;
    a.axt[(size_t)e * a.N + nu] = p;
}

// Hookean springs: F_mu = Q_mu - Q_{mu-1}, Q_mu = r_{mu+1} - r_mu within a
// chain (unwrapped positions).  Overwrites F.
__device__ inline void spring_entry(int N, int bpc, const double *__restrict__ pos,
                                    double *__restrict__ F, int mu)
{
    if (mu >= N) return;
    const int b = mu % bpc;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        double f = 0.0;
        if (b + 1 < bpc) f += pos[3 * (mu + 1) + i] - pos[3 * mu + i];
        if (b > 0) f -= pos[3 * mu + i] - pos[3 * (mu - 1) + i];
        F[3 * mu + i] = f;
    }
}

// Gaussian noise: element e uses block g = e/4, counter (g, step lo, step hi,
// 0x52505942), key (seed lo, seed hi); u = (x + 1/2) 2^-32; Box-Muller
// z0 = rho cos(2 pi u1), z1 = rho sin(2 pi u1), rho = sqrt(-2 ln u0), z2/z3
// from (u2, u3).  Scaled by sqrt(dt).
__device__ inline void noise_entry(double *__restrict__ out, int64_t count, uint64_t seed,
                                   uint64_t step, double sdt, int64_t g)
{
    if (4 * g >= count) return;
    const uint4 x = philox10(make_uint4((uint32_t)g, (uint32_t)step, (uint32_t)(step >> 32),
                                        0x52505942u),
                             make_uint2((uint32_t)seed, (uint32_t)(seed >> 32)));
    const double k = 1.0 / 4294967296.0;
    const double u0 = ((double)x.x + 0.5) * k, u1 = ((double)x.y + 0.5) * k;
    const double u2 = ((double)x.z + 0.5) * k, u3 = ((double)x.w + 0.5) * k;
    const double rho0 = sqrt(-2.0 * log(u0)), rho1 = sqrt(-2.0 * log(u2));
    double s1, c1, s3, c3;
    sincospi(2.0 * u1, &s1, &c1);
    sincospi(2.0 * u3, &s3, &c3);
    const double z[4] = {rho0 * c1, rho0 * s1, rho1 * c3, rho1 * s3};
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (4 * g + j < count) out[4 * g + j] = z[j] * sdt;
}

// The interval and the coefficients of one order, n0 + b, into
// ctab[order][SERIES_ORDERS] (256 threads).  explicit_: [dmin, dmax] given,
// and b = 0 writes the scalars and, with st, the adaptive state (as
// k_cheb_coeffs); otherwise both are there already.
__device__ inline void series_coeffs_order(const CoefArgs &a, int b)
{
    const double lo = a.explicit_ ? a.dmin : a.scal[0], hi = a.explicit_ ? a.dmax : a.scal[1];
    const int n = a.n0 + b;
    if (a.explicit_ && b == 0 && threadIdx.x == 0) {
        a.scal[0] = lo;
        a.scal[1] = hi;
        a.scal[2] = 2.0 / (hi - lo);
        a.scal[3] = (hi + lo) / (hi - lo);
        if (a.st) {
            a.st->done = 0;
            a.st->n_used = 0;
            a.st->n_start = a.n0;
            a.st->last_etol = 0;
        }
    }
    const double h = 0.5 * (hi - lo), mid = 0.5 * (hi + lo);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double f[2];   // sqrt at the nodes of this lane
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int j = 1 + lane + 64 * k;
        f[k] = j <= n ? sqrt(h * cospi((j - 0.5) / n) + mid) : 0.0;
    }
    for (int p = w; p < n; p += 4) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int j = 1 + lane + 64 * k;
            if (j <= n) s += f[k] * cospi(p * ((j - 0.5) / n));
        }
#pragma unroll
        for (int x = 32; x >= 1; x >>= 1) s += __shfl_xor(s, x);
        if (lane == 0) a.ctab[(size_t)n * SERIES_ORDERS + p] = 2.0 * s / n;
    }
}

}  // namespace rpy
