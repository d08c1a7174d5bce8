// rpy_sf.h -- structure factors of a product's input vectors, shared by the
// tile-product kernels (arXiv:1203.6208, eq. DF, reciprocal sum taken
// per product as S_k = sum_mu {cos, sin}(k.r_mu) v_mu).
#pragma once
#include "rpy_internal.h"

namespace rpy {

// e^{i 2 pi n.s} for bead table tab[3][nmax+1] (n_x >= 0 on the half space).
__device__ inline double2 kphase(const KVec &kv, const double2 *tab, int nm1)
{
    double2 ex = tab[kv.nx];
    double2 ey = tab[nm1 + (kv.ny < 0 ? -kv.ny : kv.ny)];
    double2 ez = tab[2 * nm1 + (kv.nz < 0 ? -kv.nz : kv.nz)];
    if (kv.ny < 0) ey.y = -ey.y;
    if (kv.nz < 0) ez.y = -ez.y;
    const double2 xy = make_double2(ex.x * ey.x - ex.y * ey.y, ex.x * ey.y + ex.y * ey.x);
    return make_double2(xy.x * ez.x - xy.y * ez.y, xy.x * ez.y + xy.y * ez.x);
}

// The T_k of one input vector for a column of wave vectors (n_x, n_y, *), summed
// over every bead by one workgroup of NW waves:
//   C_k = sum_mu cos(k.r_mu) v_mu,   S_k = sum_mu sin(k.r_mu) v_mu,
//   T_k = 2 m(k) (I - khat khat) (C_k, S_k)   -> tk[k][j]        (eq. DF, third term).
// Thread t takes the beads t, t + 64 NW, ...  With E = e^{i 2 pi (n_x s_x + n_y s_y)}
// from the axis tables, a bead's share of n_z and of -n_z is built from the
// four products of (Re E, Im E) v with cos and sin of 2 pi n_z s_z: 12
// multiply-adds per pair of wave vectors.  A workgroup takes NZ values of n_z
// (12 NZ sums per thread); it is bound by the latency of its loads and of its
// reduction (DPP inside 4 lanes, then LDS, in a fixed order), and re-reads the tables of
// (n_x, n_y) and v from L2 for every NZ wave vectors and their mirrors.  NZ = 4 beside
// FP64 tiles and alone (N = 16000, 7947 wave vectors: 92 us, with 2: 134 us; N = 2000,
// two vectors per pair of the reverse mode: 25 us), NZ = 2 beside the shorter FP32
// and BF16 streams, whose workgroups need the wave slots more than the
// bandwidth (FP32, N = 2000: 13.2 against 15.1 us).
// One wave vector per thread group with sincospi of every bead instead: FP32 37.9 ->
// 34.3 us at N = 4000 and 18.4 -> 13.2 us at N = 2000, FP64 22.9 -> 18.7 us at
// N = 2000; alone, with a launch that sums partials, 180 -> 92 us at N = 16000.
// With `fold`, T of a pair (n_x, n_y, +-n_z) is stored as the four vectors the
// back-projection by columns multiplies with cos and sin of 2 pi n_z s_z:
//   [pair][j][A, B, C, D] = Tc+ + Tc-, Ts+ - Ts-, Ts+ + Ts-, Tc- - Tc+.
// axt[axis (nmax + 1) + j][N] = e^{i 2 pi j s_axis}: bead-contiguous.
constexpr int SF_AHEAD = 2;   // beads whose loads go out together
struct SfCol {
    int nx, ny, nz0, cnt;   // the column, the first n_z and how many (at most NZ)
    int k0, both;           // index of n_z = 0 among the wave vectors; -n_z is one too
    int p0, pad;            // index of the pair (n_x, n_y, +-nz0) in the folded layout
};
// A column of the folded T_k: its pairs (n_x, n_y, +-n_z), n_z = 0, 1, ..., stand at p0,
// p0 + 1, ...; `len` is their number, rounded up to FOLD_STEP with zeros.
struct FoldCol {
    int nx, ny, p0, len;
};
constexpr int FOLD_STEP = 2;

// x of the lane CTRL names (a DPP control: a permutation inside 16 lanes, on
// the vector unit and not through LDS).
template <int CTRL> __device__ inline double dpp(double x)
{
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_ROR4 = 0x124, DPP_ROR8 = 0x128;

// Sums over 16 lanes, in a fixed order: lane q receives that of component
// min(q & 3, 2).  Two exchanges that halve the components, then two rotations, all
// on the vector unit: four shuffles per component through LDS instead take
// 50.3 against 44.6 us for three FP64 vectors at N = 2000, 18.4 against 16.6 us for
// one on FP32 tiles.
__device__ inline double sum16x3(double r0, double r1, double r2, int q)
{
    const bool b0 = q & 1, b1 = q & 2;
    const double a = (b0 ? r1 : r0) + dpp<DPP_XOR1>(b0 ? r0 : r1);
    const double b = r2 + dpp<DPP_XOR1>(r2);
    double r = (b1 ? b : a) + dpp<DPP_XOR2>(b1 ? a : b);
    r += dpp<DPP_ROR4>(r);
    r += dpp<DPP_ROR8>(r);
    return r;
}

// LDS: sf_lds<NW, NZ>() doubles.
template <int NW, int NZ> constexpr int sf_lds() { return 12 * NZ * (17 * NW + 1); }
template <int NW, int NZ>
__device__ __forceinline__ void sf_column(const SfCol *__restrict__ cols, int b, int N, int nm1,
                                          int rhs_cap, int j, int n3, int fold,
                                          const KCoef *__restrict__ kcoef, const double2 *axt,
                                          const double *v, double *__restrict__ tk, double *smem)
{
    constexpr int NT = 64 * NW, NS = 12 * NZ;
    const SfCol col = cols[b];
    const double2 *tx = axt + (size_t)col.nx * N, *ty = axt + (size_t)(nm1 + abs(col.ny)) * N;
    const double2 *tz = axt + (size_t)(2 * nm1 + col.nz0) * N, *t1 = axt + (size_t)(2 * nm1 + 1) * N;
    v += (size_t)j * n3;
    const double sy = col.ny < 0 ? -1.0 : 1.0;
    double a[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) a[i] = 0.0;
#pragma unroll 1
    for (int m0 = threadIdx.x; m0 < N; m0 += SF_AHEAD * NT) {
        double2 ex[SF_AHEAD], ey[SF_AHEAD], z[SF_AHEAD], z1[SF_AHEAD];
        double x[SF_AHEAD][3];
#pragma unroll
        for (int u = 0; u < SF_AHEAD; ++u) {
            const int mu = min(m0 + u * NT, N - 1);
            ex[u] = tx[mu];
            ey[u] = ty[mu];
            z[u] = tz[mu];
            z1[u] = t1[mu];
            x[u][0] = v[3 * mu];
            x[u][1] = v[3 * mu + 1];
            x[u][2] = v[3 * mu + 2];
        }
        __asm__ volatile("" ::: "memory");   // the loads of all beads before any use
#pragma unroll
        for (int u = 0; u < SF_AHEAD; ++u) {
            const double on = m0 + u * NT < N ? 1.0 : 0.0;
            const double eyi = sy * ey[u].y;
            const double er = on * (ex[u].x * ey[u].x - ex[u].y * eyi);
            const double ei = on * (ex[u].x * eyi + ex[u].y * ey[u].x);
            double zr = z[u].x, zi = z[u].y;
#pragma unroll
            for (int q = 0; q < NZ; ++q) {
                double *s = a + 12 * q;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const double w = er * x[u][c], y = ei * x[u][c];
                    s[c] = fma(w, zr, s[c]);
                    s[3 + c] = fma(y, zi, s[3 + c]);
                    s[6 + c] = fma(y, zr, s[6 + c]);
                    s[9 + c] = fma(w, zi, s[9 + c]);
                }
                const double t = zr * z1[u].x - zi * z1[u].y;
                zi = zr * z1[u].y + zi * z1[u].x;
                zr = t;
            }
        }
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        a[i] += dpp<DPP_XOR1>(a[i]);
        a[i] += dpp<DPP_XOR2>(a[i]);
    }
    // [sum][17 NW]: the 16 groups of 4 lanes of each wave, padded
    constexpr int LD = 17 * NW;
    if ((lane & 3) == 0) {
#pragma unroll
        for (int i = 0; i < NS; ++i) smem[i * LD + 17 * w + (lane >> 2)] = a[i];
    }
    __syncthreads();
    double *sum = smem + NS * LD;
    for (int e = threadIdx.x; e < NS * 4; e += NT) {   // 4 threads per sum
        const int i = e >> 2, p = e & 3;
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < 4 * NW; ++k) s += smem[i * LD + 17 * (k >> 2) + 4 * p + (k & 3)];
        s += dpp<DPP_XOR1>(s);
        s += dpp<DPP_XOR2>(s);
        if (p == 0) sum[i] = s;
    }
    __syncthreads();
    // thread (n_z, its sign, cos or sin half)
    const int q = threadIdx.x >> 2, neg = threadIdx.x >> 1 & 1, half = threadIdx.x & 1;
    if (q >= col.cnt) return;
    const int nz = col.nz0 + q, k = col.k0 + (neg ? -nz : nz);
    // n_z = 0 once; n = 0 never
    const bool have = neg ? nz != 0 && col.both : k >= 0;
    double o0 = 0.0, o1 = 0.0, o2 = 0.0;
    if (have) {
        const double sg = (half != 0) == (neg != 0) ? -1.0 : 1.0;   // C: A1 -/+ A2, S: A3 +/- A4
        const double *s = sum + 12 * q + 6 * half;
        const double s0 = s[0] + sg * s[3], s1 = s[1] + sg * s[4], s2 = s[2] + sg * s[5];
        const KCoef kc = kcoef[k];
        const double h = kc.hx * s0 + kc.hy * s1 + kc.hz * s2;
        o0 = kc.w * (s0 - kc.hx * h);
        o1 = kc.w * (s1 - kc.hy * h);
        o2 = kc.w * (s2 - kc.hz * h);
    }
    if (!fold) {
        if (!have) return;
        double *o = tk + ((size_t)k * rhs_cap + j) * 6 + 3 * half;
        o[0] = o0;
        o[1] = o1;
        o[2] = o2;
        return;
    }
    // own and mirrored T: half 0: Tc+ + Tc- and Tc- - Tc+, half 1: Ts+ + Ts- and Ts+ - Ts-
    const double p0 = dpp<DPP_XOR2>(o0), p1 = dpp<DPP_XOR2>(o1), p2 = dpp<DPP_XOR2>(o2);
    const double so = neg && half ? -1.0 : 1.0, sp = neg && !half ? -1.0 : 1.0;
    double *o = tk + ((size_t)(col.p0 + q) * rhs_cap + j) * 12 + 3 * (neg ? (half ? 1 : 3) : (half ? 2 : 0));
    o[0] = so * o0 + sp * p0;
    o[1] = so * o1 + sp * p1;
    o[2] = so * o2 + sp * p2;
}

}  // namespace rpy
