// rpy_apply.hip -- the product y = D.V (stored real-space tiles + reciprocal
// sum per product) and the Fixman-Chebyshev recurrence epilogue
// (arXiv:1203.6208, eq. DFmodified and eq. cheb1-cheb3).
#include <hip/hip_ext.h>

#include "rpy_internal.h"
#include "rpy_sf.h"

namespace rpy {

#define RPY_RHS_GROUPS(m, BODY)                                              \
    for (int j0 = 0; j0 < (m);) {                                            \
        const int mc = ((m) - j0) >= 4 ? 4 : ((m) - j0);                     \
        if (mc == 4) { constexpr int MC = 4; BODY; }                         \
        else if (mc == 3) { constexpr int MC = 3; BODY; }                    \
        else if (mc == 2) { constexpr int MC = 2; BODY; }                    \
        else { constexpr int MC = 1; BODY; }                                 \
        j0 += mc;                                                            \
    }

// ------------------------------------------------------------------ SYMV
// Loads of a packed plane row (64 values of one bead row and one entry of
// the 3 x 3 blocks): lane q (0..15) of a 16-lane row group owns the bead
// columns col(q, e), e = 0..3, read with 16-byte (FP64, FP32) or 8-byte
// (BF16) loads that are contiguous across the row group: allocating loads
// when CACHED, else non-temporal ones.
template <typename T> struct P6;
template <> struct P6<double> {
    typedef double d2v __attribute__((ext_vector_type(2)));
    struct raw_t {
        d2v u, v;
    };
    static constexpr bool hoist = false;
    __device__ static int col(int q, int e) { return 32 * (e >> 1) + 2 * q + (e & 1); }
    template <bool CACHED> __device__ static raw_t raw(const double *row, int q)
    {
        const d2v *a = reinterpret_cast<const d2v *>(row + 2 * q);
        const d2v *b = reinterpret_cast<const d2v *>(row + 32 + 2 * q);
        if constexpr (CACHED) return {*a, *b};
        else return {__builtin_nontemporal_load(a), __builtin_nontemporal_load(b)};
    }
    __device__ static void cvt(const raw_t &r, double a[4])
    {
        a[0] = r.u.x;
        a[1] = r.u.y;
        a[2] = r.v.x;
        a[3] = r.v.y;
    }
};
template <> struct P6<float> {
    typedef float raw_t __attribute__((ext_vector_type(4)));
    static constexpr bool hoist = false;
    __device__ static int col(int q, int e) { return 4 * q + e; }
    template <bool CACHED> __device__ static raw_t raw(const float *row, int q)
    {
        const raw_t *a = reinterpret_cast<const raw_t *>(row + 4 * q);
        if constexpr (CACHED) return *a;
        else return __builtin_nontemporal_load(a);
    }
    __device__ static void cvt(const raw_t &u, double a[4])
    {
        a[0] = u.x;
        a[1] = u.y;
        a[2] = u.z;
        a[3] = u.w;
    }
};
template <> struct P6<uint16_t> {
    typedef uint32_t raw_t __attribute__((ext_vector_type(2)));
    static constexpr bool hoist = true;
    __device__ static int col(int q, int e) { return 4 * q + e; }
    template <bool CACHED> __device__ static raw_t raw(const uint16_t *row, int q)
    {
        const raw_t *a = reinterpret_cast<const raw_t *>(row + 4 * q);
        if constexpr (CACHED) return *a;
        else return __builtin_nontemporal_load(a);
    }
    __device__ static void cvt(const raw_t &u, double a[4])
    {
        a[0] = __uint_as_float(u.x << 16);
        a[1] = __uint_as_float(u.x & 0xFFFF0000u);
        a[2] = __uint_as_float(u.y << 16);
        a[3] = __uint_as_float(u.y & 0xFFFF0000u);
    }
};

// Product on the packed tiles (6 planes per bead row, tile[t][i][c][j]),
// FP64, FP32 or BF16 entries, FP64 arithmetic.  The first nsf
// workgroups compute T_k of one vector for a column of wave vectors each
// (sf_column; spread through an FP64 launch instead, two vectors take 80.5 against
// 78.4 us at N = 4000, one vector the same); each further workgroup (NW waves) takes
// one stored tile (I, J), in stored order or, when `flip`, in reverse order
// (each tile's results go to its own slots, so the order changes no value).
// Wave w, row group g (16 lanes), lane q: bead rows i = 4 NW it + 4 w + g
// (it < 16 / NW); lane q owns the bead columns jb(e) = P6<T>::col(q, e),
// e = 0..3, of every plane.  With B the symmetric 3 x 3 block of (i, j), the
// row sums of B x_j over the 16 lanes give A_IJ x_J -> part[J][j][rows of I];
// for off-diagonal tiles each lane also accumulates B x_i for its columns,
// and the 4 row groups and the NW waves are combined in a fixed order ->
// part[I][j][rows of J].  Diagonal tiles hold both (i, j) and (j, i) and
// take row sums only.
// Four vectors need 274 VGPRs, one wave per SIMD; capped at 256 (two waves,
// a few spills) the FP64 launch takes 132 us instead of 176 us at N = 4000.
// Three and four vectors run at two waves per SIMD.
// Waves per tile workgroup: 4, or 2 for BF16 tiles with one vector.  Those
// short, cache-resident rows are latency-bound: two waves of 32 rows each,
// every next row loaded while the current one is used, take 24.4 us at
// N = 4000 against 26.2 us for four waves with all of a lane's rows loaded
// at once (eight: 44.4 us).  FP32 tiles keep four waves (34.4 us; eight 47.3).
template <typename T, int M> constexpr int symv_waves() { return sizeof(T) == 2 && M == 1 ? 2 : 4; }

// n_z values per structure-factor workgroup of the launch (rpy_sf.h).
template <typename T> constexpr int symv_nz() { return sizeof(T) == 8 ? 4 : 2; }

template <typename T, int M, bool CACHED, int NW = symv_waves<T, M>()>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(M >= 3 ? 2 : 1, 8))) void k_symv6(int N, int n3, int n3pad, int rhs_cap, int j0,
                                               int nsf, int flip, int hot, int nm1, int fold,
                                               const SfCol *__restrict__ cols,
                                               const KCoef *__restrict__ kcoef,
                                               const double2 *__restrict__ axt,
                                               double *__restrict__ tk,
                                               const int2 *__restrict__ tile_ij,
                                               const T *__restrict__ tiles,
                                               const double *__restrict__ v,
                                               double *__restrict__ part,
                                               const int *__restrict__ gate)
{
    extern __shared__ double smem[];
    if (gate && *gate) return;   // a product past the settled adaptive order
    const int bid = blockIdx.x, ntl = (int)gridDim.x - nsf;
    if (bid < nsf) {
        sf_column<NW, symv_nz<T>()>(cols, bid / M, N, nm1, rhs_cap, j0 + bid % M, n3, fold, kcoef,
                                    axt, v, tk, smem);
        return;
    }
    double(*sx)[TS] = reinterpret_cast<double(*)[TS]>(smem);                    // [M][TS]
    double(*scol)[M][TS] = reinterpret_cast<double(*)[M][TS]>(smem + M * TS);  // [NW][M][TS]
    constexpr int NT = 64 * NW, RPI = 4 * NW, NIT = TB / RPI;   // threads, rows per pass, passes
    constexpr bool HOIST = P6<T>::hoist && NW == 4;
    const int ord = bid - nsf;
    const int t = flip ? ntl - 1 - ord : ord;
    if constexpr (CACHED) {
        constexpr bool HOT = true;
#include "rpy_symv_tile.inc"
    } else if (((long)ord + 1) * hot / ntl != (long)ord * hot / ntl) {
        // one of the `hot` tiles of a larger array, spread evenly over it
        constexpr bool HOT = true;
#include "rpy_symv_tile.inc"
    } else {
        constexpr bool HOT = false;
#include "rpy_symv_tile.inc"
    }
}

template <typename T, int M> static size_t symv_lds(const Ctx &)
{
    // sx occupies M*TS doubles, then scol[NW][M][TS]; or the structure factors
    constexpr int NW = symv_waves<T, M>(), tile = M * TS + NW * M * TS, sf = sf_lds<NW, symv_nz<T>()>();
    return sizeof(double) * (tile > sf ? tile : sf);
}

template <typename T, int M>
static void symv_launch(const Ctx &c, const T *tiles, const double *v, int j0, hipStream_t s)
{
    const SfCols &cols = symv_nz<T>() == 4 ? c.sf4 : c.sf2;
    const int nsf = cols.n * M;
    const size_t lds = symv_lds<T, M>(c);
    // Allocating loads, with the tile order reversed on every other launch,
    // for arrays that fit the Infinity Cache (each product then starts on the
    // tiles the previous one read last); otherwise stored order, allocating
    // loads for as many tiles as fit and non-temporal ones, which do not evict them, for the rest.
    const size_t bytes = (size_t)c.ntiles * TILE6 * sizeof(T);
    const bool cached = bytes <= TILE_CACHE_BYTES;
    const int hot = cached || !own_tiles<T>(c) ? 0 : (int)(TILE_CACHE_BYTES / (TILE6 * sizeof(T)));
    const int flip = cached ? (int)(c.symv_calls++ & 1u) : 0;
    // when profiled, the dispatch itself records the start and end events,
    // so that they time the kernel alone (null events: a plain launch)
    hipEvent_t e0 = c.prof_ev0, e1 = c.prof_ev1;
    c.prof_ev0 = c.prof_ev1 = nullptr;
    if (cached)
        hipExtLaunchKernelGGL((k_symv6<T, M, true>), dim3(nsf + c.ntiles), dim3(64 * symv_waves<T, M>()),
                              (uint32_t)lds, s, e0, e1, 0u, c.N, c.n3, c.n3pad, c.rhs_cap, j0, nsf,
                              flip, hot, c.nmax + 1, c.fold, cols.d, c.kcoef, c.axt, c.fold ? c.tkf : c.tk, c.tile_ij,
                              tiles, v, c.part, c.gate);
    else
        hipExtLaunchKernelGGL((k_symv6<T, M, false>), dim3(nsf + c.ntiles), dim3(64 * symv_waves<T, M>()),
                              (uint32_t)lds, s, e0, e1, 0u, c.N, c.n3, c.n3pad, c.rhs_cap, j0, nsf,
                              flip, hot, c.nmax + 1, c.fold, cols.d, c.kcoef, c.axt, c.fold ? c.tkf : c.tk, c.tile_ij,
                              tiles, v, c.part, c.gate);
}

template <typename T>
static void symv_group(const Ctx &c, const T *tiles, const double *v, int j0, int mc,
                       hipStream_t s)
{
    if (mc == 4) symv_launch<T, 4>(c, tiles, v, j0, s);
    else if (mc == 3) symv_launch<T, 3>(c, tiles, v, j0, s);
    else if (mc == 2) symv_launch<T, 2>(c, tiles, v, j0, s);
    else symv_launch<T, 1>(c, tiles, v, j0, s);
}

void launch_symv(const Ctx &c, int prec, const double *v, int j0, int mc, hipStream_t s)
{
    if (prec == RPY_PREC_F32)
        symv_group<float>(c, c.p32, v, j0, mc, s);
    else if (prec == RPY_PREC_BF16)
        symv_group<uint16_t>(c, c.p16, v, j0, mc, s);
    else
        symv_group<double>(c, c.d64, v, j0, mc, s);
}

// ------------------------------------------------------- structure factors
// Grid (columns of wave vectors, vectors).
__global__ __launch_bounds__(256) void k_sf(int N, int nm1, int rhs_cap, int n3, int fold,
                                            const SfCol *__restrict__ cols,
                                            const KCoef *__restrict__ kcoef,
                                            const double2 *__restrict__ axt,
                                            const double *__restrict__ v, double *__restrict__ tk,
                                            const int *__restrict__ gate)
{
    __shared__ double smem[sf_lds<4, 4>()];
    if (gate && *gate) return;
    sf_column<4, 4>(cols, blockIdx.x, N, nm1, rhs_cap, blockIdx.y, n3, fold, kcoef, axt, v, tk, smem);
}

void launch_sf(const Ctx &c, const double *v, int m, int fold, hipStream_t s)
{
    hipLaunchKernelGGL(k_sf, dim3(c.sf4.n, m), dim3(256), 0, s, c.N, c.nmax + 1, c.rhs_cap, c.n3,
                       fold, c.sf4.d, c.kcoef, c.axt, v, fold ? c.tkf : c.tk, c.gate);
}

// ------------------------------------- reciprocal back-projection + epilogue
// Workgroup: B beads x S = 1024 / B slices (16 waves; lane = bead (low bits) and
// sub-slice (high bits); slice u = (64 / B) wave + sub).  Slice u owns the wave
// vectors [u nk/S, (u+1) nk/S) and the tile columns K = u, u+S, ...:
//   y_u = sum_K part[K][j][3 nu + c] + sum_k cos(k.r_nu) Tc_k + sin(k.r_nu) Ts_k
// with k.r_nu = 2 pi n.s_nu.  The wave vectors are sorted by (n_x, n_y) and
// then n_z, so inside a run of equal (n_x, n_y) the phase advances by
// e^{i 2 pi s_z}; a run starts from the product of the bead's phase-table
// entries (staged in LDS), with no transcendental call.  Slices are combined in a fixed order (xor tree over the
// sub-slices, then the 16 waves in LDS), then the epilogue of `mode`:
//   EPI_APPLY      out = y
//   EPI_CHEB_FIRST V_1 = ya y - yb V_0, acc = (c_0/2) V_0 + c_1 V_1, dv = y
//   EPI_CHEB_NEXT  V_p = 2 (ya y - yb V_{p-1}) - V_{p-2}, acc += c_p V_p
//   EPI_ADJ        adjoint step mu_p = c_p g + 2 (ya y - yb mu_{p+1}) - mu_{p+2}
//                  (g = acc, read only; mu_{p+2} = 0 when vprev2 is null),
//                  dv = xs ya mu_p
// The epilogue of `mode` for one entry: bead-component index o of the vector
// block, y the product's value, (pv, pv2, pa) the recurrence operands; with
// `trial` the entry's terms of the fused trial's dot products.
__device__ __forceinline__ void epi_entry(const EpiArgs &f, size_t o, double yy, double pv, double pv2,
                                          double pa, bool trial, double &ta, double &tb2)
{
    const double ya = f.scal ? f.scal[2] : 0.0, yb = f.scal ? f.scal[3] : 0.0;
    double vnew = 0.0;   // the vector this epilogue produces
    if (f.mode == EPI_APPLY) {
        f.vout[o] = yy;
    } else if (f.mode == EPI_CHEB_FIRST) {
        const double v1 = ya * yy - yb * pv;
        f.vout[o] = v1;
        f.acc[o] = 0.5 * f.scal[8] * pv + f.scal[9] * v1;
        if (f.dv) f.dv[o] = yy;
        vnew = v1;
    } else if (f.mode == EPI_CHEB_NEXT) {
        const double vp = 2.0 * (ya * yy - yb * pv) - pv2;
        f.vout[o] = vp;
        f.acc[o] = pa + f.scal[8 + f.p] * vp;
        vnew = vp;
    } else {
        const double mp = f.scal[8 + f.p] * pa + 2.0 * (ya * yy - yb * pv) - pv2;
        f.vout[o] = mp;
        f.dv[o] = f.xs * ya * mp;
    }
    if (!trial) return;
    // the terms in k_trial_sum's order; V_p from the register
    const double *vh = f.vhist + o;
    const double v0 = vh[0];
    double d = -0.5 * f.scal[8] * v0;
    // eight stored terms loaded at a time (a load per term
    // in turn left each trial's epilogue at about 18 us)
    for (int q0 = 0; q0 < f.trial_n; q0 += 8) {
        double t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int q = q0 + u;
            t[u] = q < f.trial_n && q != f.p ? vh[(size_t)q * f.ps] : vnew;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (q0 + u < f.trial_n) d += f.scal[8 + q0 + u] * t[u];
    }
    f.ds[o] = d;
    ta = d * d;
    tb2 = v0 * f.ddw[o];
}

// B = 8 while one workgroup per compute unit covers the box (the wave-vector loop is a
// chain of LDS reads, half as long as with 16), else 16.  Product of one vector on BF16 tiles:
// N = 800 14.2 against 15.4 us, 2000 16.6 against 17.8; N = 2100 18.0 against 19.2 with 8 and
// 20.8 with 32; three vectors N = 2000 37.8 against 39.9, N = 2100 41.5 against 48.7.
constexpr int EPI_B8_MAX = 2048;
static int epi_beads(int N) { return N <= EPI_B8_MAX ? 8 : 16; }
// When `staged` (nk <= 1024, at most epi_stage_per<M>() x 1024 values of tk,
// and the tables fit the workgroup's LDS), the wave vectors and this
// launch's 6 M values of tk per k are copied to LDS once per workgroup --
// [nk + 1] KVec then [nk][M][6] + 1 -- with every load issued before the
// first LDS write (clamped indices; the copies of the clamped loads land in
// the slack entries, so no write is conditional).  The per-thread counts
// cover the 618 half-space wave vectors of alpha L = 6 for 1-4 vectors.
template <int M> constexpr int epi_stage_per() { return M == 1 ? 6 : M == 2 ? 8 : M == 3 ? 11 : 15; }
template <int M, int B>
__global__ __launch_bounds__(1024) void k_kspace_epi(int N, int n3, int n3pad, int nbt, int nk,
                                                     int nmax, int rhs_cap, int j0, int staged,
                                                     const KVec *kvec,
                                                     const double2 *__restrict__ etab,
                                                     const double *__restrict__ part,
                                                     const double *tk_g, EpiArgs f,
                                                     const int *__restrict__ gate)
{
    constexpr int S = 1024 / B;   // slices
    static_assert(3 * B <= 64, "the entries are lanes of the first wave");
    __shared__ double red[16][3][B];
    extern __shared__ double lds[];
    if (gate && *gate) return;
    const int nm1 = nmax + 1;
    double2 *tabs = reinterpret_cast<double2 *>(lds);          // [B][3 nm1]
    double *stage = lds + 2 * B * 3 * nm1;
    // Loads that do not depend on the staged tables are issued first: the
    // bead's tile-column partials and, for the 3 B threads that apply
    // the epilogue, the recurrence operands.
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int bl = lane % B, sub = lane / B;
    const int u = 64 / B * w + sub;
    const int nu = blockIdx.x * B + bl;
    const bool live = nu < N;
    double y[M][3];
#pragma unroll
    for (int j = 0; j < M; ++j) y[j][0] = y[j][1] = y[j][2] = 0.0;
    if (live) {
        for (int K = u; K < nbt; K += S) {
#pragma unroll
            for (int j = 0; j < M; ++j) {
                const double *pp = part + ((size_t)K * rhs_cap + j0 + j) * n3pad + 3 * nu;
                y[j][0] += pp[0];
                y[j][1] += pp[1];
                y[j][2] += pp[2];
            }
        }
    }
    const int eb = (int)threadIdx.x / 3, ec = (int)threadIdx.x % 3;
    const int ebead = blockIdx.x * B + eb;
    const bool eth = threadIdx.x < 3 * B && ebead < N;
    double pv[M], pv2[M], pa[M];
#pragma unroll
    for (int j = 0; j < M; ++j) {
        const size_t o = (size_t)(j0 + j) * n3 + 3 * (size_t)ebead + ec;
        pv[j] = eth && f.mode != EPI_APPLY ? f.vprev[o] : 0.0;
        pv2[j] = eth && f.vprev2 && (f.mode == EPI_CHEB_NEXT || f.mode == EPI_ADJ) ? f.vprev2[o]
                                                                                    : 0.0;
        pa[j] = eth && (f.mode == EPI_CHEB_NEXT || f.mode == EPI_ADJ) ? f.acc[o] : 0.0;
    }
    // the phase tables e^{i 2 pi j s_a} of the workgroup's beads (zero past N)
    const int ntab = B * 3 * nm1;
    const size_t tab0 = (size_t)blockIdx.x * B * 3 * nm1;
    const int nlive = min(B, N - (int)blockIdx.x * B) * 3 * nm1;
    for (int e = threadIdx.x; e < ntab; e += blockDim.x)
        tabs[e] = e < nlive ? etab[tab0 + e] : make_double2(0.0, 0.0);
    if (staged) {
        KVec *kd = reinterpret_cast<KVec *>(stage);
        double *td = stage + 2 * (nk + 1);
        const int ntk = nk * 6 * M;
        const KVec kv0 = kvec[min((int)threadIdx.x, nk - 1)];
        constexpr int SP = epi_stage_per<M>();
        double tv[SP];
#pragma unroll
        for (int i = 0; i < SP; ++i) {
            const int e = min((int)threadIdx.x + 1024 * i, ntk - 1);
            const int k = e / (6 * M), r = e % (6 * M);
            tv[i] = tk_g[((size_t)k * rhs_cap + j0) * 6 + r];
        }
        kd[min((int)threadIdx.x, nk)] = kv0;
#pragma unroll
        for (int i = 0; i < SP; ++i) td[min((int)threadIdx.x + 1024 * i, ntk)] = tv[i];
    }
    __syncthreads();
    const int klo = (int)((long)u * nk / S), khi = (int)((long)(u + 1) * nk / S);
    const double2 *tb = tabs + bl * 3 * nm1;
    const double2 ez = nm1 > 1 ? tb[2 * nm1 + 1] : make_double2(1.0, 0.0);   // e^{i 2 pi s_z}
    const double ezr = ez.x, ezi = ez.y;
    // The loop is written out once per source of the tables, so that each
    // copy reads through a pointer of known address space (LDS reads when
    // staged; a pointer that may be either compiles to generic loads).
    auto kloop = [&](const KVec *kv_s, const double *tk_s, int tk_ld) {
        double cs = 1.0, sn = 0.0;
        int px = -(1 << 30), py = 0, pz = 0;
        for (int k = klo; k < khi; ++k) {
            const KVec kv = kv_s[k];
            if (kv.nx == px && kv.ny == py && kv.nz == pz + 1) {
                const double c2 = cs * ezr - sn * ezi;
                sn = cs * ezi + sn * ezr;
                cs = c2;
            } else {   // a run start: the phase from the bead's tables
                const double2 e = kphase(kv, tb, nm1);
                cs = e.x;
                sn = e.y;
            }
            px = kv.nx;
            py = kv.ny;
            pz = kv.nz;
            const double *tt = tk_s + (size_t)k * tk_ld;
#pragma unroll
            for (int j = 0; j < M; ++j)
#pragma unroll
                for (int c = 0; c < 3; ++c) y[j][c] += cs * tt[6 * j + c] + sn * tt[6 * j + 3 + c];
        }
    };
    if (staged)
        kloop(reinterpret_cast<const KVec *>(stage), stage + 2 * (nk + 1), 6 * M);
    else
        kloop(kvec, tk_g + (size_t)j0 * 6, 6 * rhs_cap);
    // the fused trial, as k_trial_sum: skipped once the order is settled or
    // below the call's first order
    const bool trial = f.trial_n > 0 && (f.mode == EPI_CHEB_FIRST || f.mode == EPI_CHEB_NEXT) &&
                       !f.adapt->done && f.trial_n >= f.adapt->n_start;
#pragma unroll
    for (int j = 0; j < M; ++j) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            double v = y[j][c];
#pragma unroll
            for (int x = B; x <= 32; x <<= 1) v += __shfl_xor(v, x);
            if (sub == 0) red[w][c][bl] = v;
        }
        __syncthreads();
        double ta = 0.0, tb2 = 0.0;   // this entry's share of the trial's dot products
        if (eth) {
            double yy = 0.0;
#pragma unroll
            for (int ww = 0; ww < 16; ++ww) yy += red[ww][ec][eb];
            epi_entry(f, (size_t)(j0 + j) * n3 + 3 * (size_t)ebead + ec, yy, pv[j], pv2[j], pa[j], trial,
                      ta, tb2);
        }
        if (trial && w == 0) {   // the 3 B entries are lanes of the first wave
#pragma unroll
            for (int o2 = 32; o2 >= 1; o2 >>= 1) {
                ta += __shfl_xor(ta, o2);
                tb2 += __shfl_xor(tb2, o2);
            }
            if (lane == 0) {
                double *tp = f.tpart + ((size_t)(j0 + j) * gridDim.x + blockIdx.x) * 2;
                tp[0] = ta;
                tp[1] = tb2;
            }
        }
        if (j + 1 < M) __syncthreads();   // red is rewritten by the next vector
    }
}

// The same by columns of wave vectors, for wave-vector sets past the staged limit.  Workgroup:
// 64 beads (lane = bead), 16 waves that share the columns (n_x, n_y, *) in
// contiguous parts of about equal numbers of pairs +-n_z (wsplit).  Every T is
// the same for all lanes and is read through the scalar cache; with b = 2 pi n_z s_z
//   X += cos b A + sin b B,   Y += cos b C + sin b D
// over a column's pairs (12 multiply-adds and a rotation per two wave vectors), then
//   y += Re E X + Im E Y,   E = e^{i 2 pi (n_x s_x + n_y s_y)}.
// Bound by the latency of the scalar loads (about twice the time of the
// multiply-adds; four waves per SIMD).  N = 16000, 7947 wave vectors: 62 us where
// the form above, unstaged, took 230 (each vector a workgroup row of its
// own: four in one pass over the columns 305 us, in four rows 251; N = 2000: 207 and 46).  With
// the 618 wave vectors of alpha L = 6 the staged form stays ahead: 7.2 against 9.5 us at
// N = 2000, 8.2 against 10.0 us at N = 4000.
constexpr int COL_BEADS = 64;
static_assert(3 * COL_BEADS / 64 <= 8, "trial_chunks covers this form");
constexpr int COL_TRIAL = 3 * COL_BEADS / 64;   // waves that hold entries
__global__ __launch_bounds__(1024) void k_kspace_cols(int N, int n3, int n3pad, int nbt, int nm1,
                                                      int rhs_cap,
                                                      const int *__restrict__ wsplit,
                                                      const FoldCol *__restrict__ cols,
                                                      const double2 *__restrict__ axt,
                                                      const double *__restrict__ part,
                                                      const double *__restrict__ fold, EpiArgs f,
                                                      const int *__restrict__ gate)
{
    __shared__ double red[16][3][COL_BEADS];
    if (gate && *gate) return;
    const int j = blockIdx.y, lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nu = min((int)blockIdx.x * COL_BEADS + lane, N - 1);
    const int c0 = wsplit[w], c1 = wsplit[w + 1];
    const double2 *tx = axt + nu, *ty = tx + (size_t)nm1 * N;
    const double2 e1 = tx[(size_t)(2 * nm1 + 1) * N];   // e^{i 2 pi s_z}
    FoldCol nxt = cols[c0];
    double2 nex = tx[(size_t)nxt.nx * N], ney = ty[(size_t)abs(nxt.ny) * N];
    double y[3] = {0.0, 0.0, 0.0};
    for (int K = w; K < nbt; K += 16) {
        const double *pp = part + ((size_t)K * rhs_cap + j) * n3pad + 3 * (size_t)nu;
        y[0] += pp[0];
        y[1] += pp[1];
        y[2] += pp[2];
    }
    const int eb = (int)threadIdx.x / 3, ec = (int)threadIdx.x % 3;
    const int ebead = blockIdx.x * COL_BEADS + eb;
    const bool eth = threadIdx.x < 3 * COL_BEADS && ebead < N;
    for (int c = c0; c < c1; ++c) {
        const FoldCol col = nxt;
        const double2 ex = nex, ey = ney;
        nxt = cols[min(c + 1, c1 - 1)];
        nex = tx[(size_t)nxt.nx * N];
        ney = ty[(size_t)abs(nxt.ny) * N];
        double X[3] = {0.0, 0.0, 0.0}, Y[3] = {0.0, 0.0, 0.0};
        double zr = 1.0, zi = 0.0;
        const double *t = fold + ((size_t)col.p0 * rhs_cap + j) * 12;
#pragma unroll 1
        for (int p = 0; p < col.len; p += FOLD_STEP, t += (size_t)FOLD_STEP * 12 * rhs_cap) {
#pragma unroll
            for (int u = 0; u < FOLD_STEP; ++u) {
                const double *s = t + (size_t)u * 12 * rhs_cap;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    X[i] = fma(zr, s[i], X[i]);
                    X[i] = fma(zi, s[3 + i], X[i]);
                    Y[i] = fma(zr, s[6 + i], Y[i]);
                    Y[i] = fma(zi, s[9 + i], Y[i]);
                }
                const double r = zr * e1.x - zi * e1.y;
                zi = zr * e1.y + zi * e1.x;
                zr = r;
            }
        }
        const double eyi = col.ny < 0 ? -ey.y : ey.y;
        const double er = ex.x * ey.x - ex.y * eyi, ei = ex.x * eyi + ex.y * ey.x;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            y[i] = fma(er, X[i], y[i]);
            y[i] = fma(ei, Y[i], y[i]);
        }
    }
    // as k_kspace_epi: the fused trial is skipped once the order is settled
    const bool trial = f.trial_n > 0 && (f.mode == EPI_CHEB_FIRST || f.mode == EPI_CHEB_NEXT) &&
                       !f.adapt->done && f.trial_n >= f.adapt->n_start;
#pragma unroll
    for (int i = 0; i < 3; ++i) red[w][i][lane] = y[i];
    __syncthreads();
    if (w >= COL_TRIAL) return;   // the 3 COL_BEADS entries are the lanes of three waves
    double ta = 0.0, tb2 = 0.0;
    if (eth) {
        const size_t o = (size_t)j * n3 + 3 * (size_t)ebead + ec;
        const bool next = f.mode == EPI_CHEB_NEXT || f.mode == EPI_ADJ;
        const double pv = f.mode != EPI_APPLY ? f.vprev[o] : 0.0;
        const double pv2 = next && f.vprev2 ? f.vprev2[o] : 0.0, pa = next ? f.acc[o] : 0.0;
        double yy = 0.0;
#pragma unroll
        for (int ww = 0; ww < 16; ++ww) yy += red[ww][ec][eb];
        epi_entry(f, o, yy, pv, pv2, pa, trial, ta, tb2);
    }
    if (trial) {
#pragma unroll
        for (int o2 = 32; o2 >= 1; o2 >>= 1) {
            ta += __shfl_xor(ta, o2);
            tb2 += __shfl_xor(tb2, o2);
        }
        if (lane == 0) {
            double *tp = f.tpart + (((size_t)j * gridDim.x + blockIdx.x) * COL_TRIAL + w) * 2;
            tp[0] = ta;
            tp[1] = tb2;
        }
    }
}

void launch_kspace_epi(const Ctx &c, const EpiArgs &f, hipStream_t s)
{
    const dim3 b(1024);
    if (c.fold) {
        hipLaunchKernelGGL(k_kspace_cols, dim3((c.N + COL_BEADS - 1) / COL_BEADS, f.m), b, 0, s, c.N,
                           c.n3, c.n3pad, c.nslot, c.nmax + 1, c.rhs_cap, c.fold_split, c.fold_cols,
                           c.axt, c.part, c.tkf, f, c.gate);
        return;
    }
    const int beads = epi_beads(c.N);
    const dim3 g((c.N + beads - 1) / beads);
    const size_t tabs = sizeof(double) * 2 * beads * 3 * (size_t)(c.nmax + 1);
    const size_t red = sizeof(double) * 16 * 3 * beads;   // static
#define RPY_EPI(MC, B)                                                                          \
    hipLaunchKernelGGL((k_kspace_epi<MC, B>), g, b, tabs + (staged ? lds : 0), s, c.N, c.n3,    \
                       c.n3pad, c.nslot, c.nk, c.nmax, c.rhs_cap, j0, staged, c.kvec, c.etab,   \
                       c.part, c.tk, f, c.gate)
    RPY_RHS_GROUPS(f.m, {
        const size_t lds = sizeof(double) * ((size_t)c.nk * (2 + 6 * MC) + 3);
        const int staged = c.nk <= 1024 &&
                           (size_t)c.nk * 6 * MC <= (size_t)1024 * epi_stage_per<MC>() &&
                           tabs + lds + red <= (size_t)c.lds_max;
        if (beads == 8) RPY_EPI(MC, 8);
        else RPY_EPI(MC, 16);
    });
#undef RPY_EPI
}

// ------------------------------------------------- Chebyshev coefficients
// scal[0] = d_min, scal[1] = d_max, scal[2] = 2/(d_max - d_min),
// scal[3] = (d_max + d_min)/(d_max - d_min), scal[8 + p] = c_p with
//   c_p = (2/n) sum_{j=1..n} sqrt(h x_j + m) cos(p theta_j),
//   theta_j = pi (j - 1/2)/n, x_j = cos theta_j, h = (d_max-d_min)/2, m = (d_max+d_min)/2.
// One 1024-thread workgroup: wave w sums the nodes of coefficients
// p = w, w+16, ... with a lane-parallel sum in a fixed order.
__device__ void cheb_coeffs_block(int n, double lo, double hi, double *__restrict__ scal)
{
    const double h = 0.5 * (hi - lo), mid = 0.5 * (hi + lo);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int p = w; p < n; p += 16) {
        double s = 0.0;
        for (int j = 1 + lane; j <= n; j += 64) {
            const double u = (j - 0.5) / n;
            s += sqrt(h * cospi(u) + mid) * cospi(p * u);
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
        if (lane == 0) scal[8 + p] = 2.0 * s / n;
    }
}

// The interval and the coefficients.  rule = RPY_BOUNDS_PAPER derives the
// interval from du = D.U+ first, RPY_BOUNDS_DILUTE from du = [D.U+, D.U-]
// (fixed-order tree reductions).  With st
// (an adaptive call) the order is the call's first one, adapt_floor if >= 2
// or else eq. nint, nint(sqrt(d_max/d_min)) + 1 rounded half away from zero,
// clamped to [2, adapt_max]; the call's state is reset.
__global__ __launch_bounds__(1024) void k_cheb_coeffs(int nbeads, int n, int rule, double C,
                                                      double dmin, double dmax,
                                                      const double *__restrict__ du,
                                                      double *__restrict__ scal,
                                                      int adapt_floor, int adapt_max,
                                                      AdaptState *__restrict__ st)
{
    __shared__ double red[1024];
    __shared__ double bounds[2];
    __shared__ int order;
    const int tid = threadIdx.x;
    if (rule == RPY_BOUNDS_PAPER || rule == RPY_BOUNDS_DILUTE) {
        // U.D.U / 3N for U+ (du[0 .. 3N)) and, for the dilute rule, U-
        // (du[3N .. 6N) = D.U-, signs (-1)^i)
        const int n3 = 3 * nbeads;
        double uf[2];
        for (int q = 0; q < (rule == RPY_BOUNDS_DILUTE ? 2 : 1); ++q) {
            const double *d = du + (size_t)q * n3;
            double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
            int i = tid;
            for (; i + 3 * 1024 < n3; i += 4 * 1024) {
                s0 += q && (i & 1) ? -d[i] : d[i];   // 1024 is even: the four share a sign
                s1 += q && (i & 1) ? -d[i + 1024] : d[i + 1024];
                s2 += q && (i & 1) ? -d[i + 2048] : d[i + 2048];
                s3 += q && (i & 1) ? -d[i + 3072] : d[i + 3072];
            }
            for (; i < n3; i += 1024) s0 += q && (i & 1) ? -d[i] : d[i];
            red[tid] = (s0 + s1) + (s2 + s3);
            __syncthreads();
            for (int h = 512; h > 0; h >>= 1) {
                if (tid < h) red[tid] += red[tid + h];
                __syncthreads();
            }
            uf[q] = red[0] / n3;
            __syncthreads();
        }
        if (tid == 0) {
            if (rule == RPY_BOUNDS_PAPER) {   // eq. fmax, fmin
                const double np6 = pow((double)nbeads, 0.6);
                const double lmax = 0.35 * np6 * uf[0];
                bounds[0] = lmax / (C * np6);
                bounds[1] = lmax;
            } else {   // eq. lmax-lmin-dilute with d_max = 2 lmax, d_min = lmin / 2
                bounds[0] = 0.5 * uf[1];
                bounds[1] = 2.0 * uf[0];
            }
        }
    } else if (tid == 0) {
        bounds[0] = dmin;
        bounds[1] = dmax;
    }
    __syncthreads();
    const double lo = bounds[0], hi = bounds[1];
    if (tid == 0) {
        int k = n;
        if (st) {
            const double r = round(sqrt(hi / lo)) + 1.0;   // compared in FP64: no overflow
            k = adapt_floor >= 2 ? adapt_floor : (r < (double)adapt_max ? (int)r : adapt_max);
            k = k < 2 ? 2 : (k > adapt_max ? adapt_max : k);
            st->done = 0;
            st->n_used = 0;
            st->n_start = k;
            st->last_etol = 0;
        }
        order = k;
    }
    __syncthreads();
    cheb_coeffs_block(order, lo, hi, scal);
    if (tid == 0) {
        scal[0] = lo;
        scal[1] = hi;
        scal[2] = 2.0 / (hi - lo);
        scal[3] = (hi + lo) / (hi - lo);
    }
}

void launch_cheb_coeffs(const Ctx &c, int n_cheb, int rule, double C, double dmin, double dmax,
                        const double *du, hipStream_t s, int adapt_floor, int adapt_max)
{
    hipLaunchKernelGGL(k_cheb_coeffs, dim3(1), dim3(1024), 0, s, c.N, n_cheb, rule, C, dmin,
                       dmax, du, c.scal, adapt_floor, adapt_max,
                       adapt_floor >= 0 ? c.adapt : nullptr);
}

// ------------------------------------------------------ adaptive order
// Trial order n of an adaptive call (eq. nint, then the E_f criterion).
// Both kernels return at once when the call's order is settled or n is below
// its first order.  k_trial_sum: grid (chunks of 256 entries, m);
//   dS = sum_{q<n} c_q V_q - (c_0/2) V_0      (eq. cheb1, c_q in scal[8..])
// and the chunk's dS.dS and dW.(D dW) by a fixed-order tree.
__global__ __launch_bounds__(256) void k_trial_sum(int n3, int n, size_t ps,
                                                   const AdaptState *__restrict__ st,
                                                   const double *__restrict__ scal,
                                                   const double *__restrict__ vh,
                                                   const double *__restrict__ ddw,
                                                   double *__restrict__ ds,
                                                   double *__restrict__ part)
{
    __shared__ double ra[256], rb[256];
    if (st->done || n < st->n_start) return;
    const int j = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
    double a = 0.0, b = 0.0;
    if (i < n3) {
        const size_t o = (size_t)j * n3 + i;
        const double v0 = vh[o];
        double d = -0.5 * scal[8] * v0;
        for (int q = 0; q < n; ++q) d += scal[8 + q] * vh[(size_t)q * ps + o];
        ds[o] = d;
        a = d * d;
        b = v0 * ddw[o];
    }
    ra[threadIdx.x] = a;
    rb[threadIdx.x] = b;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            ra[threadIdx.x] += ra[threadIdx.x + h];
            rb[threadIdx.x] += rb[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        double *o = part + ((size_t)j * gridDim.x + blockIdx.x) * 2;
        o[0] = ra[0];
        o[1] = rb[0];
    }
}

// k_trial_check (one workgroup): the chunks summed in order per right-hand
// side, E_f = sqrt(|dS.dS - dW.D.dW| / dW.D.dW); the order is settled when
// every E_f < tol or n = nmax (e_f written, statistics updated, the ETOL
// count raised when the tolerance was missed), else the coefficients of
// order n + 1 replace those of order n.
__global__ __launch_bounds__(1024) void k_trial_check(int m, int nchunk, int n, int nmax,
                                                      double tol, AdaptState *__restrict__ st,
                                                      const double *__restrict__ part,
                                                      double *__restrict__ scal,
                                                      double *__restrict__ e_f)
{
    __shared__ double ra[1024], rb[1024];
    __shared__ double ef[MAX_RHS];
    __shared__ int settle;
    if (st->done || n < st->n_start) return;
    const int tid = threadIdx.x;
    for (int j = 0; j < m; ++j) {
        double a = 0.0, b = 0.0;
        for (int c = tid; c < nchunk; c += 1024) {
            a += part[((size_t)j * nchunk + c) * 2];
            b += part[((size_t)j * nchunk + c) * 2 + 1];
        }
        ra[tid] = a;
        rb[tid] = b;
        __syncthreads();
        for (int h = 512; h > 0; h >>= 1) {
            if (tid < h) {
                ra[tid] += ra[tid + h];
                rb[tid] += rb[tid + h];
            }
            __syncthreads();
        }
        if (tid == 0) ef[j] = sqrt(fabs(ra[0] - rb[0]) / rb[0]);
        __syncthreads();
    }
    if (tid == 0) {
        double worst = 0.0;
        for (int j = 0; j < m; ++j) worst = ef[j] > worst ? ef[j] : worst;
        const bool ok = worst < tol;
        settle = ok || n >= nmax;
        if (settle) {
            for (int j = 0; j < m; ++j) e_f[j] = ef[j];
            st->done = 1;
            st->n_used = n;
            st->last_etol = ok ? 0 : 1;
            if (!ok) {
                st->etol += 1;
                st->missed += 1;
            }
            st->calls += 1;
            st->sum_orders += n;
            if (n > st->max_order) st->max_order = n;
        }
    }
    __syncthreads();
    if (!settle) cheb_coeffs_block(n + 1, scal[0], scal[1], scal);
}

void launch_trial(const Ctx &c, int m, int n, int nmax, double tol, size_t ps,
                  const double *ddw, double *ds, double *e_f, hipStream_t s)
{
    const int nchunk = (c.n3 + 255) / 256;
    hipLaunchKernelGGL(k_trial_sum, dim3(nchunk, m), dim3(256), 0, s, c.n3, n, ps, c.adapt,
                       c.scal, c.vhist, ddw, ds, c.tpart);
    hipLaunchKernelGGL(k_trial_check, dim3(1), dim3(1024), 0, s, m, nchunk, n, nmax, tol,
                       c.adapt, c.tpart, c.scal, e_f);
}

int epi_trial_chunks(const Ctx &c)
{
    if (c.fold) return (c.N + COL_BEADS - 1) / COL_BEADS * COL_TRIAL;
    const int b = epi_beads(c.N);
    return (c.N + b - 1) / b;   // its workgroups
}

void launch_trial_check(const Ctx &c, int m, int nchunk, int n, int nmax, double tol, double *e_f,
                        hipStream_t s)
{
    hipLaunchKernelGGL(k_trial_check, dim3(1), dim3(1024), 0, s, m, nchunk, n, nmax, tol,
                       c.adapt, c.tpart, c.scal, e_f);
}

int trial_chunks(int N)
{
    const int a = (3 * N + 255) / 256, b = (N + COL_BEADS - 1) / COL_BEADS * 8;   // of any form: at most one per 8 beads
    const int r = N <= ROWS_MAX ? rows_trial_chunks(N) : 0;
    return a > b ? (a > r ? a : r) : (b > r ? b : r);
}

// E_f = sqrt(|dS.dS - dW.(D dW)| / dW.(D dW)), one workgroup per RHS.
__global__ __launch_bounds__(256) void k_sqrt_error(int n3, const double *__restrict__ dw,
                                                    const double *__restrict__ ddw,
                                                    const double *__restrict__ ds,
                                                    double *__restrict__ e_f)
{
    __shared__ double r1[256], r2[256];
    const int j = blockIdx.x;
    double a = 0.0, b = 0.0;
    for (int i = threadIdx.x; i < n3; i += blockDim.x) {
        const size_t o = (size_t)j * n3 + i;
        a += ds[o] * ds[o];
        b += dw[o] * ddw[o];
    }
    r1[threadIdx.x] = a;
    r2[threadIdx.x] = b;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h) {
            r1[threadIdx.x] += r1[threadIdx.x + h];
            r2[threadIdx.x] += r2[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) e_f[j] = sqrt(fabs(r1[0] - r2[0]) / r2[0]);
}

void launch_sqrt_error(const Ctx &c, int m, const double *dw, const double *ddw,
                       const double *ds, double *e_f, hipStream_t s)
{
    hipLaunchKernelGGL(k_sqrt_error, dim3(m), dim3(256), 0, s, c.n3, dw, ddw, ds, e_f);
}

__global__ void k_fill(double *p, double v, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
__global__ void k_copy(double *dst, const double *src, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}
void launch_fill(double *p, double v, size_t n, hipStream_t s)
{
    if (n == 0) return;
    hipLaunchKernelGGL(k_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, v, n);
}
void launch_copy(double *dst, const double *src, size_t n, hipStream_t s)
{
    if (n == 0) return;
    hipLaunchKernelGGL(k_copy, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, dst, src, n);
}

}  // namespace rpy
