// rpy_series.hip -- the whole Chebyshev series of one vector in one launch, for
// boxes of at most SERIES_MAX beads whose tensor is stored by rows
// (rpy_rows.hip).
//
// Such a product is a few microseconds of work behind four of launch.  Here a
// term takes 2.0 us at N = 100, with the trials of the adaptive order 2.5
// at N = 400, and 4.8 at N = 1000 (one launch per term: 3.9, 5.6 plus the check of each
// order, and 12.3),
// bound by the round trip of the new vector through memory:
// every wave keeps its bead row of D in registers for the whole series, and the
// workgroups pass each new vector to each other through memory: every double
// travels as two 8-byte words that carry half of it and the number of the
// term (the flag-in-data words of low-latency collective protocols), so a reader polls
// the words themselves until all of them are of the term it waits for -- no barrier, no fence, no separate flag, only relaxed
// atomic accesses at device scope.  Two slots suffice: a workgroup writes V_{p+2}
// after it has read all of V_{p+1}, so every workgroup has read all of V_p by then.
//
// The wait needs all workgroups on the device at once (64 or, adaptive, 128 at most; past
// 512 beads one per 4 beads, 256 at most).  rpy_create checks that the device holds them
// (series_use), and the host keeps those that nearly fill it from starting beside another.
// So they are, unless enough other kernels (or series of another process) run at the same time, or
// the stream may use only a part of the compute units, that
// some are only partly resident; so every wait is bounded: a workgroup that has
// waited for its limit raises a flag, all of them leave, and the finishing
// kernel, one workgroup that waits for nobody, then runs the series alone.
#include "rpy_internal.h"
#include "rpy_pairs.h"
#include "rpy_prelude.h"

namespace rpy {

// Bead rows per workgroup (B), waves per row (WPR), column blocks of 128 per wave
// (NB; 24 registers each): up to SERIES_SMALL beads (8, 1, 4) for a fixed order and (4, 2, 2)
// for the adaptive one, else (SR_B, SR_WPR, SR_NBW).
// Series of 20 terms, N = 100 / 400: (8, 1, 4) 45.9 / 53.1 us, (4, 2, 2) 47.6 / 53.7, (4, 1, 4)
// 54.8 / 63.0, (8, 2, 2) 55.0 / 61.6; adaptive to 33 terms: 85.7 / 122.0, 80.8 / 99.0 (the trials'
// sums beside the row in half the registers), 93.5 / 122.6, 93.8 / 105.9.
// N = 1000, per term: (4, 4, 2) 4.8 us; (4, 2, 4) 8.6 and (8, 2, 4) 8.2, whose
// rows spill; (8, 1, 8) 13.3.
constexpr int SR_SMALL = SERIES_SMALL;
constexpr int SR_B = 4, SR_WPR = 4, SR_NBW = 2;
static_assert(SR_WPR * SR_NBW * 128 == SERIES_MAX, "a row in registers");
static_assert((SERIES_MAX + SR_B - 1) / SR_B <= SERIES_GROUPS && SR_SMALL / 4 <= SERIES_GROUPS,
              "workgroups in the partial sums");
typedef double sr2 __attribute__((ext_vector_type(2)));
typedef unsigned long long word_t;

__device__ inline void put(word_t *p, double v, uint32_t ep)
{
    const word_t b = (word_t)__double_as_longlong(v), e = (word_t)ep << 32;
    __hip_atomic_store(p, e | (b & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(p + 1, e | (b >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Polls the n <= NW doubles q, q + stride, ... of this thread until all carry
// ep.  False if the wait ran out or another workgroup's did.
template <int NW>
__device__ inline bool take(const word_t *src, int q, int stride, int n, uint32_t ep, double *v,
                            int *abort_flag, long long limit)
{
    const long long t0 = wall_clock64();
    if (limit < 0) {   // tests: no wait is granted
        __hip_atomic_store(abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return false;
    }
    for (int it = 0;; ++it) {
        word_t w[NW][2];
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const int e = q + k * stride;
            if (e < n) {
                w[k][0] = __hip_atomic_load(src + 2 * e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                w[k][1] = __hip_atomic_load(src + 2 * e + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                w[k][0] = w[k][1] = (word_t)ep << 32;
            }
        }
        bool all = true;
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            all = all && (uint32_t)(w[k][0] >> 32) == ep && (uint32_t)(w[k][1] >> 32) == ep;
            v[k] = __longlong_as_double((long long)((w[k][1] << 32) | (w[k][0] & 0xffffffffull)));
        }
        if (all) return true;
        if ((it & 15) == 15 &&
            (__hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ||
             wall_clock64() - t0 > limit)) {
            __hip_atomic_store(abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// The arithmetic below is written with its fused operations spelled out, so that the finishing
// kernel, which runs a series again alone, rounds as the series kernel does.

// y += the lane's two columns of a column block times their vector entries x.
__device__ inline void row_block(const sr2 (&d)[6], const double *x, double &y0, double &y1, double &y2)
{
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const double x0 = x[3 * q], x1 = x[3 * q + 1], x2 = x[3 * q + 2];
        y0 = fma(d[2][q], x2, fma(d[1][q], x1, fma(d[0][q], x0, y0)));
        y1 = fma(d[4][q], x2, fma(d[3][q], x1, fma(d[1][q], x0, y1)));
        y2 = fma(d[5][q], x2, fma(d[4][q], x1, fma(d[2][q], x0, y2)));
    }
}

// V_1 = Y V_0 and V_p = 2 Y V_{p-1} - V_{p-2} from y = D V.
__device__ inline double cheb_one(double ya, double yb, double y, double v) { return fma(ya, y, -(yb * v)); }
__device__ inline double cheb_next(double ya, double yb, double y, double v, double vp)
{
    return fma(2.0, cheb_one(ya, yb, y, v), -vp);
}
// The sum of a fixed order, from its first two terms.
__device__ inline double cheb_sum2(const double *ct, double v0, double v1)
{
    return fma(ct[1], v1, 0.5 * ct[0] * v0);
}

// A wave's part of its row's product with its columns x of the staged vector:
// component l & 3 in lane l.
template <int NB>
__device__ inline double row_dot(const sr2 (&d)[NB][6], int nb, const double *x, int lane)
{
    double y0 = 0.0, y1 = 0.0, y2 = 0.0;
#pragma unroll
    for (int u = 0; u < NB; ++u)
        if (u < nb) row_block(d[u], x + 6 * (lane + 64 * u), y0, y1, y2);
    return wave_sum3(y0, y1, y2, lane);
}

// dS of order n from the history lanes (V_q in lane q & 63, set q >> 6).
__device__ inline double trial_sum(const double (&h)[2][3], int n, const double *ct, int lane)
{
    double t0 = 0.0, t1 = 0.0, t2 = 0.0;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int q = 64 * s + lane;
        const double c = q < n ? (q ? ct[q] : 0.5 * ct[0]) : 0.0;
        t0 = fma(c, h[s][0], t0);
        t1 = fma(c, h[s][1], t1);
        t2 = fma(c, h[s][2], t2);
    }
    return wave_sum3(t0, t1, t2, lane);
}

// The sum of a row's three entries (lanes 0 .. 2).
__device__ inline double row_sum(double q) { return __shfl(q, 0) + __shfl(q, 1) + __shfl(q, 2); }

// The two sums over G workgroups from their parts pr (zero past the last), in every lane.
__device__ inline void group_sums(const double *pr, int G, int lane, double &sa, double &sb)
{
    sa = pr[2 * lane];
    sb = pr[2 * lane + 1];
    for (int g = 64; g < G; g += 64) {
        sa += pr[2 * (g + lane)];
        sb += pr[2 * (g + lane) + 1];
    }
#pragma unroll
    for (int x = 32; x >= 1; x >>= 1) {
        sa += __shfl_xor(sa, x);
        sb += __shfl_xor(sb, x);
    }
}

__device__ inline bool settles(double a, double b, int n, int nmax, double tol, double &ef)
{
    ef = sqrt(fabs(a - b) / b);
    return (ef > 0.0 ? ef : 0.0) < tol || n >= nmax;   // as k_trial_check
}

// WEU: waves per SIMD at least.  (4, 2, 2) takes 157 VGPRs, one workgroup per compute unit; past
// 256 beads it is kept to 128 (a few spills: N = 400 adaptive 99.0 against 94.2 us), two per
// compute unit, so that four such kernels (one per hardware queue) are resident together.
template <int B, int WPR, int NB, int WEU = 1>
__global__ __launch_bounds__(64 * B * WPR) __attribute__((amdgpu_waves_per_eu(WEU, 8))) void k_series(SeriesArgs a)
{
    constexpr int NT = 64 * B * WPR, X = 3 * 128 * NB * WPR, NW = (X + NT - 1) / NT;
    static_assert(2 * SERIES_GROUPS <= NT, "a thread per partial sum");
    __shared__ double sx[2][X];
    __shared__ double tred[B][2], pr[2 * SERIES_GROUPS];
    __shared__ double pd[2][WPR > 1 ? WPR : 1][B][4];   // the row parts of its waves
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r = w % B, h0 = w / B;   // row of the workgroup, wave of the row
    const int i = blockIdx.x * B + r, ic = min(i, a.N - 1), n3 = 3 * a.N;
    const int nb = min(max(a.ld / 128 - NB * h0, 0), NB), G = gridDim.x;
    const bool eth = i < a.N && h0 == 0 && lane < 3;   // lanes that own the row's entries
    const size_t o = 3 * (size_t)ic + min(lane, 2);
    const double *row = a.drow + (size_t)ic * 6 * a.ld + 128 * NB * h0 + 2 * lane;
    sr2 d[NB][6];
#pragma unroll
    for (int u = 0; u < NB; ++u)
#pragma unroll
        for (int e = 0; e < 6; ++e)
            d[u][e] = u < nb ? *reinterpret_cast<const sr2 *>(row + (size_t)e * a.ld + 128 * u)
                             : sr2{0.0, 0.0};
    for (int z = threadIdx.x; z < X; z += NT) {
        sx[0][z] = z < n3 ? a.dw[z] : 0.0;
        sx[1][z] = a.F && z < n3 ? a.F[z] : 0.0;
    }
    // the row's product with sx[s]: the waves' parts in order, in every wave of the row (q: the
    // two buffers of the parts alternate between products with no barrier between)
    auto dot = [&](int s, int q) {
        double y = row_dot<NB>(d, nb, sx[s] + 3 * 128 * NB * h0, lane);
        if constexpr (WPR > 1) {
            if (lane < 4) pd[q][h0][r][lane] = y;
            __syncthreads();
            y = pd[q][0][r][lane & 3];
#pragma unroll
            for (int k = 1; k < WPR; ++k) y += pd[q][k][r][lane & 3];
        }
        return y;
    };
    const double ya = a.scal[2], yb = a.scal[3];
    const bool adapt = a.st != nullptr;
    const int nmax = a.n, nst = adapt ? a.st->n_start : 0;
    __syncthreads();
    const double v0 = sx[0][o];
    double dd;   // D dW
    if (a.have_ddw) dd = a.ddw[o];
    else dd = dot(0, 0);
    if (a.F) {
        const double f = dot(1, 1);
        if (eth) a.ud[o] = f;
    }
    if (!a.have_ddw && eth) a.ddw[o] = dd;
    double vp = v0, v = cheb_one(ya, yb, dd, v0);   // V_0, V_1
    if (eth && nmax > 2) put(a.words + 2 * o, v, a.epoch + 1);
    __syncthreads();
    for (int z = threadIdx.x; z < X; z += NT) sx[1][z] = 0.0;   // zero past 3N
    double acc = 0.0, h[2][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}}, t = 0.0;
    const double *ct = a.coef;   // fixed order: its coefficients
    auto keep = [&](int p, double x) {   // V_p into its history lane
        const double x0 = __shfl(x, 0), x1 = __shfl(x, 1), x2 = __shfl(x, 2);
#pragma unroll
        for (int s = 0; s < 2; ++s)
            if (p == 64 * s + lane) {
                h[s][0] = x0;
                h[s][1] = x1;
                h[s][2] = x2;
            }
    };
    // this workgroup's share of dS.dS and dW.D dW, to every workgroup
    auto share = [&](double s, uint32_t ep) {
        const double q3 = row_sum(eth ? s * s : 0.0), r3 = row_sum(eth ? v0 * dd : 0.0);
        if (lane == 0 && h0 == 0) {
            tred[r][0] = q3;
            tred[r][1] = r3;
        }
        __syncthreads();
        if (threadIdx.x < 2) {
            double z = tred[0][threadIdx.x];
#pragma unroll
            for (int k = 1; k < B; ++k) z += tred[k][threadIdx.x];
            put(a.part + 2 * ((ep & 1) * 2 * SERIES_GROUPS + 2 * blockIdx.x + threadIdx.x), z, ep);
        }
    };
    // the sums over all workgroups, in their order; false: the wait ran out
    auto collect = [&](uint32_t ep, double &sa, double &sb) {
        double z[1] = {0.0};
        bool ok = true;
        if ((int)threadIdx.x < 2 * G)
            ok = take<1>(a.part + 2 * (ep & 1) * 2 * SERIES_GROUPS, threadIdx.x, 0, 2 * G, ep, z, a.abort_flag,
                         a.limit);
        if (threadIdx.x < 2 * SERIES_GROUPS) pr[threadIdx.x] = (int)threadIdx.x < 2 * G ? z[0] : 0.0;
        if (__syncthreads_or(!ok)) return false;
        group_sums(pr, G, lane, sa, sb);
        return true;
    };
    if (adapt) {
        keep(0, v0);
        keep(1, v);
        if (2 >= nst) {
            t = trial_sum(h, 2, a.coef + 2 * SERIES_ORDERS, lane);
            share(t, a.epoch + 2);
        }
    } else {
        acc = cheb_sum2(ct, v0, v);
    }
    int n = 2;   // order of the last trial
    bool done = false;
    double ef = 0.0;
    for (int p = 2; p < nmax && !done; ++p) {
        // V_{p-1} from all workgroups
        double *x = sx[p & 1];
        double z[NW];
        const bool ok = take<NW>(a.words + (size_t)((p - 1) & 1 ? 0 : 1) * 2 * 3 * SERIES_MAX,
                                threadIdx.x, NT, n3, a.epoch + p - 1, z, a.abort_flag, a.limit);
#pragma unroll
        for (int k = 0; k < NW; ++k)
            if ((int)threadIdx.x + NT * k < n3) x[threadIdx.x + NT * k] = z[k];
        if (__syncthreads_or(!ok)) return;
        const double y = dot(p & 1, 0);
        const double vn = cheb_next(ya, yb, y, v, vp);
        if (adapt && p >= nst) {   // the trial of order p, formed before this product
            double sa, sb;
            if (!collect(a.epoch + p, sa, sb)) return;
            n = p;
            done = settles(sa, sb, p, nmax, a.tol, ef);
            if (done) break;
        }
        vp = v;
        v = vn;
        if (eth && p + 1 < nmax)
            put(a.words + (size_t)(p & 1 ? 0 : 1) * 2 * 3 * SERIES_MAX + 2 * o, v, a.epoch + p);
        if (adapt) {
            keep(p, v);
            if (p + 1 >= nst) {
                t = trial_sum(h, p + 1, a.coef + (size_t)(p + 1) * SERIES_ORDERS, lane);
                share(t, a.epoch + p + 1);
            }
        } else {
            acc = fma(ct[p], v, acc);
        }
    }
    if (adapt && !done) {   // the trial of the largest order
        double sa, sb;
        if (!collect(a.epoch + nmax, sa, sb)) return;
        n = nmax;
        settles(sa, sb, n, nmax, a.tol, ef);
    }
    if (eth) a.out[o] = adapt ? t : acc;
    if (!adapt && a.want_ef) {
        share(acc, a.epoch + nmax + 1);
        if (blockIdx.x == 0) {
            double sa, sb;
            if (!collect(a.epoch + nmax + 1, sa, sb)) return;
            settles(sa, sb, 0, 1, 0.0, ef);
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.rec->n = n;
        a.rec->ef = ef;
    }
}

// One workgroup.  If the series above gave up, all of it again, alone: the rows
// from memory, a row per wave with the sums split as there (B rows per workgroup, WPR waves per
// row, NB column blocks per wave), so that the result is the same to the bit; the terms in vh
// (adaptive order: all; else a ring of three).
// Then what follows the series: the adaptive state as k_trial_check leaves it,
// E_f, the Euler update and the copies of drift and noise.
constexpr int SF_NT = 1024;
template <int B, int WPR, int NB>
__global__ __launch_bounds__(SF_NT) void k_series_finish(SeriesArgs a, double *pos, double dt4,
                                                         double *drift, double *noise, double *e_f)
{
    __shared__ double sx[3 * SERIES_MAX];
    __shared__ double rsum[SERIES_MAX][2], pr[2 * SERIES_GROUPS];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, n3 = 3 * a.N;
    const bool adapt = a.st != nullptr;
    int n = a.rec->n;
    double ef = a.rec->ef;
    const bool redo = *a.abort_flag != 0;   // uniform
    if (redo) {
        const int nmax = a.n, nst = adapt ? a.st->n_start : 0, G = (a.N + B - 1) / B;
        const double ya = a.scal[2], yb = a.scal[3];
        // every row's product with the vector x in memory: use(o, y) in the lanes of its
        // entries o
        auto product = [&](const double *x, auto use) {
            __syncthreads();
            for (int z = threadIdx.x; z < 3 * SERIES_MAX; z += SF_NT) sx[z] = z < n3 ? x[z] : 0.0;
            __syncthreads();
            for (int i = w; i < a.N; i += SF_NT / 64) {
                double y = 0.0;
#pragma unroll 1
                for (int h = 0; h < WPR; ++h) {
                    const double *row = a.drow + (size_t)i * 6 * a.ld + 128 * NB * h + 2 * lane;
                    const int nb = min(max(a.ld / 128 - NB * h, 0), NB);
                    double y0 = 0.0, y1 = 0.0, y2 = 0.0;
#pragma unroll 1
                    for (int u = 0; u < nb; ++u) {
                        sr2 d[6];
#pragma unroll
                        for (int e = 0; e < 6; ++e)
                            d[e] = *reinterpret_cast<const sr2 *>(row + (size_t)e * a.ld + 128 * u);
                        row_block(d, sx + 3 * 128 * NB * h + 6 * (lane + 64 * u), y0, y1, y2);
                    }
                    const double s = wave_sum3(y0, y1, y2, lane);
                    y = h ? y + s : s;
                }
                if (lane < 3) use(3 * i + lane, y);
            }
            __syncthreads();
        };
        // out.out and dW.D dW
        auto sums = [&](double &sa, double &sb) {
            for (int i = w; i < a.N; i += SF_NT / 64) {
                const int o = 3 * i + min(lane, 2);
                const double s = a.out[o], v0 = a.dw[o], dd = a.ddw[o];
                const double q3 = row_sum(lane < 3 ? s * s : 0.0), r3 = row_sum(lane < 3 ? v0 * dd : 0.0);
                if (lane == 0) {
                    rsum[i][0] = q3;
                    rsum[i][1] = r3;
                }
            }
            __syncthreads();
            if (threadIdx.x < 2 * SERIES_GROUPS) {
                const int g = threadIdx.x >> 1, c = threadIdx.x & 1;
                double z = 0.0;
                if (g < G) {
                    z = rsum[g * B][c];
                    for (int k = 1; k < B; ++k) z += g * B + k < a.N ? rsum[g * B + k][c] : 0.0;
                }
                pr[threadIdx.x] = z;
            }
            __syncthreads();
            group_sums(pr, G, lane, sa, sb);
            __syncthreads();
        };
        auto term = [&](int p) { return a.vh + (size_t)(adapt ? p : p % 3) * a.ps; };
        if (!a.have_ddw) product(a.dw, [&](int o, double y) { a.ddw[o] = y; });
        if (a.F) product(a.F, [&](int o, double y) { a.ud[o] = y; });
        for (int z = threadIdx.x; z < n3; z += SF_NT) {
            const double v0 = a.dw[z], v1 = cheb_one(ya, yb, a.ddw[z], v0);
            term(0)[z] = v0;
            term(1)[z] = v1;
            if (!adapt) a.out[z] = cheb_sum2(a.coef, v0, v1);
        }
        bool done = false;
        ef = 0.0;
        for (int p = 1; p < nmax && !done; ++p) {
            if (p > 1)
                product(term(p - 1), [&](int o, double y) {
                    const double v = cheb_next(ya, yb, y, term(p - 1)[o], term(p - 2)[o]);
                    term(p)[o] = v;
                    if (!adapt) a.out[o] = fma(a.coef[p], v, a.out[o]);
                });
            n = p + 1;
            if (!adapt || n < nst) continue;
            __syncthreads();
            for (int i = w; i < a.N; i += SF_NT / 64) {
                double h[2][3];
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int c = 0; c < 3; ++c)
                        h[s][c] = 64 * s + lane < n ? term(64 * s + lane)[3 * i + c] : 0.0;
                const double t = trial_sum(h, n, a.coef + (size_t)n * SERIES_ORDERS, lane);
                if (lane < 3) a.out[3 * i + lane] = t;
            }
            __syncthreads();
            double sa, sb;
            sums(sa, sb);
            done = settles(sa, sb, n, nmax, a.tol, ef);
        }
        __syncthreads();
        if (!adapt && a.want_ef) {
            double sa, sb;
            sums(sa, sb);
            settles(sa, sb, 0, 1, 0.0, ef);
        }
        __syncthreads();
    }
    for (int z = threadIdx.x; z < n3; z += SF_NT) {
        const double s = a.out[z];
        if (noise) noise[z] = s;
        if (drift) drift[z] = a.ud[z];
        if (pos) pos[z] = pos[z] + dt4 * a.ud[z] + s / 1.4142135623730951;
    }
    if (threadIdx.x == 0) {
        if (e_f) *e_f = ef;
        if (redo) {
            a.abort_flag[0] = 0;
            ++a.abort_flag[1];
        }
        if (adapt) {
            AdaptState *st = a.st;
            const bool ok = (ef > 0.0 ? ef : 0.0) < a.tol;
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
}

__global__ __launch_bounds__(256) void k_series_coeffs(CoefArgs a) { series_coeffs_order(a, blockIdx.x); }

CoefArgs series_coef_args(const Ctx &c, int n0, int explicit_, double dmin, double dmax, AdaptState *st)
{
    return CoefArgs{n0, explicit_, dmin, dmax, c.scal, c.series_coef, st};
}

void launch_series_coeffs(const Ctx &c, int n0, int n1, int explicit_, double dmin, double dmax,
                          AdaptState *st, hipStream_t s)
{
    hipLaunchKernelGGL(k_series_coeffs, dim3(n1 - n0 + 1), dim3(256), 0, s,
                       series_coef_args(c, n0, explicit_, dmin, dmax, st));
}

struct SeriesForm {
    void (*kernel)(SeriesArgs);
    void (*finish)(SeriesArgs, double *, double, double *, double *, double *);
    int rows, threads;
};

static SeriesForm series_form(int N, bool adaptive)
{
    if (N > SR_SMALL)
        return {k_series<SR_B, SR_WPR, SR_NBW>, k_series_finish<SR_B, SR_WPR, SR_NBW>, SR_B, 64 * SR_B * SR_WPR};
    if (!adaptive) return {k_series<8, 1, 4>, k_series_finish<8, 1, 4>, 8, 512};
    return {N <= SR_SMALL / 2 ? k_series<4, 2, 2> : k_series<4, 2, 2, 4>, k_series_finish<4, 2, 2>, 4, 512};
}

int series_groups(int N, bool adaptive)
{
    const int r = series_form(N, adaptive).rows;
    return (N + r - 1) / r;
}

int series_per_cu(int N, bool adaptive)
{
    const SeriesForm f = series_form(N, adaptive);
    int per = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, reinterpret_cast<const void *>(f.kernel),
                                                     f.threads, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return per;
}

void launch_series(const SeriesArgs &a, hipStream_t s)
{
    const SeriesForm f = series_form(a.N, a.st != nullptr);
    hipLaunchKernelGGL(f.kernel, dim3((a.N + f.rows - 1) / f.rows), dim3(f.threads), 0, s, a);
}

void launch_series_finish(const SeriesArgs &a, double *pos, double dt4, double *drift, double *noise,
                          double *e_f, hipStream_t s)
{
    hipLaunchKernelGGL(series_form(a.N, a.st != nullptr).finish, dim3(1), dim3(SF_NT), 0, s, a, pos, dt4, drift,
                       noise, e_f);
}

}  // namespace rpy
