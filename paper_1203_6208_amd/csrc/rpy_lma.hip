// rpy_lma.hip -- the low-memory form of the diffusion-tensor product
// (arXiv:1203.6208, section "Low memory algorithm"): nothing of size N x N is
// stored; every product recomputes the real-space sum (self term, M1 over
// the images within r_c, the overlap form below 2a) from a cell list, and
// takes the reciprocal sum from the structure factors of its input as the
// stored form does.  Requires max(r_c, 2a) < L/3, so that cells of that side
// number at least 3 per axis and the 27 cells around a bead's cell hold every
// bead any of whose images is within reach (each pair then has one such image
// at most).
#include "rpy_internal.h"
#include "rpy_pairs.h"

namespace rpy {

// out[j][k] = in[j][beads[k]] (3 components), j < m: positions or vectors in
// cell order.
__global__ void k_lma_gather(int N, int m, int n3, const int *__restrict__ beads,
                             const double *__restrict__ in, double *__restrict__ out,
                             const int *__restrict__ gate)
{
    if (gate && *gate) return;   // a product past the settled adaptive order
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= m * N) return;
    const int j = e / N, k = e % N;
    const int b = beads[k];
    const double *src = in + (size_t)j * n3 + 3 * (size_t)b;
    double *dst = out + (size_t)j * n3 + 3 * (size_t)k;
    dst[0] = src[0];
    dst[1] = src[1];
    dst[2] = src[2];
}

void launch_lma_build(const Ctx &c, hipStream_t s)
{
    launch_cell_list_into(c.N, c.L, c.lma_nc, c.rt, c.lma_start, c.lma_beads, s);
    hipLaunchKernelGGL(k_lma_gather, dim3((c.N + 255) / 256), dim3(256), 0, s, c.N, 1, c.n3,
                       c.lma_beads, c.rt, c.rt_sorted, nullptr);
}

// Real-space product, matrix-free.  One wave per home bead h (sorted index), 4
// waves per workgroup (two beads per
// wave in turn 229 against 221 us at N = 16000, four 246: the last waves).  The 27 cells around its cell are 9 rows of three cells in
// x, each contiguous in cell order except where it wraps (at most 18 runs, whose bounds
// the first 18 lanes fetch together); inside a run the periodic shift is
// the same for all beads.  The 64 lanes test a run's candidates, LMA_CAND groups of 64
// loaded together (|h - shift - x_k|^2 against r_c^2 and (2a)^2; with max(r_c, 2a) < L/3 no
// image but the shifted one can pass), and append those
// that pass to a per-wave LDS queue (ballot + prefix count).  Whenever 128 are
// queued every lane evaluates two: the 3 x 3 pair blocks of their minimum images
// (the self term for k = h) times v_k.  Only about a sixth of the stencil is within
// reach, so the expensive pair terms run on full waves.  The lanes are
// combined by a fixed tree; the result goes to part slot 0 at the bead's
// own index.  Every step of the walk is deterministic.
// N = 16000, one vector: 197 us; with the 27 cells in turn, one group of candidates at
// a time tested on its minimum image and one pair per lane evaluated, 352 us (N = 2000: 26 and
// 114 us).  Bound by the FP64 instructions of the tests and of the polynomials.
constexpr int LMA_CAND = 2;   // one vector, N = 16000: 197 us; four groups 217, six 218
constexpr int LMA_QCAP = 128 + 64 * LMA_CAND;

// R queued pairs k[r] of home h, those with live[r]; NP > 0: by the polynomial pair form
// with NP terms (rpy_pairs.h), else by erfc and exp.
template <int M, int NP, int R>
__device__ __forceinline__ void lma_pairs(double hx, double hy, double hz, const int (&k)[R],
                                          const bool (&live)[R], int h, const PairConst &p,
                                          SmoothCoef coef, const double *__restrict__ rt_s,
                                          const double *__restrict__ vs, int n3, int j0,
                                          double acc[M][3])
{
    double d[R][3], r2[R], v[R][M][3];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const double *x = rt_s + 3 * (size_t)k[r];
        d[r][0] = x[0];
        d[r][1] = x[1];
        d[r][2] = x[2];
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const double *vk = vs + (size_t)(j0 + j) * n3 + 3 * (size_t)k[r];
            v[r][j][0] = vk[0];
            v[r][j][1] = vk[1];
            v[r][j][2] = vk[2];
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        d[r][0] = hx - d[r][0];
        d[r][1] = hy - d[r][1];
        d[r][2] = hz - d[r][2];
#pragma unroll
        for (int i = 0; i < 3; ++i) d[r][i] -= p.L * rint(d[r][i] * p.invL);
        r2[r] = d[r][0] * d[r][0] + d[r][1] * d[r][1] + d[r][2] * d[r][2];
    }
    double c1[R], w[R];
    if constexpr (NP > 0) smooth_images<R, NP>(r2, p, coef, c1, w);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        double b[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        const bool self = k[r] == h;
        if constexpr (NP > 0) {
            const double a = live[r] ? (self ? p.self_coeff : c1[r]) : 0.0,
                         q = live[r] && !self ? w[r] : 0.0;
            const double qx = q * d[r][0], qy = q * d[r][1];
            b[0] = fma(qx, d[r][0], a);
            b[1] = qx * d[r][1];
            b[2] = qx * d[r][2];
            b[3] = fma(qy, d[r][1], a);
            b[4] = qy * d[r][2];
            b[5] = fma(q * d[r][2], d[r][2], a);
        } else if (live[r]) {
            if (self) b[0] = b[3] = b[5] = p.self_coeff;
            else add_image(d[r][0], d[r][1], d[r][2], p, b);
        }
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const double v0 = v[r][j][0], v1 = v[r][j][1], v2 = v[r][j][2];
            acc[j][0] += b[0] * v0 + b[1] * v1 + b[2] * v2;
            acc[j][1] += b[1] * v0 + b[3] * v1 + b[4] * v2;
            acc[j][2] += b[2] * v0 + b[4] * v1 + b[5] * v2;
        }
    }
}

// Four waves per SIMD (at most 128 VGPRs; the erfc form spills a few values
// to scratch) ran the N = 32000 product 1.3x faster than the three that 169
// VGPRs allow; five or six waves were slower.
template <int M, int NP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_lma_real(int N, int n3, int n3pad, int rhs_cap, int j0,
                                                  double L, int nc, PairConst p,
                                                  const double *coef_g,
                                                  const int *__restrict__ start,
                                                  const int *__restrict__ beads,
                                                  const double *__restrict__ rt_s,
                                                  const double *__restrict__ vs,
                                                  double *__restrict__ part,
                                                  const int *__restrict__ gate)
{
    __shared__ int queue[4][LMA_QCAP];
    if (gate && *gate) return;
    constexpr int R = NP > 0 && M <= 2 ? 2 : 1;   // pairs per lane (registers)
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int *q = queue[w];
    const SmoothCoef coef = smooth_ptr(coef_g);
    const int h = blockIdx.x * 4 + w;   // wave-uniform
    if (h >= N) return;
    const double hx = rt_s[3 * (size_t)h], hy = rt_s[3 * (size_t)h + 1],
                 hz = rt_s[3 * (size_t)h + 2];
    int cx = (int)(hx / L * nc), cy = (int)(hy / L * nc), cz = (int)(hz / L * nc);
    cx = min(max(cx, 0), nc - 1);
    cy = min(max(cy, 0), nc - 1);
    cz = min(max(cz, 0), nc - 1);
    // lane 2 r + s: run s of row r = 3 (oz + 1) + oy + 1, s = 1 the wrapped cell
    int lo = 0, hi = 0;
    if (lane < 18) {
        const int r = lane >> 1, ey = (cy + r % 3 - 1 + nc) % nc, ez = (cz + r / 3 - 1 + nc) % nc;
        const int *row = start + (ez * nc + ey) * nc;
        int xa = max(cx - 1, 0), xb = min(cx + 2, nc);
        if (lane & 1) {
            xa = cx == 0 ? nc - 1 : 0;
            xb = cx == 0 || cx == nc - 1 ? xa + 1 : xa;
        }
        lo = row[xa];
        hi = row[xb];
    }
    double acc[M][3];
#pragma unroll
    for (int j = 0; j < M; ++j) acc[j][0] = acc[j][1] = acc[j][2] = 0.0;
    int qn = 0;   // queued candidates (wave-uniform)
    for (int run = 0; run < 18; ++run) {
        const int k0 = __builtin_amdgcn_readlane(lo, run), k1 = __builtin_amdgcn_readlane(hi, run);
        if (k0 == k1) continue;
        const int oy = (run >> 1) % 3 - 1, oz = run / 6 - 1;
        const double sx = run & 1 ? (cx == 0 ? hx + L : hx - L) : hx;
        const double sy = cy + oy < 0 ? hy + L : cy + oy >= nc ? hy - L : hy;
        const double sz = cz + oz < 0 ? hz + L : cz + oz >= nc ? hz - L : hz;
        for (int base = k0; base < k1; base += 64 * LMA_CAND) {
            double x[LMA_CAND][3];
#pragma unroll
            for (int u = 0; u < LMA_CAND; ++u) {
                const double *xk = rt_s + 3 * (size_t)min(base + 64 * u + lane, k1 - 1);
                x[u][0] = xk[0];
                x[u][1] = xk[1];
                x[u][2] = xk[2];
            }
#pragma unroll
            for (int u = 0; u < LMA_CAND; ++u) {
                const int k = base + 64 * u + lane;
                const double dx = sx - x[u][0], dy = sy - x[u][1], dz = sz - x[u][2];
                const double r2 = dx * dx + dy * dy + dz * dz;
                const bool in = k < k1 && (r2 <= p.rc2 || r2 < p.a2x4);
                const unsigned long long mask = __ballot(in);
                if (in) q[qn + lanes_below(mask)] = k;
                qn += __popcll(mask);
            }
            if (qn >= 64 * R) {
                pair_wave_sync();
                do {   // from the end of the queue
                    qn -= 64 * R;
                    int kk[R];
                    bool live[R];
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        kk[r] = q[qn + 64 * r + lane];
                        live[r] = true;
                    }
                    lma_pairs<M, NP, R>(hx, hy, hz, kk, live, h, p, coef, rt_s, vs, n3, j0, acc);
                } while (qn >= 64 * R);
                pair_wave_sync();   // read before the next candidates overwrite it
            }
        }
    }
    pair_wave_sync();
    if (qn > 0) {
        int kk[R];
        bool live[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            live[r] = 64 * r + lane < qn;
            kk[r] = live[r] ? q[64 * r + lane] : h;
        }
        lma_pairs<M, NP, R>(hx, hy, hz, kk, live, h, p, coef, rt_s, vs, n3, j0, acc);
    }
    const int nu = beads[h];
#pragma unroll
    for (int j = 0; j < M; ++j) {
        const double s = wave_sum3(acc[j][0], acc[j][1], acc[j][2], lane);
        if (lane < 3) part[(size_t)(j0 + j) * n3pad + 3 * (size_t)nu + lane] = s;
    }
}

void launch_lma_real(const Ctx &c, const double *v, int m, hipStream_t s)
{
    hipLaunchKernelGGL(k_lma_gather, dim3((m * c.N + 255) / 256), dim3(256), 0, s, c.N, m, c.n3,
                       c.lma_beads, v, c.v_sorted, c.gate);
    const dim3 g((c.N + 3) / 4);
#define RPY_LMA_REAL_NP(MC, NP)                                                                 \
    hipLaunchKernelGGL((k_lma_real<MC, NP>), g, dim3(256), 0, s, c.N, c.n3, c.n3pad, c.rhs_cap, \
                       j0, c.L, c.lma_nc, c.pc, c.smooth, c.lma_start, c.lma_beads,             \
                       c.rt_sorted, c.v_sorted, c.part, c.gate)
#define RPY_LMA_REAL(MC)                                               \
    do {                                                               \
        if (c.smooth_np == SMOOTH_NP[0]) RPY_LMA_REAL_NP(MC, SMOOTH_NP[0]); \
        else if (c.smooth_np) RPY_LMA_REAL_NP(MC, SMOOTH_NP[1]);       \
        else RPY_LMA_REAL_NP(MC, 0);                                   \
    } while (0)
    for (int j0 = 0; j0 < m;) {   // groups of 4, 2, 1 vectors
        const int mc = (m - j0) >= 4 ? 4 : (m - j0) >= 2 ? 2 : 1;
        if (mc == 4) RPY_LMA_REAL(4);
        else if (mc == 2) RPY_LMA_REAL(2);
        else RPY_LMA_REAL(1);
        j0 += mc;
    }
#undef RPY_LMA_REAL
#undef RPY_LMA_REAL_NP
}

}  // namespace rpy
