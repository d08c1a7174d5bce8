// rpy_rows.hip -- the complete tensor by rows, for small FP64 boxes.
//
// With few beads a product of the tile form is two launches whose time is
// latency: the structure factors and the back-projection cost as much for one
// box of 100 beads as for 2000.  Here the reciprocal sum of eq. DF is added to
// the stored pair blocks once per set of positions, and every bead row is
// stored over all columns, drow[i][c][j] (6 planes of ld doubles, c = xx, xy,
// xz, yy, yz, zz): a row's result is then complete inside one wave, so a
// product and its recurrence step are one launch with nothing to reduce
// across workgroups.
#include "rpy_internal.h"
#include "rpy_pairs.h"

namespace rpy {

// Up to this many beads a wave takes one row and four waves share its wave
// vectors; above, two rows and two waves (weights loaded half as often).
// Measured with the wrap, us: N = 100 12.8 against 19.3, N = 400 28.1 / 25.1,
// N = 512 33.8 / 30.6; two rows per wave with no sharing, N = 1000 at 1398
// wave vectors: 141 against 113; four rows per wave lose everywhere.
constexpr int ROWS_KS_MAX = 256;
// Rows beyond the L2 caches (8 x 4 MB): walked in alternating order.
constexpr size_t ROWS_L2_BYTES = (size_t)28 << 20;

// ------------------------------------------------------------------- build
// The reciprocal part of a pair block.  The weights 2 m(k)(I - khat khat) are
// even under the sign change of any component of n up to the sign of the
// off-diagonal entries, so the sum over the half space is one over the octant
// n >= 0, with X = 2 pi n_x d_x / L and Y, Z likewise:
//   D_aa = sum W_aa cos X cos Y cos Z,    D_xy = sum W_xy sin X sin Y cos Z,
//   D_xz = sum W_xz sin X cos Y sin Z,    D_yz = sum W_yz cos X sin Y sin Z,
// W including the number of sign choices and, off the diagonal, the sign -1
// of the sine products.  Per (n_x, n_y) the sums over n_z run first: six
// multiply-adds per octant vector, 210 of them for |n|^2 <= 44.
// The weights are a stream in the order n_x, n_y, n_z, in chunks of two n_z
// (zero past the cutoff), wk[chunk][2][6]; the chunks of n_x start at off[n_x].
// They come through scalar loads straight into the multiply-adds, each chunk
// loaded while the one before it is used.  This call takes n_x = x0, x0 + KS,
// ... (KS waves share a row); ex, ey, ez: e^{i 2 pi d_a / L} of G pairs.
template <int NZ, int G, int KS>
__device__ inline void recip_block(int nmax, int n2max, int x0,
                                   const __attribute__((address_space(4))) int *off, SmoothCoef wk,
                                   const double2 (&ex)[G], const double2 (&ey)[G],
                                   const double2 (&ez)[G], double (*b)[6])
{
    constexpr int NCH = (NZ + 1) / 2;
    double cz[G][2 * NCH], sz[G][2 * NCH], cx[G], sx[G], kx[G], ky[G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
        cz[q][0] = 1.0;
        sz[q][0] = 0.0;
#pragma unroll
        for (int z = 1; z < 2 * NCH; ++z) {
            cz[q][z] = cz[q][z - 1] * ez[q].x - sz[q][z - 1] * ez[q].y;
            sz[q][z] = cz[q][z - 1] * ez[q].y + sz[q][z - 1] * ez[q].x;
        }
        // e^{i x0 X} and the step e^{i KS X}
        cx[q] = kx[q] = 1.0;
        sx[q] = ky[q] = 0.0;
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            const double c2 = kx[q] * ex[q].x - ky[q] * ex[q].y;
            ky[q] = kx[q] * ex[q].y + ky[q] * ex[q].x;
            kx[q] = c2;
            if (i + 1 == x0) {
                cx[q] = kx[q];
                sx[q] = ky[q];
            }
        }
    }
    for (int nx = x0; nx <= nmax; nx += KS) {
        SmoothCoef p = wk + (size_t)12 * off[nx];
        double cur[12], nxt[12];
#pragma unroll
        for (int e = 0; e < 12; ++e) cur[e] = p[e];
        double cy[G], sy[G];
#pragma unroll
        for (int q = 0; q < G; ++q) {
            cy[q] = 1.0;
            sy[q] = 0.0;
        }
        int rem = n2max - nx * nx;   // of |n|^2 for n_z
        for (int ny = 0; rem >= 0; ++ny) {
            double a[G][6];
#pragma unroll
            for (int q = 0; q < G; ++q)
#pragma unroll
                for (int e = 0; e < 6; ++e) a[q][e] = 0.0;
#pragma unroll
            for (int k = 0; k < NCH; ++k) {
                if (rem < 4 * k * k) break;   // uniform
                p += 12;
                // as in smooth_images: this chunk's coefficients have arrived
                // before the next chunk's loads are issued
                __asm__ volatile("" : "+s"(p), "+s"(cur[0]), "+s"(cur[11]));
#pragma unroll
                for (int q = 0; q < G; ++q)
                    __asm__ volatile("" : "+s"(p), "+v"(a[q][0]), "+v"(a[q][5]));
#pragma unroll
                for (int e = 0; e < 12; ++e) nxt[e] = p[e];
#pragma unroll
                for (int z = 0; z < 2; ++z)
#pragma unroll
                    for (int e = 0; e < 6; ++e) {
                        if (k + z == 0 && (e == 2 || e == 4)) continue;   // sin 0
#pragma unroll
                        for (int q = 0; q < G; ++q)
                            a[q][e] = fma(cur[6 * z + e],
                                          e == 2 || e == 4 ? sz[q][2 * k + z] : cz[q][2 * k + z],
                                          a[q][e]);
                    }
#pragma unroll
                for (int e = 0; e < 12; ++e) cur[e] = nxt[e];
            }
#pragma unroll
            for (int q = 0; q < G; ++q) {
                const double cc = cx[q] * cy[q], ss = sx[q] * sy[q], sc = sx[q] * cy[q],
                             cs = cx[q] * sy[q];
                b[q][0] = fma(cc, a[q][0], b[q][0]);
                b[q][1] = fma(ss, a[q][1], b[q][1]);
                b[q][2] = fma(sc, a[q][2], b[q][2]);
                b[q][3] = fma(cc, a[q][3], b[q][3]);
                b[q][4] = fma(cs, a[q][4], b[q][4]);
                b[q][5] = fma(cc, a[q][5], b[q][5]);
                const double c2 = cy[q] * ey[q].x - sy[q] * ey[q].y;
                sy[q] = cy[q] * ey[q].y + sy[q] * ey[q].x;
                cy[q] = c2;
            }
            rem -= 2 * ny + 1;
        }
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const double c2 = cx[q] * kx[q] - sx[q] * ky[q];
            sx[q] = cx[q] * ky[q] + sx[q] * kx[q];
            cx[q] = c2;
        }
    }
}

// Workgroup: R = 4 G / KS rows of the tile (I, J), I <= J; lane = bead of J.  A
// row group of G rows belongs to KS waves, each with its share of the wave
// vectors (the first of them also takes the real-space terms), summed in LDS
// in a fixed order.  Off the diagonal the mirrored blocks (equal, every pair
// block being symmetric and even) go out as well, as runs of R columns.
// Bounded by its multiply-adds, 1834 per pair at |n|^2 <= 44 and 3714 at 77:
// 62 us at N = 1000 and 106 us there with the larger set (35 TFLOP/s).
template <int NP, int NF, int NZ, int G, int KS>
__global__ __launch_bounds__(256) void k_build_rows(int N, int nmax, int n2max, int ld,
                                                    const int2 *__restrict__ tile_ij,
                                                    const double *__restrict__ rt,
                                                    const double2 *__restrict__ etab, PairConst p,
                                                    const double *coef, const int *off,
                                                    const double *wk, double *__restrict__ drow)
{
    constexpr int R = 4 * G / KS, SPLIT = TB / R;
    constexpr int QN = 8 / KS * pair_queue<NF, G>(), SN = 4 * G * 6 * (TB + 1);
    __shared__ double sI[TS], sJ[TS];
    __shared__ double buf[QN > SN ? QN : SN];
    const int t = blockIdx.x / SPLIT, part = blockIdx.x % SPLIT;
    const int2 ij = tile_ij[t];
    const int I = ij.x, J = ij.y;
    if (I * TB + part * R >= N) return;
    const int nI = N - I * TB, nJ = N - J * TB;   // valid beads (may exceed TB)
    if (threadIdx.x < TS) {
        const int e = threadIdx.x;
        sI[e] = e / 3 < nI ? rt[3 * (size_t)I * TB + e] : 0.0;
        sJ[e] = e / 3 < nJ ? rt[3 * (size_t)J * TB + e] : 0.0;
    }
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = w / KS, ks = w % KS;   // row group, share of the wave vectors
    const int nm1 = nmax + 1, row0 = part * R + grp * G;
    // e^{i 2 pi s} of the lane's bead and the rows (entry 1 of the tables)
    const double2 *tj = etab + (size_t)min(J * TB + lane, N - 1) * 3 * nm1 + 1;
    const double2 jx = tj[0], jy = tj[nm1], jz = tj[2 * nm1];
    double2 ex[G], ey[G], ez[G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
        const double2 *ti = etab + (size_t)min(I * TB + row0 + q, N - 1) * 3 * nm1 + 1;
        const double2 ix = ti[0], iy = ti[nm1], iz = ti[2 * nm1];
        ex[q] = make_double2(ix.x * jx.x + ix.y * jx.y, ix.y * jx.x - ix.x * jx.y);
        ey[q] = make_double2(iy.x * jy.x + iy.y * jy.y, iy.y * jy.x - iy.x * jy.y);
        ez[q] = make_double2(iz.x * jz.x + iz.y * jz.y, iz.y * jz.x - iz.x * jz.y);
    }
    __syncthreads();
    double b[G][6];
#pragma unroll
    for (int q = 0; q < G; ++q)
#pragma unroll
        for (int e = 0; e < 6; ++e) b[q][e] = 0.0;
    if (ks == KS - 1) {   // the share with the fewest wave vectors
        double *qa = buf + 2 * grp * pair_queue<NF, G>(), *qb = qa + pair_queue<NF, G>();
        build_rows<TB, NP, NF, G>(p, smooth_ptr(coef), sI, sJ, nI, nJ, I == J, lane, row0, 1, qa,
                                  qb, [&](const int *, int, const double (*r)[6]) {
#pragma unroll
            for (int q = 0; q < G; ++q)
#pragma unroll
                for (int e = 0; e < 6; ++e) b[q][e] = r[q][e];
        });
    }
    recip_block<NZ, G, KS>(nmax, n2max, ks, (const __attribute__((address_space(4))) int *)off,
                           smooth_ptr(wk), ex, ey, ez, b);
    __syncthreads();   // every wave is done with its queue
    // buf[w][q][e][column]
#pragma unroll
    for (int q = 0; q < G; ++q)
#pragma unroll
        for (int e = 0; e < 6; ++e) buf[((w * G + q) * 6 + e) * (TB + 1) + lane] = b[q][e];
    __syncthreads();
    auto entry = [&](int r, int e, int c) {   // row r of the workgroup, column c
        if (part * R + r >= nI || c >= nJ) return 0.0;
        const double *o = buf + ((r / G * KS * G + r % G) * 6 + e) * (TB + 1) + c;
        double s = o[0];
#pragma unroll
        for (int k = 1; k < KS; ++k) s += o[k * G * 6 * (TB + 1)];
        return s;
    };
    for (int z = threadIdx.x; z < R * 6 * TB; z += 256) {
        const int c = z % TB, e = z / TB % 6, r = z / (6 * TB);
        if (part * R + r < nI)
            drow[((size_t)(I * TB + part * R + r) * 6 + e) * ld + J * TB + c] = entry(r, e, c);
    }
    if (I == J) return;
    for (int z = threadIdx.x; z < 6 * TB * R; z += 256) {
        const int r = z % R, c = z / R % TB, e = z / (R * TB);
        if (c < nJ)
            drow[((size_t)(J * TB + c) * 6 + e) * ld + I * TB + part * R + r] = entry(r, e, c);
    }
}

// The weight stream and offsets above (one chunk past the end, which the last
// chunk's prefetch reads); false where the form does not apply (no polynomial
// pair terms, or more than 9 values of n_z).
bool make_rows_weights(const Ctx &c, std::vector<int> &off, std::vector<double> &w)
{
    if (!c.smooth_np || c.nmax > 8) return false;
    off.clear();
    w.clear();
    const double vol = c.L * c.L * c.L, al2 = c.alpha * c.alpha;
    for (int x = 0; x <= c.nmax; ++x) {
        off.push_back((int)(w.size() / 12));
        for (int y = 0; x * x + y * y <= c.n2max; ++y)
            for (int z = 0; x * x + y * y + (z & ~1) * (z & ~1) <= c.n2max; ++z) {
                const int n2 = x * x + y * y + z * z;
                double o[6] = {};
                if (n2 > 0 && n2 <= c.n2max) {
                    const double n[3] = {(double)x, (double)y, (double)z};
                    const double k2 = 4.0 * M_PI * M_PI * n2 / (c.L * c.L);
                    const double mk = (c.a - c.a * c.a * c.a * k2 / 3.0) *
                                      (1.0 + k2 / (4.0 * al2) + k2 * k2 / (8.0 * al2 * al2)) *
                                      (6.0 * M_PI / (k2 * vol)) * exp(-k2 / (4.0 * al2));
                    const double m = mk * (x ? 2 : 1) * (y ? 2 : 1) * (z ? 2 : 1);
                    for (int a = 0, e = 0; a < 3; ++a)
                        for (int b = a; b < 3; ++b, ++e)
                            // off the diagonal -khat_a khat_b times -1 for the sines
                            o[e] = a == b ? m * (1.0 - n[a] * n[a] / n2) : m * n[a] * n[b] / n2;
                }
                w.insert(w.end(), o, o + 6);
            }
    }
    w.insert(w.end(), 12, 0.0);
    return true;
}

template <int NP, int NF, int NZ> static void build_rows_launch(const Ctx &c, hipStream_t s)
{
#define RPY_BR_KS(G, KS)                                                                       \
    hipLaunchKernelGGL((k_build_rows<NP, NF, NZ, G, KS>), dim3(c.ntiles * TB * KS / (4 * G)),  \
                       dim3(256), 0, s, c.N, c.nmax, c.n2max, c.row_ld, c.tile_ij, c.rt, c.etab, \
                       c.pc, c.smooth, c.row_off, c.row_wk, c.drow)
    if (c.N <= ROWS_KS_MAX) RPY_BR_KS(1, 4);
    else RPY_BR_KS(2, 2);
#undef RPY_BR_KS
}

void launch_build_rows(const Ctx &c, hipStream_t s)
{
    const bool single = c.pc.reach * c.pc.reach < 0.5 * c.L * c.L;   // as launch_build_tiles
#define RPY_BR(NP, NF)                                               \
    do {                                                             \
        if (rows_nz(c.nmax) == 7) build_rows_launch<NP, NF, 7>(c, s); \
        else build_rows_launch<NP, NF, 9>(c, s);                     \
    } while (0)
    if (c.smooth_np == SMOOTH_NP[0]) {
        if (single) RPY_BR(SMOOTH_NP[0], 3);
        else RPY_BR(SMOOTH_NP[0], 7);
    } else {
        if (single) RPY_BR(SMOOTH_NP[1], 3);
        else RPY_BR(SMOOTH_NP[1], 7);
    }
#undef RPY_BR
}

// ----------------------------------------------------------------- product
// y = D v and the epilogue of f.mode (as k_kspace_epi) for M vectors.
// Workgroup: ROW_BEADS bead rows, WPR waves each; wave h of a row takes the
// column blocks (128 columns: lane l the columns 2 l and 2 l + 1) ROW_U h ..
// ROW_U (h + 1) - 1, all of them loaded at once and before the vectors are
// staged in LDS, so that a product waits for memory once.  The lanes' sums
// are combined by a fixed xor tree that leaves component c in lane c, then the
// waves of a row in order.
// One vector, per product with its recurrence step: N = 100 3.8 us, 400 5.6,
// 1000 11.4 (48 MB), against 15.5, 15.9 and 24 us (at 618 wave vectors) in two launches by
// tiles.  As many vectors per launch as stage in the workgroup's LDS (24 ld bytes each, all
// four up to 1280 beads): with 64 KiB of it three vectors at N = 1000 take 26 instead of 17.8 us, four
// at N = 1280 47 instead of 35.
// flip: workgroups in reverse order (keeping blockIdx mod 8, the XCD), so that
// a product starts on the rows its XCD's L2 read last.
constexpr int ROW_U = 4;
constexpr int ROW_BEADS = 4;
typedef double row2 __attribute__((ext_vector_type(2)));

template <int M, int WPR>
__global__ __launch_bounds__(64 * ROW_BEADS * WPR) void k_row(int N, int n3, int ld, int j0,
                                                              int flip, const double *drow,
                                                              const double *__restrict__ v,
                                                              EpiArgs f,
                                                              const int *__restrict__ gate)
{
    extern __shared__ double sx[];   // [M][3 ld], zero past 3N
    __shared__ double part[WPR > 1 ? ROW_BEADS * (WPR - 1) * M * 4 : 1];
    __shared__ double tred[ROW_BEADS][2];
    if (gate && *gate) return;   // a product past the settled adaptive order
    constexpr int NT = 64 * ROW_BEADS * WPR;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r = w % ROW_BEADS, h = w / ROW_BEADS;
    int blk = blockIdx.x;
    if (flip) blk = 8 * ((gridDim.x - (blk & 7) + 7) / 8 - 1 - (blk >> 3)) + (blk & 7);
    const int i = blk * ROW_BEADS + r;
    const bool live = i < N;
    const double *row = drow + (size_t)min(i, N - 1) * 6 * ld + 2 * lane;
    const int b0 = ROW_U * h, nb = ld / 128;
    row2 d[ROW_U][6];
#pragma unroll
    for (int u = 0; u < ROW_U; ++u)
        if (b0 + u < nb) {
#pragma unroll
            for (int e = 0; e < 6; ++e)
                d[u][e] = *reinterpret_cast<const row2 *>(row + (size_t)e * ld + 128 * (b0 + u));
        }
    // the recurrence operands of the row's 3 entries (lanes 0 .. 2)
    const bool eth = live && h == 0 && lane < 3;
    double pv[M], pv2[M], pa[M];
#pragma unroll
    for (int j = 0; j < M; ++j) {
        const size_t o = (size_t)(j0 + j) * n3 + 3 * (size_t)i + lane;
        pv[j] = eth && f.mode != EPI_APPLY ? f.vprev[o] : 0.0;
        pv2[j] = eth && f.vprev2 && (f.mode == EPI_CHEB_NEXT || f.mode == EPI_ADJ) ? f.vprev2[o] : 0.0;
        pa[j] = eth && (f.mode == EPI_CHEB_NEXT || f.mode == EPI_ADJ) ? f.acc[o] : 0.0;
    }
    for (int z = threadIdx.x; z < M * 3 * ld; z += NT) {
        const int j = z / (3 * ld), q = z % (3 * ld);
        sx[z] = q < n3 ? v[(size_t)(j0 + j) * n3 + q] : 0.0;
    }
    __syncthreads();
    double yr[M];   // component `lane` of the row's product
#pragma unroll
    for (int j = 0; j < M; ++j) {
        double y0 = 0.0, y1 = 0.0, y2 = 0.0;
#pragma unroll
        for (int u = 0; u < ROW_U; ++u)
            if (b0 + u < nb) {
                const double *x = sx + (size_t)j * 3 * ld + 6 * (lane + 64 * (b0 + u));
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const double x0 = x[3 * q], x1 = x[3 * q + 1], x2 = x[3 * q + 2];
                    y0 += d[u][0][q] * x0 + d[u][1][q] * x1 + d[u][2][q] * x2;
                    y1 += d[u][1][q] * x0 + d[u][3][q] * x1 + d[u][4][q] * x2;
                    y2 += d[u][2][q] * x0 + d[u][4][q] * x1 + d[u][5][q] * x2;
                }
            }
        yr[j] = wave_sum3(y0, y1, y2, lane);
    }
    if constexpr (WPR > 1) {
        if (h > 0 && lane < 4)
#pragma unroll
            for (int j = 0; j < M; ++j) part[((r * (WPR - 1) + h - 1) * M + j) * 4 + lane] = yr[j];
        __syncthreads();
        if (h == 0 && lane < 4)
#pragma unroll
            for (int k = 0; k < WPR - 1; ++k)
#pragma unroll
                for (int j = 0; j < M; ++j) yr[j] += part[((r * (WPR - 1) + k) * M + j) * 4 + lane];
    }
    const double ya = f.scal ? f.scal[2] : 0.0, yb = f.scal ? f.scal[3] : 0.0;
    const bool trial = f.trial_n > 0 && (f.mode == EPI_CHEB_FIRST || f.mode == EPI_CHEB_NEXT) &&
                       !f.adapt->done && f.trial_n >= f.adapt->n_start;
    if (!trial && h > 0) return;
#pragma unroll
    for (int j = 0; j < M; ++j) {
        const size_t o = (size_t)(j0 + j) * n3 + 3 * (size_t)min(i, N - 1) + min(lane, 2);
        const double yy = yr[j];
        double vnew = 0.0;
        if (eth) {
            if (f.mode == EPI_APPLY) {
                f.vout[o] = yy;
            } else if (f.mode == EPI_CHEB_FIRST) {
                vnew = ya * yy - yb * pv[j];
                f.vout[o] = vnew;
                f.acc[o] = 0.5 * f.scal[8] * pv[j] + f.scal[9] * vnew;
                if (f.dv) f.dv[o] = yy;
            } else if (f.mode == EPI_CHEB_NEXT) {
                vnew = 2.0 * (ya * yy - yb * pv[j]) - pv2[j];
                f.vout[o] = vnew;
                f.acc[o] = pa[j] + f.scal[8 + f.p] * vnew;
            } else {
                vnew = f.scal[8 + f.p] * pa[j] + 2.0 * (ya * yy - yb * pv[j]) - pv2[j];
                f.vout[o] = vnew;
                f.dv[o] = f.xs * ya * vnew;
            }
        }
        if (trial) {   // uniform over the grid: the terms of dS over the lanes, V_p from its lanes
            if (h == 0) {
                const double v0 = __shfl(vnew, 0), v1 = __shfl(vnew, 1), v2 = __shfl(vnew, 2);
                const size_t ob = (size_t)(j0 + j) * n3 + 3 * (size_t)min(i, N - 1);
                const double *vh = f.vhist + ob;
                double t0 = 0.0, t1 = 0.0, t2 = 0.0;
                for (int q = lane; q < f.trial_n; q += 64) {
                    const double c = q ? f.scal[8 + q] : 0.5 * f.scal[8];
                    const double *t = vh + (size_t)q * f.ps;
                    t0 += c * (q == f.p ? v0 : t[0]);
                    t1 += c * (q == f.p ? v1 : t[1]);
                    t2 += c * (q == f.p ? v2 : t[2]);
                }
                const double t = wave_sum3(t0, t1, t2, lane);
                const double tt = eth ? t * t : 0.0, tb = eth ? vh[lane] * f.ddw[o] : 0.0;
                if (eth) f.ds[o] = t;
                const double ta = __shfl(tt, 0) + __shfl(tt, 1) + __shfl(tt, 2);
                const double tc = __shfl(tb, 0) + __shfl(tb, 1) + __shfl(tb, 2);
                if (lane == 0) {
                    tred[r][0] = ta;
                    tred[r][1] = tc;
                }
            }
            __syncthreads();
            if (threadIdx.x < 2) {
                double s = tred[0][threadIdx.x];
#pragma unroll
                for (int k = 1; k < ROW_BEADS; ++k) s += tred[k][threadIdx.x];
                f.tpart[((size_t)(j0 + j) * gridDim.x + blk) * 2 + threadIdx.x] = s;
            }
            __syncthreads();   // tred is rewritten by the next vector
        }
    }
}

int rows_trial_chunks(int N) { return (N + ROW_BEADS - 1) / ROW_BEADS; }

template <int M> static void row_launch(const Ctx &c, int j0, const double *v, const EpiArgs &f,
                                        hipStream_t s)
{
    const dim3 g((c.N + ROW_BEADS - 1) / ROW_BEADS);
    const size_t lds = (size_t)24 * c.row_ld * M;
    const int flip = (size_t)c.N * 6 * c.row_ld * sizeof(double) > ROWS_L2_BYTES
                         ? (int)(c.symv_calls++ & 1u) : 0;
#define RPY_ROW(WPR)                                                                              \
    hipLaunchKernelGGL((k_row<M, WPR>), g, dim3(64 * ROW_BEADS * WPR), lds, s, c.N, c.n3, c.row_ld, \
                       j0, flip, c.drow, v, f, c.gate)
    if (c.row_ld <= 128 * ROW_U) RPY_ROW(1);
    else if (c.row_ld <= 256 * ROW_U) RPY_ROW(2);
    else RPY_ROW(3);
#undef RPY_ROW
}

void launch_row_product(const Ctx &c, const double *v, const EpiArgs &f, hipStream_t s)
{
    static_assert(ROWS_MAX <= 3 * 128 * ROW_U, "a row is at most three waves");
    for (int j0 = 0; j0 < f.m;) {
        int mc = f.m - j0 < 4 ? f.m - j0 : 4;
        while (mc > 1 && (size_t)24 * c.row_ld * mc > (size_t)c.lds_max - 2048) --mc;   // static LDS below 2 KiB
        if (mc == 4) row_launch<4>(c, j0, v, f, s);
        else if (mc == 3) row_launch<3>(c, j0, v, f, s);
        else if (mc == 2) row_launch<2>(c, j0, v, f, s);
        else row_launch<1>(c, j0, v, f, s);
        j0 += mc;
    }
}

}  // namespace rpy
