// bsde_setup.hip -- gfx950 kernels of the least-squares set-up: the basis
// matrix B of the grid points (Section 3.2, the polynomial projection
// operator of eq. (3.1) restricted to the index set of Section 3.3) and the
// pieces of its pseudo-inverse B^+ = R^{-1} Q' by CholeskyQR2:
//
//   G1 = B'B,  R1 = chol(G1),  Q1 = B R1^{-1},
//   G2 = Q1'Q1, R2 = chol(G2),  B^+' = Q1 R2^{-1} R2^{-T} R1^{-T}.
//
// The Gram products, the tall-skinny products and the p x p steps run on the
// FP64 matrix cores (v_mfma_f64_16x16x4f64) over 16 x 16 tiles: the two
// Cholesky factorisations, the triangular inverses and the p x p products
// in one workgroup with the matrices in LDS when p <= kSmallFactorP
// (small_factor_kernel), else each in a kernel of its own (chol_kernel,
// tri_inv_kernel, prod_nt_kernel).  The whole set-up is stream-ordered.
//
// Matrices over the points are column-major with a leading dimension that
// is a multiple of 64 (each basis function's values over the points are
// contiguous); padding rows and columns hold zeros.
#include "bsde_common.h"

#include <hip/hip_runtime.h>

namespace bsde {

typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f64x4 mma64(double a, double b, f64x4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// B[c][i] = prod_v T_{nu_cv}(z_v(point i)) with z_0 = 2t/T - 1 and
// z_j = (x_j - mid_j) scale_j; zero for i >= n or c >= pa.  A workgroup takes
// 64 points and a range of columns: the Chebyshev values of its points go to
// LDS once (one division and eta FMAs per point and variate instead of per
// column), each column's factors with a positive degree to a packed list, and
// a column then costs one LDS read and multiplication per such factor.  Bound
// by the 8 bytes written per entry: at n = 81,920, p = 364 62 us (3.9 TB/s)
// against 829 us with the recurrences redone for every column.
constexpr int kBasisCols = 32; // columns of a workgroup
__global__ __launch_bounds__(256) void basis_matrix_kernel(
    const double *__restrict__ pts, int n, int ld, int dp,
    const int8_t *__restrict__ nu, int pa, int pap, int eta,
    const double *__restrict__ mid, const double *__restrict__ scale, double T,
    double *__restrict__ B)
{
    extern __shared__ double Tz[]; // [variate][degree][64 points]
    __shared__ unsigned long long factors[kBasisCols];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lane, c0 = blockIdx.y * kBasisCols;
    if (threadIdx.x < kBasisCols) {
        // the rows of Tz a column multiplies, a byte each (at most
        // min(eta, dp) <= 6 of them, rows below 11 x 9), 0xff past the last
        const int c = c0 + (int)threadIdx.x;
        unsigned long long f = ~0ull;
        if (c < pa)
            for (int w = dp - 1; w >= 0; --w) {
                const int a = nu[(size_t)c * dp + w];
                if (a) f = (f << 8) | (unsigned long long)(w * (eta + 1) + a);
            }
        factors[threadIdx.x] = f;
    }
    for (int w = wave; w < dp; w += 4) {
        double z = 0.0;
        if (i < n) {
            const double *row = pts + (size_t)i * dp;
            z = w == 0 ? 2.0 * row[0] / T - 1.0 : (row[w] - mid[w - 1]) * scale[w - 1];
        }
        double t0 = 1.0, t1 = z;
        double *out = Tz + (size_t)w * (eta + 1) * 64 + lane;
        out[64] = z;
        for (int k = 1; k < eta; ++k) {
            const double t2 = 2.0 * z * t1 - t0;
            t0 = t1;
            t1 = t2;
            out[(k + 1) * 64] = t1;
        }
    }
    __syncthreads();
    for (int c = c0 + wave; c < min(c0 + kBasisCols, pap); c += 4) {
        double v = i < n && c < pa ? 1.0 : 0.0;
        for (unsigned long long f = factors[c - c0]; (f & 0xff) != 0xff; f >>= 8)
            v *= Tz[(int)(f & 0xff) * 64 + lane];
        B[(size_t)c * ld + i] = i < n ? v : 0.0;
    }
}

// Partial Gram matrices: workgroup (pair, chunk) forms the 64 x 64 block
// (bi, bj), bi <= bj, of A'A over the rows of its chunk, a wave Q x Q tiles of
// 16 x 16 of it.  A chunk of 64 rows is one batch of loads, so that its time
// is their latency once and not four times (n = 1000, p = 221: 23 -> 9 us;
// n = 81,920, p = 364: 365 -> 266 us).  SINGLE: a wave is a workgroup of its own
// (blockIdx.z).
// The rows assigned to the four k-slots of an MFMA are permuted so that
// each lane reads 4 consecutive rows of one column (32 contiguous bytes,
// a whole 128-byte line per 4 lanes): in step t of a 16-row group at s,
// k-slot kk takes row s + 4 kk + t, the same for both operands.
// partial[chunk][r][c] holds the block's entries (r in bi's rows).
template <int Q, bool SINGLE = false>
__global__ __launch_bounds__(SINGLE ? 64 : 64 * (4 / Q) * (4 / Q)) void gram_partial_kernel(
    const double *__restrict__ A, int ld, int pap, int rows_per_chunk,
    const int2 *__restrict__ pairs, double *__restrict__ partial)
{
    const int2 pr = pairs[blockIdx.x];
    const int chunk = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = SINGLE ? blockIdx.z : threadIdx.x >> 6;
    // the wave's tiles of the block: Q x Q from (qa, qb)
    const int qa = 4 * pr.x + Q * (wave / (4 / Q)), qb = 4 * pr.y + Q * (wave % (4 / Q));
    const int r0 = chunk * rows_per_chunk;
    const int r1 = min(ld, r0 + rows_per_chunk);
    const int tiles = pap >> 4;
    int nti = 0, ntj = 0;
    const double *pa[Q], *pb[Q];
#pragma unroll
    for (int t = 0; t < Q; ++t) {
        const int ti = qa + t, tj = qb + t;
        nti += ti < tiles;
        ntj += tj < tiles;
        pa[t] = A + (size_t)(min(ti, tiles - 1) * 16 + (lane & 15)) * ld + 4 * (lane >> 4);
        pb[t] = A + (size_t)(min(tj, tiles - 1) * 16 + (lane & 15)) * ld + 4 * (lane >> 4);
    }
    f64x4 acc[Q][Q];
#pragma unroll
    for (int a = 0; a < Q; ++a)
#pragma unroll
        for (int b = 0; b < Q; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
    auto load = [&](const double *p, double *v) {
        const double2 x = *(const double2 *)p, y = *(const double2 *)(p + 2);
        v[0] = x.x; v[1] = x.y; v[2] = y.x; v[3] = y.y;
    };
    // (tiles beyond the last repeat it, and are not stored)
#pragma unroll 4
    for (int s = r0; s < r1; s += 16) {
        double va[Q][4], vb[Q][4];
#pragma unroll
        for (int t = 0; t < Q; ++t) {
            load(pa[t] + s, va[t]);
            load(pb[t] + s, vb[t]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int a = 0; a < Q; ++a)
#pragma unroll
                for (int b = 0; b < Q; ++b) acc[a][b] = mma64(va[a][k], vb[b][k], acc[a][b]);
    }
    double *out = partial + (size_t)chunk * pap * pap;
#pragma unroll
    for (int a = 0; a < Q; ++a)
#pragma unroll
        for (int b = 0; b < Q; ++b)
            if (a < nti && b < ntj) {
                const int col = (qb + b) * 16 + (lane & 15);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int row = (qa + a) * 16 + (lane >> 4) + 4 * v;
                    out[(size_t)row * pap + col] = acc[a][b][v];
                }
            }
}

// G[r][c] (pa x pa, row-major) = sum over chunks of the partial entry of
// the upper block holding (r, c) or (c, r): 256 / PARTS entries a workgroup,
// the chunks of each split over PARTS lanes whose sums are added in order
template <int PARTS>
__global__ __launch_bounds__(256) void gram_reduce_kernel(const double *__restrict__ partial,
                                                          int chunks, int pap, int pa,
                                                          double *__restrict__ G)
{
    constexpr int E = 256 / PARTS;
    __shared__ double sum[PARTS][E];
    const int e = threadIdx.x % E, part = threadIdx.x / E;
    const int idx = blockIdx.x * E + e;
    int r = idx / pa, c = idx % pa;
    if ((r >> 6) > (c >> 6)) {
        const int x = r;
        r = c;
        c = x;
    }
    double s = 0.0;
    if (idx < pa * pa)
        for (int k = part; k < chunks; k += PARTS)
            s += partial[((size_t)k * pap + r) * pap + c];
    if constexpr (PARTS > 1) {
        sum[part][e] = s;
        __syncthreads();
    }
    if (part == 0 && idx < pa * pa) {
        for (int q = 1; q < PARTS; ++q) s += sum[q][e];
        G[idx] = s;
    }
}

// Y = A X for A (ld x pap, column-major, rows >= n zero) and X (pap x pap,
// row-major; upper triangular when upper is set): one wave per block of
// 16 NR rows and 16 NC columns of Y', so that the A operand is X' (coalesced
// rows of X) and the B operand is A' (16 consecutive rows of A per k).  The
// operands of the next 4 KU steps of k are loaded before the products of the
// present ones.  Blocks of one row range follow each other on one XCD (the
// launch order goes round the eight), so that its rows of A are read from
// that XCD's L2 after the first.  Column c of the result goes to Y +
// colmap[c] * ldy (c < ncols) for rows < nrows.
template <int NC, int NR, int KU>
__global__ __launch_bounds__(64) void gemm_ax_kernel(
    const double *__restrict__ A, int ld, const double *__restrict__ X,
    int pap, int upper, double *__restrict__ Y, int ldy, int nrows,
    const int *__restrict__ colmap, int ncols, int nrb, int ncb,
    const int *__restrict__ skip)
{
    // a failed factorisation upstream (skip != 0) leaves Y untouched
    if (skip && *skip != 0) return;
    const int per = (int)gridDim.x / 8; // the grid is a multiple of 8
    const int id = (int)(blockIdx.x % 8) * per + (int)blockIdx.x / 8;
    if (id >= nrb * ncb) return;
    const int lane = threadIdx.x;
    const int i0 = (id / ncb) * 16 * NR;
    const int c0 = (id % ncb) * 16 * NC;
    const int ntc = min(NC, (pap - c0) >> 4), ntr = min(NR, (ld - i0) >> 4);
    const int kend = upper ? min(pap, c0 + 16 * NC) : pap; // multiples of 16
    f64x4 acc[NC][NR];
#pragma unroll
    for (int a = 0; a < NC; ++a)
#pragma unroll
        for (int b = 0; b < NR; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
    const double *xa = X + (size_t)(lane >> 4) * pap + c0 + (lane & 15);
    const double *ab = A + (size_t)(lane >> 4) * ld + i0 + (lane & 15);
    double va[KU][NC], vb[KU][NR], na[KU][NC], nb[KU][NR];
    auto fetch = [&](int k, double(&fa)[KU][NC], double(&fb)[KU][NR]) {
#pragma unroll
        for (int u = 0; u < KU; ++u) {
#pragma unroll
            for (int a = 0; a < NC; ++a)
                fa[u][a] = a < ntc ? xa[(size_t)(k + 4 * u) * pap + 16 * a] : 0.0;
#pragma unroll
            for (int b = 0; b < NR; ++b)
                fb[u][b] = b < ntr ? ab[(size_t)(k + 4 * u) * ld + 16 * b] : 0.0;
        }
    };
    fetch(0, va, vb);
    for (int k = 0; k < kend; k += 4 * KU) {
        if (k + 4 * KU < kend) fetch(k + 4 * KU, na, nb);
#pragma unroll
        for (int u = 0; u < KU; ++u)
#pragma unroll
            for (int a = 0; a < NC; ++a)
#pragma unroll
                for (int b = 0; b < NR; ++b)
                    if (a < ntc) acc[a][b] = mma64(va[u][a], vb[u][b], acc[a][b]);
#pragma unroll
        for (int u = 0; u < KU; ++u) {
#pragma unroll
            for (int a = 0; a < NC; ++a) va[u][a] = na[u][a];
#pragma unroll
            for (int b = 0; b < NR; ++b) vb[u][b] = nb[u][b];
        }
    }
#pragma unroll
    for (int a = 0; a < NC; ++a)
#pragma unroll
        for (int b = 0; b < NR; ++b) {
            const int i = i0 + 16 * b + (lane & 15);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int c = c0 + 16 * a + (lane >> 4) + 4 * v;
                if (a < ntc && c < ncols && i < nrows)
                    Y[(size_t)(colmap ? colmap[c] : c) * ldy + i] = acc[a][b][v];
            }
        }
}

// ---------------------------------------------------------------------------
// Factorisations over 16 x 16 tiles.  An accumulator tile of the matrix cores
// holds row (lane >> 4) + 4 v, column lane & 15 in element v, which is also
// the layout of the B operand of its four steps of k: a tile computed by one
// product feeds the next without moving.
// ---------------------------------------------------------------------------
// orders a wave's LDS accesses (they complete in issue order; the fences keep
// the compiler from moving them)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// the value of lane k (compile-time) of the wave
__device__ __forceinline__ double lane_value(double x, int k)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, k);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), k);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// acc + A B for the 16 x 16 tiles A at a (element (i, k) at a[i * rs + k * cs])
// and B = b in tile layout
__device__ __forceinline__ f64x4 tile_mul(const double *a, int rs, int cs, f64x4 b, f64x4 acc)
{
    const int i = threadIdx.x & 15, k = (threadIdx.x & 63) >> 4;
    double v[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = a[(size_t)i * rs + (size_t)(4 * s + k) * cs];
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = mma64(v[s], b[s], acc);
    return acc;
}
__device__ __forceinline__ f64x4 tile_load(const double *m, int ld)
{
    const int c = threadIdx.x & 15, r = (threadIdx.x & 63) >> 4;
    f64x4 t;
#pragma unroll
    for (int v = 0; v < 4; ++v) t[v] = m[(size_t)(r + 4 * v) * ld + c];
    return t;
}

// 1 / sqrt(x), x > 0: the hardware estimate y (relative error 2^-24) and the
// series of (1 - e)^{-1/2}, e = 1 - x y^2, to second order
__device__ __forceinline__ double rsqrt_pos(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// Upper Cholesky factor R of a 16 x 16 diagonal tile and R^{-1}, by one wave.
// d: the tile (row stride 17), replaced by R; di: the inverse.  Lane c < 16
// holds column c of the tile, lane 16 + c column c of the identity (the upper
// half of the wave repeats them): the row operations that turn the tile into
// R turn the identity into R^{-T}.  live: rows before the padding.  False
// when a live pivot is not positive or its square root not above floor.
__device__ __forceinline__ bool chol_tile(double (*d)[17], double (*di)[17], int live,
                                          double floor)
{
    const int c = threadIdx.x & 15;
    const bool unit = threadIdx.x & 16;
    double a[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const double v = d[r][c];
        a[r] = unit ? (r == c ? 1.0 : 0.0) : v;
    }
    bool ok = true;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const double piv = lane_value(a[j], j);
        if (j < live && (!(piv > 0.0) || !(sqrt(piv) > floor))) ok = false;
        a[j] *= rsqrt_pos(piv);
#pragma unroll
        for (int r = j + 1; r < 16; ++r)
            a[r] = fma(-lane_value(a[j], r), a[j], a[r]); // of a tile's column, kept for r <= c
    }
    wave_sync();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        if (unit) di[c][r] = a[r]; // (zero below the diagonal as computed)
        else d[r][c] = c >= r ? a[r] : 0.0;
    }
    wave_sync();
    return ok;
}

// R'R = G (pa x pa, row-major; padded to nt tiles with the identity) by one
// workgroup of NW waves, row block after row block: the tiles of a row block
// are G minus the products of the finished rows above, one wave a tile (TW
// tiles a wave), the first wave factors the diagonal tile, and the others
// are multiplied by its inverse's transpose.  R (row stride ldr) gets the
// tiles on and above the diagonal, dinv the inverses of the diagonal tiles
// (16 x 16 each).  The rank test is on every pivot: positive, and its square
// root above rel_tol times that of the largest diagonal entry of G; false
// when one fails.
template <int NW, int TW>
__device__ __forceinline__ bool chol_blocks(const double *G, int pa, int nt, double rel_tol, double *R,
                            int ldr, double *dinv)
{
    __shared__ double d[16][17], di[16][17];
    __shared__ double dmax[NW];
    __shared__ int bad;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 15, r = lane >> 4;
    double m = 0.0;
    for (int j = threadIdx.x; j < pa; j += NW * 64) m = fmax(m, G[(size_t)j * pa + j]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
    if (lane == 0) dmax[wave] = m;
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
    for (int w = 0; w < NW; ++w) m = fmax(m, dmax[w]);
    const double floor = rel_tol * sqrt(m);
    for (int b = 0; b < nt; ++b) {
        f64x4 s[TW];
#pragma unroll
        for (int q = 0; q < TW; ++q) {
            const int t = b + wave + q * NW;
            if (t >= nt) continue;
            f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll (TW > 4 ? 2 : 4)
            for (int k = 0; k < b; ++k) {
                const double *row = R + (size_t)16 * k * ldr;
                acc = tile_mul(row + 16 * b, 1, ldr, tile_load(row + 16 * t, ldr), acc);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gr = 16 * b + r + 4 * v, gc = 16 * t + c;
                const double g = gr < pa && gc < pa ? G[(size_t)gr * pa + gc]
                                                    : (gr == gc ? 1.0 : 0.0);
                s[q][v] = g - acc[v];
            }
        }
        if (wave == 0) {
#pragma unroll
            for (int v = 0; v < 4; ++v) d[r + 4 * v][c] = s[0][v];
            wave_sync();
            const bool ok = chol_tile(d, di, pa - 16 * b, floor);
            if (!ok && lane == 0) bad = 1;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                R[(size_t)(16 * b + r + 4 * v) * ldr + 16 * b + c] = d[r + 4 * v][c];
                dinv[(size_t)b * 256 + (r + 4 * v) * 16 + c] = di[r + 4 * v][c];
            }
        }
        __syncthreads();
        if (bad) return false;
#pragma unroll
        for (int q = 0; q < TW; ++q) {
            const int t = b + wave + q * NW;
            if (t >= nt || t == b) continue;
            const f64x4 o = tile_mul(&di[0][0], 1, 17, s[q], f64x4{0.0, 0.0, 0.0, 0.0});
#pragma unroll
            for (int v = 0; v < 4; ++v)
                R[(size_t)(16 * b + r + 4 * v) * ldr + 16 * t + c] = o[v];
        }
        __syncthreads();
    }
    return true;
}

// One wave: column block j of X = R^{-1} (row stride ldx), tile after tile
// from the diagonal up: X_ij = -R_ii^{-1} sum_{i < k <= j} R_ik X_kj
__device__ __forceinline__ void tri_inv_column(const double *R, int ldr, const double *dinv, int j, double *X,
                               int ldx)
{
    const int lane = threadIdx.x & 63;
    const int c = lane & 15, r = lane >> 4;
    auto put = [&](int i, f64x4 t) {
#pragma unroll
        for (int v = 0; v < 4; ++v) X[(size_t)(16 * i + r + 4 * v) * ldx + 16 * j + c] = t[v];
        wave_sync();
    };
    put(j, tile_load(dinv + (size_t)j * 256, 16));
    for (int i = j - 1; i >= 0; --i) {
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int k = i + 1; k <= j; ++k)
            acc = tile_mul(R + (size_t)16 * i * ldr + 16 * k, ldr, 1,
                           tile_load(X + (size_t)16 * k * ldx + 16 * j, ldx), acc);
        const f64x4 o = tile_mul(dinv + (size_t)i * 256, 16, 1, acc,
                                 f64x4{0.0, 0.0, 0.0, 0.0});
        put(i, f64x4{-o[0], -o[1], -o[2], -o[3]});
    }
}

// C tile (bi, bj) = sum over k0 <= k < nt of A_bi,k (B_bj,k)' (row strides lda,
// ldb; both upper triangular or zero-padded as k0 allows)
__device__ __forceinline__ f64x4 prod_nt_tile(const double *A, int lda, const double *B, int ldb,
                                              int bi, int bj, int k0, int nt)
{
    const int c = threadIdx.x & 15, r = (threadIdx.x & 63) >> 4;
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int k = k0; k < nt; ++k) {
        f64x4 b; // B' tile: element (kk, col) = B[col][kk]
#pragma unroll
        for (int s = 0; s < 4; ++s) b[s] = B[(size_t)(16 * bj + c) * ldb + 16 * k + 4 * s + r];
        acc = tile_mul(A + (size_t)16 * bi * lda + 16 * k, lda, 1, b, acc);
    }
    return acc;
}

// Small bases (nt = pap / 16 <= 4 tiles), one workgroup of four waves with the
// matrices in LDS.  Stage 1 (R1 from G1): X1 = R1^{-1} (pap x pap, zero in
// the padding), the right factor of Q1 = B X1.  Stage 2 (R2 from G2): Xp = P'
// with P = R2^{-1} R2^{-T} R1^{-T}, the right factor of B^+' = Q1 P.  status:
// 0, or the stage whose rank test failed (stage 2 does nothing when stage 1
// failed).  Latency-bound (16 dependent pivots a tile): 8 us at p = 15, 31 us
// at p = 56; one wave over scalar LDS elements took 21 and 325 us.
__global__ __launch_bounds__(256) void small_factor_kernel(
    const double *__restrict__ G, int pa, int pap, double rel_tol, int stage,
    double *__restrict__ X1, double *__restrict__ Xp, int *__restrict__ status)
{
    constexpr int L = kSmallFactorP + 1;
    __shared__ double R[kSmallFactorP * L], Y[kSmallFactorP * L], dinv[4 * 256];
    const int nt = pap >> 4, wave = threadIdx.x >> 6;
    const int c = threadIdx.x & 15, r = (threadIdx.x & 63) >> 4;
    if (stage == 2 && *status != 0) return;
    if (!chol_blocks<4, 1>(G, pa, nt, rel_tol, R, L, dinv)) {
        if (threadIdx.x == 0) *status = stage;
        return;
    }
    for (int e = threadIdx.x; e < kSmallFactorP * L; e += 256) Y[e] = 0.0;
    __syncthreads();
    if (wave < nt) tri_inv_column(R, L, dinv, wave, Y, L);
    __syncthreads();
    if (stage == 1) {
        for (int e = threadIdx.x; e < pap * pap; e += 256) {
            const int row = e / pap, col = e % pap;
            X1[e] = row < pa && col < pa ? Y[row * L + col] : 0.0;
        }
        if (threadIdx.x == 0) *status = 0;
        return;
    }
    for (int t = wave; t < nt * nt; t += 4) { // T2 = Y Y' over R
        const int bi = t / nt, bj = t % nt;
        const f64x4 v = prod_nt_tile(Y, L, Y, L, bi, bj, max(bi, bj), nt);
#pragma unroll
        for (int q = 0; q < 4; ++q) R[(16 * bi + r + 4 * q) * L + 16 * bj + c] = v[q];
    }
    __syncthreads();
    for (int t = wave; t < nt * nt; t += 4) { // Xp = T2 X1'
        const int bi = t / nt, bj = t % nt;
        const f64x4 v = prod_nt_tile(R, L, X1, pap, bi, bj, bj, nt);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = 16 * bi + r + 4 * q, col = 16 * bj + c;
            Xp[(size_t)row * pap + col] = row < pa && col < pa ? v[q] : 0.0;
        }
    }
    if (threadIdx.x == 0) *status = 0;
}

// The factorisation of a larger basis: one workgroup of eight waves, R (pap x
// pap) in global memory (it stays in the L2).  A chain of pap / 16 row
// blocks, two thirds of it the dependent pivots of the diagonal tiles (350
// cycles each): 103 us at p = 221, 275 us at p = 364, 119 and 299 us with a
// quotient and a root in that chain and the inverse after it (on the host,
// with the copies: 1.3 ms at p = 221, 5 ms at p = 364).  With the tiles in
// registers and the rows in LDS it takes as long: 107 us.
template <int NW>
__device__ __forceinline__ void chol_workgroup(const double *G, int pa, int pap, double rel_tol,
                                               int stage, double *R, double *dinv, int *status)
{
    if (stage == 2 && *status != 0) return;
    const bool ok = chol_blocks<NW, (kFactorTiles + NW - 1) / NW>(G, pa, pap >> 4, rel_tol, R, pap,
                                                                  dinv);
    if (threadIdx.x == 0) *status = ok ? 0 : stage;
}
__global__ __launch_bounds__(512) void chol_kernel(const double *__restrict__ G, int pa, int pap,
                                                   double rel_tol, int stage, double *R,
                                                   double *dinv, int *__restrict__ status)
{
    chol_workgroup<8>(G, pa, pap, rel_tol, stage, R, dinv, status);
}
// Beside a path kernel that fills the GPU: four waves of at most 168 registers.
// A workgroup that needs more of a compute unit than one of the path kernel's
// leaves when it ends would wait for the last of them.
__global__ __launch_bounds__(256, 3) void chol_beside_kernel(
    const double *__restrict__ G, int pa, int pap, double rel_tol, int stage, double *R,
    double *dinv, int *__restrict__ status)
{
    chol_workgroup<4>(G, pa, pap, rel_tol, stage, R, dinv, status);
}

// X = R^{-1} (pap x pap, zero below the diagonal and in the padding): a
// workgroup per column block, the products of a tile split over its four
// waves and added in order, the column block in LDS in tile layout
__global__ __launch_bounds__(256) void tri_inv_kernel(const double *__restrict__ R, int pa,
                                                      int pap, const double *__restrict__ dinv,
                                                      double *__restrict__ X,
                                                      const int *__restrict__ status)
{
    extern __shared__ double xs[]; // [tile][v][lane], then four tiles of sums
    if (*status != 0) return;
    const int j = blockIdx.x, nt = pap >> 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 15, r = lane >> 4;
    double *red = xs + (size_t)nt * 256;
    auto tile = [&](const double *base) {
        return f64x4{base[lane], base[64 + lane], base[128 + lane], base[192 + lane]};
    };
    auto put = [&](double *base, f64x4 t) {
#pragma unroll
        for (int v = 0; v < 4; ++v) base[64 * v + lane] = t[v];
    };
    if (wave == 0) put(xs + (size_t)j * 256, tile_load(dinv + (size_t)j * 256, 16));
    __syncthreads();
    for (int i = j - 1; i >= 0; --i) {
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int k = i + 1 + wave; k <= j; k += 4)
            acc = tile_mul(R + (size_t)16 * i * pap + 16 * k, pap, 1, tile(xs + (size_t)k * 256),
                           acc);
        put(red + wave * 256, acc);
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int w = 1; w < 4; ++w) {
                const f64x4 t = tile(red + w * 256);
                acc = f64x4{acc[0] + t[0], acc[1] + t[1], acc[2] + t[2], acc[3] + t[3]};
            }
            const f64x4 o = tile_mul(dinv + (size_t)i * 256, 16, 1, acc,
                                     f64x4{0.0, 0.0, 0.0, 0.0});
            put(xs + (size_t)i * 256, f64x4{-o[0], -o[1], -o[2], -o[3]});
        }
        __syncthreads();
    }
    for (int k = wave; k < nt; k += 4) {
        const f64x4 t = k <= j ? tile(xs + (size_t)k * 256) : f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 16 * k + r + 4 * v, col = 16 * j + c;
            X[(size_t)row * pap + col] = row < pa && col < pa ? t[v] : 0.0;
        }
    }
}

// C = A B' (pap x pap each, B upper triangular, A too when both is set): a
// wave per 16 x 16 tile
__global__ __launch_bounds__(64) void prod_nt_kernel(const double *__restrict__ A,
                                                     const double *__restrict__ B, int pap,
                                                     int both, double *__restrict__ C,
                                                     const int *__restrict__ status)
{
    if (*status != 0) return;
    const int bi = blockIdx.x, bj = blockIdx.y;
    const f64x4 v = prod_nt_tile(A, pap, B, pap, bi, bj, both ? max(bi, bj) : bj, pap >> 4);
    const int c = threadIdx.x & 15, r = threadIdx.x >> 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) C[(size_t)(16 * bi + r + 4 * q) * pap + 16 * bj + c] = v[q];
}

// Doubles of workspace launch_factor needs
size_t factor_workspace(int pap)
{
    if (pap <= kSmallFactorP) return 0;
    // R, the second stage's R2^{-1} and R2^{-1} R2^{-T}, the diagonal inverses
    return 3 * (size_t)pap * pap + (size_t)(pap >> 4) * 256;
}

// One stage of the factorisation from the Gram matrix G (pa x pa): stage 1
// writes X1 = R1^{-1}, stage 2 Xp = P' (both pap x pap).  beside: other kernels
// fill the GPU meanwhile
hipError_t launch_factor(const double *G, int pa, int pap, double rel_tol, int stage,
                         double *X1, double *Xp, double *work, int *status, bool beside,
                         hipStream_t s)
{
    const int nt = pap >> 4;
    if (pa < 1 || pap != pad16(pa) || nt > kFactorTiles || (stage != 1 && stage != 2))
        return hipErrorInvalidValue;
    if (pap <= kSmallFactorP) {
        small_factor_kernel<<<1, 256, 0, s>>>(G, pa, pap, rel_tol, stage, X1, Xp, status);
        return hipGetLastError();
    }
    const size_t sq = (size_t)pap * pap;
    double *R = work, *Y = work + sq, *T2 = work + 2 * sq, *dinv = work + 3 * sq;
    if (beside)
        chol_beside_kernel<<<1, 256, 0, s>>>(G, pa, pap, rel_tol, stage, R, dinv, status);
    else
        chol_kernel<<<1, 512, 0, s>>>(G, pa, pap, rel_tol, stage, R, dinv, status);
    tri_inv_kernel<<<nt, 256, (nt + 4) * 256 * sizeof(double), s>>>(R, pa, pap, dinv,
                                                                  stage == 1 ? X1 : Y, status);
    if (stage == 2) {
        prod_nt_kernel<<<dim3(nt, nt), 64, 0, s>>>(Y, Y, pap, 1, T2, status);
        prod_nt_kernel<<<dim3(nt, nt), 64, 0, s>>>(T2, X1, pap, 0, Xp, status);
    }
    return hipGetLastError();
}

hipError_t launch_basis_matrix(const double *pts, int n, int ld, int dp,
                               const int8_t *nu, int pa, int pap, int eta,
                               const double *mid, const double *scale,
                               double T, double *B, hipStream_t s)
{
    // the packed factor lists hold seven row indices below 255
    if (eta < 1 || (eta < dp ? eta : dp) > 7 || dp * (eta + 1) > 255) return hipErrorInvalidValue;
    dim3 grid(ld / 64, (pap + kBasisCols - 1) / kBasisCols);
    basis_matrix_kernel<<<grid, 256, sizeof(double) * dp * (eta + 1) * 64, s>>>(
        pts, n, ld, dp, nu, pa, pap, eta, mid, scale, T, B);
    return hipGetLastError();
}

hipError_t launch_gram(const double *A, int ld, int pap, int rows_per_chunk,
                       int chunks, const int2 *pairs, int npairs,
                       double *partial, int pa, double *G, bool beside, hipStream_t s)
{
    // Beside a path kernel, single waves of one tile (42 registers) find room
    // in what its waves leave free; workgroups of four waves of 120 waited for
    // its end (d = 5, p = 84: 67 us an iteration against 1550).
    // Otherwise one wave a block reads the least (n = 81,920, p = 364: 266 us against
    // 407 with four); where that leaves SIMDs idle (1024 of them), four waves
    // share it (n = 1000, p = 221: 9 us against 14; n = 10,933, p = 56: 8
    // against 14)
    if (beside)
        gram_partial_kernel<1, true><<<dim3(npairs, chunks, 16), 64, 0, s>>>(
            A, ld, pap, rows_per_chunk, pairs, partial);
    else if (npairs * chunks < 1024)
        gram_partial_kernel<2><<<dim3(npairs, chunks), 256, 0, s>>>(A, ld, pap, rows_per_chunk,
                                                                  pairs, partial);
    else
        gram_partial_kernel<4><<<dim3(npairs, chunks), 64, 0, s>>>(A, ld, pap, rows_per_chunk,
                                                                 pairs, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // eight lanes an entry where one would leave the chip idle (p = 56, 171
    // chunks: 48 -> 7 us); p = 364 has 132,496 entries, and one lane each
    // reads whole lines (66 us against 84)
    if (pa * pa < 65536)
        gram_reduce_kernel<8><<<(pa * pa + 31) / 32, 256, 0, s>>>(partial, chunks, pap, pa, G);
    else
        gram_reduce_kernel<1><<<(pa * pa + 255) / 256, 256, 0, s>>>(partial, chunks, pap, pa, G);
    return hipGetLastError();
}

// Y = A X (gemm_ax_kernel).  Blocks of 32 x 32 read each operand half as
// often as 16 x 16 ones and leave the registers for several waves a SIMD;
// they are taken when there are two for each of the 1024 SIMDs (n = 81,920,
// p = 364, whole / triangular X: 471 / 323 us against 683 / 407; n = 40,960,
// p = 84: 27 / 23 us against 32 / 25).  With fewer most of the chip would
// wait for one wave's chain of k steps (n = 16,384, p = 56: 13 us against 11;
// n = 1000, p = 221: 19 us against 11).  64 x 64 blocks take 790 and 93 us at
// the first and last of these sizes.
hipError_t launch_gemm_ax(const double *A, int ld, const double *X, int pap, bool upper,
                          double *Y, int ldy, int nrows, const int *colmap,
                          int ncols, hipStream_t s, const int *skip)
{
    auto launch = [&](auto nc, auto ku) {
        constexpr int B = decltype(nc)::value;
        const int cb = (pap + 16 * B - 1) / (16 * B), rb = (ld + 16 * B - 1) / (16 * B);
        gemm_ax_kernel<B, B, decltype(ku)::value>
            <<<dim3((unsigned)((cb * rb + 7) / 8 * 8)), 64, 0, s>>>(
                A, ld, X, pap, upper ? 1 : 0, Y, ldy, nrows, colmap, ncols, rb, cb, skip);
        return hipGetLastError();
    };
    if (((pap + 31) / 32) * (ld / 32) >= 2048)
        return launch(std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{});
    return launch(std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{});
}

} // namespace bsde
