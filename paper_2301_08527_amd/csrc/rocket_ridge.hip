// ROCKET transform library for MI355X (gfx950): ridge regressor on the pooled features
// (paper section 3 part (3), section 3.3).  See include/rocket.h for the contract.
//
// Model: minimise ||y - X w - b||^2 + alpha ||w||^2 with an unpenalised intercept.  With
// n examples and p >> n features the fit works in the n x n dual system
//     a = (Xc Xc^T + alpha I)^-1 yc,   w = Xc^T a,   b = mean(y) - mean(X) . w
// (Xc, yc centred).  Everything is fp64 on fp32 features, and every sum has a fixed order
// (no atomics), so a fit is reproducible bit for bit.  Kernels, in launch order:
//   rr_col_sums, rr_means       column means of X and the mean target (rows split over the grid)
//   rr_gram                     partial 64 x 64 tiles of Xc Xc^T on the fp64 matrix cores
//                               (v_mfma_f64_16x16x4f64), one wavefront per (tile pair, slice of
//                               the p features); operands go from global memory straight into
//                               the MFMA operand registers, centred on the way
//   rr_gram_finish              sums the slices, adds alpha on the diagonal, writes the lower
//                               triangle of the (n+1) x (n+1) system whose last row is yc
//   per 32 columns: rr_step     Cholesky of the 32 x 32 diagonal block and the rows below it solved against
//                               that block, 16 columns at a time in each wavefront's registers (the second
//                               half updated by the first through LDS and the MFMA units), then the rank-32
//                               update of what is left, 32 x 32 tiles on the MFMA units (rr_panel and
//                               rr_trailing where much is left).  The row of yc takes part like any
//                               other row, so when the factorisation ends it holds L^-1 yc (forward
//                               substitution costs nothing extra).
//   rr_back_substitute          L^T a = L^-1 yc, panel by panel, one workgroup, with the inverses of the diagonal
//                               blocks that a workgroup of the next panel's launch makes (rr_invert_block)
//   rr_coef_partial, rr_coef_finish, rr_intercept     w = Xc^T a and b
//   rr_predict                  yhat = X w + b, one workgroup per row
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <type_traits>
#include <utility>

#include "rocket_internal.hpp"

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d4u __attribute__((ext_vector_type(4), aligned(8)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // rows of X start at any multiple of 4 bytes

constexpr int kGramTile = 64;       // rows of one Gram tile (4 x 4 MFMA tiles per wavefront)
constexpr int kNB = 32;             // panel width of the factorisation
constexpr int kMaxExamples = 32768; // (n+1)^2 doubles of workspace: 8.6 GB at this size
constexpr int kGramWaves = 2048;    // wavefronts the Gram kernel aims for (256 CUs x 4 SIMDs x 2)
constexpr int kMaxRowSplits = 16;
// Rows of X whose loads a lane of the column sums and of the coefficients has on their way together (added in order, so the
// sums are the same bits): one column is a chain of trips to memory otherwise.  677 x 20,000: rr_col_sums 18.2 -> 10.5 us
// (54 MB), rr_coef_partial 16.2 -> 11.0, and the sums of their splits, loaded together too, 5.5 -> 3.6 and 6.1 -> 4.7.
// Slices of fewer rows load their last row again: whole fits of 8 x 3,000 43.3 -> 42.8 us, of 2 x 500 35.8 -> 36.3, of
// 1 x 200,000 480 -> 483.
constexpr int kRowsInFlight = 16;
#ifndef RK_FUSED_TILES
#define RK_FUSED_TILES 48
#endif
// 32-row tiles left up to which a panel and its update are one launch.  Beyond it the factoring that every tile repeats costs
// more than the second launch.  Whole fits with 64 features in us, by the number of tiles at which the line lies (0: always
// two launches; 2,000: always one):
//      n       0      32      40      48      64    2,000
//    500     301     193     193     193     193     193
//  1,000     656     455     455     455     455     455
//  1,500   1,189     982     945     922     922     922
//  2,000   1,920   1,724   1,690   1,666   1,663   1,666
//  2,500   2,746   2,535   2,494   2,474   2,479   2,561
//  3,000   4,077   3,869   3,830   3,806   3,818   4,042
//  3,500   5,205   5,002   4,967   4,944   4,972   5,538
constexpr int kFusedTiles = RK_FUSED_TILES;
constexpr int kWideRow = 2048;      // features from which a prediction's row takes 1,024 lanes

// D = A B + C on one wavefront: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16] and holds
// D[4 v + l / 16][l % 16] in element v of the result.
__device__ __forceinline__ d4 rr_mfma(double a, double b, d4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

__device__ __forceinline__ double rr_lane(double v, int lane)   // v of a given lane, to all lanes (lane: wave-uniform)
{
    const long long bits = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane(static_cast<int>(bits), lane);
    const int hi = __builtin_amdgcn_readlane(static_cast<int>(bits >> 32), lane);
    return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}

// part[r][j] = sum of X[i][j] over the rows i of slice r, j < p; column p is the target vector
__global__ __launch_bounds__(256) void rr_col_sums(const float *__restrict__ X, const float *__restrict__ y, int n,
                                                   int p, int rows_per, double *__restrict__ part)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j > p) return;
    const int i0 = blockIdx.y * rows_per, i1 = min(n, i0 + rows_per);
    const float *src = j < p ? X + j : y;
    const size_t pitch = j < p ? p : 1;
    double s = 0.0;
    for (int i = i0; i < i1; i += kRowsInFlight) {
        float v[kRowsInFlight];
#pragma unroll
        for (int e = 0; e < kRowsInFlight; ++e) v[e] = src[min(i + e, i1 - 1) * pitch];
#pragma unroll
        for (int e = 0; e < kRowsInFlight; ++e) s += i + e < i1 ? static_cast<double>(v[e]) : 0.0;
    }
    part[static_cast<size_t>(blockIdx.y) * (p + 1) + j] = s;
}

// means[j] = mean_i X[i][j] for j < p; means[p] = mean_i y[i]
__global__ __launch_bounds__(256) void rr_means(const double *__restrict__ part, int splits, int n, int p,
                                                double *__restrict__ means)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j > p) return;
    double s = 0.0;
    double v[kMaxRowSplits];
#pragma unroll
    for (int r = 0; r < kMaxRowSplits; ++r) v[r] = part[static_cast<size_t>(min(r, splits - 1)) * (p + 1) + j];
#pragma unroll
    for (int r = 0; r < kMaxRowSplits; ++r) s += r < splits ? v[r] : 0.0;
    means[j] = s / static_cast<double>(n);
}

// One wavefront per (pair of 64-row tiles ti <= tj, slice of the features).  Work items are dealt
// so that one XCD (workgroup ids go round the eight of them) takes all tile pairs of a slice one
// after the other: the slab of X for that slice then stays in that XCD's L2.  The order of the
// features inside a step of 16 is permuted (lane q = l / 16 takes features 4q..4q+3 as one
// 16-byte load); a sum does not care, and both operands use the same permutation.  Of a pair of equal tiles only the blocks on
// and above the diagonal are computed, and the loads of a step are on their way while the last quarter of the step before is
// multiplied (1,024 clk of the matrix unit): 677 x 20,000 whole fits 452 -> 439 us, 70 x 30,000 136 -> 127.  What bounds it is
// the matrix unit with the conversions, which do not run beside it (f64 both): together 160 of the launch's 200 us.
template <bool DIAG>
__device__ __forceinline__ void rr_gram_pair(const float *__restrict__ X, const double *__restrict__ means, int n, int p, int ti, int tj,
                                             int kbeg, int kend, double *__restrict__ dst)
{
    const int l = threadIdx.x, r = l & 15, q = l >> 4;

    const float *pa[4], *pb[4];   // rows past n repeat row n - 1: their results are never stored
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        pa[a] = X + static_cast<size_t>(min(ti * kGramTile + 16 * a + r, n - 1)) * p;
        pb[a] = X + static_cast<size_t>(min(tj * kGramTile + 16 * a + r, n - 1)) * p;
    }
    d4 acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};

    f4u xa[4], xb[4];
    d4 mu;
    auto load = [&](int k0) {
        const int k = k0 + 4 * q;
        if (k0 + 16 <= kend) {
#pragma unroll
            for (int a = 0; a < 4; ++a) xa[a] = *reinterpret_cast<const f4u *>(pa[a] + k);
            if (!DIAG) {
#pragma unroll
                for (int a = 0; a < 4; ++a) xb[a] = *reinterpret_cast<const f4u *>(pb[a] + k);
            }
            mu = *reinterpret_cast<const d4 *>(means + k);
        } else {   // ragged end of the features: absent ones enter as 0 - 0
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool ok = k + e < kend;
                mu[e] = ok ? means[k + e] : 0.0;
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    xa[a][e] = ok ? pa[a][k + e] : 0.0f;
                    if (!DIAG) xb[a][e] = ok ? pb[a][k + e] : 0.0f;
                }
            }
        }
    };
    load(kbeg);
    for (int k0 = kbeg; k0 < kend; k0 += 16) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double am[4], bm[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) am[a] = static_cast<double>(xa[a][e]) - mu[e];
#pragma unroll
            for (int a = 0; a < 4; ++a) bm[a] = DIAG ? am[a] : static_cast<double>(xb[a][e]) - mu[e];
            if (e == 3) {       // the step's features have all been converted: the next ones come while the last are multiplied
                __builtin_amdgcn_sched_barrier(0);
                if (k0 + 16 < kend) load(k0 + 16);      // uniform
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = DIAG ? a : 0; b < 4; ++b) acc[a][b] = rr_mfma(am[a], bm[b], acc[a][b]);
        }
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = DIAG ? a : 0; b < 4; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) dst[(16 * a + 4 * v + q) * kGramTile + 16 * b + r] = acc[a][b][v];
}

__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void rr_gram(const float *__restrict__ X, const double *__restrict__ means, int n, int p, int tiles, int pairs, int chunk, int splits,
             double *__restrict__ part)
{
    const int total = pairs * splits, per = (total + 7) / 8;
    const int w = (blockIdx.x % 8) * per + blockIdx.x / 8;
    if (blockIdx.x / 8 >= per || w >= total) return;
    const int split = w / pairs, pair = w % pairs;
    int ti = 0, rem = pair;
    while (rem >= tiles - ti) { rem -= tiles - ti; ++ti; }
    const int tj = ti + rem, kbeg = split * chunk, kend = min(p, kbeg + chunk);
    double *dst = part + (static_cast<size_t>(pair) * splits + split) * (kGramTile * kGramTile);
    if (ti == tj) rr_gram_pair<true>(X, means, n, p, ti, tj, kbeg, kend, dst);
    else rr_gram_pair<false>(X, means, n, p, ti, tj, kbeg, kend, dst);
}

// M (n+1 rows, leading dimension ld): the lower triangle of Xc Xc^T + alpha I in rows 0..n-1,
// yc in row n.  grid.x = tile pairs + 1 (the last one writes row n), grid.y = 16 slabs of a tile.
__global__ __launch_bounds__(256) void rr_gram_finish(const double *__restrict__ part, int tiles, int pairs, int splits,
                                                      int n, int ld, double alpha, const float *__restrict__ y,
                                                      const double *__restrict__ means, int p, double *__restrict__ M)
{
    if (static_cast<int>(blockIdx.x) == pairs) {
        for (int j = blockIdx.y * 256 + threadIdx.x; j < n; j += 16 * 256)
            M[static_cast<size_t>(n) * ld + j] = static_cast<double>(y[j]) - means[p];
        return;
    }
    int ti = 0, rem = blockIdx.x;
    while (rem >= tiles - ti) { rem -= tiles - ti; ++ti; }
    const int tj = ti + rem;
    const int e = blockIdx.y * 256 + threadIdx.x;
    const double *src = part + static_cast<size_t>(blockIdx.x) * splits * (kGramTile * kGramTile) + e;
    double s = 0.0;
#pragma unroll 8
    for (int c = 0; c < splits; ++c) s += src[static_cast<size_t>(c) * (kGramTile * kGramTile)];
    const int gi = ti * kGramTile + e / kGramTile, gj = tj * kGramTile + e % kGramTile;
    if (gi < n && gj < n && gj >= gi) M[static_cast<size_t>(gj) * ld + gi] = s + (gi == gj ? alpha : 0.0);
}

// LDS that one wavefront alone writes and reads: its accesses take effect in order, so only the compiler has to keep them so.
__device__ __forceinline__ void rr_wave_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 1/sqrt(x): the hardware's estimate (about 2^-24) and one third-order step, y (1 + e/2 + 3 e^2/8) with e = 1 - x y^2, whose
// error (e^3) is far below that of the last rounding.  NaN for x <= 0, as the square root would give.  rr_half spells the same
// steps out between its updates, operation by operation: the two change together.
__device__ __forceinline__ double rr_rsqrt(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// Keeps a value's computation where it stands: left alone the compiler turns the updates below around, so that a column's are
// one dependent chain, each waiting for its own two readlanes.
__device__ __forceinline__ void rr_here(double &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void rr_here_s(double &v) { asm volatile("" : "+s"(v)); }

// Columns K0 .. K0 + 15 of the 64 rows in the lanes: factored, and taken out of those of them that follow.  The chain from one
// column's diagonal to the next (readlane, reciprocal square root, five dependent operations) runs between the updates of
// the columns after it, which do not need its result.
template <int K0>
__device__ __forceinline__ void rr_half(double (&row)[kNB])
{
    constexpr int kEnd = K0 + 16;
    const int l = threadIdx.x & 63;
    double inv = rr_rsqrt(rr_lane(row[K0], K0));
#pragma unroll
    for (int k = K0; k < kEnd; ++k) {
        const double lrk = row[k] * inv;
        row[k] = l == k ? inv : lrk;
        if (k + 1 == kEnd) break;
        row[k + 1] = fma(-lrk, rr_lane(lrk, k + 1), row[k + 1]);   // meaningful where column <= lane
        rr_here(row[k + 1]);
        const double d = rr_lane(row[k + 1], k + 1);
        double y = __builtin_amdgcn_rsq(d), xy = 0.0, e = 0.0, f = 0.0, ye = 0.0;
        rr_here(y);
        const int others = kEnd - (k + 2);
        int stage = 0;
        double next = others > 0 ? rr_lane(lrk, k + 2) : 0.0;      // an update ahead: a readlane's result takes two cycles of waiting
#pragma unroll
        for (int i = 0; i <= others; ++i) {
#pragma unroll
            for (; stage < 4 && 5 * i >= (stage + 1) * others; ++stage) {      // rr_rsqrt, a step at a time
                if (stage == 0) { xy = -d * y; rr_here(xy); }
                if (stage == 1) { e = fma(xy, y, 1.0); rr_here(e); }
                if (stage == 2) { f = fma(0.375, e, 0.5); ye = y * e; rr_here(f); rr_here(ye); }
                if (stage == 3) { inv = fma(ye, f, y); rr_here(inv); }
            }
            if (i < others) {
                const int j = k + 2 + i;
                const double factor = next;
                if (i + 1 < others) {
                    next = rr_lane(lrk, j + 1);
                    rr_here_s(next);
                }
                row[j] = fma(-lrk, factor, row[j]);
                rr_here(row[j]);
            }
        }
    }
}

// One panel of the factorisation for 32 rows, inside one wavefront.  Lanes 0..31 hold the rows of the diagonal block at
// (k0, k0) of width nb <= 32 (padded with the identity; right of the diagonal they hold what stood there, which no other lane
// reads), lanes 32..63 the rows first .. first + 31 of M below it (rows past the last repeat it).  Column by column, in two
// halves of 16, all 64 rows are scaled and updated with values of lanes 0..31 that come through
// readlane: the same instructions factor the block and solve the rows against it.  Afterwards lanes 0..31 hold the factor
// with the reciprocals of its diagonal, lanes 32..63 the rows of L.  Between the two halves of the columns the second is
// updated by the first on the matrix unit, through `half` (LDS of this wavefront alone), which does in 12 instructions what
// takes 256 x (two readlanes + one multiply-add).  What bounds it is the chain of 32 columns.  Fit and prediction, 137 x 3,000
// and 677 x 20,000: 105.3 -> 94.5 and 576.7 -> 517.5 us.  Relative error of the coefficients against 80-bit sums, before -> now
// (2-norm, four data sets each): 33 x 300 1.1e-15 -> 1.3e-15, 64 x 500 2.06e-15 -> 2.08e-15, 137 x 1,000 3.78e-15 ->
// 3.81e-15, 200 x 900 at alpha = 0.001 6.4e-15 -> 6.2e-15, 260 x 1,300 7.4e-15 -> 7.2e-15.
constexpr int kHalfPitch = 18;      // doubles a row of `half`: 16-byte reads, and rows start in different banks
__device__ __forceinline__ void rr_factor_rows(const double *__restrict__ M, int ld, int nrows, int k0, int nb, int first,
                                               double (&row)[kNB], double (&half)[64][kHalfPitch])
{
    const int l = threadIdx.x & 63, r = l & 15, q = l >> 4;
    const double *src = M + static_cast<size_t>(l < kNB ? k0 + min(l, nb - 1) : min(first + l - kNB, nrows - 1)) * ld + k0;
    if (nb == kNB) {
#pragma unroll
        for (int c = 0; c < kNB; c += 2) {
            const double2 v = *reinterpret_cast<const double2 *>(src + c);   // ld and k0 are even, M is 256-byte aligned
            row[c] = v.x;
            row[c + 1] = v.y;
        }
    } else {
#pragma unroll
        for (int c = 0; c < kNB; ++c) row[c] = l >= nb && l < kNB ? (c == l ? 1.0 : 0.0) : c < nb ? src[c] : 0.0;
    }
    rr_half<0>(row);
    // rows 16..63: row[16 + c] -= sum over k < 16 of row[k] * (row 16 + c)[k]; lane q takes four neighbouring k of its row
#pragma unroll
    for (int c = 0; c < 16; ++c) half[l][c] = row[c];
    rr_wave_lds();
    double op[3][4];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int e = 0; e < 4; ++e) op[a][e] = half[16 + 16 * a + r][4 * q + e];
    d4 sum[3] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int a = 0; a < 3; ++a) sum[a] = rr_mfma(op[a][e], op[0][e], sum[a]);
    rr_wave_lds();
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int v = 0; v < 4; ++v) half[16 + 16 * a + 4 * v + q][r] = sum[a][v];
    rr_wave_lds();
#pragma unroll
    for (int c = 0; c < 16; ++c) row[16 + c] -= half[l][c];
    rr_half<16>(row);
}

// The lanes' results to memory: the rows of L go, transposed, to the upper triangle of M (L[i][k] to M[k][i]; nobody reads
// there before the back substitution, whose reads they suit), the factored block to D.
__device__ __forceinline__ void rr_store_rows(double *__restrict__ M, int ld, int nrows, int k0, int nb, int first,
                                              const double (&row)[kNB])
{
    const int l = threadIdx.x & 63;
    const int i = first + l - kNB;
    if (l < kNB || i >= nrows) return;
#pragma unroll
    for (int c = 0; c < kNB; ++c)
        if (c < nb) M[static_cast<size_t>(k0 + c) * ld + i] = row[c];
}

__device__ __forceinline__ void rr_store_block(double *__restrict__ D, int k0, const double (&row)[kNB])
{
    const int l = threadIdx.x & 63;
    if (l >= kNB) return;
    double *dst = D + static_cast<size_t>(k0 / kNB) * (kNB * kNB) + l * kNB;
#pragma unroll
    for (int c = 0; c < kNB; ++c) dst[c] = c <= l ? row[c] : 0.0;
}

// A factored diagonal block (32 x 32: the rows of L, with the reciprocals of its diagonal) to L^-1, in place, by one wavefront, through
// `block` (LDS of this wavefront alone).  The two 16 x 16 blocks on the diagonal side by side, lane m row m of its block's inverse,
// with no value of another lane; the one below them, -C^-1 B A^-1, on the matrix unit.  The back substitution multiplies by these
// instead of substituting; a panel's block is inverted beside the next panel, which it does not hold up.
constexpr int kBlockPitch = kNB + 1;
__device__ __forceinline__ void rr_invert_block(double *__restrict__ D, double *block)
{
    const int l = threadIdx.x & 63, r = l & 15, q = l >> 4, corner = l & 16;       // lanes 32..63 repeat lanes 0..31
#pragma unroll
    for (int i = 0; i < kNB * kNB / 64; ++i) block[(2 * i + (l >> 5)) * kBlockPitch + (l & 31)] = D[64 * i + l];
    rr_wave_lds();
    double u[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) u[c] = c == r ? 1.0 : 0.0;
#pragma unroll
    for (int k = 15; k >= 0; --k) {
        const double *row = block + (corner + k) * kBlockPitch + corner;
        u[k] *= row[k];
#pragma unroll
        for (int c = 0; c < k; ++c) {
            u[c] = fma(-row[c], u[k], u[c]);
            rr_here(u[c]);
        }
    }
    rr_wave_lds();
    if (l < kNB) {
#pragma unroll
        for (int c = 0; c < 16; ++c) block[l * kBlockPitch + corner + c] = u[c];
    }
    rr_wave_lds();
    // a product with the block below: of its 16 inner indices lane q takes 4 q .. 4 q + 3, on both sides
    auto times = [&](int lrow, int lcol, int rrow, int rcol) {
        d4 sum = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            sum = rr_mfma(block[(lrow + r) * kBlockPitch + lcol + 4 * q + e], block[(rrow + 4 * q + e) * kBlockPitch + rcol + r], sum);
        rr_wave_lds();
#pragma unroll
        for (int v = 0; v < 4; ++v) block[(16 + 4 * v + q) * kBlockPitch + r] = sum[v];
        rr_wave_lds();
    };
    times(16, 0, 0, 0);         // B A^-1
    times(16, 16, 16, 0);       // C^-1 (B A^-1)
#pragma unroll
    for (int i = 0; i < kNB * kNB / 64; ++i) {
        const int m = 2 * i + (l >> 5), c = l & 31;
        const double v = block[m * kBlockPitch + c];
        D[64 * i + l] = m >= 16 && c < 16 ? -v : v;
    }
}

// One panel in one launch: a workgroup of two wavefronts per 32 x 32 tile (ti >= tj) of what is left.  Each wavefront factors
// the diagonal block itself and solves the 32 rows of one side of the tile; the rows meet in LDS and the tile gets its
// rank-32 update.  The factoring is repeated by every tile, on units that would idle: a step takes its latency as long as the
// tiles are about as many as the chip holds at once, which is why only the triangle is launched: with the empty half of the
// square beside it two workgroups share a CU from 17 tiles a side on instead of 23 (a panel 10 us instead of 7.2).  A panel at
// n = 677: 30 us as two launches, 10.5 as one launch of the square whose updates waited for their readlanes, 7.3 now.
__global__ __launch_bounds__(128) void rr_step(double *__restrict__ M, int ld, int nrows, int k0, int nb,
                                               double *__restrict__ D)
{
    __shared__ double side[2][32][kNB + 1];
    if (k0 > 0 && blockIdx.x + 1 == gridDim.x) {        // the last workgroup: the block of the panel before
        if (threadIdx.x < 64) rr_invert_block(D + static_cast<size_t>(k0 / kNB - 1) * (kNB * kNB), &side[0][0][0]);
        return;
    }
    // tile blockIdx.x of the lower triangle, row by row; the root is off by one at most (48 rows of tiles)
    int ti = static_cast<int>((sqrtf(8.0f * static_cast<float>(blockIdx.x) + 1.0f) - 1.0f) * 0.5f);
    if ((ti + 1) * (ti + 2) / 2 <= static_cast<int>(blockIdx.x)) ++ti;
    if (ti * (ti + 1) / 2 > static_cast<int>(blockIdx.x)) --ti;
    const int tj = static_cast<int>(blockIdx.x) - ti * (ti + 1) / 2;
    __shared__ __attribute__((aligned(16))) double half[2][64][kHalfPitch];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, r = l & 15, q = l >> 4;
    const int first = k0 + nb, rows = nrows - first, cols = rows - 1;   // the row of yc has no column
    double old[2][4];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int gi = ti * 32 + 16 * w + 4 * v + q, gj = tj * 32 + 16 * b + r;
            old[b][v] = 0.0;
            if (gi < rows && gj < cols && gj <= gi) old[b][v] = M[static_cast<size_t>(first + gi) * ld + first + gj];
        }
    double row[kNB];
    const int mine = first + 32 * (w == 0 ? ti : tj);
    rr_factor_rows(M, ld, nrows, k0, nb, mine, row, half[w]);
    if (l >= kNB) {
#pragma unroll
        for (int c = 0; c < kNB; ++c) side[w][l - kNB][c] = row[c];
    }
    if (ti == tj && w == 0) rr_store_rows(M, ld, nrows, k0, nb, mine, row);
    if (ti == 0 && w == 1) rr_store_block(D, k0, row);
    __syncthreads();
    d4 acc[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const double av = side[0][16 * w + r][8 * q + e];
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[b] = rr_mfma(av, side[1][16 * b + r][8 * q + e], acc[b]);
    }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int gi = ti * 32 + 16 * w + 4 * v + q, gj = tj * 32 + 16 * b + r;
            if (gi < rows && gj < cols && gj <= gi) M[static_cast<size_t>(first + gi) * ld + first + gj] = old[b][v] - acc[b][v];
        }
}

// Larger systems: the panel alone, one wavefront per 32 rows below the diagonal block.  The rows also go, packed 32 to a row,
// to P for the trailing update.
__global__ __launch_bounds__(64) void rr_panel(double *__restrict__ M, int ld, int nrows, int k0, int nb,
                                               double *__restrict__ P, double *__restrict__ D)
{
    const int l = threadIdx.x, first = k0 + nb, mine = first + 32 * static_cast<int>(blockIdx.x);
    __shared__ __attribute__((aligned(16))) double half[64][kHalfPitch];
    static_assert(64 * kHalfPitch >= kNB * kBlockPitch, "the block to be inverted lies there");
    if (k0 > 0 && blockIdx.x + 1 == gridDim.x) {        // as in rr_step
        rr_invert_block(D + static_cast<size_t>(k0 / kNB - 1) * (kNB * kNB), &half[0][0]);
        return;
    }
    double row[kNB];
    rr_factor_rows(M, ld, nrows, k0, nb, mine, row, half);
    rr_store_rows(M, ld, nrows, k0, nb, mine, row);
    if (blockIdx.x == 0) rr_store_block(D, k0, row);
    const int i = mine + l - kNB;
    if (l < kNB || i >= nrows) return;
    double *pk = P + static_cast<size_t>(i - first) * kNB;
#pragma unroll
    for (int c = 0; c < kNB; ++c) pk[c] = row[c];
}

// C -= P P^T on the lower triangle of what lies below and right of the panel: one wavefront per
// 32 x 32 tile (ti >= tj), 2 x 2 MFMA tiles, the 32 columns of P in 8 steps (lane q = l / 16
// takes columns 8q..8q+7 of its row; same permutation on both sides).  rows = rows of P (the row
// of yc included), cols = columns still to be factored (rows - 1: yc has no column).
__global__ __launch_bounds__(64) void rr_trailing(double *__restrict__ M, int ld, int first, int rows, int cols,
                                                  const double *__restrict__ P)
{
    const int ti = blockIdx.y, tj = blockIdx.x;
    if (tj > ti) return;
    const int l = threadIdx.x, r = l & 15, q = l >> 4;
    double av[2][8], bv[2][8];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const double *sa = P + static_cast<size_t>(min(ti * 32 + 16 * a + r, rows - 1)) * kNB + 8 * q;
        const double *sb = P + static_cast<size_t>(min(tj * 32 + 16 * a + r, rows - 1)) * kNB + 8 * q;
#pragma unroll
        for (int e = 0; e < 8; ++e) { av[a][e] = sa[e]; bv[a][e] = sb[e]; }
    }
    d4 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[a][b] = rr_mfma(av[a][e], bv[b][e], acc[a][b]);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gi = ti * 32 + 16 * a + 4 * v + q, gj = tj * 32 + 16 * b + r;
                if (gi < rows && gj < cols && gj <= gi) M[static_cast<size_t>(first + gi) * ld + first + gj] -= acc[a][b][v];
            }
}

// One workgroup.  The upper triangle of M holds L^T, its column n z = L^-1 yc, D the inverted diagonal blocks, the last one as it was
// factored.  Solves L^T a = z from the last panel to the first: the first wavefront multiplies a panel's right-hand sides by its block
// (the chain of 32 x (multiply, readlane, multiply-add) that a substitution is was 2.6 of the 3.3 us of a panel), then
// everyone takes it out of the right-hand sides above it.  Eight lanes share a row, so that a load instruction takes whole
// lines (a lane that walks a row of its own finds its lines evicted before it has used them), each keeps its own part of the
// row's right-hand side, and the parts meet when the row's panel comes up.  Group g owns rows g, g + 64, ...; rows from
// kBackRows on are in `a`.  The factors of the next panel are on their way while the panel before is solved.  n = 677: 72 -> 45 us;
// whole fits 677 x 20,000 470 -> 452 us, 1,000 x 500 469 -> 419, 2,000 x 3,000 1,936 -> 1,745.  Relative errors of the coefficients
// against 80-bit sums (2-norm, rms of four data sets), substituted -> multiplied: 33 x 300 1.29e-15 -> 1.34e-15, 64 x 500 2.08e-15
// both, 137 x 1,000 3.81e-15 -> 3.79e-15, 200 x 900 at alpha = 0.001 6.18e-15 -> 6.17e-15, 260 x 1,300 7.22e-15 -> 7.17e-15.
constexpr int kBackThreads = 512;
constexpr int kBackGroups = kBackThreads / 8;
constexpr int kBackOwn = 16;
constexpr int kBackRows = kBackGroups * kBackOwn;
__global__ __launch_bounds__(kBackThreads) void rr_back_substitute(const double *__restrict__ M, int ld, int n,
                                                                   const double *__restrict__ D, double *a)
{
    __shared__ __attribute__((aligned(16))) double rhs[kNB], found[kNB];
    __shared__ double block[2][kNB][kNB + 1];
    const int t = threadIdx.x, c = t & 31, g = t >> 5;
    const int group = t >> 3, part = t & 7;
    const int last = (n - 1) / kNB * kNB;
    double mine[kBackOwn], factor[kBackOwn][4];      // this lane's columns of a panel: 2 part, 2 part + 1, and 16 further on
#pragma unroll
    for (int o = 0; o < kBackOwn; ++o) {
        const int j = group + o * kBackGroups;
        mine[o] = part == 0 && j < n ? M[static_cast<size_t>(j) * ld + n] : 0.0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = last + 2 * part + 16 * (e / 2) + e % 2;
            factor[o][e] = j < last && m < n ? M[static_cast<size_t>(j) * ld + m] : 0.0;
        }
    }
    for (int j = t + kBackRows; j < n; j += kBackThreads) a[j] = M[static_cast<size_t>(j) * ld + n];
    const double *src_block = D + static_cast<size_t>(last / kNB) * (kNB * kNB) + t;
    block[0][g][c] = src_block[0];
    block[0][g + 16][c] = src_block[512];
    int turn = 0;
    __syncthreads();
    for (int k0 = last; k0 >= 0; k0 -= kNB, turn ^= 1) {
        double next0 = 0.0, next1 = 0.0;
        if (k0 > 0) {
            src_block -= kNB * kNB;
            next0 = src_block[0];
            next1 = src_block[512];
        }
        if (k0 < kBackRows) {      // a panel's rows have one place among their owners': 32 divides kBackGroups
            const int at = group - k0 % kBackGroups;
            if (at >= 0 && at < kNB) {
                double v = 0.0;
#pragma unroll
                for (int o = 0; o < kBackOwn; ++o)
                    if (o == k0 / kBackGroups) v = mine[o];     // 0 past the last
                v += __shfl_xor(v, 1);
                v += __shfl_xor(v, 2);
                v += __shfl_xor(v, 4);
                if (part == 0) rhs[at] = v;
            }
        } else if (t < kNB) {
            rhs[t] = k0 + t < n ? a[k0 + t] : 0.0;
        }
        __syncthreads();
        if (t < 64) {
            double x = 0.0;
            if (k0 == last) {
                double v = rhs[c];
                const double inv = block[turn][c][c];
#pragma unroll 16
                for (int m = kNB - 1; m >= 0; --m) {
                    const double xm = rr_lane(v * inv, m);
                    if (c == m) x = xm;
                    v = fma(-block[turn][m][c], xm, v);          // meaningful where c < m
                }
            } else {        // lane (c, half of the panel)
                const int from = t >> 5 << 4;
                double s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int m = 0; m < kNB / 2; m += 2) {
                    s0 = fma(block[turn][from + m][c], rhs[from + m], s0);
                    s1 = fma(block[turn][from + m + 1][c], rhs[from + m + 1], s1);
                }
                x = s0 + s1;
                x += __shfl_xor(x, 32);
            }
            if (t < kNB) {
                found[t] = x;
                if (k0 + t < n) a[k0 + t] = x;
            }
        }
        block[turn ^ 1][g][c] = next0;
        block[turn ^ 1][g + 16][c] = next1;
        __syncthreads();
        const double2 x0 = *reinterpret_cast<const double2 *>(found + 2 * part);
        const double2 x1 = *reinterpret_cast<const double2 *>(found + 16 + 2 * part);
#pragma unroll
        for (int o = 0; o < kBackOwn; ++o) {
            if (o * kBackGroups >= k0) continue;
            mine[o] = fma(-factor[o][0], x0.x, mine[o]);     // rows from k0 on have been solved: nobody reads theirs again
            mine[o] = fma(-factor[o][1], x0.y, mine[o]);
            mine[o] = fma(-factor[o][2], x1.x, mine[o]);
            mine[o] = fma(-factor[o][3], x1.y, mine[o]);
            rr_here(mine[o]);      // now, and not after the next factors have come to stand beside these
        }
#pragma unroll
        for (int o = 0; o < kBackOwn; ++o) {
            if (o * kBackGroups >= k0 - kNB) continue;
            // rows that need no more repeat the last one that does; ld is a multiple of 4, M 256-byte aligned
            const int j = min(group + o * kBackGroups, k0 - kNB - 1);
            const double2 *src = reinterpret_cast<const double2 *>(M + static_cast<size_t>(j) * ld + k0 - kNB) + part;
            const double2 f0 = src[0], f1 = src[8];
            factor[o][0] = f0.x;
            factor[o][1] = f0.y;
            factor[o][2] = f1.x;
            factor[o][3] = f1.y;
        }
        if (k0 > kBackRows) {
            for (int j = t + kBackRows; j < k0; j += kBackThreads) {
                double s = a[j];
#pragma unroll 4
                for (int m = 0; m < kNB; ++m) s = fma(k0 + m < n ? -M[static_cast<size_t>(j) * ld + k0 + m] : 0.0, found[m], s);
                a[j] = s;
            }
            __syncthreads();
        }
    }
}
static_assert(kBackThreads == 16 * kNB, "the diagonal blocks are copied as two halves");
static_assert(kBackGroups % kNB == 0 && kBackRows % kNB == 0, "panels do not straddle the owners");

// wpart[r][j] = sum over the rows i of slice r of a[i] * (X[i][j] - mean_j)
__global__ __launch_bounds__(256) void rr_coef_partial(const float *__restrict__ X, const double *__restrict__ means,
                                                       const double *__restrict__ a, int n, int p, int rows_per,
                                                       double *__restrict__ wpart)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= p) return;
    const int i0 = blockIdx.y * rows_per, i1 = min(n, i0 + rows_per);
    const double mu = means[j];
    double s = 0.0;
    for (int i = i0; i < i1; i += kRowsInFlight) {
        float v[kRowsInFlight];
#pragma unroll
        for (int e = 0; e < kRowsInFlight; ++e) v[e] = X[static_cast<size_t>(min(i + e, i1 - 1)) * p + j];
#pragma unroll
        for (int e = 0; e < kRowsInFlight; ++e)
            if (i + e < i1) s = fma(a[i + e], static_cast<double>(v[e]) - mu, s);
    }
    wpart[static_cast<size_t>(blockIdx.y) * p + j] = s;
}

template <int NT>
__device__ __forceinline__ double rr_block_sum(double v)
{
    __shared__ double part[NT / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) s += part[w];
    __syncthreads();
    return s;
}

// w[j] = sum_r wpart[r][j]; bpart[block] = sum over the block's j of mean_j * w[j]
__global__ __launch_bounds__(256) void rr_coef_finish(const double *__restrict__ wpart, int splits, int p,
                                                      const double *__restrict__ means, double *__restrict__ w,
                                                      double *__restrict__ bpart)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    double s = 0.0;
    if (j < p) {
        double v[kMaxRowSplits];
#pragma unroll
        for (int r = 0; r < kMaxRowSplits; ++r) v[r] = wpart[static_cast<size_t>(min(r, splits - 1)) * p + j];
#pragma unroll
        for (int r = 0; r < kMaxRowSplits; ++r) s += r < splits ? v[r] : 0.0;
        w[j] = s;
        s *= means[j];
    }
    s = rr_block_sum<256>(s);
    if (threadIdx.x == 0) bpart[blockIdx.x] = s;
}

// b = mean(y) - sum_j mean_j * w[j]   (one workgroup over the block sums)
__global__ __launch_bounds__(256) void rr_intercept(const double *__restrict__ means, const double *__restrict__ bpart,
                                                    int blocks, int p, double *__restrict__ b)
{
    double s = 0.0;
    for (int j = threadIdx.x; j < blocks; j += 256) s += bpart[j];
    s = rr_block_sum<256>(s);
    if (threadIdx.x == 0) b[0] = means[p] - s;
}

// pred[i] = b + sum_j X[i][j] * w[j]: one workgroup of NT lanes per row, four neighbouring columns per lane and round (rows
// start at any multiple of 4 bytes) and two rounds in flight.  Few rows are a matter of latency, so long rows take 1,024
// lanes: 1 x 20,000 23 -> 4.6 us.
template <int NT>
__global__ __launch_bounds__(NT) void rr_predict(const float *__restrict__ X, int p, const double *__restrict__ w,
                                                 const double *__restrict__ b, double *__restrict__ pred)
{
    const float *row = X + static_cast<size_t>(blockIdx.x) * p;
    const int whole = p & ~3;
    d4 s4 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
    for (int j = 4 * static_cast<int>(threadIdx.x); j < whole; j += 4 * NT) {
        const f4u x = *reinterpret_cast<const f4u *>(row + j);
        const d4u c = *reinterpret_cast<const d4u *>(w + j);
#pragma unroll
        for (int e = 0; e < 4; ++e) s4[e] = fma(static_cast<double>(x[e]), c[e], s4[e]);
    }
    double s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
    if (static_cast<int>(threadIdx.x) < p - whole) s = fma(static_cast<double>(row[whole + threadIdx.x]), w[whole + threadIdx.x], s);
    s = rr_block_sum<NT>(s);
    if (threadIdx.x == 0) pred[blockIdx.x] = s + b[0];
}

inline size_t up256(size_t v) { return (v + 255) / 256 * 256; }

}  // namespace

#define RR_HIP(call)                                                                   \
    do {                                                                               \
        hipError_t e_ = (call);                                                        \
        if (e_ != hipSuccess)                                                          \
            return rk_fail(ROCKET_EHIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

namespace {

// Where the pieces of the workspace lie and how the work is cut, for n examples and p features.
struct RidgePlan {
    int ld;            // leading dimension of the (n+1)-row system
    int tiles, pairs;  // 64-row tiles of the Gram matrix and pairs ti <= tj of them
    int chunk, splits; // features per slice (a multiple of 16) and slices
    int row_splits, rows_per;
    size_t off_means, off_M, off_dual, off_P, off_D, off_scratch, bytes;
};

RidgePlan ridge_plan(int n, int p)
{
    RidgePlan q;
    q.ld = (n + 1 + 3) / 4 * 4;
    q.tiles = (n + kGramTile - 1) / kGramTile;
    q.pairs = q.tiles * (q.tiles + 1) / 2;
    const int want = std::max(1, std::min(64, kGramWaves / q.pairs));
    q.chunk = std::max(64, ((p + want - 1) / want + 15) / 16 * 16);
    q.splits = (p + q.chunk - 1) / q.chunk;
    q.row_splits = std::max(1, std::min(kMaxRowSplits, n / 32));
    q.rows_per = (n + q.row_splits - 1) / q.row_splits;
    q.row_splits = (n + q.rows_per - 1) / q.rows_per;
    const size_t coef_blocks = (static_cast<size_t>(p) + 255) / 256;
    const size_t scratch = std::max({static_cast<size_t>(q.row_splits) * (p + 1),
                                     static_cast<size_t>(q.pairs) * q.splits * kGramTile * kGramTile,
                                     static_cast<size_t>(q.row_splits) * p + coef_blocks});
    size_t at = 0;
    q.off_means = at;   at += up256(static_cast<size_t>(p + 1) * 8);
    q.off_M = at;       at += up256(static_cast<size_t>(n + 1) * q.ld * 8);
    q.off_dual = at;    at += up256(static_cast<size_t>(n) * 8);
    q.off_P = at;       at += up256(static_cast<size_t>(n + 1) * kNB * 8);
    q.off_D = at;       at += up256(static_cast<size_t>((n + kNB - 1) / kNB) * kNB * kNB * 8);
    q.off_scratch = at; at += up256(scratch * 8);
    q.bytes = at;
    return q;
}

}  // namespace

extern "C" size_t rocket_ridge_workspace_bytes(int32_t n, int32_t p)
{
    if (n < 1 || p < 1 || n > kMaxExamples) return 0;
    return ridge_plan(n, p).bytes;
}

extern "C" int rocket_ridge_fit(const float *features_dev, const float *targets_dev, int32_t n, int32_t p, double alpha,
                                double *coef_dev, double *intercept_dev, void *ws, size_t ws_bytes, void *hip_stream)
{
    if (!features_dev || !targets_dev || !coef_dev || !intercept_dev)
        return rk_fail(ROCKET_EINVAL, "rocket_ridge_fit: NULL pointer");
    if (n < 1 || p < 1) return rk_fail(ROCKET_EINVAL, "rocket_ridge_fit: n and p must be >= 1");
    if (n > kMaxExamples) return rk_fail(ROCKET_EINVAL, "rocket_ridge_fit: at most 32768 examples (the dual system is stored densely)");
    if (!(alpha > 0.0) || !std::isfinite(alpha)) return rk_fail(ROCKET_EINVAL, "rocket_ridge_fit: alpha must be positive and finite");
    const RidgePlan q = ridge_plan(n, p);
    if (!ws || ws_bytes < q.bytes)
        return rk_fail(ROCKET_EWORKSPACE, "rocket_ridge_fit: workspace of " + std::to_string(q.bytes) + " bytes required");
    if (reinterpret_cast<uintptr_t>(ws) % 256 != 0) return rk_fail(ROCKET_EWORKSPACE, "rocket_ridge_fit: workspace must be 256-byte aligned");
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    char *base = static_cast<char *>(ws);
    double *means = reinterpret_cast<double *>(base + q.off_means);
    double *M = reinterpret_cast<double *>(base + q.off_M);
    double *dual = reinterpret_cast<double *>(base + q.off_dual);
    double *P = reinterpret_cast<double *>(base + q.off_P);
    double *D = reinterpret_cast<double *>(base + q.off_D);
    double *scratch = reinterpret_cast<double *>(base + q.off_scratch);

    hipLaunchKernelGGL(rr_col_sums, dim3((p + 1 + 255) / 256, q.row_splits), dim3(256), 0, stream, features_dev,
                       targets_dev, n, p, q.rows_per, scratch);
    hipLaunchKernelGGL(rr_means, dim3((p + 1 + 255) / 256), dim3(256), 0, stream, scratch, q.row_splits, n, p, means);
    const int items = q.pairs * q.splits;
    hipLaunchKernelGGL(rr_gram, dim3((items + 7) / 8 * 8), dim3(64), 0, stream, features_dev, means, n, p, q.tiles,
                       q.pairs, q.chunk, q.splits, scratch);
    hipLaunchKernelGGL(rr_gram_finish, dim3(q.pairs + 1, 16), dim3(256), 0, stream, scratch, q.tiles, q.pairs, q.splits,
                       n, q.ld, alpha, targets_dev, means, p, M);
    const int nrows = n + 1;
    for (int k0 = 0; k0 < n; k0 += kNB) {
        const int nb = std::min(kNB, n - k0);
        const int first = k0 + nb, rows = nrows - first;   // rows >= 1: the row of yc is always below
        const int t = (rows + 31) / 32, more = k0 > 0 ? 1 : 0;      // a workgroup more inverts the block of the panel before
        if (t <= kFusedTiles) {
            hipLaunchKernelGGL(rr_step, dim3(t * (t + 1) / 2 + more), dim3(128), 0, stream, M, q.ld, nrows, k0, nb, D);
        } else {   // so many rows are left that the panel is 32 columns wide and columns follow it
            hipLaunchKernelGGL(rr_panel, dim3(t + more), dim3(64), 0, stream, M, q.ld, nrows, k0, nb, P, D);
            hipLaunchKernelGGL(rr_trailing, dim3(t, t), dim3(64), 0, stream, M, q.ld, first, rows, rows - 1, P);
        }
    }
    hipLaunchKernelGGL(rr_back_substitute, dim3(1), dim3(kBackThreads), 0, stream, M, q.ld, n, D, dual);
    const int coef_blocks = (p + 255) / 256;
    double *wpart = scratch, *bpart = scratch + static_cast<size_t>(q.row_splits) * p;
    hipLaunchKernelGGL(rr_coef_partial, dim3(coef_blocks, q.row_splits), dim3(256), 0, stream, features_dev, means, dual,
                       n, p, q.rows_per, wpart);
    hipLaunchKernelGGL(rr_coef_finish, dim3(coef_blocks), dim3(256), 0, stream, wpart, q.row_splits, p, means, coef_dev,
                       bpart);
    hipLaunchKernelGGL(rr_intercept, dim3(1), dim3(256), 0, stream, means, bpart, coef_blocks, p, intercept_dev);
    RR_HIP(hipGetLastError());
    return ROCKET_OK;
}

extern "C" int rocket_ridge_predict(const float *features_dev, int32_t m, int32_t p, const double *coef_dev,
                                    const double *intercept_dev, double *pred_dev, void *hip_stream)
{
    if (!features_dev || !coef_dev || !intercept_dev || !pred_dev)
        return rk_fail(ROCKET_EINVAL, "rocket_ridge_predict: NULL pointer");
    if (m < 1 || p < 1) return rk_fail(ROCKET_EINVAL, "rocket_ridge_predict: m and p must be >= 1");
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (p >= kWideRow) hipLaunchKernelGGL(rr_predict<1024>, dim3(m), dim3(1024), 0, stream, features_dev, p, coef_dev, intercept_dev, pred_dev);
    else hipLaunchKernelGGL(rr_predict<256>, dim3(m), dim3(256), 0, stream, features_dev, p, coef_dev, intercept_dev, pred_dev);
    RR_HIP(hipGetLastError());
    return ROCKET_OK;
}
