// Panel factorisation of the blocked Householder QR (Alg. 1 step 3) by
// CholeskyQR2 with Householder reconstruction: panels stored in float64 or
// float32, every sum, factorisation and product in float64 (a float32 panel's
// rows are rounded to float32 where they are stored, and the second pass's
// Gram is of the stored rows).
//
// The unblocked panel (k_qr_panel) needs one grid-wide exchange per column.
// Here a 64-column panel P (M x 64, row-major, in place) takes three passes
// over its rows and two single-block factorisations:
//   1. k_cq_gram + k_cq_reduce: G = P^T P (partial Grams of 256-row slabs on
//      the matrix cores, then a fixed-order sum);
//   2. k_cq_factor (pass 1): column scaling D = diag(sqrt(G_jj)), Cholesky
//      D^{-1} G D^{-1} = U1^T U1, R1 = U1 D and W1 = R1^{-1};
//   3. k_cq_apply_gram + k_cq_reduce: P <- Q1 = P W1 fused with the Gram of Q1;
//   4. k_cq_factor (pass 2): Cholesky of Q1's Gram = U2^T U2 (Q = Q1 U2^{-1},
//      R = U2 R1), and the Householder reconstruction (Ballard, Demmel,
//      Grigori, Jacquelin, Knight and Nguyen, "Reconstructing Householder
//      vectors from tall-skinny QR", 2015) of Q's top 64 x 64 block: with
//      S = diag(s_j), Q S - [I; 0] = Y (-T Y_1^T) is an LU factorisation
//      without pivoting whose unit lower factor Y holds the Householder vectors
//      of a QR of P and whose pivots give tau_j = -U_jj = 1 + |c_j|, s_j =
//      -sign(c_j) chosen column by column from the current pivot c_j (so
//      |U_jj| >= 1 and the elimination is stable); the QR's triangular factor
//      is S R.  The panel's top block gets S R and Y_1;
//   5. k_cq_apply: the rows below become Y_2 = Q1 (U2^{-1} S U^{-1}) = Q1 (U S U2)^{-1}.
// The panel is left exactly as the unblocked kernel leaves it: S R on and
// above the diagonal, the vectors below it (unit diagonal implied), tau.
//
// CholeskyQR2 is accurate while the scaled panel's condition number stays
// well below u^{-1/2} (its first pass squares it).  The sketches of the RFM
// systems here have scaled panel conditions up to 3.2e6 (8x8-box system, all
// 200 panels; unscaled up to 2e13).  A panel whose first Cholesky meets a
// non-positive pivot or a pivot ratio below the caller's threshold is flagged
// (status 1) and factored by the unblocked kernel instead, on the untouched
// panel; a second Cholesky failure (status 2) leaves Q1 in the panel, which the
// unblocked kernel then factors, multiplying its R by R1 at the end.  Every sum runs in a fixed order.
#include "common.h"

namespace rfmls {
namespace {

constexpr int kNb = 64;      // panel width
constexpr int kSlab = 256;   // rows per partial Gram (tall panels)
// Panels under this many rows take 128-row slabs (two 16-row groups per
// wavefront): twice the workgroups, so a short panel's Gram and apply passes
// use more of the GPU, their partial Grams still few enough to sum (Helmholtz
// sketch, 12,800 rows: 0.155 -> 0.146 ms per panel; 64-row slabs 0.147).
constexpr int64_t kShortPanelRows = 32768;
inline int64_t slab_rows(int64_t M) { return M >= kShortPanelRows ? kSlab : 128; }

typedef double v4d __attribute__((ext_vector_type(4)));

// status: 0 CholeskyQR2 used; 1 first Cholesky failed (panel untouched);
// 2 second Cholesky failed (panel holds Q1, R1 in Rc)

// Operand layout of v_mfma_f64_16x16x4f64 (D += A B, A 16 x 4, B 4 x 16): lane
// l = 16 lk + lr holds A[lr][lk] and B[lk][lr]; accumulator register r holds
// D[lk + 4 r][lr].

// A Gram is kept as its ten upper 16 x 16 tiles (a, b), a <= b, each row-major, which
// is also the order r * 64 + lane of the accumulator registers.
constexpr int kGramTiles = 10;
constexpr int kGramLen = kGramTiles * 256;
__device__ __forceinline__ int gram_at(int i, int j) {  // entry (i, j), either triangle
  const int a = i >> 4, b = j >> 4;
  const bool up = a <= b;
  const int a2 = up ? a : b, b2 = up ? b : a, ii = up ? i : j, jj = up ? j : i;
  return (a2 * 4 - a2 * (a2 - 1) / 2 + b2 - a2) * 256 + (ii & 15) * 16 + (jj & 15);
}
// gp = the sum of the four wavefronts' tiles in wave order; S holds 4 kGramLen doubles.
// One pass out and one back: adding them one wavefront at a time in a shared copy took
// a read, an add and a write of every entry and a barrier per wavefront (1,600 / 3,200
// column sketches, with W's loads issued together: Gram 7.5 -> 5.5 us, fused apply + Gram
// 16.0 / 18.0 -> 10.5 / 12.2, apply 8.7 / 10.2 -> 5.3 / 7.1; Helmholtz solve 24.1 -> 23.5 ms).
__device__ __forceinline__ void sum_tiles(const v4d (&acc)[kGramTiles], double* __restrict__ S,
                                          double* __restrict__ gp) {
  const int t = threadIdx.x;
  const int lane = t & 63, w = t >> 6;
#pragma unroll
  for (int q = 0; q < kGramTiles; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) S[w * kGramLen + q * 256 + r * 64 + lane] = acc[q][r];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kGramTiles; ++q) {
    const int e = q * 256 + t;
    gp[e] = ((S[e] + S[kGramLen + e]) + S[2 * kGramLen + e]) + S[3 * kGramLen + e];
  }
}

// Partial Gram of rows [z S, (z + 1) S) of P (S = 64 NG) on the matrix cores.
// Wave w takes the 16 NG rows from z S + 16 NG w and accumulates the ten upper
// 16 x 16 tiles of their Gram; each lane loads its operands straight from P
// (lane (lr, lk) reads row 4 s + lk, columns 16 q + lr: every 16 lanes read
// 128 contiguous bytes), no LDS staging.  The four waves' tiles are then added
// in wave order through LDS (sum_tiles).
template <typename TS, int NG>
__global__ void __launch_bounds__(256) k_cq_gram(const TS* __restrict__ P, int64_t ld, int64_t M,
                                                 double* __restrict__ Gpart, const int* __restrict__ status) {
  if (status && *status) return;
  __shared__ double S[4 * kGramLen];
  const int t = threadIdx.x;
  const int lane = t & 63, w = t >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  v4d acc[10];
#pragma unroll
  for (int q = 0; q < 10; ++q) acc[q] = v4d{0.0, 0.0, 0.0, 0.0};
  const int64_t r0 = (int64_t)blockIdx.x * (64 * NG) + 16 * NG * w;
  // all the wavefront's rows' operands loaded first (rows past M read row
  // M - 1 and are replaced by zeros, so the loads carry no branch)
  double x[4 * NG][4];
#pragma unroll
  for (int s = 0; s < 4 * NG; ++s) {
    const int64_t row = r0 + 4 * s + lk;
    const int64_t rr = row < M ? row : M - 1;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double v = (double)P[rr * ld + 16 * q + lr];
      x[s][q] = row < M ? v : 0.0;
    }
  }
#pragma unroll
  for (int s = 0; s < 4 * NG; ++s) {
    int tile = 0;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = a; b < 4; ++b, ++tile)
        acc[tile] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[s][a], x[s][b], acc[tile], 0, 0, 0);
  }
  sum_tiles(acc, S, Gpart + (int64_t)blockIdx.x * kGramLen);
}

// G = sum of the nslab partials in slab order.  Block b takes entries
// 16 b .. 16 b + 15; its 16 slices of threads sum every 16th partial, then the
// 16 slice sums are added in order.  With reset, the panel's status is set to 0
// (first pass: a new panel).
__global__ void __launch_bounds__(256) k_cq_reduce(const double* __restrict__ Gpart, int nslab,
                                                   double* __restrict__ G, int* __restrict__ status, int reset) {
  if (!reset && *status) return;
  __shared__ double red[16][17];
  const int t = threadIdx.x;
  const int el = t & 15, zq = t >> 4;
  const int e = blockIdx.x * 16 + el;
  double s = 0.0;
#pragma unroll 4
  for (int z = zq; z < nslab; z += 16) s += Gpart[(int64_t)z * kGramLen + e];
  red[zq][el] = s;
  __syncthreads();
  if (t < 16) {
    double tot = 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) tot += red[q][t];
    G[blockIdx.x * 16 + t] = tot;
  }
  if (reset && blockIdx.x == 0 && t == 0) *status = 0;
}

// ---------------------------------------------------------------------------
// 64 x 64 factorisations in LDS by one block of 256 threads, blocked by 16:
// the eliminations of a 16-row (or 16-column) block on one wavefront in
// registers (values passed by v_readlane), every product of blocks on the
// matrix cores.
// ---------------------------------------------------------------------------
constexpr int kB = 16;
constexpr int kLd = kNb + 1;  // LDS row stride of a 64 x 64 matrix
typedef double Mat[kNb][kLd];
typedef double Blk[kB][kB + 1];

// Tile (ti, tj) of D -= op(A) B with K = 16, for LDS matrices of kLd columns (D, A
// and B do not overlap): op(A) = A (a column block) or, with TA, A^T (A a row block).
template <bool TA>
__device__ __forceinline__ void rank16_tile(double* D, const double* A, const double* B, int ti, int tj, int lane) {
  const int lr = lane & 15, lk = lane >> 4;
  double* d = D + (16 * ti + lk) * kLd + 16 * tj + lr;
  const double* ap = TA ? A + lk * kLd + 16 * ti + lr : A + (16 * ti + lr) * kLd + lk;
  const double* bp = B + lk * kLd + 16 * tj + lr;
  v4d acc;
  double a[4], b[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    a[s] = ap[4 * s * (TA ? kLd : 1)];
    b[s] = bp[4 * s * kLd];
    acc[s] = d[4 * s * kLd];
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[s], b[s], acc, 0, 0, 0);
#pragma unroll
  for (int r = 0; r < 4; ++r) d[4 * r * kLd] = acc[r];
}

// Orders a wavefront's LDS writes before its later LDS reads (no block barrier).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 1 / x and 1 / sqrt(x) (x finite, positive for the root) by the hardware estimate,
// good to 2^-24 or so, and one third-order step (to about an ulp): dependent chains a
// third as long as the library's.
__device__ __forceinline__ double rcp2(double x) {
  const double y = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, y, 1.0);
  return fma(y, fma(e, e, e), y);
}
__device__ __forceinline__ double rsq2(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// Z = inverse of the diagonal block at k0 of the upper triangular U, by one
// wavefront: lane l < 16 forms column l by a column sweep with U's entries read
// uniformly from LDS (what lies below the diagonal is not read).
__device__ __forceinline__ void diag_inverse(const Mat& U, int k0, Blk& Z, int l) {
  double rd[kB], acc[kB];
#pragma unroll
  for (int i = 0; i < kB; ++i) {
    rd[i] = rcp2(U[k0 + i][k0 + i]);
    acc[i] = (i == l) ? 1.0 : 0.0;
  }
#pragma unroll
  for (int m2 = kB - 1; m2 >= 0; --m2) {
    const double zm = (m2 <= l) ? acc[m2] * rd[m2] : 0.0;
    acc[m2] = zm;
#pragma unroll
    for (int i = 0; i < m2; ++i) acc[i] = fma(-U[k0 + i][k0 + m2], zm, acc[i]);
  }
  if (l < kB)
#pragma unroll
    for (int i = 0; i < kB; ++i) Z[i][l] = acc[i];
}

// Block row kb of the Cholesky factor A = U^T U (A symmetric, kept whole; U written
// over A with zeros below the diagonal of the diagonal block), by one wavefront:
// 16 rows, columns k0 = 16 kb .. 63, lane l holding column k0 + l.  Step s takes
// the pivot from lane s (v_readlane), scales the lanes' row s entries to U's
// row s and subtracts u_s,i u_s,l from the rows i > s below it, u_s,i read
// from lane i; the whole block row of U comes out of the one elimination (no
// product with the diagonal block's inverse) and no LDS round trip sits on the
// chain.  mn / mx follow the pivots u_kk; *bad is set on a non-positive or
// non-finite pivot.  With Z (kb > 0), 16 of the lanes past the columns carry the
// identity through the same steps, which leaves U_kb^{-T}: Z = U_kb^{-1}.
__device__ __forceinline__ void chol_panel(Mat& A, int kb, int l, double* mn, double* mx, bool* bad, Blk* Z) {
  const int k0 = kb * kB;
  const bool act = l < kNb - k0;
  const int zc = l - (kNb - k0);  // column of the identity
  double d[kB];
#pragma unroll
  for (int i = 0; i < kB; ++i) {
    const double a = A[k0 + i][act ? k0 + l : k0];
    d[i] = act ? a : (i == zc ? 1.0 : 0.0);
  }
#pragma unroll
  for (int s2 = 0; s2 < kB; ++s2) {
    const double piv = lane_read(d[s2], s2);
    *bad |= !(piv > 0.0 && piv < INFINITY);
    const double r = rsq2(piv);
    *mn = fmin(*mn, piv * r);
    *mx = fmax(*mx, piv * r);
    const double us = d[s2] * r;  // u_{s,l} for l >= s
    // u_{s,i} from the unscaled row, whose readlanes need not wait for r
#pragma unroll
    for (int i = s2 + 1; i < kB; ++i) d[i] = fma(-(lane_read(d[s2], i) * r), us, d[i]);
    d[s2] = l >= s2 ? us : 0.0;
  }
  if (act)
#pragma unroll
    for (int i = 0; i < kB; ++i) A[k0 + i][k0 + l] = d[i];
  else if (Z && zc < kB)
#pragma unroll
    for (int i = 0; i < kB; ++i) (*Z)[zc][i] = d[i];
}

// Columns k0 .. k0 + 15 of the reconstruction's LU (see k_cq_factor), rows k0 .. 63,
// by one wavefront, lane i holding row i.  Step j: the current pivot e_j by
// readlane, s_j = -sign(e_j), row j minus s_j times U2's row j (whose diagonal is
// positive, so the pivot's size is |e_j| + u_jj), multipliers and the panel's
// remaining columns.  A gets the multipliers below the diagonal and U~ on and
// above it, tau_j = |pivot| / u_jj.  Then the same rows of U~ in the columns right of
// the panel, a column per lane: unit lower forward substitution with the multipliers
// out of the registers (readlane), minus s_i U2; or, for the last panel, which has
// none, Z = the inverse of its diagonal block, a column per lane, by a column sweep.
__device__ __forceinline__ void recon_panel(Mat& A, const Mat& U2, int kb, int i, double* sg, double* tau, Blk& Z) {
  const int k0 = kb * kB;
  const int c = k0 + kB + i;  // this lane's column right of the panel
  const bool right = c < kNb;
  double p[kB], u[kB], x[kB];
#pragma unroll
  for (int m = 0; m < kB; ++m) {
    p[m] = A[i][k0 + m];
    u[m] = U2[i][k0 + m];  // row i of U2 (used on the panel's own rows only)
  }
  double pv = 1.0;  // this row's pivot
#pragma unroll
  for (int j = 0; j < kB; ++j) {
    const int pr = k0 + j;
    const double ej = lane_read(p[j], pr);
    const double ujj = lane_read(u[j], pr);
    const double rp = rcp2(ej + copysign(ujj, ej));  // the pivot e_j - s_j u_jj
    const double cj = i == pr ? copysign(1.0, ej) : 0.0;
    const double pj = i > pr ? p[j] : 0.0;
#pragma unroll
    for (int m = j; m < kB; ++m) p[m] = fma(cj, u[m], p[m]);
    const double lij = pj * rp;
    pv = i == pr ? p[j] : pv;
    p[j] = i > pr ? lij : p[j];
#pragma unroll
    for (int m = j + 1; m < kB; ++m) p[m] = fma(-lij, lane_read(p[m], pr), p[m]);
  }
  const double sv = -copysign(1.0, pv), rv = rcp2(pv);
  if (i >= k0) {
#pragma unroll
    for (int m = 0; m < kB; ++m) A[i][k0 + m] = p[m];
    if (i < k0 + kB) {
      sg[i] = sv;
      tau[i] = fabs(pv) / U2[i][i];
    }
  }
  if (kb == kNb / kB - 1) {
#pragma unroll
    for (int m = 0; m < kB; ++m) x[m] = m == i ? 1.0 : 0.0;
#pragma unroll
    for (int m = kB - 1; m >= 0; --m) {
      x[m] = m <= i ? x[m] * lane_read(rv, k0 + m) : 0.0;
#pragma unroll
      for (int q = 0; q < m; ++q) x[q] = fma(-lane_read(p[m], k0 + q), x[m], x[q]);
    }
    if (i < kB)
#pragma unroll
      for (int m = 0; m < kB; ++m) Z[m][i] = x[m];
    return;
  }
#pragma unroll
  for (int m = 0; m < kB; ++m)
    x[m] = fma(-lane_read(sv, k0 + m), U2[k0 + m][right ? c : k0], A[k0 + m][right ? c : k0]);
#pragma unroll
  for (int m = 0; m < kB; ++m) {
#pragma unroll
    for (int q = m + 1; q < kB; ++q) x[q] = fma(-lane_read(p[m], k0 + q), x[m], x[q]);
  }
  if (right)
#pragma unroll
    for (int m = 0; m < kB; ++m) A[k0 + m][c] = x[m];
}

// R1 <- U2 R1 (both upper triangular, zeros below the diagonal inside the diagonal
// blocks) by one wavefront on the matrix cores: block column by block column, the
// blocks from the top down, each needing only the blocks of R1 at and below it.
__device__ __forceinline__ void upper_product(const Mat& U2, Mat& R1, int lane) {
  const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int tj = 0; tj < kNb / kB; ++tj)
#pragma unroll
    for (int ti = 0; ti <= tj; ++ti) {
      v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int k = 4 * ti; k < 4 * (tj + 1); ++k)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(U2[16 * ti + lr][4 * k + lk], R1[4 * k + lk][16 * tj + lr], acc, 0,
                                                   0, 0);
      wave_sync();
#pragma unroll
      for (int r = 0; r < 4; ++r) R1[16 * ti + lk + 4 * r][16 * tj + lr] = acc[r];
      wave_sync();
    }
}

// Block column tj of W = U^{-1} for the upper triangular U (Z the inverses of its
// diagonal blocks) by one wavefront, block back substitution from the bottom up:
// W_k = -Z_k (sum_{k < j <= tj} U_kj W_j), w[k] in the accumulator layout.  A register
// r of it holds rows lk + 4 r, so taking K in that order makes w[j] the next product's
// operand as it stands: no LDS round trip and no barrier.
__device__ __forceinline__ void upper_inverse_col(const Mat& U, const Blk* Z, int tj, int lane, v4d (&w)[kNb / kB]) {
  const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int j = 0; j < kNb / kB; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) w[j][r] = j == tj ? Z[j][lk + 4 * r][lr] : 0.0;
#pragma unroll
  for (int k = kNb / kB - 2; k >= 0; --k) {
    if (k >= tj) continue;
    v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = k + 1; j < kNb / kB; ++j)
      if (j <= tj)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(U[16 * k + lr][16 * j + lk + 4 * r], w[j][r], acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      w[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(Z[k][lr][lk + 4 * r], -acc[r], w[k], 0, 0, 0);
  }
}

// One Cholesky step of CholeskyQR2 on the reduced Gram G.
// pass 1 (column-scaled Gram D^{-1} G D^{-1} = U^T U): R1 = U D into Rc and
//   Wk = R1^{-1} = D^{-1} U^{-1} (the operand of the fused apply + Gram).
// pass 2 (Gram of Q1 = U2^T U2): R = U2 R1 into the panel's top block as S R,
//   and the Householder reconstruction of Q = Q1 U2^{-1}: with S = diag(s_j),
//   Q's top block gives Q S - I = L U (no pivoting, s_j = -sign of the current
//   pivot).  Multiplied by S U2 from the right that is
//     A - S U2 = L U~,  A = Q1's top block,  U~ = U S U2,
//   so the elimination runs on A and U2 directly: Q's top block and U2^{-1} are
//   not formed, the current pivot e_j is u2_jj times Q's, tau_j = -u_jj = |u~_jj| /
//   u2_jj, and the rows below become Q1bot U2^{-1} S U^{-1} = Q1bot U~^{-1}: one
//   triangular inverse, Wk = U~^{-1}, where U2^{-1} and U^{-1} and two products with
//   them were formed before.  L goes below the diagonal of the panel's top block.
// A pivot ratio u_min / u_max below min_pivot_ratio (or a non-positive pivot)
// sets *status = pass and leaves everything else untouched.
//
// Bound by the eliminations' chains (a step per column), so independent ones run
// beside each other, one wavefront each: stage kb has block row kb of the Cholesky
// factor (wavefront 0; in pass 1 its diagonal block's inverse comes out of the same
// elimination), the reconstruction's panel kb - 1 (1; the last with its diagonal
// block's inverse), the inverse of an earlier diagonal block of U~ (2) and at the end
// U2 R1 (3); the trailing tiles after a stage are shared by all four, and each
// wavefront forms a block column of the inverse by itself.  Average of the two passes
// 27.5 us; with the diagonal inverses as stages of their own, trailing and inverse
// products with barriers inside and the library's rsqrt and divisions on the chains it
// was 37.7 (4x4-box solve 8.8 -> 8.35 ms, Helmholtz 25.3 -> 24.4 ms).  A step of a
// 16-column elimination takes about 400 (Cholesky) and 500 clocks (reconstruction) at
// some 75 instructions; shortening its dependent chain changes nothing, so one
// wavefront's issue rate is what is left.
template <typename TS>
__global__ void __launch_bounds__(256) k_cq_factor(const double* __restrict__ G, double* __restrict__ Wk,
                                                   double* __restrict__ Rc, TS* __restrict__ P, int64_t ld,
                                                   TS* __restrict__ tau, int* __restrict__ status, int pass,
                                                   double min_pivot_ratio) {
  if (pass == 2 && *status) return;
  __shared__ Mat M0, M2, M3;
  __shared__ Blk Z[kNb / kB];
  __shared__ double dsc[kNb], rdsc[kNb];
  __shared__ double sg[kNb], tj[kNb];
  __shared__ int bad_s;
  __shared__ double ext[2];
  constexpr int kBlocks = kNb / kB;
  const int t = threadIdx.x;
  const int lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  // thread t takes element (t / 64 + 4 q, t % 64), q < 16, of every 64 x 64
  // operand; each operand's 16 loads are issued together
  const int er = t >> 6, ec = t & 63;
  double gv[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) gv[q] = G[gram_at(er + 4 * q, ec)];
  const double gjj = G[gram_at(ec, ec)];
  if (pass == 2) {
    // the panel's top block (Q1's) into M3, R1 into M2
    double pv[16], rv[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      pv[q] = (double)P[(int64_t)(er + 4 * q) * ld + ec];
      rv[q] = Rc[(er + 4 * q) * kNb + ec];
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      M3[er + 4 * q][ec] = pv[q];
      M2[er + 4 * q][ec] = rv[q];
    }
  }
  if (t == 0) bad_s = 0;
  if (pass == 1) {
    __syncthreads();
    if (t < kNb) {
      const double dj = sqrt(gjj > 0.0 ? gjj : 0.0);
      dsc[t] = dj;
      rdsc[t] = dj > 0.0 ? 1.0 / dj : 0.0;
      if (!(dj > 0.0)) bad_s = 1;
    }
    __syncthreads();
    const double rj = rdsc[ec];
#pragma unroll
    for (int q = 0; q < 16; ++q) M0[er + 4 * q][ec] = gv[q] * rdsc[er + 4 * q] * rj;
  } else {
#pragma unroll
    for (int q = 0; q < 16; ++q) M0[er + 4 * q][ec] = gv[q];
  }
  __syncthreads();
  double mn = 1e300, mx = 0.0;  // pivots, uniform on wavefront 0
  bool ok = !bad_s;
  for (int kb = 0; kb < kBlocks + (pass == 2 ? 1 : 0) && ok; ++kb) {
    const int k0 = kb * kB;
    if (w == 0 && kb < kBlocks) {
      bool bad = false;
      chol_panel(M0, kb, lane, &mn, &mx, &bad, pass == 1 && kb > 0 ? &Z[kb] : nullptr);
      if (lane == 0) {
        if (bad) bad_s = 1;
        ext[0] = mn;
        ext[1] = mx;
      }
    }
    if (pass == 1) {
      if (w == 1 && kb == 1) diag_inverse(M0, 0, Z[0], lane);
    } else {
      if (w == 1 && kb > 0) recon_panel(M3, M0, kb - 1, lane, sg, tj, Z[kBlocks - 1]);
      if (w == 2 && kb > 1) diag_inverse(M3, k0 - 2 * kB, Z[kb - 2], lane);
      if (w == 3 && kb == kBlocks) upper_product(M0, M2, lane);
    }
    __syncthreads();
    ok = !bad_s;
    // the trailing blocks of the Cholesky block row just formed (upper tiles, all
    // that is read) and of the panel just reconstructed
    const int nt = kBlocks - 1 - kb;  // tile rows right of block row kb
    int q = w;
    for (int ti = 0; ti < nt; ++ti)
      for (int tc = ti; tc < nt; ++tc, q = q == 0 ? 3 : q - 1)
        if (q == 0)
          rank16_tile<true>(&M0[k0 + kB][k0 + kB], &M0[k0][k0 + kB], &M0[k0][k0 + kB], ti, tc, lane);
    if (pass == 2 && kb > 0 && kb < kBlocks)
      for (int e = 0; e < (nt + 1) * (nt + 1); ++e, q = q == 0 ? 3 : q - 1)
        if (q == 0)
          rank16_tile<false>(&M3[k0][k0], &M3[k0][k0 - kB], &M3[k0 - kB][k0], e / (nt + 1), e % (nt + 1), lane);
    if (kb < kBlocks - 1 + (pass == 2 ? 1 : 0)) __syncthreads();
  }
  if (!ok || !(ext[0] >= min_pivot_ratio * ext[1])) {
    if (t == 0) *status = pass;
    return;
  }
  // the inverse's block column w, and 16 elements a thread of the rest
  const int lr = lane & 15, lk = lane >> 4;
  v4d wc[kBlocks];
  if (pass == 1) {
    upper_inverse_col(M0, Z, w, lane, wc);  // U^{-1}
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int i = er + 4 * q;
      Rc[i * kNb + ec] = i <= ec ? M0[i][ec] * dsc[ec] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < kBlocks; ++k)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * k + lk + 4 * r;
        Wk[i * kNb + 16 * w + lr] = wc[k][r] * rdsc[i];
      }
    return;
  }
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int i = er + 4 * q;
    const double a = sg[i] * M2[i][ec], b = M3[i][ec];
    P[(int64_t)i * ld + ec] = (TS)(i <= ec ? a : b);
  }
  if (t < kNb) tau[t] = (TS)tj[t];
  upper_inverse_col(M3, Z, w, lane, wc);  // U~^{-1} (above the diagonal blocks M3 holds U~)
#pragma unroll
  for (int k = 0; k < kBlocks; ++k)
#pragma unroll
    for (int r = 0; r < 4; ++r) Wk[(16 * k + lk + 4 * r) * kNb + 16 * w + lr] = wc[k][r];
}

// A operands of P W for one row: lane (lr, lk) of a wavefront takes row lr of
// a 16-row group, and step t of the product's K range one of its columns,
// kcol(t, lk): with E = 16 / sizeof(TS), step t takes column 4E (t / E) + E lk +
// t % E, so that the lane reads E adjacent columns at a time, by one 16-byte load
// where the row start and ld allow it (V16) and one by one otherwise; the K order,
// and so every bit of the product, is the same.  The four lanes of a step hold four
// distinct columns inside the 4E-column chunk of the step, all 64 columns are covered
// once, and the steps t < 4 (q + 1) hold every column <= 16 q + 15.
template <typename TS>
__device__ __forceinline__ int kcol(int t, int lk) {
  constexpr int E = 16 / (int)sizeof(TS);
  return 4 * E * (t / E) + E * lk + t % E;
}
template <typename TS, bool V16>
__device__ __forceinline__ void load_arow(double (&a)[16], const TS* __restrict__ row, int lk, bool in) {
  if constexpr (V16 && sizeof(TS) == 8) {
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const double2 v = *(const double2*)(row + 8 * m + 2 * lk);
      a[2 * m] = in ? v.x : 0.0;
      a[2 * m + 1] = in ? v.y : 0.0;
    }
  } else if constexpr (V16) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const float4 v = *(const float4*)(row + 16 * m + 4 * lk);
      a[4 * m] = in ? (double)v.x : 0.0;
      a[4 * m + 1] = in ? (double)v.y : 0.0;
      a[4 * m + 2] = in ? (double)v.z : 0.0;
      a[4 * m + 3] = in ? (double)v.w : 0.0;
    }
  } else {
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const double v = (double)row[kcol<TS>(t, lk)];
      a[t] = in ? v : 0.0;
    }
  }
}
// D = A W for a 16-row group, W upper triangular (zeros below its diagonal
// are skipped: tile q's K range stops at column 16 q + 15).  Accumulator
// register r of tile q holds D[lk + 4 r][16 q + lr].
template <typename TS>
__device__ __forceinline__ void group_times_upper(const double (&a)[16], const double (*Ws)[kNb + 1], int lr, int lk,
                                                  v4d (&acc)[4]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    const int kk = kcol<TS>(t, lk);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (t < 4 * (q + 1)) acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t], Ws[kk][16 * q + lr], acc[q], 0, 0, 0);
  }
}

// Rows [r_begin, M) of P <- P W (W 64 x 64 upper triangular) on the matrix
// cores, in place: wave w of a block takes 16 rows, reads all 64 of their
// columns (A operands, in registers) before it writes them.  Runs when
// *status == 0.
template <typename TS, bool V16>
__global__ void __launch_bounds__(256) k_cq_apply(TS* __restrict__ P, int64_t ld, int64_t r_begin, int64_t M,
                                                  const double* __restrict__ W, const int* __restrict__ status) {
  if (*status) return;
  __shared__ double Ws[kNb][kNb + 1];
  const int t = threadIdx.x;
  const int lane = t & 63, w = t >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const int64_t rbase = r_begin + (int64_t)blockIdx.x * 64 + 16 * w;
  const int64_t ra = rbase + lr;
  const int64_t rc = ra < M ? ra : M - 1;  // rows past M: row M - 1, replaced by zeros
  double a[16];
  load_arow<TS, V16>(a, P + rc * ld, lk, ra < M);
#pragma unroll
  for (int q = 0; q < kNb * kNb / 256; ++q) Ws[(t >> 6) + 4 * q][t & 63] = W[t + 256 * q];
  __syncthreads();
  v4d acc[4];
  group_times_upper<TS>(a, Ws, lr, lk, acc);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t row = rbase + lk + 4 * r;
    if (row < M)
#pragma unroll
      for (int q = 0; q < 4; ++q) P[row * ld + 16 * q + lr] = (TS)acc[q][r];
  }
}

// First pass's apply fused with the second pass's Gram: rows
// [z S, (z + 1) S) of P (S = 64 NG) <- P W (W upper triangular; matrix cores,
// in place) and the partial Gram of the new rows.  Wave w takes NG groups of 16
// rows from z S + 16 NG w; a group's product tiles (D[lk + 4 r][16 q + lr] in
// register r of tile q) are already the Gram's operands for K-step r.  The
// waves' Gram tiles are added in wave order through LDS.  Runs when
// *status == 0.
template <typename TS, bool V16, int NG>
__global__ void __launch_bounds__(256) k_cq_apply_gram(TS* __restrict__ P, int64_t ld, int64_t M,
                                                       const double* __restrict__ W, double* __restrict__ Gpart,
                                                       const int* __restrict__ status) {
  if (*status) return;
  __shared__ double S[4 * kGramLen];
  double(*Ws)[kNb + 1] = (double(*)[kNb + 1])S;
  const int t = threadIdx.x;
  const int lane = t & 63, w = t >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  // the four groups' operands loaded first (rows past M read row M - 1 and
  // are replaced by zeros, so the loads carry no branch)
  double ag[NG][16];
#pragma unroll
  for (int grp = 0; grp < NG; ++grp) {
    const int64_t ra = (int64_t)blockIdx.x * (64 * NG) + 16 * NG * w + 16 * grp + lr;
    const int64_t rc = ra < M ? ra : M - 1;
    load_arow<TS, V16>(ag[grp], P + rc * ld, lk, ra < M);
  }
#pragma unroll
  for (int q = 0; q < kNb * kNb / 256; ++q) Ws[(t >> 6) + 4 * q][t & 63] = W[t + 256 * q];
  __syncthreads();
  v4d gacc[10];
#pragma unroll
  for (int q = 0; q < 10; ++q) gacc[q] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int grp = 0; grp < NG; ++grp) {
    const int64_t rbase = (int64_t)blockIdx.x * (64 * NG) + 16 * NG * w + 16 * grp;
    v4d acc[4];
    group_times_upper<TS>(ag[grp], Ws, lr, lk, acc);
    if constexpr (sizeof(TS) < sizeof(double)) {
      // the Gram below is of the rows as stored
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[q][r] = (double)(TS)acc[q][r];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = rbase + lk + 4 * r;
      if (row < M)
#pragma unroll
        for (int q = 0; q < 4; ++q) P[row * ld + 16 * q + lr] = (TS)acc[q][r];
    }
    // rows past M hold exact zeros (zero operands) and add nothing
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int tile = 0;
#pragma unroll
      for (int a2 = 0; a2 < 4; ++a2)
#pragma unroll
        for (int b = a2; b < 4; ++b, ++tile)
          gacc[tile] = __builtin_amdgcn_mfma_f64_16x16x4f64(acc[a2][r], acc[b][r], gacc[tile], 0, 0, 0);
    }
  }
  __syncthreads();  // every wavefront is done with Ws
  sum_tiles(gacc, S, Gpart + (int64_t)blockIdx.x * kGramLen);
}

}  // namespace

// Partial Grams of an M-row panel.
static int64_t cq_nslab(int64_t M) { return (M + slab_rows(M) - 1) / slab_rows(M); }

int64_t cholqr_workspace_doubles(int64_t M) {
  // room for the most partials of any panel of at most M rows
  const int64_t ms = M < kShortPanelRows - 1 ? M : kShortPanelRows - 1;
  const int64_t a = cq_nslab(M), b = cq_nslab(ms);
  return (a > b ? a : b) * kNb * kNb + 3 * kNb * kNb + 64;
}

// Enqueues CholeskyQR2 and the reconstruction on the 64-column panel P
// (M >= 64 rows, stored as TS, all arithmetic in float64); ws holds
// cholqr_workspace_doubles(M) doubles.  A pass whose Cholesky pivot ratio falls
// below min_ratio1 (first pass) or min_ratio2 (second) sets the status.  The
// caller then launches the unblocked kernel gated on *status != 0, with R1
// (cholqr_r1).
template <typename TS>
static rfmls_status cholqr_panel(rfmls_handle* h, TS* P, int64_t ld, int64_t M, TS* tau, double* ws, int* status,
                                 double min_ratio1, double min_ratio2) {
  hipStream_t st = h->stream;
  const int64_t nslab = cq_nslab(M);
  const bool tall = slab_rows(M) == kSlab;
  // G, Wk and Rc sit after the most partials any panel of this QR writes
  double* Gpart = ws;
  double* G = ws + (cholqr_workspace_doubles(M) - 3 * kNb * kNb - 64);
  double* Wk = G + kNb * kNb;
  double* Rc = Wk + kNb * kNb;
  if (tall)
    hipLaunchKernelGGL((k_cq_gram<TS, 4>), dim3((unsigned)nslab), dim3(256), 0, st, (const TS*)P, ld, M, Gpart,
                       (const int*)nullptr);
  else
    hipLaunchKernelGGL((k_cq_gram<TS, 2>), dim3((unsigned)nslab), dim3(256), 0, st, (const TS*)P, ld, M, Gpart,
                       (const int*)nullptr);
  hipLaunchKernelGGL(k_cq_reduce, dim3(kGramLen / 16), dim3(256), 0, st, (const double*)Gpart, (int)nslab, G, status,
                     1);
  hipLaunchKernelGGL(k_cq_factor<TS>, dim3(1), dim3(256), 0, st, (const double*)G, Wk, Rc, P, ld, tau, status, 1,
                     min_ratio1);
  // 16-byte operand loads when every row start allows them
  const bool v16 = ld % (16 / (int64_t)sizeof(TS)) == 0 && reinterpret_cast<uintptr_t>(P) % 16 == 0;
  if (v16 && tall)
    hipLaunchKernelGGL((k_cq_apply_gram<TS, true, 4>), dim3((unsigned)nslab), dim3(256), 0, st, P, ld, M,
                       (const double*)Wk, Gpart, (const int*)status);
  else if (v16)
    hipLaunchKernelGGL((k_cq_apply_gram<TS, true, 2>), dim3((unsigned)nslab), dim3(256), 0, st, P, ld, M,
                       (const double*)Wk, Gpart, (const int*)status);
  else if (tall)
    hipLaunchKernelGGL((k_cq_apply_gram<TS, false, 4>), dim3((unsigned)nslab), dim3(256), 0, st, P, ld, M,
                       (const double*)Wk, Gpart, (const int*)status);
  else
    hipLaunchKernelGGL((k_cq_apply_gram<TS, false, 2>), dim3((unsigned)nslab), dim3(256), 0, st, P, ld, M,
                       (const double*)Wk, Gpart, (const int*)status);
  hipLaunchKernelGGL(k_cq_reduce, dim3(kGramLen / 16), dim3(256), 0, st, (const double*)Gpart, (int)nslab, G, status,
                     0);
  hipLaunchKernelGGL(k_cq_factor<TS>, dim3(1), dim3(256), 0, st, (const double*)G, Wk, Rc, P, ld, tau, status, 2,
                     min_ratio2);
  if (M > kNb) {
    const dim3 grid((unsigned)((M - kNb + 63) / 64));
    if (v16)
      hipLaunchKernelGGL((k_cq_apply<TS, true>), grid, dim3(256), 0, st, P, ld, (int64_t)kNb, M, (const double*)Wk,
                         (const int*)status);
    else
      hipLaunchKernelGGL((k_cq_apply<TS, false>), grid, dim3(256), 0, st, P, ld, (int64_t)kNb, M, (const double*)Wk,
                         (const int*)status);
  }
  RFMLS_HIP(h, hipGetLastError());
  return RFMLS_OK;
}

rfmls_status run_cholqr_panel(rfmls_handle* h, double* P, int64_t ld, int64_t M, double* tau, double* ws,
                              int* status, double min_ratio1, double min_ratio2) {
  return cholqr_panel<double>(h, P, ld, M, tau, ws, status, min_ratio1, min_ratio2);
}
rfmls_status run_cholqr_panel(rfmls_handle* h, float* P, int64_t ld, int64_t M, float* tau, double* ws, int* status,
                              double min_ratio1, double min_ratio2) {
  return cholqr_panel<float>(h, P, ld, M, tau, ws, status, min_ratio1, min_ratio2);
}

const double* cholqr_r1(const double* ws, int64_t M) {
  return ws + (cholqr_workspace_doubles(M) - 3 * kNb * kNb - 64) + 2 * kNb * kNb;
}

}  // namespace rfmls
