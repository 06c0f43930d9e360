// CSSVDP-LSQR preconditioner (Alg. 2 step 3): the truncated SVD of the sketch
// SA through its R factor (SA = Q R, so SA and R share Sigma and V), and
// P = V_r Sigma_r^{-1} with r = #{sigma_i > rcond sigma_1} (Sec. 3.2: the
// LAPACK-style threshold, rcond times the largest singular value).
//
// SVD of R by one-sided (Hestenes) Jacobi, preconditioned by a second QR
// (Drmac and Veselic): R^T = Q2 R2, and plane rotations J applied on the right
// make the columns of M = R2^T J mutually orthogonal, so M = U Sigma with
// sigma_k = ||M_k||, and R = U Sigma (Q2 J)^T: V = Q2 J.  The rotations are
// accumulated, and P = Q2 J Sigma^{-1} is formed from them rather than from the
// normalised columns: R P = M Sigma^{-1} then has orthonormal columns to the
// stopping tolerance however wide the spread of sigma, so SA P = Q U keeps the
// conditioning Thm 3.4 relies on.
//
// Ordering: columns in groups of 32; a sweep first rotates the pairs inside every
// group and then takes the round-robin (circle) schedule over the groups, Gp = the
// group count rounded up to even: each of its Gp - 1 steps gives Gp / 2 disjoint
// group pairs, whose 32 x 32 cross pairs are rotated.  A step works on 64-column
// blocks through their Gram matrices, three launches for all blocks at once:
//   k_jac_gram   G = X^T X of a block's 64 columns X (split over rows);
//   k_jac_solve  the rotations, from G alone: W = product of the rotations of 32
//                rounds of 32 disjoint pairs;
//   k_jac_apply  X <- X W for the block's columns of M and of J.
// At most 32 columns, one group, take their sweeps in one launch (k_jac_small).
// A pair (p, q) is rotated when |m_p . m_q| > tol ||m_p|| ||m_q||; the sweeps stop
// when a sweep, whose every block starts from a fresh Gram, rotates none.
// Against rotating 8 columns at a time in registers (a step per 4-column group
// pair): the same rotations in an eighth of the passes over M and J, their
// products on the matrix cores, and no block-wide reduction over n rows per
// round.  Measured at n = 1,600 (31,360 x 1,600 Helmholtz system): 16 sweeps of 399
// steps of 52 us before; 13 or 14 sweeps of 50 steps of 11 (Gram) + 25 (rotations)
// + 19 us (apply, 4.3 TB/s) now, whole CSSVDP solve 340 -> 53 ms.
//
// Layout: M and J column-major (column k contiguous, ld = ldm), columns and rows
// padded with zeros to whole groups and 32-row tiles; float64 throughout.
#include <cmath>
#include <cstring>
#include <type_traits>

#include "common.h"

namespace rfmls {
namespace {

// out[c * ldo + r] = in[r * ldi + c] * (rowscale ? rowscale[r] : 1), an LDS-tiled
// transpose of a rows x cols matrix; with order, row r is read from row order[r]
constexpr int kTr = 32;
__global__ void __launch_bounds__(kTr * 8)
    k_transpose_scale(const double* __restrict__ in, int64_t ldi, int64_t rows, int64_t cols,
                      const double* __restrict__ rowscale, const int32_t* __restrict__ order,
                      double* __restrict__ out, int64_t ldo) {
  __shared__ double t[kTr][kTr + 1];
  const int64_t r0 = (int64_t)blockIdx.y * kTr, c0 = (int64_t)blockIdx.x * kTr;
  const int tx = threadIdx.x % kTr, ty = threadIdx.x / kTr;
  for (int k = ty; k < kTr; k += 8) {
    const int64_t r = r0 + k, c = c0 + tx;
    double v = 0.0;
    if (r < rows && c < cols) v = in[(order ? (int64_t)order[r] : r) * ldi + c] * (rowscale ? rowscale[r] : 1.0);
    t[k][tx] = v;
  }
  __syncthreads();
  for (int k = ty; k < kTr; k += 8) {
    const int64_t c = c0 + k, r = r0 + tx;
    if (r < rows && c < cols) out[c * ldo + r] = t[tx][k];
  }
}

// rank[i] = place of row i of R (n x n, upper triangular, row-major) by descending
// norm, ties by index; the norms' bit patterns order them (NaN first).
__global__ void __launch_bounds__(256)
    k_row_norms(const double* __restrict__ R, int64_t n, unsigned long long* __restrict__ nb) {
  __shared__ double scratch[256 / 64];
  const int64_t i = blockIdx.x;
  double s = 0.0;
  for (int64_t j = i + threadIdx.x; j < n; j += 256) s += R[i * n + j] * R[i * n + j];
  s = block_sum(s, scratch);
  if (threadIdx.x == 0) nb[i] = (unsigned long long)__double_as_longlong(fabs(s));
}
__global__ void __launch_bounds__(256)
    k_norm_order(const unsigned long long* __restrict__ nb, int64_t n, int32_t* __restrict__ order) {
  __shared__ unsigned long long t[256];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const unsigned long long mine = i < n ? nb[i] : 0ull;
  int32_t rank = 0;
  for (int64_t j0 = 0; j0 < n; j0 += 256) {
    __syncthreads();
    if (j0 + threadIdx.x < n) t[threadIdx.x] = nb[j0 + threadIdx.x];
    __syncthreads();
    const int lim = (int)(n - j0 < 256 ? n - j0 : 256);
    for (int k = 0; k < lim; ++k) rank += (t[k] > mine || (t[k] == mine && j0 + k < i)) ? 1 : 0;
  }
  if (i < n) order[rank] = (int32_t)i;
}

// M[k ldm + i] = R2[k][i] for i >= k, else 0: column k of L = R2^T is row k of
// the upper-triangular R2 (row-major, ld2); zeros in the padding (ncp columns)
__global__ void k_upper_rows_to_cols(const double* __restrict__ R2, int64_t ld2, int64_t n, int64_t ncp,
                                     double* __restrict__ M, int64_t ldm) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < ncp * ldm;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = e / ldm, i = e % ldm;
    M[e] = (k < n && i < n && i >= k) ? R2[k * ld2 + i] : 0.0;
  }
}

__global__ void k_eye_cols(double* __restrict__ J, int64_t n, int64_t ldm) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n * ldm;
       e += (int64_t)gridDim.x * blockDim.x)
    J[e] = (e / ldm == e % ldm) ? 1.0 : 0.0;
}

// counters of one sweep over more than one group: [0] = bits of the largest |cos| met, [1] = rotations,
// [2] = blocks that rotated (and so wrote their columns of M and J)
__global__ void k_zero_counters(unsigned long long* ctr) {
  if (threadIdx.x < 3) ctr[threadIdx.x] = 0ull;
}

// group of step t at slot `slot` in the circle schedule over Gp groups: slot 0
// stays, the others turn
__device__ __forceinline__ int64_t circle(int64_t slot, int64_t t, int64_t Gp) {
  return slot == 0 ? 0 : (slot - 1 + t) % (Gp - 1) + 1;
}

typedef double v4d __attribute__((ext_vector_type(4)));
typedef double d2v __attribute__((ext_vector_type(2)));

constexpr int kJb = 32;         // columns per group
constexpr int kJw = 2 * kJb;    // columns per block
constexpr int kSolveWaves = 4;  // wavefronts of k_jac_solve
constexpr int kGramRows = 64;   // rows a workgroup's four wavefronts take per step

// First columns of block `blk`'s two groups in step t of a sweep: t < 0 is the
// step inside the groups (neighbouring groups share a block), t >= 0 the circle
// schedule's step t.
__device__ __forceinline__ void jac_block(int64_t blk, int64_t t, int64_t Gp, int64_t* c1, int64_t* c2) {
  *c1 = kJb * (t < 0 ? 2 * blk : circle(blk, t, Gp));
  *c2 = kJb * (t < 0 ? 2 * blk + 1 : circle(Gp - 1 - blk, t, Gp));
}

// Partial Gram of block blockIdx.y's 64 columns over rows [z rows, (z + 1) rows),
// z = blockIdx.x (rows a multiple of kGramRows, the padding rows are zeros): ten
// upper 16 x 16 tiles on the matrix cores, every fourth 16-row step to a
// wavefront, operands straight from M with the K order permuted (lane (lr, lk)
// reads rows 4 lk .. 4 lk + 3 of column lr: 128 contiguous bytes per column and
// step).  The wavefronts' tiles are added in order through LDS and the full
// symmetric 64 x 64 partial is written.  Bound by reading M once per step.
__global__ void __launch_bounds__(256)
    k_jac_gram(const double* __restrict__ M, int64_t ldm, int64_t Gp, int64_t t, int64_t rows,
               double* __restrict__ part) {
  __shared__ double S[4][10][4][64];  // wavefront, tile, register, lane
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  int64_t c1, c2;
  jac_block(blockIdx.y, t, Gp, &c1, &c2);
  const int64_t r0 = (int64_t)blockIdx.x * rows, r1 = r0 + rows < ldm ? r0 + rows : ldm;
  const double* col[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) col[g] = M + ((g < 2 ? c1 + 16 * g : c2 + 16 * (g - 2)) + lr) * ldm + 4 * lk;
  v4d acc[10];
#pragma unroll
  for (int q = 0; q < 10; ++q) acc[q] = v4d{0.0, 0.0, 0.0, 0.0};
  for (int64_t r = r0 + 16 * w; r < r1; r += kGramRows) {
    double a[4][4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const d2v x = *(const d2v*)(col[g] + r), y = *(const d2v*)(col[g] + r + 2);
      a[g][0] = x[0];
      a[g][1] = x[1];
      a[g][2] = y[0];
      a[g][3] = y[1];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int tile = 0;
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = p; q < 4; ++q, ++tile)
          acc[tile] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[p][j], a[q][j], acc[tile], 0, 0, 0);
    }
  }
#pragma unroll
  for (int q = 0; q < 10; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) S[w][q][r][lane] = acc[q][r];
  __syncthreads();
  // wavefront w adds the four sums of register w of every tile
  double* o = part + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * (kJw * kJw);
  {
    int tile = 0;
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int q = p; q < 4; ++q, ++tile) {
        const double v = ((S[0][tile][w][lane] + S[1][tile][w][lane]) + S[2][tile][w][lane]) + S[3][tile][w][lane];
        const int i = 16 * p + lk + 4 * w, j = 16 * q + lr;
        o[i * kJw + j] = v;
        if (p != q) o[j * kJw + i] = v;
      }
  }
}

// v of lane (lane ^ mask) within 32 lanes, on the DPP path where it has the pattern
template <int MASK>
__device__ __forceinline__ double lane_xor(double v) {
  if constexpr (MASK == 1) return dpp_move<0xB1>(v);         // quad_perm(1, 0, 3, 2)
  else if constexpr (MASK == 2) return dpp_move<0x4E>(v);    // quad_perm(2, 3, 0, 1)
  else if constexpr (MASK == 7) return dpp_move<0x141>(v);   // row_half_mirror
  else if constexpr (MASK == 15) return dpp_move<0x140>(v);  // row_mirror
  else return __shfl_xor(v, MASK, 64);
}

// 1 / sqrt(x), x in [2^-4, 2^4], from the hardware's estimate (2^-24) by one third-order
// step, the rounding of x y taken out of 1 - x y^2: the last rounding is what is left.
__device__ __forceinline__ double rsqrt3(double x) {
  const double y = __builtin_amdgcn_rsq(x), h = x * y;
  const double e = fma(-fma(x, y, -h), y, fma(-h, y, 1.0));
  return fma(y * e, fma(e, 0.375, 0.5), y);
}
__device__ __forceinline__ int exp_of(double x) { return __builtin_amdgcn_frexp_exp(x); }

// The rotation of a pair from aa = ||x_p||^2, bb = ||x_q||^2, ab = x_p . x_q:
// [c s; -s c] on (x_p, x_q) that zeroes x_p . x_q: t = s / c the root of smaller
// magnitude of t^2 + 2 zeta t - 1 = 0, zeta = (bb - aa) / (2 ab), as
// t = sign(d) e / (|d| + sqrt(d^2 + e^2)) with d = bb - aa and e = 2 ab.  Identity (and
// false) when |ab| <= tol ||x_p|| ||x_q||.  d and e, and aa, bb and ab for the cosine,
// are first scaled by powers of two, so that neither columns hundreds of decades apart
// nor subnormal products leave the range of the square roots.  The chain of dependent
// operations is what a round waits for, so roots and quotient are hardware estimates
// refined in the open, the last root and the quotient by their own residuals, instead of
// the library's sequences, and lose nothing to them: over 4 M pairs up to 290 decades
// apart |t|, c, s and the cosine are off by at most 3.5, 1.8, 4.4 and 2.2 u, the same
// formula by the library's square roots and divisions by 4.6, 2.4, 5.8 and 3.4 (CSSVDP
// solve at 1,600 columns: 53.4 ms, 58.1 with those).
__device__ __forceinline__ bool jac_rotation(double aa, double bb, double ab, double tol, double* cs, double* sn,
                                             double* tn, double* rel_out) {
  const bool some = aa > 0.0 && bb > 0.0;
  const int ka = exp_of(aa) >> 1, kb = exp_of(bb) >> 1;
  const double sab = ldexp(aa, -2 * ka) * ldexp(bb, -2 * kb);  // in [1/4, 4)
  const double rel = some ? fabs(ldexp(ab, -ka - kb)) * rsqrt3(sab) : 0.0;
  *rel_out = rel;
  const bool go = rel > tol;
  const double d0 = go ? bb - aa : 1.0, e0 = go ? 2.0 * ab : 0.0;
  const int k = -exp_of(fmax(fabs(d0), fabs(e0)));
  const double d = fabs(ldexp(d0, k)), e = ldexp(d0 < 0.0 ? -e0 : e0, k);
  const double g = fma(d, d, e * e);  // in [1/4, 2)
  const double y = rsqrt3(g), h0 = g * y;
  const double den = d + fma(fma(-h0, h0, g), 0.5 * y, h0);  // d + sqrt(g), in [1/2, 5/2)
  const double v0 = __builtin_amdgcn_rcp(den), v = fma(fma(-den, v0, 1.0), v0, v0);
  const double q = e * v, t = fma(fma(-den, q, e), v, q);
  const double c = go ? rsqrt3(fma(t, t, 1.0)) : 1.0;
  *tn = t;
  *cs = c;
  *sn = c * t;
  return go;
}

// v + (v of the lane 32 away), on every lane
__device__ __forceinline__ double half_sum(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
         __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}

// The rotations of one block from its Gram G (the sum of nz partials in order),
// one workgroup per block.  With W the product of the
// rotations so far and H = G W, the rotated columns' product m_p . m_q is
// w_p . h_q, so only W's and H's columns are rotated (one-sided) and a round
// needs one sum over 64 rows per pair; the norms follow each rotation (no worse than
// summed from W and H again, 1e-15 to 6e-14 of their size either way, G's own rounding;
// a sweep without a rotation has only fresh sums in it).  Lane i of
// a half wavefront holds eight rows of column i (p) and of its partner (q) of W
// and H.
//   Cross step (t >= 0): p = i and q = 32 + (i ^ x); x runs over all 32 values in
//   Gray-code order over the basis 1, 2, 7, 15, 16, so the q columns move to their
//   next lanes by one DPP pattern a round.
//   Inside the groups (t < 0): both groups at once, pairs (i, i ^ x), x = 1 .. 31,
//   each lane forming its own column of the pair.
// Bound by the 32 rounds' chain (a 64-row sum over LDS with one barrier, then the
// rotation's scalar chain): 44 us with eight wavefronts, library square roots and
// divisions and one partial Gram's loads in flight, 25 us now; W goes to Wout, and moved[block] tells
// whether any pair was rotated.
__global__ void __launch_bounds__(64 * kSolveWaves)
    k_jac_solve(const double* __restrict__ part, int nz, int64_t t, double tol, double* __restrict__ Wout,
                int* __restrict__ moved, unsigned long long* __restrict__ ctr) {
  constexpr int NR = kJw / (2 * kSolveWaves);  // rows a half wavefront holds
  __shared__ double buf[2][kSolveWaves][2][kJb];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = lane & 31;
  const int row0 = 2 * NR * w + NR * (lane >> 5);
  const double* G = part + (int64_t)blockIdx.x * nz * (kJw * kJw);
  double wp[NR], wq[NR], hp[NR], hq[NR];
  double aa = 0.0, bb = 0.0;
#pragma unroll
  for (int k = 0; k < NR; ++k) hp[k] = hq[k] = 0.0;
#pragma unroll 4
  for (int z = 0; z < nz; ++z) {  // several partials' loads in flight
    const double* Gz = G + (int64_t)z * (kJw * kJw);
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      hp[k] += Gz[(row0 + k) * kJw + i];
      hq[k] += Gz[(row0 + k) * kJw + kJb + i];
    }
    aa += Gz[i * kJw + i];
    bb += Gz[(kJb + i) * kJw + kJb + i];
  }
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    wp[k] = row0 + k == i ? 1.0 : 0.0;
    wq[k] = row0 + k == kJb + i ? 1.0 : 0.0;
  }
  // pairwise sums, short chains: over a lane's rows, and over the wavefronts
  auto row_dot = [](const double (&a)[NR], const double (&b)[NR]) {
    double p[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) p[k] = a[k] * b[k];
#pragma unroll
    for (int o = NR / 2; o > 0; o >>= 1)
#pragma unroll
      for (int k = 0; k < o; ++k) p[k] += p[k + o];
    return p[0];
  };
  auto wave_total = [](const double (&b)[kSolveWaves][2][kJb], int which, int c) {
    double p[kSolveWaves];
#pragma unroll
    for (int k = 0; k < kSolveWaves; ++k) p[k] = b[k][which][c];
#pragma unroll
    for (int o = kSolveWaves / 2; o > 0; o >>= 1)
#pragma unroll
      for (int k = 0; k < o; ++k) p[k] += p[k + o];
    return p[0];
  };
  double offmax = 0.0;
  int nrot = 0, x = 0;
  if (t >= 0) {
    auto round = [&](int par) {
      const double dot = half_sum(row_dot(wp, hq));
      if (lane < kJb) buf[par][w][0][i] = dot;
      __syncthreads();
      const double ab = wave_total(buf[par], 0, i);
      double cs, sn, tn, rel;
      if (jac_rotation(aa, bb, ab, tol, &cs, &sn, &tn, &rel)) ++nrot;
      offmax = rel > offmax ? rel : offmax;
      aa -= tn * ab;
      bb += tn * ab;
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        const double a = wp[k], b = wq[k], c = hp[k], d = hq[k];
        wp[k] = cs * a - sn * b;
        wq[k] = sn * a + cs * b;
        hp[k] = cs * c - sn * d;
        hq[k] = sn * c + cs * d;
      }
    };
    auto turn = [&](auto mask) {
      constexpr int kM = decltype(mask)::value;
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        wq[k] = lane_xor<kM>(wq[k]);
        hq[k] = lane_xor<kM>(hq[k]);
      }
      bb = lane_xor<kM>(bb);
      x ^= kM;
    };
    for (int o = 0; o < 4; ++o) {
      round(0);
      turn(std::integral_constant<int, 1>());
      round(1);
      turn(std::integral_constant<int, 2>());
      round(0);
      turn(std::integral_constant<int, 1>());
      round(1);
      turn(std::integral_constant<int, 7>());
      round(0);
      turn(std::integral_constant<int, 1>());
      round(1);
      turn(std::integral_constant<int, 2>());
      round(0);
      turn(std::integral_constant<int, 1>());
      round(1);
      if (o == 1) turn(std::integral_constant<int, 16>());
      else if (o != 3) turn(std::integral_constant<int, 15>());
    }
  } else {
    for (int m = 1; m < kJb; ++m) {
      const int par = m & 1;
      double pw[NR], ph[NR], qw[NR], qh[NR];  // the partners' columns
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        pw[k] = __shfl_xor(wp[k], m, 64);
        ph[k] = __shfl_xor(hp[k], m, 64);
        qw[k] = __shfl_xor(wq[k], m, 64);
        qh[k] = __shfl_xor(hq[k], m, 64);
      }
      const double pa = __shfl_xor(aa, m, 64), pb = __shfl_xor(bb, m, 64);
      const bool low = (i ^ m) > i;
      // both lanes of a pair read the lower column's sum
      const double d1 = half_sum(row_dot(wp, ph)), d2 = half_sum(row_dot(wq, qh));
      if (lane < kJb) {
        buf[par][w][0][i] = d1;
        buf[par][w][1][i] = d2;
      }
      __syncthreads();
      const int il = low ? i : i ^ m;
      const double ab1 = wave_total(buf[par], 0, il), ab2 = wave_total(buf[par], 1, il);
      auto own = [&](double (&ow)[NR], double (&oh)[NR], const double (&tw)[NR], const double (&th)[NR], double& on,
                     double tnorm, double ab) {
        double cs, sn, tn, rel;
        if (jac_rotation(low ? on : tnorm, low ? tnorm : on, ab, tol, &cs, &sn, &tn, &rel) && low) ++nrot;
        offmax = rel > offmax ? rel : offmax;
        on += low ? -tn * ab : tn * ab;
        const double s = low ? -sn : sn;
#pragma unroll
        for (int k = 0; k < NR; ++k) {
          ow[k] = cs * ow[k] + s * tw[k];
          oh[k] = cs * oh[k] + s * th[k];
        }
      };
      own(wp, hp, pw, ph, aa, pa, ab1);
      own(wq, hq, qw, qh, bb, pb, ab2);
    }
  }
  double* Wb = Wout + (int64_t)blockIdx.x * (kJw * kJw);
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    Wb[(row0 + k) * kJw + i] = wp[k];
    Wb[(row0 + k) * kJw + kJb + (i ^ x)] = wq[k];
  }
  // every wavefront has the same counts; the first reports them
  if (w == 0) {
    int nr = lane < kJb ? nrot : 0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      nr += __shfl_xor(nr, off, 64);
      const double o = __shfl_xor(offmax, off, 64);
      offmax = o > offmax ? o : offmax;
    }
    if (lane == 0) {
      moved[blockIdx.x] = nr;
      if (offmax > 0.0) atomicMax(&ctr[0], (unsigned long long)__double_as_longlong(offmax));
      if (nr) {
        atomicAdd(&ctr[1], (unsigned long long)nr);
        atomicAdd(&ctr[2], 1ull);
      }
    }
  }
}

// X <- X W on the 64 columns of block blockIdx.y of M (blockIdx.z = 0) and J (1),
// 32 rows a wavefront: lane (lr, lk) holds rows 2 lr, 2 lr + 1 of columns 4 s + lk
// (16-byte loads), all 64 columns read before any is written.  Output column
// j = 16 q + lk + 4 r of W^T X^T sits in accumulator register r.  Bound by reading
// and writing M and J once per step, with the matrix cores close behind.
__global__ void __launch_bounds__(256)
    k_jac_apply(double* __restrict__ M, double* __restrict__ J, int64_t ldm, int64_t Gp, int64_t t,
                const double* __restrict__ Wall, const int* __restrict__ moved) {
  if (moved[blockIdx.y] == 0) return;
  __shared__ double Ws[kJw][kJw + 2];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const double* W = Wall + (int64_t)blockIdx.y * (kJw * kJw);
  for (int e = tid; e < kJw * kJw; e += 256) Ws[e / kJw][e % kJw] = W[e];
  int64_t c1, c2;
  jac_block(blockIdx.y, t, Gp, &c1, &c2);
  double* X = blockIdx.z ? J : M;
  const int64_t r = (int64_t)blockIdx.x * 128 + 32 * w;
  const bool live = r < ldm;  // uniform per wavefront
  d2v x[16];
  if (live)
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const int k = 4 * s + lk;
      x[s] = *(const d2v*)(X + (s < 8 ? c1 + k : c2 + k - kJb) * ldm + r + 2 * lr);
    }
  __syncthreads();
  if (!live) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    v4d a0 = {0.0, 0.0, 0.0, 0.0}, a1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const double a = Ws[4 * s + lk][16 * q + lr];
      a0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, x[s][0], a0, 0, 0, 0);
      a1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, x[s][1], a1, 0, 0, 0);
    }
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int j = 16 * q + lk + 4 * rr;
      *(d2v*)(X + (j < kJb ? c1 + j : c2 + j - kJb) * ldm + r + 2 * lr) = d2v{a0[rr], a1[rr]};
    }
  }
}

// Up to `sweeps` sweeps over at most 32 columns (the one group there is) in one launch,
// by one workgroup that holds M and J in registers: thread (c, g) has rows 4 g .. 4 g + 3
// of column c.  Pairs (c, c ^ x), x = 1 .. w - 1, w a power of two that covers the
// columns; a round sums the pair's three products over LDS, from the columns themselves,
// and both columns' threads form the rotation.  Ends after a sweep without a rotation.
// ctr: the last sweep's largest |cos| and rotations, the sweeps, and how many rotated.
// Bound by the rounds' chain.  Against the three launches of each step of a sweep and a
// host wait for every sweep: 8 columns 0.69 -> 0.28 ms with the QRs, 32 columns 0.93 -> 0.50.
__global__ void __launch_bounds__(256)
    k_jac_small(double* __restrict__ M, double* __restrict__ J, int w, double tol, int sweeps,
                unsigned long long* __restrict__ ctr) {
  __shared__ double buf[2][8][2][kJb];
  const int c = threadIdx.x & (kJb - 1), g = threadIdx.x / kJb;
  double m[4], j[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    m[k] = M[c * kJb + 4 * g + k];
    j[k] = J[c * kJb + 4 * g + k];
  }
  double off = 0.0;
  int rotated = 0, sweep = 0, moving = 0, par = 0;
  while (sweep < sweeps) {
    ++sweep;
    rotated = 0;
    off = 0.0;
    for (int x = 1; x < w; ++x, par ^= 1) {
      double pm[4], pj[4];  // the partner's rows
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        pm[k] = __shfl_xor(m[k], x, 64);
        pj[k] = __shfl_xor(j[k], x, 64);
      }
      buf[par][g][0][c] = (m[0] * m[0] + m[1] * m[1]) + (m[2] * m[2] + m[3] * m[3]);
      buf[par][g][1][c] = (m[0] * pm[0] + m[1] * pm[1]) + (m[2] * pm[2] + m[3] * pm[3]);
      __syncthreads();
      const bool low = (c ^ x) > c;
      const int p = low ? c : c ^ x, q = low ? c ^ x : c;
      double aa = 0.0, bb = 0.0, ab = 0.0;
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        aa += buf[par][r][0][p];
        bb += buf[par][r][0][q];
        ab += buf[par][r][1][p];  // both columns' threads read the lower one's
      }
      double cs, sn, tn, rel;
      const bool go = jac_rotation(aa, bb, ab, tol, &cs, &sn, &tn, &rel);
      rotated += __popcll(__ballot(go && low)) / 2;  // (a wavefront holds every column twice)
      off = rel > off ? rel : off;
      const double s = low ? -sn : sn;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        m[k] = cs * m[k] + s * pm[k];
        j[k] = cs * j[k] + s * pj[k];
      }
    }
    if (rotated == 0) break;  // the same in every thread
    ++moving;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    M[c * kJb + 4 * g + k] = m[k];
    J[c * kJb + 4 * g + k] = j[k];
  }
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) {
    const double v = __shfl_xor(off, o, 64);
    off = v > off ? v : off;
  }
  if (threadIdx.x == 0) {
    ctr[0] = (unsigned long long)__double_as_longlong(off);
    ctr[1] = (unsigned long long)rotated;
    ctr[2] = (unsigned long long)sweep;
    ctr[3] = (unsigned long long)moving;
  }
}

// sigma[k] = ||M_k|| (fixed-order block sum), one block per column
__global__ void __launch_bounds__(256)
    k_col_norms(const double* __restrict__ M, int64_t n, int64_t ldm, double* __restrict__ sigma) {
  __shared__ double scratch[256 / 64];
  const int64_t k = blockIdx.x;
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 256) s += M[k * ldm + i] * M[k * ldm + i];
  s = block_sum(s, scratch);
  if (threadIdx.x == 0) sigma[k] = sqrt(s);
}

}  // namespace

int64_t svd_max_n() { return 16384; }

rfmls_status run_build_svd_precond(rfmls_handle* h, int64_t n, const double* SA, int64_t ld,
                                   rfmls_dtype store, double rcond, int max_sweeps,
                                   rfmls_precond_t* P) {
  if (n > svd_max_n())
    return fail(h, RFMLS_E_ARG, "SVD preconditioner: n = %lld exceeds %lld", (long long)n,
                (long long)svd_max_n());
  hipStream_t st = h->stream;
  P->n = n;
  P->nt = (n + kTile - 1) / kTile;
  P->store = store;
  P->full = 1;
  // R (normalised, row-major) kept for export, as for the QR preconditioner
  RFMLS_CHECK(run_extract_R(h, n, SA, ld, P));
  const int64_t ldm = (n + 31) / 32 * 32;  // 256-byte aligned columns, whole 32-row tiles
  // column groups of kJb, rounded up to an even count
  const int64_t Gn = (n + kJb - 1) / kJb;
  const int64_t Gp = Gn + (Gn & 1);
  const int64_t ncp = Gp * kJb, nblk = Gp / 2;
  // row chunks of the Gram products: about a workgroup per compute unit over the
  // blocks, at most 8 (each is one more partial for the rotations to add)
  int64_t nz = ((int64_t)h->num_cus + nblk - 1) / nblk;
  if (nz > 8) nz = 8;
  int64_t zrows = ((ldm + nz - 1) / nz + kGramRows - 1) / kGramRows * kGramRows;
  nz = (ldm + zrows - 1) / zrows;
  void* pw;
  RFMLS_CHECK(workspace(h, WS_SVD,
                        sizeof(double) * (2 * (size_t)ncp * ldm + (size_t)n + (size_t)(nz + 1) * nblk * kJw * kJw) +
                            64 + sizeof(int) * (size_t)nblk,
                        &pw));
  double* Mc = (double*)pw;
  double* Jc = Mc + (size_t)ncp * ldm;
  double* gram = Jc + (size_t)ncp * ldm;
  double* Wb = gram + (size_t)nz * nblk * kJw * kJw;
  double* d = Wb + (size_t)nblk * kJw * kJw;
  unsigned long long* ctr = (unsigned long long*)(d + n);
  int* moved = (int*)(ctr + 8);
  RFMLS_HIP(h, hipMalloc(&P->sigma, sizeof(double) * (size_t)n));
  // Preconditioning of the sweeps (Drmac and Veselic): the QR of R^T,
  // R^T = Q2 R2, gives R = R2^T Q2^T; Jacobi then runs on the columns of
  // L = R2^T (the rows of R2): L J = U Sigma, so R's right singular vectors are
  // V = Q2 J.  The QR's rotation towards triangular form leaves L closer to
  // orthogonal columns, and the cyclic sweeps need about a third fewer passes.
  const int64_t ld2 = (n + 127) / 128 * 128;
  void* p2;
  RFMLS_CHECK(workspace(h, WS_SVD2, sizeof(double) * ((size_t)n * ld2 + 3 * (size_t)n), &p2));
  double* Rt = (double*)p2;
  double* tau2 = Rt + (size_t)n * ld2;
  {
    dim3 g(ceil_div(n, kTr), ceil_div(n, kTr));
    // the rows of R by descending norm: (Pi R)^T = Q2 R2 leaves V = Q2 J as it is
    // (only U's rows are permuted), and sorted columns in the second QR bring
    // L nearer to orthogonal columns (15 -> 13 sweeps at 640 columns)
    unsigned long long* nb = (unsigned long long*)(tau2 + n);
    int32_t* order = (int32_t*)(nb + n);
    // (not for the few columns of k_jac_small: two launches for a sweep at most)
    if (n > kJb) {
      hipLaunchKernelGGL(k_row_norms, dim3((unsigned)n), dim3(256), 0, st, (const double*)P->Rdense, n, nb);
      hipLaunchKernelGGL(k_norm_order, dim3(ceil_div(n, 256)), dim3(256), 0, st, (const unsigned long long*)nb, n, order);
    }
    hipLaunchKernelGGL(k_transpose_scale, g, dim3(kTr * 8), 0, st, (const double*)P->Rdense, n, n, n,
                       (const double*)nullptr, (const int32_t*)(n > kJb ? order : nullptr), Rt, ld2);
    RFMLS_HIP(h, hipGetLastError());
  }
  RFMLS_CHECK(run_qr(h, n, n, ld2, RFMLS_F64, Rt, ld2, tau2));
  {
    int flag = 0;
    RFMLS_HIP(h, hipMemcpyAsync(&flag, h->dev_flags, sizeof(int), hipMemcpyDeviceToHost, st));
    RFMLS_HIP(h, hipStreamSynchronize(st));
    if (flag) {
      (void)hipMemset(h->dev_flags, 0, sizeof(int));
      return fail(h, RFMLS_E_HIP, "SVD preconditioner: QR panel hand-over timed out");
    }
  }
  {
    const unsigned g = ceil_div(ncp * ldm, 256) < 4096 ? ceil_div(ncp * ldm, 256) : 4096;
    hipLaunchKernelGGL(k_upper_rows_to_cols, dim3(g), dim3(256), 0, st, (const double*)Rt, ld2, n, ncp, Mc, ldm);
    hipLaunchKernelGGL(k_eye_cols, dim3(g), dim3(256), 0, st, Jc, ncp, ldm);
    RFMLS_HIP(h, hipGetLastError());
  }
  // stopping tolerance on |cos(m_p, m_q)|: a few units of the rounding of the
  // blocked dot products (LAPACK's one-sided Jacobi takes sqrt(n) eps)
  const double eps = 2.220446049250313e-16;
  const double tol = (sqrt((double)n) > 8.0 ? sqrt((double)n) : 8.0) * eps;
  unsigned long long* pin = (unsigned long long*)((char*)h->pinned + 3072);
  P->sweeps = 0;
  P->off = 0.0;
  bool converged = false;
  // the counters of a sweep (or of several in one launch)
  auto read_counters = [&](int words) -> rfmls_status {
    RFMLS_HIP(h, hipGetLastError());
    RFMLS_HIP(h, hipMemcpyAsync(pin, ctr, words * sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    RFMLS_HIP(h, hipStreamSynchronize(st));
    const unsigned long long bits = pin[0];
    memcpy(&P->off, &bits, sizeof(P->off));
    converged = pin[1] == 0ull;
    if (!(P->off == P->off)) return fail(h, RFMLS_E_BREAKDOWN, "SVD preconditioner: non-finite column products");
    return RFMLS_OK;
  };
  if (n <= kJb) {
    int w = 2;
    while (w < n) w *= 2;
    while (!converged && P->sweeps < max_sweeps) {
      const int most = max_sweeps - P->sweeps < 64 ? max_sweeps - P->sweeps : 64;
      {
        Trace tr(h, "svd_jacobi_sweep", 32.0 * (double)n * (double)n, 0.0);
        hipLaunchKernelGGL(k_jac_small, dim3(1), dim3(256), 0, st, Mc, Jc, w, tol, most, ctr);
      }
      RFMLS_CHECK(read_counters(4));
      P->sweeps += (int)pin[2];
      if (h->trace && !h->trace_recs.empty())
        h->trace_recs.back().flops = 9.0 * (double)n * (double)n * (double)n * (double)pin[3];
    }
  }
  while (n > kJb && !converged && P->sweeps < max_sweeps) {
    hipLaunchKernelGGL(k_zero_counters, dim3(1), dim3(64), 0, st, ctr);
    {
      // (bytes and flops set below from the sweep's counts)
      Trace tr(h, "svd_jacobi_sweep", 0.0, 0.0);
      for (int64_t t = -1; t < Gp - 1; ++t) {
        hipLaunchKernelGGL(k_jac_gram, dim3((unsigned)nz, (unsigned)nblk), dim3(256), 0, st, (const double*)Mc, ldm,
                           Gp, t, zrows, gram);
        hipLaunchKernelGGL(k_jac_solve, dim3((unsigned)nblk), dim3(64 * kSolveWaves), 0, st, (const double*)gram, (int)nz, t, tol,
                           Wb, moved, ctr);
        hipLaunchKernelGGL(k_jac_apply, dim3(ceil_div(ldm, 128), (unsigned)nblk, 2), dim3(256), 0, st, Mc, Jc, ldm,
                           Gp, t, (const double*)Wb, (const int*)moved);
      }
    }
    RFMLS_CHECK(read_counters(3));
    ++P->sweeps;
    if (h->trace && !h->trace_recs.empty()) {
      // algorithmic bytes of the sweep: every step reads all n columns of M for
      // the Gram matrices; a block that rotated reads and writes its 64 columns
      // of M and J.  Flops: the Grams' upper triangles and the products with W.
      const double steps = (double)Gp, rblocks = (double)pin[2];
      h->trace_recs.back().bytes = 8.0 * (double)n * ((double)n * steps + 4.0 * kJw * rblocks);
      h->trace_recs.back().flops =
          (double)n * (steps * (double)nblk * kJw * (kJw + 1) + 4.0 * kJw * kJw * rblocks);
    }
  }
  // singular values, rank and P = J diag(d), d_k = 1 / sigma_k above the threshold, else 0
  hipLaunchKernelGGL(k_col_norms, dim3((unsigned)n), dim3(256), 0, st, (const double*)Mc, n, ldm, P->sigma);
  std::vector<double> sig(n), dh(n);
  RFMLS_HIP(h, hipMemcpyAsync(sig.data(), P->sigma, sizeof(double) * n, hipMemcpyDeviceToHost, st));
  RFMLS_HIP(h, hipStreamSynchronize(st));
  double smax = 0.0;
  for (double v : sig) {
    if (!(v == v)) return fail(h, RFMLS_E_BREAKDOWN, "SVD preconditioner: non-finite singular value");
    smax = v > smax ? v : smax;
  }
  if (rcond <= 0.0) rcond = (double)n * 1.1102230246251565e-16;
  const double thr = rcond * smax;
  int64_t r = 0;
  for (int64_t k = 0; k < n; ++k) {
    const bool keep = smax > 0.0 && sig[k] > thr;
    dh[k] = keep ? 1.0 / sig[k] : 0.0;
    r += keep ? 1 : 0;
  }
  P->rank = r;
  if (r == 0) return fail(h, RFMLS_E_RANK, "SVD preconditioner: every singular value is below rcond * sigma_1");
  RFMLS_HIP(h, hipMemcpyAsync(d, dh.data(), sizeof(double) * n, hipMemcpyHostToDevice, st));
  void* px;
  RFMLS_CHECK(workspace(h, WS_TRSM, sizeof(double) * (size_t)n * (size_t)n, &px));
  double* Pd = (double*)px;
  {
    // Pd[i][k] = J[i][k] d[k]: J is stored as columns, so row k of Jc is column k of J
    dim3 g(ceil_div(n, kTr), ceil_div(n, kTr));
    hipLaunchKernelGGL(k_transpose_scale, g, dim3(kTr * 8), 0, st, (const double*)Jc, ldm, n, n,
                       (const double*)d, (const int32_t*)nullptr, Pd, n);
    RFMLS_HIP(h, hipGetLastError());
  }
  // P = V diag(d) = Q2 (J diag(d))
  RFMLS_CHECK(apply_householder(h, Rt, ld2, n, n, tau2, Pd, n, n));
  // dh must stay alive until the upload above has been consumed
  RFMLS_HIP(h, hipStreamSynchronize(st));
  RFMLS_CHECK(pack_precond(h, P, Pd));
  if (!converged)
    return fail(h, RFMLS_W_NOCONV, "SVD preconditioner: %d Jacobi sweeps left |cos| = %.3e > %.3e",
                P->sweeps, P->off, tol);
  return RFMLS_OK;
}

}  // namespace rfmls
