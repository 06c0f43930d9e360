// LSQR on the preconditioned operator B = A R^{-1} (Alg. 1 steps 4-6 with the
// preconditioner applied inside the iteration, Remark 3.2), textbook
// Paige-Saunders recurrences with every scalar kept on the device.
//
// Products used by one iteration:
//   z = X v            triangular product with the packed X = R^{-1}  (k_trmv_*)
//   u^ = A z - a u     SpMV over each row's column runs                (k_spmv_runs)
//   q = A^T u          the same with the explicit transpose            (k_spmv_runs)
//   v^ = X^T q - b v   transposed triangular product                   (k_trmvT_*)
// followed by the plane rotation and the updates of y and w.  u and v are kept
// unnormalised (beta u, alpha v): the pass that would only scale a vector by its
// new norm is folded into the next product (LazyScale), and the scalars of an
// iteration are formed by every workgroup of the update kernel from the partial
// sums.  An iteration is seven launches (five for small preconditioners, whose
// triangular products need no second pass) instead of eleven.  Norms are
// reduced in a fixed order (per-block partials, then a fixed tree), so runs
// are bitwise reproducible.  The host only polls a device "done" flag every
// few iterations; kernels launched after the stop return immediately.
#include <mutex>

#include "common.h"
#include "lsqr_dev.h"

namespace rfmls {
namespace {

constexpr int kThreads = 256;
constexpr int kSpmvMaxBlocks = 2048;

__device__ __forceinline__ double inv_or_0(double x) { return x > 0.0 ? 1.0 / x : 0.0; }

// sum sq[0..nsq) in a fixed order, on every thread of the block
__device__ double reduce_partials(const double* __restrict__ sq, int nsq, double* scratch) {
  double t = 0.0;
  for (int i = threadIdx.x; i < nsq; i += blockDim.x) t += sq[i];
  return block_sum(t, scratch);
}

// The scalars of out = s acc - c prev (every thread of the block calls it).
__device__ __forceinline__ void lazy_scale(const LazyScale& L, double* scratch, double* s, double* c) {
  *s = L.s;
  *c = L.c;
  if (L.sq) {
    const double nu = sqrt(reduce_partials(L.sq, L.nsq, scratch));
    if (blockIdx.x == 0 && threadIdx.x == 0) *L.norm = nu;
    *s *= inv_or_0(nu);
    if (L.cden) *c *= nu * inv_or_0(*L.cden);
  } else {
    if (L.sdiv) *s *= inv_or_0(*L.sdiv);
    if (L.cnum) *c *= *L.cnum * inv_or_0(*L.cden);
  }
}

// Takes the state an iteration left in `next` (k_lsqr_step) into `st`, with the
// sums of its y and w and the stopping tests (S1 needs ||y_k||, known only once
// every workgroup of the update is done).  One workgroup; nothing when there is
// no uncommitted state, so it may run both at the end of a poll interval and in
// the next iteration's first kernel.  That kernel's other workgroups use nothing
// of the state but the stop flag, whose being set early or late by one kernel
// changes no result.
__device__ void commit_state(const LsqrCommit& cm, double* scratch) {
  // every load issued before the first use: the state of an iteration that left
  // none is read for nothing
  LsqrDev s = *cm.next;
  double y2 = 0.0, w2 = 0.0;
  for (int i = threadIdx.x; i < cm.n; i += blockDim.x) {
    y2 += cm.ysq[i];
    w2 += cm.wsq[i];
  }
  if (!s.fresh) return;  // uniform
  y2 = block_sum(y2, scratch);
  w2 = block_sum(w2, scratch);
  if (threadIdx.x != 0) return;
  cm.next->fresh = 0;
  s.fresh = 0;
  if (!s.done) {
    s.ynorm = sqrt(y2);
    s.w2 = w2;
    const double anorm = sqrt(s.anorm2);
    const double rtol = cm.consistent ? s.btol * s.bnorm : s.btol * s.bnorm + s.atol * anorm * s.ynorm;
    int istop = 0;
    if (s.normr <= rtol) istop = 1;
    else if (s.pending) istop = s.pending;
    else if (s.itn >= s.itmax) istop = 7;
    if (istop) {
      s.istop = istop;
      s.done = 1;
    }
  }
  *cm.st = s;
}
__global__ void __launch_bounds__(kThreads) k_commit(LsqrCommit cm) {
  __shared__ double scratch[kThreads / 64];
  commit_state(cm, scratch);
}

// Sum over groups of L = 8 or 32 neighbouring lanes, on each of them, on the DPP path
// (quad permutations and a mirror of 8 lanes; 32: the two 16-lane rows' sums).
template <int L>
__device__ __forceinline__ double group_sum(double v) {
  if constexpr (L == 8) {
    v += dpp_move<0xB1>(v);   // quad_perm(1, 0, 3, 2)
    v += dpp_move<0x4E>(v);   // quad_perm(2, 3, 0, 1)
    v += dpp_move<0x141>(v);  // row_half_mirror
    return v;
  } else {
    static_assert(L == 32, "group");
    v = row16_sum(v);
    return v + __shfl_xor(v, 16, 64);
  }
}

// Sums of 16 rows over the wavefront's lanes (a[q]: this lane's part of row q):
// halving exchanges, 17 in all instead of six per row; every lane receives row
// lane / 4.
__device__ __forceinline__ double rows16_sum(double (&a)[16], int lane) {
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) {
    const bool hi = lane & (4 * o);
#pragma unroll
    for (int q = 0; q < o; ++q) {
      const double keep = hi ? a[q + o] : a[q], give = hi ? a[q] : a[q + o];
      a[q] = keep + __shfl_xor(give, 4 * o, 64);
    }
  }
  double s = a[0];
  s += __shfl_xor(s, 2, 64);
  s += __shfl_xor(s, 1, 64);
  return s;
}

// ---------------------------------------------------------------------------
// Triangular products with the packed tiles of X (64 x 64, upper triangle)
// ---------------------------------------------------------------------------
// z = X v: block e handles tile row I = tab[e].x, tiles J in [J_0 + k C, J_0 + (k+1) C)
// with J_0 = row_first(I) (I for the triangular packing, 0 for the full grid).
// Thread (c = lane, w = wave) accumulates rows w + 4q of the tile row against
// column c, then each row is summed across the wavefront.
template <typename TS>
__global__ void __launch_bounds__(kThreads)
    k_trmv_part(const TS* __restrict__ Xpk, int64_t nt, int64_t n, int full, const int2* __restrict__ tab,
                int C, int maxk, const double* __restrict__ v, double* __restrict__ part,
                const int* __restrict__ done) {
  if (done && *done) return;
  const int2 e = tab[blockIdx.x];
  const int64_t I = e.x;
  const int k = e.y;
  const int64_t J0 = row_first(I, full) + (int64_t)k * C;
  const int64_t J1 = J0 + C < nt ? J0 + C : nt;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double acc[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) acc[q] = 0.0;
  // two tiles' loads in flight per iteration (sums in the same order)
#pragma unroll 2
  for (int64_t J = J0; J < J1; ++J) {
    const TS* t = Xpk + ptile(I, J, nt, full) * (int64_t)(kTile * kTile);
    const int64_t gc = J * kTile + lane;
    const double vc = gc < n ? v[gc] : 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[q] += (double)t[(w + 4 * q) * kTile + lane] * vc;
  }
  const double s = rows16_sum(acc, lane);
  if ((lane & 3) == 0) part[((int64_t)I * maxk + k) * kTile + w + 4 * (lane >> 2)] = s;
}

// p = X^T q: block e handles tile column J = tab[e].x, tiles I in [k C, min((k+1) C, col_end(J))).
template <typename TS>
__global__ void __launch_bounds__(kThreads)
    k_trmvT_part(const TS* __restrict__ Xpk, int64_t nt, int64_t n, int full, const int2* __restrict__ tab,
                 int C, int maxk, const double* __restrict__ qv, double* __restrict__ part,
                 const int* __restrict__ done) {
  if (done && *done) return;
  __shared__ double red[4][kTile];
  const int2 e = tab[blockIdx.x];
  const int64_t J = e.x;
  const int k = e.y;
  const int64_t I0 = (int64_t)k * C;
  const int64_t Iend = col_end(J, nt, full);
  const int64_t I1 = I0 + C < Iend ? I0 + C : Iend;
  const int lane = threadIdx.x & 63;
  // the wavefront index as a uniform value: the 16 entries of qv a wavefront
  // needs per tile are then scalar loads, with no branch for the bound test
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double acc0 = 0.0, acc1 = 0.0;  // two chains over alternate rows
#pragma unroll 2
  for (int64_t I = I0; I < I1; ++I) {
    const TS* t = Xpk + ptile(I, J, nt, full) * (int64_t)(kTile * kTile);
#pragma unroll
    for (int q = 0; q < 16; q += 2) {
      const int r = w + 4 * q;
      const int64_t gr = I * kTile + r;
      const double q0 = gr < n ? qv[gr] : 0.0;
      const double q1 = gr + 4 < n ? qv[gr + 4] : 0.0;
      acc0 += (double)t[r * kTile + lane] * q0;
      acc1 += (double)t[(r + 4) * kTile + lane] * q1;
    }
  }
  const double acc = acc0 + acc1;
  red[w][lane] = acc;
  __syncthreads();
  if (w == 0)
    part[((int64_t)J * maxk + k) * kTile + lane] =
        (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// out[i] = s sum_k part[row(i)][k] - c prev[i];  partial sum of squares per block.
// nk(I) = number of chunks of tile row/column I (trans: ceil(col_end(I)/C), else
// ceil((nt - row_first(I))/C)).
// A block handles tile rows I (64 outputs each, grid-stride); its four
// wavefronts sum every fourth partial of each output (independent loads in
// flight), and the four quarter sums are added in a fixed order.  With a commit,
// the last block only commits.
constexpr int kRedMaxBlocks = 2048;

__global__ void __launch_bounds__(kThreads)
    k_tri_reduce(const double* __restrict__ part, int64_t nt, int64_t n, int full, int C, int maxk, int trans,
                 LazyScale sc, const double* prev, double* out, double* __restrict__ sq,
                 const int* __restrict__ done, LsqrCommit cm) {
  __shared__ double scratch[kThreads / 64];
  __shared__ double quarter[kThreads / 64][kTile];
  unsigned nblk = gridDim.x;
  if (cm.st) {
    if (blockIdx.x == --nblk) {
      commit_state(cm, scratch);
      return;
    }
  }
  if (done && *done) return;
  const int r = threadIdx.x & (kTile - 1);
  const int q = threadIdx.x / kTile;
  double s1 = 0.0, cf = 0.0;
  bool scaled = false;
  double ss = 0.0;
  for (int64_t I = blockIdx.x; I < nt; I += nblk) {
    const int64_t i = I * kTile + r;
    const int64_t nk = trans ? (col_end(I, nt, full) + C - 1) / C : (nt - row_first(I, full) + C - 1) / C;
    double s = 0.0;
    if (i < n)
      for (int64_t k = q; k < nk; k += kThreads / kTile) s += part[(I * maxk + k) * kTile + r];
    quarter[q][r] = s;
    if (!scaled) {  // after the first sums' loads have been issued
      lazy_scale(sc, scratch, &s1, &cf);
      scaled = true;
    }
    __syncthreads();
    if (q == 0 && i < n) {
      double t = s1 * ((quarter[0][r] + quarter[1][r]) + (quarter[2][r] + quarter[3][r]));
      if (prev && cf != 0.0) t -= cf * prev[i];
      out[i] = t;
      ss += t * t;
    }
    __syncthreads();
  }
  if (sq) {
    ss = block_sum(ss, scratch);
    if (threadIdx.x == 0) sq[blockIdx.x] = ss;
  }
}

// The triangular products of a preconditioner of at most kSmallTiles tile rows in
// one launch: a workgroup of eight wavefronts per 16 outputs, the tiles of its
// row (column) dealt to the wavefronts in turn and their sums added in order, so
// no partial sums go through memory.  There, the second launch of the two-pass
// form costs more than the coarser split (a workgroup here reads at most 256 KB
// of X): n = 1,600, X v 7.4 + 3.8 -> 6.3 us, X^T q 5.1 + 3.8 -> 8.2; n = 200, 7.4 +
// 2.9 -> 3.7 and 3.8 + 2.9 -> 3.9.  Wider ones need the split over tiles to keep
// every compute unit reading.
constexpr int64_t kSmallTiles = 32;
constexpr int kSmallWaves = 8;

__device__ __forceinline__ void small_store(double v, int64_t i, bool live, double s1, double cf, const double* prev,
                                            double* out, double* sq) {
  double t = 0.0;
  if (live) {
    t = s1 * v;
    if (prev && cf != 0.0) t -= cf * prev[i];
    out[i] = t;
  }
  if (sq) {  // lanes 0 .. 15 of wavefront 0
    t = row16_sum(t * t);
    if (threadIdx.x == 0) sq[blockIdx.x] = t;
  }
}

template <typename TS>
__global__ void __launch_bounds__(64 * kSmallWaves)
    k_trmv_small(const TS* __restrict__ Xpk, int64_t nt, int64_t n, int full, const double* __restrict__ v,
                 LazyScale sc, const double* prev, double* out, double* __restrict__ sq,
                 const int* __restrict__ done, LsqrCommit cm) {
  __shared__ double scratch[kSmallWaves];
  __shared__ double red[kSmallWaves][16];
  if (cm.st && blockIdx.x == gridDim.x - 1) {
    commit_state(cm, scratch);
    return;
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t I = blockIdx.x >> 2;
  const int r0 = 16 * (blockIdx.x & 3);
  // lane (lr, lk) takes columns 16 p + lr of rows lk + 4 q; the next tile's loads in
  // flight during this one's products, the first tile's issued with the stop flag's
  const int lr = lane & 15, lk = lane >> 4;
  TS x[16];
  double vc[4];
  auto load = [&](int64_t J) {
    const TS* t = Xpk + ptile(I, J, nt, full) * (int64_t)(kTile * kTile) + (r0 + lk) * kTile + lr;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int64_t gc = J * kTile + 16 * p + lr;
      vc[p] = gc < n ? v[gc] : 0.0;
#pragma unroll
      for (int q = 0; q < 4; ++q) x[4 * q + p] = t[4 * q * kTile + 16 * p];
    }
  };
  int64_t J = row_first(I, full) + w;
  if (J < nt) load(J);
  if (done && *done) return;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  while (J < nt) {
    double pr[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) pr[e] = (double)x[e] * vc[e & 3];
    J += kSmallWaves;
    if (J < nt) load(J);
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] += (pr[4 * q] + pr[4 * q + 1]) + (pr[4 * q + 2] + pr[4 * q + 3]);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double s = row16_sum(acc[q]);
    if (lr == 0) red[w][lk + 4 * q] = s;
  }
  double s1, cf;
  lazy_scale(sc, scratch, &s1, &cf);
  __syncthreads();
  if (threadIdx.x < 16) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < kSmallWaves; ++q) t += red[q][threadIdx.x];
    const int64_t i = I * kTile + r0 + threadIdx.x;
    small_store(t, i, i < n, s1, cf, prev, out, sq);
  }
}

template <typename TS>
__global__ void __launch_bounds__(64 * kSmallWaves)
    k_trmvT_small(const TS* __restrict__ Xpk, int64_t nt, int64_t n, int full, const double* __restrict__ qv,
                  LazyScale sc, const double* prev, double* out, double* __restrict__ sq,
                  const int* __restrict__ done, LsqrCommit cm) {
  __shared__ double scratch[kSmallWaves];
  __shared__ double red[kSmallWaves][16];
  if (cm.st && blockIdx.x == gridDim.x - 1) {
    commit_state(cm, scratch);
    return;
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const int64_t J = blockIdx.x >> 2;
  const int c0 = 16 * (blockIdx.x & 3);
  const int64_t Iend = col_end(J, nt, full);
  TS x[16];
  double y[16];
  auto load = [&](int64_t I) {  // as in k_trmv_small
    const TS* t = Xpk + ptile(I, J, nt, full) * (int64_t)(kTile * kTile) + c0 + lr;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int r = 4 * q + lk;
      const int64_t gr = I * kTile + r;
      x[q] = t[r * kTile];
      y[q] = gr < n ? qv[gr] : 0.0;
    }
  };
  int64_t I = w;
  if (I < Iend) load(I);
  if (done && *done) return;
  double acc0 = 0.0, acc1 = 0.0;
  while (I < Iend) {
    double p[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) p[q] = (double)x[q] * y[q];
    I += kSmallWaves;
    if (I < Iend) load(I);
#pragma unroll
    for (int q = 0; q < 16; q += 2) {
      acc0 += p[q];
      acc1 += p[q + 1];
    }
  }
  double s = acc0 + acc1;
  s += __shfl_xor(s, 16, 64);
  s += __shfl_xor(s, 32, 64);
  if (lane < 16) red[w][lane] = s;
  double s1, cf;
  lazy_scale(sc, scratch, &s1, &cf);
  __syncthreads();
  if (threadIdx.x < 16) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < kSmallWaves; ++q) t += red[q][threadIdx.x];
    const int64_t i = J * kTile + c0 + threadIdx.x;
    small_store(t, i, i < n, s1, cf, prev, out, sq);
  }
}

// ---------------------------------------------------------------------------
// CSR SpMV: out[row] = s (A x)[row] - c prev[row]; half a wavefront (32
// lanes) per row, two entries per lane in flight (measured on the RFM matrix
// and its transpose: 5.2-5.9 TB/s against 3.8-4.3 for a wavefront per row).
// ---------------------------------------------------------------------------
constexpr int kSpvLanes = 32;

__global__ void __launch_bounds__(kThreads)
    k_spmv(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
           const double* __restrict__ val, int64_t rows, const double* __restrict__ x, LazyScale sc,
           const double* prev, double* out, double* __restrict__ sq, const int* __restrict__ done, LsqrCommit cm) {
  __shared__ double scratch[kThreads / 64];
  unsigned nblk = gridDim.x;
  if (cm.st) {
    if (blockIdx.x == --nblk) {
      commit_state(cm, scratch);
      return;
    }
  }
  if (done && *done) return;
  const int lane = threadIdx.x & (kSpvLanes - 1);
  const int64_t sub = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / kSpvLanes;
  const int64_t nsub = (int64_t)nblk * (kThreads / kSpvLanes);
  double sA, cf;
  lazy_scale(sc, scratch, &sA, &cf);
  double ss = 0.0;
  for (int64_t row = sub; row < rows; row += nsub) {
    const int64_t lo = rp[row], hi = rp[row + 1];
    double s0 = 0.0, s1 = 0.0;
    int64_t e = lo + lane;
    for (; e + kSpvLanes < hi; e += 2 * kSpvLanes) {
      s0 += val[e] * x[col[e]];
      s1 += val[e + kSpvLanes] * x[col[e + kSpvLanes]];
    }
    if (e < hi) s0 += val[e] * x[col[e]];
    const double t = group_sum<kSpvLanes>(s0 + s1);
    if (lane == 0) {
      double o = sA * t;
      if (prev && cf != 0.0) o -= cf * prev[row];
      out[row] = o;
      ss += o * o;
    }
  }
  if (sq) {
    ss = block_sum(ss, scratch);
    if (threadIdx.x == 0) sq[blockIdx.x] = ss;
  }
}

// ---------------------------------------------------------------------------
// Column runs.  The rows of an RFM matrix cover the basis functions of one or
// two boxes, contiguous column ranges, and the rows of its transpose a few
// blocks of collocation points.  Row i is described as at most kMaxRuns runs
// of consecutive columns: run k starts at column rcol[i kMaxRuns + k] and
// ends before entry rend[i kMaxRuns + k] of the row (counted from rp[i]); the
// SpMV then reads 8 bytes per entry (its value) instead of 12 and x in
// contiguous stretches.  nrun[i] = -1 marks a row with more runs, which takes
// the column-index path.
// ---------------------------------------------------------------------------
// lanes per row of the run SpMV for matrices whose rows average fewer than
// 512 entries (more rows in flight per wavefront: spmv_A 0.054 -> 0.048 ms on
// the 8x8-box system's 216-entry rows, 0.060 -> 0.055 ms on the Helmholtz
// system's 446-entry rows; 4 lanes and 16 were slower); longer rows keep 32
constexpr int kSpvLanesShort = 8;

__global__ void __launch_bounds__(kThreads)
    k_find_runs(const int64_t* __restrict__ rp, const int32_t* __restrict__ col, int64_t rows,
                int32_t* __restrict__ nrun, int32_t* __restrict__ rcol, int32_t* __restrict__ rend,
                const int* __restrict__ skip) {
  if (skip && *skip) return;
  const int lane = threadIdx.x & (kSpvLanes - 1);
  const int half = (threadIdx.x & 63) >> 5;
  const int64_t sub = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / kSpvLanes;
  const int64_t nsub = (int64_t)gridDim.x * (kThreads / kSpvLanes);
  for (int64_t row = sub; row < rows; row += nsub) {
    const int64_t lo = rp[row], hi = rp[row + 1];
    int cnt = 0;  // runs found so far (uniform over the row's 32 lanes)
    for (int64_t b = lo; b < hi; b += kSpvLanes) {
      const int64_t e = b + lane;
      const bool in = e < hi;
      const int32_t c = in ? col[e] : 0;
      const int32_t pc = (in && e > lo) ? col[e - 1] : 0;
      const bool start = in && (e == lo || c != pc + 1);
      const unsigned bits = (unsigned)(__ballot(start) >> (32 * half));
      const int idx = cnt + __popc(bits & ((1u << lane) - 1u));
      if (start && idx < kMaxRuns) {
        rcol[row * kMaxRuns + idx] = c;
        if (idx > 0) rend[row * kMaxRuns + idx - 1] = (int32_t)(e - lo);
      }
      cnt += __popc(bits);
    }
    if (lane == 0) {
      if (cnt >= 1 && cnt <= kMaxRuns) rend[row * kMaxRuns + cnt - 1] = (int32_t)(hi - lo);
      nrun[row] = cnt <= kMaxRuns ? cnt : -1;
    }
  }
}

// k_spmv over column runs (rows marked -1 take the column-index path), L
// lanes per row.  A row's pointers, run count and first run are loaded
// together, and the next row's while this one is summed, so a row costs one
// memory latency instead of three.
template <int L>
__global__ void __launch_bounds__(kThreads)
    k_spmv_runs(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                const double* __restrict__ val, int64_t rows, const int32_t* __restrict__ nrun,
                const int32_t* __restrict__ rcol, const int32_t* __restrict__ rend,
                const double* __restrict__ x, LazyScale sc, const double* prev, double* out,
                double* __restrict__ sq, const int* __restrict__ done, LsqrCommit cm) {
  __shared__ double scratch[kThreads / 64];
  unsigned nblk = gridDim.x;
  if (cm.st) {
    if (blockIdx.x == --nblk) {
      commit_state(cm, scratch);
      return;
    }
  }
  const int lane = threadIdx.x & (L - 1);
  const int64_t sub = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / L;
  const int64_t nsub = (int64_t)nblk * (kThreads / L);
  int64_t lo = 0, hi = 0;
  int nr = 0;
  int32_t e0 = 0, c0 = 0;
  if (sub < rows) {
    lo = rp[sub];
    hi = rp[sub + 1];
    nr = nrun[sub];
    e0 = rend[sub * kMaxRuns];
    c0 = rcol[sub * kMaxRuns];
  }
  if (done && *done) return;  // its load goes out with the first row's
  double sA, cf;
  lazy_scale(sc, scratch, &sA, &cf);
  double ss = 0.0;
  for (int64_t row = sub; row < rows; row += nsub) {
    const int64_t nrow = row + nsub;
    int64_t nlo = 0, nhi = 0;
    int nnr = 0;
    int32_t ne0 = 0, nc0 = 0;
    if (nrow < rows) {
      nlo = rp[nrow];
      nhi = rp[nrow + 1];
      nnr = nrun[nrow];
      ne0 = rend[nrow * kMaxRuns];
      nc0 = rcol[nrow * kMaxRuns];
    }
    double s0 = 0.0, s1 = 0.0;
    if (nr < 0) {
      int64_t e = lo + lane;
      for (; e + L < hi; e += 2 * L) {
        s0 += val[e] * x[col[e]];
        s1 += val[e + L] * x[col[e + L]];
      }
      if (e < hi) s0 += val[e] * x[col[e]];
    } else {
      const double* vr = val + lo;
      int32_t off = 0;
      for (int k = 0; k < nr; ++k) {
        const int32_t end = k == 0 ? e0 : rend[row * kMaxRuns + k];
        const double* xr = x + (k == 0 ? c0 : rcol[row * kMaxRuns + k]);  // column of entry off
        // four entries per lane in flight (the transposes' rows run to
        // thousands of entries: 0.085 -> 0.064 ms on the Helmholtz A^T)
        int32_t e = off + lane;
        for (; e + 3 * L < end; e += 4 * L) {
          s0 += vr[e] * xr[e - off];
          s1 += vr[e + L] * xr[e + L - off];
          s0 += vr[e + 2 * L] * xr[e + 2 * L - off];
          s1 += vr[e + 3 * L] * xr[e + 3 * L - off];
        }
        for (; e < end; e += L) s0 += vr[e] * xr[e - off];
        off = end;
      }
    }
    const double t = group_sum<L>(s0 + s1);
    if (lane == 0) {
      double o = sA * t;
      if (prev && cf != 0.0) o -= cf * prev[row];
      out[row] = o;
      ss += o * o;
    }
    lo = nlo;
    hi = nhi;
    nr = nnr;
    e0 = ne0;
    c0 = nc0;
  }
  if (sq) {
    ss = block_sum(ss, scratch);
    if (threadIdx.x == 0) sq[blockIdx.x] = ss;
  }
}

// ---------------------------------------------------------------------------
// Vector helpers
// ---------------------------------------------------------------------------
// out = a x + b y
__global__ void k_axpby(int64_t len, double a, const double* x, double b, const double* y, double* out) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len;
       i += (int64_t)gridDim.x * blockDim.x) {
    double o = a * x[i];
    if (y) o += b * y[i];
    out[i] = o;
  }
}

// out[0] = sqrt(sum sq[0..nsq)) in the fixed order of reduce_partials (one block)
__global__ void __launch_bounds__(kThreads) k_sqrt_sum(const double* __restrict__ sq, int nsq,
                                                       double* __restrict__ out) {
  __shared__ double red[kThreads / 64];
  const double t = reduce_partials(sq, nsq, red);
  if (threadIdx.x == 0) out[0] = sqrt(t);
}

// per-block sums of squares of x, which is also copied to out when given
__global__ void __launch_bounds__(kThreads) k_copy_sumsq(const double* x, int64_t len, double* out,
                                                         double* __restrict__ sq) {
  __shared__ double scratch[kThreads / 64];
  double t = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < len;
       i += (int64_t)gridDim.x * kThreads) {
    const double v = x[i];
    if (out) out[i] = v;
    t += v * v;
  }
  t = block_sum(t, scratch);
  if (threadIdx.x == 0) sq[blockIdx.x] = t;
}

// ---------------------------------------------------------------------------
// LSQR scalars
// ---------------------------------------------------------------------------
// beta_1 = ||b|| from the partial sums: set up the state.
__global__ void __launch_bounds__(kThreads)
    k_lsqr_begin(LsqrDev* st, LsqrDev* next, const double* __restrict__ sq, int nsq, double atol, double btol,
                 double conlim, int64_t itmax) {
  __shared__ double scratch[kThreads / 64];
  const double beta = sqrt(reduce_partials(sq, nsq, scratch));
  if (threadIdx.x != 0) return;
  LsqrDev s{};
  s.atol = atol;
  s.btol = btol;
  s.conlim = conlim;
  s.itmax = itmax;
  s.beta = s.bnorm = s.phibar = beta;
  s.istop = 7;
  if (!isfinite(beta)) {  // a non-finite right-hand side: breakdown, not "x = 0 is exact"
    s.istop = -3;
    s.done = 1;
  } else if (!(beta > 0.0)) {
    s.istop = 0;
    s.done = 1;
  }
  *st = s;
  next->fresh = 0;
}

// After alpha_1 (sq: the partial sums of its vector).
__global__ void __launch_bounds__(kThreads) k_lsqr_begin2(LsqrDev* st, const double* __restrict__ sq, int nsq) {
  if (st->done) return;
  __shared__ double scratch[kThreads / 64];
  const double alpha = sqrt(reduce_partials(sq, nsq, scratch));
  if (threadIdx.x != 0) return;
  st->alpha = st->alpha_prev = st->rhobar = alpha;
  st->normr = st->beta;
  st->normar = alpha * st->beta;
  st->w2 = 1.0;  // w_1 = v_1
  if (!isfinite(alpha)) {
    st->istop = -3;
    st->done = 1;
  } else if (!(alpha > 0.0)) {
    st->istop = 0;
    st->done = 1;
  }
}

// y_1 = 0 and w_1 = v^/alpha (v^ = alpha v), or of the backward's shadow vector
// vt_1 = u^/(beta alpha), which is also kept in vt; wsq (optional): the partial sums
// of ||w_1||^2
__global__ void __launch_bounds__(kThreads)
    k_lsqr_first_w(const LsqrDev* __restrict__ st, const double* __restrict__ v, int over_beta, double* vt, double* w,
                   double* y, int64_t n, double* __restrict__ wsq) {
  __shared__ double scratch[kThreads / 64];
  double f = inv_or_0(st->alpha);
  if (over_beta) f *= inv_or_0(st->beta);
  double sw = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
    const double wi = v[i] * f;
    if (vt) vt[i] = wi;
    w[i] = wi;
    y[i] = 0.0;
    sw += wi * wi;
  }
  if (!wsq) return;
  sw = block_sum(sw, scratch);
  if (threadIdx.x == 0) wsq[blockIdx.x] = sw;
}
__global__ void __launch_bounds__(kThreads) k_lsqr_w2(LsqrDev* st, const double* __restrict__ wsq, int nsq) {
  __shared__ double scratch[kThreads / 64];
  const double t = reduce_partials(wsq, nsq, scratch);
  if (threadIdx.x == 0) st->w2 = t;
}

// The rest of iteration k after alpha v^ (asq: the partial sums of its squares)
// and beta (in the state): plane rotation, y += phi/rho w, w = v - theta/rho w,
// partial sums of ||y||^2 and ||w||^2.  Every workgroup forms the same scalars from
// the committed state; the first leaves the new one in `next` (commit_state).
//   backward (vt given): v is the beta u of the iteration; the shadow vector vt =
//   (u - beta vt) / alpha takes v's part.
__global__ void __launch_bounds__(kThreads)
    k_lsqr_step(const LsqrDev* __restrict__ st, LsqrDev* next, const double* __restrict__ asq, int nasq,
                const double* __restrict__ v, double* vt, double* w, double* y, int64_t n, double* __restrict__ ysq,
                double* __restrict__ wsq) {
  __shared__ double scratch[kThreads / 64];
  // the state, the partial sums and the first entries of the vectors are loaded
  // together (one memory round trip), then the stop flag is looked at
  LsqrDev s = *st;
  double a2 = 0.0;
  for (int i = threadIdx.x; i < nasq; i += kThreads) a2 += asq[i];
  const int64_t i0 = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const bool in0 = i0 < n;
  const double w0 = in0 ? w[i0] : 0.0, y0 = in0 ? y[i0] : 0.0, v0 = in0 ? v[i0] : 0.0;
  const double vt0 = vt && in0 ? vt[i0] : 0.0;
  if (s.done) return;
  const double alpha = sqrt(block_sum(a2, scratch));
  const double beta = s.beta;
  s.alpha = alpha;
  s.itn += 1;
  s.anorm2 += s.alpha_prev * s.alpha_prev + beta * beta;
  const double rho = hypot(s.rhobar, beta);
  s.pending = 0;
  const bool good = rho > 0.0 && isfinite(rho);
  if (good) {
    const double c = s.rhobar / rho;
    const double sn = beta / rho;
    const double theta = sn * alpha;
    s.rhobar = -c * alpha;
    const double phi = c * s.phibar;
    s.phibar = sn * s.phibar;
    s.phi_rho = phi / rho;
    s.theta_rho = theta / rho;
    s.ddnorm += s.w2 / (rho * rho);
    const double anorm = sqrt(s.anorm2);
    s.acond = anorm * sqrt(s.ddnorm);
    s.normr = s.phibar;
    s.normar = s.phibar * alpha * fabs(c);
    if (s.normr == 0.0 || s.normar <= s.atol * anorm * s.normr) s.pending = 2;
    else if (s.conlim > 0.0 && s.acond >= s.conlim) s.pending = 3;
    s.alpha_prev = alpha;
  } else {
    s.istop = isfinite(rho) ? 1 : -3;
    s.done = 1;
    s.phi_rho = 0.0;
    s.theta_rho = 0.0;
  }
  s.fresh = 1;
  if (blockIdx.x == 0 && threadIdx.x == 0) *next = s;
  if (!good) return;
  const double a = s.phi_rho, b = s.theta_rho;
  const double ia = inv_or_0(alpha), ib = inv_or_0(beta);
  double sy = 0.0, sw = 0.0;
  for (int64_t i = i0; i < n; i += (int64_t)gridDim.x * kThreads) {
    const bool first = i == i0;
    const double wi = first ? w0 : w[i];
    const double yi = (first ? y0 : y[i]) + a * wi;
    double vi = first ? v0 : v[i];
    if (vt) {
      vi = (vi * ib - beta * (first ? vt0 : vt[i])) * ia;
      vt[i] = vi;
    } else {
      vi *= ia;
    }
    const double wn = vi - b * wi;
    y[i] = yi;
    w[i] = wn;
    sy += yi * yi;
    sw += wn * wn;
  }
  sy = block_sum(sy, scratch);
  sw = block_sum(sw, scratch);
  if (threadIdx.x == 0) {
    ysq[blockIdx.x] = sy;
    wsq[blockIdx.x] = sw;
  }
}

// dA[e] += r_i w_j - lam_i x_j on the pattern of A
__global__ void k_pattern_grad(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                               int64_t m, const double* __restrict__ r, const double* __restrict__ w,
                               const double* __restrict__ lam, const double* __restrict__ x,
                               double* __restrict__ dA, int accumulate) {
  const int lane = threadIdx.x & 63;
  const int64_t wid = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x / 64);
  for (int64_t row = wid; row < m; row += nw) {
    const double ri = r[row], li = lam[row];
    for (int64_t e = rp[row] + lane; e < rp[row + 1]; e += 64) {
      const int32_t j = col[e];
      const double g = ri * w[j] - li * x[j];
      dA[e] = accumulate ? dA[e] + g : g;
    }
  }
}

// ---------------------------------------------------------------------------
// Dense products with the explicit B = A R^{-1} (row-major m x n, Alg. 1 step 4).
// ---------------------------------------------------------------------------
// out[i] = s (B v)[i] - c prev[i]; one wavefront per
// row, four independent partial sums per lane, a fixed-order tree across the
// wavefront; per-block sums of squares of out into sq.
__global__ void __launch_bounds__(kThreads)
    k_gemv(const double* __restrict__ B, int64_t ldb, int64_t m, int64_t n,
           const double* __restrict__ v, LazyScale sc, const double* prev, double* out, double* __restrict__ sq,
           const int* __restrict__ done) {
  if (done && *done) return;
  __shared__ double scratch[kThreads / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double sA, cf;
  lazy_scale(sc, scratch, &sA, &cf);
  double ss = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * (kThreads / 64) + w; i < m; i += (int64_t)gridDim.x * (kThreads / 64)) {
    const double* row = B + i * ldb;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    int64_t j = lane;
    for (; j + 192 < n; j += 256) {
      a0 += row[j] * v[j];
      a1 += row[j + 64] * v[j + 64];
      a2 += row[j + 128] * v[j + 128];
      a3 += row[j + 192] * v[j + 192];
    }
    for (; j < n; j += 64) a0 += row[j] * v[j];
    double t = wave_sum((a0 + a1) + (a2 + a3));
    if (lane == 0) {
      t = sA * t;
      if (prev && cf != 0.0) t -= cf * prev[i];
      out[i] = t;
      ss += t * t;
    }
  }
  if (sq) {
    ss = block_sum(ss, scratch);
    if (threadIdx.x == 0) sq[blockIdx.x] = ss;
  }
}

// part[z][j] = sum over the rows i of slice z of B[i][j] u[i]: block (x, z)
// covers the kThreads columns from kThreads x and rows [z rps, (z + 1) rps).
// Bound by HBM (B once): a thread keeps kGemvTRows rows' loads of its column
// in flight, and the slices are chosen so that the grid fills the GPU
// (gemvT_slices).  On the 32,805 x 2,619 operator (687 MB), with the sum of the
// slices: 401 us with two columns per thread, one row in flight and 64 slices
// (1.7 TB/s), 120 us now (5.7 TB/s).
constexpr int kGemvTRows = 8;
__global__ void __launch_bounds__(kThreads)
    k_gemvT_part(const double* __restrict__ B, int64_t ldb, int64_t m, int64_t n,
                 const double* __restrict__ u, int64_t rps, double* __restrict__ part,
                 const int* __restrict__ done) {
  if (done && *done) return;
  const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.y * rps;
  const int64_t r1 = r0 + rps < m ? r0 + rps : m;
  if (j >= n) return;
  const double* p = B + r0 * ldb + j;
  double a0 = 0.0, a1 = 0.0;  // even and odd rows
  int64_t i = r0;
  for (; i + kGemvTRows <= r1; i += kGemvTRows, p += kGemvTRows * ldb) {
    double b[kGemvTRows];
#pragma unroll
    for (int k = 0; k < kGemvTRows; ++k) b[k] = p[k * ldb];
#pragma unroll
    for (int k = 0; k < kGemvTRows; k += 2) {
      a0 += b[k] * u[i + k];
      a1 += b[k + 1] * u[i + k + 1];
    }
  }
  for (; i < r1; ++i, p += ldb) a0 += *p * u[i];
  part[(int64_t)blockIdx.y * n + j] = a0 + a1;
}

// out[j] = s sum_z part[z][j] - c prev[j]; per-block sums of squares.  A block
// takes 64 columns at a time (grid-stride); its four wavefronts sum every
// fourth slice, and the four sums are added in a fixed order.
__global__ void __launch_bounds__(kThreads)
    k_gemvT_reduce(const double* __restrict__ part, int nz, int64_t n, LazyScale sc, const double* prev, double* out,
                   double* __restrict__ sq, const int* __restrict__ done) {
  if (done && *done) return;
  __shared__ double scratch[kThreads / 64];
  __shared__ double quarter[kThreads / 64][64];
  const int c = threadIdx.x & 63, q = threadIdx.x >> 6;
  double s1, cf;
  lazy_scale(sc, scratch, &s1, &cf);
  double ss = 0.0;
  for (int64_t j0 = (int64_t)blockIdx.x * 64; j0 < n; j0 += (int64_t)gridDim.x * 64) {
    const int64_t j = j0 + c;
    double t = 0.0;
    if (j < n) {
#pragma unroll 4
      for (int z = q; z < nz; z += kThreads / 64) t += part[(int64_t)z * n + j];
    }
    quarter[q][c] = t;
    __syncthreads();
    if (q == 0 && j < n) {
      t = s1 * ((quarter[0][c] + quarter[1][c]) + (quarter[2][c] + quarter[3][c]));
      if (prev && cf != 0.0) t -= cf * prev[j];
      out[j] = t;
      ss += t * t;
    }
    __syncthreads();
  }
  if (sq) {
    ss = block_sum(ss, scratch);
    if (threadIdx.x == 0) sq[blockIdx.x] = ss;
  }
}

}  // namespace

// ===========================================================================
// Host drivers
// ===========================================================================
struct Ctx {
  rfmls_handle* h;
  const rfmls_csr* A;
  const rfmls_csr* AT;
  const rfmls_precond_t* P;
  const double* Bm = nullptr;  // explicit B = A R^{-1} (row-major), or null: implicit operator
  int64_t ldbm = 0;
  double* gpart = nullptr;     // slice partials of B^T u
  hipStream_t st;
  // work vectors
  double *u, *v, *w, *y, *z, *q, *t, *r, *xs;
  double *sqA, *sqB, *sqY, *sqW;
  double* hn;  // device doubles for norms read by the host
  LsqrDev* dst;   // the state, and after it the iteration's uncommitted one
  IterGraph* graph = nullptr;  // captured poll interval of the loop, or null: eager launches
  // column runs of A and A^T (null: the column-index SpMV)
  const int32_t *nrunA = nullptr, *rcolA = nullptr, *rendA = nullptr;
  const int32_t *nrunAT = nullptr, *rcolAT = nullptr, *rendAT = nullptr;
};

static unsigned spmv_blocks(int64_t rows) {
  const int64_t b = (rows + kThreads / kSpvLanes - 1) / (kThreads / kSpvLanes);
  return (unsigned)(b < kSpmvMaxBlocks ? (b > 0 ? b : 1) : kSpmvMaxBlocks);
}
static unsigned vec_blocks(int64_t len) {
  const int64_t b = (len + kThreads - 1) / kThreads;
  return (unsigned)(b < 1024 ? (b > 0 ? b : 1) : 1024);
}

int tri_reduce_blocks(int64_t n) {
  const int64_t b = ceil_div(n, kTile);
  return (int)(b < kRedMaxBlocks ? (b > 0 ? b : 1) : kRedMaxBlocks);
}

rfmls_status tri_apply(rfmls_handle* h, const rfmls_precond_t* P, int trans, const double* in,
                       double* out, const LazyScale& sc, const double* prev, double* sq, int* nsq,
                       const int* done, const LsqrCommit& commit) {
  const int64_t n = P->n, nt = P->nt;
  const int C = P->chunk;
  const int maxk = (int)((nt + C - 1) / C);
  hipStream_t st = h->stream;
  double* part = (double*)P->part;
  const double esz = P->store == RFMLS_F64 ? 8.0 : 4.0;
  const int full = P->full;
  const double tri_elems = full ? (double)n * (double)n : (double)n * (double)(n + 1) / 2.0;
  const unsigned extra = commit.st ? 1u : 0u;
  // algorithmic: the stored entries of X once (n(n+1)/2, or n^2 for the full
  // SVD preconditioner), the input vector, the output
  const char* name = full ? (trans ? "gemv_Pt" : "gemv_P") : (trans ? "trmv_Xt" : "trmv_X");
  if (nt <= kSmallTiles) {
    Trace tr(h, name, esz * tri_elems + 16.0 * (double)n, 2.0 * tri_elems);
    const unsigned nb = ceil_div(n, 16);
    if (P->store == RFMLS_F64)
      hipLaunchKernelGGL(trans ? k_trmvT_small<double> : k_trmv_small<double>, dim3(nb + extra),
                         dim3(64 * kSmallWaves), 0, st, (const double*)P->Xpk, nt, n, full, in, sc, prev, out, sq, done,
                         commit);
    else
      hipLaunchKernelGGL(trans ? k_trmvT_small<float> : k_trmv_small<float>, dim3(nb + extra), dim3(64 * kSmallWaves),
                         0, st, (const float*)P->Xpk, nt, n, full, in, sc, prev, out, sq, done, commit);
    if (nsq) *nsq = (int)nb;
    RFMLS_HIP(h, hipGetLastError());
    return RFMLS_OK;
  }
  {
  Trace tr(h, name, esz * tri_elems + 16.0 * (double)n, 2.0 * tri_elems);
  if (!trans) {
    if (P->store == RFMLS_F64)
      hipLaunchKernelGGL(k_trmv_part<double>, dim3((unsigned)P->ntab), dim3(kThreads), 0, st,
                         (const double*)P->Xpk, nt, n, full, P->tab_row, C, maxk, in, part, done);
    else
      hipLaunchKernelGGL(k_trmv_part<float>, dim3((unsigned)P->ntab), dim3(kThreads), 0, st,
                         (const float*)P->Xpk, nt, n, full, P->tab_row, C, maxk, in, part, done);
  } else {
    if (P->store == RFMLS_F64)
      hipLaunchKernelGGL(k_trmvT_part<double>, dim3((unsigned)P->ntab), dim3(kThreads), 0, st,
                         (const double*)P->Xpk, nt, n, full, P->tab_col, C, maxk, in, part, done);
    else
      hipLaunchKernelGGL(k_trmvT_part<float>, dim3((unsigned)P->ntab), dim3(kThreads), 0, st,
                         (const float*)P->Xpk, nt, n, full, P->tab_col, C, maxk, in, part, done);
  }
  }
  Trace tr2(h, "tri_reduce", 8.0 * (double)nt * maxk * kTile + 16.0 * (double)n, 0.0);
  const int nb = tri_reduce_blocks(n);
  hipLaunchKernelGGL(k_tri_reduce, dim3((unsigned)nb + extra), dim3(kThreads), 0, st, part, nt, n,
                     full, C, maxk, trans, sc, prev, out, sq, done, commit);
  if (nsq) *nsq = nb;
  RFMLS_HIP(h, hipGetLastError());
  return RFMLS_OK;
}


void find_runs(hipStream_t st, const rfmls_csr* M, int32_t* nrun, int32_t* rcol, int32_t* rend, const int* skip) {
  hipLaunchKernelGGL(k_find_runs, dim3(spmv_blocks(M->m)), dim3(kThreads), 0, st, M->row_ptr, M->col, M->m, nrun, rcol,
                     rend, skip);
}

static rfmls_status spmv(Ctx& c, const rfmls_csr* M, const double* x, double* out,
                         const LazyScale& sc = LazyScale(), const double* prev = nullptr, double* sq = nullptr,
                         int* nblk = nullptr, const int* done = nullptr, const LsqrCommit& commit = LsqrCommit()) {
  const unsigned nb = spmv_blocks(M->m);
  const unsigned extra = commit.st ? 1u : 0u;
  const int32_t* nrun = M == c.A ? c.nrunA : c.nrunAT;
  const int32_t* rcol = M == c.A ? c.rcolA : c.rcolAT;
  const int32_t* rend = M == c.A ? c.rendA : c.rendAT;
  // algorithmic: values once (and the column indices, unless the rows are
  // described by their column runs: then a run count and at least one run per
  // row), row pointers, x gathered once, out written (and prev read when used)
  const double idx_bytes = nrun ? 4.0 * (double)M->m * (1 + 2) : 4.0 * (double)M->nnz;
  Trace tr(c.h, M == c.A ? "spmv_A" : "spmv_At",
           8.0 * (double)M->nnz + idx_bytes + 8.0 * (double)(M->m + 1) + 8.0 * (double)M->n +
               8.0 * (double)M->m * (prev ? 2.0 : 1.0),
           2.0 * (double)M->nnz);
  if (nrun && M->nnz < 512 * M->m) {
    const int64_t b = (M->m + kThreads / kSpvLanesShort - 1) / (kThreads / kSpvLanesShort);
    const unsigned nbs = (unsigned)(b < kSpmvMaxBlocks ? (b > 0 ? b : 1) : kSpmvMaxBlocks);
    hipLaunchKernelGGL(k_spmv_runs<kSpvLanesShort>, dim3(nbs + extra), dim3(kThreads), 0, c.st, M->row_ptr, M->col,
                       M->val, M->m, nrun, rcol, rend, x, sc, prev, out, sq, done, commit);
    if (nblk) *nblk = (int)nbs;
    RFMLS_HIP(c.h, hipGetLastError());
    return RFMLS_OK;
  }
  if (nrun)
    hipLaunchKernelGGL(k_spmv_runs<kSpvLanes>, dim3(nb + extra), dim3(kThreads), 0, c.st, M->row_ptr, M->col, M->val,
                       M->m, nrun, rcol, rend, x, sc, prev, out, sq, done, commit);
  else
    hipLaunchKernelGGL(k_spmv, dim3(nb + extra), dim3(kThreads), 0, c.st, M->row_ptr, M->col, M->val, M->m,
                       x, sc, prev, out, sq, done, commit);
  if (nblk) *nblk = (int)nb;
  RFMLS_HIP(c.h, hipGetLastError());
  return RFMLS_OK;
}

// Products with the explicit B (Ctx::Bm): out = s B v - c prev over the m rows,
// and out = s B^T u - c prev over the n columns (slice partials, then a
// fixed-order sum); each writes per-block sums of squares to sq and returns
// their count in *nblk.
// Row slices of B^T u: about eight workgroups per compute unit over the column
// blocks, each slice at least 64 rows.
static int64_t gemvT_slices(const rfmls_handle* h, int64_t m, int64_t n) {
  const int64_t cb = ceil_div(n, kThreads);
  const int64_t want = (8 * (int64_t)h->num_cus + cb - 1) / cb, most = (m + 63) / 64;
  const int64_t z = want < most ? want : most;
  return z > 0 ? z : 1;
}
static rfmls_status bmul(Ctx& c, const double* v, const LazyScale& sc, const double* prev, double* out, double* sq,
                         const int* done, int* nblk) {
  const int64_t m = c.A->m, n = c.A->n;
  const int64_t b = (m + kThreads / 64 - 1) / (kThreads / 64);
  const unsigned nb = (unsigned)(b < kSpmvMaxBlocks ? (b > 0 ? b : 1) : kSpmvMaxBlocks);
  Trace tr(c.h, "gemv_B", 8.0 * (double)m * (double)n + 8.0 * (double)n + 8.0 * (double)m * (prev ? 2.0 : 1.0),
           2.0 * (double)m * (double)n);
  hipLaunchKernelGGL(k_gemv, dim3(nb), dim3(kThreads), 0, c.st, c.Bm, c.ldbm, m, n, v, sc, prev, out, sq, done);
  *nblk = (int)nb;
  RFMLS_HIP(c.h, hipGetLastError());
  return RFMLS_OK;
}
static rfmls_status btmul(Ctx& c, const double* u, const LazyScale& sc, const double* prev, double* out, double* sq,
                          const int* done, int* nblk) {
  const int64_t m = c.A->m, n = c.A->n;
  const int64_t ns = gemvT_slices(c.h, m, n);
  const int64_t rps = m > ns ? (m + ns - 1) / ns : 1;
  const int nz = (int)((m + rps - 1) / rps);
  const unsigned nr = (unsigned)tri_reduce_blocks(n);
  {
    Trace tr(c.h, "gemvT_B", 8.0 * (double)m * (double)n + 8.0 * (double)m + 8.0 * (double)nz * (double)n,
             2.0 * (double)m * (double)n);
    hipLaunchKernelGGL(k_gemvT_part, dim3(ceil_div(n, kThreads), (unsigned)nz), dim3(kThreads), 0, c.st,
                       c.Bm, c.ldbm, m, n, u, rps, c.gpart, done);
    hipLaunchKernelGGL(k_gemvT_reduce, dim3(nr), dim3(kThreads), 0, c.st, (const double*)c.gpart, nz, n,
                       sc, prev, out, sq, done);
  }
  *nblk = (int)nr;
  RFMLS_HIP(c.h, hipGetLastError());
  return RFMLS_OK;
}

// The state as of the last commit, through the pinned staging buffer.
static rfmls_status read_state(Ctx& c, LsqrDev* out) {
  LsqrDev* pin = (LsqrDev*)((char*)c.h->pinned + 2048);
  RFMLS_HIP(c.h, hipMemcpyAsync(pin, c.dst, sizeof(LsqrDev), hipMemcpyDeviceToHost, c.st));
  RFMLS_HIP(c.h, hipStreamSynchronize(c.st));
  *out = *pin;
  return RFMLS_OK;
}

static LsqrCommit commit_of(const Ctx& c, int consistent) {
  LsqrCommit cm;
  cm.st = c.dst;
  cm.next = c.dst + 1;
  cm.ysq = c.sqY;
  cm.wsq = c.sqW;
  cm.n = (int)vec_blocks(c.A->n);
  cm.consistent = consistent;
  return cm;
}

// Runs `iteration` (which enqueues one iteration on c.st) up to itmax times, the
// host reading the committed state after every `every` iterations; with
// c.graph the poll interval is captured once and replayed.  *s: the final state.
template <class F>
static rfmls_status run_iterations(Ctx& c, int64_t itmax, int every, int consistent, LsqrDev* s, F&& iteration) {
  rfmls_handle* h = c.h;
  const LsqrCommit cm = commit_of(c, consistent);
  auto interval = [&](int64_t count) -> rfmls_status {
    for (int64_t k = 0; k < count; ++k) RFMLS_CHECK(iteration());
    hipLaunchKernelGGL(k_commit, dim3(1), dim3(kThreads), 0, c.st, cm);
    RFMLS_HIP(h, hipGetLastError());
    return RFMLS_OK;
  };
  if (c.graph && !h->trace) {
    // the poll interval's launches recorded once per call, then replayed
    if (!c.graph->exec)
      RFMLS_CHECK(capture_graph(h, c.graph, [&]() -> rfmls_status {
        const hipStream_t s0 = c.st;
        c.st = h->stream;
        const rfmls_status r = interval(every);
        c.st = s0;
        return r;
      }));
    *s = LsqrDev{};
    for (int64_t it = 0; it < itmax && !s->done; it += every) {
      RFMLS_HIP(h, hipGraphLaunch(c.graph->exec, c.st));
      RFMLS_CHECK(read_state(c, s));
    }
    return RFMLS_OK;
  }
  *s = LsqrDev{};
  for (int64_t it = 0; it < itmax && !s->done; it += every) {
    RFMLS_CHECK(interval(itmax - it < every ? itmax - it : every));
    RFMLS_CHECK(read_state(c, s));
  }
  return RFMLS_OK;
}

// One LSQR iteration (Golub-Kahan step, plane rotation, updates of y and w),
// enqueued on c.st.  c.u and c.v hold beta u and alpha v.
static rfmls_status lsqr_iteration(Ctx& c) {
  rfmls_handle* h = c.h;
  LsqrDev* st = c.dst;
  const int* done = &st->done;
  const LsqrCommit cm = commit_of(c, 0);
  int nb = 0, nred = 0;
  // beta' u' = A (X v) - alpha u, with v = v^/alpha and u = u^/beta
  LazyScale su;
  su.sdiv = &st->alpha;
  su.c = 1.0;
  su.cnum = &st->alpha;
  su.cden = &st->beta;
  if (c.Bm) {
    // B v uses the state at once, so the commit goes before it
    hipLaunchKernelGGL(k_commit, dim3(1), dim3(kThreads), 0, c.st, cm);
    RFMLS_CHECK(bmul(c, c.v, su, c.u, c.u, c.sqA, done, &nb));
  } else {
    RFMLS_CHECK(tri_apply(h, c.P, 0, c.v, c.z, LazyScale(), nullptr, nullptr, nullptr, done, cm));
    RFMLS_CHECK(spmv(c, c.A, c.z, c.u, su, c.u, c.sqA, &nb, done));
  }
  // alpha' v' = X^T (A^T u') - beta' v, with u' = u^'/beta', beta' from the partial sums
  LazyScale sv;
  sv.c = 1.0;
  sv.sq = c.sqA;
  sv.nsq = nb;
  sv.norm = &st->beta;
  sv.cden = &st->alpha;
  if (c.Bm) {
    RFMLS_CHECK(btmul(c, c.u, sv, c.v, c.v, c.sqB, done, &nred));
  } else {
    RFMLS_CHECK(spmv(c, c.AT, c.u, c.q, LazyScale(), nullptr, nullptr, nullptr, done));
    RFMLS_CHECK(tri_apply(h, c.P, 1, c.q, c.v, sv, c.v, c.sqB, &nred, done));
  }
  hipLaunchKernelGGL(k_lsqr_step, dim3(vec_blocks(c.A->n)), dim3(kThreads), 0, c.st, (const LsqrDev*)st, st + 1,
                     (const double*)c.sqB, nred, (const double*)c.v, (double*)nullptr, c.w, c.y, c.A->n, c.sqY, c.sqW);
  RFMLS_HIP(h, hipGetLastError());
  return RFMLS_OK;
}

// One LSQR sweep for min ||A X y - rhs||; on return c.y holds y and *s the
// final state.  rhs is an m-vector (device).
static rfmls_status lsqr_sweep(Ctx& c, const double* rhs, const rfmls_opts* o, int64_t itmax, LsqrDev* s) {
  rfmls_handle* h = c.h;
  const int64_t m = c.A->m, n = c.A->n;
  const unsigned vbn = vec_blocks(n), vbm = vec_blocks(m);
  LsqrDev* st = c.dst;
  const int* done = &st->done;
  // beta_1 u_1 = rhs
  hipLaunchKernelGGL(k_copy_sumsq, dim3(vbm), dim3(kThreads), 0, c.st, rhs, m, c.u, c.sqA);
  hipLaunchKernelGGL(k_lsqr_begin, dim3(1), dim3(kThreads), 0, c.st, st, st + 1, (const double*)c.sqA, (int)vbm,
                     o->atol, o->btol, o->conlim, itmax);
  // alpha_1 v_1 = B^T u_1 = X^T (A^T u_1) (or the explicit B^T u_1)
  LazyScale s1;
  s1.sdiv = &st->beta;
  int nred = 0;
  if (c.Bm) {
    RFMLS_CHECK(btmul(c, c.u, s1, nullptr, c.v, c.sqB, done, &nred));
  } else {
    RFMLS_CHECK(spmv(c, c.AT, c.u, c.q, LazyScale(), nullptr, nullptr, nullptr, done));
    RFMLS_CHECK(tri_apply(h, c.P, 1, c.q, c.v, s1, nullptr, c.sqB, &nred, done));
  }
  hipLaunchKernelGGL(k_lsqr_begin2, dim3(1), dim3(kThreads), 0, c.st, st, (const double*)c.sqB, nred);
  // y = 0, w_1 = v_1 (unconditional: y is used when the sweep stops at once too)
  hipLaunchKernelGGL(k_lsqr_first_w, dim3(vbn), dim3(kThreads), 0, c.st, (const LsqrDev*)st, (const double*)c.v, 0,
                     (double*)nullptr, c.w, c.y, n, (double*)nullptr);
  RFMLS_HIP(h, hipGetLastError());
  return run_iterations(c, itmax, o->check_every > 0 ? o->check_every : 8, 0, s,
                        [&]() -> rfmls_status { return lsqr_iteration(c); });
}

// Doubles of device memory one single-right-hand-side solve works in: the
// vectors and partial sums (make_ctx's layout) and the LSQR state after them.
static int64_t ctx_doubles(int64_t m, int64_t n) { return 4 * m + 8 * n + 4 * kSpmvMaxBlocks + 64; }
constexpr int64_t kStateDoubles = (2 * sizeof(LsqrDev) + 255) / 256 * 32;

// Bytes of the column-run descriptors of `rows` matrix rows.
static int64_t runs_bytes(int64_t rows) { return (int64_t)sizeof(int32_t) * rows * (1 + 2 * kMaxRuns); }

// base: device memory of at least ctx_doubles + kStateDoubles doubles followed
// by runs_bytes(m + n) bytes, or null for the handle's workspace
static rfmls_status make_ctx(rfmls_handle* h, const rfmls_csr* A, const rfmls_csr* AT,
                             const rfmls_precond_t* P, Ctx& c, double* base = nullptr) {
  c.h = h;
  c.A = A;
  c.AT = AT;
  c.P = P;
  c.st = h->stream;
  const int64_t m = A->m, n = A->n;
  const size_t nvec = (size_t)ctx_doubles(m, n);
  void* p = base;
  if (!base) RFMLS_CHECK(workspace(h, WS_LSQR_VEC, sizeof(double) * nvec, &p));
  double* d = (double*)p;
  c.u = d;
  d += m;
  c.r = d;
  d += m;
  c.t = d;
  d += m;
  d += m;  // spare m-vector
  c.v = d;
  d += n;
  c.w = d;
  d += n;
  c.y = d;
  d += n;
  c.z = d;
  d += n;
  c.q = d;
  d += n;
  c.xs = d;
  d += n;
  d += 2 * n;  // spare
  c.sqA = d;
  d += kSpmvMaxBlocks;
  c.sqB = d;
  d += kSpmvMaxBlocks;
  c.sqY = d;
  d += kSpmvMaxBlocks;
  c.sqW = d;
  d += kSpmvMaxBlocks;
  c.hn = d;
  void* ps = base ? (void*)(base + nvec) : nullptr;
  if (!base) RFMLS_CHECK(workspace(h, WS_LSQR_SCAL, sizeof(LsqrDev) * 2, &ps));
  c.dst = (LsqrDev*)ps;
  {
    // column runs of A and A^T, after the state in the caller's scratch or in
    // the handle's workspace
    const int64_t ra = A->m, rt = AT ? AT->m : 0;
    void* pr = base ? (void*)(base + nvec + kStateDoubles) : nullptr;
    if (!base) RFMLS_CHECK(workspace(h, WS_LSQR_RUNS, (size_t)runs_bytes(ra + rt), &pr));
    int32_t* q = (int32_t*)pr;
    auto carve = [&](const rfmls_csr* M, int64_t rows, const int32_t** nr, const int32_t** rc, const int32_t** re) {
      int32_t* n0 = q;
      int32_t* c0 = n0 + rows;
      int32_t* e0 = c0 + rows * kMaxRuns;
      q = e0 + rows * kMaxRuns;
      find_runs(c.st, M, n0, c0, e0);
      *nr = n0;
      *rc = c0;
      *re = e0;
    };
    if (ra > 0) carve(A, ra, &c.nrunA, &c.rcolA, &c.rendA);
    if (rt > 0) carve(AT, rt, &c.nrunAT, &c.rcolAT, &c.rendAT);
    RFMLS_HIP(h, hipGetLastError());
  }
  return RFMLS_OK;
}

// ||v|| of a device vector into c.hn[k] (read by the host later)
static rfmls_status norm_to(Ctx& c, const double* v, int64_t len, int k) {
  const unsigned nb = vec_blocks(len);
  hipLaunchKernelGGL(k_copy_sumsq, dim3(nb), dim3(kThreads), 0, c.st, v, len, (double*)nullptr, c.sqY);
  hipLaunchKernelGGL(k_sqrt_sum, dim3(1), dim3(kThreads), 0, c.st, (const double*)c.sqY, (int)nb, c.hn + k);
  RFMLS_HIP(c.h, hipGetLastError());
  return RFMLS_OK;
}

// One right-hand side at a time; Bm (row-major m x n, or null) is the explicit
// operator B = A R^{-1}.
static rfmls_status solve_impl(rfmls_handle* h, const rfmls_csr* A, const rfmls_csr* AT,
                               const rfmls_precond_t* P, const double* Bm, int64_t ldbm,
                               const double* B, int64_t ldb, int64_t nrhs, double* X, int64_t ldx,
                               double* Rout, int64_t ldr, const rfmls_opts* o, rfmls_info* info,
                               double* base = nullptr) {
  Ctx c;
  RFMLS_CHECK(make_ctx(h, A, AT, P, c, base));
  // the allocation-free variant launches eagerly (instantiating a graph allocates)
  IterGraph graph;
  if (o->graph && !base) c.graph = &graph;
  if (Bm) {
    void* p;
    RFMLS_CHECK(workspace(h, WS_GEMV, sizeof(double) * (size_t)gemvT_slices(h, A->m, A->n) * (size_t)A->n, &p));
    c.Bm = Bm;
    c.ldbm = ldbm;
    c.gpart = (double*)p;
  }
  const int64_t m = A->m, n = A->n;
  const int64_t itmax = o->itmax > 0 ? o->itmax : n;
  const unsigned vbn = vec_blocks(n), vbm = vec_blocks(m);
  // r = b - A x
  LazyScale residual;
  residual.s = -1.0;
  residual.c = -1.0;
  rfmls_status ret = RFMLS_OK;
  for (int64_t k = 0; k < nrhs; ++k) {
    const double* b = B + k * ldb;
    double* x = X + k * ldx;
    rfmls_info inf{};
    double* rres = c.r;
    // from x = 0 the first sweep takes b itself; from a given x every sweep
    // solves for the correction from the true residual r = b - A x
    const bool warm = o->x_init != 0;
    if (warm) {
      RFMLS_CHECK(norm_to(c, b, m, 2));
      RFMLS_CHECK(spmv(c, A, x, rres, residual, b));
    }
    for (int sweep = 0; sweep <= o->refine; ++sweep) {
      const bool from_zero = sweep == 0 && !warm;
      const double* rhs = from_zero ? b : rres;
      LsqrDev s;
      RFMLS_CHECK(lsqr_sweep(c, rhs, o, itmax, &s));
      if (s.istop < 0) return fail(h, RFMLS_E_BREAKDOWN, "non-finite value in LSQR");
      if (sweep == 0) {
        inf.itn_first = s.itn;
        inf.istop = s.istop;
        inf.normr_est = s.normr;
        inf.normar_est = s.normar;
        inf.anorm_est = sqrt(s.anorm2);
        inf.acond_est = s.acond;
        if (!warm) inf.normb = s.bnorm;
        if (s.istop == 7) ret = RFMLS_W_NOCONV;
      }
      inf.itn += s.itn;
      inf.istop_last = s.istop;
      // x (+)= X y
      RFMLS_CHECK(tri_apply(h, P, 0, c.y, from_zero ? x : c.xs));
      if (!from_zero)
        hipLaunchKernelGGL(k_axpby, dim3(vbn), dim3(kThreads), 0, c.st, n, 1.0, (const double*)x, 1.0,
                           (const double*)c.xs, x);
      // r = b - A x
      RFMLS_CHECK(spmv(c, A, x, rres, residual, b));
      if (s.itn == 0) break;
    }
    RFMLS_CHECK(norm_to(c, rres, m, 0));
    RFMLS_CHECK(spmv(c, AT, rres, c.q));
    RFMLS_CHECK(norm_to(c, c.q, n, 1));
    double* pin = (double*)((char*)h->pinned + 3072);
    RFMLS_HIP(h, hipMemcpyAsync(pin, c.hn, 3 * sizeof(double), hipMemcpyDeviceToHost, c.st));
    if (Rout)
      hipLaunchKernelGGL(k_axpby, dim3(vbm), dim3(kThreads), 0, c.st, m, 1.0, (const double*)rres, 0.0,
                         (const double*)nullptr, Rout + k * ldr);
    RFMLS_HIP(h, hipGetLastError());
    RFMLS_HIP(h, hipStreamSynchronize(c.st));
    inf.normr = pin[0];
    inf.normar = pin[1];
    if (warm) inf.normb = pin[2];
    if (info) info[k] = inf;
  }
  RFMLS_HIP(h, hipStreamSynchronize(c.st));
  return ret;
}

rfmls_status run_solve(rfmls_handle* h, const rfmls_csr* A, const rfmls_csr* AT,
                       const rfmls_precond_t* P, const double* B, int64_t ldb, int64_t nrhs,
                       double* X, int64_t ldx, double* Rout, int64_t ldr, const rfmls_opts* o,
                       rfmls_info* info) {
  return solve_impl(h, A, AT, P, nullptr, 0, B, ldb, nrhs, X, ldx, Rout, ldr, o, info);
}

// ---------------------------------------------------------------------------
// Allocation-free variant of the single-right-hand-side solve: its device
// scratch (the vectors, partial sums and LSQR state of make_ctx) lives in one
// file-scope array.  Each device holds its own copy of the array (allocated
// when the library's code object is loaded on that device, kept until the
// process ends); host code reaches it only through the address that
// hipGetSymbolAddress returns for the current device, never through the
// array's name, which on the host is only a stand-in for the symbol.
// ---------------------------------------------------------------------------
namespace noalloc {
constexpr int64_t kScratchDoubles = (int64_t)1 << 22;  // 32 MiB
static __device__ __align__(256) double scratch[kScratchDoubles];
constexpr int kMaxDevices = 64;
static std::mutex mu;
static double* dev_ptr[kMaxDevices] = {};
}  // namespace noalloc

// Called by rfmls_create with h->device current: record this device's
// address of the scratch array (once per device).
rfmls_status noalloc_scratch_init(rfmls_handle* h) {
  std::lock_guard<std::mutex> lk(noalloc::mu);
  if (h->device < 0 || h->device >= noalloc::kMaxDevices)
    return fail(h, RFMLS_E_ARG, "device %d out of range for the allocation-free scratch", h->device);
  if (noalloc::dev_ptr[h->device]) return RFMLS_OK;
  void* p = nullptr;
  hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(noalloc::scratch));
  if (e != hipSuccess || !p) {
    (void)hipGetLastError();
    return fail(h, RFMLS_E_HIP, "hipGetSymbolAddress(scratch) on device %d: %s", h->device,
                hipGetErrorString(e));
  }
  noalloc::dev_ptr[h->device] = (double*)p;
  return RFMLS_OK;
}

int64_t noalloc_scratch_bytes() { return noalloc::kScratchDoubles * (int64_t)sizeof(double); }

int64_t noalloc_needed_bytes(int64_t m, int64_t n) {
  return (ctx_doubles(m, n) + kStateDoubles) * (int64_t)sizeof(double) + runs_bytes(m + n);
}

rfmls_status run_solve_noalloc(rfmls_handle* h, const rfmls_csr* A, const rfmls_csr* AT,
                               const rfmls_precond_t* P, const double* B, int64_t ldb, int64_t nrhs,
                               double* X, int64_t ldx, double* Rout, int64_t ldr, const rfmls_opts* o,
                               rfmls_info* info) {
  double* base = nullptr;
  {
    std::lock_guard<std::mutex> lk(noalloc::mu);
    base = (h->device >= 0 && h->device < noalloc::kMaxDevices) ? noalloc::dev_ptr[h->device] : nullptr;
  }
  if (!base) return fail(h, RFMLS_E_HIP, "rfmls_solve_noalloc: no scratch address for device %d", h->device);
  if (noalloc_needed_bytes(A->m, A->n) > noalloc_scratch_bytes())
    return fail(h, RFMLS_E_ARG, "rfmls_solve_noalloc: m = %lld, n = %lld need %lld bytes of scratch, above the "
                "%lld-byte limit", (long long)A->m, (long long)A->n, (long long)noalloc_needed_bytes(A->m, A->n),
                (long long)noalloc_scratch_bytes());
  return solve_impl(h, A, AT, P, nullptr, 0, B, ldb, nrhs, X, ldx, Rout, ldr, o, info, base);
}

rfmls_status run_solve_explicit(rfmls_handle* h, const rfmls_csr* A, const rfmls_csr* AT,
                                const rfmls_precond_t* P, const double* Bm, int64_t ldbm,
                                const double* B, int64_t ldb, int64_t nrhs, double* X, int64_t ldx,
                                double* Rout, int64_t ldr, const rfmls_opts* o, rfmls_info* info) {
  return solve_impl(h, A, AT, P, Bm, ldbm, B, ldb, nrhs, X, ldx, Rout, ldr, o, info);
}

// Backward: LSQR on the consistent system B^T lam = c (c = X^T g), operator
// M = B^T (n x m), tracking lam = B z through the shadow vectors vt, wt (v = B vt).
rfmls_status run_backward(rfmls_handle* h, const rfmls_csr* A, const rfmls_csr* AT,
                          const rfmls_precond_t* P, const double* Xs, int64_t ldx,
                          const double* Rres, int64_t ldr, const double* G, int64_t ldg,
                          int64_t nrhs, double* dB, int64_t lddb, double* dAval,
                          const rfmls_opts* o, rfmls_info* info) {
  Ctx c;
  RFMLS_CHECK(make_ctx(h, A, AT, P, c));
  const int64_t m = A->m, n = A->n;
  const int64_t itmax = o->itmax > 0 ? o->itmax : m;
  const unsigned vbn = vec_blocks(n), vbm = vec_blocks(m);
  // roles: un = beta u (n-vector), vm = alpha v (m-vector), vt/wt/zz shadows (n-vectors)
  double* un = c.z;   // n
  double* vm = c.t;   // m
  double* vt = c.w;   // n
  double* wt = c.q;   // n
  double* zz = c.y;   // n
  double* tmpn = c.xs;  // n
  double* lam = c.r;  // m
  LsqrDev* st = c.dst;
  const int* done = &st->done;
  const LsqrCommit cm = commit_of(c, 1);
  rfmls_status ret = RFMLS_OK;
  IterGraph graph;  // one capture serves every right-hand side (same buffers)
  if (o->graph) c.graph = &graph;
  for (int64_t k = 0; k < nrhs; ++k) {
    int nred = 0, nb = 0;
    // beta_1 u_1 = c = X^T g
    RFMLS_CHECK(tri_apply(h, P, 1, G + k * ldg, un, LazyScale(), nullptr, c.sqB, &nred));
    hipLaunchKernelGGL(k_lsqr_begin, dim3(1), dim3(kThreads), 0, c.st, st, st + 1, (const double*)c.sqB, nred, o->atol,
                       o->btol, o->conlim, itmax);
    // alpha_1 v_1 = M^T u_1 = A (X u_1);  vt_1 = u_1 / alpha_1
    LazyScale s1;
    s1.sdiv = &st->beta;
    RFMLS_CHECK(tri_apply(h, P, 0, un, tmpn, LazyScale(), nullptr, nullptr, nullptr, done));
    RFMLS_CHECK(spmv(c, A, tmpn, vm, s1, nullptr, c.sqA, &nb, done));
    hipLaunchKernelGGL(k_lsqr_begin2, dim3(1), dim3(kThreads), 0, c.st, st, (const double*)c.sqA, nb);
    hipLaunchKernelGGL(k_lsqr_first_w, dim3(vbn), dim3(kThreads), 0, c.st, (const LsqrDev*)st, (const double*)un, 1,
                       vt, wt, zz, n, c.sqW);
    hipLaunchKernelGGL(k_lsqr_w2, dim3(1), dim3(kThreads), 0, c.st, st, (const double*)c.sqW, (int)vbn);
    RFMLS_HIP(h, hipGetLastError());
    LsqrDev s;
    RFMLS_CHECK(run_iterations(c, itmax, o->check_every > 0 ? o->check_every : 8, 1, &s, [&]() -> rfmls_status {
      // beta' u' = X^T (A^T v) - alpha u, with v = v^/alpha and u = u^/beta
      LazyScale su;
      su.sdiv = &st->alpha;
      su.c = 1.0;
      su.cnum = &st->alpha;
      su.cden = &st->beta;
      RFMLS_CHECK(spmv(c, AT, vm, tmpn, LazyScale(), nullptr, nullptr, nullptr, done, cm));
      RFMLS_CHECK(tri_apply(h, P, 1, tmpn, un, su, un, c.sqB, &nred, done));
      // alpha' v' = A (X u') - beta' v, with u' = u^'/beta', beta' from the partial sums;
      // vt' = (u' - beta' vt) / alpha' in k_lsqr_step
      LazyScale sv;
      sv.c = 1.0;
      sv.sq = c.sqB;
      sv.nsq = nred;
      sv.norm = &st->beta;
      sv.cden = &st->alpha;
      RFMLS_CHECK(tri_apply(h, P, 0, un, tmpn, LazyScale(), nullptr, nullptr, nullptr, done));
      RFMLS_CHECK(spmv(c, A, tmpn, vm, sv, vm, c.sqA, &nb, done));
      hipLaunchKernelGGL(k_lsqr_step, dim3(vbn), dim3(kThreads), 0, c.st, (const LsqrDev*)st, st + 1,
                         (const double*)c.sqA, nb, (const double*)un, vt, wt, zz, n, c.sqY, c.sqW);
      RFMLS_HIP(h, hipGetLastError());
      return RFMLS_OK;
    }));
    if (s.istop < 0) return fail(h, RFMLS_E_BREAKDOWN, "non-finite value in backward LSQR");
    if (s.istop == 7) ret = RFMLS_W_NOCONV;
    if (info) {
      rfmls_info inf{};
      inf.itn = inf.itn_first = s.itn;
      inf.istop = inf.istop_last = s.istop;
      inf.normr_est = s.normr;
      inf.normb = s.bnorm;
      info[k] = inf;
    }
    // w = X z (into tmpn), lam = A w
    RFMLS_CHECK(tri_apply(h, P, 0, zz, tmpn));
    RFMLS_CHECK(spmv(c, A, tmpn, lam));
    if (dB)
      hipLaunchKernelGGL(k_axpby, dim3(vbm), dim3(kThreads), 0, c.st, m, 1.0, (const double*)lam, 0.0,
                         (const double*)nullptr, dB + k * lddb);
    if (dAval)
      hipLaunchKernelGGL(k_pattern_grad, dim3(spmv_blocks(m)), dim3(kThreads), 0, c.st, A->row_ptr,
                         A->col, m, Rres + k * ldr, (const double*)tmpn, (const double*)lam,
                         Xs + k * ldx, dAval, k > 0 ? 1 : 0);
    RFMLS_HIP(h, hipGetLastError());
  }
  RFMLS_HIP(h, hipStreamSynchronize(c.st));
  return ret;
}

}  // namespace rfmls
