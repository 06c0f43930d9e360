// Lockstep LSQR for a block of right-hand sides (up to kBlk = 32 at a time).
//
// Each column runs exactly the single-right-hand-side recurrences of lsqr.hip
// (its own alpha, beta, rotation, stopping test); the columns only share the
// passes over the matrices:
//   Z = X V        triangular product with the packed X = R^{-1}: each 64 x 64
//                  tile of X meets a 64 x 32 block of V on the matrix cores
//                  (v_mfma_f64_16x16x4f64), so X is streamed once per
//                  iteration for all 32 columns instead of 32 times
//   U = A Z - U a  CSR SpMM: 64-row groups times LDS-staged 32-wide input windows
//                  on the matrix cores
//   Q = A^T U      the same with the transpose
//   V = X^T Q - V b
// Vectors are interleaved row-major blocks (element (i, c) at i * 32 + c).  As in
// the single-column loop, u and v are kept unnormalised (beta u, alpha v): the next
// product divides by the norm (BlkScale), and the update kernel's workgroups form the
// rotation themselves, so that no pass only scales a block and no launch only
// computes scalars.
// A column that has stopped keeps its y and x; the host polls one
// "all columns done" flag every few iterations.
#include <algorithm>
#include <cstring>

#include "common.h"
#include "lsqr_dev.h"
#include "runs.h"

namespace rfmls {

constexpr int kBlk = 32;

namespace {

constexpr int kThreads = 256;
constexpr int kSpmmMaxBlocks = 2048;  // capacity of the per-column partial-sum buffers
// Producers of per-column partial sums use at most these many blocks (grid-
// stride loops).
constexpr int kSpmmBlocks = 512;
constexpr int kRowBlocks = 1024;  // 8-row blocks: enough loads in flight for the row-wise passes

typedef double v4d __attribute__((ext_vector_type(4)));

struct BlockState {
  LsqrDev col[kBlk];
  int all_done;  // (in the uncommitted state: whether it holds an iteration)
  int pad[15];
};

__device__ __forceinline__ bool all_done(const BlockState* st) { return st->all_done != 0; }
__device__ __forceinline__ double inv_or_0(double x) { return x > 0.0 ? 1.0 / x : 0.0; }

constexpr int kStride = (int)(sizeof(LsqrDev) / sizeof(double));  // between columns' states, in doubles
static_assert(sizeof(LsqrDev) % sizeof(double) == 0, "LsqrDev must be a whole number of doubles");

// Per-column sums of squares: producers leave partials sq[block][32], k_blk_presum
// folds them into kPre rows, and every consumer adds those itself.
constexpr int kPre = 32;
__device__ __forceinline__ double blk_total(const double* __restrict__ pre, int c) {
  double v[kPre];
#pragma unroll
  for (int z = 0; z < kPre; ++z) v[z] = pre[z * kBlk + c];
#pragma unroll
  for (int o = kPre / 2; o > 0; o >>= 1)
#pragma unroll
    for (int z = 0; z < o; ++z) v[z] += v[z + o];
  return v[0];
}

// Scalars of column c in out = s acc - c prev; the fields as LazyScale's (common.h),
// each pointer at column 0's value, columns kStride apart; pre: the folded sums of
// the block just multiplied, whose norm one thread per column (writer) stores in
// norm while the column is active.
struct BlkScale {
  double s = 1.0, c = 0.0;
  const double* sdiv = nullptr;
  const double *cnum = nullptr, *cden = nullptr;
  const double* pre = nullptr;
  double* norm = nullptr;
};
__device__ __forceinline__ void blk_scale(const BlkScale& B, int c, bool writer, double* s, double* cf) {
  *s = B.s;
  *cf = B.c;
  if (B.pre) {
    const double nu = sqrt(blk_total(B.pre, c));
    if (writer && B.norm) B.norm[c * kStride] = nu;
    *s *= inv_or_0(nu);
    if (B.cden) *cf *= nu * inv_or_0(B.cden[c * kStride]);
  } else {
    if (B.sdiv) *s *= inv_or_0(B.sdiv[c * kStride]);
    if (B.cnum) *cf *= B.cnum[c * kStride] * inv_or_0(B.cden[c * kStride]);
  }
}

// Takes the state an iteration left in next into st, with the sums of its y and w
// and the stopping tests, by one workgroup of kThreads (commit_state of the
// single-column loop, per column).
struct BlkCommit {
  BlockState* st = nullptr;
  BlockState* next = nullptr;
  const double *ysq = nullptr, *wsq = nullptr;
  int n = 0;
  int consistent = 0;
};
__device__ void all_done_update(BlockState* st) {
  int all = 1;
  for (int c = 0; c < kBlk; ++c) all &= st->col[c].done != 0;
  st->all_done = all;
}
__device__ void commit_block(const BlkCommit& cm, double (*red)[kBlk]) {
  if (!cm.next->all_done) return;  // uniform
  const int c = threadIdx.x % kBlk, rsub = threadIdx.x / kBlk;
  constexpr int kR = kThreads / kBlk;
  double y2 = 0.0, w2 = 0.0;
#pragma unroll 4
  for (int b = rsub; b < cm.n; b += kR) {
    y2 += cm.ysq[b * kBlk + c];
    w2 += cm.wsq[b * kBlk + c];
  }
  red[rsub][c] = y2;
  red[kR + rsub][c] = w2;
  __syncthreads();
  if (rsub == 0) {
    y2 = w2 = 0.0;
    for (int q = 0; q < kR; ++q) {
      y2 += red[q][c];
      w2 += red[kR + q][c];
    }
    LsqrDev s = cm.next->col[c];
    if (s.fresh) {
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
      cm.st->col[c] = s;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    cm.next->all_done = 0;
    all_done_update(cm.st);
  }
}
__global__ void __launch_bounds__(kThreads) k_blk_commit(BlkCommit cm) {
  __shared__ double red[2 * kThreads / kBlk][kBlk];
  commit_block(cm, red);
}

// ---------------------------------------------------------------------------
// Triangular products with 64 x 32 blocks on the matrix cores.
// Wave w computes rows 16 w .. 16 w + 15 of the 64-row output block, both
// 16-column halves.  Operand layout of v_mfma_f64_16x16x4f64: lane l holds
// A[l % 16][l / 16] and B[l / 16][l % 16]; accumulator register r holds
// D[l / 16 + 4 r][l % 16].
// ---------------------------------------------------------------------------
// Z = X V for a 64-row tile row: each 64 x 64 tile of X is staged in LDS with
// coalesced loads (the next tile prefetched into registers meanwhile), as is
// the matching 64 x 32 block of V; the MFMA operands are then read from LDS.
// Reading the A operand (16 rows x 4 columns per instruction) straight from
// HBM would fetch 32-byte pieces of 16 different rows per load.
template <typename TS>
__global__ void __launch_bounds__(kThreads)
    k_trmm_part(const TS* __restrict__ Xpk, int64_t nt, int64_t n, int full, const int2* __restrict__ tab,
                int C, int maxk, const double* __restrict__ V, double* __restrict__ part,
                const BlockState* __restrict__ st, BlkCommit cm) {
  // the last workgroup commits the iteration before; the others use nothing of the
  // state but the stop word, whose early or late setting changes no result
  const bool committing = cm.st && blockIdx.x == gridDim.x - 1;
  if (!committing && st && all_done(st)) return;
  constexpr int kPer = kTile * kTile / kThreads;  // 16 X elements per thread per tile
  __shared__ TS Xs[kTile][kTile + 1];
  __shared__ double Vs[kTile][kBlk + 1];
  if (committing) {
    commit_block(cm, (double (*)[kBlk])&Vs[0][0]);
    return;
  }
  const int2 e = tab[blockIdx.x];
  const int64_t I = e.x;
  const int k = e.y;
  const int64_t J0 = row_first(I, full) + (int64_t)k * C;
  const int64_t J1 = J0 + C < nt ? J0 + C : nt;
  const int tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  v4d acc0 = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
  TS xr[kPer];
  double vr[kTile * kBlk / kThreads];  // 8 V elements per thread
  auto fetch = [&](int64_t J) {
    const TS* t = Xpk + ptile(I, J, nt, full) * (int64_t)(kTile * kTile);
#pragma unroll
    for (int q = 0; q < kPer; ++q) xr[q] = t[tid + q * kThreads];
#pragma unroll
    for (int q = 0; q < kTile * kBlk / kThreads; ++q) {
      const int idx = tid + q * kThreads;  // (row, col) = (idx / 32, idx % 32)
      const int64_t r = J * kTile + idx / kBlk;
      vr[q] = r < n ? V[r * kBlk + (idx % kBlk)] : 0.0;
    }
  };
  if (J0 < J1) fetch(J0);
  for (int64_t J = J0; J < J1; ++J) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int idx = tid + q * kThreads;
      Xs[idx / kTile][idx % kTile] = xr[q];
    }
#pragma unroll
    for (int q = 0; q < kTile * kBlk / kThreads; ++q) {
      const int idx = tid + q * kThreads;
      Vs[idx / kBlk][idx % kBlk] = vr[q];
    }
    __syncthreads();
    if (J + 1 < J1) fetch(J + 1);
#pragma unroll
    for (int s4 = 0; s4 < kTile / 4; ++s4) {
      const int kk = 4 * s4 + lk;
      const double a = (double)Xs[16 * w + lr][kk];
      acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Vs[kk][lr], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Vs[kk][16 + lr], acc1, 0, 0, 0);
    }
  }
  double* o = part + ((int64_t)I * maxk + k) * (kTile * kBlk);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = 16 * w + lk + 4 * r;
    o[row * kBlk + lr] = acc0[r];
    o[row * kBlk + 16 + lr] = acc1[r];
  }
}

// P = X^T Q for a 64-column tile column J: tiles I in [k C, min((k+1) C, J+1)),
// staged in LDS like k_trmm_part (the operand is the tile read transposed).
template <typename TS>
__global__ void __launch_bounds__(kThreads)
    k_trmmT_part(const TS* __restrict__ Xpk, int64_t nt, int64_t n, int full, const int2* __restrict__ tab,
                 int C, int maxk, const double* __restrict__ Qv, double* __restrict__ part,
                 const BlockState* __restrict__ st, BlkCommit cm) {
  // the last workgroup commits the iteration before; the others use nothing of the
  // state but the stop word, whose early or late setting changes no result
  const bool committing = cm.st && blockIdx.x == gridDim.x - 1;
  if (!committing && st && all_done(st)) return;
  constexpr int kPer = kTile * kTile / kThreads;
  __shared__ TS Xs[kTile][kTile + 1];
  __shared__ double Qs[kTile][kBlk + 1];
  if (committing) {
    commit_block(cm, (double (*)[kBlk])&Qs[0][0]);
    return;
  }
  const int2 e = tab[blockIdx.x];
  const int64_t J = e.x;
  const int k = e.y;
  const int64_t I0 = (int64_t)k * C;
  const int64_t Iend = col_end(J, nt, full);
  const int64_t I1 = I0 + C < Iend ? I0 + C : Iend;
  const int tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  v4d acc0 = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
  TS xr[kPer];
  double qr[kTile * kBlk / kThreads];
  auto fetch = [&](int64_t I) {
    const TS* t = Xpk + ptile(I, J, nt, full) * (int64_t)(kTile * kTile);
#pragma unroll
    for (int q = 0; q < kPer; ++q) xr[q] = t[tid + q * kThreads];
#pragma unroll
    for (int q = 0; q < kTile * kBlk / kThreads; ++q) {
      const int idx = tid + q * kThreads;
      const int64_t r = I * kTile + idx / kBlk;
      qr[q] = r < n ? Qv[r * kBlk + (idx % kBlk)] : 0.0;
    }
  };
  if (I0 < I1) fetch(I0);
  for (int64_t I = I0; I < I1; ++I) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int idx = tid + q * kThreads;
      Xs[idx / kTile][idx % kTile] = xr[q];
    }
#pragma unroll
    for (int q = 0; q < kTile * kBlk / kThreads; ++q) {
      const int idx = tid + q * kThreads;
      Qs[idx / kBlk][idx % kBlk] = qr[q];
    }
    __syncthreads();
    if (I + 1 < I1) fetch(I + 1);
#pragma unroll
    for (int s4 = 0; s4 < kTile / 4; ++s4) {
      const int kk = 4 * s4 + lk;  // row of the X tile = column of X^T
      const double a = (double)Xs[kk][16 * w + lr];
      acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Qs[kk][lr], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Qs[kk][16 + lr], acc1, 0, 0, 0);
    }
  }
  double* o = part + ((int64_t)J * maxk + k) * (kTile * kBlk);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = 16 * w + lk + 4 * r;
    o[row * kBlk + lr] = acc0[r];
    o[row * kBlk + 16 + lr] = acc1[r];
  }
}

// out[i][c] = s_c sum_k part[...][i][c] - coef_c prev[i][c]; per-column partial sums of
// squares.  Thread (i, c) with c = tid % 32.
__global__ void __launch_bounds__(kThreads)
    k_blk_tri_reduce(const double* __restrict__ part, int64_t nt, int64_t n, int full, int C, int maxk,
                     int trans, BlkScale sc, const double* prev, double* out, double* __restrict__ sq,
                     const BlockState* __restrict__ st) {
  if (st && all_done(st)) return;
  __shared__ double red[kThreads / kBlk][kBlk];
  const int c = threadIdx.x % kBlk;
  const int rsub = threadIdx.x / kBlk;
  const bool act = !st || !st->col[c].done;
  double s1, cf;
  blk_scale(sc, c, blockIdx.x == 0 && rsub == 0 && act, &s1, &cf);
  double ss = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * (kThreads / kBlk) + rsub; i < n;
       i += (int64_t)gridDim.x * (kThreads / kBlk)) {
    const int64_t I = i / kTile;
    const int r = (int)(i % kTile);
    const int64_t nk = trans ? (col_end(I, nt, full) + C - 1) / C : (nt - row_first(I, full) + C - 1) / C;
    double s = 0.0;
    // the partials in chunk order; the loads of eight at a time are in flight together
    const double* pp = part + ((I * maxk) * kTile + r) * kBlk + c;
    int64_t kq = 0;
    for (; kq + 8 <= nk; kq += 8) {
      double v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = pp[(kq + q) * kTile * kBlk];
#pragma unroll
      for (int q = 0; q < 8; ++q) s += v[q];
    }
    for (; kq < nk; ++kq) s += pp[kq * kTile * kBlk];
    s *= s1;
    if (prev && cf != 0.0) s -= cf * prev[i * kBlk + c];
    if (act) out[i * kBlk + c] = s;
    ss += s * s;
  }
  if (sq) {
    red[rsub][c] = ss;
    __syncthreads();
    if (rsub == 0) {
      double t = 0.0;
      for (int q = 0; q < kThreads / kBlk; ++q) t += red[q][c];
      sq[blockIdx.x * kBlk + c] = t;
    }
  }
}

// Entries [*b, *e) of row r in split z of nsplit: the columns in the z-th of
// nsplit ranges cut at equal-count points of the group's first row r0 (binary
// searches; malformed rows give some range, never one outside the row).
__device__ __forceinline__ void spmm_split_range(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                 int64_t r0, int64_t r, int nsplit, int z, int64_t* b_out,
                                                 int64_t* e_out) {
  const int64_t b = rp[r], e = rp[r + 1];
  const int64_t f0 = rp[r0], len0 = rp[r0 + 1] - rp[r0];
  const int32_t lo = z == 0 ? INT32_MIN : (len0 > 0 ? col[f0 + (int64_t)z * len0 / nsplit] : INT32_MAX);
  const int32_t hi = z == nsplit - 1 ? INT32_MAX : (len0 > 0 ? col[f0 + (int64_t)(z + 1) * len0 / nsplit] : INT32_MAX);
  int64_t a = b, c2 = e;
  while (a < c2) {
    const int64_t mid = (a + c2) / 2;
    if (col[mid] < lo) a = mid + 1;
    else c2 = mid;
  }
  int64_t a2 = a, c3 = e;
  if (hi != INT32_MAX) {
    while (a2 < c3) {
      const int64_t mid = (a2 + c3) / 2;
      if (col[mid] < hi) a2 = mid + 1;
      else c3 = mid;
    }
  } else {
    a2 = e;
  }
  *b_out = a;
  *e_out = a2;
}

// CSR SpMM on the matrix cores:
//   out[row][c] = s_c (M Xin)[row][c] - coef_c prev[row][c],  c < 32,
// plus per-column partial sums of squares of out.  Rows go in groups of
// kSpmmGroup (64), wavefront w of a workgroup rows 16 w .. 16 w + 15; a group's
// (ascending) column indices are walked in windows of W input rows, each
// starting at a multiple of 4: the window's 32-wide input rows are staged in
// LDS, the group's entries that fall in it are scattered into a dense 64 x W
// tile (zeros elsewhere), and each wavefront multiplies its 16 x W slab by the
// W x 32 window (v_mfma_f64_16x16x4f64, two 16 x 16 output tiles).  Rows of one
// RFM box share their column runs, so the tile is nearly dense and every staged
// input row serves 64 rows through the matrix cores.  Column j always falls in
// the K step of its aligned quad j / 4, so every output is the same ordered sum
// of quads whatever W is: the window width changes no result.
//
// The walk depends only on the matrix, so k_spmm_walk runs it once per solve
// and records descriptors: per work item its windows, per window its start
// column, per window and row the row's first entry in it and their number (the
// row's entries in order until the first one outside the window).  k_spmm then
// only loads and multiplies.  Malformed input (columns out of order or out of
// range) ends a prefix early and cannot make either kernel read outside Xin or
// LDS.
//
// Split groups (nsplit > 1, for matrices with few long rows): work item
// (group, z) takes only the entries whose column lies in the z-th of nsplit
// ranges cut at equal-count points of the group's first row, and writes its
// raw sums to part[z][row][32]; k_spmm_merge adds the nsplit parts in order and
// applies the scaling, the subtraction and the sums of squares.
constexpr int kSpmmGroup = 64;
constexpr int kDescCntShift = 48;  // descriptor: first entry | count << 48

// One pass of the window walk over every work item.  Count pass: wcount[item]
// = its number of windows.  Fill pass (wptr = exclusive scan of the counts):
// window k of the item (global index wptr[item] + k) gets its start in
// wstart[k] and, for each of the group's 64 rows, the descriptor in
// wdesc[k * 64 + row].
template <int W, bool Fill>
__global__ void __launch_bounds__(kThreads)
    k_spmm_walk(const int64_t* __restrict__ rp, const int32_t* __restrict__ col, int64_t rows, int nsplit,
                int32_t* __restrict__ wcount, const int64_t* __restrict__ wptr, int32_t* __restrict__ wstart,
                int64_t* __restrict__ wdesc) {
  static_assert(W % 32 == 0 && W <= 128, "window");
  constexpr int kH = (W + 63) / 64;
  __shared__ int64_t cur[kSpmmGroup], endp[kSpmmGroup];
  __shared__ int wmin[4];
  __shared__ int w0_s;
  const int tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6;
  const int64_t ngroups = (rows + kSpmmGroup - 1) / kSpmmGroup;
  for (int64_t wi = blockIdx.x; wi < ngroups * nsplit; wi += gridDim.x) {
    const int64_t gi = wi / nsplit;
    const int z = (int)(wi % nsplit);
    const int64_t r0 = gi * kSpmmGroup;
    if (tid < kSpmmGroup) {
      const int64_t r = r0 + tid;
      int64_t b = r < rows ? rp[r] : 0, e = r < rows ? rp[r + 1] : 0;
      if (nsplit > 1 && r < rows) spmm_split_range(rp, col, r0, r, nsplit, z, &b, &e);
      cur[tid] = b;
      endp[tid] = e;
    }
    __syncthreads();
    if (w == 0) {
      // first window: the smallest first column of the group
      int m0 = cur[lane] < endp[lane] ? col[cur[lane]] : INT32_MAX;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        const int o = __shfl_xor(m0, off, 64);
        m0 = o < m0 ? o : m0;
      }
      if (lane == 0) w0_s = m0;
    }
    __syncthreads();
    int w0 = w0_s == INT32_MAX ? INT32_MAX : (w0_s & ~3);
    int64_t k = Fill ? wptr[wi] : 0;
    while (w0 != INT32_MAX) {  // uniform
      // each row's in-window prefix: its entries in order until the first one
      // outside the window; its next column is none if the row is finished,
      // its first entry left if the window took none of it, else at least
      // w0 + W (it took entries up to the first that is not in the window,
      // whose column, the columns ascending, lies beyond it)
      const int lb = (int)((int64_t)w0 + W < (int64_t)INT32_MAX ? (int64_t)w0 + W : (int64_t)INT32_MAX - 1);
      int nxt = INT32_MAX;
      for (int rr = 0; rr < 16; ++rr) {
        const int row = 16 * w + rr;
        const int64_t base = cur[row], end = endp[row];
        int fb = W, c0 = 0;
#pragma unroll
        for (int h = 0; h < kH; ++h) {
          const int j = lane + 64 * h;
          const int64_t e = base + j;
          const bool in = j < W && e < end;
          const int cj = in ? col[e] : 0;
          if (h == 0) c0 = cj;
          const int cc = cj - w0;
          const bool ok = in && cc >= 0 && cc < W;
          const unsigned long long bad = __ballot(j < W && !ok);
          if (bad) {
            const int f = 64 * h + __builtin_ctzll(bad);
            fb = f < fb ? f : fb;
          }
        }
        int rn;
        if (base + fb >= end) rn = INT32_MAX;
        else if (fb == 0) rn = __builtin_amdgcn_readlane(c0, 0);
        else rn = lb;
        nxt = rn < nxt ? rn : nxt;
        if (lane == 0) {
          if (Fill) wdesc[k * kSpmmGroup + row] = base | ((int64_t)fb << kDescCntShift);
          cur[row] = base + fb;
        }
      }
      if (lane == 0) wmin[w] = nxt;
      if (Fill && tid == 0) wstart[k] = w0;
      __syncthreads();
      int wn = wmin[0];
#pragma unroll
      for (int q = 1; q < 4; ++q) wn = wmin[q] < wn ? wmin[q] : wn;
      w0 = wn == INT32_MAX ? INT32_MAX : (wn & ~3);
      ++k;
      __syncthreads();
    }
    if (!Fill && tid == 0) wcount[wi] = (int32_t)k;
  }
}

template <int W>
__global__ void __launch_bounds__(kThreads)
    k_spmm(const int32_t* __restrict__ col, const double* __restrict__ val, int64_t rows, int64_t ncols,
           const double* __restrict__ Xin, BlkScale sc, const double* prev, double* out, double* __restrict__ sq,
           const BlockState* __restrict__ st, int nsplit,
           double* __restrict__ part, const int64_t* __restrict__ wptr, const int32_t* __restrict__ wstart,
           const int64_t* __restrict__ wdesc) {
  static_assert(W % 32 == 0 && W <= 128, "window");
  if (st && all_done(st)) return;
  __shared__ double Xs[W][kBlk];
  __shared__ double At[kSpmmGroup][W + 1];
  __shared__ double red[kThreads / 16][kBlk];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  double sA[2], cf[2];
  bool act[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int c = 16 * q + lr;
    act[q] = !st || !st->col[c].done;
    if (nsplit == 1) blk_scale(sc, c, blockIdx.x == 0 && w == 0 && lk == 0 && act[q], &sA[q], &cf[q]);
  }
  double ss[2] = {0.0, 0.0};
  // Window data in registers: the input rows [w0, w0 + W) (coalesced, 32
  // doubles per row) and, per wavefront, each of its 16 rows' entries in the
  // window (64 lanes over consecutive entries).  The next window's are loaded
  // while the matrix cores work on the current one.
  constexpr int kXPer = W * kBlk / kThreads;
  constexpr int kH = (W + 63) / 64;
  double xr[kXPer];
  int cj[16][kH];
  double vj[16][kH];
  int w0 = 0;
  auto load = [&](int64_t k) {
    w0 = wstart[k];
#pragma unroll
    for (int q = 0; q < kXPer; ++q) {
      const int e = tid + q * kThreads;
      const int64_t r = (int64_t)w0 + e / kBlk;
      xr[q] = (r >= 0 && r < ncols) ? Xin[r * kBlk + (e % kBlk)] : 0.0;
    }
#pragma unroll
    for (int rr = 0; rr < 16; ++rr) {
      const int64_t d = wdesc[k * kSpmmGroup + 16 * w + rr];
      const int64_t base = d & ((1ll << kDescCntShift) - 1);
      const int cnt = (int)(d >> kDescCntShift);
#pragma unroll
      for (int h = 0; h < kH; ++h) {
        const int j = lane + 64 * h;
        const bool in = j < cnt;
        cj[rr][h] = in ? col[base + j] : -1;
        vj[rr][h] = in ? val[base + j] : 0.0;
      }
    }
  };
  const int64_t items = ((rows + kSpmmGroup - 1) / kSpmmGroup) * nsplit;
  // the last items first: a matrix's last rows (the RFM's interface rows, two
  // boxes' columns each) have the most windows, and blocks are dispatched in order
  for (int64_t wb = blockIdx.x; wb < items; wb += gridDim.x) {
    const int64_t wi = items - 1 - wb;
    const int64_t gi = wi / nsplit;
    const int z = (int)(wi % nsplit);
    const int64_t r0 = gi * kSpmmGroup;
    const int64_t kb = wptr[wi], ke = wptr[wi + 1];
    v4d acc[2] = {v4d{0.0, 0.0, 0.0, 0.0}, v4d{0.0, 0.0, 0.0, 0.0}};
    if (kb < ke) load(kb);
    for (int64_t k = kb; k < ke; ++k) {
      // the tile starts empty (the previous window's products are done)
      for (int e = tid; e < kSpmmGroup * W; e += kThreads) At[e / W][e % W] = 0.0;
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kXPer; ++q) {
        const int e = tid + q * kThreads;
        Xs[e / kBlk][e % kBlk] = xr[q];
      }
#pragma unroll
      for (int rr = 0; rr < 16; ++rr)
#pragma unroll
        for (int h = 0; h < kH; ++h)
          if (cj[rr][h] >= 0) At[16 * w + rr][cj[rr][h] - w0] = vj[rr][h];
      __syncthreads();
      if (k + 1 < ke) load(k + 1);
      // the wavefront's 16 x W slab times the W x 32 window
#pragma unroll 4
      for (int s4 = 0; s4 < W / 4; ++s4) {
        const double a = At[16 * w + lr][4 * s4 + lk];
        const double b0 = Xs[4 * s4 + lk][lr], b1 = Xs[4 * s4 + lk][16 + lr];
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b0, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b1, acc[1], 0, 0, 0);
      }
      __syncthreads();
    }
    // register r of tile q: row 16 w + lk + 4 r, column 16 q + lr
    if (nsplit > 1) {
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t row = r0 + 16 * w + lk + 4 * r;
          if (row < rows) part[((int64_t)z * rows + row) * kBlk + 16 * q + lr] = acc[q][r];
        }
      continue;
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t row = r0 + 16 * w + lk + 4 * r;
        const int c = 16 * q + lr;
        if (row < rows) {
          double o = sA[q] * acc[q][r];
          if (prev && cf[q] != 0.0) o -= cf[q] * prev[row * kBlk + c];
          if (act[q]) out[row * kBlk + c] = o;
          ss[q] += o * o;
        }
      }
  }
  if (sq) {
    // per column: the 16 lane groups (4 per wavefront) in order
#pragma unroll
    for (int q = 0; q < 2; ++q) red[4 * w + lk][16 * q + lr] = ss[q];
    __syncthreads();
    if (tid < kBlk) {
      double t = 0.0;
      for (int g = 0; g < kThreads / 16; ++g) t += red[g][tid];
      sq[blockIdx.x * kBlk + tid] = t;
    }
  }
}

// out[row][c] = s_c sum_z part[z][row][c] (z in order) - cf_c prev[row][c] for the
// rows of a split SpMM; per-column sums of squares per block as k_spmm's.
__global__ void __launch_bounds__(kThreads)
    k_spmm_merge(const double* __restrict__ part, int nsplit, int64_t rows, BlkScale sc, const double* prev,
                 double* out, double* __restrict__ sq, const BlockState* __restrict__ st) {
  if (st && all_done(st)) return;
  __shared__ double red[kThreads / kBlk][kBlk];
  const int c = threadIdx.x % kBlk, rsub = threadIdx.x / kBlk;
  const bool act = !st || !st->col[c].done;
  double sA, cf;
  blk_scale(sc, c, blockIdx.x == 0 && rsub == 0 && act, &sA, &cf);
  double ss = 0.0;
  for (int64_t row = (int64_t)blockIdx.x * (kThreads / kBlk) + rsub; row < rows;
       row += (int64_t)gridDim.x * (kThreads / kBlk)) {
    double a = 0.0;
#pragma unroll 8
    for (int z = 0; z < nsplit; ++z) a += part[((int64_t)z * rows + row) * kBlk + c];
    double o = sA * a;
    if (prev && cf != 0.0) o -= cf * prev[row * kBlk + c];
    if (act) out[row * kBlk + c] = o;
    ss += o * o;
  }
  if (sq) {
    red[rsub][c] = ss;
    __syncthreads();
    if (threadIdx.x < kBlk) {
      double t = 0.0;
      for (int q = 0; q < kThreads / kBlk; ++q) t += red[q][threadIdx.x];
      sq[blockIdx.x * kBlk + threadIdx.x] = t;
    }
  }
}

// ---------------------------------------------------------------------------
// SpMM over column runs.  Consecutive rows of an RFM matrix (the collocation
// points of one box, face or interface) and of its transpose (the features of
// one box) hold the same runs of consecutive columns, so up to 64 such rows, a
// "piece", are dense blocks: each run's entries are a rows x length slab whose
// row r lies contiguous at val + rp[r], and its input rows are contiguous too.
// The slabs are read straight into the matrix cores' operand registers; no
// column index is read, nothing is scattered through LDS and there is no
// window walk.
//
// Bound: HBM for the values (8 bytes an entry) beside the float64 matrix
// cores (64 flops an entry; the two take about equally long).  Split: one
// workgroup per (piece, K chunk); its four wavefronts take every fourth
// 16-entry step of each run for all 64 rows, so an input row is read once per
// piece, and their sums are added in a fixed order through LDS.  Inside a step
// the K order is permuted: lane (lr, lk) holds entries 4 lk .. 4 lk + 3 of row
// lr (two 16-byte loads, 128 contiguous bytes per row over the four lanes) and
// columns 2 lr, 2 lr + 1 of the input rows (16-byte loads); instruction j
// multiplies entries 4 lk + j.
// Measured, 32 columns, Helmholtz system (37.1 M entries, A and A^T): 82 us on
// average (3.6 TB/s of values, 29 TFLOP/s) where the windowed kernel took 139
// (A) and 530 us (A^T) and its walk 2 ms a call; 32 right-hand sides 42.1 ->
// 14.1 ms.  See spmm_prepare for which matrices take this kernel.
// ---------------------------------------------------------------------------
constexpr int kRunStep = 16;
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

struct RunMat {
  const int64_t* rp;
  const double* val;
  const int32_t *nrun, *rcol, *rend;  // column runs (find_runs), kMaxRuns per row
  const int2* pieces;                 // first row, rows
  int64_t npieces, rows;
  int nsplit;
  int64_t kchunk;                     // entries per K chunk, a multiple of kRunStep
};

// Pieces of each 64-row group (group_pieces).  Count pass: pcount[group]; fill
// pass: pieces from pptr[group] on, and their number in *total.  bad is set when a row has no run description
// or a run leaves the matrix's columns.
template <bool Fill>
__global__ void __launch_bounds__(kThreads)
    k_run_pieces(int64_t rows, int64_t ncols, const int32_t* __restrict__ nrun, const int32_t* __restrict__ rcol,
                 const int32_t* __restrict__ rend, int32_t* __restrict__ pcount, const int64_t* __restrict__ pptr,
                 int2* __restrict__ pieces, int* __restrict__ bad, int64_t* __restrict__ total) {
  // set before, by the probe or the count pass (whose own setting it leaves counts and
  // places unwritten that nothing then reads)
  if (*bad) return;
  const int lane = threadIdx.x & 63;
  const int64_t ngroups = (rows + kPieceRows - 1) / kPieceRows;
  const int64_t nw = (int64_t)gridDim.x * (kThreads / 64);
  if (Fill && blockIdx.x == 0 && threadIdx.x == 0) *total = pptr[ngroups];
  for (int64_t g = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6); g < ngroups; g += nw) {
    unsigned long long starts, lives, wrong;
    group_pieces(g, rows, ncols, nrun, rcol, rend, &starts, &lives, &wrong);
    if (!Fill) {
      if (lane == 0) {
        pcount[g] = __popcll(starts);
        if (wrong) atomicOr(bad, 1);
      }
    } else if (starts >> lane & 1) {
      const unsigned long long below = starts & ((1ull << lane) - 1ull);
      pieces[pptr[g] + __popcll(below)] = make_int2((int)(g * kPieceRows + lane), piece_len(starts, lives, lane));
    }
  }
}

template <int NG>
__device__ __forceinline__ void run_piece_product(const RunMat& M, int64_t row0, int nrows, int64_t e0, int64_t e1,
                                                  int w, int lr, int lk, const double* __restrict__ Xin,
                                                  v4d (&acc)[4][2]) {
  const double* ar[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const int r = 16 * g + lr;  // rows past the piece repeat its last (their sums are not stored)
    ar[g] = M.val + M.rp[row0 + (r < nrows ? r : nrows - 1)];
  }
  struct Step {
    double a[NG][4], b[4][2];
  };
  auto mma = [&](const Step& s) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        acc[g][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(s.a[g][j], s.b[j][0], acc[g][0], 0, 0, 0);
        acc[g][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(s.a[g][j], s.b[j][1], acc[g][1], 0, 0, 0);
      }
  };
  const int nr = M.nrun[row0];
  int32_t off = 0;
  for (int k = 0; k < nr; ++k) {
    const int32_t end = M.rend[row0 * kMaxRuns + k];
    const int64_t s0 = off > e0 ? off : e0, s1 = end < e1 ? end : e1;
    // input row of entry e: (column of the run's first entry) + e - off
    const double* xr = Xin + ((int64_t)M.rcol[row0 * kMaxRuns + k] - off) * kBlk + 2 * lr;
    off = end;
    if (s0 >= s1) continue;
    auto load = [&](Step& s, int64_t step) {
      const int64_t e = s0 + step * kRunStep + 4 * lk;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const d2u* p = (const d2u*)(ar[g] + e);
        const d2u x = p[0], y = p[1];
        s.a[g][0] = x[0];
        s.a[g][1] = x[1];
        s.a[g][2] = y[0];
        s.a[g][3] = y[1];
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const d2u v = *(const d2u*)(xr + (e + j) * kBlk);
        s.b[j][0] = v[0];
        s.b[j][1] = v[1];
      }
    };
    const int64_t nfull = (s1 - s0) / kRunStep;
    int64_t st = w;
    if (st < nfull) {
      // the next step's loads in flight during this one's products
      Step A, B;
      load(A, st);
      for (;;) {
        const bool m1 = st + 4 < nfull;
        if (m1) load(B, st + 4);
        mma(A);
        st += 4;
        if (!m1) break;
        const bool m2 = st + 4 < nfull;
        if (m2) load(A, st + 4);
        mma(B);
        st += 4;
        if (!m2) break;
      }
    }
    if ((s1 - s0) % kRunStep != 0 && nfull % 4 == w) {
      // the run's last entries: lanes past its end read its last entry and multiply zeros
      Step T;
      const int64_t e = s0 + nfull * kRunStep + 4 * lk;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool in = e + j < s1;
        const int64_t ec = in ? e + j : s1 - 1;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const double v = ar[g][ec];
          T.a[g][j] = in ? v : 0.0;
        }
        const d2u v = *(const d2u*)(xr + ec * kBlk);
        T.b[j][0] = in ? v[0] : 0.0;
        T.b[j][1] = in ? v[1] : 0.0;
      }
      mma(T);
    }
  }
}

// last_first: the workgroups dispatched first take the last pieces (an RFM
// matrix's last rows, the interfaces, have the longest runs).  The order decides
// only which workgroup is which slot; a slot's pieces, their order and its
// partial sums are the same.
__global__ void __launch_bounds__(kThreads, 2)
    k_spmm_runs(RunMat M, int last_first, const double* __restrict__ Xin, BlkScale sc, const double* prev, double* out,
                double* __restrict__ sq, const BlockState* __restrict__ st, double* __restrict__ part) {
  if (st && all_done(st)) return;
  __shared__ double buf[4][4][4][64];  // wavefront, row group, register, lane
  __shared__ double red[kThreads / 16][kBlk];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  double sA[2], cf[2];
  bool act[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int c = 2 * lr + q;
    act[q] = !st || !st->col[c].done;
    if (M.nsplit == 1) blk_scale(sc, c, blockIdx.x == 0 && w == 0 && lk == 0 && act[q], &sA[q], &cf[q]);
  }
  double ss[2] = {0.0, 0.0};
  const int64_t items = M.npieces * M.nsplit;
  const unsigned slot = last_first ? gridDim.x - 1 - blockIdx.x : blockIdx.x;
  for (int64_t wi = slot; wi < items; wi += gridDim.x) {
    const int z = (int)(wi % M.nsplit);
    const int2 pc = M.pieces[wi / M.nsplit];
    const int64_t row0 = pc.x;
    const int ng = (pc.y + 15) >> 4;
    const int64_t e0 = (int64_t)z * M.kchunk, e1 = z == M.nsplit - 1 ? INT32_MAX : e0 + M.kchunk;
    v4d acc[4][2];
#pragma unroll
    for (int g = 0; g < 4; ++g) acc[g][0] = acc[g][1] = v4d{0.0, 0.0, 0.0, 0.0};
    if (ng == 4) run_piece_product<4>(M, row0, pc.y, e0, e1, w, lr, lk, Xin, acc);
    else if (ng == 3) run_piece_product<3>(M, row0, pc.y, e0, e1, w, lr, lk, Xin, acc);
    else if (ng == 2) run_piece_product<2>(M, row0, pc.y, e0, e1, w, lr, lk, Xin, acc);
    else run_piece_product<1>(M, row0, pc.y, e0, e1, w, lr, lk, Xin, acc);
    // wavefront w adds the four sums of row group w, one column half at a time
    double tot[2][4];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      __syncthreads();
#pragma unroll
      for (int g = 0; g < 4; ++g)
        if (g < ng)
#pragma unroll
          for (int r = 0; r < 4; ++r) buf[w][g][r][lane] = acc[g][q][r];
      __syncthreads();
      if (w < ng)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          tot[q][r] = ((buf[0][w][r][lane] + buf[1][w][r][lane]) + buf[2][w][r][lane]) + buf[3][w][r][lane];
    }
    if (w >= ng) continue;
    // register r: row 16 w + lk + 4 r, columns 2 lr and 2 lr + 1
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int rl = 16 * w + lk + 4 * r;
      if (rl >= pc.y) continue;
      const int64_t row = row0 + rl;
      if (M.nsplit > 1) {
        *(d2u*)(part + ((int64_t)z * M.rows + row) * kBlk + 2 * lr) = d2u{tot[0][r], tot[1][r]};
        continue;
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int c = 2 * lr + q;
        double o = sA[q] * tot[q][r];
        if (prev && cf[q] != 0.0) o -= cf[q] * prev[row * kBlk + c];
        if (act[q]) out[row * kBlk + c] = o;
        ss[q] += o * o;
      }
    }
  }
  if (sq && M.nsplit == 1) {
    red[4 * w + lk][2 * lr] = ss[0];
    red[4 * w + lk][2 * lr + 1] = ss[1];
    __syncthreads();
    if (threadIdx.x < kBlk) {
      double t = 0.0;
      for (int g = 0; g < kThreads / 16; ++g) t += red[g][threadIdx.x];
      sq[slot * kBlk + threadIdx.x] = t;
    }
  }
}

// pre[z][c] = sum of sq[b][c] over b = z, z + kPre, ... < nsq (workgroup z; fixed order)
__global__ void __launch_bounds__(kThreads) k_blk_presum(const double* __restrict__ sq, int nsq,
                                                         double* __restrict__ pre,
                                                         const BlockState* __restrict__ st) {
  if (st && all_done(st)) return;
  __shared__ double red[kThreads / kBlk][kBlk];
  const int c = threadIdx.x % kBlk, rsub = threadIdx.x / kBlk;
  double t = 0.0;
#pragma unroll 4
  for (int b = blockIdx.x + kPre * rsub; b < nsq; b += kPre * (kThreads / kBlk)) t += sq[b * kBlk + c];
  red[rsub][c] = t;
  __syncthreads();
  if (rsub == 0) {
    double s = 0.0;
    for (int q = 0; q < kThreads / kBlk; ++q) s += red[q][c];
    pre[blockIdx.x * kBlk + c] = s;
  }
}
// out[c] = sqrt of the folded sums
__global__ void k_blk_norm_out(const double* __restrict__ pre, double* __restrict__ out) {
  if (threadIdx.x < kBlk) out[threadIdx.x] = sqrt(blk_total(pre, threadIdx.x));
}

__global__ void k_blk_fill(double* p, int64_t len, double v) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < len;
       e += (int64_t)gridDim.x * blockDim.x)
    p[e] = v;
}

// per-column sums of squares of a len x 32 block, which is also copied to out when given
__global__ void __launch_bounds__(kThreads) k_blk_sumsq(const double* __restrict__ x, int64_t len,
                                                        double* __restrict__ out, double* __restrict__ sq) {
  __shared__ double red[kThreads / kBlk][kBlk];
  const int c = threadIdx.x % kBlk, rsub = threadIdx.x / kBlk;
  double t = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * (kThreads / kBlk) + rsub; i < len;
       i += (int64_t)gridDim.x * (kThreads / kBlk)) {
    const double v = x[i * kBlk + c];
    if (out) out[i * kBlk + c] = v;
    t += v * v;
  }
  red[rsub][c] = t;
  __syncthreads();
  if (rsub == 0) {
    double s = 0.0;
    for (int q = 0; q < kThreads / kBlk; ++q) s += red[q][c];
    sq[blockIdx.x * kBlk + c] = s;
  }
}

// beta_1 from the folded sums: set up the states.
__global__ void k_blk_begin(BlockState* st, BlockState* next, const double* __restrict__ pre, double atol, double btol,
                            double conlim, int64_t itmax) {
  const int c = threadIdx.x;
  if (c < kBlk) {
    const double beta = sqrt(blk_total(pre, c));
    LsqrDev d{};
    d.atol = atol;
    d.btol = btol;
    d.conlim = conlim;
    d.itmax = itmax;
    d.beta = d.bnorm = d.phibar = beta;
    d.istop = 7;
    if (!isfinite(beta)) {  // a non-finite right-hand side: breakdown, not "x = 0 is exact"
      d.istop = -3;
      d.done = 1;
    } else if (!(beta > 0.0)) {
      d.istop = 0;
      d.done = 1;
    }
    st->col[c] = d;
    next->col[c].fresh = 0;
  }
  if (c == 0) next->all_done = 0;
  __syncthreads();
  if (c == 0) all_done_update(st);
}

// alpha_1 from the folded sums.
__global__ void k_blk_begin2(BlockState* st, const double* __restrict__ pre) {
  const int c = threadIdx.x;
  if (c < kBlk) {
    LsqrDev& d = st->col[c];
    if (!d.done) {
      const double alpha = sqrt(blk_total(pre, c));
      d.alpha = d.alpha_prev = d.rhobar = alpha;
      d.normr = d.beta;
      d.normar = alpha * d.beta;
      d.w2 = 1.0;  // w_1 = v_1
      if (!isfinite(alpha)) {
        d.istop = -3;
        d.done = 1;
      } else if (!(alpha > 0.0)) {
        d.istop = 0;
        d.done = 1;
      }
    }
  }
  __syncthreads();
  if (c == 0) all_done_update(st);
}
__global__ void k_blk_w2(BlockState* st, const double* __restrict__ pre) {
  if (threadIdx.x < kBlk) st->col[threadIdx.x].w2 = blk_total(pre, threadIdx.x);
}

// y_1 = 0 and w_1 = v^/alpha, or of the backward's shadow vector vt_1 = u^/(beta alpha),
// also kept in vt; wsq (optional): partial sums of ||w_1||^2
__global__ void __launch_bounds__(kThreads)
    k_blk_first_w(const BlockState* __restrict__ st, const double* __restrict__ v, int over_beta, double* vt, double* w,
                  double* y, int64_t n, double* __restrict__ wsq) {
  __shared__ double red[kThreads / kBlk][kBlk];
  const int c = threadIdx.x % kBlk, rsub = threadIdx.x / kBlk;
  double f = inv_or_0(st->col[c].alpha);
  if (over_beta) f *= inv_or_0(st->col[c].beta);
  double sw = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * (kThreads / kBlk) + rsub; i < n;
       i += (int64_t)gridDim.x * (kThreads / kBlk)) {
    const int64_t e = i * kBlk + c;
    const double wi = f > 0.0 ? v[e] * f : 0.0;
    if (vt) vt[e] = wi;
    w[e] = wi;
    y[e] = 0.0;
    sw += wi * wi;
  }
  if (!wsq) return;
  red[rsub][c] = sw;
  __syncthreads();
  if (rsub == 0) {
    double tw = 0.0;
    for (int q = 0; q < kThreads / kBlk; ++q) tw += red[q][c];
    wsq[blockIdx.x * kBlk + c] = tw;
  }
}

// The rest of iteration k after alpha v^ (apre: its folded sums) and beta (in the
// state): plane rotation, y += phi/rho w, w = v - theta/rho w and the partial sums of
// ||y||^2 and ||w||^2, per active column (k_lsqr_step of the single-column loop;
// vt given: the backward's shadow vector takes v's part).  Every thread forms its
// column's scalars; the first workgroup leaves the new states in next.
__global__ void __launch_bounds__(kThreads)
    k_blk_step(const BlockState* __restrict__ st, BlockState* next, const double* __restrict__ apre,
               const double* __restrict__ v, double* vt, double* w, double* y, int64_t n, double* __restrict__ ysq,
               double* __restrict__ wsq) {
  if (all_done(st)) return;
  __shared__ double ry[kThreads / kBlk][kBlk], rw[kThreads / kBlk][kBlk];
  const int c = threadIdx.x % kBlk, rsub = threadIdx.x / kBlk;
  LsqrDev s = st->col[c];
  const double alpha = sqrt(blk_total(apre, c));
  const double beta = s.beta;
  bool act = !s.done;
  if (act) {
    s.alpha = alpha;
    s.itn += 1;
    s.anorm2 += s.alpha_prev * s.alpha_prev + beta * beta;
    const double rho = hypot(s.rhobar, beta);
    s.pending = 0;
    if (rho > 0.0 && isfinite(rho)) {
      const double cs = s.rhobar / rho;
      const double sn = beta / rho;
      const double theta = sn * alpha;
      s.rhobar = -cs * alpha;
      const double phi = cs * s.phibar;
      s.phibar = sn * s.phibar;
      s.phi_rho = phi / rho;
      s.theta_rho = theta / rho;
      s.ddnorm += s.w2 / (rho * rho);
      const double anorm = sqrt(s.anorm2);
      s.acond = anorm * sqrt(s.ddnorm);
      s.normr = s.phibar;
      s.normar = s.phibar * alpha * fabs(cs);
      if (s.normr == 0.0 || s.normar <= s.atol * anorm * s.normr) s.pending = 2;
      else if (s.conlim > 0.0 && s.acond >= s.conlim) s.pending = 3;
      s.alpha_prev = alpha;
    } else {
      s.istop = isfinite(rho) ? 1 : -3;
      s.done = 1;
      s.phi_rho = 0.0;
      s.theta_rho = 0.0;
      act = false;
    }
    s.fresh = 1;
    if (blockIdx.x == 0 && rsub == 0) next->col[c] = s;
  } else if (blockIdx.x == 0 && rsub == 0) {
    next->col[c].fresh = 0;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) next->all_done = 1;
  const double a = s.phi_rho, b = s.theta_rho;
  const double ia = inv_or_0(alpha), ib = inv_or_0(beta);
  double sy = 0.0, sw = 0.0;
  if (act)
    for (int64_t i = (int64_t)blockIdx.x * (kThreads / kBlk) + rsub; i < n;
         i += (int64_t)gridDim.x * (kThreads / kBlk)) {
      const int64_t e = i * kBlk + c;
      const double wi = w[e];
      const double yi = y[e] + a * wi;
      double vi = v[e];
      if (vt) {
        vi = (vi * ib - beta * vt[e]) * ia;
        vt[e] = vi;
      } else {
        vi *= ia;
      }
      const double wn = vi - b * wi;
      y[e] = yi;
      w[e] = wn;
      sy += yi * yi;
      sw += wn * wn;
    }
  ry[rsub][c] = sy;
  rw[rsub][c] = sw;
  __syncthreads();
  if (rsub == 0) {
    double ty = 0.0, tw = 0.0;
    for (int q = 0; q < kThreads / kBlk; ++q) {
      ty += ry[q][c];
      tw += rw[q][c];
    }
    ysq[blockIdx.x * kBlk + c] = ty;
    wsq[blockIdx.x * kBlk + c] = tw;
  }
}

// column-major (ld) <-> interleaved block conversions
__global__ void k_gather_block(const double* __restrict__ B, int64_t ldb, int64_t k0, int64_t nb,
                               int64_t len, double* __restrict__ out) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < len * kBlk;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = e / kBlk, c = e % kBlk;
    out[e] = c < nb ? B[(k0 + c) * ldb + i] : 0.0;
  }
}
__global__ void k_scatter_block(const double* __restrict__ in, int64_t len, int64_t k0, int64_t nb,
                                double* __restrict__ X, int64_t ldx) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < len * kBlk;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = e / kBlk, c = e % kBlk;
    if (c < nb) X[(k0 + c) * ldx + i] = in[e];
  }
}
__global__ void k_blk_axpy(double* x, const double* __restrict__ dx, int64_t len) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < len * kBlk;
       e += (int64_t)gridDim.x * blockDim.x)
    x[e] += dx[e];
}

// dA[e] (+)= sum_c (r[i][c] w[j][c] - lam[i][c] x[j][c]) on the pattern of A; one wavefront
// per row, lanes over the row's entries; the 32 columns of each block row are contiguous.
__global__ void __launch_bounds__(kThreads)
    k_blk_pattern_grad(const int64_t* __restrict__ rp, const int32_t* __restrict__ col, int64_t m,
                       const double* __restrict__ r, const double* __restrict__ w,
                       const double* __restrict__ lam, const double* __restrict__ x,
                       double* __restrict__ dA, int accumulate) {
  const int lane = threadIdx.x & 63;
  const int64_t wid = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  const int64_t nw = (int64_t)gridDim.x * (kThreads / 64);
  for (int64_t row = wid; row < m; row += nw) {
    const double* ri = r + row * kBlk;
    const double* li = lam + row * kBlk;
    for (int64_t e = rp[row] + lane; e < rp[row + 1]; e += 64) {
      const int64_t j = col[e];
      const double* wj = w + j * kBlk;
      const double* xj = x + j * kBlk;
      double g = 0.0;
#pragma unroll 8
      for (int c = 0; c < kBlk; ++c) g += ri[c] * wj[c] - li[c] * xj[c];
      dA[e] = accumulate ? dA[e] + g : g;
    }
  }
}

// The same over the pieces of an RFM matrix, on the matrix cores: the entries of a
// piece are nrows x (run length) blocks, each the product over K = 64 of [r, -lam] of
// its rows with [w, x] of its columns.  A workgroup takes a piece (a K chunk's span of
// its entries where M is chunked) and holds its rows' operands in LDS; the
// wavefronts take its 16-entry steps in turn.  K runs 8 columns to a lane group, so
// that a lane's operands are 64 contiguous bytes; a piece's rows have the same number
// of entries, hence row i's entries at i times that.
// Bound by the 8 B per entry written (and read, from the second block of columns on).
// 6.9 M entries, 7 columns: 518 us entry by entry (k_blk_pattern_grad, which takes
// matrices without pieces), 51 us here (the 7-column backward 5.4 -> 4.9 ms).
__global__ void __launch_bounds__(kThreads)
    k_run_pattern_grad(RunMat M, const double* __restrict__ r, const double* __restrict__ w,
                       const double* __restrict__ lam, const double* __restrict__ x, double* __restrict__ dA,
                       int accumulate) {
  constexpr int kC = kBlk / 4;  // columns per lane group
  __shared__ double As[kPieceRows][2 * kBlk + 1];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int64_t items = M.npieces * M.nsplit;
  for (int64_t wi = blockIdx.x; wi < items; wi += gridDim.x) {
    const int z = (int)(wi % M.nsplit);
    const int2 pc = M.pieces[wi / M.nsplit];
    const int64_t row0 = pc.x;
    const int ng = (pc.y + 15) >> 4;
    const int64_t e0 = (int64_t)z * M.kchunk, e1 = z == M.nsplit - 1 ? INT32_MAX : e0 + M.kchunk;
    const int nr = M.nrun[row0];
    if (nr < 1) continue;
    const int64_t len = M.rend[row0 * kMaxRuns + nr - 1];
    double* out = dA + M.rp[row0];
    __syncthreads();  // the item before has read As
    for (int e = threadIdx.x; e < 16 * ng * kBlk; e += kThreads) {
      const int rl = e / kBlk, c = e % kBlk;  // rows past the piece repeat its last (not stored)
      const int64_t o = (row0 + (rl < pc.y ? rl : pc.y - 1)) * kBlk + c;
      As[rl][c] = r[o];
      As[rl][kBlk + c] = -lam[o];
    }
    __syncthreads();
    int32_t off = 0;
    for (int k = 0; k < nr; ++k) {
      const int32_t end = M.rend[row0 * kMaxRuns + k];
      const int64_t s0 = off > e0 ? off : e0, s1 = end < e1 ? end : e1;
      const int64_t j0 = (int64_t)M.rcol[row0 * kMaxRuns + k] - off;  // column of entry e: j0 + e
      off = end;
      for (int64_t eb = s0 + 16 * wv; eb < s1; eb += 64) {
        const int64_t e = eb + lr < s1 ? eb + lr : s1 - 1;  // lanes past the run's end: not stored
        const int64_t o = (j0 + e) * kBlk + kC * lk;
        double b[2 * kC];
#pragma unroll
        for (int s = 0; s < kC; ++s) {
          b[s] = w[o + s];
          b[kC + s] = x[o + s];
        }
        for (int g = 0; g < ng; ++g) {
          v4d p = {0.0, 0.0, 0.0, 0.0}, q = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int s = 0; s < kC; ++s) {
            p = __builtin_amdgcn_mfma_f64_16x16x4f64(As[16 * g + lr][kC * lk + s], b[s], p, 0, 0, 0);
            q = __builtin_amdgcn_mfma_f64_16x16x4f64(As[16 * g + lr][kBlk + kC * lk + s], b[kC + s], q, 0, 0, 0);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int rl = 16 * g + lk + 4 * i;
            if (rl >= pc.y || eb + lr >= s1) continue;
            double* d = out + rl * len + eb + lr;
            const double v = p[i] + q[i];
            *d = accumulate ? *d + v : v;
          }
        }
      }
    }
  }
}

unsigned grid_for(int64_t elems) {
  const int64_t b = (elems + kThreads - 1) / kThreads;
  return (unsigned)(b < 4096 ? (b > 0 ? b : 1) : 4096);
}
unsigned rows_grid(int64_t rows) {  // blocks of 8 rows x 32 columns, grid-stride beyond kRowBlocks
  const int64_t b = (rows + (kThreads / kBlk) - 1) / (kThreads / kBlk);
  return (unsigned)(b < kRowBlocks ? (b > 0 ? b : 1) : kRowBlocks);
}
// k_blk_pattern_grad: four rows a wavefront, grid-stride beyond kSpmmBlocks
unsigned pattern_grid(int64_t rows) {
  const int64_t b = (rows + 15) / 16;
  return (unsigned)(b < kSpmmBlocks ? (b > 0 ? b : 1) : kSpmmBlocks);
}

// SpMM launch shapes: 64-row groups; the window width (columns of the input
// block staged in LDS at a time) is chosen per matrix by the autotuner below.
// It changes neither the order of any sum nor the rows each block handles (so
// not the norm partials either), so every candidate gives bitwise the same
// result.  Grids stop at kSpmmGrid blocks (grid-stride over the groups beyond):
// up to 2048 groups one block each.
constexpr unsigned kSpmmGrid = kSpmmMaxBlocks;
struct SpmmShape {
  const void* fn;
  int group, win;
  unsigned max_blocks;  // grid cap (grid-stride over the groups beyond it)
  int last_first = 0;   // k_spmm_runs: order in which the pieces are taken
};
// the hand-picked shape (used when tuning is off, and the tuner's reference) is
// the first; runs: the matrix takes k_spmm_runs, whose shapes differ in the
// order the pieces are taken
SpmmShape spmm_shape(bool runs) {
  if (runs) return {nullptr, kPieceRows, 0, kSpmmGrid, 1};
  return {(const void*)k_spmm<64>, kSpmmGroup, 64, kSpmmGrid};
}
static std::vector<SpmmShape> spmm_candidates(bool runs) {
  std::vector<SpmmShape> c;
  c.push_back(spmm_shape(runs));
  if (runs) {
    c.push_back({nullptr, kPieceRows, 0, kSpmmGrid, 0});
  } else {
    c.push_back({(const void*)k_spmm<32>, kSpmmGroup, 32, kSpmmGrid});
    c.push_back({(const void*)k_spmm<128>, kSpmmGroup, 128, kSpmmGrid});
  }
  return c;
}
// Split row groups of a matrix with fewer than 4 groups per compute unit and
// long rows (at least 4 windows of 64 per split) so that the grid covers the
// chip: nsplit = ceil(4 CUs / groups), at most 8.
int spmm_split(const rfmls_csr* M, int num_cus) {
  const int64_t ng = (M->m + kSpmmGroup - 1) / kSpmmGroup;
  const int64_t target = 4 * (int64_t)num_cus;
  if (ng <= 0 || ng >= target || M->nnz / M->m < 8 * 64) return 1;
  const int64_t sp = (target + ng - 1) / ng;
  const int64_t win = M->nnz / M->m / 64;  // windows of 64 columns of a row
  int64_t k = sp < 8 ? sp : 8;
  while (k > 1 && win / k < 4) --k;
  return (int)k;
}
// Window descriptors of one matrix for the window width W (built by
// spmm_build_desc, see k_spmm_walk).
struct SpmmDesc {
  int W = 0;  // 0: not built
  int nsplit = 1;
  int64_t items = 0, nwin = 0;
  int64_t* wptr = nullptr;    // items + 1 window offsets
  int32_t* wstart = nullptr;  // nwin window starts
  int64_t* wdesc = nullptr;   // nwin x 64 row descriptors
};
struct BCtx {
  rfmls_handle* h;
  const rfmls_csr* A;
  const rfmls_csr* AT;
  const rfmls_precond_t* P;
  hipStream_t st;
  double *U, *V, *W, *Y, *Z, *Q, *Rr, *Xb, *Bb, *DX;
  double *sqA, *sqB, *sqY, *sqW, *part;
  double *preA, *preB, *hn;  // folded sums (kPre x 32), and norms read by the host
  double* spart;  // partial sums of split SpMM groups (nsplit x rows x 32)
  SpmmDesc dA, dAT;  // SpMM window descriptors of A and A^T (k_spmm_walk)
  RunMat rA{}, rAT{};  // A and A^T as pieces of dense runs (npieces 0: the windowed kernel)
  BlockState* dst;  // the states, and after them the iteration's uncommitted ones
  IterGraph* graph = nullptr;  // captured poll interval of the loop, or null: eager launches
};

// Runs the lockstep loop: `iteration` (which enqueues one iteration on c.st) up
// to itmax times, the host polling the "all columns done" word after every
// `every` iterations; with c.graph the poll interval is captured once and replayed.
template <class F>
static rfmls_status run_loop(BCtx& c, int64_t itmax, int every, int consistent, F&& iteration);

BlkCommit commit_of(const BCtx& c, int consistent) {
  BlkCommit cm;
  cm.st = c.dst;
  cm.next = c.dst + 1;
  cm.ysq = c.sqY;
  cm.wsq = c.sqW;
  cm.n = (int)rows_grid(c.A->n);
  cm.consistent = consistent;
  return cm;
}
// Folds a producer's nsq rows of partial sums into pre.
rfmls_status presum(BCtx& c, const double* sq, int nsq, double* pre, const BlockState* stp) {
  hipLaunchKernelGGL(k_blk_presum, dim3(kPre), dim3(kThreads), 0, c.st, sq, nsq, pre, stp);
  RFMLS_HIP(c.h, hipGetLastError());
  return RFMLS_OK;
}

rfmls_status tri_block(BCtx& c, int trans, const double* in, double* out, const BlkScale& sc = BlkScale(),
                       const double* prev = nullptr, double* sq = nullptr, const BlockState* stp = nullptr,
                       const BlkCommit& cm = BlkCommit()) {
  const rfmls_precond_t* P = c.P;
  const int64_t n = P->n, nt = P->nt;
  const int C = P->chunk;
  const int maxk = (int)((nt + C - 1) / C);
  const double esz = P->store == RFMLS_F64 ? 8.0 : 4.0;
  const int full = P->full;
  const double tri = full ? (double)n * (double)n : (double)n * (double)(n + 1) / 2.0;
  {
    Trace tr(c.h, full ? (trans ? "gemm_Pt" : "gemm_P") : (trans ? "trmm_Xt" : "trmm_X"),
             esz * tri + 2.0 * 8.0 * kBlk * (double)n, 2.0 * tri * kBlk);
    if (!trans) {
      if (P->store == RFMLS_F64)
        hipLaunchKernelGGL(k_trmm_part<double>, dim3((unsigned)P->ntab + (cm.st ? 1u : 0u)), dim3(kThreads), 0, c.st,
                           (const double*)P->Xpk, nt, n, full, P->tab_row, C, maxk, in, c.part, stp, cm);
      else
        hipLaunchKernelGGL(k_trmm_part<float>, dim3((unsigned)P->ntab + (cm.st ? 1u : 0u)), dim3(kThreads), 0, c.st,
                           (const float*)P->Xpk, nt, n, full, P->tab_row, C, maxk, in, c.part, stp, cm);
    } else {
      if (P->store == RFMLS_F64)
        hipLaunchKernelGGL(k_trmmT_part<double>, dim3((unsigned)P->ntab + (cm.st ? 1u : 0u)), dim3(kThreads), 0, c.st,
                           (const double*)P->Xpk, nt, n, full, P->tab_col, C, maxk, in, c.part, stp, cm);
      else
        hipLaunchKernelGGL(k_trmmT_part<float>, dim3((unsigned)P->ntab + (cm.st ? 1u : 0u)), dim3(kThreads), 0, c.st,
                           (const float*)P->Xpk, nt, n, full, P->tab_col, C, maxk, in, c.part, stp, cm);
    }
  }
  hipLaunchKernelGGL(k_blk_tri_reduce, dim3(rows_grid(n)), dim3(kThreads), 0, c.st, (const double*)c.part,
                     nt, n, full, C, maxk, trans, sc, prev, out, sq, stp);
  RFMLS_HIP(c.h, hipGetLastError());
  return RFMLS_OK;
}

// The tuned launch shape of products with M on this handle, if a matrix of M's
// shape (rows, columns, stored entries) that the same kernel takes has been tuned: a
// rebuilt transpose (same matrix at a new address) is not tuned again, a matrix of
// another structure has candidates of its own.
static bool spmm_lookup(rfmls_handle* h, const rfmls_csr* M, bool runs, SpmmShape* out) {
  if (!h->tune) return false;
  for (const TuneRec& t : h->tuned)
    if (t.rows == M->m && t.cols == M->n && t.nnz == M->nnz && t.runs == runs && !strcmp(t.kernel, "spmm")) {
      const std::vector<SpmmShape> cands = spmm_candidates(runs);
      if (t.choice >= 0 && t.choice < (int)cands.size()) {
        *out = cands[t.choice];
        return true;
      }
    }
  return false;
}

// Window descriptors of M (A or A^T of the context) for width W: a count pass
// of the window walk, the scan of the counts, one host read of the total,
// and the fill pass.  Synchronises the stream; refused while a graph is
// being captured (the solve loops prepare them before capturing).
template <int W>
static void spmm_walk_launch(BCtx& c, const rfmls_csr* M, int nsplit, unsigned grid, int32_t* cnt, int64_t* wptr,
                             int32_t* wstart, int64_t* wdesc, bool fill) {
  if (fill)
    hipLaunchKernelGGL((k_spmm_walk<W, true>), dim3(grid), dim3(kThreads), 0, c.st, M->row_ptr, M->col, M->m, nsplit,
                       cnt, (const int64_t*)wptr, wstart, wdesc);
  else
    hipLaunchKernelGGL((k_spmm_walk<W, false>), dim3(grid), dim3(kThreads), 0, c.st, M->row_ptr, M->col, M->m, nsplit,
                       cnt, (const int64_t*)wptr, wstart, wdesc);
}
static rfmls_status spmm_build_desc(BCtx& c, const rfmls_csr* M, int W, SpmmDesc* d) {
  rfmls_handle* h = c.h;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(c.st, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone)
    return fail(h, RFMLS_E_HIP, "SpMM: window descriptors requested while capturing a graph");
  const bool isA = M == c.A;
  const int nsplit = spmm_split(M, h->num_cus);
  const int64_t items = ((M->m + kSpmmGroup - 1) / kSpmmGroup) * nsplit;
  const unsigned grid = (unsigned)(items < 4096 ? (items > 0 ? items : 1) : 4096);
  void* p1;
  RFMLS_CHECK(workspace(h, isA ? WS_SPMM_WPTR_A : WS_SPMM_WPTR_AT,
                        sizeof(int64_t) * (size_t)(items + 1) + sizeof(int32_t) * (size_t)(items + 1), &p1));
  int64_t* wptr = (int64_t*)p1;
  int32_t* cnt = (int32_t*)(wptr + items + 1);
  auto walk = [&](bool fill, int32_t* ws, int64_t* wd) {
    if (W == 32) spmm_walk_launch<32>(c, M, nsplit, grid, cnt, wptr, ws, wd, fill);
    else if (W == 128) spmm_walk_launch<128>(c, M, nsplit, grid, cnt, wptr, ws, wd, fill);
    else spmm_walk_launch<64>(c, M, nsplit, grid, cnt, wptr, ws, wd, fill);
  };
  walk(false, nullptr, nullptr);
  RFMLS_CHECK(scan_counts(h, cnt, items, wptr));
  int64_t nwin = 0;
  RFMLS_HIP(h, hipMemcpyAsync(&nwin, wptr + items, sizeof(int64_t), hipMemcpyDeviceToHost, c.st));
  RFMLS_HIP(h, hipStreamSynchronize(c.st));
  void* p2;
  RFMLS_CHECK(workspace(h, isA ? WS_SPMM_WDESC_A : WS_SPMM_WDESC_AT,
                        sizeof(int64_t) * (size_t)(nwin > 0 ? nwin : 1) * kSpmmGroup +
                            sizeof(int32_t) * (size_t)(nwin > 0 ? nwin : 1) + 64,
                        &p2));
  int64_t* wdesc = (int64_t*)p2;
  int32_t* wstart = (int32_t*)(wdesc + (nwin > 0 ? nwin : 1) * kSpmmGroup);
  walk(true, wstart, wdesc);
  RFMLS_HIP(h, hipGetLastError());
  d->W = W;
  d->nsplit = nsplit;
  d->items = items;
  d->nwin = nwin;
  d->wptr = wptr;
  d->wstart = wstart;
  d->wdesc = wdesc;
  if (c.AT == c.A) c.dAT = c.dA = *d;
  return RFMLS_OK;
}

static rfmls_status spmm_launch(BCtx& c, const rfmls_csr* M, const SpmmShape& sh, const double* x, const BlkScale& sc,
                                const double* prev, double* out, double* sq, const BlockState* stp, int* nblk);
static const RunMat& run_mat(const BCtx& c, const rfmls_csr* M) { return M == c.A ? c.rA : c.rAT; }

// Autotuner of the SpMM launch shape for M: the first time a
// matrix of M's shape and kernel is used on this handle (with tuning on), every candidate of
// spmm_candidates runs on M with a zero input block of 32 columns into
// scratch (xin: M->n x 32, out: M->m x 32, sq: the partials), once to warm up
// and then three times between HIP events; the candidate with the smallest
// median is kept for M on this handle.  Synchronises the stream; never called
// while a graph is being captured.
static rfmls_status spmm_tune(BCtx& c, const rfmls_csr* M, double* xin, double* out, double* sq) {
  rfmls_handle* h = c.h;
  const bool runs = run_mat(c, M).npieces > 0;
  SpmmShape dummy;
  if (!h->tune || M->m < 1 || spmm_lookup(h, M, runs, &dummy)) return RFMLS_OK;
  const std::vector<SpmmShape> cands = spmm_candidates(runs);
  hipLaunchKernelGGL(k_blk_fill, dim3(grid_for(M->n * kBlk)), dim3(kThreads), 0, c.st, xin, M->n * kBlk, 0.0);
  hipEvent_t ev[4];
  for (auto& e : ev) RFMLS_HIP(h, hipEventCreate(&e));
  std::vector<double> med(cands.size(), 0.0);
  rfmls_status st = RFMLS_OK;
  const bool trace = h->trace;
  h->trace = false;  // the trial launches are not part of any traced step
  for (size_t k = 0; k < cands.size() && st >= 0; ++k) {
    float t[3];
    st = spmm_launch(c, M, cands[k], xin, BlkScale(), nullptr, out, sq, nullptr, nullptr);
    for (int r = 0; r < 3 && st >= 0; ++r) {
      hipEventRecord(ev[0], c.st);
      st = spmm_launch(c, M, cands[k], xin, BlkScale(), nullptr, out, sq, nullptr, nullptr);
      hipEventRecord(ev[1], c.st);
      if (hipEventSynchronize(ev[1]) != hipSuccess || hipEventElapsedTime(&t[r], ev[0], ev[1]) != hipSuccess)
        st = fail(h, RFMLS_E_HIP, "SpMM autotuner: event timing failed");
    }
    if (st >= 0) {
      std::sort(t, t + 3);
      med[k] = t[1];
    }
  }
  h->trace = trace;
  for (auto& e : ev) hipEventDestroy(e);
  if (st < 0) return st;
  size_t best = 0;
  for (size_t k = 1; k < cands.size(); ++k)
    if (med[k] < med[best]) best = k;
  TuneRec rec{};
  snprintf(rec.kernel, sizeof(rec.kernel), "spmm");
  rec.runs = runs;
  rec.rows = M->m;
  rec.cols = M->n;
  rec.nnz = M->nnz;
  rec.choice = (int)best;
  if (runs)
    snprintf(rec.desc, sizeof(rec.desc), "runs, pieces of %d rows, %s first", cands[best].group,
             cands[best].last_first ? "last" : "first");
  else
    snprintf(rec.desc, sizeof(rec.desc), "group %d window %d grid %u", cands[best].group, cands[best].win,
             cands[best].max_blocks);
  rec.ms_best = med[best];
  rec.ms_default = med[0];
  rec.candidates = (int)cands.size();
  h->tuned.push_back(rec);
  return RFMLS_OK;
}

// Column runs and pieces of A and A^T (once per call, from the matrices as they
// are), and which of the two kernels each takes.  Synchronises the stream once;
// called before any capture of the loop.
//
// The run kernel takes a matrix whose rows all have a run description and whose
// pieces average at least kRunMinRows rows: a piece's products run on 16-row
// tiles, so shorter pieces leave most of the matrix cores' rows empty.  The
// windowed kernel (which needs no structure) takes the rest.  The line by pieces of h
// rows at random places, B = A X over 1,024 columns, windowed against runs (ms): 20,000
// rows of 200 entries, h = 2 / 4 / 6 / 12: 2.85, 2.84, 2.85, 2.70 against 3.11, 1.79,
// 1.41, 1.00; of 8 runs of 4: h = 4 / 6 2.89, 2.79 against 2.55, 1.97; 100,000 rows of
// 20: h = 4 / 6 / 8 4.69, 3.80, 2.93 against 4.77, 3.60, 2.79.
constexpr int64_t kRunMinRows = 6;
constexpr int64_t kRunMaxSplit = 32;
static rfmls_status spmm_prepare(BCtx& c) {
  rfmls_handle* h = c.h;
  const rfmls_csr* mats[2] = {c.A, c.AT};
  const int nm = c.A == c.AT ? 1 : 2;
  size_t bytes = 256;
  for (int i = 0; i < nm; ++i) {
    const int64_t rows = mats[i]->m, ng = (rows + kPieceRows - 1) / kPieceRows;
    bytes += sizeof(int2) * (size_t)rows + (sizeof(int64_t) + sizeof(int32_t)) * (size_t)(ng + 2) +
             sizeof(int32_t) * (size_t)rows * (1 + 2 * kMaxRuns) + 64;
  }
  void* pr;
  RFMLS_CHECK(workspace(h, WS_SPMM_RUNS, bytes, &pr));
  // flags of both matrices and the numbers of pieces, in one copy
  int* bad = (int*)pr;
  int64_t* total = (int64_t*)pr + 2;
  char* q = (char*)pr + 256;
  RunMat* out[2] = {&c.rA, &c.rAT};
  int64_t* pptr[2];
  auto carve = [&](size_t b) {
    char* r = q;
    q += (b + 7) / 8 * 8;
    return r;
  };
  for (int i = 0; i < nm; ++i) {
    const rfmls_csr* M = mats[i];
    const int64_t rows = M->m, ng = (rows + kPieceRows - 1) / kPieceRows;
    int2* pieces = (int2*)carve(sizeof(int2) * (size_t)rows);
    pptr[i] = (int64_t*)carve(sizeof(int64_t) * (size_t)(ng + 1));
    int32_t* pcount = (int32_t*)carve(sizeof(int32_t) * (size_t)(ng + 1));
    int32_t* nrun = (int32_t*)carve(sizeof(int32_t) * (size_t)rows * (1 + 2 * kMaxRuns));
    int32_t* rcol = nrun + rows;
    int32_t* rend = rcol + rows * kMaxRuns;
    *out[i] = RunMat{M->row_ptr, M->val, nrun, rcol, rend, pieces, 0, rows, 1, 0};
    if (rows > 0) {
      const int* skip = probe_pieces(c.st, M, bad + i);
      find_runs(c.st, M, nrun, rcol, rend, skip);
      const unsigned g = (unsigned)(ng < 4096 ? (ng + 3) / 4 : 1024);
      hipLaunchKernelGGL(k_run_pieces<false>, dim3(g), dim3(kThreads), 0, c.st, rows, M->n, (const int32_t*)nrun,
                         (const int32_t*)rcol, (const int32_t*)rend, pcount, (const int64_t*)nullptr,
                         (int2*)nullptr, bad + i, (int64_t*)nullptr);
      RFMLS_CHECK(scan_counts(h, pcount, ng, pptr[i], skip));
      hipLaunchKernelGGL(k_run_pieces<true>, dim3(g), dim3(kThreads), 0, c.st, rows, M->n, (const int32_t*)nrun,
                         (const int32_t*)rcol, (const int32_t*)rend, pcount, (const int64_t*)pptr[i], pieces,
                         bad + i, total + i);
    }
  }
  RFMLS_HIP(h, hipGetLastError());
  const int64_t* pin = (const int64_t*)((char*)h->pinned + 1024);
  RFMLS_HIP(h, hipMemcpyAsync((char*)h->pinned + 1024, pr, 4 * sizeof(int64_t), hipMemcpyDeviceToHost, c.st));
  RFMLS_HIP(h, hipStreamSynchronize(c.st));
  const int* badh = (const int*)pin;
  int64_t need = 0;
  for (int i = 0; i < nm; ++i) {
    const rfmls_csr* M = mats[i];
    RunMat& r = *out[i];
    const int64_t np = pin[2 + i];
    if (M->m < 1 || badh[i] || np * kRunMinRows > M->m) continue;
    r.npieces = np;
    // K chunks where the pieces alone give fewer than four workgroups per
    // compute unit: each at least 256 entries of an average row (four steps per
    // wavefront; with 64, a 6.9 M entry matrix's products with 240- and 3,600-entry
    // rows took 25.9 + 7.2 us for the merge each, with 256 23.2 us and one merge of
    // 5.0 for the two; 192 gives 26.6, 384 25.1), at most kRunMaxSplit; a chunk is a
    // whole number of steps and the last also takes what longer rows have beyond it
    const int64_t len = (M->nnz + M->m - 1) / M->m;
    int64_t sp = (4 * (int64_t)h->num_cus + np - 1) / np;
    if (sp > len / 256) sp = len / 256;
    if (sp > kRunMaxSplit) sp = kRunMaxSplit;
    if (sp < 1) sp = 1;
    r.nsplit = (int)sp;
    r.kchunk = ((len + sp - 1) / sp + kRunStep - 1) / kRunStep * kRunStep;
    const int64_t pn = sp > 1 ? sp * M->m : 0;
    need = pn > need ? pn : need;
  }
  if (nm == 1) c.rAT = c.rA;
  if (need > 0) {
    void* pp;
    RFMLS_CHECK(workspace(h, WS_SPMM_PART, sizeof(double) * (size_t)need * kBlk, &pp));
    c.spart = (double*)pp;
  }
  return RFMLS_OK;
}

// Tunes the products with A and A^T and builds the window descriptors of the
// shapes the loop will use (before any capture of the loop).
static rfmls_status spmm_tune_both(BCtx& c) {
  RFMLS_CHECK(spmm_prepare(c));
  RFMLS_CHECK(spmm_tune(c, c.A, c.Z, c.U, c.sqA));
  if (c.AT != c.A) RFMLS_CHECK(spmm_tune(c, c.AT, c.U, c.Q, c.sqA));
  for (const rfmls_csr* M : {c.A, c.AT}) {
    const bool runs = run_mat(c, M).npieces > 0;
    if (runs) continue;
    SpmmShape sh;
    if (!spmm_lookup(c.h, M, runs, &sh)) sh = spmm_shape(runs);
    SpmmDesc* d = M == c.A ? &c.dA : &c.dAT;
    if (d->W != sh.win) RFMLS_CHECK(spmm_build_desc(c, M, sh.win, d));
  }
  return RFMLS_OK;
}

rfmls_status spmm(BCtx& c, const rfmls_csr* M, const double* x, double* out, const BlkScale& sc = BlkScale(),
                  const double* prev = nullptr, double* sq = nullptr, const BlockState* stp = nullptr,
                  int* nblk = nullptr) {
  const bool runs = run_mat(c, M).npieces > 0;
  SpmmShape sh;
  if (!spmm_lookup(c.h, M, runs, &sh)) sh = spmm_shape(runs);
  return spmm_launch(c, M, sh, x, sc, prev, out, sq, stp, nblk);
}

static rfmls_status spmm_launch(BCtx& c, const rfmls_csr* M, const SpmmShape& sh, const double* x, const BlkScale& sc,
                                const double* prev, double* out, double* sq, const BlockState* stp, int* nblk) {
  const RunMat& rm = run_mat(c, M);
  const bool runs = rm.npieces > 0;
  const int64_t ng = runs ? rm.npieces : (M->m + sh.group - 1) / sh.group;
  const int nsplit = runs ? rm.nsplit : spmm_split(M, c.h->num_cus);
  const int64_t work = ng * nsplit;
  const unsigned nb = (unsigned)(work < (int64_t)sh.max_blocks ? (work > 0 ? work : 1) : sh.max_blocks);
  Trace tr(c.h, M == c.A ? "spmm_A" : "spmm_At",
           (runs ? 8.0 : 12.0) * (double)M->nnz + 8.0 * (double)(M->m + 1) +
               8.0 * kBlk * ((double)M->n + (double)M->m * (prev ? 2.0 : 1.0)),
           2.0 * kBlk * (double)M->nnz);
  BlkScale sc_v = sc;
  double* spart = c.spart;
  if (runs) {
    hipLaunchKernelGGL(k_spmm_runs, dim3(nb), dim3(kThreads), 0, c.st, rm, sh.last_first, x, sc, prev, out, sq, stp,
                       spart);
  } else {
  SpmmDesc* dsc = M == c.A ? &c.dA : &c.dAT;
  if (dsc->W != sh.win) RFMLS_CHECK(spmm_build_desc(c, M, sh.win, dsc));
  const int64_t* wptr = dsc->wptr;
  const int32_t* wstart = dsc->wstart;
  const int64_t* wdesc = dsc->wdesc;
  void* args[] = {(void*)&M->col, (void*)&M->val, (void*)&M->m, (void*)&M->n,
                  (void*)&x, (void*)&sc_v, (void*)&prev,
                  (void*)&out, (void*)&sq, (void*)&stp, (void*)&nsplit, (void*)&spart, (void*)&wptr,
                  (void*)&wstart, (void*)&wdesc};
  RFMLS_HIP(c.h, hipLaunchKernel(sh.fn, dim3(nb), dim3(kThreads), args, 0, c.st));
  }
  if (nsplit > 1) {
    const unsigned gm = rows_grid(M->m);
    hipLaunchKernelGGL(k_spmm_merge, dim3(gm), dim3(kThreads), 0, c.st, (const double*)spart, nsplit, M->m,
                       sc, prev, out, sq, stp);
    if (nblk) *nblk = (int)gm;
  } else if (nblk) {
    *nblk = (int)nb;
  }
  RFMLS_HIP(c.h, hipGetLastError());
  return RFMLS_OK;
}

rfmls_status poll_all(BCtx& c, int* done) {
  int* pin = (int*)((char*)c.h->pinned + 1024);
  RFMLS_HIP(c.h, hipMemcpyAsync(pin, &c.dst->all_done, sizeof(int), hipMemcpyDeviceToHost, c.st));
  RFMLS_HIP(c.h, hipStreamSynchronize(c.st));
  *done = *pin;
  return RFMLS_OK;
}

// One lockstep sweep for min ||A X y - rhs|| over the 32 columns of rhs (m x 32).
rfmls_status block_sweep(BCtx& c, const double* rhs, const rfmls_opts* o, int64_t itmax) {
  const int64_t m = c.A->m, n = c.A->n;
  BlockState* st = c.dst;
  const BlockState* cst = st;
  double *alpha = &st->col[0].alpha, *beta = &st->col[0].beta;
  const unsigned rn = rows_grid(n);
  // beta_1 u_1 = rhs
  hipLaunchKernelGGL(k_blk_sumsq, dim3(rows_grid(m)), dim3(kThreads), 0, c.st, rhs, m, c.U, c.sqA);
  RFMLS_CHECK(presum(c, c.sqA, (int)rows_grid(m), c.preA, nullptr));
  hipLaunchKernelGGL(k_blk_begin, dim3(1), dim3(64), 0, c.st, st, st + 1, (const double*)c.preA, o->atol, o->btol,
                     o->conlim, itmax);
  // alpha_1 v_1 = X^T (A^T u_1)
  BlkScale s1;
  s1.sdiv = beta;
  RFMLS_CHECK(spmm(c, c.AT, c.U, c.Q));
  RFMLS_CHECK(tri_block(c, 1, c.Q, c.V, s1, nullptr, c.sqB));
  RFMLS_CHECK(presum(c, c.sqB, (int)rn, c.preB, nullptr));
  hipLaunchKernelGGL(k_blk_begin2, dim3(1), dim3(64), 0, c.st, st, (const double*)c.preB);
  hipLaunchKernelGGL(k_blk_first_w, dim3(rn), dim3(kThreads), 0, c.st, cst, (const double*)c.V, 0, (double*)nullptr, c.W,
                     c.Y, n, (double*)nullptr);
  RFMLS_HIP(c.h, hipGetLastError());
  const int every = o->check_every > 0 ? o->check_every : 8;
  const BlkCommit cm = commit_of(c, 0);
  return run_loop(c, itmax, every, 0, [&]() -> rfmls_status {
    // beta' u' = A (X v) - alpha u, with v = v^/alpha and u = u^/beta
    BlkScale su;
    su.sdiv = alpha;
    su.c = 1.0;
    su.cnum = alpha;
    su.cden = beta;
    int nb = 0;
    RFMLS_CHECK(tri_block(c, 0, c.V, c.Z, BlkScale(), nullptr, nullptr, cst, cm));
    RFMLS_CHECK(spmm(c, c.A, c.Z, c.U, su, c.U, c.sqA, cst, &nb));
    RFMLS_CHECK(presum(c, c.sqA, nb, c.preA, cst));
    // alpha' v' = X^T (A^T u') - beta' v, with u' = u^'/beta', beta' from the sums
    BlkScale sv;
    sv.c = 1.0;
    sv.pre = c.preA;
    sv.norm = beta;
    sv.cden = alpha;
    RFMLS_CHECK(spmm(c, c.AT, c.U, c.Q, BlkScale(), nullptr, nullptr, cst));
    RFMLS_CHECK(tri_block(c, 1, c.Q, c.V, sv, c.V, c.sqB, cst));
    RFMLS_CHECK(presum(c, c.sqB, (int)rn, c.preB, cst));
    hipLaunchKernelGGL(k_blk_step, dim3(rn), dim3(kThreads), 0, c.st, cst, st + 1, (const double*)c.preB,
                       (const double*)c.V, (double*)nullptr, c.W, c.Y, n, c.sqY, c.sqW);
    RFMLS_HIP(c.h, hipGetLastError());
    return RFMLS_OK;
  });
}

template <class F>
static rfmls_status run_loop(BCtx& c, int64_t itmax, int every, int consistent, F&& iteration) {
  rfmls_handle* h = c.h;
  const BlkCommit cm = commit_of(c, consistent);
  auto interval = [&](int64_t count) -> rfmls_status {
    for (int64_t k = 0; k < count; ++k) RFMLS_CHECK(iteration());
    hipLaunchKernelGGL(k_blk_commit, dim3(1), dim3(kThreads), 0, c.st, cm);
    RFMLS_HIP(h, hipGetLastError());
    return RFMLS_OK;
  };
  int hd = 0;
  if (c.graph && !h->trace) {
    if (!c.graph->exec)
      RFMLS_CHECK(capture_graph(h, c.graph, [&]() -> rfmls_status {
        const hipStream_t s0 = c.st;
        c.st = h->stream;
        const rfmls_status r = interval(every);
        c.st = s0;
        return r;
      }));
    for (int64_t it = 0; it < itmax && !hd; it += every) {
      RFMLS_HIP(h, hipGraphLaunch(c.graph->exec, c.st));
      RFMLS_CHECK(poll_all(c, &hd));
    }
    return RFMLS_OK;
  }
  for (int64_t it = 0; it < itmax && !hd; it += every) {
    RFMLS_CHECK(interval(itmax - it < every ? itmax - it : every));
    RFMLS_CHECK(poll_all(c, &hd));
  }
  return RFMLS_OK;
}

rfmls_status read_block_state(BCtx& c, BlockState* out) {
  RFMLS_HIP(c.h, hipMemcpyAsync(out, c.dst, sizeof(BlockState), hipMemcpyDeviceToHost, c.st));
  RFMLS_HIP(c.h, hipStreamSynchronize(c.st));
  return RFMLS_OK;
}

// Work blocks (3 of m x 32, 7 of n x 32), partial sums and the triangular-product
// partials, carved from one workspace slot.
static rfmls_status make_bctx(rfmls_handle* h, const rfmls_csr* A, const rfmls_csr* AT,
                              const rfmls_precond_t* P, BCtx& c) {
  const int64_t m = A->m, n = A->n;
  c.h = h;
  c.A = A;
  c.AT = AT;
  c.P = P;
  c.st = h->stream;
  const int64_t maxk = (P->nt + P->chunk - 1) / P->chunk;
  const size_t nvec = (size_t)kBlk * (size_t)(3 * m + 7 * n) + (4 * (size_t)kSpmmMaxBlocks + 2 * kPre + 4) * kBlk +
                      (size_t)P->nt * maxk * kTile * kBlk;
  void* p;
  RFMLS_CHECK(workspace(h, WS_LSQR_BLK, sizeof(double) * nvec, &p));
  double* d = (double*)p;
  auto take = [&](int64_t len) {
    double* r = d;
    d += len;
    return r;
  };
  c.U = take(m * kBlk);
  c.Rr = take(m * kBlk);
  c.Bb = take(m * kBlk);
  c.V = take(n * kBlk);
  c.W = take(n * kBlk);
  c.Y = take(n * kBlk);
  c.Z = take(n * kBlk);
  c.Q = take(n * kBlk);
  c.Xb = take(n * kBlk);
  c.DX = take(n * kBlk);
  c.sqA = take(kSpmmMaxBlocks * kBlk);
  c.sqB = take(kSpmmMaxBlocks * kBlk);
  c.sqY = take(kSpmmMaxBlocks * kBlk);
  c.sqW = take(kSpmmMaxBlocks * kBlk);
  c.preA = take(kPre * kBlk);
  c.preB = take(kPre * kBlk);
  c.hn = take(4 * kBlk);
  c.part = take(P->nt * maxk * kTile * kBlk);
  {
    const int64_t need = (int64_t)spmm_split(A, h->num_cus) * A->m > (int64_t)spmm_split(AT, h->num_cus) * AT->m
                             ? (int64_t)spmm_split(A, h->num_cus) * A->m
                             : (int64_t)spmm_split(AT, h->num_cus) * AT->m;
    void* pp;
    RFMLS_CHECK(workspace(h, WS_SPMM_PART, sizeof(double) * (size_t)need * kBlk, &pp));
    c.spart = (double*)pp;
  }
  void* ps;
  RFMLS_CHECK(workspace(h, WS_LSQR_BSTATE, 2 * sizeof(BlockState), &ps));
  c.dst = (BlockState*)ps;
  return RFMLS_OK;
}

// Column norms of a len x 32 block into c.hn[32 k ..] (read by the host later).
static rfmls_status norms_to(BCtx& c, const double* x, int64_t len, int k) {
  hipLaunchKernelGGL(k_blk_sumsq, dim3(rows_grid(len)), dim3(kThreads), 0, c.st, x, len, (double*)nullptr, c.sqY);
  RFMLS_CHECK(presum(c, c.sqY, (int)rows_grid(len), c.preA, nullptr));
  hipLaunchKernelGGL(k_blk_norm_out, dim3(1), dim3(64), 0, c.st, (const double*)c.preA, c.hn + k * kBlk);
  RFMLS_HIP(c.h, hipGetLastError());
  return RFMLS_OK;
}

// ---- the explicit preconditioned matrix B = A X (Alg. 1 step 4) ----
// out[j][k] = X[j][c0 + k] for k < nb (zero beyond nb, and below the diagonal
// for the triangular X = R^{-1}): a 32-column slab of X in the lockstep block
// layout, read from the packed tiles.
template <typename TS>
__global__ void k_x_slab(const TS* __restrict__ Xpk, int64_t n, int64_t nt, int full, int64_t c0, int nb,
                         double* __restrict__ out) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n * kBlk;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = e / kBlk, c = c0 + e % kBlk;
    double v = 0.0;
    if (e % kBlk < nb && (full || j <= c))
      v = (double)Xpk[ptile(j / kTile, c / kTile, nt, full) * (int64_t)(kTile * kTile) +
                      (j % kTile) * kTile + c % kTile];
    out[e] = v;
  }
}
// B[i][c0 + k] = in[i][k] for k < nb (rows of B ldb apart)
__global__ void k_scatter_slab(const double* __restrict__ in, int64_t m, int64_t c0, int nb,
                               double* __restrict__ B, int64_t ldb) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m * kBlk;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = e / kBlk, k = e % kBlk;
    if (k < nb) B[i * ldb + c0 + k] = in[e];
  }
}

}  // namespace

rfmls_status run_solve_block(rfmls_handle* h, const rfmls_csr* A, const rfmls_csr* AT,
                             const rfmls_precond_t* P, const double* B, int64_t ldb, int64_t nrhs,
                             double* X, int64_t ldx, double* Rout, int64_t ldr, const rfmls_opts* o,
                             rfmls_info* info) {
  const int64_t m = A->m, n = A->n;
  const int64_t itmax = o->itmax > 0 ? o->itmax : n;
  BCtx c;
  RFMLS_CHECK(make_bctx(h, A, AT, P, c));
  RFMLS_CHECK(spmm_tune_both(c));
  IterGraph graph;  // one capture serves every sweep and column block (same buffers)
  if (o->graph) c.graph = &graph;
  const unsigned gm = grid_for(m * kBlk), gn = grid_for(n * kBlk);
  rfmls_status ret = RFMLS_OK;
  BlkScale residual;  // r = b - A x
  residual.s = -1.0;
  residual.c = -1.0;
  std::vector<BlockState> hs(1);
  for (int64_t k0 = 0; k0 < nrhs; k0 += kBlk) {
    const int64_t nb = nrhs - k0 < kBlk ? nrhs - k0 : kBlk;
    std::vector<rfmls_info> inf(nb);
    hipLaunchKernelGGL(k_gather_block, dim3(gm), dim3(kThreads), 0, c.st, B, ldb, k0, nb, m, c.Bb);
    // from x = 0 the first sweep takes B itself; from given starting points
    // every sweep solves for the correction from the true residual B - A X
    const bool warm = o->x_init != 0;
    if (warm) {
      hipLaunchKernelGGL(k_gather_block, dim3(gn), dim3(kThreads), 0, c.st, (const double*)X, ldx, k0, nb,
                         n, c.Xb);
      RFMLS_CHECK(spmm(c, A, c.Xb, c.Rr, residual, c.Bb));
      RFMLS_CHECK(norms_to(c, c.Bb, m, 2));
    }
    for (int sweep = 0; sweep <= o->refine; ++sweep) {
      const bool from_zero = sweep == 0 && !warm;
      RFMLS_CHECK(block_sweep(c, from_zero ? c.Bb : c.Rr, o, itmax));
      RFMLS_CHECK(read_block_state(c, hs.data()));
      int64_t itn_max = 0;
      for (int64_t q = 0; q < nb; ++q) {
        const LsqrDev& s = hs[0].col[q];
        if (s.istop < 0) return fail(h, RFMLS_E_BREAKDOWN, "non-finite value in LSQR (column %lld)", (long long)(k0 + q));
        if (sweep == 0) {
          inf[q].itn_first = s.itn;
          inf[q].istop = s.istop;
          inf[q].normr_est = s.normr;
          inf[q].normar_est = s.normar;
          inf[q].anorm_est = sqrt(s.anorm2);
          inf[q].acond_est = s.acond;
          if (!warm) inf[q].normb = s.bnorm;
          if (s.istop == 7) ret = RFMLS_W_NOCONV;
        }
        inf[q].itn += s.itn;
        inf[q].istop_last = s.istop;
        if (s.itn > itn_max) itn_max = s.itn;
      }
      // x (+)= X y ; r = b - A x
      RFMLS_CHECK(tri_block(c, 0, c.Y, from_zero ? c.Xb : c.DX));
      if (!from_zero)
        hipLaunchKernelGGL(k_blk_axpy, dim3(gn), dim3(kThreads), 0, c.st, c.Xb, (const double*)c.DX, n);
      RFMLS_CHECK(spmm(c, A, c.Xb, c.Rr, residual, c.Bb));
      if (itn_max == 0) break;
    }
    // true residual norms per column
    RFMLS_CHECK(norms_to(c, c.Rr, m, 0));
    RFMLS_CHECK(spmm(c, AT, c.Rr, c.Q));
    RFMLS_CHECK(norms_to(c, c.Q, n, 1));
    double* pin = (double*)((char*)h->pinned + 1024);
    RFMLS_HIP(h, hipMemcpyAsync(pin, c.hn, 3 * kBlk * sizeof(double), hipMemcpyDeviceToHost, c.st));
    hipLaunchKernelGGL(k_scatter_block, dim3(gn), dim3(kThreads), 0, c.st, (const double*)c.Xb, n, k0, nb, X, ldx);
    if (Rout)
      hipLaunchKernelGGL(k_scatter_block, dim3(gm), dim3(kThreads), 0, c.st, (const double*)c.Rr, m, k0, nb, Rout, ldr);
    RFMLS_HIP(h, hipGetLastError());
    RFMLS_HIP(h, hipStreamSynchronize(c.st));
    for (int64_t q = 0; q < nb; ++q) {
      inf[q].normr = pin[q];
      inf[q].normar = pin[kBlk + q];
      if (warm) inf[q].normb = pin[2 * kBlk + q];
      if (info) info[k0 + q] = inf[q];
    }
  }
  return ret;
}


// Backward in lockstep blocks of 32: for each column, LSQR on the consistent
// system B^T lam = X^T g with operator M = B^T = X^T A^T (n x m), from lam = 0,
// tracking the shadow vectors vt (v = B vt) and z (lam = B z); then w = X z,
// lam = A w, dB = lam and dA += r w^T - lam x^T on A's pattern (summed over
// the right-hand sides).  Same per-column recurrences as the single-column
// backward.
rfmls_status run_backward_block(rfmls_handle* h, const rfmls_csr* A, const rfmls_csr* AT,
                                const rfmls_precond_t* P, const double* Xs, int64_t ldx,
                                const double* Rres, int64_t ldr, const double* G, int64_t ldg,
                                int64_t nrhs, double* dB, int64_t lddb, double* dAval,
                                const rfmls_opts* o, rfmls_info* info) {
  const int64_t m = A->m, n = A->n;
  const int64_t itmax = o->itmax > 0 ? o->itmax : m;
  BCtx c;
  RFMLS_CHECK(make_bctx(h, A, AT, P, c));
  RFMLS_CHECK(spmm_tune_both(c));
  IterGraph graph;
  if (o->graph) c.graph = &graph;
  // roles: un (n), vm (m), vt, wt, zz shadows (n), tmp (n), lam (m), gathered blocks
  double* un = c.V;
  double* vm = c.U;
  double* vt = c.W;
  double* wt = c.Q;
  double* zz = c.Y;
  double* tmp = c.Z;
  double* lam = c.Rr;
  double* Gb = c.Xb;
  double* Xg = c.DX;
  double* Rg = c.Bb;
  const unsigned gm = grid_for(m * kBlk), gn = grid_for(n * kBlk);
  const int every = o->check_every > 0 ? o->check_every : 8;
  const BlockState* cst = c.dst;
  double *alpha = &c.dst->col[0].alpha, *beta = &c.dst->col[0].beta;
  const unsigned rn = rows_grid(n);
  const BlkCommit cm = commit_of(c, 1);
  rfmls_status ret = RFMLS_OK;
  std::vector<BlockState> hs(1);
  for (int64_t k0 = 0; k0 < nrhs; k0 += kBlk) {
    const int64_t nb = nrhs - k0 < kBlk ? nrhs - k0 : kBlk;
    hipLaunchKernelGGL(k_gather_block, dim3(gn), dim3(kThreads), 0, c.st, G, ldg, k0, nb, n, Gb);
    // beta_1 u_1 = X^T g
    RFMLS_CHECK(tri_block(c, 1, Gb, un, BlkScale(), nullptr, c.sqB));
    RFMLS_CHECK(presum(c, c.sqB, (int)rn, c.preB, nullptr));
    hipLaunchKernelGGL(k_blk_begin, dim3(1), dim3(64), 0, c.st, c.dst, c.dst + 1, (const double*)c.preB, o->atol,
                       o->btol, o->conlim, itmax);
    // alpha_1 v_1 = A (X u_1);  vt_1 = u_1 / alpha_1;  w_1 = vt_1
    BlkScale s1;
    s1.sdiv = beta;
    int nbk = 0;
    RFMLS_CHECK(tri_block(c, 0, un, tmp));
    RFMLS_CHECK(spmm(c, A, tmp, vm, s1, nullptr, c.sqA, nullptr, &nbk));
    RFMLS_CHECK(presum(c, c.sqA, nbk, c.preA, nullptr));
    hipLaunchKernelGGL(k_blk_begin2, dim3(1), dim3(64), 0, c.st, c.dst, (const double*)c.preA);
    hipLaunchKernelGGL(k_blk_first_w, dim3(rn), dim3(kThreads), 0, c.st, cst, (const double*)un, 1, vt, wt, zz, n,
                       c.sqW);
    RFMLS_CHECK(presum(c, c.sqW, (int)rn, c.preB, nullptr));
    hipLaunchKernelGGL(k_blk_w2, dim3(1), dim3(64), 0, c.st, c.dst, (const double*)c.preB);
    RFMLS_HIP(h, hipGetLastError());
    RFMLS_CHECK(run_loop(c, itmax, every, 1, [&]() -> rfmls_status {
      // beta' u' = X^T (A^T v) - alpha u, with v = v^/alpha and u = u^/beta
      BlkScale su;
      su.sdiv = alpha;
      su.c = 1.0;
      su.cnum = alpha;
      su.cden = beta;
      RFMLS_CHECK(spmm(c, AT, vm, tmp, BlkScale(), nullptr, nullptr, cst));
      RFMLS_CHECK(tri_block(c, 1, tmp, un, su, un, c.sqB, cst, cm));
      RFMLS_CHECK(presum(c, c.sqB, (int)rn, c.preB, cst));
      // alpha' v' = A (X u') - beta' v, with u' = u^'/beta', beta' from the sums;
      // vt' = (u' - beta' vt) / alpha' in k_blk_step
      BlkScale sv;
      sv.c = 1.0;
      sv.pre = c.preB;
      sv.norm = beta;
      sv.cden = alpha;
      RFMLS_CHECK(tri_block(c, 0, un, tmp, BlkScale(), nullptr, nullptr, cst));
      RFMLS_CHECK(spmm(c, A, tmp, vm, sv, vm, c.sqA, cst, &nbk));
      RFMLS_CHECK(presum(c, c.sqA, nbk, c.preA, cst));
      hipLaunchKernelGGL(k_blk_step, dim3(rn), dim3(kThreads), 0, c.st, cst, c.dst + 1, (const double*)c.preA,
                         (const double*)un, vt, wt, zz, n, c.sqY, c.sqW);
      RFMLS_HIP(h, hipGetLastError());
      return RFMLS_OK;
    }));
    RFMLS_CHECK(read_block_state(c, hs.data()));
    for (int64_t q = 0; q < nb; ++q) {
      const LsqrDev& st = hs[0].col[q];
      if (st.istop < 0)
        return fail(h, RFMLS_E_BREAKDOWN, "non-finite value in backward LSQR (column %lld)", (long long)(k0 + q));
      if (st.istop == 7) ret = RFMLS_W_NOCONV;
      if (info) {
        rfmls_info inf{};
        inf.itn = inf.itn_first = st.itn;
        inf.istop = inf.istop_last = st.istop;
        inf.normr_est = st.normr;
        inf.normb = st.bnorm;
        info[k0 + q] = inf;
      }
    }
    // w = X z, lam = A w
    RFMLS_CHECK(tri_block(c, 0, zz, tmp));
    RFMLS_CHECK(spmm(c, A, tmp, lam));
    if (dB)
      hipLaunchKernelGGL(k_scatter_block, dim3(gm), dim3(kThreads), 0, c.st, (const double*)lam, m, k0, nb, dB, lddb);
    if (dAval) {
      hipLaunchKernelGGL(k_gather_block, dim3(gm), dim3(kThreads), 0, c.st, Rres, ldr, k0, nb, m, Rg);
      hipLaunchKernelGGL(k_gather_block, dim3(gn), dim3(kThreads), 0, c.st, Xs, ldx, k0, nb, n, Xg);
      const RunMat& rm = c.rA;
      Trace tr(h, "pattern_grad_blk",
               (rm.npieces > 0 ? 8.0 : 16.0) * (double)A->nnz + 8.0 * (double)(m + 1) + 16.0 * kBlk * (double)(m + n),
               4.0 * kBlk * (double)A->nnz);
      const int64_t items = rm.npieces * rm.nsplit;
      if (items > 0)
        hipLaunchKernelGGL(k_run_pattern_grad, dim3((unsigned)(items < 65536 ? items : 65536)), dim3(kThreads), 0, c.st,
                           rm, (const double*)Rg, (const double*)tmp, (const double*)lam, (const double*)Xg, dAval,
                           k0 > 0 ? 1 : 0);
      else
        hipLaunchKernelGGL(k_blk_pattern_grad, dim3(pattern_grid(m)), dim3(kThreads), 0, c.st, A->row_ptr, A->col, m,
                           (const double*)Rg, (const double*)tmp, (const double*)lam, (const double*)Xg, dAval,
                           k0 > 0 ? 1 : 0);
    }
    RFMLS_HIP(h, hipGetLastError());
  }
  RFMLS_HIP(h, hipStreamSynchronize(c.st));
  return ret;
}

// B = A X in slabs of 32 columns: X's slab in the block layout, one lockstep
// SpMM with A (the kernel the multi-right-hand-side solve uses), the m x 32
// result scattered into B's rows.
rfmls_status run_form_B(rfmls_handle* h, const rfmls_csr* A, const rfmls_precond_t* P, double* Bmat,
                        int64_t ldb) {
  const int64_t m = A->m, n = A->n;
  BCtx c;
  RFMLS_CHECK(make_bctx(h, A, A, P, c));
  RFMLS_CHECK(spmm_tune_both(c));
  const unsigned gn = grid_for(n * kBlk), gm = grid_for(m * kBlk);
  for (int64_t c0 = 0; c0 < n; c0 += kBlk) {
    const int nb = (int)(n - c0 < kBlk ? n - c0 : kBlk);
    if (P->store == RFMLS_F64)
      hipLaunchKernelGGL(k_x_slab<double>, dim3(gn), dim3(kThreads), 0, c.st, (const double*)P->Xpk, n,
                         P->nt, P->full, c0, nb, c.Xb);
    else
      hipLaunchKernelGGL(k_x_slab<float>, dim3(gn), dim3(kThreads), 0, c.st, (const float*)P->Xpk, n,
                         P->nt, P->full, c0, nb, c.Xb);
    RFMLS_CHECK(spmm(c, A, c.Xb, c.U));
    hipLaunchKernelGGL(k_scatter_slab, dim3(gm), dim3(kThreads), 0, c.st, (const double*)c.U, m, c0, nb,
                       Bmat, ldb);
    RFMLS_HIP(h, hipGetLastError());
  }
  return RFMLS_OK;
}

}  // namespace rfmls
