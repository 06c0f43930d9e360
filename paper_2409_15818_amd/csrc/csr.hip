// Deterministic transpose of a CSR matrix (A^T as CSR, used for the products
// A^T u of Alg. 1 step 5).  A stable counting sort by column: rows are cut
// into chunks; per chunk and column the entries are counted, the counts are
// scanned over chunks (giving every (chunk, column) pair its first slot), and
// each chunk then walks its rows in order, so every row of A^T lists its
// entries in ascending row-of-A order.  No floating-point arithmetic.
//
// A matrix whose rows come in pieces with the same column runs (runs.h: the rows
// of one RFM box, face or interface) is sorted piece by piece instead: a piece of
// r rows puts r consecutive entries into each of its columns, so the counting and
// the walk handle one entry per piece and column, and the values are moved as
// dense 64 x 64 tiles through LDS, read and written in whole segments (the
// entry-by-entry walk writes 12 bytes at a time into as many different rows of A^T
// as the row has entries).  Both give the same A^T.  Which of the two runs is
// decided on the device (mode), so the call neither waits nor leaves a capture;
// the kernels of the other return at once.
// Measured on the 105,840 x 9,450 system of 44.5 M entries: 2.72 ms entry by entry
// (count 0.21, scan 0.24, walk 2.26), 0.44 ms piece by piece (runs 0.07, counts and
// places 0.06, tiles 0.25 at 3.6 TB/s); Helmholtz solve 29.2 -> 27.3 ms.
#include "common.h"
#include "runs.h"

namespace rfmls {
namespace {

constexpr int kColPass = 16384;  // columns handled per LDS pass

__global__ void __launch_bounds__(256)
    k_tr_hist(const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col, int64_t m,
              int64_t n, int64_t rc, int32_t* __restrict__ hist, const int* __restrict__ mode) {
  if (mode && *mode) return;
  __shared__ int32_t cnt[kColPass];
  const int64_t k = blockIdx.x;
  const int64_t rlo = k * rc, rhi = rlo + rc < m ? rlo + rc : m;
  const int64_t elo = row_ptr[rlo], ehi = row_ptr[rhi];
  for (int64_t c0 = 0; c0 < n; c0 += kColPass) {
    const int64_t cw = n - c0 < kColPass ? n - c0 : kColPass;
    for (int t = threadIdx.x; t < cw; t += 256) cnt[t] = 0;
    __syncthreads();
    for (int64_t e = elo + threadIdx.x; e < ehi; e += 256) {
      const int64_t c = (int64_t)col[e] - c0;
      if (c >= 0 && c < cw) atomicAdd(&cnt[c], 1);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < cw; t += 256) hist[k * n + c0 + t] = cnt[t];
    __syncthreads();
  }
}

// hist[k][c] <- exclusive prefix over k; count[c] <- total.  Runs when *mode == when
// (mode null: always).  Eight chunks' loads in flight per thread.
__global__ void k_tr_colscan(int32_t* __restrict__ hist, int64_t nchunk, int64_t n,
                             int32_t* __restrict__ count, const int* __restrict__ mode, int when) {
  if (mode && (*mode != 0) != (when != 0)) return;
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  int32_t run = 0;
  for (int64_t k0 = 0; k0 < nchunk; k0 += 8) {
    int32_t v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = k0 + q < nchunk ? hist[(k0 + q) * n + c] : 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (k0 + q < nchunk) hist[(k0 + q) * n + c] = run;
      run += v[q];
    }
  }
  count[c] = run;
}

__global__ void __launch_bounds__(256)
    k_tr_fill(const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
              const double* __restrict__ val, int64_t m, int64_t n, int64_t rc,
              const int32_t* __restrict__ hist, const int64_t* __restrict__ at_ptr,
              int32_t* __restrict__ at_col, double* __restrict__ at_val, const int* __restrict__ mode) {
  if (mode && *mode) return;
  __shared__ int32_t cur[kColPass];
  const int64_t k = blockIdx.x;
  const int64_t rlo = k * rc, rhi = rlo + rc < m ? rlo + rc : m;
  for (int64_t c0 = 0; c0 < n; c0 += kColPass) {
    const int64_t cw = n - c0 < kColPass ? n - c0 : kColPass;
    for (int t = threadIdx.x; t < cw; t += 256) cur[t] = hist[k * n + c0 + t];
    __syncthreads();
    for (int64_t i = rlo; i < rhi; ++i) {
      const int64_t lo = row_ptr[i], hi = row_ptr[i + 1];
      for (int64_t e = lo + threadIdx.x; e < hi; e += 256) {
        const int64_t c = (int64_t)col[e] - c0;
        if (c >= 0 && c < cw) {
          const int64_t pos = at_ptr[c0 + c] + cur[c];
          cur[c] += 1;  // columns are unique within a row: no two threads share c
          at_col[pos] = (int32_t)i;
          at_val[pos] = val[e];
        }
      }
      __syncthreads();
    }
  }
}

// ---- piece by piece ----
// Per 64-row group: the rows that start a piece, and the entries of one row of each
// of its pieces (elen, summed over the group's pieces).  bad: see group_pieces.
__global__ void __launch_bounds__(256)
    k_tr_groups(int64_t m, int64_t n, const int32_t* __restrict__ nrun, const int32_t* __restrict__ rcol,
                const int32_t* __restrict__ rend, unsigned long long* __restrict__ gstart, int32_t* __restrict__ elen,
                int* __restrict__ bad) {
  if (*bad) return;  // (what it leaves unwritten is not read then)
  const int lane = threadIdx.x & 63;
  const int64_t ng = (m + kPieceRows - 1) / kPieceRows;
  const int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (g >= ng) return;  // uniform per wavefront
  unsigned long long starts, lives, wrong;
  group_pieces(g, m, n, nrun, rcol, rend, &starts, &lives, &wrong);
  const int64_t row = g * kPieceRows + lane;
  int len = 0;
  if (starts >> lane & 1) {
    const int k = nrun[row];
    len = k > 0 ? rend[row * kMaxRuns + k - 1] : 0;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) len += __shfl_xor(len, o, 64);
  if (lane == 0) {
    gstart[g] = starts;
    elen[g] = len;
    if (wrong) atomicOr(bad, 1);
  }
}
__global__ void k_clear_flag(int* bad) { *bad = 0; }
// bad = 1 where a sample says that the rows have no pieces to speak of, else 0.  The
// sample is up to 16 groups spread over the matrix, one a wavefront; a row of another
// length or first column than the row before starts a piece.  More than a fifth of the
// sampled rows doing so is beyond what either use of the pieces takes (one in eight
// entries here, one in six rows in the lockstep products): the kernels that find the
// runs and pieces then return at once.  Without it a 2,000,000 x 20,000 matrix of 12
// scattered entries a row spent 0.55 of 6.95 ms on runs that the entry-by-entry transpose
// then did not use.  One workgroup, bound by its scattered loads: 64 groups and the last
// columns too took 16 us.
constexpr int kProbeGroups = 16;
__global__ void __launch_bounds__(64 * kProbeGroups)
    k_probe_pieces(const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col, int64_t m, int* bad) {
  __shared__ int found[kProbeGroups][2];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t ng = (m + kPieceRows - 1) / kPieceRows;
  const int64_t row = w * (ng > kProbeGroups ? ng / kProbeGroups : 1) * kPieceRows + lane;
  const bool live = row < m;
  const int64_t lo = row_ptr[live ? row : m], hi = row_ptr[live ? row + 1 : m];
  const int len = (int)(hi - lo), first = len > 0 ? col[lo] : -1;
  // (every lane takes part in both shuffles)
  const int len1 = __shfl_up(len, 1, 64), first1 = __shfl_up(first, 1, 64);
  const int starts = __popcll(__ballot(live && (lane == 0 || len1 != len || first1 != first)));
  const int rows = __popcll(__ballot(live));
  if (lane == 0) {
    found[w][0] = starts;
    found[w][1] = rows;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int s = 0, r = 0;
    for (int q = 0; q < kProbeGroups; ++q) {
      s += found[q][0];
      r += found[q][1];
    }
    *bad = 5 * s > r;
  }
}
// mode = 1: every row described, and the pieces' entry lists fit their buffer
__global__ void k_tr_mode(const int* __restrict__ bad, const int64_t* __restrict__ eptr, int64_t ng, int64_t cap,
                          int* __restrict__ mode) {
  *mode = !*bad && eptr[ng] <= cap;
}

// Calls f(row0, rows, entries, first entry slot) for the pieces of group g in order
// (uniform over the workgroup).
template <class F>
__device__ __forceinline__ void each_piece(int64_t g, int64_t m, const unsigned long long* __restrict__ gstart,
                                           const int64_t* __restrict__ eptr, const int32_t* __restrict__ nrun,
                                           const int32_t* __restrict__ rend, F&& f) {
  const unsigned long long starts = gstart[g];
  const int64_t left = m - g * kPieceRows;
  const unsigned long long lives = left >= kPieceRows ? ~0ull : (1ull << left) - 1ull;
  int64_t slot = eptr[g];
  for (unsigned long long s = starts; s; s &= s - 1) {
    const int r = __builtin_ctzll(s);
    const int64_t row = g * kPieceRows + r;
    const int k = nrun[row];
    const int len = k > 0 ? rend[row * kMaxRuns + k - 1] : 0;
    f(row, piece_len(starts, lives, r), len, slot);
    slot += len;
  }
}
// Column of entry e of a row with the given runs.
__device__ __forceinline__ int entry_col(int64_t row, int e, int k, const int32_t* __restrict__ rcol,
                                         const int32_t* __restrict__ rend) {
  int off = 0, c = 0;
  for (int q = 0; q < k; ++q) {
    const int end = rend[row * kMaxRuns + q];
    if (e >= off && e < end) c = rcol[row * kMaxRuns + q] + (e - off);
    off = end;
  }
  return c;
}

// hist[chunk][c] = entries of column c in the chunk's groups (count pass), then with
// hist the exclusive prefix over chunks: pos[slot + e] = first place in A^T of entry
// e of each piece (walk pass, pieces in order).
template <bool Walk>
__global__ void __launch_bounds__(256)
    k_tr_piece_walk(int64_t m, int64_t n, int64_t gc, const unsigned long long* __restrict__ gstart,
                    const int64_t* __restrict__ eptr, const int32_t* __restrict__ nrun,
                    const int32_t* __restrict__ rcol, const int32_t* __restrict__ rend, int32_t* __restrict__ hist,
                    const int64_t* __restrict__ at_ptr, int32_t* __restrict__ pos, const int* __restrict__ mode) {
  if (!*mode) return;
  __shared__ int32_t cnt[kColPass];
  const int64_t k = blockIdx.x, ng = (m + kPieceRows - 1) / kPieceRows;
  const int64_t glo = k * gc, ghi = glo + gc < ng ? glo + gc : ng;
  for (int64_t c0 = 0; c0 < n; c0 += kColPass) {
    const int cw = (int)(n - c0 < kColPass ? n - c0 : kColPass);
    for (int t = threadIdx.x; t < cw; t += 256) cnt[t] = Walk ? hist[k * n + c0 + t] : 0;
    __syncthreads();
    for (int64_t g = glo; g < ghi; ++g)
      each_piece(g, m, gstart, eptr, nrun, rend, [&](int64_t row, int nr, int len, int64_t slot) {
        const int kr = nrun[row];
        for (int e = threadIdx.x; e < len; e += 256) {
          const int64_t c = entry_col(row, e, kr, rcol, rend);
          if (c >= c0 && c < c0 + cw) {  // a piece's columns are distinct: no two threads share one
            if (Walk) pos[slot + e] = (int32_t)(at_ptr[c] + cnt[c - c0]);
            cnt[c - c0] += nr;
          }
        }
        __syncthreads();
      });
    if (!Walk) {
      for (int t = threadIdx.x; t < cw; t += 256) hist[k * n + c0 + t] = cnt[t];
      __syncthreads();
    }
  }
}

// The values and row numbers of every piece into A^T, 64 entries of the piece's rows
// at a time through LDS.  Bound by HBM: A's values read and A^T's values and columns
// written once, in segments of a piece's height.
__global__ void __launch_bounds__(256)
    k_tr_piece_fill(const int64_t* __restrict__ row_ptr, const double* __restrict__ val, int64_t m,
                    const unsigned long long* __restrict__ gstart, const int64_t* __restrict__ eptr,
                    const int32_t* __restrict__ nrun, const int32_t* __restrict__ rend,
                    const int32_t* __restrict__ pos, int32_t* __restrict__ at_col, double* __restrict__ at_val,
                    const int* __restrict__ mode) {
  if (!*mode) return;
  __shared__ double tile[kPieceRows][65];
  __shared__ int64_t rp[kPieceRows];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t ng = (m + kPieceRows - 1) / kPieceRows;
  for (int64_t g = blockIdx.x; g < ng; g += gridDim.x)
    each_piece(g, m, gstart, eptr, nrun, rend, [&](int64_t row, int nr, int len, int64_t slot) {
      __syncthreads();  // the previous piece's tiles are out
      if (threadIdx.x < nr) rp[threadIdx.x] = row_ptr[row + threadIdx.x];
      __syncthreads();
      for (int e0 = 64 * blockIdx.y; e0 < len; e0 += 64 * gridDim.y) {
        const int e = e0 + lane;
        double v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const int r = w + 4 * q;
          v[q] = (r < nr && e < len) ? val[rp[r] + e] : 0.0;
        }
        int32_t p[16];  // of columns e0 + w + 4 q
#pragma unroll
        for (int q = 0; q < 16; ++q) p[q] = e0 + w + 4 * q < len ? pos[slot + e0 + w + 4 * q] : 0;
#pragma unroll
        for (int q = 0; q < 16; ++q) tile[w + 4 * q][lane] = v[q];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const int c = w + 4 * q;
          if (e0 + c < len && lane < nr) {
            const int64_t o = (int64_t)p[q] + lane;
            at_val[o] = tile[lane][c];
            at_col[o] = (int32_t)(row + lane);
          }
        }
        __syncthreads();
      }
    });
}

}  // namespace

// The sample is a launch of 4.9 us more for a matrix of pieces (whole transposes, 8,000 x
// 1,200 of 150 a row 52 to 58 us, 100,000 x 9,000 of 160 199 us) and spares one without
// them the runs and their counts, which go by rows: 105,000 rows of 10 scattered entries
// 276 us without and 244 with, 600,000 of 20 1.64 and 1.51 ms, 2,000,000 of 12 6.94 and
// 6.40.  A system of fewer rows is likely the former, and one of these rows takes at
// least 0.15 ms.
constexpr int64_t kProbeMinRows = (int64_t)1 << 18;
const int* probe_pieces(hipStream_t st, const rfmls_csr* M, int* bad) {
  if (M->m < kProbeMinRows) {
    hipLaunchKernelGGL(k_clear_flag, dim3(1), dim3(1), 0, st, bad);
    return nullptr;
  }
  hipLaunchKernelGGL(k_probe_pieces, dim3(1), dim3(64 * kProbeGroups), 0, st, M->row_ptr, M->col, M->m, bad);
  return bad;
}

rfmls_status run_transpose(rfmls_handle* h, const rfmls_csr* A, int64_t* rp, int32_t* at_col,
                           double* at_val) {
  const int64_t m = A->m, n = A->n;
  int64_t rc = (m + 1023) / 1024;
  if (rc < 32) rc = 32;
  const int64_t nchunk = m > 0 ? (m + rc - 1) / rc : 0;
  void *p_hist, *p_count;
  RFMLS_CHECK(workspace(h, WS_TRANSPOSE, sizeof(int32_t) * (size_t)(nchunk > 0 ? nchunk : 1) * (size_t)n, &p_hist));
  RFMLS_CHECK(workspace(h, WS_SKETCH_COUNT, sizeof(int32_t) * (size_t)(n + 1), &p_count));
  int32_t* hist = (int32_t*)p_hist;
  int32_t* count = (int32_t*)p_count;
  Trace tr(h, "transpose", 2.0 * (12.0 * (double)A->nnz) + 8.0 * (double)(m + n + 2), 0.0);
  // Piece by piece where a matrix is large enough for the extra small launches
  // (about 12, 40 us) to pay: the 10,752 x 1,600 system of 1.2 M entries is even or
  // just faster (9.86 -> 9.74 ms a solve).  Pieces must average at least kTrPieceRows
  // rows over the entries, or their entry lists would approach the matrix's own size.
  constexpr int64_t kTrPieceMinNnz = (int64_t)1 << 20;
  constexpr int64_t kTrPieceRows = 8;
  const bool try_pieces = A->nnz >= kTrPieceMinNnz && m > 0;
  const int64_t ng = (m + kPieceRows - 1) / kPieceRows, cap = A->nnz / kTrPieceRows;
  const int64_t gc = (ng + 127) / 128;  // groups per chunk
  const int64_t nch = gc > 0 ? (ng + gc - 1) / gc : 0;
  int* mode = nullptr;
  unsigned long long* gstart = nullptr;
  int64_t* eptr = nullptr;
  int32_t *nrun = nullptr, *rcol = nullptr, *rend = nullptr, *pos = nullptr, *phist = nullptr;
  if (try_pieces) {
    void* pw;
    const size_t runs_b = sizeof(int32_t) * (size_t)m * (1 + 2 * kMaxRuns);
    RFMLS_CHECK(workspace(h, WS_TR_PIECES,
                          256 + sizeof(int64_t) * (size_t)(2 * ng + 2) + sizeof(int32_t) * (size_t)(ng + 2) + runs_b +
                              sizeof(int32_t) * ((size_t)cap + (size_t)nch * (size_t)n + 16),
                          &pw));
    int* bad = (int*)pw;
    mode = bad + 1;
    gstart = (unsigned long long*)((char*)pw + 256);
    eptr = (int64_t*)(gstart + ng);
    int32_t* elen = (int32_t*)(eptr + ng + 1);
    nrun = elen + ng + 2;
    rcol = nrun + m;
    rend = rcol + m * kMaxRuns;
    pos = rend + m * kMaxRuns;
    phist = pos + cap;
    const int* skip = probe_pieces(h->stream, A, bad);
    find_runs(h->stream, A, nrun, rcol, rend, skip);
    hipLaunchKernelGGL(k_tr_groups, dim3(ceil_div(ng, 4)), dim3(256), 0, h->stream, m, n, (const int32_t*)nrun,
                       (const int32_t*)rcol, (const int32_t*)rend, gstart, elen, bad);
    RFMLS_CHECK(scan_counts(h, elen, ng, eptr, skip));
    hipLaunchKernelGGL(k_tr_mode, dim3(1), dim3(1), 0, h->stream, (const int*)bad, (const int64_t*)eptr, ng, cap, mode);
    hipLaunchKernelGGL(k_tr_piece_walk<false>, dim3((unsigned)nch), dim3(256), 0, h->stream, m, n, gc,
                       (const unsigned long long*)gstart, (const int64_t*)eptr, (const int32_t*)nrun,
                       (const int32_t*)rcol, (const int32_t*)rend, phist, (const int64_t*)nullptr, pos,
                       (const int*)mode);
    hipLaunchKernelGGL(k_tr_colscan, dim3(ceil_div(n, 256)), dim3(256), 0, h->stream, phist, nch, n, count,
                       (const int*)mode, 1);
    RFMLS_HIP(h, hipGetLastError());
  }
  if (nchunk > 0) {
    hipLaunchKernelGGL(k_tr_hist, dim3((unsigned)nchunk), dim3(256), 0, h->stream, A->row_ptr,
                       A->col, m, n, rc, hist, (const int*)mode);
    hipLaunchKernelGGL(k_tr_colscan, dim3(ceil_div(n, 256)), dim3(256), 0, h->stream, hist, nchunk,
                       n, count, (const int*)mode, 0);
  } else {
    RFMLS_HIP(h, hipMemsetAsync(count, 0, sizeof(int32_t) * (size_t)n, h->stream));
  }
  RFMLS_HIP(h, hipGetLastError());
  RFMLS_CHECK(scan_counts(h, count, n, rp));
  if (try_pieces) {
    hipLaunchKernelGGL(k_tr_piece_walk<true>, dim3((unsigned)nch), dim3(256), 0, h->stream, m, n, gc,
                       (const unsigned long long*)gstart, (const int64_t*)eptr, (const int32_t*)nrun,
                       (const int32_t*)rcol, (const int32_t*)rend, phist, (const int64_t*)rp, pos, (const int*)mode);
    // about eight workgroups per compute unit over the groups, at most 32
    const int64_t most = 32 * (int64_t)h->num_cus;
    int64_t ys = (8 * (int64_t)h->num_cus + ng - 1) / ng;
    if (ys > 8) ys = 8;
    hipLaunchKernelGGL(k_tr_piece_fill, dim3((unsigned)(ng < most ? ng : most), (unsigned)ys), dim3(256), 0, h->stream, A->row_ptr, A->val,
                       m, (const unsigned long long*)gstart, (const int64_t*)eptr, (const int32_t*)nrun,
                       (const int32_t*)rend, (const int32_t*)pos, at_col, at_val, (const int*)mode);
    RFMLS_HIP(h, hipGetLastError());
  }
  if (nchunk > 0) {
    hipLaunchKernelGGL(k_tr_fill, dim3((unsigned)nchunk), dim3(256), 0, h->stream, A->row_ptr,
                       A->col, A->val, m, n, rc, hist, rp, at_col, at_val, (const int*)mode);
    RFMLS_HIP(h, hipGetLastError());
  }
  return RFMLS_OK;
}

}  // namespace rfmls
