// Blocked Householder QR of the sketch SA (s x n, row-major, in place):
// Alg. 1 step 3.  Only R is needed; Q is never formed, and the rows of a sparse
// sketch are first sorted by where they start (sort_rows), so that s below is the
// number of rows that have started.
//
// Two levels of blocking.  Outer blocks of kOuter = 256 or 512 columns
// are factored panel by panel (kMaxNb = 64 columns each); the trailing matrix
// right of an outer block is then updated once, with K = kOuter, which keeps
// that update -- most of the flops -- on the matrix cores instead of bound by
// HBM traffic.
//
// Inner panel at column p0 (M = s - p0 rows):
//   k_qr_panel   unblocked Householder on the M x 64 panel, spread over G
//                co-resident workgroups (rows held in registers); each column
//                needs one grid-wide sum of sigma = sum_{i>j} a_ij^2, d_c =
//                sum_{i>j} a_ij a_ic and the pivot row, after which every
//                workgroup forms the same reflector and applies it to its rows;
//   inside the outer block: W = V^T [V | C] (split-K GEMM), T from V^T V
//                (the inverse of its strict upper part plus diag(1/tau), by
//                back substitution), C <- C - V (T^T W).
// Outer block at column k0 (M0 = s - k0 rows, V_o = its kOuter Householder vectors):
//   W = V_o^T [V_o | C] (split-K GEMM; the first kOuter columns are the Gram V_o^T V_o),
//   W' = T_o^T W_C without forming T_o's off-diagonal blocks: T_o's block
//   recurrence T_o[:q, q] = -T_o[:q, :q] (V_:q^T V_q) T_qq turns the product
//   into a forward substitution by blocks with the Gram's blocks and the
//   panels' T (k_qr_outer_wp),  then C <- C - V_o W'.
// All reductions run in a fixed order, so the factorisation is deterministic.
#include "common.h"
#include "gemm.h"

namespace rfmls {
namespace {

constexpr int kMaxNb = 64;
// CholeskyQR2 panels: at least this many rows, and the first Cholesky's pivot ratio
// below which a panel falls back to the unblocked kernel (scaled panel condition
// near u^{-1/2}).  The unblocked kernel exchanges sums between workgroups for every
// column, 190 to 230 us a panel at 128 to 1,024 rows, CholeskyQR2's passes and
// factorisations about 100 us (2x2-box solve 3.0 -> 2.4 ms against a limit of 1,024
// rows, when they took 120).
constexpr int64_t kCholqrMinRows = 128;
constexpr double kCholqrMinPivot = 1e-7;

// Cross-block exchange of the panel kernel.  Every value crosses blocks in a
// "low-latency" slot: the float64 travels as two 64-bit words (its low or high
// 32 bits, and a tag in the upper 32 bits), each written and read with one
// relaxed agent-scope atomic, which is coherent across the XCDs' separate L2
// caches.  A reader accepts the value once both words carry the tag it
// expects, so no flag, counter or store-completion wait sits on the critical
// path: a hand-over costs one store propagation plus one load round trip.
// Tags are the column's index in the matrix + 1, unique within one QR; the
// slots are zeroed once per QR (a stale value from an earlier panel carries
// another tag).
__device__ __forceinline__ void ll_put(uint64_t* slot, double v, unsigned tag) {
  const uint64_t x = (uint64_t)__double_as_longlong(v);
  const uint64_t t = (uint64_t)tag << 32;
  __hip_atomic_store(&slot[0], (x & 0xffffffffull) | t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(&slot[1], (x >> 32) | t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Wait (bounded) for the value tagged `tag`; on time-out flag the error, clear
// the block's `ok` and return 0.
__device__ __forceinline__ bool ll_try(uint64_t* p, unsigned tag, double* v) {
  const uint64_t a = __hip_atomic_load(&p[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint64_t b = __hip_atomic_load(&p[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if ((unsigned)(a >> 32) != tag || (unsigned)(b >> 32) != tag) return false;
  *v = __longlong_as_double((long long)((a & 0xffffffffull) | (b << 32)));
  return true;
}
constexpr int kSpinLimit = 1 << 20;
__device__ __forceinline__ double ll_wait(const uint64_t* slot, unsigned tag, int* err, int* ok) {
  uint64_t* p = const_cast<uint64_t*>(slot);
  double v = 0.0;
  for (int spins = 0; !ll_try(p, tag, &v); ++spins) {
    if (spins > kSpinLimit) {
      atomicExch(err, 1);
      *ok = 0;
      return 0.0;
    }
    __builtin_amdgcn_s_sleep(4);
  }
  return v;
}
// Two values polled together (one round trip per attempt for both).  Every
// workgroup polls the same few slots here (the totals and the pivot row), so
// the attempts are spaced out: 24 x 64 clocks between them measured about 1%
// faster on the whole panel than back-to-back polls (fewer reads queue at
// those cache lines), and two polls kept in flight 8% slower.
__device__ __forceinline__ void ll_wait2(const uint64_t* s0, const uint64_t* s1, unsigned tag,
                                         double* v0, double* v1, int* err, int* ok) {
  uint64_t* p0 = const_cast<uint64_t*>(s0);
  uint64_t* p1 = const_cast<uint64_t*>(s1);
  bool d0 = false, d1 = false;
  for (int spins = 0;; ++spins) {
    if (!d0) d0 = ll_try(p0, tag, v0);
    if (!d1) d1 = ll_try(p1, tag, v1);
    if (d0 && d1) return;
    if (spins > kSpinLimit) {
      atomicExch(err, 1);
      *ok = 0;
      *v0 = *v1 = 0.0;
      return;
    }
    __builtin_amdgcn_s_sleep(24);
  }
}

// Unblocked Householder QR of an M x nb panel (nb <= 64) spread over G
// co-resident workgroups of NT = 1024 threads (16 wavefronts), one per CU.
// Thread (c = lane, rg = wavefront) of block g holds rows
// r0 + rg + 16 q (q < Q, r0 = g rpw, rpw = 16 Q) of column c in registers;
// all lanes of a wavefront hold the same rows, so column j reaches every lane
// by v_readlane from lane j (no LDS).  Block 0 holds rows 0 .. rpw-1 >= nb-1.
//
// Column j needs one grid-wide sum: sigma = sum_{i>j} a_ij^2 and
// d_c = sum_{i>j} a_ij a_ic (c > j), plus the pivot row a_jc from block 0.
// Each block publishes its partial sums (slots r1[j&1][c][g]) and block 0 the
// pivot row (rp[j&1][c]).  With G >= 64 blocks, block c sums the G partials of
// column c (each of its first G threads waits for one, then a fixed-order
// wavefront tree and an ordered sum of the wavefront results) and publishes
// the total (r2[j&1][c]); every block then reads the nb - j totals.  With
// fewer blocks every block sums all G partials itself (16 threads per column,
// each over blocks p, p + 16, ..., then those 16 partial sums in order).  Every
// block thus receives bit-identical totals and forms the same reflector (LAPACK
// dlarfg convention: beta = -sign(alpha) ||(alpha, x)||, tau = (beta -
// alpha)/beta, v = [1; x/(alpha-beta)]), computed once per block by the thread
// of column j, and applies it to its rows.  Slots of column j are reused by
// column j + 2 only: a block can publish column j + 2 only after every block
// has published column j + 1, which each does after reading column j.
//   ll  slots, 16 bytes each: r1 [2][64][G], rp [2][64], r2 [2][64]

constexpr int kPanelThreads = 1024;
constexpr int kPanelGroups = kPanelThreads / 64;  // wavefronts per block
constexpr int kPanelMaxBlocks = kPanelThreads;    // a reducer thread per block
__host__ __device__ constexpr int64_t ll_words(int64_t G) { return 2 * (2 * kMaxNb * G + 4 * kMaxNb); }

template <typename T, int Q>
__global__ void __launch_bounds__(kPanelThreads)
    k_qr_panel(T* __restrict__ P, int64_t ld, int64_t M, int nb, int rpw, T* __restrict__ tau,
               uint64_t* __restrict__ ll, int* __restrict__ err, unsigned tag0, const int* __restrict__ run_if,
               const double* __restrict__ R1) {
  static_assert(kPanelGroups * Q >= kMaxNb, "block 0 must hold the panel's top rows");
  // gated launch (after a CholeskyQR2 attempt): every block reads the same
  // flag and leaves before any exchange when the panel is already factored
  if (run_if && *run_if == 0) return;
  __shared__ double red[2 * kMaxNb];               // totals, then the pivot row
  __shared__ double grp[kPanelGroups][kMaxNb];     // per-wavefront partials
  __shared__ double part[kPanelGroups][kMaxNb];    // partial sums of the totals
  __shared__ double piv[kMaxNb];                   // pivot row (block 0)
  __shared__ double refl[3];                       // beta, tau, 1/(alpha - beta)
  __shared__ int ok;
  const int G = gridDim.x;
  const int g = blockIdx.x;
  const int tid = threadIdx.x;
  const int c = tid & 63;
  const int rg = tid >> 6;  // wavefront index: uniform within a wavefront
  const int64_t r0 = (int64_t)g * rpw;
  const int nr = (int)(M - r0 < rpw ? (M - r0 > 0 ? M - r0 : 0) : rpw);
  uint64_t* r1 = ll;                                // [2][kMaxNb][G] slots
  uint64_t* rp = ll + 2 * (2 * kMaxNb * (int64_t)G);  // [2][kMaxNb]
  uint64_t* r2 = rp + 2 * (2 * kMaxNb);               // [2][kMaxNb]
  if (tid == 0) ok = 1;

  // rows beyond the panel are held as zeros and contribute nothing
  T a[Q];
  const int64_t rstep = (int64_t)kPanelGroups * ld;  // between a thread's rows
  {
    const T* pr = P + (r0 + rg) * ld + c;
#pragma unroll
    for (int q = 0; q < Q; ++q, pr += rstep) {
      const int li = rg + kPanelGroups * q;
      a[q] = (li < nr && c < nb) ? *pr : T(0);
    }
  }

  const bool top = (g == 0);
  for (int j = 0; j < nb; ++j) {
    const unsigned tag = tag0 + (unsigned)j + 1u;
    const int par = j & 1;
    const int L = nb - j;
    // Only block 0 holds rows i <= j (li > j is uniform per wavefront).
    if (top && rg == (j % kPanelGroups)) {  // pivot row j lives in this wavefront
      const int qj = j / kPanelGroups;
      double pv = 0.0;
#pragma unroll
      for (int q = 0; q < Q; ++q) pv = (q == qj) ? (double)a[q] : pv;
      piv[c] = pv;
    }
    // ---- local partials over rows i > j: sum_i a_ij a_ic ----
    // (up to 16 rows per thread, a_ij of the wavefront's rows is kept for the
    // update below, column j not changing in between; more rows would spill)
    constexpr bool kKeep = Q <= 16;
    double s = 0.0;
    T aj[kKeep ? Q : 1];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int li = rg + kPanelGroups * q;
      // rows li >= kMaxNb > j always take part (compile-time for large q)
      if (kPanelGroups * q >= kMaxNb || !top || li > j) {
        const T v = (T)lane_read(a[q], j);
        if constexpr (kKeep) aj[q] = v;
        s += (double)v * (double)a[q];
      } else if constexpr (kKeep) {
        aj[q] = T(0);
      }
    }
    grp[rg][c] = s;
    __syncthreads();
    if (tid < 64 && c >= j && c < nb) {
      double t = 0.0;
#pragma unroll
      for (int q = 0; q < kPanelGroups; ++q) t += grp[q][c];
      ll_put(&r1[2 * (((int64_t)par * kMaxNb + c) * G + g)], t, tag);
      if (top) ll_put(&rp[2 * (par * kMaxNb + c)], piv[c], tag);
    }
    // ---- totals ----
    double tot = 0.0;  // thread c (< 64): total of column c
    if (G >= kMaxNb) {
      if (g >= j && g < nb) {  // this block sums column g (block-uniform branch)
        double v = 0.0;
        if (tid < G) v = ll_wait(&r1[2 * (((int64_t)par * kMaxNb + g) * G + tid)], tag, err, &ok);
        v = wave_sum(v);
        if (c == 0) part[rg][0] = v;
        __syncthreads();
        if (tid == 0) {
          double t = 0.0;
#pragma unroll
          for (int q = 0; q < kPanelGroups; ++q) t += part[q][0];
          ll_put(&r2[2 * (par * kMaxNb + g)], t, tag);
        }
      }
    } else {
      if (c >= j && c < nb) {
        double t = 0.0;
        for (int gg = rg; gg < G; gg += kPanelGroups)
          t += ll_wait(&r1[2 * (((int64_t)par * kMaxNb + c) * G + gg)], tag, err, &ok);
        part[rg][c] = t;
      }
      __syncthreads();
      if (tid < 64 && c >= j && c < nb) {
#pragma unroll
        for (int q = 0; q < kPanelGroups; ++q) tot += part[q][c];
      }
    }
    if (tid < 64 && c >= j && c < nb) {
      double pc;
      if (G >= kMaxNb)
        ll_wait2(&r2[2 * (par * kMaxNb + c)], &rp[2 * (par * kMaxNb + c)], tag, &tot, &pc, err, &ok);
      else
        pc = ll_wait(&rp[2 * (par * kMaxNb + c)], tag, err, &ok);
      red[c - j] = tot;
      red[L + c - j] = pc;
      if (c == j) {  // the reflector, once per block
        const double alpha = pc, sigma = tot;
        double beta = alpha, tj = 0.0, scal = 0.0;
        if (sigma != 0.0) {
          const double nrm = sqrt(alpha * alpha + sigma);
          beta = alpha >= 0.0 ? -nrm : nrm;
          tj = (beta - alpha) / beta;
          scal = 1.0 / (alpha - beta);
        }
        refl[0] = beta;
        refl[1] = tj;
        refl[2] = scal;
        if (top) tau[j] = (T)tj;
      }
    }
    __syncthreads();
    if (!ok) return;  // a partner block did not answer (error flag set)
    // ---- apply H_j to rows i >= j of columns c > j; column j becomes v ----
    const double beta = refl[0], tj = refl[1], scal = refl[2];
    const bool upd = (c > j && c < nb && tj != 0.0);
    const double f = upd ? tj * (red[L + c - j] + scal * red[c - j]) : 0.0;
    const double sf = scal * f;
    // one multiply-add per row below the diagonal, with no per-lane branch:
    // a - sf v_j on the columns updated, scal v_j on column j (it becomes v),
    // a + 0 v_j (exactly a) on the columns left alone
    const double kv = upd ? -sf : (c == j ? scal : 0.0);
    const bool keep = (c != j);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int li = rg + kPanelGroups * q;
      if (kPanelGroups * q >= kMaxNb || !top || li > j) {
        double vj;
        if constexpr (kKeep) vj = (double)aj[q];
        else vj = lane_read(a[q], j);  // read before lane j rewrites it
        a[q] = (T)fma(kv, vj, keep ? (double)a[q] : 0.0);
      } else if (li == j) {
        a[q] = (T)(upd ? (double)a[q] - f : (c == j ? beta : (double)a[q]));
      }
    }
    // no barrier here: the next writes of red, refl and part follow the next
    // column's first __syncthreads, and piv / grp are not read after this point
  }
  T* pw_row = P + (r0 + rg) * ld + c;
  // an opaque copy: otherwise the compiler reuses the Q row addresses of the
  // initial loads here and keeps them alive (spilled) across the whole kernel
  asm volatile("" : "+v"(pw_row));
#pragma unroll
  for (int q = 0; q < Q; ++q, pw_row += rstep) {
    const int li = rg + kPanelGroups * q;
    if (li < nr && c < nb) *pw_row = a[q];
  }
  // after a failed second Cholesky the panel was Q1: its R times R1 (64 x 64 upper
  // triangular, terms in order), by the workgroup that holds the top rows
  if (run_if && *run_if == 2 && top) {
    __syncthreads();
    double o[kMaxNb / kPanelGroups];
#pragma unroll
    for (int q = 0; q < kMaxNb / kPanelGroups; ++q) {
      const int r = rg + kPanelGroups * q;
      double s = 0.0;
      for (int k = r; k <= c; ++k) s = fma((double)P[(int64_t)r * ld + k], R1[k * kMaxNb + c], s);
      o[q] = s;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kMaxNb / kPanelGroups; ++q) {
      const int r = rg + kPanelGroups * q;
      if (c >= r) P[(int64_t)r * ld + c] = (T)o[q];
    }
  }
}

// T (nb x nb upper triangular, row-major) of the compact-WY form H_1 ... H_nb =
// I - V T V^T from tau and the Gram V^T V (the leading nb columns of W, nb x ldw),
// and W' = T^T W_C for the ncol columns of W after it.
// T is the inverse of U = (strictly upper part of V^T V) + diag(1/tau): that
// is the matrix form of the column recursion T[:j, j] = -tau_j T[:j, :j]
// V_:j^T v_j (Schreiber and Van Loan).  Column k of T solves U t = e_k by
// back substitution on one wavefront (lane i holds row i), t_l = tau_l x_l
// from the bottom up, so 1/tau is never formed and a reflector with tau_j = 0
// (H_j = I) leaves row and column j zero, as the recursion does; a column of W'
// solves U^T w' = w the same way from the top down, so it needs no T and both
// go in one launch.  One wavefront per column, 16 to a workgroup, each workgroup
// staging the Gram: the first ceil(nb / 16) form T, the others W' (none for
// ncol = 0).  Bound by the loads and the 64-step chains.  Forming T first and
// multiplying by it in a second launch took 8.5 + 11.3 us for 192 columns; this 8.1
// (Helmholtz solve 26.4 -> 25.7 ms).
template <typename T>
__global__ void __launch_bounds__(1024)
    k_qr_T_wp(const T* __restrict__ W, int64_t ldw, int nb, const T* __restrict__ tau, T* __restrict__ Tout,
              int64_t ldt, int64_t ncol, T* __restrict__ Wp, int64_t ldwp) {
  // Us[i][l] = (V^T V)_il for i < l < nb, zero elsewhere, so the updates below
  // need no per-row test (rows that are done subtract exactly 0)
  __shared__ double Us[kMaxNb][kMaxNb + 1];
  __shared__ double Ws[kMaxNb][16 + 1];
  __shared__ double ts[kMaxNb + 3];  // three zero entries below index 0 (steps past l = 0)
  constexpr int kCols = 16;          // columns per workgroup
  const int tid = threadIdx.x;
  const int nT = (nb + kCols - 1) / kCols;
  const int64_t c0 = ((int64_t)blockIdx.x - nT) * kCols;
  // clamped addresses, unused values dropped by selects: the loads go out together
  double g[kMaxNb * kMaxNb / 1024];
#pragma unroll
  for (int q = 0; q < kMaxNb * kMaxNb / 1024; ++q) {
    const int e = tid + 1024 * q, i = e / kMaxNb, l = e % kMaxNb;
    g[q] = (double)W[(int64_t)min(i, nb - 1) * ldw + min(l, nb - 1)];
  }
  const double tv = tid < kMaxNb + 3 ? (double)tau[min(max(tid - 3, 0), nb - 1)] : 0.0;
  if (c0 >= 0) {
    const int k = tid / kCols;
    const int64_t c = c0 + tid % kCols;
    const double v = (double)W[(int64_t)min(k, nb - 1) * ldw + nb + (c < ncol ? c : ncol - 1)];
    Ws[k][tid % kCols] = k < nb ? v : 0.0;
  }
#pragma unroll
  for (int q = 0; q < kMaxNb * kMaxNb / 1024; ++q) {
    const int e = tid + 1024 * q, i = e / kMaxNb, l = e % kMaxNb;
    Us[i][l] = i < l && l < nb ? g[q] : 0.0;
  }
  if (tid < kMaxNb + 3) ts[tid] = tid >= 3 && tid - 3 < nb ? tv : 0.0;
  __syncthreads();
  const int lane = tid & 63, w = tid >> 6;
  if (c0 < 0) {
    const int k = (int)blockIdx.x * kCols + w;
    if (k >= nb) return;  // uniform within the wavefront (no barrier follows)
    double x = lane == k ? 1.0 : 0.0, t = 0.0;
    // four steps per group, their LDS reads issued together; steps past l = 0
    // read tau = 0 and column 0 of Us (zeros) and change nothing
    for (int l0 = k; l0 >= 0; l0 -= 4) {
      double u[4], tt[4];
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const int l = l0 - d;
        u[d] = Us[lane][l > 0 ? l : 0];
        tt[d] = ts[l + 3];
      }
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const int l = l0 - d;
        const double tl = tt[d] * lane_read(x, l > 0 ? l : 0);  // x_l is final once rows > l are done
        if (lane == l) t = tl;
        x -= u[d] * tl;
      }
    }
    if (lane < nb) Tout[(int64_t)lane * ldt + k] = (T)(lane <= k ? t : 0.0);
    return;
  }
  double x = Ws[lane][w], t = 0.0;
  for (int l0 = 0; l0 < kMaxNb; l0 += 4) {  // tau = 0 past nb
    double u[4], tt[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      u[d] = Us[l0 + d][lane];
      tt[d] = ts[l0 + d + 3];
    }
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const double tl = tt[d] * lane_read(x, l0 + d);  // x_l is final once rows < l are done
      if (lane == l0 + d) t = tl;
      x -= u[d] * tl;
    }
  }
  Ws[lane][w] = t;
  __syncthreads();
  const int k = tid / kCols;
  const int64_t c = c0 + tid % kCols;
  if (k < nb && c < ncol) Wp[(int64_t)k * ldwp + c] = (T)Ws[k][tid % kCols];
}
template <typename T>
void launch_T_wp(hipStream_t st, const T* W, int64_t ldw, int nb, const T* tau, T* Tout, int64_t ldt, int64_t ncol = 0,
                 T* Wp = nullptr, int64_t ldwp = 0) {
  hipLaunchKernelGGL(k_qr_T_wp<T>, dim3((unsigned)((nb + 15) / 16 + (ncol + 15) / 16)), dim3(1024), 0, st, W, ldw, nb,
                     tau, Tout, ldt, ncol, Wp, ldwp);
}

// W = the sum of the nsplit slices of Wz in slice order, 16 bytes a thread (len a
// multiple of 32, slices 16-byte aligned), eight slices' loads in flight: bound by
// reading the slices (4^3-box float32 sketch 176 -> 125 us, one element a thread before).
template <typename T>
__global__ void __launch_bounds__(256) k_sum_slices(const T* __restrict__ Wz, int64_t zstride, int nsplit, int64_t len,
                                                    T* __restrict__ W) {
  constexpr int E = 16 / sizeof(T);
  typedef T vec __attribute__((ext_vector_type(E)));
  for (int64_t e = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * E; e < len;
       e += (int64_t)gridDim.x * blockDim.x * E) {
    double acc[E] = {};
    int z = 0;
    for (; z + 8 <= nsplit; z += 8) {
      vec v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = *(const vec*)(Wz + (int64_t)(z + q) * zstride + e);
#pragma unroll
      for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int i = 0; i < E; ++i) acc[i] += (double)v[q][i];
    }
    for (; z < nsplit; ++z) {
      const vec v = *(const vec*)(Wz + (int64_t)z * zstride + e);
#pragma unroll
      for (int i = 0; i < E; ++i) acc[i] += (double)v[i];
    }
    vec o;
#pragma unroll
    for (int i = 0; i < E; ++i) o[i] = (T)acc[i];
    *(vec*)(W + e) = o;
  }
}

// The same sum for one panel's V^T [V | C] (a short range over many slices):
// a workgroup per 64 elements, its four wavefronts summing every fourth slice,
// the four partial sums then added in a fixed order.
template <typename T>
__global__ void __launch_bounds__(256)
    k_sum_slices_narrow(const T* __restrict__ Wz, int64_t zstride, int nsplit, int64_t len,
                        T* __restrict__ W) {
  __shared__ double part[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t e = (int64_t)blockIdx.x * 64 + lane;
  double acc = 0.0;
  if (e < len) {
#pragma unroll 4
    for (int z = w; z < nsplit; z += 4) acc += (double)Wz[(int64_t)z * zstride + e];
  }
  part[w][lane] = acc;
  __syncthreads();
  if (w == 0 && e < len) W[e] = (T)((part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]));
}

__global__ void k_zero_u64(uint64_t* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0ull;
}

// Outer block width: 512 columns for float32, whose trailing update then
// reads and writes the trailing matrix half as often (4^3-box sketch: 2.5% less
// QR time than 256), and for float64 from 12,800 columns on (4^3-box, 25,600
// columns: 1.3% less solve time; 8x8-box, 12,800 columns: QR phase 327.8 ->
// 325.1 ms, the trailing products' 9 ms saved less the inner 64-column
// products, which grow with the width); narrower float64 systems keep 256.
constexpr int64_t kOuterMax = 512;
template <typename T>
int64_t outer_width(int64_t n) { return sizeof(T) == 4 || n >= 12800 ? 512 : 256; }
inline int64_t pad32(int64_t x) { return (x + 31) / 32 * 32; }

// Row slices of an inner panel's split-K product V^T [V | C]: its output is
// only 64 rows by at most kOuter columns, so the slices are what fills the
// GPU.  256-row slices from 32,768 rows on, 128 below (8x8-box sketch, QR
// phase 325.4 -> 323.6 ms against 512-row slices; Helmholtz sketch, 12,800
// rows, 20.35 -> 19.74 ms; 128-row slices on the 8x8-box sketch 325-327 ms,
// the slice sums' extra reads outweighing the fuller grid).
inline int64_t inner_split(int64_t M) { return M >= 32768 ? 256 : 128; }
// most slices any panel of an s-row sketch takes
inline int64_t inner_slices_max(int64_t s) {
  const int64_t a = (s + inner_split(s) - 1) / inner_split(s);
  const int64_t ms = s < 32767 ? s : 32767;
  const int64_t b = (ms + 127) / 128;
  return a > b ? a : b;
}
// Row slices of an outer block's V^T [V | C] below its masked top rows:
// 4096 rows from 32,768 rows on (2% faster than 8192 on the 8x8-box sketch,
// net of the longer slice sum; 2048 there measured even).  Below, the largest of
// 4096, 2048 and kOuterSplitShort rows that leaves 64 x 64 tiles times slices for
// kOuterMinTiles workgroups over the nl columns from the block on (Helmholtz sketch,
// 12,800 rows: V^T C 4.07 -> 3.15 ms per solve with 1024 rows against 4096; 2048 rows
// 3.45 ms, 8192 rows 6.6 ms), since every slice is written and read once more.
// 8x8-box sketch in sorted order, under 32,768 rows: the slice sum 112 -> 36 us against
// 1024 rows, the product even.
// nl and not the product's own columns decides, so that a product split by
// columns (look-ahead) keeps every column's sums.
constexpr int64_t kOuterSplitShort = 1024;
constexpr int64_t kOuterMinTiles = 2048;
inline int64_t outer_split(int64_t M0, int64_t bw, int64_t nl) {
  if (M0 >= 32768) return 4096;
  int64_t sp = 4096;
  while (sp > kOuterSplitShort && (bw / 64) * ((nl + 63) / 64) * ((M0 + sp - 1) / sp) < kOuterMinTiles) sp /= 2;
  return sp;
}
// most slices any outer block of an s-row sketch takes (the masked top rows
// and a ragged tail included)
inline int64_t outer_slices_max(int64_t s) {
  const int64_t a = (s + 4095) / 4096;
  const int64_t ms = s < 32767 ? s : 32767;
  const int64_t b = (ms + kOuterSplitShort - 1) / kOuterSplitShort;
  return (a > b ? a : b) + 2;
}

// W' = T_o^T W_C for an outer block of NQ 64-column panels, without forming
// T_o's blocks above the diagonal.  Since T_o[:q0, q] = -T_o[:q0, :q0]
// G[:q0, q] T_q (G = V_o^T V_o, q the panel at column q0, T_q its T), block
// row q of T_o^T W_C is
//   W'_q = T_q^T (W_q - G[:q0, q]^T W'[:q0]),
// a forward substitution by blocks that every column runs on its own.  G's
// blocks above the diagonal are read from G (rows ldg apart), each T_q (upper
// triangular, zeros stored below the diagonal) from the diagonal 64-blocks of
// Td (rows ldt apart), W_C from W (NQ * 64 rows, ldw apart).  One workgroup
// per 16 columns; wavefront w forms rows 16 w .. 16 w + 15 of each 64-row
// block on the matrix cores, in float64 for either storage type, and the rows
// of W' formed so far stay in LDS.
template <typename T, int NQ>
__global__ void __launch_bounds__(256)
    k_qr_outer_wp(const T* __restrict__ W, int64_t ldw, const T* __restrict__ G, int64_t ldg,
                  const T* __restrict__ Td, int64_t ldt, int64_t ncol, T* __restrict__ Wp, int64_t ldwp) {
  typedef double v4d __attribute__((ext_vector_type(4)));
  constexpr int SW = 16;
  __shared__ double Xs[NQ * kMaxNb][SW + 1];  // W' rows formed so far
  __shared__ double Ys[kMaxNb][SW + 1];       // W_q - G[:q0, q]^T W'[:q0]
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const int i0 = 16 * w;
  const int64_t col = (int64_t)blockIdx.x * SW + lr;
  const bool cin = col < ncol;
  // operand layout of v_mfma_f64_16x16x4f64: lane (lr, lk) holds A[lr][lk] and
  // B[lk][lr]; accumulator register r holds D[lk + 4 r][lr]
  for (int q = 0; q < NQ; ++q) {
    const int q0 = kMaxNb * q;
    // G[:q0, q]^T W'[:q0]: A[i][k] = G[k][q0 + i], B[k][c] = W'[k][c], K in
    // chunks of 64 (the next chunk's operands loaded during this one's
    // products), two accumulators (even and odd steps)
    v4d acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = {0.0, 0.0, 0.0, 0.0};
    const T* ga = G + q0 + i0 + lr;
    double a[16];
    if (q0 > 0)
#pragma unroll
      for (int j = 0; j < 16; ++j) a[j] = (double)ga[(int64_t)(4 * j + lk) * ldg];
    for (int kc = 0; kc < q0; kc += 64) {
      double an[16];
      const bool more = kc + 64 < q0;
      if (more)
#pragma unroll
        for (int j = 0; j < 16; ++j) an[j] = (double)ga[(int64_t)(kc + 64 + 4 * j + lk) * ldg];
#pragma unroll
      for (int j = 0; j < 16; j += 2) {
        acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[j], Xs[kc + 4 * j + lk][lr], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[j + 1], Xs[kc + 4 * j + 4 + lk][lr], acc1, 0, 0, 0);
      }
      if (more)
#pragma unroll
        for (int j = 0; j < 16; ++j) a[j] = an[j];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + lk + 4 * r;
      const double wv = cin ? (double)W[(int64_t)(q0 + i) * ldw + col] : 0.0;
      Ys[i][lr] = wv - (acc0[r] + acc1[r]);
    }
    __syncthreads();
    // W'_q = T_q^T Y: A[i][k] = T_q[k][i], zero for k > i, so the K range of
    // rows i0 .. i0 + 15 ends at i0 + 16
    const T* ta = Td + (int64_t)q0 * ldt + q0 + i0 + lr;
    const int nk = 4 * (w + 1);
    double tv[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) tv[j] = (double)ta[(int64_t)(4 * j + lk) * ldt];  // inside the block
    v4d o0 = {0.0, 0.0, 0.0, 0.0}, o1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 16; j += 2) {
      if (j < nk) {
        o0 = __builtin_amdgcn_mfma_f64_16x16x4f64(tv[j], Ys[4 * j + lk][lr], o0, 0, 0, 0);
        o1 = __builtin_amdgcn_mfma_f64_16x16x4f64(tv[j + 1], Ys[4 * j + 4 + lk][lr], o1, 0, 0, 0);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + lk + 4 * r;
      const double v = o0[r] + o1[r];
      Xs[q0 + i][lr] = v;
      if (cin) Wp[(int64_t)(q0 + i) * ldwp + col] = (T)v;
    }
    __syncthreads();
  }
}

// The Gram's 64-blocks above the diagonal (rows ldw apart in W) into the same
// places of To (rows ldt apart), whose diagonal blocks hold the panels' T:
// what k_qr_outer_wp needs when a later product reuses the outer block.
template <typename T>
__global__ void k_qr_keep_gram(const T* __restrict__ W, int64_t ldw, int bw, T* __restrict__ To, int64_t ldt) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)bw * bw) return;
  const int r = (int)(e / bw), c = (int)(e % bw);
  if (r / kMaxNb < c / kMaxNb) To[(int64_t)r * ldt + c] = W[(int64_t)r * ldw + c];
}

// ---------------------------------------------------------------------------
// Row order of a sparse sketch.  R does not depend on the order of SA's rows, and
// a row takes part in the elimination only from the column of its first nonzero
// on.  A sketch row is the sum of a few rows of A, each over one or two boxes'
// columns, so its first nonzero lies anywhere in [0, n).  Sorted by the 64-column
// panel of their first nonzero, the rows of panel k and before fill rows
// [0, act[k]) and those below are still zero in panel k's columns: every product
// and panel of the QR runs over act[k] - p rows instead of s - p.  On the
// 8x8-box sketch (51,200 x 12,800, 2.2 rows of A per sketch row) that is 0.41 of
// the flops, on the 4^3-box one 0.48, on the Helmholtz one 0.72.  Measured, whole
// solves: 8x8-box 368 -> 248 ms (the trailing products 115 -> 57, V^T C 117 -> 60
// ms, the rows' move 3 ms), 4^3-box float32 703 -> 505 ms, Helmholtz 30.2 -> 29.8,
// 4x4-box 11.2 -> 11.0 ms.
// ---------------------------------------------------------------------------
// key[i] = panel of row i's first nonzero (npan for a zero row); one wavefront per row.
// cnt[0 .. npan] = 0.
template <typename T>
__global__ void __launch_bounds__(256)
    k_row_keys(const T* __restrict__ SA, int64_t ld, int64_t s, int64_t n, int npan, int32_t* __restrict__ key,
               int32_t* __restrict__ cnt) {
  if (blockIdx.x == 0)
    for (int k = threadIdx.x; k <= npan; k += 256) cnt[k] = 0;
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= s) return;
  const T* p = SA + row * ld;
  int k = npan;
  constexpr int kAhead = 4;  // panels read together: the search is a chain of loads
  for (int64_t c0 = 0; c0 < n; c0 += kAhead * kMaxNb) {
    T v[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const int64_t c = c0 + q * kMaxNb + lane;
      v[q] = c < n ? p[c] : T(0);
    }
    int f = npan;
#pragma unroll
    for (int q = kAhead - 1; q >= 0; --q)
      if (__ballot(v[q] != T(0))) f = (int)(c0 / kMaxNb) + q;
    if (f < npan) {  // uniform
      k = f;
      break;
    }
  }
  if (lane == 0) key[row] = k;
}

// cnt[k] += rows of key k, counted in LDS by chunks of kCountRows (npan < kCountKeys: a
// sketch has at most 512 rows a compute unit, and as many columns).
constexpr int kCountRows = 4096, kCountKeys = 4096;
__global__ void __launch_bounds__(1024)
    k_row_counts(const int32_t* __restrict__ key, int64_t s, int npan, int32_t* __restrict__ cnt) {
  __shared__ int32_t c[kCountKeys];
  for (int k = threadIdx.x; k <= npan; k += 1024) c[k] = 0;
  __syncthreads();
  const int64_t i0 = (int64_t)blockIdx.x * kCountRows;
#pragma unroll
  for (int q = 0; q < kCountRows / 1024; ++q) {
    const int64_t i = i0 + q * 1024 + threadIdx.x;
    if (i < s) atomicAdd(&c[key[i]], 1);
  }
  __syncthreads();
  for (int k = threadIdx.x; k <= npan; k += 1024)
    if (c[k]) atomicAdd(&cnt[k], c[k]);
}

// Stable sort of the rows by key: workgroup k starts after the rows of smaller keys and
// lists its own in ascending order.
__global__ void __launch_bounds__(1024)
    k_row_order(const int32_t* __restrict__ key, int64_t s, const int32_t* __restrict__ cnt, int32_t* __restrict__ perm) {
  __shared__ int wsum[16];
  const int k = blockIdx.x;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (cnt[k] == 0) return;  // uniform
  int below = 0;
  for (int q = threadIdx.x; q < k; q += 1024) below += cnt[q];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) below += __shfl_xor(below, off, 64);
  if (lane == 0) wsum[w] = below;
  __syncthreads();
  int base = 0;
#pragma unroll
  for (int q = 0; q < 16; ++q) base += wsum[q];
  for (int64_t i0 = 0; i0 < s; i0 += 1024) {
    const int64_t i = i0 + threadIdx.x;
    const bool mine = i < s && key[i] == k;
    const unsigned long long b = __ballot(mine);
    __syncthreads();  // the previous round's sums have been read
    if (lane == 0) wsum[w] = __popcll(b);
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      before += q < w ? wsum[q] : 0;
      all += wsum[q];
    }
    if (mine) perm[base + before + __popcll(b & ((1ull << lane) - 1ull))] = (int32_t)i;
    base += all;
  }
}

// out[i][c] = in[row(i)][c], c < width; row(i) = perm[i], or i without perm
template <typename T>
__global__ void __launch_bounds__(256)
    k_move_rows(const T* __restrict__ in, int64_t ldi, const int32_t* __restrict__ perm, int64_t width,
                T* __restrict__ out, int64_t ldo) {
  const int64_t i = blockIdx.x;
  const T* p = in + (perm ? (int64_t)perm[i] : i) * ldi;
  T* o = out + i * ldo;
  for (int64_t c = threadIdx.x; c < width; c += 256) o[c] = p[c];
}

// Panel launch shapes (rows per thread Q, rows per block 16 Q), increasing.
// The largest are the largest that compile without spills at 1024 threads.
struct PanelShape {
  int q;
  const void* fn;
  int64_t rpw() const { return (int64_t)kPanelGroups * q; }
};
template <typename T>
const PanelShape* panel_shapes() {
  static const PanelShape s[] = {{4, (const void*)k_qr_panel<T, 4>},
                                 {8, (const void*)k_qr_panel<T, 8>},
                                 {16, (const void*)k_qr_panel<T, 16>},
                                 {32, (const void*)k_qr_panel<T, 32>},
                                 {0, nullptr}};
  return s;
}

// The smallest shape whose grid (G = ceil(M / rows per block)) fits one block
// per CU: fewer rows per thread means less arithmetic per column on the
// critical path, and one block per CU keeps the SIMDs' shares equal (two
// blocks on some CUs would double their work per column).
template <typename T>
rfmls_status pick_panel_shape(rfmls_handle* h, int64_t M, PanelShape* out, int64_t* G_out) {
  for (const PanelShape* sh = panel_shapes<T>(); sh->q != 0; ++sh) {
    int per_cu = 0;
    RFMLS_HIP(h, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, sh->fn, kPanelThreads, 0));
    int64_t gmax = per_cu >= 1 ? (int64_t)h->num_cus : 0;
    if (gmax > kPanelMaxBlocks) gmax = kPanelMaxBlocks;
    const int64_t G = (M + sh->rpw() - 1) / sh->rpw();
    if (G <= gmax) {
      *out = *sh;
      *G_out = G;
      return RFMLS_OK;
    }
  }
  return fail(h, RFMLS_E_ARG, "QR panel of %lld rows does not fit one co-resident grid",
              (long long)M);
}

template <typename T>
GemmArgs<T> vt_gemm(T* P, int64_t ld, int64_t M, int64_t vcols, int64_t ncols, T* out,
                    int64_t ldo, int64_t ksplit) {
  // out_z = V^T [V | C] over row slices: V = the vcols Householder vectors
  // stored below the diagonal of P, C the next ncols - vcols columns; rows of
  // out are ldo apart, slices vcols ldo apart
  GemmArgs<T> g;
  g.M = vcols;
  g.N = ncols;
  g.K = M;
  g.A = P;
  g.lda = ld;
  g.transA = 1;
  g.a_vmask = 1;
  g.B = P;
  g.ldb = ld;
  g.b_vcols = vcols;
  g.C = out;
  g.ldc = ldo;
  g.alpha = T(1);
  g.beta = T(0);
  g.ksplit = ksplit;
  g.c_zstride = vcols * ldo;
  return g;
}

template <typename T>
GemmArgs<T> v_update(T* P, int64_t ld, int64_t M, int64_t vcols, int64_t ncols, const T* Wp,
                     int64_t ldwp) {
  // C <- C - V Wp, C = the ncols columns right of the vcols Householder vectors
  // (rows of Wp ldwp apart)
  GemmArgs<T> g;
  g.M = M;
  g.N = ncols;
  g.K = vcols;
  g.A = P;
  g.lda = ld;
  g.a_vmask = 1;
  g.B = Wp;
  g.ldb = ldwp;
  g.C = P + vcols;
  g.ldc = ld;
  g.alpha = T(-1);
  g.beta = T(1);
  return g;
}

// Rows that a panel or an outer block works on: all s, or with sorted rows the
// act[k] rows whose first nonzero lies in panel k or before it.
struct RowCounts {
  int64_t s = 0, n = 0;  // the sketch's rows and columns
  std::vector<int64_t> act;  // per 64-column panel; empty: s
  int64_t at(int64_t col) const { return act.empty() ? s : act[(size_t)(col / kMaxNb)]; }
};

// Buffers of one outer block's panels: tau and the diagonal 64-blocks of T_o
// (written by the panels), and the inner products' slices, Gram and T^T W.
template <typename T>
struct PanelBufs {
  T* tau;
  T* To;
  T* Wz;
  T* W;
  T* Wp;
};

// The inner panels of the outer block [k0, k0 + bw) of SA, each factored and
// applied to the rest of the block, on h->stream; tau_out (if given) receives
// the block's tau.
template <typename T>
rfmls_status qr_block_panels(rfmls_handle* h, const RowCounts& rows, int64_t k0, int64_t bw, int64_t kOuter, T* SA,
                             int64_t ld, const PanelBufs<T>& pb, uint64_t* ll, double* cq_ws, int* cq_status, T* tau_out) {
  hipStream_t st = h->stream;
  for (int64_t p0 = k0; p0 < k0 + bw; p0 += kMaxNb) {
    const int jb = (int)(k0 + bw - p0 < kMaxNb ? k0 + bw - p0 : kMaxNb);
    const int64_t M = rows.at(p0) - p0;
    const int64_t split_in = inner_split(M);
    PanelShape sh;
    int64_t G = 0;
    RFMLS_CHECK(pick_panel_shape<T>(h, M, &sh, &G));
    const int64_t rpw = sh.rpw();
    T* P = SA + p0 * ld + p0;
    T* tau_p = pb.tau + (p0 - k0);
    int rpw_i = (int)rpw;
    unsigned tag0 = (unsigned)p0;
    const int* run_if = nullptr;
    const double* r1 = nullptr;
    // Householder on an M x jb panel: sum_j 4 (M - j)(jb - j) flops; panel
    // read and written once (the method's work, whichever way it is factored)
    const double pf = 4.0 * (double)M * jb * (jb + 1) / 2.0;
    if (cq_ws && jb == kMaxNb && M >= kCholqrMinRows) {
      // 64-column panels: CholeskyQR2 + reconstruction in float64 arithmetic;
      // the unblocked kernel below then runs only for a panel it flagged
      Trace tr(h, "qr_panel_cq", 2.0 * sizeof(T) * (double)M * jb, pf);
      const double thr1 = h->qr_panel == 2 ? 2.0 : kCholqrMinPivot;
      const double thr2 = h->qr_panel == 3 ? 2.0 : kCholqrMinPivot;
      RFMLS_CHECK(run_cholqr_panel(h, P, ld, M, tau_p, cq_ws, cq_status, thr1, thr2));
      run_if = cq_status;
      r1 = cholqr_r1(cq_ws, M);
    }
    void* args[] = {(void*)&P,     (void*)&ld, (void*)&M,            (void*)&jb,   (void*)&rpw_i,
                    (void*)&tau_p, (void*)&ll, (void*)&h->dev_flags, (void*)&tag0, (void*)&run_if,
                    (void*)&r1};
    const void* fn = sh.fn;
    {
      Trace tr(h, run_if ? "qr_panel_fallback" : "qr_panel", run_if ? 0.0 : 2.0 * sizeof(T) * (double)M * jb,
               run_if ? 0.0 : pf);
      // The gated launch after CholeskyQR2 on the main stream is an ordinary
      // launch: nothing else runs beside it, so its G <= one-per-CU workgroups
      // are all resident when it does run (its waits are bounded either way),
      // and the cooperative launch's own overhead (about 15 us per panel,
      // 200 panels on the 8x8-box sketch) is not paid when it does nothing.
      if (run_if && !h->qr_lookahead)
        RFMLS_HIP(h, hipLaunchKernel(fn, dim3((unsigned)G), dim3(kPanelThreads), args, 0, st));
      else
        RFMLS_HIP(h, hipLaunchCooperativeKernel(fn, dim3((unsigned)G), dim3(kPanelThreads), args, 0, st));
    }
    const int64_t rem = k0 + bw - (p0 + jb);
    if (rem <= 0) continue;
    const int64_t ncols = jb + rem;
    const int64_t ldw = pad32(ncols), ldwp = pad32(rem);
    const int64_t nsp = (M + split_in - 1) / split_in;
    {
      Trace tr(h, "qr_inner_VtC", sizeof(T) * ((double)M * ncols + (double)nsp * jb * ncols),
               2.0 * (double)jb * ncols * M);
      RFMLS_HIP(h, (gemm<T, GemmRole::QrInnerVtC>(vt_gemm<T>(P, ld, M, jb, ncols, pb.Wz, ldw, split_in), st)));
      hipLaunchKernelGGL(k_sum_slices_narrow<T>, dim3(ceil_div(jb * ldw, 64)), dim3(256), 0, st, (const T*)pb.Wz,
                         (int64_t)jb * ldw, (int)nsp, (int64_t)jb * ldw, pb.W);
    }
    {
      Trace tr(h, "qr_inner_T", sizeof(T) * 2.0 * jb * ncols, 2.0 * (double)jb * jb * rem);
      // this panel's T is also a diagonal block of the outer block's T_o
      T* Tq = pb.To + (p0 - k0) * kOuter + (p0 - k0);
      launch_T_wp<T>(st, pb.W, ldw, jb, tau_p, Tq, kOuter, rem, pb.Wp, ldwp);
    }
    {
      Trace tr(h, "qr_inner_update", sizeof(T) * (2.0 * (double)M * rem + (double)M * jb),
               2.0 * (double)M * rem * jb);
      RFMLS_HIP(h, (gemm<T, GemmRole::QrInnerUpdate>(v_update<T>(P, ld, M, jb, rem, pb.Wp, ldwp), st)));
    }
    RFMLS_HIP(h, hipGetLastError());
  }
  // every reflector's tau, for a caller that applies Q afterwards
  if (tau_out)
    RFMLS_HIP(h, hipMemcpyAsync(tau_out + k0, pb.tau, sizeof(T) * (size_t)bw, hipMemcpyDeviceToDevice, st));
  return RFMLS_OK;
}

// Buffers of the trailing update: the outer products' slices, W = V^T [.],
// and W' = T_o^T W.
template <typename T>
struct TrailBufs {
  T* Wz;
  T* W;
  T* Wp;
};

// Trailing update C <- C - V T_o^T (V^T C) with the outer block [k0, k0 + bw)
// (V below its diagonal in SA) for the nc columns starting off columns right
// of the block (nc_m of them the method's own, the rest tile padding within
// the room).  With gram, off must be 0: the product then also covers V itself,
// and T_o is built from that Gram (its diagonal 64-blocks from the panels,
// except the last panel's); without, T_o must already hold the block's T.
template <typename T>
rfmls_status qr_block_trailing(rfmls_handle* h, const RowCounts& rows, int64_t k0, int64_t bw, int64_t kOuter, T* SA,
                               int64_t ld, int64_t off, int64_t nc, int64_t nc_m, bool gram, const T* tau, T* To,
                               const TrailBufs<T>& tb, bool keep_gram = false) {
  hipStream_t st = h->stream;
  const int64_t M0 = rows.at(k0 + bw - 1) - k0;
  const int64_t split_out = outer_split(M0, bw, rows.n - k0);
  T* P0 = SA + k0 * ld + k0;
  const int64_t vc = gram ? bw : 0;  // V's own columns in the product
  const int64_t ncols = vc + nc, ncols_m = vc + nc_m;
  const int64_t ldw = pad32(ncols), ldwp = pad32(nc);
  T* Bc = P0 + bw + off;  // first product column when V is not included
  // V^T [V | C] (or V^T C) in row slices summed in order: rows [0, bw) hold the
  // triangle of V (masked, general kernel); the rows below are clear of every
  // mask, so a whole number of 16-row chunks of them goes to the clean-only
  // kernel in split_out-row slices, and a tail of fewer than 16 rows (if any) to the
  // general kernel without masks
  const int64_t Kc = (M0 - bw) / 16 * 16, Kt = M0 - bw - Kc;
  const int64_t nsc = (Kc + split_out - 1) / split_out;
  const int64_t nsp = 1 + nsc + (Kt > 0 ? 1 : 0);
  const int64_t zs = bw * ldw;
  auto product = [&](int64_t r0, int64_t nr, T* out, int64_t ksplit) {
    GemmArgs<T> g = vt_gemm<T>(P0 + r0 * ld, ld, nr, bw, ncols, out, ldw, ksplit);
    if (!gram) {
      g.B = Bc + r0 * ld;
      g.b_vcols = 0;
    }
    return g;
  };
  {
    Trace tr(h, gram ? "qr_gemm_VtC" : "qr_gemm_VtC_rest",
             sizeof(T) * ((double)M0 * ncols_m + 2.0 * (double)nsp * bw * ncols_m), 2.0 * (double)bw * ncols_m * M0);
    {
      // op(A) = V^T of the top rows is upper triangular (the mask zeroes the
      // rest): each row tile starts its K range at its own first row
      GemmArgs<T> gt = product(0, bw, tb.Wz, 0);
      gt.a_upper = 1;
      RFMLS_HIP(h, (gemm<T, GemmRole::QrVtC>(gt, st)));
    }
    if (Kc > 0) {
      GemmArgs<T> gc = product(bw, Kc, tb.Wz + zs, split_out);
      gc.a_vmask = 0;
      gc.b_vcols = 0;
      // the kOuter / 64 row tiles of a B strip run together (56 -> 59 TFLOP/s,
      // float64, 256-column blocks) on one XCD (then 481 -> 469 ms on the
      // 4^3-box float64 solve's 512-column blocks, equal at 256)
      gc.tile_order = 3;
      RFMLS_HIP(h, (gemm_clean<T, GemmRole::QrVtC>(gc, st)));
    }
    if (Kt > 0) {
      GemmArgs<T> gr = product(bw + Kc, Kt, tb.Wz + (1 + nsc) * zs, 0);
      gr.a_vmask = 0;
      gr.b_vcols = 0;
      RFMLS_HIP(h, (gemm<T, GemmRole::QrVtC>(gr, st)));
    }
    const int64_t per = 256 * 16 / sizeof(T);  // elements a workgroup sums at a time
    hipLaunchKernelGGL(k_sum_slices<T>, dim3(ceil_div(bw * ldw, per) < 4096 ? ceil_div(bw * ldw, per) : 4096),
                       dim3(256), 0, st, (const T*)tb.Wz, bw * ldw, (int)nsp, zs, tb.W);
  }
  if (gram) {
    // the last panel's T (no inner update followed it) from the Gram's
    // diagonal block; the other panels wrote theirs into To's diagonal
    Trace tr(h, "qr_outer_T", sizeof(T) * 2.0 * kMaxNb * kMaxNb, 2.0 * (double)kMaxNb * kMaxNb * kMaxNb / 3.0);
    const int64_t q0 = (bw - 1) / kMaxNb * kMaxNb;
    const int jq = (int)(bw - q0);
    launch_T_wp<T>(st, tb.W + q0 * ldw + q0, ldw, jq, tau + q0, To + q0 * kOuter + q0, kOuter);
    if (keep_gram)
      hipLaunchKernelGGL(k_qr_keep_gram<T>, dim3((unsigned)ceil_div(bw * bw, 256)), dim3(256), 0, st,
                         (const T*)tb.W, ldw, (int)bw, To, kOuter);
  }
  {
    // W' = T_o^T W[:, C's columns] by forward substitution with the Gram's
    // blocks (from this product, or kept in To by an earlier one) and the
    // panels' T
    Trace tr(h, "qr_outer_Wp", sizeof(T) * 2.0 * (double)bw * nc_m, (double)bw * bw * nc_m);
    const T* Gp = gram ? tb.W : To;
    const int64_t ldg = gram ? ldw : kOuter;
    const unsigned nb = (unsigned)ceil_div(nc, 16);
    if (bw == 4 * kMaxNb)
      hipLaunchKernelGGL((k_qr_outer_wp<T, 4>), dim3(nb), dim3(256), 0, st, (const T*)(tb.W + vc), ldw, Gp, ldg,
                         (const T*)To, kOuter, nc, tb.Wp, ldwp);
    else if (bw == 8 * kMaxNb)
      hipLaunchKernelGGL((k_qr_outer_wp<T, 8>), dim3(nb), dim3(256), 0, st, (const T*)(tb.W + vc), ldw, Gp, ldg,
                         (const T*)To, kOuter, nc, tb.Wp, ldwp);
    else
      return fail(h, RFMLS_E_ARG, "outer block of %lld columns", (long long)bw);
  }
  {
    Trace tr(h, gram ? "qr_gemm_update" : "qr_gemm_update_rest",
             sizeof(T) * (2.0 * (double)M0 * nc_m + (double)M0 * bw + (double)bw * nc_m), 2.0 * (double)M0 * nc_m * bw);
    // rows [0, bw) meet the triangle of V (masked, general kernel); the rows
    // below are clear of it and take the clean-only kernel
    {
      // V's top rows are lower triangular (the mask zeroes the rest): each
      // row tile ends its K range at its own last row
      GemmArgs<T> gt = v_update<T>(P0, ld, bw, bw, nc, tb.Wp, ldwp);
      gt.C = P0 + bw + off;
      gt.a_lower = 1;
      RFMLS_HIP(h, (gemm<T, GemmRole::QrTrailingUpdate>(gt, st)));
    }
    if (M0 > bw) {
      GemmArgs<T> gu = v_update<T>(P0 + bw * ld, ld, M0 - bw, bw, nc, tb.Wp, ldwp);
      gu.C = P0 + bw * ld + bw + off;
      gu.a_vmask = 0;
      gu.tile_order = 2;  // bands of 32 tile rows: 53.8 -> 56.5 TFLOP/s (float64, 51200 x 12800)
      RFMLS_HIP(h, (gemm_clean<T, GemmRole::QrTrailingUpdate>(gu, st)));
    }
  }
  RFMLS_HIP(h, hipGetLastError());
  return RFMLS_OK;
}

// Second stream and its two events for the look-ahead (created on first use).
rfmls_status lookahead_stream(rfmls_handle* h) {
  if (h->la_stream) return RFMLS_OK;
  if (hipStreamCreateWithFlags(&h->la_stream, hipStreamNonBlocking) != hipSuccess) {
    h->la_stream = nullptr;
    return fail(h, RFMLS_E_HIP, "QR look-ahead: could not create its stream");
  }
  for (int i = 0; i < 2; ++i)
    if (hipEventCreateWithFlags(&h->la_event[i], hipEventDisableTiming) != hipSuccess)
      return fail(h, RFMLS_E_HIP, "QR look-ahead: could not create its events");
  return RFMLS_OK;
}

// Sorts SA's rows by the panel of their first nonzero where that saves at least
// a tenth of the QR's work, and gives the rows each panel works on.  tmp (tmp_len
// elements) holds a slab of columns during the move: a slab's rows are gathered
// into tmp in the new order and copied back, the rows still zero there left where
// they are (nothing reads them until a later slab moves them).
//   act[k]  at least the panel's rows (so that R's rows exist), and at least
//           kCholqrMinRows of them, so that the first panels of a sparse sketch
//           stay on CholeskyQR2; whole multiples of 64 keep the clean kernels.
// Costs a host wait for the counts (40 to 60 us with the search; the order is formed only
// where it is used), so small sketches, where the panels' latency is most of the time, and
// narrow ones, which have little work to save, keep their order.  The lines by sketches of
// some rows dense and the others starting anywhere, factored sorted against as given (ms):
// 1,448 x 362 at 0.50 of the work 1.41 against 1.35, 2,048 x 512 at 0.44 1.52 against 1.44;
// 2,896 x 724 (2^21 elements) at 0.43 2.52 against 2.52, 4,096 x 1,024 at 0.82, 0.64 and 0.41
// 3.10, 3.07 and 3.05 against 3.03; 6,400 x 1,600 at 0.97, 0.90, 0.82, 0.64 and 0.40 5.25,
// 5.24, 5.17, 5.08 and 4.95 against 5.16.  Columns: 131,072 x 64 0.37 against 0.32 and 60,000
// x 200 1.02 against 0.97 (0.40 and 1.21 with unblocked panels), 9,000 x 250 1.07 against
// 1.00, 33,500 x 320 1.30 against 1.41.
constexpr int64_t kSortMinElems = (int64_t)1 << 21;
constexpr int64_t kSortMinCols = 256;
template <typename T>
rfmls_status sort_rows(rfmls_handle* h, int64_t s, int64_t n, int64_t kOuter, T* SA, int64_t ld, T* tmp,
                       int64_t tmp_len, RowCounts* rows) {
  rows->s = s;
  rows->act.clear();
  if (s * n < kSortMinElems || n < kSortMinCols || n >= kMaxNb * (kCountKeys - 1) || s >= INT32_MAX) return RFMLS_OK;
  hipStream_t st = h->stream;
  const int64_t npan = (n + kMaxNb - 1) / kMaxNb;
  void* p;
  RFMLS_CHECK(workspace(h, WS_QR_ORDER, sizeof(int32_t) * (size_t)(2 * s + npan + 1), &p));
  int32_t* key = (int32_t*)p;
  int32_t* perm = key + s;
  int32_t* cnt = perm + s;
  std::vector<int32_t> c((size_t)npan + 1);
  {
    Trace tr(h, "qr_row_order", 4.0 * 3.0 * (double)s, 0.0);
    hipLaunchKernelGGL(k_row_keys<T>, dim3(ceil_div(s, 4)), dim3(256), 0, st, (const T*)SA, ld, s, n, (int)npan, key,
                       cnt);
    hipLaunchKernelGGL(k_row_counts, dim3(ceil_div(s, kCountRows)), dim3(1024), 0, st, (const int32_t*)key, s, (int)npan,
                       cnt);
    RFMLS_HIP(h, hipGetLastError());
  }
  RFMLS_HIP(h, hipMemcpyAsync(c.data(), cnt, sizeof(int32_t) * c.size(), hipMemcpyDeviceToHost, st));
  RFMLS_HIP(h, hipStreamSynchronize(st));
  std::vector<int64_t> act((size_t)npan);
  double plain = 0.0, sorted = 0.0;
  int64_t started = 0;
  for (int64_t k = 0; k < npan; ++k) {
    const int64_t p0 = k * kMaxNb;
    started += c[(size_t)k];
    int64_t a = started;
    a = a > p0 + kMaxNb + kCholqrMinRows ? a : p0 + kMaxNb + kCholqrMinRows;
    a = (a + kMaxNb - 1) / kMaxNb * kMaxNb;
    if (k > 0 && act[(size_t)k - 1] > a) a = act[(size_t)k - 1];
    act[(size_t)k] = a < s ? a : s;
    plain += (double)(s - p0) * (double)(n - p0);
    sorted += (double)(act[(size_t)k] - p0) * (double)(n - p0);
  }
  if (sorted > 0.9 * plain) return RFMLS_OK;
  // slabs of whole panels, as many columns as tmp holds for the rows that the
  // outer block of the slab's last panel works on (its V spans the whole block,
  // so a panel's zeros are needed down to there)
  const int64_t po = kOuter / kMaxNb;
  auto moved = [&](int64_t k) {
    const int64_t e = (k / po + 1) * po - 1;
    return act[(size_t)(e < npan ? e : npan - 1)];
  };
  if (moved(npan - 1) * kMaxNb > tmp_len) return RFMLS_OK;
  hipLaunchKernelGGL(k_row_order, dim3((unsigned)npan + 1), dim3(1024), 0, st, (const int32_t*)key, s,
                     (const int32_t*)cnt, perm);
  for (int64_t k0 = 0; k0 < npan;) {
    int64_t k1 = k0 + 1;
    while (k1 < npan && moved(k1) * (k1 + 1 - k0) * kMaxNb <= tmp_len) ++k1;
    const int64_t c0 = k0 * kMaxNb, w = (k1 * kMaxNb < n ? k1 * kMaxNb : n) - c0, na = moved(k1 - 1);
    Trace tr(h, "qr_row_move", 2.0 * sizeof(T) * (double)na * (double)w, 0.0);
    hipLaunchKernelGGL(k_move_rows<T>, dim3((unsigned)na), dim3(256), 0, st, (const T*)(SA + c0), ld,
                       (const int32_t*)perm, w, tmp, w);
    hipLaunchKernelGGL(k_move_rows<T>, dim3((unsigned)na), dim3(256), 0, st, (const T*)tmp, w, (const int32_t*)nullptr,
                       w, SA + c0, ld);
    k0 = k1;
  }
  RFMLS_HIP(h, hipGetLastError());
  rows->act.swap(act);
  return RFMLS_OK;
}

// n_room >= n columns of SA may be written: the big trailing products round
// their column count up to the tile width inside that room (full tiles, no
// ragged edge); the extra columns only ever hold values nothing reads.
//
// Look-ahead (rfmls_qr_lookahead, float64 CholeskyQR2 panels only): after the
// panels of outer block k, the trailing update first covers only block k + 1's
// columns; block k + 1's panels then run on a second stream while the main
// stream updates the remaining columns, and the main stream waits for them
// before block k + 1's own trailing update.  The split is by columns, every
// column's sums run in the same order, and the two streams touch disjoint
// columns and buffers (T_o and tau alternate between two copies, the panels
// have their own product buffers), so the factors are bitwise the same.
template <typename T>
rfmls_status qr_impl(rfmls_handle* h, int64_t s, int64_t n, int64_t n_room, T* SA, int64_t ld, T* tau_out) {
  const int64_t kOuter = outer_width<T>(n);
  // a sketch with more rows than a panel's grid can hold is refused as it stands, also
  // where sorted rows would leave every panel fewer
  PanelShape widest;
  int64_t blocks = 0;
  RFMLS_CHECK(pick_panel_shape<T>(h, s, &widest, &blocks));
  const int64_t nsp_in_max = inner_slices_max(s);
  const int64_t nsp_out_max = outer_slices_max(s);
  void *p_tau, *p_part, *p_wz, *p_w, *p_wp, *p_to, *p_in;
  RFMLS_CHECK(workspace(h, WS_QR_TAU, sizeof(T) * 2 * kOuterMax, &p_tau));
  RFMLS_CHECK(workspace(h, WS_QR_PART, sizeof(uint64_t) * ll_words(kPanelMaxBlocks), &p_part));
  // rows of the products W, W' are padded to 32 elements (128-byte aligned
  // rows for every column count)
  const int64_t npad = pad32(n_room);
  const size_t wz_out = (size_t)nsp_out_max * kOuter * (size_t)npad;
  RFMLS_CHECK(workspace(h, WS_QR_W, sizeof(T) * wz_out, &p_wz));
  RFMLS_CHECK(workspace(h, WS_QR_WR, sizeof(T) * kOuter * (size_t)npad, &p_w));
  RFMLS_CHECK(workspace(h, WS_QR_WP, sizeof(T) * kOuter * (size_t)npad, &p_wp));
  RFMLS_CHECK(workspace(h, WS_QR_T, sizeof(T) * 2 * kOuter * kOuter, &p_to));
  // the panels' own product buffers: slices, Gram and T^T W of at most
  // 64 x kOuter each
  const int64_t kop = pad32(kOuter);
  const size_t in_wz = (size_t)nsp_in_max * kMaxNb * kop, in_w = (size_t)kMaxNb * kop;
  RFMLS_CHECK(workspace(h, WS_QR_INNER, sizeof(T) * (in_wz + 2 * in_w), &p_in));
  // CholeskyQR2 panels (rfmls_qr_panel_mode): workspace for the largest
  // panel and one status word after it
  double* cq_ws = nullptr;
  int* cq_status = nullptr;
  if (h->qr_panel != 1 && s >= kCholqrMinRows) {
    const int64_t nd = cholqr_workspace_doubles(s);
    void* p_cq;
    RFMLS_CHECK(workspace(h, WS_CHOLQR, sizeof(double) * (size_t)(nd + 8), &p_cq));
    cq_ws = (double*)p_cq;
    cq_status = (int*)(cq_ws + nd);
  }
  // only panels that never wait on each other's workgroups may run beside the
  // trailing products: CholeskyQR2 in its normal mode
  const bool lookahead = h->qr_lookahead && cq_ws && h->qr_panel == 0;
  if (lookahead) RFMLS_CHECK(lookahead_stream(h));
  hipStream_t st = h->stream;
  T* tau2[2] = {(T*)p_tau, (T*)p_tau + kOuterMax};
  T* To2[2] = {(T*)p_to, (T*)p_to + kOuter * kOuter};
  const TrailBufs<T> tb = {(T*)p_wz, (T*)p_w, (T*)p_wp};
  T* in = (T*)p_in;
  uint64_t* ll = (uint64_t*)p_part;
  {
    // the panels' exchange slots, zeroed once: their tags are column indices
    const int64_t nll = ll_words(kPanelMaxBlocks);
    hipLaunchKernelGGL(k_zero_u64, dim3(ceil_div(nll, 256) < 512 ? ceil_div(nll, 256) : 512), dim3(256), 0, st, ll,
                       nll);
  }
  auto bufs = [&](int64_t blk) {
    PanelBufs<T> pb = {tau2[blk & 1], To2[blk & 1], in, in + in_wz, in + in_wz + in_w};
    return pb;
  };
  // the rows' order is free when no reflector is applied afterwards
  RowCounts rows;
  rows.s = s;
  rows.n = n;
  if (!tau_out) RFMLS_CHECK(sort_rows<T>(h, s, n, kOuter, SA, ld, tb.Wz, (int64_t)wz_out, &rows));
  // block k + 1's panels all CholeskyQR2-eligible (64 columns, enough rows)
  auto cq_block = [&](int64_t k1, int64_t bw1) {
    for (int64_t p = k1; p < k1 + bw1; p += kMaxNb)
      if (rows.at(p) - p < kCholqrMinRows) return false;
    return bw1 % kMaxNb == 0;
  };
  RFMLS_CHECK(qr_block_panels<T>(h, rows, 0, n < kOuter ? n : kOuter, kOuter, SA, ld, bufs(0), ll, cq_ws, cq_status,
                                 tau_out));
  int64_t blk = 0;
  for (int64_t k0 = 0; k0 < n; k0 += kOuter, ++blk) {
    const int64_t bw = n - k0 < kOuter ? n - k0 : kOuter;
    if (n - k0 - bw <= 0) break;
    const int64_t k1 = k0 + bw, bw1 = n - k1 < kOuter ? n - k1 : kOuter;
    // columns right of the block, rounded up to the widest tile (128) within
    // the room; the method's own are the traced work
    const int64_t ntr = (n_room < (n + 127) / 128 * 128 ? n_room : (n + 127) / 128 * 128) - k0 - bw;
    const int64_t ntr_m = n - k0 - bw;
    const PanelBufs<T> pb = bufs(blk), pb1 = bufs(blk + 1);
    if (lookahead && ntr_m > kOuter && cq_block(k1, bw1)) {
      // block k + 1's columns first, its panels on the second stream, the rest here
      RFMLS_CHECK(qr_block_trailing<T>(h, rows, k0, bw, kOuter, SA, ld, 0, kOuter, kOuter, true, pb.tau, pb.To, tb,
                                       true));
      RFMLS_HIP(h, hipEventRecord(h->la_event[0], st));
      RFMLS_HIP(h, hipStreamWaitEvent(h->la_stream, h->la_event[0], 0));
      h->stream = h->la_stream;
      const rfmls_status ps =
          qr_block_panels<T>(h, rows, k1, bw1, kOuter, SA, ld, pb1, ll, cq_ws, cq_status, tau_out);
      const hipError_t er = hipEventRecord(h->la_event[1], h->la_stream);
      h->stream = st;
      RFMLS_CHECK(ps);
      RFMLS_HIP(h, er);
      const rfmls_status ts = qr_block_trailing<T>(h, rows, k0, bw, kOuter, SA, ld, kOuter, ntr - kOuter,
                                                   ntr_m - kOuter, false, pb.tau, pb.To, tb);
      RFMLS_HIP(h, hipStreamWaitEvent(st, h->la_event[1], 0));
      RFMLS_CHECK(ts);
    } else {
      RFMLS_CHECK(qr_block_trailing<T>(h, rows, k0, bw, kOuter, SA, ld, 0, ntr, ntr_m, true, pb.tau, pb.To, tb));
      RFMLS_CHECK(qr_block_panels<T>(h, rows, k1, bw1, kOuter, SA, ld, pb1, ll, cq_ws, cq_status, tau_out));
    }
  }
  return RFMLS_OK;
}

}  // namespace

rfmls_status run_qr(rfmls_handle* h, int64_t s, int64_t n, int64_t n_room, rfmls_dtype dt, void* SA,
                    int64_t ld, void* tau_out) {
  if (n_room < n || n_room > ld) n_room = n;
  if (dt == RFMLS_F64) return qr_impl<double>(h, s, n, n_room, (double*)SA, ld, (double*)tau_out);
  return qr_impl<float>(h, s, n, n_room, (float*)SA, ld, (float*)tau_out);
}

// Y <- Q Y with Q = H_0 H_1 ... H_{n-1} of a float64 Householder QR left by
// run_qr in P (s x n, vectors below the diagonal, tau from its tau_out): the
// 64-column panels from last to first, each as Y <- (I - V T V^T) Y with
// T from the panel's Gram V^T V and tau, i.e. W = V^T Y, W' = T W, Y -= V W'.
rfmls_status apply_householder(rfmls_handle* h, const double* P, int64_t ld, int64_t s, int64_t n,
                               const double* tau, double* Y, int64_t ldy, int64_t ny) {
  hipStream_t st = h->stream;
  const int64_t ldw = (ny + 31) / 32 * 32;
  void* pw;
  RFMLS_CHECK(workspace(h, WS_APPLYQ, sizeof(double) * (size_t)(2 * kMaxNb * kMaxNb + 2 * kMaxNb * ldw), &pw));
  double* G = (double*)pw;
  double* Tq = G + kMaxNb * kMaxNb;
  double* W = Tq + kMaxNb * kMaxNb;
  double* Wp = W + kMaxNb * ldw;
  for (int64_t p0 = (n - 1) / kMaxNb * kMaxNb; p0 >= 0; p0 -= kMaxNb) {
    const int jb = (int)(n - p0 < kMaxNb ? n - p0 : kMaxNb);
    const int64_t M = s - p0;
    double* V = const_cast<double*>(P) + p0 * ld + p0;
    RFMLS_HIP(h, (gemm<double, GemmRole::Generic>(vt_gemm<double>(V, ld, M, jb, jb, G, kMaxNb, 0), st)));
    launch_T_wp<double>(st, G, kMaxNb, jb, tau + p0, Tq, kMaxNb);
    GemmArgs<double> gw;  // W = V^T Y[p0:, :]
    gw.M = jb;
    gw.N = ny;
    gw.K = M;
    gw.A = V;
    gw.lda = ld;
    gw.transA = 1;
    gw.a_vmask = 1;
    gw.B = Y + p0 * ldy;
    gw.ldb = ldy;
    gw.C = W;
    gw.ldc = ldw;
    RFMLS_HIP(h, (gemm<double, GemmRole::Generic>(gw, st)));
    GemmArgs<double> gt;  // W' = T W (T upper triangular)
    gt.M = jb;
    gt.N = ny;
    gt.K = jb;
    gt.A = Tq;
    gt.lda = kMaxNb;
    gt.a_upper = 1;
    gt.B = W;
    gt.ldb = ldw;
    gt.C = Wp;
    gt.ldc = ldw;
    RFMLS_HIP(h, (gemm<double, GemmRole::Generic>(gt, st)));
    GemmArgs<double> gu;  // Y[p0:, :] -= V W'
    gu.M = M;
    gu.N = ny;
    gu.K = jb;
    gu.A = V;
    gu.lda = ld;
    gu.a_vmask = 1;
    gu.B = Wp;
    gu.ldb = ldw;
    gu.C = Y + p0 * ldy;
    gu.ldc = ldy;
    gu.alpha = -1.0;
    gu.beta = 1.0;
    RFMLS_HIP(h, (gemm<double, GemmRole::Generic>(gu, st)));
  }
  RFMLS_HIP(h, hipGetLastError());
  return RFMLS_OK;
}

}  // namespace rfmls
