// Symmetric FP64 eigensolver for the rank-sized Gram matrices of the
// Gram-SVD truncation (App. A.2: G_A = V_A S_A^2 V_A^T, G_B = V_B S_B^2 V_B^T,
// and the Gram of M for its SVD).
//
// Pipeline (one job per matrix, several jobs run side by side):
//   1. Householder tridiagonalisation A = Q T Q^T (the only step with O(n)
//      sequential dependences): the matrix in one block's registers up to
//      order 192, above that the rows split over 16 to 64 blocks' registers.
//   2. Eigenpairs of T by divide and conquer from 8x8 leaves, all levels in
//      one persistent launch: the merges up to 64 rows on one block each, above
//      that one wavefront per secular root and products in tiles over the
//      blocks, with grid barriers between the phases.
//   3. Back-transformation V = Q Z, a wavefront per kept vector, with the
//      descending order, sign gauge (largest |entry| positive) and clip rule.
// The same divide and conquer also serves the small SVD of M (section 5).
#include <float.h>
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "gemm_tile.h"
#include "grid_sync.h"
#include "tt_internal.h"

namespace tt {

namespace {

constexpr double U64 = 1.1102230246251565e-16;  // 2^-53

struct EigJobs {
  EigJob j[4];
};

struct Work {
  double *d, *e, *tau, *w, *H, *Z;
};
__device__ inline Work work_of(const EigJob& J, int N) {
  Work W;
  W.d = J.work;
  W.e = W.d + N;
  W.tau = W.e + N;
  W.w = W.tau + N;
  W.H = W.w + N;
  W.Z = W.H + (size_t)N * N;
  return W;
}

__host__ __device__ inline int next_pow2(int n) {
  int p = 1;
  while (p < n) p <<= 1;
  return p;
}

// Work area of one job at capacity N, before the grid-barrier words: d, e,
// tau, w (4 N), reflectors (N x N), then the divide-and-conquer area.
// d, e, tau, w, H (N x N), then an area that the divide and conquer uses
// and, before it, the grid reductions' exchange buffers (k_gebrd's
// double-buffered partials of up to 64 blocks, more than the divide and
// conquer for small N).
__host__ __device__ inline size_t eig_work_main(int N) {
  const size_t N2 = next_pow2(N);
  const size_t dc = 2 * N2 * N2 + 17 * N2 + 64;
  const size_t grid = 2 * ((size_t)N + 64 * (size_t)N + 256) + 64;
  return 4 * (size_t)N + (size_t)N * N + N2 + (dc > grid ? dc : grid);
}

// Lane exchange inside rows of 16 lanes by DPP, on both halves of a double.
template <int CTRL>
__device__ inline double dpp_d(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = (int)b, hi = (int)(b >> 32);
  const int lo2 = __builtin_amdgcn_mov_dpp(lo, CTRL, 0xf, 0xf, true);
  const int hi2 = __builtin_amdgcn_mov_dpp(hi, CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi2 << 32) | (unsigned int)lo2);
}
__device__ inline double lane_d(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sum over the 64 lanes of a wavefront, returned on every lane, in a fixed
// order: inside each row of 16 lanes, pairs (lane ^ 1), quads (lane ^ 2),
// half rows (mirror of 8) and rows (mirror of 16), by DPP moves; then the four
// row sums, read from lanes 0, 16, 32 and 48.  At every stage the lanes of a
// row hold bitwise-equal sums (the two operands of each addition only swap),
// so every lane returns the same value.  Call with the whole wavefront active.
__device__ inline double wave_sum(double v) {
  v += dpp_d<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_d<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_d<0x141>(v);  // row_half_mirror
  v += dpp_d<0x140>(v);  // row_mirror
  return (lane_d(v, 0) + lane_d(v, 16)) + (lane_d(v, 32) + lane_d(v, 48));
}

// 1 / sqrt(x) to about an ulp for x well inside the normal range: the hardware
// estimate and one third-order step.
__device__ inline double rsqrt_d(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}
// 1 / x likewise (two Newton steps).
__device__ inline double rcp_d(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(y, fma(-x, y, 1.0), y);
  return fma(y, fma(-x, y, 1.0), y);
}

// Householder scalars of a column with first entry alpha and squared norm
// sumsq below it: H = I - tau v v^T, v = [1, scal x], takes it to beta e_1.  The
// square root and the two divisions are on every reduction's sequential
// chain, so within the range where rsqrt_d and rcp_d hold they come from
// those.
__device__ inline void householder(double alpha, double sumsq, double& tau, double& scal,
                                   double& beta) {
  if (sumsq == 0.0) {
    tau = 0.0;
    scal = 0.0;
    beta = alpha;
    return;
  }
  const double h2 = fma(alpha, alpha, sumsq);
  if (h2 > 0x1p-900 && h2 < 0x1p900) {
    const double r = rsqrt_d(h2);
    double nrm = h2 * r;
    nrm = fma(fma(-nrm, nrm, h2), 0.5 * r, nrm);
    beta = -copysign(nrm, alpha);
    tau = fma(fabs(alpha), r, 1.0);
    scal = rcp_d(alpha - beta);
  } else {
    beta = -copysign(sqrt(h2), alpha);
    tau = (beta - alpha) / beta;
    scal = 1.0 / (alpha - beta);
  }
}

// Barrier that orders LDS only: waits for this wavefront's LDS accesses
// (lgkmcnt 0), not for its global stores, then s_barrier.  For loops whose
// global stores nothing in the kernel reads back; the signal fences keep the
// compiler from moving memory accesses across it.
__device__ inline void lds_barrier() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0xC07F);  // vmcnt 63, expcnt 7, lgkmcnt 0
  __builtin_amdgcn_s_barrier();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Orders one wavefront's LDS accesses (its lanes' writes before their reads),
// for code that one wavefront runs alone.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Deterministic block-wide sum (fixed combination order).
template <int NT>
__device__ double block_sum(double v, double* red) {
  v = wave_sum(v);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < NT / 64; ++i) s += red[i];
  return s;
}

// ---------------------------------------------------------------------------
// 1. Householder tridiagonalisation (lower form): for k = 0..n-3, H_k =
// I - tau_k v v^T with v = [1, x_2..]/(alpha - beta) annihilates A[k+2:, k].
constexpr int SYR_MAX = 192;  // orders reduced in registers by k_sytrd_reg

// Large orders (n > SYR_MAX): the matrix does not fit one CU's registers,
// and one block streaming the trailing matrix from L2 is bound by that CU's
// share of the memory system.  Instead P blocks per job each keep 16 rows, 4 to
// a wavefront, in registers for the whole reduction, and step k, which needs
// T_k (the matrix after reflectors 0..k-1), runs as:
//   - every wavefront forms row k of T_k from row k of T_{k-1} (published by
//     its owner) and the previous reflector's (v, w), and v_k, tau_k from it,
//     redundantly (same data and fixed-order sums, so identical everywhere);
//   - each applies T_k = T_{k-1} - v w^T - w v^T to its rows and in the same
//     pass forms p_k = tau_k T_k,22 v_k on them and its share of p_k^T v_k;
//     the owner of row k+1 publishes it;
//   - one grid barrier; w_k = p_k - (tau_k / 2)(p_k^T v_k) v_k then follows
//     from the published p_k and the partial dots summed in a fixed order.
// Only p, the partial dots and one row cross blocks per step, by relaxed
// agent-scope accesses (xput, xget).  Bound by the exchange: at order 322
// (32 blocks) a step is about 1.7 us of barrier, 1.0 us of loads behind it,
// 0.5 us of the row and its reflector and 0.7 us of updates.  With the rows in
// LDS and a barrier that released and acquired it was 2.4, 0.7, 0.9 and 2.1.
// An eigensolve of order 206, 322, 641, 1024, before and now: 1364 -> 984,
// 2244 -> 1579, 6174 -> 5039, 11790 -> 9575 us.
// The launch is an ordinary one (a cooperative one would drain the queue on every
// call, also when all jobs are small and the kernel returns at once), so its
// blocks must be resident together beside those of other streams' launches.  A
// process has 4 hardware queues and the chip 256 CUs: every launch with grid
// barriers keeps to GRID_CUS CUs, but the reductions of capacities above
// SYG_WIDE, which keep to GRID_CUS_WIDE.  A launch has two jobs, the two sides of a
// bond.  Up to SYG_WIDE a block has at most 256 registers a lane and two fit a CU;
// above, a block takes a CU (about 430 registers; in 256 it spills, and orders
// 641 and 897 took 5836 and 11532 us instead of 5113 and 8370).  So contexts may
// step at the same time as long as their CUs add up to 256: four of them, or two
// above SYG_WIDE.  (With three jobs a launch and one block a CU, as it was, a launch
// took 96 CUs up to order 512 and 192 above, and two contexts could wait for
// each other's CUs.)
// Every wait is bounded by SYTRD_SPIN_MAX polls, after which the barrier-timeout
// flag is raised and the kernel runs out.
// Outputs (d, e, tau, reflectors in H): d, e the tridiagonal, row k of H and
// tau[k] the reflector H_k = I - tau_k v v^T (v_{k+1} = 1).
constexpr int GRID_CUS = 64, GRID_CUS_WIDE = 128;
constexpr int SYG_WIDE = 512;
constexpr int SYTRD_GRID_P = 64;
constexpr int SYTRD_GRID_T = 256;
constexpr int SYTRD_GRID_NMAX = 1024;  // largest order
constexpr int SYG_R = 4;  // rows of a wavefront
constexpr int SYG_T = SYTRD_GRID_NMAX / 64;  // columns per lane at most
constexpr unsigned SYTRD_SPIN_MAX = 1u << 24;
static_assert(SYTRD_GRID_P <= SYNC_MAXP && SYTRD_GRID_NMAX < (int)(GRID_ORD_DC - GRID_ORD_REDUCE),
              "a flag a block, an ordinal a column");

struct SytrdGridBufs {
  double *Rp, *Pv, *Dv;  // published rows (2 x N), p (2 x N), wavefront partial dots (2 x 4 P)
};
__device__ __host__ inline SytrdGridBufs sytrd_grid_bufs(double* work, int N) {
  // inside the divide-and-conquer area, which is free until the reduction ends
  const size_t N2 = next_pow2(N);
  double* z = work + 4 * (size_t)N + (size_t)N * N + N2;
  SytrdGridBufs B;
  B.Rp = z;
  B.Pv = z + 2 * (size_t)N;
  B.Dv = B.Pv + 2 * (size_t)N;
  return B;
}

// A job's barrier flags (grid_sync.h).
constexpr size_t SYNC_DOUBLES = SYNC_MAXP / 2;
__device__ inline unsigned* grid_flags(double* work, int N) {
  return reinterpret_cast<unsigned*>(work + eig_work_main(N));
}

// Barrier with ordinal `ordinal` over the P <= SYNC_MAXP blocks of one launch:
// each block stores its ordinal into its own flag (a release store after the
// block barrier, which orders the block's earlier stores before it); one wave
// polls all P flags with coherent loads, then an acquire fence.  No
// read-modify-write, so no serialisation on one address.
__device__ inline void grid_barrier(unsigned* flag, unsigned ordinal, int P, int* s_abort,
                                    int* dims) {
  __syncthreads();
  if (threadIdx.x < 64 && !*s_abort) {
    const int lane = threadIdx.x;
    if (lane == 0)
      __hip_atomic_store(&flag[blockIdx.x], ordinal, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    unsigned spins = 0;
    while (true) {
      bool ok = true;
      for (int q = lane; q < P; q += 64)
        ok = ok && grid_arrived(
                       __hip_atomic_load(&flag[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), ordinal);
      if (__all(ok)) break;
      __builtin_amdgcn_s_sleep(1);
      if (++spins > SYTRD_SPIN_MAX) {
        if (lane == 0) {
          *s_abort = 1;
          atomicOr(&dims[D_FLAG], FLAG_BARRIER);
        }
        break;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  __syncthreads();
}

// Exchange between the blocks of a launch without fences: the values are
// written and read with relaxed agent-scope accesses, which pass the caches
// that are not coherent across XCDs, so a barrier needs neither the write-back
// nor the invalidation of an L2 that release and acquire take.
__device__ inline void xput(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline double xget(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// grid_barrier for values exchanged by xput and xget: every wavefront waits for
// its stores' acknowledgements (vmcnt 0) before the block's flag is raised.
__device__ inline void grid_barrier_relaxed(unsigned* flag, unsigned ordinal, int P, int* s_abort,
                                            int* dims) {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt 0, expcnt 7, lgkmcnt 15
  __syncthreads();
  if (threadIdx.x < 64 && !*s_abort) {
    const int lane = threadIdx.x;
    if (lane == 0)
      __hip_atomic_store(&flag[blockIdx.x], ordinal, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned spins = 0;
    while (true) {
      bool ok = true;
      for (int q = lane; q < P; q += 64)
        ok = ok && grid_arrived(
                       __hip_atomic_load(&flag[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), ordinal);
      if (__all(ok)) break;
      if (++spins > SYTRD_SPIN_MAX) {
        if (lane == 0) {
          *s_abort = 1;
          atomicOr(&dims[D_FLAG], FLAG_BARRIER);
        }
        break;
      }
    }
  }
  __syncthreads();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// One block's part, for n <= 64 NT on P blocks of 4 wavefronts: wavefront w of block b
// holds the rows b + P (w + 4 r), r < 4, a lane the columns lane + 64 t.
template <int NT>
__device__ void sytrd_grid_rows(const EigJob& J, int* __restrict__ dims, int N, int n, int P,
                                double* lds, int* s_abort) {
  const int b = blockIdx.x;
  Work W = work_of(J, N);
  const SytrdGridBufs G = sytrd_grid_bufs(J.work, N);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double* lv = lds + wave * 3 * NT * 64;  // v_{k-1}, w_{k-1}, v_k of this wavefront
  double* lw = lv + NT * 64;
  double* ln = lw + NT * 64;
  double a[SYG_R][NT], v[NT], w[NT];
#pragma unroll
  for (int r = 0; r < SYG_R; ++r) {
    const int i = b + P * (wave + SYTRD_GRID_T / 64 * r);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int j = lane + 64 * t;
      a[r][t] = i < n && j < n ? J.A[(long long)i * J.lda + j] : 0.0;
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) v[t] = w[t] = 0.0;
  unsigned* flags = grid_flags(J.work, N);
  unsigned ordinal = GRID_ORD_REDUCE;
  const bool writer = b == 0 && wave == 0;
  double taup = 0.0;
  for (int k = 0; k <= n - 2; ++k) {
    // w_{k-1} on indices >= k from the published p_{k-1} and partial dots,
    // fused with row k of T_k; all loads of the step in flight together
    const int par = (k - 1) & 1;
    const double* pp = G.Pv + (size_t)par * N;
    const double* src = G.Rp + (size_t)par * N;
    double x[NT], hc = 0.0, ppk = 0.0;
    if (k == 0) {
#pragma unroll
      for (int t = 0; t < NT; ++t) x[t] = lane + 64 * t < n ? J.A[lane + 64 * t] : 0.0;
    } else {
      double pv[NT], dp[SYTRD_GRID_P / 16];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int j = lane + 64 * t;
        const bool live = j >= k && j < n;
        pv[t] = live ? xget(pp + j) : 0.0;
        x[t] = live ? xget(src + j) : 0.0;
      }
#pragma unroll
      for (int m = 0; m < SYTRD_GRID_P / 16; ++m)
        dp[m] = lane + 64 * m < 4 * P ? xget(G.Dv + (size_t)par * 4 * SYTRD_GRID_P + lane + 64 * m) : 0.0;
      ppk = xget(pp + k);
      double s = 0.0;
#pragma unroll
      for (int m = 0; m < SYTRD_GRID_P / 16; ++m) s += dp[m];
      hc = 0.5 * taup * wave_sum(s);
      const double wk0 = ppk - hc;  // v_{k-1} starts with 1
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        w[t] = lane + 64 * t >= k ? pv[t] - hc * v[t] : 0.0;
        x[t] = x[t] - w[t] - wk0 * v[t];
      }
    }
    double part = 0.0, al = 0.0;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int j = lane + 64 * t;
      lv[j] = v[t];
      lw[j] = w[t];
      if (j >= k + 2) part += x[t] * x[t];
      if (j == k + 1) al = x[t];
    }
    if (k == n - 2) break;
    const double sumsq = wave_sum(part), alpha = wave_sum(al);
    double tau, scal, beta;
    householder(alpha, sumsq, tau, scal, beta);
    double vn[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int j = lane + 64 * t;
      vn[t] = j > k + 1 ? x[t] * scal : j == k + 1 ? 1.0 : 0.0;
      ln[j] = vn[t];
    }
    wave_sync();
    // own rows: T_k = T_{k-1} - v w^T - w v^T, and p_k = tau T_k,22 v_k
    double acc[SYG_R], wpart = 0.0;
#pragma unroll
    for (int r = 0; r < SYG_R; ++r) {
      acc[r] = 0.0;
      const int i = b + P * (wave + SYTRD_GRID_T / 64 * r);
      if (i <= k || i >= n) continue;
      const double vi = lv[i], wi = lw[i];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (64 * t + 63 <= k) continue;
        a[r][t] = a[r][t] - vi * w[t] - wi * v[t];
        acc[r] += a[r][t] * vn[t];
      }
      if (i == k + 1) {
        double* rpub = G.Rp + (size_t)(k & 1) * N;
#pragma unroll
        for (int t = 0; t < NT; ++t)
          if (lane + 64 * t > k && lane + 64 * t < n) xput(rpub + lane + 64 * t, a[r][t]);
      }
    }
#pragma unroll
    for (int r = 0; r < SYG_R; ++r) acc[r] = wave_sum(acc[r]);
#pragma unroll
    for (int r = 0; r < SYG_R; ++r) {
      const int i = b + P * (wave + SYTRD_GRID_T / 64 * r);
      if (i <= k || i >= n) continue;
      const double pv = tau * acc[r];
      if (lane == 0) xput(G.Pv + (size_t)(k & 1) * N + i, pv);
      wpart += pv * ln[i];
    }
    if (lane == 0) xput(G.Dv + (size_t)(k & 1) * 4 * SYTRD_GRID_P + 4 * b + wave, wpart);
#pragma unroll
    for (int t = 0; t < NT; ++t) v[t] = vn[t];
    taup = tau;
    grid_barrier_relaxed(flags, ++ordinal, P, s_abort, dims);
    if (writer) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int j = lane + 64 * t;
        if (j == k) W.d[k] = x[t];
        if (j > k && j < n) W.H[(long long)k * N + j] = v[t];
      }
      if (lane == 0) {
        W.e[k] = beta;
        W.tau[k] = tau;
      }
    }
  }
  // the last 2 x 2 block of T_{n-2}, from its owners' rows of T_{n-3}
  wave_sync();
#pragma unroll
  for (int r = 0; r < SYG_R; ++r) {
    const int i = b + P * (wave + SYTRD_GRID_T / 64 * r);
    if (i < n - 2 || i >= n) continue;
    const double vi = lv[i], wi = lw[i];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int j = lane + 64 * t;
      const double y = a[r][t] - vi * w[t] - wi * v[t];
      if (j == i) W.d[i] = y;
      if (i == n - 2 && j == n - 1) {
        W.e[i] = y;
        W.tau[i] = 0.0;
      }
    }
  }
}

// Blocks of a live order n: 16 rows to a block, 4 to a wavefront.
__device__ __host__ inline int sytrd_grid_blocks(int n) {
  return n <= 256 ? 16 : n <= 512 ? 32 : SYTRD_GRID_P;
}
__device__ __host__ inline int sytrd_grid_chunks(int n) {
  return n <= 256 ? 4 : n <= 384 ? 6 : n <= 512 ? 8 : n <= 704 ? 11 : 16;
}
inline size_t sytrd_grid_lds(int N) {
  return (size_t)sytrd_grid_chunks(N) * 64 * 3 * (SYTRD_GRID_T / 64) * 8;
}
// Jobs of a launch.
constexpr int SYG_JOBS = 2;
static_assert(SYG_JOBS * (SYG_WIDE / 16) / 2 <= GRID_CUS && SYG_JOBS * SYTRD_GRID_P <= GRID_CUS_WIDE,
              "CUs of a launch");

// Jobs q0 and q0 + 1.  WIDE: capacities above SYG_WIDE.  Up to there 256 registers a
// lane do, and two blocks fit a CU.
template <bool WIDE>
__global__ __launch_bounds__(SYTRD_GRID_T) __attribute__((amdgpu_waves_per_eu(WIDE ? 1 : 2))) void k_sytrd_grid(
    EigJobs jobs, int q0, int* __restrict__ dims, int N) {
  extern __shared__ double lds[];
  __shared__ int s_abort;
  const EigJob J = jobs.j[q0 + blockIdx.y];
  const int n = dims[J.n_idx];
  if (n <= SYR_MAX) return;  // k_sytrd_reg (the same decision on all blocks of the job)
  const int P = sytrd_grid_blocks(n);
  if (blockIdx.x >= P) return;
  if (threadIdx.x == 0) s_abort = 0;
  __syncthreads();
  if (n <= 256) sytrd_grid_rows<4>(J, dims, N, n, P, lds, &s_abort);
  else if (n <= 384) sytrd_grid_rows<6>(J, dims, N, n, P, lds, &s_abort);
  else if (!WIDE || n <= 512) sytrd_grid_rows<8>(J, dims, N, n, P, lds, &s_abort);
  else if (n <= 704) sytrd_grid_rows<11>(J, dims, N, n, P, lds, &s_abort);
  else sytrd_grid_rows<16>(J, dims, N, n, P, lds, &s_abort);
}

// The same reduction with the matrix in registers (n <= SYR_MAX), one block
// per matrix: wavefront w holds the columns 16 w .. 16 w + 15, lane 16 g + c of
// it column j = 16 w + c and the rows i = g (mod 4), shifted: before step k,
// a[r] = A(4 (s + r) + g, j) with s = floor(k / 4), so rows k and k + 1 are always
// in a[0] or a[1] and no register is picked by a run-time index.  Row factors
// reach the multiply-adds without an LDS read or a move: a vector's entries
// are held one per lane, entry 4 (s + 16 m + c) + g in register m of lane
// 16 g + c, and v_fmac_f64 takes lane c of each row of 16 as its broadcast
// operand (row_newbcast), so one instruction is one row of every column.
// (The earlier form, each row over two lanes, read both vectors from LDS for
// every column it updated, and was bound by those reads: 160 broadcast pairs
// a lane and step.)  A Householder step k has two block barriers:
//   the lanes of rows k and k + 1 have published them in LDS (row k as x, zero
//   up to entry k + 1); (B1)
//   every wavefront sums x's norm and forms tau, beta, scal; y_j = sum_i
//   A(i, j) x_i over its columns, the four row groups added by row swaps; by
//   symmetry p_j = tau (A(k+1, j) + scal y_j) with v = [1, scal x];
//   p and each wavefront's share of p.v to LDS; (B2)
//   with K = tau p.v / 2 and u_i = p_i - 2 K v_i, A(i, j) -= v_i p_j + u_i v_j
//   (= v w^T + w v^T with w = p - K v), and the rows k + 1 and k + 2 are
//   published.
// Rows are taken in groups of 32 (8 registers); a group wholly past n, and a
// wavefront whose columns are all done, is skipped by a scalar branch.
// Entries past n are zero, and stay so.  The loop issues no global memory
// access: the reflectors and d, e, tau stay in LDS and are written out after
// it.  One matrix, before and now: order 62
// 86 -> 68 us, 142 303 -> 199 us, 160 350 -> 237 us, 192 (k_sytrd_grid before)
// 1013 -> 315 us.  (With wavefronts whose columns are done still forming the
// step's scalars, 142 took 229 us: three wavefronts then shared a SIMD.)
constexpr int SYR_WAVES = SYR_MAX / 16;
constexpr int SYR_T = 64 * SYR_WAVES;
constexpr int SYR_RC = SYR_MAX / 4;   // rows a lane holds
constexpr int SYR_PUB = SYR_MAX + 64; // entries of a published vector (read by whole wavefronts)
static_assert(SYR_MAX % 64 == 0, "row groups of 32, vector registers of 64");
// offset of v_k (n - 1 - k entries) in the packed reflector store
__device__ inline int refl_off(int k, int n) { return k * (n - 1) - k * (k - 1) / 2; }

// y[t % 4] += x(lane 8 H + t of the row of 16) a[t], t < 8.  The leading s_nop
// covers the two wait states between a vector write of x and its use as a
// DPP operand, which the compiler does not see inside the block.
#define TT_FMAC_BC(d, x, a, n) "v_fmac_f64_dpp " d ", " x ", " a " row_newbcast:" n " row_mask:0xf bank_mask:0xf\n\t"
template <int H>
__device__ __forceinline__ void fmac8_dot(double (&y)[4], double x, const double* a) {
  if (H == 0)
    asm("s_nop 1\n\t" TT_FMAC_BC("%0", "%4", "%5", "0") TT_FMAC_BC("%1", "%4", "%6", "1")
        TT_FMAC_BC("%2", "%4", "%7", "2") TT_FMAC_BC("%3", "%4", "%8", "3")
        TT_FMAC_BC("%0", "%4", "%9", "4") TT_FMAC_BC("%1", "%4", "%10", "5")
        TT_FMAC_BC("%2", "%4", "%11", "6") TT_FMAC_BC("%3", "%4", "%12", "7")
        : "+v"(y[0]), "+v"(y[1]), "+v"(y[2]), "+v"(y[3])
        : "v"(x), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]));
  else
    asm("s_nop 1\n\t" TT_FMAC_BC("%0", "%4", "%5", "8") TT_FMAC_BC("%1", "%4", "%6", "9")
        TT_FMAC_BC("%2", "%4", "%7", "10") TT_FMAC_BC("%3", "%4", "%8", "11")
        TT_FMAC_BC("%0", "%4", "%9", "12") TT_FMAC_BC("%1", "%4", "%10", "13")
        TT_FMAC_BC("%2", "%4", "%11", "14") TT_FMAC_BC("%3", "%4", "%12", "15")
        : "+v"(y[0]), "+v"(y[1]), "+v"(y[2]), "+v"(y[3])
        : "v"(x), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]));
}
// a[t] += x(lane 8 H + t) p + u(lane 8 H + t) q, t < 8.
template <int H>
__device__ __forceinline__ void fmac8_rank2(double* a, double x, double p, double u, double q) {
  if (H == 0)
    asm("s_nop 1\n\t" TT_FMAC_BC("%0", "%8", "%9", "0") TT_FMAC_BC("%1", "%8", "%9", "1")
        TT_FMAC_BC("%2", "%8", "%9", "2") TT_FMAC_BC("%3", "%8", "%9", "3")
        TT_FMAC_BC("%4", "%8", "%9", "4") TT_FMAC_BC("%5", "%8", "%9", "5")
        TT_FMAC_BC("%6", "%8", "%9", "6") TT_FMAC_BC("%7", "%8", "%9", "7")
        TT_FMAC_BC("%0", "%10", "%11", "0") TT_FMAC_BC("%1", "%10", "%11", "1")
        TT_FMAC_BC("%2", "%10", "%11", "2") TT_FMAC_BC("%3", "%10", "%11", "3")
        TT_FMAC_BC("%4", "%10", "%11", "4") TT_FMAC_BC("%5", "%10", "%11", "5")
        TT_FMAC_BC("%6", "%10", "%11", "6") TT_FMAC_BC("%7", "%10", "%11", "7")
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7])
        : "v"(x), "v"(p), "v"(u), "v"(q));
  else
    asm("s_nop 1\n\t" TT_FMAC_BC("%0", "%8", "%9", "8") TT_FMAC_BC("%1", "%8", "%9", "9")
        TT_FMAC_BC("%2", "%8", "%9", "10") TT_FMAC_BC("%3", "%8", "%9", "11")
        TT_FMAC_BC("%4", "%8", "%9", "12") TT_FMAC_BC("%5", "%8", "%9", "13")
        TT_FMAC_BC("%6", "%8", "%9", "14") TT_FMAC_BC("%7", "%8", "%9", "15")
        TT_FMAC_BC("%0", "%10", "%11", "8") TT_FMAC_BC("%1", "%10", "%11", "9")
        TT_FMAC_BC("%2", "%10", "%11", "10") TT_FMAC_BC("%3", "%10", "%11", "11")
        TT_FMAC_BC("%4", "%10", "%11", "12") TT_FMAC_BC("%5", "%10", "%11", "13")
        TT_FMAC_BC("%6", "%10", "%11", "14") TT_FMAC_BC("%7", "%10", "%11", "15")
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7])
        : "v"(x), "v"(p), "v"(u), "v"(q));
}
// Sum over the four rows of 16 lanes, lane by lane, the same bits on all four:
// the row swaps put two rows' (two pairs of rows') values side by side.
__device__ inline double rows_sum(double v) {
  unsigned long long b = (unsigned long long)__double_as_longlong(v);
  auto l = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
  auto h = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  v = __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
      __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
  b = (unsigned long long)__double_as_longlong(v);
  l = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
  h = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
         __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
}

// LDS of the register reduction: published row k (x), row k + 1, p; d, e, tau;
// the packed reflectors (v_k, rows k + 1 .. n - 1, from refl_off(k)).
struct SyrLds {
  double xs[SYR_PUB], as[SYR_PUB], ps[SYR_PUB];
  double red[SYR_WAVES];  // each wavefront's share of p.v (zero past the live ones)
  double sde[3][SYR_MAX];
  double al, dk;  // A(k, k + 1), A(k, k)
  double refl[SYR_MAX * (SYR_MAX - 1) / 2];
};

__global__ __launch_bounds__(SYR_T) void k_sytrd_reg(EigJobs jobs, int* __restrict__ dims, int N) {
  const EigJob J = jobs.j[blockIdx.x];
  const int n = dims[J.n_idx];
  grid_clear(grid_flags(J.work, N), threadIdx.x, SYR_T);
  if (n < 1 || n > SYR_MAX) return;  // k_sytrd_grid
  // the wavefront index is uniform: in a scalar register
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = (n + 15) >> 4;
  if (wave >= nw) return;  // before any barrier
  __shared__ __align__(16) SyrLds L;
  const double* A = J.A;
  const long long lda = J.lda;
  Work W = work_of(J, N);
  const int tid = threadIdx.x, l = tid & 63, g = l >> 4, c = l & 15, T = 64 * nw;
  const int j = 16 * wave + c;  // this lane's column
  double a[SYR_RC];
  // the lower triangle
#pragma unroll
  for (int r = 0; r < SYR_RC; ++r) {
    const int i = 4 * r + g;
    a[r] = i < n && j < n ? A[i >= j ? i * lda + j : j * lda + i] : 0.0;
  }
  for (int e = tid; e < 3 * SYR_PUB; e += T) L.xs[e] = 0.0;  // xs, as, ps
  if (tid < SYR_WAVES) L.red[tid] = 0.0;
  __syncthreads();
  // rows k (register r0 of the lanes g0) and k + 1 (r1, g1)
  auto publish = [&](int k, double x, int g0, double y, int g1) {
    if (g == g0 && j < n) {
      L.xs[j] = j >= k + 2 ? x : 0.0;
      if (j == k + 1) L.al = x;
      if (j == k) L.dk = x;
    }
    if (g == g1 && j < n) L.as[j] = y;
  };
  publish(0, a[0], 0, a[0], 1);
  // step k = 4 s + Q
  auto step = [&](const int k, auto qtag) {
    constexpr int Q = decltype(qtag)::value;
    const int s4 = k & ~3;
    lds_barrier();  // (B1)
    // a wavefront whose columns are all done only keeps the barriers' count
    const bool live = 16 * wave + 15 > k;
    if (!live) {
      if (g == 0) L.ps[j] = 0.0;
      if (l == 0) L.red[wave] = 0.0;
      lds_barrier();  // (B2)
      return;
    }
    const double alpha = L.al, dkk = L.dk;
    double xm[3], y[4] = {0.0, 0.0, 0.0, 0.0}, part = 0.0;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      xm[m] = s4 + 64 * m < n ? L.xs[s4 + 64 * m + 4 * c + g] : 0.0;
      part = fma(xm[m], xm[m], part);
    }
    const double xj = L.xs[j], aj = L.as[j];
#pragma unroll
    for (int q = 0; q < SYR_RC / 8; ++q) {
      if (s4 + 32 * q >= n) continue;
      if (q & 1) fmac8_dot<1>(y, xm[q / 2], a + 8 * q);
      else fmac8_dot<0>(y, xm[q / 2], a + 8 * q);
    }
    const double sumsq = wave_sum(part);
    double tau, scal, beta;
    householder(alpha, sumsq, tau, scal, beta);
    const double yj = rows_sum((y[0] + y[1]) + (y[2] + y[3]));
    const double vj = j == k + 1 ? 1.0 : scal * xj;
    const double pj = j > k ? tau * fma(scal, yj, aj) : 0.0;
    if (g == 0) {
      if (j < n) {
        L.ps[j] = pj;
        if (j > k) L.refl[refl_off(k, n) + j - k - 1] = vj;
      }
    }
    // the four row groups hold the same p_j v_j: a sum over one row of lanes
    double kp = pj * vj;
    kp += dpp_d<0xB1>(kp);
    kp += dpp_d<0x4E>(kp);
    kp += dpp_d<0x141>(kp);
    kp += dpp_d<0x140>(kp);
    if (l == 0) {
      L.red[wave] = kp;
      if (wave == nw - 1) {  // live to the end
        L.sde[0][k] = dkk;
        L.sde[1][k] = beta;
        L.sde[2][k] = tau;
      }
    }
    lds_barrier();  // (B2)
    {
      double kd[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int w = 0; w < SYR_WAVES; ++w) kd[w & 3] += L.red[w];
      const double K2 = tau * ((kd[0] + kd[1]) + (kd[2] + kd[3]));  // 2 K
      double nv[3], nu[3];
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        const int i = s4 + 64 * m + 4 * c + g;
        const double pm = s4 + 64 * m < n ? L.ps[i] : 0.0;
        const double vm = i == k + 1 ? 1.0 : scal * xm[m];
        nv[m] = -vm;
        nu[m] = fma(K2, vm, -pm);
      }
#pragma unroll
      for (int q = 0; q < SYR_RC / 8; ++q) {
        if (s4 + 32 * q >= n) continue;
        if (q & 1) fmac8_rank2<1>(a + 8 * q, nv[q / 2], pj, nu[q / 2], vj);
        else fmac8_rank2<0>(a + 8 * q, nv[q / 2], pj, nu[q / 2], vj);
      }
    }
    if (Q == 3) {  // the next step's rows start four further on
#pragma unroll
      for (int r = 0; r + 1 < SYR_RC; ++r) a[r] = a[r + 1];
      a[SYR_RC - 1] = 0.0;
    }
    publish(k + 1, a[0], (Q + 1) & 3, Q == 2 ? a[1] : a[0], (Q + 2) & 3);
  };
  for (int k = 0; k + 2 < n; k += 4) {
    step(k, std::integral_constant<int, 0>());
    if (k + 3 < n) step(k + 1, std::integral_constant<int, 1>());
    if (k + 4 < n) step(k + 2, std::integral_constant<int, 2>());
    if (k + 5 < n) step(k + 3, std::integral_constant<int, 3>());
  }
  // the last published rows hold the last 2 x 2 block (n = 1: row 0 alone)
  __syncthreads();
  if (tid == 0) {
    if (n >= 2) {
      W.d[n - 2] = L.dk;
      W.e[n - 2] = L.al;
      W.tau[n - 2] = 0.0;
      W.d[n - 1] = L.as[n - 1];
    } else {
      W.d[0] = L.dk;
    }
  }
  for (int k = tid; k + 2 < n; k += T) {
    W.d[k] = L.sde[0][k];
    W.e[k] = L.sde[1][k];
    W.tau[k] = L.sde[2][k];
  }
  for (int k = wave; k + 2 < n; k += nw) {
    const int off = refl_off(k, n);
    for (int i = k + 1 + l; i < n; i += 64) W.H[(long long)k * N + i] = L.refl[off + i - k - 1];
  }
}

// ---------------------------------------------------------------------------
// 2. Tridiagonal eigenproblem by divide and conquer (Cuppen), bottom-up from
// leaves of 8 rows.  T is torn at every off-diagonal e_m into blocks coupled by
// rank-one terms |e_m| w w^T, w = e_m + sign(e_m) e_{m+1}; each merge of two
// solved halves solves  D + rho z z^T  (z = last row of Q_left, sign-scaled
// first row of Q_right).  Deflation removes tiny z_j and near-equal d_j
// (Givens); the remaining roots come from the secular equation
//   1 + rho sum_j z_j^2 / (d_j - lambda) = 0,
// solved in the shifted variable lambda = d_origin + tau; the eigenvectors
// use the Loewner-recomputed z^ so that they are orthogonal to working
// accuracy.  Vector updates Q <- Q_rot U are tiled products (dc_subtree, dc_update_tile).
struct DC {
  double *lam, *Qa, *Qb, *dsl, *dro, *rc, *rs, *rtau, *zhat, *dK, *zK, *mrho;
  int *perm, *Kslot, *rp, *rq, *mk, *mnrot, *mm2;
};
__device__ inline DC dc_of(const Work& W, int N) {
  const int N2 = next_pow2(N);
  DC D;
  double* p = W.Z;
  D.lam = p; p += N2;
  D.Qa = p; p += (size_t)N2 * N2;
  D.Qb = p; p += (size_t)N2 * N2;
  double** dv[] = {&D.dsl, &D.dro, &D.rc, &D.rs, &D.rtau, &D.zhat, &D.dK, &D.zK, &D.mrho};
  for (double** q : dv) { *q = p; p += N2; }
  int** iv[] = {&D.perm, &D.Kslot, &D.rp, &D.rq, &D.mk, &D.mnrot, &D.mm2};
  for (int** q : iv) { *q = reinterpret_cast<int*>(p); p += N2; }
  return D;
}

// Leaves of DC_LEAF rows, solved directly: leaf r holds rows
// [DC_LEAF r, DC_LEAF (r + 1)) of
// T torn only at its two boundary off-diagonals (its diagonal loses |e| at a
// torn boundary; inside the leaf T keeps its off-diagonals).  One wavefront
// runs the implicit QL iteration with Wilkinson's shift on a leaf, in
// registers with compile-time indexes: every lane carries the same d and e
// (scaled by a power of two to a largest entry near 1), lane i row i of the
// vectors.  A found eigenvalue goes to LDS with its vector and the arrays
// shift down by one, so one copy of the iteration's code serves all eight.
// An off-diagonal is dropped at u / 8 of the leaf's Frobenius norm (the
// merges above deflate at 8 u ||T|| anyway) or at u of its diagonal neighbours.
// The eigenvalues are sorted ascending with their vectors, and written where
// the merges up to blocks of 8 would have left them: lam[leaf] and the
// diagonal block of Q.
// Bound by the instructions of the rotations (some 90 a leaf at 8 rows, one
// reciprocal root and about 45 instructions each, which a lone wavefront
// issues every 7 cycles): 15 us at order 16, 26 at 62, with the first loads.
// Cyclic Jacobi through LDS, a lane per entry, took 8 us more at order 16 and 25 at 62.

// The implicit QL iteration on a leaf's d, e, v (rows past nb are decoupled
// zeros; an off-diagonal at or below `tiny` is dropped): emit(l, eigenvalue,
// this lane's entry of its vector) for l < nb.  Returns whether every
// eigenvalue split off within LEAF_MAXIT iterations (it takes two or three).
constexpr int DC_LEAF = 8;
constexpr int LEAF_MAXIT = 40;
template <typename Emit>
__device__ __forceinline__ bool leaf_ql(double (&d)[DC_LEAF], double (&e)[DC_LEAF], double (&v)[DC_LEAF], int nb,
                                        double tiny, Emit emit) {
  bool conv = true;
  for (int l = 0; l < nb; ++l) {
    int it = 0;
    for (; it < LEAF_MAXIT; ++it) {
      // the unreduced block that starts at 0 ends at row m; dm = d[m]
      int m = 0;
      double dm = d[0];
      bool open = true;
#pragma unroll
      for (int k = 0; k < DC_LEAF - 1; ++k) {
        const double ae = fabs(e[k]);
        const bool drop = ae <= tiny || ae <= U64 * (fabs(d[k]) + fabs(d[k + 1]));
        e[k] = open && drop ? 0.0 : e[k];
        open = open && !drop;
        m = open ? k + 1 : m;
        dm = open ? d[k + 1] : dm;
      }
      m = __builtin_amdgcn_readfirstlane(m);  // the same on every lane
      if (m == 0) break;
      // shift: the eigenvalue of the leading 2 x 2 nearer d[0]
      const double del = d[1] - d[0], two = 2.0 * e[0];
      const double hyp = sqrt(del * del + two * two);
      double g = dm - d[0] + e[0] * two / (del + copysign(hyp, del));
      double c = 1.0, s = 1.0, p = 0.0;
#pragma unroll
      for (int i = DC_LEAF - 2; i >= 0; --i) {
        if (i < m) {
          const double f = s * e[i], b = c * e[i];
          const double h = f * f + g * g;
          const double rh = h > 1e-280 ? rsqrt_d(h) : 0.0;
          if (i + 1 < m) e[i + 1] = h * rh;
          s = f * rh;
          c = rh > 0.0 ? g * rh : 1.0;
          const double dn = d[i + 1] - p;
          const double w = (d[i] - dn) * s + 2.0 * c * b;
          p = s * w;
          d[i + 1] = dn + p;
          g = c * w - b;
          const double x = v[i + 1], y = v[i];
          v[i + 1] = s * y + c * x;
          v[i] = c * y - s * x;
        }
      }
      d[0] -= p;
      e[0] = g;
    }
    conv = conv && it < LEAF_MAXIT;
    emit(l, d[0], v[0]);
#pragma unroll
    for (int k = 0; k + 1 < DC_LEAF; ++k) {
      d[k] = d[k + 1];
      e[k] = e[k + 1];
      v[k] = v[k + 1];
    }
    d[DC_LEAF - 1] = 0.0;
    e[DC_LEAF - 1] = 0.0;
    v[DC_LEAF - 1] = 0.0;
  }
  return conv;
}

struct LeafLds {
  double lam[DC_LEAF], V[DC_LEAF][DC_LEAF + 1];
};

// Leaf `leaf` of job J, by the calling wavefront (lane = threadIdx.x % 64), its
// eigenvalues to lam[0 .. 7].
__device__ void dc_leaf_wave(const EigJob& J, int* __restrict__ dims, int N, int leaf,
                             double* lam, LeafLds& L) {
  const int n = max(0, dims[J.n_idx]);
  Work W = work_of(J, N);
  DC D = dc_of(W, N);
  const int N2 = next_pow2(N);
  const int r0 = leaf * DC_LEAF;
  if (r0 >= n) return;
  const int nb = min(DC_LEAF, n - r0);
  const int lane = threadIdx.x & 63, row = lane & (DC_LEAF - 1);
  // e[k]: off-diagonal (k, k + 1); rows past nb are decoupled zeros
  double d[DC_LEAF], e[DC_LEAF], v[DC_LEAF];
#pragma unroll
  for (int k = 0; k < DC_LEAF; ++k) {
    d[k] = k < nb ? W.d[r0 + k] : 0.0;
    e[k] = k < nb && r0 + k + 1 < n ? W.e[r0 + k] : 0.0;
    v[k] = k == row ? 1.0 : 0.0;
  }
  if (r0 > 0) d[0] -= fabs(W.e[r0 - 1]);
#pragma unroll
  for (int k = 0; k < DC_LEAF; ++k)
    if (k == nb - 1) {
      d[k] -= fabs(e[k]);
      e[k] = 0.0;
    }
  double big = 0.0;
#pragma unroll
  for (int k = 0; k < DC_LEAF; ++k) big = fmax(big, fmax(fabs(d[k]), fabs(e[k])));
  const int ex = big > 0.0 && big <= DBL_MAX ? ilogb(big) : 0;
  double fro = 0.0;
#pragma unroll
  for (int k = 0; k < DC_LEAF; ++k) {
    d[k] = ldexp(d[k], -ex);
    e[k] = ldexp(e[k], -ex);
    fro += d[k] * d[k] + 2.0 * e[k] * e[k];
  }
  // a leaf with a NaN is flagged and solved as a zero one, so that the places
  // below stay a permutation (numbers give numbers)
  const bool nan = !(fro == fro);
#pragma unroll
  for (int k = 0; k < DC_LEAF; ++k) {
    d[k] = nan ? 0.0 : d[k];
    e[k] = nan ? 0.0 : e[k];
  }
  const bool conv = leaf_ql(d, e, v, nb, 0.125 * U64 * sqrt(nan ? 0.0 : fro), [&](int l, double x, double y) {
    if (lane == 0) L.lam[l] = x;
    if (lane < DC_LEAF) L.V[lane][l] = y;
  });
  wave_sync();
  // ascending (stable: the index breaks ties), an entry a lane
  const int i = lane / DC_LEAF, k = lane % DC_LEAF;
  if (k < nb) {
    const double x = L.lam[k];
    int pos = 0;
    for (int j = 0; j < nb; ++j) pos += L.lam[j] < x || (L.lam[j] == x && j < k);
    if (i < nb) D.Qa[(size_t)(r0 + i) * N2 + r0 + pos] = L.V[i][k];
    if (i == 0) lam[pos] = ldexp(x, ex);
  }
  if ((nan || !conv) && lane == 0) atomicOr(&dims[D_FLAG], FLAG_EIG);
}

// Dynamic LDS of the phases above the one-block merges, per merge element: the sort and
// deflation (4 doubles, 3 ints); the tiles with the permutation and the
// rotations staged, up to VEC_STAGE_MAX rows (7 doubles, 6 ints), or not (5
// doubles, 3 ints), beside their panel.
constexpr int PREP_BYTES_PER = 4 * 8 + 3 * 4;
constexpr int VEC_STAGE_MAX = 1024;
constexpr int VEC_BYTES_STAGED = 7 * 8 + 6 * 4;
constexpr int VEC_BYTES_GLOBAL = 5 * 8 + 3 * 4;

// Sums and products over groups of L lanes (64: the wavefront; 8: aligned
// groups, which may be active by themselves), the result on every lane.
template <int L>
__device__ inline double grp_sum(double v) {
  if (L == 64) return wave_sum(v);
  v += dpp_d<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_d<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_d<0x141>(v);  // row_half_mirror
  if (L == 16) v += dpp_d<0x140>(v);  // row_mirror
  return v;
}
template <int L>
__device__ inline double grp_prod(double v) {
  v *= dpp_d<0xB1>(v);
  v *= dpp_d<0x4E>(v);
  v *= dpp_d<0x141>(v);
  if (L == 64) {
    v *= dpp_d<0x140>(v);
    v = (lane_d(v, 0) * lane_d(v, 16)) * (lane_d(v, 32) * lane_d(v, 48));
  }
  return v;
}

// The tridiagonal solver's blocks: DC_T threads; the lowest DC_SUB rows' merges stay
// on one block; above, a merge's products are taken in tiles of DC_RT rows by
// DC_CT columns, the update matrix in panels of DC_KC rows.
constexpr int DC_T = 512;
constexpr int DC_SUB = 64;
constexpr int DC_RT = 64;
constexpr int DC_CT = 32;
constexpr int DC_PLD = DC_CT + 4;  // panel stride: k rows 4 apart fall on other banks
constexpr int DC_ZSPLIT = 256;     // S from which z^ is a phase of its own
template <bool STAGE> constexpr int dc_kc() { return STAGE ? 256 : 128; }

// One root of the secular equation f(tau) = 1 + rho sum_j z_j^2 / (delta_j - tau)
// (delta_j = d_j - d_o, o the nearer end of the root's interval), by a group
// of L lanes (`lane` within it), d and z in LDS.  f is increasing between the
// poles delta_i < tau < delta_{i+1}; the root is kept in a bracket [lo, hi]
// with f(lo) < 0 < f(hi).  Each iteration replaces the terms up to pole
// `split`, psi, and those after it, phi, each by a / (delta - t) + b matching
// value and slope at the current iterate at their nearest pole (the two-pole
// rational model of Bunch, Nielsen and Sorensen, 1978); the model's root in
// the bracket is the next iterate (bisection when it falls outside, or is not a
// number: the model's divisions and root take the fast forms).  The
// first iterate is the interval's middle, whose sign picks the origin, and
// its model keeps the exact weights of both neighbours.  When an iteration
// leaves f's sign unchanged and reduces |f| by less than 10x, the next step
// swaps to the fixed-weight model (exact weight on the origin pole, fitted weight on the
// other neighbour), and back, as LAPACK's dlaed4 does between its middle-way
// and fixed-weight steps (Li, 1993).  Stops when |f| is at the level of its
// evaluation error, 8u (1 + rho sum |terms|), or at a relative change of 2u.
// Bound by the chain of an iteration (pole sums, their reduction, the model's
// square root and division, some 700 cycles), so the number of iterations
// counts: starting from the middle's exact-weight model takes about 4
// evaluations, where both bracket ends were evaluated first and the first
// iterate was their geometric mean it took 8.
constexpr int ROOT_MAXIT = 100;
template <int L>
__device__ inline void dc_root(const double* d, const double* z, int nk, int i, double rho,
                               int lane, double& tau_out, double& dor_out, bool& ok) {
  if (nk == 1) {
    tau_out = rho * z[0] * z[0];
    dor_out = d[0];
    ok = tau_out == tau_out && tau_out != 0.0;
    return;
  }
  const bool inner = i < nk - 1;
  const int split = inner ? i : nk - 2;
  const double ds = d[split], dn = d[split + 1];
  const double ws = rho * z[split] * z[split], wn = rho * z[split + 1] * z[split + 1];
  const double gap = dn - ds;
  bool right = !inner;  // the origin is pole split + 1
  double dor = right ? dn : ds;
  double lo, hi, x;
  if (inner) {
    x = 0.5 * gap;
    lo = 0.0;
    hi = x;
  } else {
    // all other terms are negative, so tau* >= rho z_o^2
    lo = 0.5 * wn;
    hi = rho;
    x = 0.5 * rho;
  }
  double pl = ds - dor, pr = dn - dor;
  double tau = 0.0, fprev = 0.0;
  bool fw = false;
  int it = 0;
  for (; it < ROOT_MAXIT; ++it) {
    // psi, psi', phi, phi' at x
    double ps = 0.0, dps = 0.0, ph = 0.0, dph = 0.0;
    for (int j = lane; j < nk; j += L) {
      const double r = rcp_d((d[j] - dor) - x);
      const double zj = z[j];
      const double t = zj * zj * r;
      if (j <= split) {
        ps += t;
        dps = fma(t, r, dps);
      } else {
        ph += t;
        dph = fma(t, r, dph);
      }
    }
    ps = grp_sum<L>(ps);
    dps = grp_sum<L>(dps);
    ph = grp_sum<L>(ph);
    dph = grp_sum<L>(dph);
    const double f = 1.0 + rho * (ps + ph);
    if (it == 0 && inner) {
      // Safe brackets from the secular function itself: for the root on the
      // origin's right, f(tau) <= 1 + 2 rho / gap - rho z_o^2 / tau, so
      // tau* >= rho z_o^2 / (1 + 2 rho / gap); symmetrically on the left.
      if (f >= 0.0) {
        hi = x;
        lo = 0.5 * ws / (1.0 + 2.0 * rho / gap);
      } else {
        right = true;
        dor = dn;
        pl = ds - dor;
        pr = 0.0;
        x = -(gap - x);
        lo = x;
        hi = -0.5 * wn / fmax(1.0, 2.0 * rho / gap);
      }
      // an end that underflowed to zero would sit on the origin's pole
      if (lo == 0.0) lo = hi * 0x1p-60;
      if (hi == 0.0) hi = lo * 0x1p-60;
    }
    // converged once f is at the level of its own rounding error
    if (f == 0.0 || fabs(f) <= 8.0 * U64 * (1.0 + rho * (fabs(ph) + fabs(ps)))) { tau = x; break; }
    if (it > 0 || !inner) {
      if (f < 0.0) lo = x;
      else hi = x;
    }
    if (hi - lo <= 4.0 * U64 * fmax(fabs(lo), fabs(hi))) { tau = 0.5 * (lo + hi); break; }
    // when f keeps its sign and falls by less than a factor of 10, the
    // other model takes the next step
    if (it > 0 && inner && f * fprev > 0.0 && fabs(f) > 0.1 * fabs(fprev)) fw = !fw;
    fprev = f;
    // model: a0 + al / (pl - t) + ga / (pr - t) = 0
    const double el = pl - x, er = pr - x;
    double al, ga, a0;
    if (it == 0) {
      al = ws;
      ga = wn;
      a0 = f - al * rcp_d(el) - ga * rcp_d(er);
    } else if (fw) {
      // fixed weight: the origin pole keeps its exact weight rho z_o^2; the
      // other neighbouring pole's weight and the constant match f and f'
      // at x.  It converges where the two-pole fit does not: a root next to
      // a pole of tiny weight, beside a heavy pole one step away.
      const double fp = rho * (dps + dph);
      const double eo = right ? er : el, eq = right ? el : er;
      const double wo = right ? wn : ws;
      const double ro = rcp_d(eo), wq = (fp - wo * ro * ro) * eq * eq;
      a0 = f - wo * ro - wq * rcp_d(eq);
      al = right ? wq : wo;
      ga = right ? wo : wq;
    } else {
      al = rho * dps * el * el;
      ga = rho * dph * er * er;
      a0 = 1.0 + rho * (ps - dps * el) + rho * (ph - dph * er);
    }
    // a0 t^2 - b t + c = 0
    const double b = a0 * (pl + pr) + al + ga;
    const double c = a0 * pl * pr + al * pr + ga * pl;
    const double disc = b * b - 4.0 * a0 * c;
    double xn = NAN;
    if (disc >= 0.0) {
      const double sq = disc > 0.0 ? disc * rsqrt_d(disc) : 0.0;
      const double qq = b >= 0.0 ? b + sq : b - sq;  // no cancellation
      const double r1 = 2.0 * c * rcp_d(qq);
      if (r1 > lo && r1 < hi) {
        xn = r1;
      } else {
        const double r2 = qq * rcp_d(2.0 * a0);
        if (r2 > lo && r2 < hi) xn = r2;
      }
    }
    if (!(xn > lo && xn < hi)) {
      xn = (lo > 0.0 && hi > 4.0 * lo) ? sqrt(lo) * sqrt(hi)
         : (hi < 0.0 && lo < 4.0 * hi) ? -sqrt(-lo) * sqrt(-hi) : 0.5 * (lo + hi);
      if (!(xn > lo && xn < hi)) { tau = 0.5 * (lo + hi); break; }
    }
    if (fabs(xn - x) <= 2.0 * U64 * fabs(xn)) { tau = xn; break; }
    x = xn;
    tau = x;
  }
  ok = tau == tau && tau != 0.0;
  if (!ok) tau = right ? lo : hi;
  ok = ok && it < ROOT_MAXIT;
  tau_out = tau;
  dor_out = dor;
}

// Loewner weight z^_j over a group of L lanes: the product over the roots of
// (d_j - lambda_i) / (d_j - d_i), so that the vectors formed with it are
// orthogonal to working accuracy whatever the roots' own errors.
template <int L>
__device__ inline double dc_zhat(const double* d, const double* dro, const double* rt, double zj,
                                 int nk, int j, double rho, int lane) {
  const double dj = d[j];
  double prod = 1.0;
  for (int i = lane; i < nk; i += L) {
    const double num = (dj - dro[i]) - rt[i];
    prod *= i != j ? num * rcp_d(dj - d[i]) : -num / rho;
  }
  return copysign(sqrt(fmax(grp_prod<L>(prod), 0.0)), zj);
}

// The deflating rotation of kept entries p < q, if they are near enough: |t c s|
// <= tol with c = z_q / r, s = z_p / r, r^2 = z_p^2 + z_q^2, tested without a square root
// or a division (the z are normalised and above tol / rho, so r^2 neither
// overflows nor underflows).
__device__ inline bool dc_near(double dp, double zp, double dq, double zq, double tol) {
  return fabs((dq - dp) * zq * zp) <= tol * (zp * zp + zq * zq);
}

// The U entry (before any rotation) of the column of root (di, ti) at pole j.
__device__ inline double dc_uent(double zh, double dj, double di, double ti, double inv) {
  return zh * rcp_d((dj - di) - ti) * inv;
}

// The rotations of one column of the update matrix W, by one thread.
// Rotation t acts on slots p_t < q_t, the q_t strictly increase with t and
// p_t >= q_{t-1} (the deflation carries its last kept slot along).  Applied
// last first, rotation t therefore meets slot p_t untouched (its U entry),
// and slot q_t untouched or as the output of rotation t + 1 on its p side,
// carried in a register; q_t is final after rotation t, and the carried slot
// is final once the next rotation does not take it.  u0(s): the U entry at
// slot s; put(s, v): the final value.
template <typename U0, typename Put>
__device__ inline void dc_rotate_column(int nrot, const int* rp, const int* rq, const double* rc,
                                        const double* rs, U0 u0, Put put) {
  int crow = -1;
  double cval = 0.0;
  for (int t = nrot - 1; t >= 0; --t) {
    const int p = rp[t], q = rq[t];
    const double c = rc[t], sn = rs[t];
    double xq;
    if (q == crow) {
      xq = cval;
    } else {
      if (crow >= 0) put(crow, cval);
      xq = u0(q);
    }
    const double xp = u0(p);
    put(q, c * xq - sn * xp);
    crow = p;
    cval = c * xp + sn * xq;
  }
  if (crow >= 0) put(crow, cval);
}

// LDS of the merges on one block: arrays of the block's DC_SUB rows, a merge's
// entries at its own rows; the update matrices of a level side by side.
struct SubLds {
  double lam[DC_SUB], dt[DC_SUB], d[DC_SUB], z[DC_SUB], rt[DC_SUB], dro[DC_SUB], ds[DC_SUB],
      zs[DC_SUB], rc[DC_SUB], rs[DC_SUB], rho[DC_SUB / DC_LEAF];
  double panel[DC_SUB * (DC_SUB + 4)];
  int perm[DC_SUB], ks[DC_SUB], kix[DC_SUB], tag[DC_SUB], rp[DC_SUB], rq[DC_SUB];
  int nk[DC_SUB / DC_LEAF], nrot[DC_SUB / DC_LEAF];
};

// Sort and deflation of a merge of up to 64 entries by one wavefront, a lane per
// entry (off: the merge's first row in the block's arrays).  The halves are
// merged by ranks (each element's rank in the other half by binary search;
// ties put the left element first).  Entries with tiny z deflate; then every
// neighbouring pair of kept ones is tested at once, and only where a pair
// is near does the sweep that carries the last kept entry along run.
__device__ inline void dc_sub_prep(SubLds& L, const double* Qs, int N2, int S, int b0, int off,
                                   int tm, int m2, double beta, int lane) {
  const double sgn = beta < 0.0 ? -1.0 : 1.0;
  const int c = lane;
  double zq = 0.0, dv = 0.0;
  if (c < m2) {
    zq = c < S ? Qs[(size_t)(b0 + S - 1) * N2 + b0 + c] : sgn * Qs[(size_t)(b0 + S) * N2 + b0 + c];
    dv = L.lam[off + c];
    L.dt[off + c] = dv;
    L.tag[off + c] = -1;
  }
  const double nz2 = wave_sum(zq * zq);
  double dmax = fabs(dv);
  for (int o = 32; o > 0; o >>= 1) dmax = fmax(dmax, __shfl_xor(dmax, o));
  const double nz = sqrt(nz2);
  const double rho = fabs(beta) * nz2;
  const double tol = 8.0 * U64 * fmax(dmax, rho);
  wave_sync();
  if (c < m2) {
    const bool left = c < S;
    const double* other = L.dt + off + (left ? S : 0);
    int lo = 0, hi = left ? m2 - S : S;
    while (lo < hi) {  // entries of the other half before this one
      const int mid = (lo + hi) >> 1;
      const double y = other[mid];
      if (left ? y < dv : y <= dv) lo = mid + 1;
      else hi = mid;
    }
    const int pos = (left ? c : c - S) + lo;
    L.perm[off + pos] = c;
    L.ds[off + pos] = dv;
    L.zs[off + pos] = nz > 0.0 ? zq / nz : 0.0;  // rows of orthogonal blocks: nz^2 = 2
  }
  wave_sync();
  double* ds = L.ds + off;
  double* zs = L.zs + off;
  const double dc = c < m2 ? ds[c] : 0.0, zc = c < m2 ? zs[c] : 0.0;
  const unsigned long long below = (1ULL << c) - 1ULL;
  unsigned long long km = __ballot(c < m2 && !(rho * fabs(zc) <= tol));
  const bool kept = (km >> c) & 1ULL;
  bool near = false;
  if (kept && (km & below)) {
    const int p = 63 - __builtin_clzll(km & below);
    near = dc_near(ds[p], zs[p], dc, zc, tol);
  }
  unsigned long long todo = __ballot(near);
  int nrot = 0;
  while (todo) {
    int q = __builtin_ctzll(todo);
    int p = 63 - __builtin_clzll(km & ((1ULL << q) - 1ULL));
    double dp = ds[p], zp = zs[p];
    bool more = true;
    while (more) {
      const double dq = ds[q], zz = zs[q];
      if (!dc_near(dp, zp, dq, zz, tol)) break;
      const double r = sqrt(zp * zp + zz * zz);
      const double ir = 1.0 / r;
      const double cs = zz * ir, sn = zp * ir;
      const double dqn = sn * sn * dp + cs * cs * dq;
      if (lane == 0) {
        L.rp[off + nrot] = p;
        L.rq[off + nrot] = q;
        L.rc[off + nrot] = cs;
        L.rs[off + nrot] = sn;
        ds[p] = cs * cs * dp + sn * sn * dq;
        zs[p] = 0.0;
        ds[q] = dqn;
        zs[q] = r;
      }
      ++nrot;
      km &= ~(1ULL << p);
      dp = dqn;
      zp = r;
      p = q;
      const unsigned long long above = q < 63 ? km & ~((2ULL << q) - 1ULL) : 0ULL;
      more = above != 0ULL;
      if (more) q = __builtin_ctzll(above);
    }
    todo &= q < 63 ? ~((2ULL << q) - 1ULL) : 0ULL;
  }
  wave_sync();
  if (c < m2) {
    const int k = __popcll(km & below);
    const bool keep = (km >> c) & 1ULL;
    if (keep) {
      L.d[off + k] = ds[c];
      L.z[off + k] = zs[c];
      L.ks[off + k] = c;
    }
    L.kix[off + c] = keep ? k + 1 : 0;
  }
  if (lane == 0) {
    L.nk[tm] = __popcll(km);
    L.nrot[tm] = nrot;
    L.rho[tm] = rho;
  }
}

// The leaves and the merges S = 8, 16, 32 of rows [DC_SUB sub, DC_SUB (sub + 1)) of
// job J, all on the calling block: no grid barrier until blocks of 64 are
// solved.  At level S a merge has 16 S threads, 8 lanes to a root, a pole
// weight or a column, so every phase of every level is one round over the
// block; eigenvalues and the merges' arrays stay in LDS, eigenvectors go
// through L2.  An eigensolve of order 62 fell from 286 to 223 us with it.
__device__ void dc_subtree(const EigJob& J, int* __restrict__ dims, int N, int sub, SubLds& L) {
  const int n = dims[J.n_idx];
  Work W = work_of(J, N);
  DC D = dc_of(W, N);
  const int N2 = next_pow2(N);
  const int base = sub * DC_SUB;
  const int tid = threadIdx.x, lane = tid & 63, l8 = tid & 7;
  bool bad = false;
  // a place that no entry takes (halves that a flagged merge left out of order)
  // still names a row of the block
  if (tid < DC_SUB) L.perm[tid] = 0;
  dc_leaf_wave(J, dims, N, sub * (DC_SUB / DC_LEAF) + (tid >> 6), L.lam + DC_LEAF * (tid >> 6),
               reinterpret_cast<LeafLds*>(L.panel)[tid >> 6]);
  __syncthreads();
  int par = 0;
  for (int S = DC_LEAF; S < DC_SUB && S < n; S *= 2, par ^= 1) {
    const double* Qs = par ? D.Qb : D.Qa;
    double* Qd = par ? D.Qa : D.Qb;
    const int w = 2 * S, T = 16 * S;
    const int tm = tid / T, tt = tid - tm * T, g = tt >> 3;
    const int off = tm * w, b0 = base + off;
    const int m2 = max(0, min(w, n - b0));
    const bool has = b0 + S < n;
    const int ld = w + 4;
    double* panel = L.panel + tm * w * ld;
    if (has && tt < 64) dc_sub_prep(L, Qs, N2, S, b0, off, tm, m2, W.e[b0 + S - 1], lane);
    __syncthreads();
    const int nk = has ? L.nk[tm] : 0, nrot = has ? L.nrot[tm] : 0;
    const double rho = has ? L.rho[tm] : 0.0;
    const double *d = L.d + off, *ds = L.ds + off;
    double *z = L.z + off, *rt = L.rt + off, *dro = L.dro + off;
    if (g < nk) {
      double tau, dor;
      bool ok;
      dc_root<8>(d, z, nk, g, rho, l8, tau, dor, ok);
      bad = bad || !ok;
      if (l8 == 0) {
        rt[g] = tau;
        dro[g] = dor;
      }
    }
    __syncthreads();
    // sorted places of the roots (ascending already) and the deflated slots
    // (by value, then slot; a root before an equal slot), the pole weights
    // (in place: group j reads and writes its own z), and a clear panel
    if (g < nk) {
      const double v = dro[g] + rt[g];
      int cnt = 0;
      for (int c = l8; c < m2; c += 8) cnt += L.kix[off + c] == 0 && ds[c] < v;
      cnt += __builtin_amdgcn_mov_dpp(cnt, 0xB1, 0xf, 0xf, true);
      cnt += __builtin_amdgcn_mov_dpp(cnt, 0x4E, 0xf, 0xf, true);
      cnt += __builtin_amdgcn_mov_dpp(cnt, 0x141, 0xf, 0xf, true);
      bad = bad || !(v == v);
      const double zh = dc_zhat<8>(d, dro, rt, z[g], nk, g, rho, l8);
      if (l8 == 0) {
        L.tag[off + g + cnt] = g;
        L.lam[off + g + cnt] = v == v ? v : DBL_MAX;
        z[g] = zh;
      }
    }
    if (has && g < m2 && L.kix[off + g] == 0) {
      const double v = ds[g];
      int cnt = 0;
      for (int c = l8; c < m2; c += 8) {
        if (L.kix[off + c] == 0) cnt += ds[c] < v || (ds[c] == v && c < g);
        if (c < nk) cnt += dro[c] + rt[c] <= v;
      }
      cnt += __builtin_amdgcn_mov_dpp(cnt, 0xB1, 0xf, 0xf, true);
      cnt += __builtin_amdgcn_mov_dpp(cnt, 0x4E, 0xf, 0xf, true);
      cnt += __builtin_amdgcn_mov_dpp(cnt, 0x141, 0xf, 0xf, true);
      bad = bad || !(v == v);
      if (l8 == 0) {
        L.tag[off + cnt] = w + g;
        L.lam[off + cnt] = v == v ? v : DBL_MAX;
      }
    }
    if (has)
      for (int e = tt; e < w * ld; e += T) panel[e] = 0.0;
    __syncthreads();
    // column g of the update matrix W = P G U: U (slot rows, output columns)
    // with the deflation's rotations G and the slot-to-row permutation P on
    // its rows, so that the new eigenvector block is the old one times W
    {
      const int tag = has && g < m2 ? L.tag[off + g] : -1;
      const bool root = tag >= 0 && tag < w;
      double di = 0.0, ti = 0.0, inv = 0.0;
      if (has && g < m2 && tag < 0) bad = true;
      if (root) {
        di = dro[tag];
        ti = rt[tag];
        double nrm = 0.0;
        for (int j = l8; j < nk; j += 8) {
          const double u = z[j] * rcp_d((d[j] - di) - ti);
          nrm = fma(u, u, nrm);
        }
        nrm = grp_sum<8>(nrm);
        if (!(nrm > 0.0) || !(nrm < DBL_MAX)) bad = true;
        inv = 1.0 / sqrt(nrm);
        for (int j = l8; j < nk; j += 8)
          panel[L.perm[off + L.ks[off + j]] * ld + g] = dc_uent(z[j], d[j], di, ti, inv);
      } else if (tag >= w && l8 == 0) {
        panel[L.perm[off + tag - w] * ld + g] = 1.0;
      }
      wave_sync();
      if (tag >= 0 && l8 == 0 && nrot > 0)
        dc_rotate_column(
            nrot, L.rp + off, L.rq + off, L.rc + off, L.rs + off,
            [&](int s) -> double {
              if (!root) return s == tag - w ? 1.0 : 0.0;
              const int j = L.kix[off + s] - 1;
              return j < 0 ? 0.0 : dc_uent(z[j], d[j], di, ti, inv);
            },
            [&](int s, double v) { panel[L.perm[off + s] * ld + g] = v; });
    }
    __syncthreads();
    // products, a 16 x 16 tile to a wavefront; the old block is block
    // diagonal (for S = 8 inside a tile: its entries off the halves count as
    // zero and are not read as anything else)
    if (has) {
      const int nt = w / 16, lr = lane & 15, lk = lane >> 4;
      for (int t = tt >> 6; t < nt * nt; t += T / 64) {
        const int i0 = 16 * (t / nt), j0 = 16 * (t % nt);
        const int k0 = S == 8 ? 0 : i0 / S * S, k1 = S == 8 ? 16 : k0 + S;
        const int row = i0 + lr;
        const double* Ar = Qs + (size_t)(b0 + row) * N2 + b0;
        gemm_f64x4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int k = k0; k < k1; k += 16)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int kk = k + 4 * lk + u;
            const double a = row < m2 && kk < m2 && (row < S) == (kk < S) ? Ar[kk] : 0.0;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, panel[kk * ld + j0 + lr], acc, 0, 0, 0);
          }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = i0 + lk + 4 * r, j = j0 + lr;
          if (i < m2 && j < m2) Qd[(size_t)(b0 + i) * N2 + b0 + j] = acc[r];
        }
      }
    } else {
      // no merge in this block: across to the other buffer
      for (int e = tt; e < m2 * m2; e += T) {
        const size_t o = (size_t)(b0 + e / m2) * N2 + b0 + e % m2;
        Qd[o] = Qs[o];
      }
    }
    __syncthreads();
  }
  if (tid < DC_SUB && base + tid < n) D.lam[base + tid] = L.lam[tid];
  if (bad) atomicOr(&dims[D_FLAG], FLAG_EIG);
  __syncthreads();
}

// Sort and deflation of merge m above the one-block levels, by a whole block; d and z
// of the kept entries stay in LDS (smem, smem + 2 S) for the roots.  Every
// block that solves roots of the merge does this for itself, from the same
// inputs in the same order; the one with pub set writes the merge's arrays
// for the update phase.  As dc_sub_prep: ranks, then all neighbouring
// pairs of kept entries tested at once; one wavefront runs the carrying sweep
// where a pair is near, from each near pair on.
// One lane's sweep over all entries, on one block between two grid barriers,
// took 18 us of a 142-order job's last two merges each.
struct PrepLds {
  double red[DC_T / 64];
  int wcnt[DC_T / 64];
  int nrot;
};
__device__ void dc_prep_block(const EigJob& J, int N, int n, int S, int par, int m, bool pub,
                              double* smem, PrepLds& R, int& nk_out, double& rho_out) {
  Work W = work_of(J, N);
  DC D = dc_of(W, N);
  const int N2 = next_pow2(N);
  const double* Qs = par ? D.Qb : D.Qa;
  const int b0 = m * 2 * S;
  const int nR = min(S, n - b0 - S), m2 = S + nR;
  double* dt = smem;            // original local order; then the kept d
  double* zt = dt + 2 * S;      // likewise z
  double* ds = zt + 2 * S;      // sorted
  double* zs = ds + 2 * S;
  int* perm = reinterpret_cast<int*>(zs + 2 * S);
  int* kl = perm + 2 * S;       // kept slots
  int* fl = kl + 2 * S;         // bit 0: near its predecessor, bit 1: rotated away
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const double beta = W.e[b0 + S - 1];
  const double sgn = beta < 0.0 ? -1.0 : 1.0;
  double part = 0.0, pmax = 0.0;
  for (int c = tid; c < m2; c += DC_T) {
    const double zq = c < S ? Qs[(size_t)(b0 + S - 1) * N2 + b0 + c]
                            : sgn * Qs[(size_t)(b0 + S) * N2 + b0 + c];
    const double dv = D.lam[b0 + c];
    zt[c] = zq;
    dt[c] = dv;
    part += zq * zq;
    pmax = fmax(pmax, fabs(dv));
  }
  const double nz2 = block_sum<DC_T>(part, R.red);
  for (int o = 32; o > 0; o >>= 1) pmax = fmax(pmax, __shfl_xor(pmax, o));
  __syncthreads();
  if (lane == 0) R.red[wv] = pmax;
  __syncthreads();
  double dmax = 0.0;
  for (int t = 0; t < DC_T / 64; ++t) dmax = fmax(dmax, R.red[t]);
  const double nz = sqrt(nz2);
  const double rho = fabs(beta) * nz2;
  const double tol = 8.0 * U64 * fmax(dmax, rho);
  for (int c = tid; c < m2; c += DC_T) {
    const double x = dt[c];
    const bool left = c < S;
    const double* other = dt + (left ? S : 0);
    int lo = 0, hi = left ? nR : S;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      const double y = other[mid];
      if (left ? y < x : y <= x) lo = mid + 1;
      else hi = mid;
    }
    const int pos = (left ? c : c - S) + lo;
    perm[pos] = c;
    ds[pos] = x;
    zs[pos] = nz > 0.0 ? zt[c] / nz : 0.0;
  }
  __syncthreads();
  // kept slots in order, by a block prefix count
  int nk0 = 0;
  for (int c0 = 0; c0 < m2; c0 += DC_T) {
    const int c = c0 + tid;
    const bool keep = c < m2 && !(rho * fabs(zs[c]) <= tol);
    const unsigned long long bal = __ballot(keep);
    if (lane == 0) R.wcnt[wv] = __popcll(bal);
    __syncthreads();
    int o = nk0 + __popcll(bal & ((1ULL << lane) - 1ULL));
    for (int t = 0; t < DC_T / 64; ++t) {
      if (t < wv) o += R.wcnt[t];
      nk0 += R.wcnt[t];
    }
    if (keep) kl[o] = c;
    __syncthreads();
  }
  int any = 0;
  for (int k = tid; k < nk0; k += DC_T) {
    const int c = kl[k];
    int near = 0;
    if (k > 0) {
      const int p = kl[k - 1];
      near = dc_near(ds[p], zs[p], ds[c], zs[c], tol);
    }
    fl[k] = near;
    any |= near;
  }
  any = __syncthreads_or(any);
  int nk = nk0;
  if (any) {
    if (wv == 0) {
      int nrot = 0, q0 = 1;  // pairs (k - 1, k) with k >= q0 hold their first values
      for (int k0 = 0; k0 < nk0; k0 += 64) {
        const unsigned long long mask = __ballot(k0 + lane < nk0 && (fl[min(k0 + lane, nk0 - 1)] & 1));
        while (true) {
          const int s = q0 - k0;
          const unsigned long long rest = s >= 64 ? 0ULL : s <= 0 ? mask : mask & ~((1ULL << s) - 1ULL);
          if (!rest) break;
          int q = k0 + __builtin_ctzll(rest), p = q - 1;
          double dp = ds[kl[p]], zp = zs[kl[p]];
          for (; q < nk0; ++q) {
            const int sp = kl[p], sq = kl[q];
            const double dq = ds[sq], zz = zs[sq];
            if (!dc_near(dp, zp, dq, zz, tol)) break;
            const double r = sqrt(zp * zp + zz * zz);
            const double ir = 1.0 / r;
            const double cs = zz * ir, sn = zp * ir;
            const double dqn = sn * sn * dp + cs * cs * dq;
            if (lane == 0) {
              if (pub) {
                D.rp[b0 + nrot] = sp;
                D.rq[b0 + nrot] = sq;
                D.rc[b0 + nrot] = cs;
                D.rs[b0 + nrot] = sn;
              }
              ds[sp] = cs * cs * dp + sn * sn * dq;
              zs[sp] = 0.0;
              fl[p] |= 2;
              ds[sq] = dqn;
              zs[sq] = r;
            }
            ++nrot;
            dp = dqn;
            zp = r;
            p = q;
          }
          q0 = q + 1;
        }
      }
      if (lane == 0) R.nrot = nrot;
    }
    __syncthreads();
    nk = 0;
    for (int k0 = 0; k0 < nk0; k0 += DC_T) {
      const int k = k0 + tid;
      const bool keep = k < nk0 && !(fl[k] & 2);
      const int c = keep ? kl[k] : 0;
      const unsigned long long bal = __ballot(keep);
      if (lane == 0) R.wcnt[wv] = __popcll(bal);
      __syncthreads();
      int o = nk + __popcll(bal & ((1ULL << lane) - 1ULL));
      for (int t = 0; t < DC_T / 64; ++t) {
        if (t < wv) o += R.wcnt[t];
        nk += R.wcnt[t];
      }
      if (keep) kl[o] = c;  // o <= k: no later round's entry
      __syncthreads();
    }
  }
  for (int k = tid; k < nk; k += DC_T) {
    const int c = kl[k];
    dt[k] = ds[c];
    zt[k] = zs[c];
    if (pub) {
      D.dK[b0 + k] = ds[c];
      D.zK[b0 + k] = zs[c];
      D.Kslot[b0 + k] = c;
    }
  }
  if (pub) {
    for (int c = tid; c < m2; c += DC_T) {
      D.perm[b0 + c] = perm[c];
      D.dsl[b0 + c] = ds[c];
    }
    if (tid == 0) {
      D.mk[m] = nk;
      D.mrho[m] = rho;
      D.mm2[m] = m2;
      D.mnrot[m] = any ? R.nrot : 0;
    }
  }
  __syncthreads();
  nk_out = nk;
  rho_out = rho;
}

// The pole weights of 8 poles of merge m, a wavefront each (S >= DC_ZSPLIT:
// nk^2 quotients are too many for every tile's block to form them all).
__device__ void dc_zhat_block(const EigJob& J, int N, int n, int S, int m, int grp, double* smem) {
  Work W = work_of(J, N);
  DC D = dc_of(W, N);
  const int b0 = m * 2 * S;
  if (b0 + S >= n) return;
  const int nk = D.mk[m];
  if (grp * 8 >= nk) return;
  double* d = smem;
  double* rt = d + 2 * S;
  double* dro = rt + 2 * S;
  for (int j = threadIdx.x; j < nk; j += DC_T) {
    d[j] = D.dK[b0 + j];
    rt[j] = D.rtau[b0 + j];
    dro[j] = D.dro[b0 + j];
  }
  __syncthreads();
  const int j = grp * 8 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (j >= nk) return;
  const double zh = dc_zhat<64>(d, dro, rt, D.zK[b0 + j], nk, j, D.mrho[m], lane);
  if (lane == 0) D.zhat[b0 + j] = zh;
}

// Tile (ti, tj) of half h of merge m: rows [64 ti, 64 ti + 64) of the half by
// columns [32 tj, 32 tj + 32) of the new eigenvector block, = the half's old
// block (mh x mh) times the matching rows of the update matrix W (dc_subtree),
// whose 32 columns this block forms in LDS: the sorted places of the
// outputs, the column norms, and the entries, panel by panel of KC rows.  A
// wavefront has a 16 x 16 product tile; lane groups of 16 take 4 consecutive
// k each (the same permutation of k on both operands), so a row of A is read
// 128 bytes at a time.  Merges of more than 1024 rows (STAGE false) read the
// permutation and the rotations from global memory, to stay within the CU's LDS.
struct TileLds {
  double di[DC_CT], ti[DC_CT], inv[DC_CT];
  int tag[DC_CT];
  int wcnt[DC_T / 64];
};
template <bool STAGE>
__device__ void dc_update_tile(const EigJob& J, int* __restrict__ dims, int N, int n, int S, int par,
                               int m, int h, int ti, int tj, double* smem, TileLds& R) {
  Work W = work_of(J, N);
  DC D = dc_of(W, N);
  const int N2 = next_pow2(N);
  const double* Qs = par ? D.Qb : D.Qa;
  double* Qd = par ? D.Qa : D.Qb;
  const int b0 = m * 2 * S, S2 = 2 * S, lim = n - b0;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int i0 = ti * DC_RT, j0 = tj * DC_CT;
  if (lim <= S) {  // no merge in this block: across to the other buffer
    if (h == 0)
      for (int e = tid; e < DC_RT * DC_CT; e += DC_T) {
        const int i = i0 + e / DC_CT, j = j0 + e % DC_CT;
        const size_t o = (size_t)(b0 + i) * N2 + b0 + j;
        if (i < lim && j < lim) Qd[o] = Qs[o];
      }
    return;
  }
  const int m2 = min(S2, lim);
  const int mh = h == 0 ? S : m2 - S;
  if (i0 >= mh || j0 >= m2) return;
  const int nk = D.mk[m], nrot = D.mnrot[m];
  const double rho = D.mrho[m];
  constexpr int KC = dc_kc<STAGE>();
  double* panel = smem;
  double* d = panel + KC * DC_PLD;
  double* zh = d + S2;
  double* rt = zh + S2;
  double* dro = rt + S2;
  double* dval = dro + S2;              // deflated values in slot order
  double* rc_s = dval + S2;             // staged rotations
  double* rs_s = rc_s + (STAGE ? S2 : 0);
  int* ks = reinterpret_cast<int*>(rs_s + (STAGE ? S2 : 0));
  int* kix = ks + S2;                   // slot -> K index + 1, 0 for a deflated slot
  int* dslot = kix + S2;
  int* perm_s = dslot + S2;
  int* rp_s = perm_s + (STAGE ? S2 : 0);
  int* rq_s = rp_s + (STAGE ? S2 : 0);
  const int* perm = STAGE ? perm_s : D.perm + b0;
  const int* rp = STAGE ? rp_s : D.rp + b0;
  const int* rq = STAGE ? rq_s : D.rq + b0;
  const double* rc = STAGE ? rc_s : D.rc + b0;
  const double* rs = STAGE ? rs_s : D.rs + b0;
  for (int c = tid; c < m2; c += DC_T) {
    if (STAGE) perm_s[c] = D.perm[b0 + c];
    kix[c] = 0;
  }
  for (int j = tid; j < nk; j += DC_T) {
    d[j] = D.dK[b0 + j];
    rt[j] = D.rtau[b0 + j];
    dro[j] = D.dro[b0 + j];
    ks[j] = D.Kslot[b0 + j];
    zh[j] = S >= DC_ZSPLIT ? D.zhat[b0 + j] : D.zK[b0 + j];
  }
  if (STAGE)
    for (int t = tid; t < nrot; t += DC_T) {
      rp_s[t] = D.rp[b0 + t];
      rq_s[t] = D.rq[b0 + t];
      rc_s[t] = D.rc[b0 + t];
      rs_s[t] = D.rs[b0 + t];
    }
  if (tid < DC_CT) R.tag[tid] = -1;
  __syncthreads();
  for (int j = tid; j < nk; j += DC_T) kix[ks[j]] = j + 1;
  if (S < DC_ZSPLIT)
    for (int j = tid >> 3; j < nk; j += DC_T / 8) {
      const double v = dc_zhat<8>(d, dro, rt, zh[j], nk, j, rho, tid & 7);
      if ((tid & 7) == 0) zh[j] = v;  // read by this group only
    }
  __syncthreads();
  // deflated slots in slot order, by a block prefix count
  int nd = 0;
  bool bad = false;
  for (int c0 = 0; c0 < m2; c0 += DC_T) {
    const int c = c0 + tid;
    const bool defl = c < m2 && kix[c] == 0;
    const unsigned long long bal = __ballot(defl);
    if (lane == 0) R.wcnt[wv] = __popcll(bal);
    __syncthreads();
    int o = nd + __popcll(bal & ((1ULL << lane) - 1ULL));
    for (int t = 0; t < DC_T / 64; ++t) {
      if (t < wv) o += R.wcnt[t];
      nd += R.wcnt[t];
    }
    if (defl) {
      const double v = D.dsl[b0 + c];
      bad = bad || !(v == v);
      dval[o] = v == v ? v : DBL_MAX;
      dslot[o] = c;
    }
    __syncthreads();
  }
  // Sorted places: the roots ascend; the deflated values nearly do (a rotated
  // one may pass a neighbour), and where they do not they are counted.  A
  // root goes before an equal slot.  Each block keeps the places of its own
  // columns; the first row tile of the left half writes the eigenvalues.
  int unsorted = 0;
  for (int k = tid; k + 1 < nd; k += DC_T) unsorted |= dval[k] > dval[k + 1];
  unsorted = __syncthreads_or(unsorted);
  auto place = [&](int pos, int tag, double v) {
    if (pos >= j0 && pos < j0 + DC_CT) {
      R.tag[pos - j0] = tag;
      if (h == 0 && ti == 0) D.lam[b0 + pos] = v;
    }
  };
  for (int i = tid; i < nk; i += DC_T) {
    const double lv = dro[i] + rt[i];
    bad = bad || !(lv == lv);
    const double v = lv == lv ? lv : DBL_MAX;
    int cnt = 0;
    if (unsorted) {
      for (int k = 0; k < nd; ++k) cnt += dval[k] < v;
    } else {
      int hi = nd;
      while (cnt < hi) {
        const int mid = (cnt + hi) >> 1;
        if (dval[mid] < v) cnt = mid + 1;
        else hi = mid;
      }
    }
    place(i + cnt, i, v);
  }
  for (int k = tid; k < nd; k += DC_T) {
    const double v = dval[k];
    int before = k;
    if (unsorted) {
      before = 0;
      for (int t = 0; t < nd; ++t) before += dval[t] < v || (dval[t] == v && t < k);
    }
    int cnt = 0, hi = nk;
    while (cnt < hi) {
      const int mid = (cnt + hi) >> 1;
      if (dro[mid] + rt[mid] <= v) cnt = mid + 1;
      else hi = mid;
    }
    place(before + cnt, S2 + dslot[k], v);
  }
  __syncthreads();
  {  // column norms, 16 lanes to a column
    const int c = tid >> 4, l16 = tid & 15;
    const int tag = j0 + c < m2 ? R.tag[c] : -1;
    double di = 0.0, tv = 0.0, inv = 0.0;
    if (j0 + c < m2 && tag < 0) bad = true;
    if (tag >= 0 && tag < S2) {
      di = dro[tag];
      tv = rt[tag];
      double nrm = 0.0;
      for (int j = l16; j < nk; j += 16) {
        const double u = zh[j] * rcp_d((d[j] - di) - tv);
        nrm = fma(u, u, nrm);
      }
      nrm = grp_sum<16>(nrm);
      if (!(nrm > 0.0) || !(nrm < DBL_MAX)) bad = true;
      inv = 1.0 / sqrt(nrm);
    }
    if (l16 == 0) {
      R.di[c] = di;
      R.ti[c] = tv;
      R.inv[c] = inv;
    }
  }
  if (bad) atomicOr(&dims[D_FLAG], FLAG_EIG);
  const int lr = lane & 15, lk = lane >> 4;
  const int iw = i0 + 16 * (wv >> 1), jw = 16 * (wv & 1);
  const bool live = iw < mh && j0 + jw < m2;
  const int arow = min(iw + lr, mh - 1);
  const double* Ar = Qs + (size_t)(b0 + h * S + arow) * N2 + b0 + h * S;
  gemm_f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int r0 = 0; r0 < mh; r0 += KC) {
    const int kr = min(KC, mh - r0), kr16 = (kr + 15) & ~15;
    const int first = h * S + r0;  // local row of the panel's first
    __syncthreads();
    for (int e = tid; e < kr16 * DC_PLD; e += DC_T) panel[e] = 0.0;
    __syncthreads();
    {
      const int c = tid & (DC_CT - 1), tag = R.tag[c];
      if (tag >= 0 && tag < S2) {
        const double di = R.di[c], tv = R.ti[c], inv = R.inv[c];
        for (int j = tid / DC_CT; j < nk; j += DC_T / DC_CT) {
          const int r = perm[ks[j]] - first;
          if (r >= 0 && r < kr) panel[r * DC_PLD + c] = dc_uent(zh[j], d[j], di, tv, inv);
        }
      } else if (tag >= S2 && tid < DC_CT) {
        const int r = perm[tag - S2] - first;
        if (r >= 0 && r < kr) panel[r * DC_PLD + c] = 1.0;
      }
    }
    if (nrot > 0) {
      __syncthreads();
      if (tid < DC_CT && R.tag[tid] >= 0) {
        const int tag = R.tag[tid];
        const bool root = tag < S2;
        const double di = R.di[tid], tv = R.ti[tid], inv = R.inv[tid];
        dc_rotate_column(
            nrot, rp, rq, rc, rs,
            [&](int s) -> double {
              if (!root) return s == tag - S2 ? 1.0 : 0.0;
              const int j = kix[s] - 1;
              return j < 0 ? 0.0 : dc_uent(zh[j], d[j], di, tv, inv);
            },
            [&](int s, double v) {
              const int r = perm[s] - first;
              if (r >= 0 && r < kr) panel[r * DC_PLD + tid] = v;
            });
      }
    }
    __syncthreads();
    if (live) {
      // whole groups of 16 k; a ragged last one is clipped to the half (the
      // panel's rows past it are zero)
      const double* Ak = Ar + r0 + 4 * lk;
      const double* Bk = panel + 4 * lk * DC_PLD + jw + lr;
      int k = 0;
#pragma unroll 4
      for (; k + 16 <= kr; k += 16) {
        double a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = Ak[k + u];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], Bk[(k + u) * DC_PLD], acc, 0, 0, 0);
      }
      if (k < kr) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double a = k + 4 * lk + u < kr ? Ak[k + u] : 0.0;
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Bk[(k + u) * DC_PLD], acc, 0, 0, 0);
        }
      }
    }
  }
  if (live)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = iw + lk + 4 * r, j = j0 + jw + lr;
      if (i < mh && j < m2) Qd[(size_t)(b0 + h * S + i) * N2 + b0 + j] = acc[r];
    }
}

// Levels of the divide and conquer at order n (merges of blocks S = 8, 16,
// ... while S < n), and which buffer holds its eigenvectors at the end
// (0: Qa, 1: Qb): the leaves write Qa and each level swaps.
__host__ __device__ inline int dc_par(int n) {
  int L = 0;
  for (int S = DC_LEAF; S < n; S *= 2) ++L;
  return L & 1;
}

// Job q's item t of a phase whose job q has cnt[q] items (t counts across
// the jobs in order).
__device__ inline bool dc_item(const int* cnt, int njobs, int t, int& q, int& r) {
  for (q = 0; q < njobs; ++q) {
    if (t < cnt[q]) {
      r = t;
      return true;
    }
    t -= cnt[q];
  }
  return false;
}

// The whole divide and conquer of up to 4 jobs in one launch of P
// persistent blocks: first every 64 rows' leaves and merges, one block each,
// then the merges above.  Each of those has two phases ended by a grid
// barrier: the sort and deflation (every block for itself) with 8 roots an
// item, then the tiles of its products, each forming its own columns of the
// update matrix; merges from S = DC_ZSPLIT on have the pole weights as a phase
// between.  A job stops at its own live order (dims), so its levels follow
// n, not the capacity N; orders up to 64 meet no barrier.  (Before, every
// level from 16 rows on had four phases, with sort, deflation and vectors of
// a merge on one block: 20 barriers at order 142, and two thirds of the time
// in phases of one or two blocks.)  An eigensolve of order 16, 62, 142, 322,
// 641, before and now: 135 -> 114, 286 -> 223, 616 -> 473, 2540 -> 2244,
// 6871 -> 6174 us.  LDS: the phases' arrays share the dynamic buffer
// (dc_fused_dyn_lds(N) bytes).
constexpr int DCF_MAXP = 64;
static_assert(DCF_MAXP <= SYNC_MAXP && DCF_MAXP <= GRID_CUS, "a flag a block, a CU a block");
__global__ __launch_bounds__(DC_T) void k_dc_fused(EigJobs jobs, int njobs, int* __restrict__ dims,
                                                   int N) {
  extern __shared__ double smem[];
  __shared__ PrepLds prep_lds;
  __shared__ TileLds tile_lds;
  __shared__ int s_abort;
  const int b = blockIdx.x, P = gridDim.x;
  unsigned* flags = grid_flags(jobs.j[0].work, N);
  if (threadIdx.x == 0) s_abort = 0;
  unsigned ord = GRID_ORD_DC;
  int nq[4] = {0, 0, 0, 0}, nmax = 0;
  for (int q = 0; q < njobs; ++q) {
    nq[q] = max(0, dims[jobs.j[q].n_idx]);  // -1: an SVD solved by k_svd_jacobi
    nmax = max(nmax, nq[q]);
  }
  if (nmax == 0) return;  // nothing to solve (every block sees the same sizes)
  int cnt[4] = {0, 0, 0, 0}, tot = 0;
  for (int q = 0; q < njobs; ++q) tot += cnt[q] = (nq[q] + DC_SUB - 1) / DC_SUB;
  for (int t = b; t < tot; t += P) {
    int q, r;
    if (dc_item(cnt, njobs, t, q, r))
      dc_subtree(jobs.j[q], dims, N, r, *reinterpret_cast<SubLds*>(smem));
  }
  static_assert(8 * sizeof(LeafLds) <= sizeof(SubLds::panel), "the leaves' LDS");
  static_assert(DC_SUB == 8 * DC_LEAF && DC_T == 8 * DC_SUB, "a wavefront a leaf, 8 lanes a row");
  // DC_SUB / DC_LEAF is a power of two: par counts the levels a job has passed
  int par = 1;  // after S = 8, 16, 32
  for (int S = DC_SUB; S < nmax; S *= 2, par ^= 1) {
    int nm[4] = {0, 0, 0, 0}, tm = 0;
    for (int q = 0; q < njobs; ++q) tm += nm[q] = nq[q] > S ? (nq[q] + 2 * S - 1) / (2 * S) : 0;
    grid_barrier(flags, ++ord, P, &s_abort, dims);
    const int X = 2 * S / 8;  // groups of 8 roots or poles of a merge
    for (int q = 0; q < njobs; ++q) cnt[q] = nm[q] * X;
    int have_q = -1, have_m = -1, nk = 0;  // the merge whose arrays are in LDS
    double rho = 0.0;
    for (int t = b; t < tm * X; t += P) {
      int q, r;
      if (!dc_item(cnt, njobs, t, q, r)) continue;
      const EigJob& J = jobs.j[q];
      const int m = r / X, grp = r % X, b0 = m * 2 * S;
      if (b0 + S >= nq[q] || grp * 8 >= min(2 * S, nq[q] - b0)) continue;
      // the item that publishes has group 0, which no earlier item of its merge precedes
      if (q != have_q || m != have_m) {
        __syncthreads();  // the previous merge's roots are done
        dc_prep_block(J, N, nq[q], S, par, m, grp == 0, smem, prep_lds, nk, rho);
        have_q = q;
        have_m = m;
      }
      const int i = grp * 8 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
      if (i >= nk) continue;
      double tau, dor;
      bool ok;
      dc_root<64>(smem, smem + 2 * S, nk, i, rho, lane, tau, dor, ok);
      if (lane == 0) {
        DC D = dc_of(work_of(J, N), N);
        D.rtau[b0 + i] = tau;
        D.dro[b0 + i] = dor;
        if (!ok) atomicOr(&dims[D_FLAG], FLAG_EIG);
      }
    }
    if (S >= DC_ZSPLIT) {
      grid_barrier(flags, ++ord, P, &s_abort, dims);
      for (int t = b; t < tm * X; t += P) {
        int q, r;
        __syncthreads();  // the previous item's LDS reads are done
        if (dc_item(cnt, njobs, t, q, r)) dc_zhat_block(jobs.j[q], N, nq[q], S, r / X, r % X, smem);
      }
    }
    grid_barrier(flags, ++ord, P, &s_abort, dims);
    const int TI = S / DC_RT, TJ = 2 * S / DC_CT, TM = 2 * TI * TJ;
    for (int q = 0; q < njobs; ++q) cnt[q] = nm[q] * TM;
    for (int t = b; t < tm * TM; t += P) {
      int q, r;
      __syncthreads();
      if (!dc_item(cnt, njobs, t, q, r)) continue;
      const int m = r / TM, e = r % TM, h = e / (TI * TJ), ti = (e / TJ) % TI, tj = e % TJ;
      if (2 * S <= VEC_STAGE_MAX)
        dc_update_tile<true>(jobs.j[q], dims, N, nq[q], S, par, m, h, ti, tj, smem, tile_lds);
      else
        dc_update_tile<false>(jobs.j[q], dims, N, nq[q], S, par, m, h, ti, tj, smem, tile_lds);
    }
  }
}

// Threshold of the clip rule: eigenvalues above it are kept.
__device__ inline double keep_threshold(const EigJob& J, const double* w, int n) {
  const double lmax = n > 0 ? w[n - 1] : 0.0;
  return fmax(J.clip * (double)n * U64 * lmax, 0.0);
}

// ---------------------------------------------------------------------------
// 3. Back-transformation V[:, n-1-j] = H_0 H_1 ... H_{n-3} q_j for the kept
// eigenvectors q_j of T (columns of the D&C result), a wavefront per vector,
// the vector in registers (lane l holds rows l + 64 c, c < NCH; row chunks
// past n are skipped by a scalar branch).  The reflectors are applied four
// at a time in compact WY form: G = H_k H_{k+1} H_{k+2} H_{k+3} = I - V T V^T
// with V = [v_k .. v_{k+3}] and T upper triangular (T_jj = tau_j,
// T(0:j-1, j) = -tau_j T(0:j-1, 0:j-1) V(:, 0:j-1)^T v_j), so G y = y - V (T
// (V^T y)): four dot products whose wavefront sums run side by side, a 4 x 4
// triangular product, one pass of axpys.  The reflectors are staged through
// LDS in chunks of whole groups (one cooperative load per chunk, every load
// in flight before the first store; rows zero outside each reflector, up to
// n rounded to 64), one wavefront forms each group's T there, and the
// sequential loop over the groups reads only LDS.
constexpr int ORM_G = 4;   // reflectors per compact WY group
constexpr int ORM_CH = 64;
// reflector doubles staged per chunk, and of them per thread: one block per
// CU (a launch has one block per four kept vectors, well under the CU
// count at the orders that matter), so a chunk may take most of the LDS;
// ch * ld stays within it for every capacity up to 1024 (ch >= 4)
constexpr int ORM_LDS_DBL = 18432;
constexpr int ORM_PER = (ORM_LDS_DBL + 255) / 256;
constexpr int ORM_BATCH = 24;  // staged doubles a thread loads before storing them
static_assert(ORM_PER % ORM_BATCH == 0, "whole staging batches");
__host__ __device__ inline int ormtr_ld(int N) { return ((N > 0 ? N : 1) + 63) & ~63; }
__host__ __device__ inline int ormtr_chunk(int N) {
  int c = ORM_LDS_DBL / ormtr_ld(N);
  c = c < ORM_G ? ORM_G : (c > ORM_CH ? ORM_CH : c);
  return c - c % ORM_G;
}
// for every live order up to N
inline size_t ormtr_lds_doubles(int N) {
  return (size_t)std::min(std::max(ORM_CH * ormtr_ld(N), ORM_G * ormtr_ld(N)), ORM_LDS_DBL) +
         (ORM_CH / ORM_G) * 16 + ORM_CH;
}

// VPW vectors per wavefront (4 VPW per block): every block stages all the
// reflectors, so at large orders (above 640), where the blocks
// outnumber the CUs and the staging traffic (blocks x reflector bytes) bounds
// the launch, each wavefront carries four vectors through the same staged
// chunks; below that one vector a wavefront is faster.  The choice follows the
// live order: at capacity 641 the back-transformations of a step of live
// orders up to 206 took 72 us on average by the capacity's choice, 26 by their own.
// SVD: the vectors of the short side instead, n = q of a tridiagonal of order
// 2 q: y is the even entries of the tridiagonal's eigenvector, normalised (the
// +-sigma pair's mixing only rescales its v-part), and the reflectors are the
// bidiagonalisation's right ones.
template <bool SVD, int NCH, int VPW>
__device__ __forceinline__ void ormtr_vectors(const EigJob& J, int* __restrict__ dims, int N, int nt,
                                              double* hs) {
  const int n = SVD ? nt / 2 : nt;
  const int par = dc_par(nt);
  Work W = work_of(J, N);
  DC D = dc_of(W, N);
  const int N2 = next_pow2(N);
  const int ch = ormtr_chunk(n), ld = ormtr_ld(n), gpc = ch / ORM_G;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int j0 = blockIdx.x * 4 * VPW;
  if (j0 >= n) return;
  const int c0 = nt - n;  // the n largest of the tridiagonal's nt
  const double* lam = D.lam + c0;
  const double thr = keep_threshold(J, D.lam, nt);
  // eigenvalues ascend, so the block's last vector is its largest
  if (!(lam[min(j0 + 4 * VPW - 1, n - 1)] > thr)) return;
  // vector v of this wavefront: j = j0 + 4 v + wave
  bool active[VPW];
  bool any = false;
#pragma unroll
  for (int v = 0; v < VPW; ++v) {
    const int j = j0 + 4 * v + wave;
    active[v] = j < n && lam[j] > thr;
    any = any || active[v];
  }
  // hs: ch reflectors (rows 0 .. ld - 1), each group's T, the taus
  double* Ts = hs + (size_t)ch * ld;
  double* taus = Ts + (size_t)gpc * 16;
  double y[VPW][NCH];
#pragma unroll
  for (int v = 0; v < VPW; ++v)
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int i = lane + 64 * c, j = j0 + 4 * v + wave;
      y[v][c] = active[v] && i < n ? (par ? D.Qb : D.Qa)[(size_t)(SVD ? 2 * i : i) * N2 + c0 + j] : 0.0;
    }
  if (SVD) {
#pragma unroll
    for (int v = 0; v < VPW; ++v) {
      double part = 0.0;
#pragma unroll
      for (int c = 0; c < NCH; ++c) part = fma(y[v][c], y[v][c], part);
      const double nrm = sqrt(wave_sum(part));
      const double inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
#pragma unroll
      for (int c = 0; c < NCH; ++c) y[v][c] *= inv;
    }
  }
  const int nref = SVD ? n - 1 : n - 2;  // reflectors 0 .. nref - 1
  const int ngrp = nref > 0 ? (nref + ORM_G - 1) / ORM_G : 0;
  for (int g1 = ngrp - 1; g1 >= 0; g1 -= gpc) {
    const int g0 = max(0, g1 - gpc + 1), kbase = ORM_G * g0, nr = ORM_G * (g1 - g0 + 1);
    __syncthreads();  // the previous chunk is no longer read
    // flat over (reflector, row), in batches of ORM_BATCH elements a thread:
    // every load of a batch in flight before its first store
    const int tot = nr * ld;
    const double tv = threadIdx.x < nr && kbase + (int)threadIdx.x < nref ? W.tau[kbase + threadIdx.x] : 0.0;
    for (int u0 = 0; u0 < ORM_PER; u0 += ORM_BATCH) {
      if (256 * u0 >= tot) break;
      double t[ORM_BATCH];
#pragma unroll
      for (int u = 0; u < ORM_BATCH; ++u) {
        const int e = threadIdx.x + 256 * (u0 + u), q = e / ld, i = e - q * ld, kk = kbase + q;
        t[u] = (e < tot && kk < nref && i > kk && i < n) ? W.H[(size_t)kk * N + i] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < ORM_BATCH; ++u) {
        const int e = threadIdx.x + 256 * (u0 + u);
        if (e < tot) hs[e] = t[u];
      }
    }
    if (threadIdx.x < nr) taus[threadIdx.x] = tv;
    __syncthreads();
    for (int gq = wave; gq <= g1 - g0; gq += 4) {
      const double* v = hs + (size_t)(ORM_G * gq) * ld;
      const int kb = kbase + ORM_G * gq;
      double d01 = 0.0, d02 = 0.0, d03 = 0.0, d12 = 0.0, d13 = 0.0, d23 = 0.0;
      for (int i = kb + 1 + lane; i < n; i += 64) {
        const double a0 = v[i], a1 = v[ld + i], a2 = v[2 * ld + i], a3 = v[3 * ld + i];
        d01 = fma(a0, a1, d01);
        d02 = fma(a0, a2, d02);
        d03 = fma(a0, a3, d03);
        d12 = fma(a1, a2, d12);
        d13 = fma(a1, a3, d13);
        d23 = fma(a2, a3, d23);
      }
      d01 = wave_sum(d01);
      d02 = wave_sum(d02);
      d03 = wave_sum(d03);
      d12 = wave_sum(d12);
      d13 = wave_sum(d13);
      d23 = wave_sum(d23);
      const double t0 = taus[ORM_G * gq], t1 = taus[ORM_G * gq + 1];
      const double t2 = taus[ORM_G * gq + 2], t3 = taus[ORM_G * gq + 3];
      const double T01 = -t1 * t0 * d01;
      const double T02 = -t2 * (t0 * d02 + T01 * d12), T12 = -t2 * t1 * d12;
      const double T03 = -t3 * ((t0 * d03 + T01 * d13) + T02 * d23);
      const double T13 = -t3 * (t1 * d13 + T12 * d23), T23 = -t3 * t2 * d23;
      if (lane < 16) {
        const int rr = lane >> 2, cc = lane & 3;
        double tv = 0.0;
        if (rr == cc) tv = rr == 0 ? t0 : rr == 1 ? t1 : rr == 2 ? t2 : t3;
        else if (rr < cc)
          tv = rr == 0 ? (cc == 1 ? T01 : cc == 2 ? T02 : T03) : rr == 1 ? (cc == 2 ? T12 : T13) : T23;
        Ts[gq * 16 + lane] = tv;
      }
    }
    __syncthreads();
    if (!any) continue;
    for (int gq = g1 - g0; gq >= 0; --gq) {
      const double* v = hs + (size_t)(ORM_G * gq) * ld;
      const int kb = kbase + ORM_G * gq;
      // one vector: the group's rows stay in registers for the update; more:
      // they are read from LDS again (registers hold the vectors)
      constexpr bool KEEP = VPW == 1;
      double vv[ORM_G][KEEP ? NCH : 1];
      double sv[VPW][ORM_G];
#pragma unroll
      for (int w = 0; w < VPW; ++w)
#pragma unroll
        for (int q = 0; q < ORM_G; ++q) sv[w][q] = 0.0;
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const int ck = KEEP ? c : 0;
#pragma unroll
        for (int q = 0; q < ORM_G; ++q) vv[q][ck] = 0.0;
        if (64 * c >= n || 64 * c + 63 <= kb) continue;  // no rows of the group here
        const int i = lane + 64 * c;
#pragma unroll
        for (int q = 0; q < ORM_G; ++q) vv[q][ck] = v[(size_t)q * ld + i];
#pragma unroll
        for (int w = 0; w < VPW; ++w)
#pragma unroll
          for (int q = 0; q < ORM_G; ++q) sv[w][q] = fma(vv[q][ck], y[w][c], sv[w][q]);
      }
      const double* T = Ts + gq * 16;
#pragma unroll
      for (int w = 0; w < VPW; ++w) {
        const double s0 = wave_sum(sv[w][0]), s1 = wave_sum(sv[w][1]);
        const double s2 = wave_sum(sv[w][2]), s3 = wave_sum(sv[w][3]);
        const double u0 = ((T[0] * s0 + T[1] * s1) + T[2] * s2) + T[3] * s3;
        const double u1 = (T[5] * s1 + T[6] * s2) + T[7] * s3;
        const double u2 = T[10] * s2 + T[11] * s3;
        const double u3 = T[15] * s3;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          if (64 * c >= n || 64 * c + 63 <= kb) continue;
          const int i = lane + 64 * c;
          const double a0 = KEEP ? vv[0][KEEP ? c : 0] : v[i];
          const double a1 = KEEP ? vv[1][KEEP ? c : 0] : v[(size_t)ld + i];
          const double a2 = KEEP ? vv[2][KEEP ? c : 0] : v[2 * (size_t)ld + i];
          const double a3 = KEEP ? vv[3][KEEP ? c : 0] : v[3 * (size_t)ld + i];
          y[w][c] -= ((a0 * u0 + a1 * u1) + a2 * u2) + a3 * u3;
        }
      }
    }
  }
#pragma unroll
  for (int w = 0; w < VPW; ++w) {
    if (!active[w]) continue;
    const int col = n - 1 - (j0 + 4 * w + wave);
    // sign gauge: the largest |entry| (first on ties) positive
    double best = -1.0, val = 0.0;
    int bi = 0x7fffffff;
#pragma unroll
    for (int c = 0; c < NCH; ++c)
      if (lane + 64 * c < n && fabs(y[w][c]) > best) {
        best = fabs(y[w][c]);
        val = y[w][c];
        bi = lane + 64 * c;
      }
    for (int o = 32; o > 0; o >>= 1) {
      const double b2 = __shfl_xor(best, o), v2 = __shfl_xor(val, o);
      const int i2 = __shfl_xor(bi, o);
      if (b2 > best || (b2 == best && i2 < bi)) {
        best = b2;
        val = v2;
        bi = i2;
      }
    }
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int i = lane + 64 * c;
      if (i < n) J.V[(size_t)i * J.ldv + col] = val < 0.0 ? -y[w][c] : y[w][c];
    }
  }
}

// Descending eigenvalues (SVD: singular values), the kept count, sq and isq, by
// one block.
template <bool SVD>
__device__ __forceinline__ void eig_counts(const EigJob& J, int* __restrict__ dims, int N, int nt) {
  const int n = SVD ? nt / 2 : nt;
  Work W = work_of(J, N);
  const double* lam = dc_of(W, N).lam;
  const double thr = keep_threshold(J, lam, nt);
  lam += nt - n;
  __shared__ int s_low, s_bad;
  const int tid = threadIdx.x;
  if (tid == 0) {
    s_low = -1;
    s_bad = 0;
  }
  __syncthreads();
  // ascending: the kept ones are those above the highest index whose value is
  // not above the threshold (a NaN counts as not above)
  int low = -1, bad = 0;
  for (int j = tid; j < n; j += 256) {
    if (!(lam[j] == lam[j])) bad = 1;
    if (!(lam[j] > thr)) low = j;
  }
  if (low >= 0) atomicMax(&s_low, low);
  if (bad) s_bad = 1;
  __syncthreads();
  const int kept = n - 1 - s_low;
  if (tid == 0) {
    dims[J.kept_idx] = kept;
    if (s_bad) atomicOr(&dims[D_FLAG], FLAG_EIG);
  }
  for (int c = tid; c < n; c += 256) {
    const double l = lam[n - 1 - c];
    J.lam[c] = l;
    if (c < kept) {
      const double s = SVD ? l : sqrt(l);
      J.sq[c] = s;
      J.isq[c] = 1.0 / s;
    }
  }
}

template <bool SVD>
__global__ __launch_bounds__(256) void k_ormtr(EigJobs jobs, int* __restrict__ dims, int N) {
  extern __shared__ double hs[];
  const EigJob J = jobs.j[blockIdx.y];
  const int nt = dims[J.n_idx];
  if (nt < 0) return;  // an SVD solved by k_svd_jacobi
  const int n = SVD ? nt / 2 : nt;
  // block 0 holds the smallest, the likeliest not kept
  if (blockIdx.x == 0) eig_counts<SVD>(J, dims, N, nt);
  if (n <= 192) ormtr_vectors<SVD, 3, 1>(J, dims, N, nt, hs);
  else if (n <= 384) ormtr_vectors<SVD, 6, 1>(J, dims, N, nt, hs);
  else if (n <= 640) ormtr_vectors<SVD, 10, 1>(J, dims, N, nt, hs);
  else ormtr_vectors<SVD, 16, 4>(J, dims, N, nt, hs);
}

// ---------------------------------------------------------------------------
// 5. Small SVD through the Golub-Kahan tridiagonal.  With M = Q_L B Q_R^T
// (B upper bidiagonal, diagonal d_i, superdiagonal e_i), the symmetric
// tridiagonal of order 2q with zero diagonal and off-diagonal
// (d_0, e_0, d_1, e_1, ..., d_{q-1}) has eigenvalues +-sigma_j, and the
// eigenvector of +sigma_j interleaves (v_j, u_j) / sqrt 2.  Its eigenpairs
// come from the divide and conquer above, so sigma_j is accurate to
// ~u sigma_1 absolutely and the vectors to ~u sigma_1 / gap.

// Small SVDs by one-sided Jacobi (Hestenes), in one 512-thread block: when
// the short side q <= JAC_QMAX and the p x q work matrix B (B = M for side 1,
// M^T for side 0; p >= q) fits LDS, its columns are orthogonalised by plane
// rotations, B V = U S, and the right vectors V (the vectors of M's short
// side) and S come out directly, with no bidiagonalisation and no
// tridiagonal eigensolve.  V is accumulated over the rotations: M is graded on
// both sides, and the tiny entries of V that couple a small singular value to
// a large column keep their relative accuracy that way, on which U = M V S^-1
// depends (forming V from the orthogonalised rows of a QR factor takes fewer
// sweeps and loses it: U's columns come out orthogonal to 1e-6, not 1e-12).
//
// A round is one latency chain: the exchange of the columns through LDS (its
// writes the largest part), the sums, the rotation's scalars, the update, a
// barrier.  So columns move in blocks of two: the nbe blocks are paired
// round-robin (nbe - 1 rounds of nbe / 2 disjoint block pairs per sweep), half
// a wavefront holds the four columns of its pair and their V columns in
// registers for a round and applies the four cross rotations as two steps of
// two independent ones (and, in round 0, the two inside the blocks).  Lane r
// holds rows 2 r, 2 r + 1 of every 64, so columns move in 16-byte LDS accesses.
// Whole calls of tt_kernel_svd (about 65 us besides this kernel) on matrices
// graded by 1e-4 along the rows and 1e-6 along the columns, before (one pair
// per 16 lanes and round, three sums a pair, divisions and square roots) and
// now: 142 x 36 411 -> 300 us, 144 x 63 984 -> 616, 96 x 32 320 -> 213, 62 x 12
// 113 -> 93.
//
// A pair (i, j) with a = |b_i|^2, b = |b_j|^2, g = b_i . b_j is rotated when
// g^2 > (p u)^2 a b, by the angle that zeroes g to the accuracy of the
// hardware's reciprocals (jacobi_rotation).  a and b are summed in round 0 of
// a sweep and follow the rotations from there by a - t g, b + t g; a sweep that
// rotates nothing, which ends the iteration, has tested summed norms only.
// More than JAC_MAXSW sweeps raise the eigensolver flag.  Singular values are
// the final column norms, sorted descending (index breaks ties); the kept
// count, the scalings and the sign gauge follow the same rules as the
// Golub-Kahan path, whose launches then return at once: the Golub-Kahan order
// dims[J.n_idx] is set to -1 to say so.
constexpr int JAC_QMAX = 64;
constexpr int JAC_PQ = 14336;   // doubles of B in LDS (112 KB: columns of p rows padded to 16)
constexpr int JAC_PMAX = 512;
constexpr int JAC_MAXSW = 40;
constexpr int JAC_T = 512;
constexpr int JAC_WAVES = JAC_T / 64;
constexpr int JAC_VLD = JAC_QMAX;
__device__ inline int jacobi_ld(int p) { return (p + 15) & ~15; }
// columns of B in LDS: an even number of blocks of two, those past q zero
__device__ inline int jacobi_cols(int q) { return (q + 3) & ~3; }
__device__ inline bool jacobi_fits(int p, int q) {
  return q >= 1 && q <= JAC_QMAX && p <= JAC_PMAX && jacobi_ld(p) * jacobi_cols(q) <= JAC_PQ;
}

// Sum over each half wavefront, the same bits on all its lanes: the first four
// steps of wave_sum on each row of 16 lanes, then the row swap puts the two
// rows' sums side by side on both.
__device__ inline double half_sum(double v) {
  v += dpp_d<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_d<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_d<0x141>(v);  // row_half_mirror
  v += dpp_d<0x140>(v);  // row_mirror
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
  const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  return __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
         __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
}

// Rotation by the smaller angle that makes columns x_i, x_j with
// d = |x_j|^2 - |x_i|^2 and g = x_i . x_j != 0 orthogonal: x_i' = c x_i - s x_j,
// x_j' = s x_i + c x_j, t = s / c = sign(d) 2 g / (|d| + sqrt(d^2 + 4 g^2)), on d
// and 2 g scaled by a power of two (exact).  t needs no more than the
// hardware's reciprocal (square root) estimates, about 2^-24: what a rotation
// leaves of g is that small part of it, and the next sweep's rotation takes it.
// c and s are (y, y t), y the estimate of 1 / sqrt(1 + t^2), scaled by
// (1 - e)^(-1/2), e = 1 - y^2 - (y t)^2 taken on the rounded pair itself, so that
// c^2 + s^2 = 1 but for the roundings of c and s.  (c from the rounded 1 + t^2
// alone, which the many small t of the last sweeps fall out of, makes c^2 + s^2
// too large by 1 to 2 u on average; that adds up over the rotations: the V of a
// graded 144 x 63 matrix was orthogonal to 1690 u in the Frobenius norm, with
// one over a square root and a division to 1110 u, and this way to 140 u.)
__device__ inline void jacobi_rotation(double d, double g, double& c, double& s, double& t) {
  const double e2 = 2.0 * g;
  const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(d), fabs(e2)));
  const double ds = __builtin_amdgcn_ldexp(d, ex), es = __builtin_amdgcn_ldexp(e2, ex);
  const double h2 = fma(ds, ds, es * es);
  const double r = __builtin_amdgcn_rcp(fma(h2, __builtin_amdgcn_rsq(h2), fabs(ds)));
  t = (ds >= 0.0 ? es : -es) * r;
  const double y = __builtin_amdgcn_rsq(fma(t, t, 1.0)), z = y * t;
  const double e = fma(-z, z, fma(-y, y, 1.0)), h = fma(0.375, e, 0.5);
  c = fma(y * e, h, y);
  s = fma(z * e, h, z);
}

// A column of 64 C rows and its V column on half a wavefront.
template <int C>
struct JacCol {
  double2 x[C], v;
  double n2;  // squared norm
};
template <int C>
__device__ inline double jac_dot(const JacCol<C>& a, const JacCol<C>& b) {
  double s0 = a.x[0].x * b.x[0].x, s1 = a.x[0].y * b.x[0].y;
#pragma unroll
  for (int c = 1; c < C; ++c) {
    s0 = fma(a.x[c].x, b.x[c].x, s0);
    s1 = fma(a.x[c].y, b.x[c].y, s1);
  }
  return half_sum(s0 + s1);
}
__device__ inline void jac_turn(double2& a, double2& b, double c, double s) {
  const double2 x = a, y = b;
  a.x = fma(c, x.x, -s * y.x);
  a.y = fma(c, x.y, -s * y.y);
  b.x = fma(s, x.x, c * y.x);
  b.y = fma(s, x.y, c * y.y);
}
// Rotates the disjoint pairs (a0, b0) and (a1, b1) where they need it; the two
// chains interleave.  Returns whether a pair of this half was rotated.
template <int C>
__device__ inline bool jac_step(JacCol<C>& a0, JacCol<C>& b0, JacCol<C>& a1, JacCol<C>& b1,
                                double tol2) {
  const double g0 = jac_dot(a0, b0), g1 = jac_dot(a1, b1);
  const bool r0 = g0 != 0.0 && g0 * g0 > tol2 * a0.n2 * b0.n2;
  const bool r1 = g1 != 0.0 && g1 * g1 > tol2 * a1.n2 * b1.n2;
  if (__any(r0 || r1)) {
    double c0, s0, t0, c1, s1, t1;
    jacobi_rotation(b0.n2 - a0.n2, g0, c0, s0, t0);
    jacobi_rotation(b1.n2 - a1.n2, g1, c1, s1, t1);
    c0 = r0 ? c0 : 1.0;
    s0 = r0 ? s0 : 0.0;
    t0 = r0 ? t0 * g0 : 0.0;
    c1 = r1 ? c1 : 1.0;
    s1 = r1 ? s1 : 0.0;
    t1 = r1 ? t1 * g1 : 0.0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      jac_turn(a0.x[c], b0.x[c], c0, s0);
      jac_turn(a1.x[c], b1.x[c], c1, s1);
    }
    jac_turn(a0.v, b0.v, c0, s0);
    jac_turn(a1.v, b1.v, c1, s1);
    a0.n2 -= t0;
    b0.n2 += t0;
    a1.n2 -= t1;
    b1.n2 += t1;
  }
  return r0 || r1;
}

// LDS of the Jacobi kernel's sweeps.
struct JacLds {
  double B[JAC_PQ];                // column j at j ld; rows p .. ld - 1, columns past q zero
  double V[JAC_QMAX * JAC_VLD];
  double n2[JAC_QMAX];             // squared norms
  double pad[2];                   // the rows past ld of a chunk of 64: zeros
  int rot[2];
};

// All sweeps over the columns in LDS (64 (C - 1) < p <= 64 C).  Returns the sweeps
// before the one that rotated nothing; maxsw when the last of them did.
template <int C>
__device__ int jacobi_sweeps(JacLds& L, int p, int q, int maxsw) {
  const int lane = threadIdx.x & 63, rl = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int k = 2 * wave + (lane >> 5);  // block pair of this half
  const int ld = jacobi_ld(p);
  const int nbe = jacobi_cols(q) / 2, npair = nbe / 2, m1 = nbe - 1;
  const double tol2 = ((double)p * U64) * ((double)p * U64);
  const bool tail = 64 * (C - 1) + 2 * rl < ld;  // this lane's rows of the last chunk
  int sw = 0;
  for (; sw < maxsw; ++sw) {
    const int flag = sw & 1;
    for (int rnd = 0; rnd < m1; ++rnd) {
      if (k < npair) {
        // round-robin: position 0 fixed, the others rotate
        int xa = k - 1 + rnd, xb = nbe - 2 - k + rnd;
        if (xa >= m1) xa -= m1;
        if (xb >= m1) xb -= m1;
        const int bi = k == 0 ? 0 : 1 + xa, bj = 1 + xb;
        JacCol<C> w[4];
        double2 *px[4], *pt[4], *pv[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const int col = 2 * (m < 2 ? bi : bj) + (m & 1);
          px[m] = reinterpret_cast<double2*>(L.B + col * ld) + rl;
          // rows past ld: read and written as the zeros they are
          pt[m] = tail ? px[m] + 32 * (C - 1) : reinterpret_cast<double2*>(L.pad);
          pv[m] = reinterpret_cast<double2*>(L.V + col * JAC_VLD) + rl;
#pragma unroll
          for (int c = 0; c < C - 1; ++c) w[m].x[c] = px[m][32 * c];
          w[m].x[C - 1] = *pt[m];
          w[m].v = *pv[m];
          w[m].n2 = L.n2[col];
        }
        bool rot = false;
        if (rnd == 0) {
#pragma unroll
          for (int m = 0; m < 4; ++m) w[m].n2 = jac_dot(w[m], w[m]);
          rot = jac_step(w[0], w[1], w[2], w[3], tol2);
        }
        rot |= jac_step(w[0], w[2], w[1], w[3], tol2);
        rot |= jac_step(w[0], w[3], w[1], w[2], tol2);
        if (rot) {
#pragma unroll
          for (int m = 0; m < 4; ++m) {
#pragma unroll
            for (int c = 0; c < C - 1; ++c) px[m][32 * c] = w[m].x[c];
            *pt[m] = w[m].x[C - 1];
            *pv[m] = w[m].v;
          }
        }
        if (rl == 0 && (rot || rnd == 0)) {
          *reinterpret_cast<double2*>(&L.n2[2 * bi]) = double2{w[0].n2, w[1].n2};
          *reinterpret_cast<double2*>(&L.n2[2 * bj]) = double2{w[2].n2, w[3].n2};
          if (rot) L.rot[flag] = 1;
        }
      }
      lds_barrier();
    }
    const int any = L.rot[flag];
    if (threadIdx.x == 0) L.rot[flag ^ 1] = 0;  // the next sweep's flag
    lds_barrier();
    if (!any) break;
  }
  return sw;
}

__global__ __launch_bounds__(JAC_T) void k_svd_jacobi(const double* __restrict__ M, int ldm,
                                                      EigJobs jobs, int* __restrict__ dims, int N,
                                                      int a_idx, int b_idx, int side_idx) {
  const EigJob J = jobs.j[0];
  grid_clear(grid_flags(J.work, N), threadIdx.x, JAC_T);
  const int a = dims[a_idx], b = dims[b_idx], side = dims[side_idx];
  const int p = side ? a : b, q = side ? b : a;
  if (!jacobi_fits(p, q)) {  // the Golub-Kahan path
    if (threadIdx.x == 0) dims[J.n_idx] = 2 * q;
    return;
  }
  __shared__ __align__(16) JacLds L;
  __shared__ double ssig[JAC_QMAX];
  __shared__ int spos[JAC_QMAX];
  __shared__ int s_kept;
  double *Bs = L.B, *Vs = L.V;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // B column-major (column j at Bs + j ld, rows p .. ld - 1 and columns past q
  // zero), V = I; both read along M's rows
  const int ld = jacobi_ld(p), nc = jacobi_cols(q);
  if (side) {
    for (int e = tid; e < ld * nc; e += JAC_T) {
      const int i = e / nc, j = e - i * nc;
      Bs[j * ld + i] = i < p && j < q ? M[(long long)i * ldm + j] : 0.0;
    }
  } else {
    for (int e = tid; e < ld * nc; e += JAC_T) {
      const int j = e / ld, i = e - j * ld;
      Bs[e] = i < p && j < q ? M[(long long)j * ldm + i] : 0.0;
    }
  }
  for (int e = tid; e < nc * JAC_VLD; e += JAC_T) Vs[e] = (e % JAC_VLD) == (e / JAC_VLD) ? 1.0 : 0.0;
  if (tid < JAC_QMAX) L.n2[tid] = 0.0;
  if (tid < 2) {
    L.rot[tid] = 0;
    L.pad[tid] = 0.0;
  }
  __syncthreads();
  // sweeps allowed: JAC_MAXSW, or fewer when the host caps them (a test of
  // the failure path: the rotations stay finite, only convergence is lost)
  const int capsw = dims[D_JAC_MAXSW];
  const int maxsw = capsw > 0 && capsw < JAC_MAXSW ? capsw : JAC_MAXSW;
  int sw;
  // C = ceil(ld / 64): every chunk but the last lies wholly within a column
  switch ((p + 63) / 64) {
    case 1: sw = jacobi_sweeps<1>(L, p, q, maxsw); break;
    case 2: sw = jacobi_sweeps<2>(L, p, q, maxsw); break;
    case 3: sw = jacobi_sweeps<3>(L, p, q, maxsw); break;
    case 4: sw = jacobi_sweeps<4>(L, p, q, maxsw); break;
    case 5: sw = jacobi_sweeps<5>(L, p, q, maxsw); break;
    case 6: sw = jacobi_sweeps<6>(L, p, q, maxsw); break;
    case 7: sw = jacobi_sweeps<7>(L, p, q, maxsw); break;
    default: sw = jacobi_sweeps<8>(L, p, q, maxsw);
  }
  if (sw == maxsw && tid == 0) atomicOr(&dims[D_FLAG], FLAG_NOCONV);
  // singular values: column norms; descending order (index breaks ties)
  for (int j = wave; j < q; j += JAC_WAVES) {
    double part = 0.0;
    for (int i = lane; i < p; i += 64) part = fma(Bs[j * ld + i], Bs[j * ld + i], part);
    const double s2 = wave_sum(part);
    if (lane == 0) ssig[j] = sqrt(s2);
  }
  __syncthreads();
  if (tid < q) {
    const double v = ssig[tid];
    if (!(v == v)) atomicOr(&dims[D_FLAG], FLAG_EIG);
    int pos = 0;
    double smax = 0.0;
    for (int kk = 0; kk < q; ++kk) {
      const double w = ssig[kk];
      pos += (w > v) || (w == v && kk < tid);
      smax = fmax(smax, w);
    }
    spos[tid] = pos;
    J.lam[pos] = v;
    // the Golub-Kahan path's clip rule at its order 2q: sigma > clip 2q u sigma_1
    const double thr = fmax(J.clip * (double)(2 * q) * U64 * smax, 0.0);
    const bool keep = v > thr;
    const unsigned long long m = __ballot(keep);
    if (keep) {
      J.sq[pos] = v;
      J.isq[pos] = 1.0 / v;
    }
    if (tid == 0) {
      s_kept = __popcll(m);
      dims[J.kept_idx] = s_kept;
      dims[J.n_idx] = -1;
    }
  }
  __syncthreads();
  // vectors in descending order, of the kept ones the largest-magnitude entry
  // (first on ties) positive; a wavefront per column, an entry per lane
  const int kept = s_kept;
  for (int j = wave; j < q; j += JAC_WAVES) {
    const int pos = spos[j];
    const double x = lane < q ? Vs[j * JAC_VLD + lane] : 0.0;
    double best = fabs(x), val = x;
    int bi = lane;
    for (int o = 32; o > 0; o >>= 1) {
      const double b2 = __shfl_xor(best, o), v2 = __shfl_xor(val, o);
      const int i2 = __shfl_xor(bi, o);
      if (b2 > best || (b2 == best && i2 < bi)) { best = b2; val = v2; bi = i2; }
    }
    if (lane < q) J.V[(size_t)lane * J.ldv + pos] = pos < kept && val < 0.0 ? -x : x;
  }
}

// Golub-Kahan bidiagonalisation of the taller orientation (p x q, p >= q): left
// reflectors zero column k below the diagonal (d_k), right reflectors zero
// row k right of the superdiagonal (e_k).  Only the right reflectors are kept
// (W.H rows, W.tau): the vectors of the short side are Q_R times the v-part
// of the tridiagonal's eigenvectors.
//
// k_gebrd: the matrix in registers, a wavefront's rows over P blocks, one
// exchange per step.  The left reflector of column k is u = e_k + s_L c,
// c = A(k+1:, k), and its product with the trailing matrix is
// y = tau_L (A(k, k+1:) + s_L sum_{i > k} A(i, k) A(i, k+1:)): each wavefront can
// form its share of that sum, and of |c|^2, from its own rows before the
// reflector exists.  Step k: every wavefront puts those two partials in LDS,
// the owner of row k the row; the block sums them, over several blocks
// publishes the sums and after a barrier adds up the P of them (relaxed
// agent-scope accesses, columns from k on); then every wavefront forms the left reflector,
// y, row k after it, and from that row the right reflector v_k, tau_R, e_k,
// redundantly, and applies both to its own rows
// (A_i -= s_L A(i, k) y, then A_i -= tau_R (A_i . v) v).  Exchange buffers are
// double-buffered by step parity: a block may write step k + 1's while another
// still reads step k's.
// One kernel for all column classes: as compiled it has 256 registers, of which 14
// spill (60 bytes a lane), and 620 scalar ones; the widest class sets that.
// Bound by latency: at 142 x 142 a step is 5.5 us, of which the block's and the
// grid's barriers take 2.1, the loads behind them 1.2, the reflectors 0.7 and
// the rows 1.3; at 128 x 128 and below, on one block, 3 us.  (With the rows
// in LDS a step took 7 us at 142 x 142.)  An SVD of order 100, 142, 192, 322,
// 897 x 896, before and now: 679 -> 620, 1461 -> 1135, 1944 -> 1435, 3927 ->
// 3102, 23292 -> 20702 us.
// Outputs: W.e[2k] = d_k, W.e[2k+1] = e_k, W.tau, right reflectors in W.H.
constexpr int GBR_T = 512;
constexpr int GBR_W = GBR_T / 64;
constexpr int GEBRD_QMAX = 1024;     // columns at most
constexpr int GEBRD_GRID_PMAX = 64;  // blocks at most: 1024 rows, 16 a block above 704 columns
static_assert(GEBRD_GRID_PMAX <= GRID_CUS, "a block fills a CU: 8 wavefronts of 256 registers");
static_assert(GEBRD_GRID_PMAX <= SYNC_MAXP && GEBRD_QMAX < (int)(GRID_ORD_DC - GRID_ORD_REDUCE),
              "a flag a block, an ordinal a column");
struct GebrdGridBufs {
  double *R, *Y, *S;  // published rows (2 x N), partial sums (2 x P x N), |c|^2 partials (2 x P)
};
__device__ __host__ inline GebrdGridBufs gebrd_grid_bufs(double* work, int N) {
  const size_t N2 = next_pow2(N);
  double* z = work + 4 * (size_t)N + (size_t)N * N + N2;
  GebrdGridBufs B;
  B.R = z;
  B.Y = z + 2 * (size_t)N;
  B.S = B.Y + 2 * (size_t)GEBRD_GRID_PMAX * N;
  return B;
}

// x, as a value that the compiler knows nothing about: a uniform condition on
// it stays one branch, where conditions it can relate to others are
// threaded into copies of the code between them, which spills the matrix.
__device__ __forceinline__ int opaque_s(int x) {
  asm volatile("" : "+s"(x));
  return x;
}

// Sums over the wavefront of four values at once: two exchanges of lane halves
// and of rows pack them, one to a row of 16 lanes, before the sums inside the
// rows.  All results on every lane.
__device__ inline double pack_add(double x, double y, bool half) {
  const unsigned long long bx = (unsigned long long)__double_as_longlong(x);
  const unsigned long long by = (unsigned long long)__double_as_longlong(y);
  const auto l = half ? __builtin_amdgcn_permlane32_swap((unsigned)bx, (unsigned)by, false, false)
                      : __builtin_amdgcn_permlane16_swap((unsigned)bx, (unsigned)by, false, false);
  const auto h = half ? __builtin_amdgcn_permlane32_swap((unsigned)(bx >> 32), (unsigned)(by >> 32), false, false)
                      : __builtin_amdgcn_permlane16_swap((unsigned)(bx >> 32), (unsigned)(by >> 32), false, false);
  return __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
         __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
}
__device__ inline void wave_sum4(double* x) {
  // rows of 16: x[0], x[2], x[1], x[3]
  double v = pack_add(pack_add(x[0], x[1], true), pack_add(x[2], x[3], true), false);
  v += dpp_d<0xB1>(v);
  v += dpp_d<0x4E>(v);
  v += dpp_d<0x141>(v);
  v += dpp_d<0x140>(v);
  x[0] = lane_d(v, 0);
  x[1] = lane_d(v, 32);
  x[2] = lane_d(v, 16);
  x[3] = lane_d(v, 48);
}

// a += x y in place: written out so that the matrix entries stay where they are
// (the compiler otherwise copies them at branches).
__device__ __forceinline__ void fmac_in_place(double& a, double x, double y) {
  asm("v_fmac_f64 %0, %1, %2" : "+v"(a) : "v"(x), "v"(y));
}

// One block's part for q <= 64 NT: of P blocks of GBR_W wavefronts, wavefront w of
// block b holds the rows 8 b + w + 8 P r, r < R, a lane the columns lane + 64 t.
template <int NT, int R>
__device__ __forceinline__ void gebrd_rows(const double* __restrict__ M, int ldm, int side, const EigJob& J,
                           int* __restrict__ dims, int N, int p, int q, int P, double* lds,
                           int* s_abort) {
  Work W = work_of(J, N);
  const GebrdGridBufs G = gebrd_grid_bufs(J.work, N);
  constexpr int LQ = NT * 64;
  constexpr int GS = R < 4 ? R : 4;  // rows taken together
  double* part = lds;                 // partial sums of the wavefronts (GBR_W x LQ)
  double* sacc = part + GBR_W * LQ;   // their sum
  double* srow2 = sacc + LQ;          // row k, by the parity of k
  double* ssq = srow2 + 2 * LQ;       // |c|^2 partials (GBR_W), then their sum in ssq[GBR_W]
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row0 = __builtin_amdgcn_readfirstlane(GBR_W * b + wave), rstep = GBR_W * P;
  double a[R][NT];
  const int si = side ? ldm : 1, sj = side ? 1 : ldm;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = row0 + rstep * r;
    const double* Mi = M + (long long)min(i, p - 1) * si;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int j = lane + 64 * t;
      const double x = Mi[(long long)min(j, q - 1) * sj];
      a[r][t] = i < p && j < q ? x : 0.0;
    }
    __builtin_amdgcn_sched_barrier(0);  // a row's loads at a time: their addresses are short-lived
  }
  if (b == 0)
    for (int i = tid; i < 2 * q; i += GBR_T) W.d[i] = 0.0;
  unsigned* flags = grid_flags(J.work, N);
  unsigned ordinal = GRID_ORD_REDUCE;
  __builtin_amdgcn_s_waitcnt(0x0F70);  // the matrix is there: no waits for it in the loop (10 us at 300 x 300)
  const bool writer = b == 0 && wave == 0;
  for (int k = 0;; ++k) {
    double* srow = srow2 + (k & 1) * LQ;
    const int kr = k - row0, pr = p - row0;  // row r is past k, below p
    // column k of rows g .. g + 3, zero where the row is done
    auto column = [&](int g, double (&c)[GS]) {
      const int lk = k & 63;
#pragma unroll
      for (int r = 0; r < GS; ++r) c[r] = 0.0;
#pragma unroll
      for (int t = 0; t < NT; ++t)
        if (opaque_s(k >> 6) == t)
#pragma unroll
          for (int r = 0; r < GS; ++r) c[r] = a[g + r][t];
#pragma unroll
      for (int r = 0; r < GS; ++r) {
        const long long x = __double_as_longlong(c[r]);
        const int m = (kr - rstep * (g + r)) >> 31;  // -1: past k
        const int lo = __builtin_amdgcn_readlane((int)x, lk) & m;
        const int hi = __builtin_amdgcn_readlane((int)(x >> 32), lk) & m;
        c[r] = __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
      }
    };
    // partials of step k over the own rows i > k, and row k from its owner
    {
      double s[NT], cc = 0.0;
#pragma unroll
      for (int t = 0; t < NT; ++t) s[t] = 0.0;
#pragma unroll
      for (int g = 0; g < R; g += GS) {
        const bool live = rstep * (g + GS - 1) > opaque_s(kr) && rstep * g < opaque_s(pr);
        if (!live) continue;
        double c[GS];
        column(g, c);
#pragma unroll
        for (int r = 0; r < GS; ++r) cc = fma(c[r], c[r], cc);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if (64 * t + 63 <= opaque_s(k)) continue;
#pragma unroll
          for (int r = 0; r < GS; ++r) s[t] = fma(c[r], a[g + r][t], s[t]);
        }
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) part[wave * LQ + lane + 64 * t] = s[t];
      if (lane == 0) ssq[wave] = cc;
      if (k % rstep == row0) {
        const int rk = k / rstep;
        double x[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) x[t] = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (r == rk)
#pragma unroll
            for (int t = 0; t < NT; ++t) x[t] = a[r][t];
        if (P == 1) {
#pragma unroll
          for (int t = 0; t < NT; ++t) srow[lane + 64 * t] = x[t];
        } else {
#pragma unroll
          for (int t = 0; t < NT; ++t)
            if (lane + 64 * t >= k && lane + 64 * t < q) xput(G.R + (size_t)(k & 1) * N + lane + 64 * t, x[t]);
        }
      }
    }
    lds_barrier();
    // the block's sums; over several blocks their exchange
    if (P == 1) {
      for (int j = tid; j < LQ; j += GBR_T) {
        double acc = 0.0;
#pragma unroll
        for (int w = 0; w < GBR_W; ++w) acc += part[w * LQ + j];
        sacc[j] = acc;
      }
      if (tid == GBR_T - 1) {
        double acc = 0.0;
#pragma unroll
        for (int w = 0; w < GBR_W; ++w) acc += ssq[w];
        ssq[GBR_W] = acc;
      }
    } else {
      const int par = k & 1;
      double* Y = G.Y + (size_t)par * GEBRD_GRID_PMAX * N;
      double* S = G.S + (size_t)par * GEBRD_GRID_PMAX;
      // columns before k are done: nothing reads their sums
      for (int j = tid; j < q; j += GBR_T) {
        if (j < k) continue;
        double acc = 0.0;
#pragma unroll
        for (int w = 0; w < GBR_W; ++w) acc += part[w * LQ + j];
        xput(Y + (size_t)b * N + j, acc);
      }
      if (tid == GBR_T - 1) {
        double acc = 0.0;
#pragma unroll
        for (int w = 0; w < GBR_W; ++w) acc += ssq[w];
        xput(S + b, acc);
      }
      grid_barrier_relaxed(flags, ++ordinal, P, s_abort, dims);
      for (int j = tid; j < q; j += GBR_T) {
        if (j < k) continue;
        double acc = 0.0;
        const double row = xget(G.R + (size_t)par * N + j);
        // many partials in flight, without a branch each (past P: the last again,
        // not added): a wait behind the barrier costs about 1 us
        const double* Yj = Y + j;
        auto sum = [&](auto batch) {
          constexpr int U = decltype(batch)::value;
          for (int u0 = 0; u0 < P; u0 += U) {
            double v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = xget(Yj + (size_t)min(u0 + u, P - 1) * N);
#pragma unroll
            for (int u = 0; u < U; ++u) acc += u0 + u < P ? v[u] : 0.0;
          }
        };
        if (P <= 8) sum(std::integral_constant<int, 8>());
        else sum(std::integral_constant<int, 32>());
        sacc[j] = acc;
        srow[j] = row;
      }
      if (wave == GBR_W - 1) {
        const double s = wave_sum(lane < P ? xget(S + lane) : 0.0);
        if (lane == 0) ssq[GBR_W] = s;
      }
    }
    lds_barrier();
    // left reflector of column k, y and row k after it, right reflector of
    // that row: every wavefront for itself
    double tl, sl, bl;
    householder(srow[k], ssq[GBR_W], tl, sl, bl);
    if (writer && lane == 0) W.e[2 * k] = bl;
    if (k == q - 1) {
      if (writer && lane == 0) W.tau[k] = 0.0;
      break;
    }
    double y[NT], v[NT], sq = 0.0, al = 0.0;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int j = lane + 64 * t;
      const bool live = j > k && j < q;
      const double rkj = live ? srow[j] : 0.0;
      y[t] = live ? tl * (rkj + sl * sacc[j]) : 0.0;
      v[t] = rkj - y[t];
      if (j > k + 1) sq = fma(v[t], v[t], sq);
      if (j == k + 1) al = v[t];
    }
    double tr, sr, br;
    householder(wave_sum(al), wave_sum(sq), tr, sr, br);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int j = lane + 64 * t;
      v[t] = j > k + 1 ? v[t] * sr : j == k + 1 ? 1.0 : 0.0;
      if (writer && j > k && j < q) W.H[(long long)k * N + j] = v[t];
    }
    if (writer && lane == 0) {
      W.e[2 * k + 1] = br;
      W.tau[k] = tr;
    }
    // own rows: A_i -= s_L A(i, k) y, then A_i -= tau_R (A_i . v) v
#pragma unroll
    for (int g = 0; g < R; g += GS) {
      if (rstep * (g + GS - 1) <= opaque_s(kr) || rstep * g >= opaque_s(pr)) continue;
      double z[4] = {0.0, 0.0, 0.0, 0.0}, u[GS];
      column(g, u);
#pragma unroll
      for (int r = 0; r < GS; ++r) u[r] *= -sl;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (64 * t + 63 <= opaque_s(k)) continue;
#pragma unroll
        for (int r = 0; r < GS; ++r) {
          fmac_in_place(a[g + r][t], u[r], y[t]);
          z[r] = fma(a[g + r][t], v[t], z[r]);
        }
      }
      wave_sum4(z);
#pragma unroll
      for (int r = 0; r < GS; ++r) z[r] *= -tr;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (64 * t + 63 <= opaque_s(k)) continue;
#pragma unroll
        for (int r = 0; r < GS; ++r) fmac_in_place(a[g + r][t], z[r], v[t]);
      }
    }
  }
}

// Blocks for a p x q matrix, p >= q: one, 16 rows a wavefront, up to 128 x 128;
// above, 4 rows a wavefront (2 past 704 columns, whose registers they fill).
// One block needs no exchange, about 3 us of a 100 x 100 step, but a CU's
// registers hold no more; with more blocks a step is near 5.5 us whatever the rows,
// so few rows a wavefront (its work between two exchanges) beat few blocks.
__device__ __host__ inline int gebrd_blocks(int p, int q) {
  if (p <= 16 * GBR_W && q <= 128) return 1;
  const int rows = q <= 256 ? 8 * GBR_W : q <= 704 ? 4 * GBR_W : 2 * GBR_W;
  return (p + rows - 1) / rows;
}
__device__ __host__ inline int gebrd_chunks(int q) {
  return q <= 128 ? 2 : q <= 192 ? 3 : q <= 256 ? 4 : q <= 384 ? 6 : q <= 512 ? 8
       : q <= 704 ? 11 : 16;
}
inline size_t gebrd_lds(int q) {
  return ((size_t)(GBR_W + 3) * 64 * gebrd_chunks(q) + GBR_W + 8) * 8;
}

__global__ __launch_bounds__(GBR_T) void k_gebrd(const double* __restrict__ M, int ldm, EigJobs jobs,
                                                 int* __restrict__ dims, int N, int a_idx, int b_idx,
                                                 int side_idx) {
  extern __shared__ double lds[];
  __shared__ int s_abort;
  const EigJob J = jobs.j[0];
  if (dims[J.n_idx] < 0) return;  // solved by k_svd_jacobi
  const int ma = dims[a_idx], mb = dims[b_idx], side = dims[side_idx];
  const int p = side ? ma : mb, q = side ? mb : ma;
  const int P = gebrd_blocks(p, q);
  if (q < 1 || (int)blockIdx.x >= P) return;
  if (threadIdx.x == 0) s_abort = 0;
  __syncthreads();
  if (P == 1) gebrd_rows<2, 16>(M, ldm, side, J, dims, N, p, q, 1, lds, &s_abort);
  else if (q <= 128) gebrd_rows<2, 8>(M, ldm, side, J, dims, N, p, q, P, lds, &s_abort);
  else if (q <= 192) gebrd_rows<3, 8>(M, ldm, side, J, dims, N, p, q, P, lds, &s_abort);
  else if (q <= 256) gebrd_rows<4, 8>(M, ldm, side, J, dims, N, p, q, P, lds, &s_abort);
  else if (q <= 384) gebrd_rows<6, 4>(M, ldm, side, J, dims, N, p, q, P, lds, &s_abort);
  else if (q <= 512) gebrd_rows<8, 4>(M, ldm, side, J, dims, N, p, q, P, lds, &s_abort);
  else if (q <= 704) gebrd_rows<11, 4>(M, ldm, side, J, dims, N, p, q, P, lds, &s_abort);
  else gebrd_rows<16, 2>(M, ldm, side, J, dims, N, p, q, P, lds, &s_abort);
}

// Dynamic LDS of k_dc_fused at capacity N: the largest of its phases' needs
// (the one-block merges; sort and deflation, tiles of the levels above).
size_t dc_fused_dyn_lds(int N) {
  size_t need = sizeof(SubLds);
  for (int S = DC_SUB; S < N; S *= 2) {
    const size_t m2 = (size_t)2 * S;
    need = std::max(need, m2 * PREP_BYTES_PER);
    need = std::max(need, m2 <= VEC_STAGE_MAX
                              ? dc_kc<true>() * DC_PLD * 8 + m2 * VEC_BYTES_STAGED
                              : dc_kc<false>() * DC_PLD * 8 + m2 * VEC_BYTES_GLOBAL);
  }
  return need;
}
// Blocks: a block each up to order 64; above, one for 8 roots or a top
// merge's tile, and for several jobs one for 8 places of a whole top merge: a
// job's items are counted so, and with fewer blocks the next job's come a round
// later (its launches in steps of two jobs of order 142 average 129 us on 64
// blocks, 141 on 36).  At most DCF_MAXP: with up to a CU's LDS each they keep to
// GRID_CUS CUs (the residence that grid barriers need, k_sytrd_grid).
int dc_fused_blocks(int N, int njobs) {
  if (N <= DC_SUB) return njobs;
  const int roots = njobs > 1 ? next_pow2(N) / 8 : (N + 7) / 8;
  return std::min(DCF_MAXP, njobs * std::max(roots, N * N / 2048));
}

}  // namespace

// ---- LDS budget of the launches with dynamic LDS -----------------------------
// A CU has 160 KiB of LDS; a launch asking for more static + dynamic LDS than
// that fails to dispatch.  These are the static sizes of the kernels launched
// with dynamic LDS as compiled for gfx950; at run time the larger of this and
// the runtime's own figure is used.
namespace {
constexpr size_t LDS_CU = 160 * 1024;
constexpr size_t ST_SYTRD_GRID = 8, ST_DC_FUSED = 1296, ST_ORMTR = 0, ST_GEBRD = 8,
                 ST_SVD_JACOBI = 148768;

size_t static_lds(const void* fn, size_t table, bool runtime) {
  if (!runtime) return table;
  hipFuncAttributes a;
  if (hipFuncGetAttributes(&a, fn) == hipSuccess && (size_t)a.sharedSizeBytes > table)
    return (size_t)a.sharedSizeBytes;
  return table;
}

void lds_note(size_t bytes, const char* name, size_t& worst, const char** which) {
  if (bytes > worst) {
    worst = bytes;
    if (which) *which = name;
  }
}

// divide and conquer at order N (eigensolve N, or Golub-Kahan order 2q)
void dc_lds(int N, bool rt, size_t& worst, const char** which) {
  lds_note(static_lds((const void*)k_dc_fused, ST_DC_FUSED, rt) + dc_fused_dyn_lds(N), "k_dc_fused",
           worst, which);
}
}  // namespace

size_t eig_lds_bytes(int N, bool runtime, const char** which) {
  size_t worst = 0;
  // (an order past the columns that its registers hold counts as not fitting)
  if (N > SYR_MAX)
    lds_note(static_lds((const void*)k_sytrd_grid<true>, ST_SYTRD_GRID, runtime) + sytrd_grid_lds(N) +
                 (N > SYTRD_GRID_NMAX ? LDS_CU : 0),
             "k_sytrd_grid", worst, which);
  dc_lds(N, runtime, worst, which);
  lds_note(static_lds((const void*)k_ormtr<false>, ST_ORMTR, runtime) + ormtr_lds_doubles(N) * 8,
           "k_ormtr", worst, which);
  return worst;
}

size_t svd_lds_bytes(int ncap2, int pcap, bool runtime, const char** which) {
  size_t worst = 0;
  lds_note(static_lds((const void*)k_svd_jacobi, ST_SVD_JACOBI, runtime), "k_svd_jacobi", worst, which);
  const int qcap = ncap2 / 2;
  const int qc = std::min(qcap, pcap);
  lds_note(static_lds((const void*)k_gebrd, ST_GEBRD, runtime) + gebrd_lds(qc) +
               (qc > GEBRD_QMAX || gebrd_blocks(pcap, qc) > GEBRD_GRID_PMAX ? LDS_CU : 0),
           "k_gebrd", worst, which);
  lds_note(static_lds((const void*)k_ormtr<true>, ST_ORMTR, runtime) + ormtr_lds_doubles(qcap) * 8,
           "k_ormtr", worst, which);
  dc_lds(ncap2, runtime, worst, which);
  return worst;
}

bool lds_fits(size_t bytes) { return bytes <= LDS_CU; }

size_t eig_work_doubles(int N) { return eig_work_main(N) + SYNC_DOUBLES; }

namespace {

// Divide and conquer of the tridiagonals (W.d, W.e) of the jobs; the
// eigenvectors end in buffer dc_par(n) of each job.
void dc_solve(const EigJobs& J, int njobs, int N, int* dims, hipStream_t s) {
  k_dc_fused<<<dc_fused_blocks(N, njobs), DC_T, dc_fused_dyn_lds(N), s>>>(J, njobs, dims, N);
}

}  // namespace

void eig_batched(const EigJob* jobs, int njobs, int N, int* dims, hipStream_t s) {
  if (njobs <= 0 || N <= 0) return;
  EigJobs J;
  for (int i = 0; i < njobs && i < 4; ++i) J.j[i] = jobs[i];
  k_sytrd_reg<<<njobs, SYR_T, 0, s>>>(J, dims, N);
  if (N > SYR_MAX) {
    const int nj = njobs < 4 ? njobs : 4;
    for (int q = 0; q < nj; q += SYG_JOBS) {
      const dim3 grid(sytrd_grid_blocks(N), std::min(SYG_JOBS, nj - q));
      if (N > SYG_WIDE) k_sytrd_grid<true><<<grid, SYTRD_GRID_T, sytrd_grid_lds(N), s>>>(J, q, dims, N);
      else k_sytrd_grid<false><<<grid, SYTRD_GRID_T, sytrd_grid_lds(N), s>>>(J, q, dims, N);
    }
  }
  dc_solve(J, njobs < 4 ? njobs : 4, N, dims, s);
  k_ormtr<false><<<dim3((N + 3) / 4, njobs), 256, ormtr_lds_doubles(N) * 8, s>>>(J, dims, N);
}

void svd_short_side(const double* M, int ldm, int a_idx, int b_idx, int side_idx,
                    const EigJob& job, int N, int pcap, int* dims, hipStream_t s) {
  if (N < 2) return;
  EigJobs J;
  J.j[0] = job;
  const int qcap = N / 2;
  k_svd_jacobi<<<1, JAC_T, 0, s>>>(M, ldm, J, dims, N, a_idx, b_idx, side_idx);
  const int qc = std::min(qcap, pcap);
  k_gebrd<<<gebrd_blocks(pcap, qc), GBR_T, gebrd_lds(qc), s>>>(M, ldm, J, dims, N, a_idx, b_idx, side_idx);
  dc_solve(J, 1, N, dims, s);
  k_ormtr<true><<<(qcap + 3) / 4, 256, ormtr_lds_doubles(qcap) * 8, s>>>(J, dims, N);
}

}  // namespace tt
