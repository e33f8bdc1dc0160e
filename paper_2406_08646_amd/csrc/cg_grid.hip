// Jacobi-CG of a mid-size system as ONE cooperative launch (paper Sec. 6:
// fewer synchronisation points, scalars on the device).
//
// What bounds the launch-per-phase solve of such a system is not its bytes
// (a 66,049-row 9-point operator is 7 MB) but two kernels an iteration, each
// a chain of dependent memory round trips (partials, row bounds, entries,
// gather, reduction) that starts from nothing: 8.2 + 5.5 us.  Here every
// workgroup keeps its rows for the whole solve: their values and 16-bit
// window columns in LDS, their vectors in registers.  What still crosses
// workgroups each iteration is the vector u that the product reads (a few
// KB per workgroup, through memory) and three sums, so an iteration is two
// exchanges between the resident workgroups.
//
// The recurrences, tests and statuses are those of the form in cg.hip that
// the solve would take without this launch, the single-reduction one
// (k_sr_update, k_sr_spmv) or the textbook one (k_cg_update, k_cg_pupdate),
// element by element; only the order in which the dots' partial sums are
// added differs.
//
// An exchange: each workgroup stores its partial sums in its slots, every
// workgroup reads all slots and adds them in the same order, so all take
// the same branches.  A double travels as two 64-bit words, each with 32 of
// its bits and the exchange's number, so a word is valid as soon as its
// number matches and needs no fence.  Slots alternate between two sets: a
// workgroup can be at most one exchange ahead of another.  u and the words
// are written and read with agent-scope accesses, which go past the XCD's
// L2; a workgroup's stores of u have completed (vmcnt 0 in every wave, then
// the barrier) before it stores its words.  The launch is cooperative, so
// every workgroup is resident; a wait that still exceeds kWaitTicks gives
// up, and the solve reports an error.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.hpp"
#include "device.hpp"

namespace spx {
namespace {

constexpr int kGridBlock = 512;
constexpr int kGridWaves = kGridBlock / 64;
constexpr int kGridMaxWg = 256;  // two values of all slots: one poll per thread
constexpr int kGridWords = 256;  // bitmap of the 64-entry blocks of x
constexpr int64_t kGridMaxRows = (int64_t)kGridWords * 32 * kWinBlock;
// Copies of the slots: workgroup b reads copy b % 8, so that 32 workgroups
// and not 256 poll the same lines (at 256 workgroups an iteration takes 6.6
// us with 8 copies, 7.0 with 2, 8.0 with 1; with one copy of two separate
// 8-byte words 11.1).
constexpr int kGridCopies = 8;
constexpr int kGridSet = kGridCopies * 2 * kGridMaxWg;  // pairs of one slot set
constexpr long long kWaitTicks = 2000000000;  // 20 s of the 100 MHz clock
typedef unsigned long long Pair __attribute__((ext_vector_type(2)));
static_assert(2 * 2 * kGridSet == kGridSlotWords, "two slot sets of word pairs");
static_assert(2 * kGridMaxWg <= kGridBlock, "a thread polls one value of one workgroup");
static_assert(2 * kGridCopies <= 64, "one wave stores a workgroup's words");

// The matrix in precision VT and each workgroup's share of it.
template <typename VT>
struct GridMat {
  int64_t n;
  const int32_t* rowptr;
  const int32_t* col;
  const VT* val;
  int rows;     // rows per workgroup (a multiple of 32)
  int entries;  // most entries of one workgroup
  int blocks;   // x blocks its LDS holds
};

struct GridLds {
  double red[2][kGridWaves];
  double tot[kGridWaves];
  uint32_t bits[kGridWords];
  uint32_t incl[kGridWords];
  int fail;
};

template <typename T>
__device__ __forceinline__ T agent_load(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void agent_store(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One 16-byte word pair, past the caches.
__device__ __forceinline__ Pair agent_load_pair(const Pair* p) {
  Pair v;
  asm volatile("global_load_dwordx4 %0, %1, off sc1\n\ts_waitcnt vmcnt(0)"
               : "=&v"(v)
               : "v"(p)
               : "memory");
  return v;
}
__device__ __forceinline__ void agent_store_pair(Pair* p, Pair v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1" : : "v"(p), "v"(v) : "memory");
}

// v[k] becomes its sum over every thread of every workgroup (N <= 2).
// Returns false when a wait gave up (the same in every thread).
template <int N>
__device__ __forceinline__ bool exchange(Pair* slots, uint32_t number, GridLds& l,
                                         double (&v)[N]) {
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const double s = wave_sum(v[k]);
    if (lane == 0) l.red[k][w] = s;
  }
  __builtin_amdgcn_s_waitcnt(0);  // this wave's stores of u are in memory
  __syncthreads();
  Pair* set = slots + (number & 1) * kGridSet;
  if (tid < kGridCopies * N) {
    const int k = tid / kGridCopies, c = tid % kGridCopies;
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < kGridWaves; ++i) s += l.red[k][i];
    const unsigned long long bits = (unsigned long long)__double_as_longlong(s);
    const unsigned long long tag = (unsigned long long)number << 32;
    Pair q;
    q.x = tag | (bits & 0xffffffffull);
    q.y = tag | (bits >> 32);
    agent_store_pair(set + (c * 2 + k) * kGridMaxWg + blockIdx.x, q);
  }
  const int k = tid / kGridMaxWg, g = tid % kGridMaxWg;
  double got = 0.0;
  if (k < N && g < (int)gridDim.x) {
    const Pair* p = set + ((blockIdx.x % kGridCopies) * 2 + k) * kGridMaxWg + g;
    Pair q;
    long long until = 0;
    for (int spin = 1;; ++spin) {
      q = agent_load_pair(p);
      if ((uint32_t)(q.x >> 32) == number && (uint32_t)(q.y >> 32) == number) break;
      if ((spin & 1023) == 0) {
        const long long now = (long long)wall_clock64();
        if (until == 0) until = now + kWaitTicks;
        if (now > until) {
          l.fail = 1;
          break;
        }
      }
    }
    got = __longlong_as_double((long long)((q.y << 32) | (q.x & 0xffffffffull)));
  }
  got = wave_sum(got);
  if (lane == 0) l.tot[w] = got;
  __syncthreads();
  constexpr int PER = kGridMaxWg / 64;
#pragma unroll
  for (int q = 0; q < N; ++q) {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < PER; ++i) s += l.tot[q * PER + i];
    v[q] = s;
  }
  return l.fail == 0;
}

// One workgroup's share in LDS: its entries' values and window columns, and
// the blocks of x that they fall in.
template <typename VT>
struct GridShare {
  VT* xs;  // the window of x
  VT* val;
  int32_t* blk;
  uint16_t* col;
  int64_t r0, r1;
  int32_t t0;
  int nblk;    // blocks of the window
  bool ready;  // the share fits
};

template <typename VT>
size_t grid_lds_bytes(int64_t entries, int64_t blocks) {
  return (size_t)(entries * (sizeof(VT) + sizeof(uint16_t)) +
                  blocks * (kWinBlock * sizeof(VT) + sizeof(int32_t)));
}

template <typename VT>
__device__ __forceinline__ GridShare<VT> grid_setup(const GridMat<VT>& A, GridLds& l, char* smem) {
  GridShare<VT> S;
  S.xs = reinterpret_cast<VT*>(smem);
  S.val = S.xs + (int64_t)A.blocks * kWinBlock;
  S.blk = reinterpret_cast<int32_t*>(S.val + A.entries);
  S.col = reinterpret_cast<uint16_t*>(S.blk + A.blocks);
  S.r0 = (int64_t)blockIdx.x * A.rows;
  S.r1 = S.r0 + A.rows < A.n ? S.r0 + A.rows : A.n;
  S.t0 = A.rowptr[S.r0];
  const int32_t t0 = S.t0, t1 = A.rowptr[S.r1];
  S.nblk = 0;
  S.ready = false;
  const int tid = threadIdx.x;
  if (tid == 0) l.fail = 0;
  if (t1 - t0 > A.entries) return S;
  for (int i = tid; i < kGridWords; i += kGridBlock) l.bits[i] = 0;
  __syncthreads();
  for (int32_t e = t0 + tid; e < t1; e += kGridBlock) {
    const int32_t d = A.col[e] / kWinBlock;
    atomicOr(&l.bits[d >> 5], 1u << (d & 31));
  }
  __syncthreads();
  if (tid < kGridWords) l.incl[tid] = __popc(l.bits[tid]);
  __syncthreads();
  for (int o = 1; o < kGridWords; o <<= 1) {
    const uint32_t v = tid < kGridWords && tid >= o ? l.incl[tid - o] : 0u;
    __syncthreads();
    if (tid < kGridWords) l.incl[tid] += v;
    __syncthreads();
  }
  S.nblk = (int)l.incl[kGridWords - 1];
  if (S.nblk > A.blocks) return S;
  if (tid < kGridWords) {
    const uint32_t w = l.bits[tid];
    uint32_t rank = l.incl[tid] - __popc(w);
    for (uint32_t m = w; m != 0; m &= m - 1) S.blk[rank++] = tid * 32 + (__ffs(m) - 1);
  }
  for (int32_t e = t0 + tid; e < t1; e += kGridBlock) {
    const int32_t c = A.col[e], d = c / kWinBlock;
    const uint32_t w = l.bits[d >> 5];
    const uint32_t r = l.incl[d >> 5] - __popc(w) + __popc(w & ((1u << (d & 31)) - 1u));
    S.col[e - t0] = (uint16_t)(r * kWinBlock + c % kWinBlock);
    S.val[e - t0] = A.val[e];
  }
  __syncthreads();
  S.ready = true;
  return S;
}

// Calls f(i, v[entry]) for every entry of the share's window, i its place
// in it (entries at n and beyond are 0), a few loads of a thread in flight
// together; AGENT: past the caches.
template <bool AGENT, typename VT, typename F>
__device__ __forceinline__ void grid_window(const VT* __restrict__ v, int64_t n,
                                            const GridShare<VT>& S, F&& f) {
  constexpr int PRE = 4;
  const int cnt = S.nblk * kWinBlock;
  for (int q0 = threadIdx.x; q0 < cnt; q0 += PRE * kGridBlock) {
    VT t[PRE];
#pragma unroll
    for (int k = 0; k < PRE; ++k) {
      const int q = q0 + k * kGridBlock;
      t[k] = VT(0);
      if (q < cnt) {
        const int64_t g = (int64_t)S.blk[q / kWinBlock] * kWinBlock + q % kWinBlock;
        if (g < n) t[k] = AGENT ? agent_load(v + g) : v[g];
      }
    }
#pragma unroll
    for (int k = 0; k < PRE; ++k) {
      const int q = q0 + k * kGridBlock;
      if (q < cnt) f(q, t[k]);
    }
  }
  __syncthreads();
}

// Entries [ra, re) of the share times its window, in entry order.
template <typename VT>
__device__ __forceinline__ VT grid_row(const GridShare<VT>& S, int32_t ra, int32_t re) {
  constexpr int U = 4;
  VT s = VT(0);
  int32_t e = ra;
  for (; e + U <= re; e += U) {
    VT a[U], x[U];
#pragma unroll
    for (int k = 0; k < U; ++k) a[k] = S.val[e + k];
#pragma unroll
    for (int k = 0; k < U; ++k) x[k] = S.xs[S.col[e + k]];
#pragma unroll
    for (int k = 0; k < U; ++k) s += a[k] * x[k];
  }
  for (; e < re; ++e) s += S.val[e] * S.xs[S.col[e]];
  return s;
}

constexpr double kGridBad = 0x1p40;  // added by a workgroup whose share does not fit

struct GridSolve {
  const int32_t* dpos;
  const double* b;
  double* x;
  double* u;  // work vector
  Pair* slots;
  CgScalars* st;
  double rtol;
  int32_t maxit;
};

// The fp64 solve.  Thread t owns rows r0 + t, r0 + t + kGridBlock, ... (RPT
// of them).  TEXTBOOK: that form, in which each workgroup keeps p on its whole
// window, as k_cg_grid_inner does, so it takes two exchanges an iteration
// too; s is then A p.
template <int RPT, bool TEXTBOOK>
__global__ __launch_bounds__(kGridBlock) void k_cg_grid(GridMat<double> A, GridSolve a) {
  extern __shared__ __align__(16) char smem[];
  __shared__ GridLds l;
  const int tid = threadIdx.x;
  const GridShare<double> S = grid_setup(A, l, smem);
  const auto stage = [&](int i, double v) { S.xs[i] = v; };
  double bad = !S.ready && tid == 0 ? kGridBad : 0.0;  // and one for each zero diagonal
  int32_t ra[RPT], re[RPT];
  double x[RPT], r[RPT], p[RPT], s[RPT], u[RPT], dinv[RPT];
  double gr[2] = {0.0, 0.0}, bf[2] = {0.0, 0.0};  // r.u, r.r; b.b, bad
  if (S.ready) grid_window<false>(a.x, A.n, S, stage);
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int64_t row = S.r0 + tid + k * kGridBlock;
    ra[k] = re[k] = 0;
    x[k] = r[k] = p[k] = s[k] = u[k] = dinv[k] = 0.0;
    if (S.ready && row < S.r1) {
      ra[k] = A.rowptr[row] - S.t0;
      re[k] = A.rowptr[row + 1] - S.t0;
      const int32_t dp = a.dpos[row];
      const double d = dp >= 0 ? S.val[dp - S.t0] : 0.0;
      if (d == 0.0)
        bad += 1.0;
      else
        dinv[k] = 1.0 / d;
      const double bi = a.b[row];
      x[k] = a.x[row];
      r[k] = bi - grid_row(S, ra[k], re[k]);
      u[k] = dinv[k] * r[k];
      agent_store(a.u + row, u[k]);
      gr[0] += r[k] * u[k];
      gr[1] += r[k] * r[k];
      bf[0] += bi * bi;
    }
  }
  bf[1] = bad;
  uint32_t number = 0;
  const bool ok = exchange(a.slots, ++number, l, gr) && exchange(a.slots, ++number, l, bf);
  double gamma = gr[0], rr = gr[1], pq = 0.0, alpha = 0.0;
  const double bb = bf[0], bnorm = sqrt(bb), thresh = a.rtol * bnorm;
  int32_t status = SPX_OK, iters = 0;
  bool run = false;
  if (!ok)
    status = kGridTimedOut;
  else if (bf[1] >= kGridBad)
    status = kGridUnfit;
  else if (bf[1] != 0.0)
    status = SPX_ZERO_DIAGONAL;
  else if (sqrt(rr) <= thresh)
    status = SPX_OK;
  else if (a.maxit <= 0)
    status = SPX_NOT_CONVERGED;
  else
    run = true;
  if (TEXTBOOK && run) {
    grid_window<true>(a.u, A.n, S, stage);
#pragma unroll
    for (int q = 0; q < RPT; ++q) p[q] = u[q];
    for (int32_t k = 1;; ++k) {
      double d[1] = {0.0};
#pragma unroll
      for (int q = 0; q < RPT; ++q) {
        s[q] = grid_row(S, ra[q], re[q]);
        d[0] += p[q] * s[q];
      }
      if (!exchange(a.slots, ++number, l, d)) {
        status = kGridTimedOut;
        break;
      }
      pq = d[0];
      if (!(pq > 0.0) || !isfinite(pq)) {
        status = SPX_BREAKDOWN;
        iters = k - 1;
        break;
      }
      alpha = gamma / pq;
      gr[0] = gr[1] = 0.0;
#pragma unroll
      for (int q = 0; q < RPT; ++q) {
        const int64_t row = S.r0 + tid + q * kGridBlock;
        x[q] = x[q] + alpha * p[q];
        r[q] = r[q] - alpha * s[q];
        u[q] = dinv[q] * r[q];
        if (row < S.r1) agent_store(a.u + row, u[q]);
        gr[0] += r[q] * u[q];
        gr[1] += r[q] * r[q];
      }
      if (!exchange(a.slots, ++number, l, gr)) {
        status = kGridTimedOut;
        break;
      }
      rr = gr[1];
      iters = k;
      if (sqrt(rr) <= thresh) break;
      if (k >= a.maxit) {
        status = SPX_NOT_CONVERGED;
        break;
      }
      const double beta = gr[0] / gamma;
      gamma = gr[0];
#pragma unroll
      for (int q = 0; q < RPT; ++q) p[q] = u[q] + beta * p[q];
      grid_window<true>(a.u, A.n, S, [&](int i, double v) { S.xs[i] = v + beta * S.xs[i]; });
    }
  } else if (run) {
    double g_prev = 0.0;
    for (int32_t k = 0;; ++k) {
      // w = A u; p = u + beta p; s = w + beta s (p = u, s = w at k = 0)
      const double beta = k == 0 ? 0.0 : gamma / g_prev;
      grid_window<true>(a.u, A.n, S, stage);
      double d[1] = {0.0};
#pragma unroll
      for (int q = 0; q < RPT; ++q) {
        const double w = grid_row(S, ra[q], re[q]);
        p[q] = k == 0 ? u[q] : u[q] + beta * p[q];
        s[q] = k == 0 ? w : w + beta * s[q];
        d[0] += w * u[q];
      }
      if (!exchange(a.slots, ++number, l, d)) {
        status = kGridTimedOut;
        break;
      }
      pq = k == 0 ? d[0] : d[0] - beta * gamma / alpha;
      if (!(pq > 0.0) || !isfinite(pq)) {
        status = SPX_BREAKDOWN;
        iters = k;
        break;
      }
      alpha = gamma / pq;
      gr[0] = gr[1] = 0.0;
#pragma unroll
      for (int q = 0; q < RPT; ++q) {
        const int64_t row = S.r0 + tid + q * kGridBlock;
        x[q] = x[q] + alpha * p[q];
        r[q] = r[q] - alpha * s[q];
        u[q] = dinv[q] * r[q];
        if (row < S.r1) agent_store(a.u + row, u[q]);
        gr[0] += r[q] * u[q];
        gr[1] += r[q] * r[q];
      }
      if (!exchange(a.slots, ++number, l, gr)) {
        status = kGridTimedOut;
        break;
      }
      g_prev = gamma;
      gamma = gr[0];
      rr = gr[1];
      iters = k + 1;
      if (sqrt(rr) <= thresh) break;
      if (iters >= a.maxit) {
        status = SPX_NOT_CONVERGED;
        break;
      }
    }
  }
  if (run) {
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const int64_t row = S.r0 + tid + q * kGridBlock;
      if (row < S.r1) a.x[row] = x[q];
    }
  }
  if (tid == 0 && status == kGridTimedOut) a.st->verify = 1;  // whichever workgroup saw it
  if (tid == 0 && blockIdx.x == 0) {
    a.st->rho[0] = gamma;
    a.st->pq = pq;
    a.st->alpha = alpha;
    a.st->rr = rr;
    a.st->bb = bb;
    a.st->bnorm = bnorm;
    a.st->thresh = thresh;
    a.st->iters = iters;
    a.st->status = status;
    a.st->done = 1;
  }
}

struct GridInner {
  float* x;
  const float* r;
  float* z;  // in: D^-1 r; then the work vector
  const float* dinv;
  Pair* slots;
  CgScalars* st;
};

// The fp32 inner solve of the mixed refinement (the recurrences of
// k_cg_update and k_cg_pupdate: fp32 vectors and product, fp64 dots) from
// x = 0, r and z = D^-1 r, with rho, the threshold and the limit in *st.
// Each workgroup keeps p on its whole window: after an exchange of r.z it
// reads its neighbours' z and updates their p itself, so the textbook form
// also takes two exchanges an iteration.
template <int RPT>
__global__ __launch_bounds__(kGridBlock) void k_cg_grid_inner(GridMat<float> A, GridInner a) {
  extern __shared__ __align__(16) char smem[];
  __shared__ GridLds l;
  if (a.st->done) return;  // nothing to refine: the same in every workgroup
  const int tid = threadIdx.x;
  const double thresh = a.st->thresh;
  const int32_t maxit = a.st->maxit;
  double rho = a.st->rho[0], rr = a.st->rr, pq = 0.0;
  const GridShare<float> S = grid_setup(A, l, smem);
  int32_t ra[RPT], re[RPT];
  float x[RPT], r[RPT], p[RPT], dinv[RPT];
  if (S.ready) grid_window<false>(a.z, A.n, S, [&](int i, float v) { S.xs[i] = v; });
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int64_t row = S.r0 + tid + k * kGridBlock;
    ra[k] = re[k] = 0;
    x[k] = r[k] = p[k] = dinv[k] = 0.0f;
    if (S.ready && row < S.r1) {
      ra[k] = A.rowptr[row] - S.t0;
      re[k] = A.rowptr[row + 1] - S.t0;
      r[k] = a.r[row];
      p[k] = a.z[row];
      dinv[k] = a.dinv[row];
    }
  }
  uint32_t number = 0;
  int32_t status = SPX_OK, iters = 0;
  double bad[1] = {!S.ready && tid == 0 ? kGridBad : 0.0};
  // also keeps every workgroup's first reads of z ahead of the first stores
  if (!exchange(a.slots, ++number, l, bad))
    status = kGridTimedOut;
  else if (bad[0] != 0.0)
    status = kGridUnfit;
  if (status == SPX_OK) {
    for (int32_t k = 1;; ++k) {
      float q[RPT];
      double d[1] = {0.0};
#pragma unroll
      for (int u = 0; u < RPT; ++u) {
        q[u] = grid_row(S, ra[u], re[u]);
        d[0] += (double)p[u] * (double)q[u];
      }
      if (!exchange(a.slots, ++number, l, d)) {
        status = kGridTimedOut;
        break;
      }
      pq = d[0];
      if (!(pq > 0.0) || !isfinite(pq)) {
        status = SPX_BREAKDOWN;
        iters = k - 1;
        break;
      }
      const float alpha = (float)(rho / pq);
      float z[RPT];
      double g[2] = {0.0, 0.0};
#pragma unroll
      for (int u = 0; u < RPT; ++u) {
        const int64_t row = S.r0 + tid + u * kGridBlock;
        x[u] = x[u] + alpha * p[u];
        r[u] = r[u] - alpha * q[u];
        z[u] = dinv[u] * r[u];
        if (row < S.r1) agent_store(a.z + row, z[u]);
        g[0] += (double)r[u] * (double)z[u];
        g[1] += (double)r[u] * (double)r[u];
      }
      if (!exchange(a.slots, ++number, l, g)) {
        status = kGridTimedOut;
        break;
      }
      rr = g[1];
      iters = k;
      if (sqrt(rr) <= thresh) break;
      if (k >= maxit) {
        status = SPX_NOT_CONVERGED;
        break;
      }
      const float beta = (float)(g[0] / rho);
      rho = g[0];
#pragma unroll
      for (int u = 0; u < RPT; ++u) p[u] = z[u] + beta * p[u];
      grid_window<true>(a.z, A.n, S, [&](int i, float v) { S.xs[i] = v + beta * S.xs[i]; });
    }
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
      const int64_t row = S.r0 + tid + u * kGridBlock;
      if (row < S.r1) a.x[row] = x[u];
    }
  }
  if (tid == 0 && status == kGridTimedOut) a.st->verify = 1;
  if (tid == 0 && blockIdx.x == 0) {
    a.st->rho[0] = rho;
    a.st->pq = pq;
    a.st->rr = rr;
    a.st->iters = iters;
    a.st->status = status;
    a.st->done = 1;
  }
}

// Slots, and (st given) the scalars, of a new solve.
__global__ void k_grid_reset(CgScalars* st, unsigned long long* slots, int32_t maxit) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < kGridSlotWords;
       i += gridDim.x * blockDim.x)
    slots[i] = 0;
  if (st && blockIdx.x == 0 && threadIdx.x == 0) {
    CgScalars z = {};
    z.maxit = maxit;
    z.stop_pos = INT32_MAX;
    *st = z;
  }
}

// Rows per workgroup: as few as use every CU, but at least kGridMinRows
// (fewer workgroups exchange faster: 4,225 rows of a 9-point operator take
// 5.3 us an iteration with 64 rows each, 5.0 with 128 or 256; 2,744 rows of
// a 27-point one 6.7 with 64 or 128, 6.8 with 256).  A workgroup needs a CU
// to itself: its share takes most of the 160 KB.
constexpr int64_t kGridLds = 155 * 1024;
constexpr int64_t kGridMinRows = 128;
constexpr int kGridMaxRpt = 4;

struct GridPlan {
  int wgs, rows, entries, blocks, rpt;
  size_t lds;
};

template <typename VT>
bool grid_plan(const Csr& M, GridPlan* g) {
  if (M.n <= 0 || M.n > kGridMaxRows) return false;
  const int64_t wgs = std::min(cu_count(), kGridMaxWg);
  const int64_t rows = std::max(ceil_div(ceil_div(M.n, wgs), 32) * 32, kGridMinRows);
  if (rows > kGridMaxRpt * kGridBlock) return false;
  // no 32 rows hold more than tile_nnz[0] entries; even, for the alignment
  // of what follows them
  const int64_t entries = (rows / 32 * M.tile_nnz[0] + 1) & ~int64_t(1);
  const int64_t left = kGridLds - (int64_t)grid_lds_bytes<VT>(entries, 0);
  const int64_t blocks = std::min<int64_t>({left / (int64_t)grid_lds_bytes<VT>(0, 1), 1022,
                                            ceil_div(M.n, kWinBlock)});
  if (left <= 0 || blocks < 1) return false;
  g->rows = (int)rows;
  g->wgs = (int)ceil_div(M.n, rows);
  g->entries = (int)entries;
  g->blocks = (int)blocks;
  g->rpt = rows <= kGridBlock ? 1 : rows <= 2 * kGridBlock ? 2 : kGridMaxRpt;
  g->lds = grid_lds_bytes<VT>(entries, blocks);
  return true;
}

// Resets the slots (and *st when given) and launches fn on the plan's grid;
// *launched is false when the device refuses it.
template <typename VT, class Args>
int grid_launch(const GridPlan& g, const void* fn, GridMat<VT>& A, Args& a, CgScalars* st,
                int64_t maxit, hipStream_t s, bool* launched) {
  *launched = false;
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)g.lds) !=
      hipSuccess) {
    (void)hipGetLastError();
    return SPX_OK;
  }
  hipLaunchKernelGGL(k_grid_reset, dim3(16), dim3(256), 0, s, st,
                     reinterpret_cast<unsigned long long*>(a.slots), (int32_t)maxit);
  SPX_CHECK_HIP(hipGetLastError());
  void* args[] = {&A, &a};
  if (hipLaunchCooperativeKernel(fn, dim3((unsigned)g.wgs), dim3(kGridBlock), args, (unsigned)g.lds,
                                 s) != hipSuccess) {
    (void)hipGetLastError();  // not resident at once here: another form takes the solve
    return SPX_OK;
  }
  *launched = true;
  return SPX_OK;
}

// Whether a refused launch says something about the device, and not only that
// s is being captured.
bool refused_for_good(hipStream_t s) {
  hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
  const bool known = hipStreamIsCapturing(s, &c) == hipSuccess;
  (void)hipGetLastError();
  return known && c == hipStreamCaptureStatusNone;
}

}  // namespace

bool grid_cg_fits(const Csr& M, bool fp32) {
  GridPlan g;
  return fp32 ? !M.grid_unfit32 && grid_plan<float>(M, &g)
              : !M.grid_unfit && grid_plan<double>(M, &g);
}

int launch_grid_cg(const Csr& M, bool textbook, const double* b, double* x, double* u,
                   double* slots, CgScalars* st, double rtol, int64_t maxit, hipStream_t s,
                   bool* launched) {
  *launched = false;
  GridPlan g;
  if (!grid_plan<double>(M, &g)) return SPX_OK;
  GridMat<double> A{M.n, M.rowptr, M.col, M.val, g.rows, g.entries, g.blocks};
  GridSolve a{M.dpos, b, x, u, reinterpret_cast<Pair*>(slots), st, rtol, (int32_t)maxit};
  auto form = [&](auto t) {
    constexpr bool T = decltype(t)::value;
    return g.rpt == 1   ? reinterpret_cast<const void*>(&k_cg_grid<1, T>)
           : g.rpt == 2 ? reinterpret_cast<const void*>(&k_cg_grid<2, T>)
                        : reinterpret_cast<const void*>(&k_cg_grid<kGridMaxRpt, T>);
  };
  const void* fn = textbook ? form(std::true_type()) : form(std::false_type());
  SPX_TRY(grid_launch(g, fn, A, a, st, maxit, s, launched));
  if (!*launched && refused_for_good(s)) M.grid_unfit = true;
  return SPX_OK;
}

int launch_grid_inner(const Csr& M, float* x, const float* r, float* z, const float* dinv,
                      double* slots, CgScalars* st, hipStream_t s, bool* launched) {
  *launched = false;
  GridPlan g;
  if (!grid_plan<float>(M, &g)) return SPX_OK;
  GridMat<float> A{M.n, M.rowptr, M.col, M.val32, g.rows, g.entries, g.blocks};
  GridInner a{x, r, z, dinv, reinterpret_cast<Pair*>(slots), st};
  const void* fn = g.rpt == 1   ? reinterpret_cast<const void*>(&k_cg_grid_inner<1>)
                   : g.rpt == 2 ? reinterpret_cast<const void*>(&k_cg_grid_inner<2>)
                                : reinterpret_cast<const void*>(&k_cg_grid_inner<kGridMaxRpt>);
  SPX_TRY(grid_launch(g, fn, A, a, (CgScalars*)nullptr, 0, s, launched));
  if (!*launched && refused_for_good(s)) M.grid_unfit32 = true;
  return SPX_OK;
}

}  // namespace spx
