// Limited-memory BFGS product p = H_k g in the paper's intermediate dense
// form (Sec. 8, dense reformulations):
//   H_k g = [I, -S R^-T] [I 0; Y^T I] diag(H0, D) [I Y; 0 I] [I; -R^-1 S^T] g
// with R = triu(S^T Y), D = diag(S^T Y) and a diagonal base operator H0
// that may change from call to call.  Evaluated right to left:
//   c = -R^-1 (S^T g);  a = h0 (g + Y c);  f = Y^T a + D c;  e = R^-T f;
//   p = a - S e.
//
// Design for gfx950.  The passes stream the history once each and are bound
// by HBM.  S and Y are stored in tiles of kTileRows rows, a tile's m columns
// (the ring's slots) back to back, so a pass reads each tile as one
// contiguous stretch (51 KB at m = 50) and the grid sweeps the array from
// end to end.  The history is loaded past the caches' replacement
// (nontemporal: 7.0 TB/s against 6.2 for a plain sweep of 4 GB) and no load
// waits for another.  Stores among the loads cost far more than their bytes
// (80 MB stored during a 4 GB sweep take 120 us, where a copy of as much
// takes 35), so a new pair is stored by a kernel of its own (by the pass
// where the history is short) and a pass holds its results in LDS and stores
// many at once.
// n = 10^7, m = 50, one update and apply: 2685 us with S and Y as whole
// columns, 80 MB apart (S^T y and S^T g 894, a and Y^T a 918, p 789, the two
// solves 14 each, at 4.4-5.1 TB/s), 2180 so (728, 716, 658, 17 and 11; 592
// for S^T g alone with no new pair still on its way to memory).
//
// The m x m matrix of pair products s_a.y_b is kept by slot; R = triu(S^T
// Y) in time order only ever reads s_a.y_b with pair a no newer than pair
// b, so an update fills the new slot's column (s_b.y_new for every held b,
// the diagonal included) from one pass over S and never reads Y.  One apply
// is three passes over the rows (S^T g, taken in the update's pass where
// there is one; then a and Y^T a in one pass over Y; then p from S),
// separated by two one-workgroup kernels that add the pass's partials and
// solve the m x m triangular system, so no workgroup waits for another and
// no fence is needed.
#include <algorithm>
#include <cmath>
#include <new>

#include "common.hpp"
#include "device.hpp"

struct spx_lbfgs {
  int device = 0;
  int64_t n = 0;
  int64_t tiles = 0;
  int m = 0;
  int count = 0;  // pairs held
  int start = 0;  // slot of the oldest pair
  double* S = nullptr;   // [tiles][m][kTileRows]
  double* Y = nullptr;
  double* SY = nullptr;  // SY[a*m + b] = s_a . y_b, by slot
  double* P = nullptr;   // partials [3 kMaxHistory][workgroups of a pass]
  double* red = nullptr; // c[kMaxHistory] | e[kMaxHistory]
  double* a = nullptr;   // [tiles][kTileRows]
};

namespace spx {
namespace {

constexpr int kMaxHistory = 64;
// Up to this many pairs the pass over S stores the new one (us an update by a
// kernel of its own and so: n = 10^7, m = 3 108 and 94, m = 4 129 and 109; n =
// 1000 10 and 7.5), above it, more streams among the stores, that takes
// longer (a step at m = 6, n = 10^7 427 and 439, at m = 5, n = 5 x 10^5 38.1
// and 39.1; m = 50 below).
constexpr int kPutInPass = 4;
constexpr int kLB = 256;
constexpr int kWaves = kLB / 64;
constexpr int kTileRows = 128;  // two rows per lane, 16-byte loads
// Tiles of results held in LDS, by columns per wave: half a CU's LDS with the
// parts of k_lb_ya, or less where eight workgroups share it.
constexpr int hold_tiles(int nc) { return nc <= 2 ? 8 : 72; }
constexpr int kWaveCols = kMaxHistory / kWaves;
constexpr int kSolve = 1024;  // threads of the reduce-and-solve kernels
constexpr int kRStride = kMaxHistory + 1;  // R in LDS, rows and columns both read by lane

typedef double dbl2 __attribute__((ext_vector_type(2)));

// The ring: logical pair b (oldest first) lives in slot start + b (mod m).
struct Ring {
  int m, start, cnt;
  __device__ __forceinline__ int slot(int b) const {
    const int s = start + b;
    return s >= m ? s - m : s;
  }
};

// Rows r and r + 1 of a caller's vector of any alignment, 0 at n and beyond.
// Without branches: a load under one makes the next wait for it.
__device__ __forceinline__ dbl2 load2(const double* __restrict__ p, int64_t r, int64_t n) {
  const double x = p[r < n ? r : n - 1], y = p[r + 1 < n ? r + 1 : n - 1];
  return dbl2{r < n ? x : 0.0, r + 1 < n ? y : 0.0};
}
// wide: the vector is 16-byte aligned and all of the tile's rows are below n.
__device__ __forceinline__ void store2(double* __restrict__ p, int64_t r, int64_t n, bool wide,
                                       dbl2 v) {
  if (wide) {
    *reinterpret_cast<dbl2*>(p + r) = v;
  } else {
    if (r < n) p[r] = v.x;
    if (r + 1 < n) p[r + 1] = v.y;
  }
}
inline __host__ __device__ bool is_wide(const void* p) {
  return (reinterpret_cast<uintptr_t>(p) & 15) == 0;
}

// Two rows of the history, read once a pass and far larger than the caches.
__device__ __forceinline__ dbl2 load_once(const double* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const dbl2*>(p));
}

// One wave's share of the ring's columns: logical columns lo .. lo + nc (NC - kWaves
// <= nc <= NC, so only the last kWaves places ask whether they hold one) and
// the offset of each in a tile.
template <int NC>
struct Cols {
  int lo, nc;
  int newest;  // place of the newest pair's column, or -1
  int off[NC];
  __device__ __forceinline__ Cols(const Ring& R, int w) {
    lo = R.cnt * w / kWaves;
    nc = R.cnt * (w + 1) / kWaves - lo;
    newest = lo + nc == R.cnt && nc > 0 ? nc - 1 : -1;
#pragma unroll
    for (int u = 0; u < NC; ++u) off[u] = R.slot(lo + u) * kTileRows;
  }
  __device__ __forceinline__ bool has(int u) const { return u < NC - kWaves || u < nc; }
  // The tile's rows of the share, 0 for a place that holds no column.
  __device__ __forceinline__ void load(dbl2 (&c)[NC], const double* tile) const {
#pragma unroll
    for (int u = 0; u < NC; ++u) {
      c[u] = dbl2{0.0, 0.0};
      if (has(u)) c[u] = load_once(tile + off[u]);
    }
  }
};

// ------------------------------------------------------------ the new pair
// Stores s and y in slot `slot` of every tile; a wave per tile.  On its own
// rather than in the pass over S that follows: at n = 10^7 this takes 50 us
// and the pass 728, and the pass with these stores in it 840.
__global__ __launch_bounds__(kLB) void k_lb_put(int64_t n, int64_t tiles, int m, int slot,
                                                const double* __restrict__ s,
                                                const double* __restrict__ y,
                                                double* __restrict__ S, double* __restrict__ Y) {
  const int64_t t = (int64_t)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (t >= tiles) return;
  const int lane = threadIdx.x & 63;
  const int64_t r = t * kTileRows + 2 * lane;
  const int64_t o = (t * m + slot) * kTileRows + 2 * lane;
  const dbl2 sv = load2(s, r, n), yv = load2(y, r, n);
  *reinterpret_cast<dbl2*>(S + o) = sv;
  *reinterpret_cast<dbl2*>(Y + o) = yv;
}

// ------------------------------------------------- transposed products
// Partials of s_b . w1 (row row1 + b of P) and, with BOTH, of s_b . w2 (row
// row2 + b) over the workgroup's tiles, for the ring's columns.  Each wave
// takes a quarter of the columns of every tile, all of a step's loads in
// flight together, so every element of the history is read once and w1 and
// w2 once per workgroup.  Every column's products are added in the same
// order with and without BOTH.  PUT: the newest pair is (s, w1) and not yet
// stored; the wave that has its column takes it from s and stores both.
template <int NC, bool BOTH, bool PUT>
__global__ __launch_bounds__(kLB) void k_lb_dots(int64_t n, int64_t tiles, double* __restrict__ S,
                                                 double* __restrict__ Y, Ring R,
                                                 const double* __restrict__ s,
                                                 const double* __restrict__ w1,
                                                 const double* __restrict__ w2,
                                                 double* __restrict__ P, int row1, int row2) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const Cols<NC> C(R, w);
  double acc[NC], acc2[BOTH ? NC : 1];
#pragma unroll
  for (int u = 0; u < NC; ++u) {
    acc[u] = 0.0;
    if constexpr (BOTH) acc2[u] = 0.0;
  }
  for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
    const int64_t r = t * kTileRows + 2 * lane;
    const dbl2 v = load2(w1, r, n);
    dbl2 v2 = {0.0, 0.0};
    if constexpr (BOTH) v2 = load2(w2, r, n);
    dbl2 c[NC];
    const int64_t o = t * R.m * kTileRows + 2 * lane;
    if constexpr (PUT) {
      dbl2 sv = {0.0, 0.0};
      if (C.newest >= 0) sv = load2(s, r, n);
#pragma unroll
      for (int u = 0; u < NC; ++u) {
        c[u] = dbl2{0.0, 0.0};
        if (C.has(u) && u != C.newest) c[u] = load_once(S + o + C.off[u]);
        if (u == C.newest) {
          c[u] = sv;
          *reinterpret_cast<dbl2*>(S + o + C.off[u]) = sv;
          *reinterpret_cast<dbl2*>(Y + o + C.off[u]) = v;
        }
      }
    } else {
      C.load(c, S + o);
    }
#pragma unroll
    for (int u = 0; u < NC; ++u) {
      acc[u] += c[u].x * v.x;
      acc[u] += c[u].y * v.y;
      if constexpr (BOTH) {
        acc2[u] += c[u].x * v2.x;
        acc2[u] += c[u].y * v2.y;
      }
    }
  }
  const int64_t G = gridDim.x, b = blockIdx.x;
#pragma unroll
  for (int u = 0; u < NC; ++u) {
    if (C.has(u)) {
      const double d = wave_sum(acc[u]);
      if (lane == 0) P[(row1 + C.lo + u) * G + b] = d;
      if constexpr (BOTH) {
        const double d2 = wave_sum(acc2[u]);
        if (lane == 0) P[(row2 + C.lo + u) * G + b] = d2;
      }
    }
  }
}

// ------------------------------------------------------ a and Y^T a
// a = h0 (g + Y c), c in red[0 ..), and the partials of f_b = y_b . a (row b
// of P) in one pass over Y: each wave holds its quarter of the columns of a
// tile in registers, the four waves' parts of Y c meet in LDS, and every
// wave adds its columns' products with the tile's a.  a is held in LDS and
// stored several tiles at a time (716 us against 749 stored tile by tile).
template <int NC, bool H0>
__global__ __launch_bounds__(kLB) void k_lb_ya(int64_t n, int64_t tiles,
                                               const double* __restrict__ Y, Ring R,
                                               const double* __restrict__ g,
                                               const double* __restrict__ h0,
                                               const double* __restrict__ red,
                                               double* __restrict__ a_out,
                                               double* __restrict__ P) {
  __shared__ dbl2 part[2][kWaves][64];
  constexpr int kHold = hold_tiles(NC);
  __shared__ dbl2 hold[kHold][64];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const Cols<NC> C(R, w);
  double f[NC], c[NC];
#pragma unroll
  for (int u = 0; u < NC; ++u) {
    f[u] = 0.0;
    c[u] = C.has(u) ? red[C.lo + u] : 0.0;
  }
  int buf = 0, held = 0;
  int64_t first = blockIdx.x;  // the tile of hold[0]
  for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x, buf ^= 1) {
    const int64_t r = t * kTileRows + 2 * lane;
    const dbl2 gv = load2(g, r, n);
    dbl2 hv = {1.0, 1.0};
    if constexpr (H0) hv = load2(h0, r, n);
    dbl2 y[NC];
    C.load(y, Y + t * R.m * kTileRows + 2 * lane);
    dbl2 s = {0.0, 0.0};
#pragma unroll
    for (int u = 0; u < NC; ++u) s += y[u] * c[u];
    part[buf][w][lane] = s;
    __syncthreads();
    dbl2 a = gv;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) a += part[buf][q][lane];
    if constexpr (H0) a = hv * a;
    // no row at n and beyond: 0 times an infinite c is not 0
    a = dbl2{r < n ? a.x : 0.0, r + 1 < n ? a.y : 0.0};
    // a place of hold belongs to one wave, which fills and empties it
    if (w == (held & (kWaves - 1))) hold[held][lane] = a;
    if (++held == kHold || t + gridDim.x >= tiles) {
      for (int i = w; i < held; i += kWaves)
        *reinterpret_cast<dbl2*>(a_out + (first + (int64_t)i * gridDim.x) * kTileRows + 2 * lane) =
            hold[i][lane];
      first = t + gridDim.x;
      held = 0;
    }
#pragma unroll
    for (int u = 0; u < NC; ++u) {
      f[u] += y[u].x * a.x;
      f[u] += y[u].y * a.y;
    }
  }
#pragma unroll
  for (int u = 0; u < NC; ++u) {
    if (C.has(u)) {
      const double d = wave_sum(f[u]);
      if (lane == 0) P[(int64_t)(C.lo + u) * gridDim.x + blockIdx.x] = d;
    }
  }
}

// --------------------------------------------------- one or two columns
// The same two passes where a quarter of the columns would leave waves
// without any: a wave per tile with all NC = cnt columns, which keeps four
// times as many bytes in flight and needs no exchange between waves.  NC = 1,
// n = 10^7, a step of 228 us with whole columns, 247 with those waves idle,
// 182 so (NC = 2 301, 270 and 226).
template <int NC>
__device__ __forceinline__ void few_partials(double (&v)[NC], double* __restrict__ P, int row) {
  __shared__ double part[NC][kWaves];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int u = 0; u < NC; ++u) {
    const double d = wave_sum(v[u]);
    if (lane == 0) part[u][w] = d;
  }
  __syncthreads();
  if (threadIdx.x < NC) {
    double d = 0.0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) d += part[threadIdx.x][q];
    P[(int64_t)(row + threadIdx.x) * gridDim.x + blockIdx.x] = d;
  }
  __syncthreads();
}

template <int NC, bool BOTH, bool PUT>
__global__ __launch_bounds__(kLB) void k_lb_few_dots(int64_t n, int64_t tiles,
                                                     double* __restrict__ S, double* __restrict__ Y,
                                                     Ring R, const double* __restrict__ s,
                                                     const double* __restrict__ w1,
                                                     const double* __restrict__ w2,
                                                     double* __restrict__ P, int row1, int row2) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  double acc[NC] = {}, acc2[NC] = {};
  for (int64_t t = (int64_t)blockIdx.x * kWaves + w; t < tiles; t += (int64_t)gridDim.x * kWaves) {
    const int64_t r = t * kTileRows + 2 * lane;
    const dbl2 v = load2(w1, r, n);
    dbl2 v2 = {0.0, 0.0}, c[NC];
    if constexpr (BOTH) v2 = load2(w2, r, n);
    const int64_t o = t * R.m * kTileRows + 2 * lane;
#pragma unroll
    for (int u = 0; u < NC; ++u) {
      if (PUT && u == NC - 1)
        c[u] = load2(s, r, n);
      else
        c[u] = load_once(S + o + R.slot(u) * kTileRows);
    }
    if constexpr (PUT) {
      *reinterpret_cast<dbl2*>(S + o + R.slot(NC - 1) * kTileRows) = c[NC - 1];
      *reinterpret_cast<dbl2*>(Y + o + R.slot(NC - 1) * kTileRows) = v;
    }
#pragma unroll
    for (int u = 0; u < NC; ++u) {
      acc[u] += c[u].x * v.x;
      acc[u] += c[u].y * v.y;
      if constexpr (BOTH) {
        acc2[u] += c[u].x * v2.x;
        acc2[u] += c[u].y * v2.y;
      }
    }
  }
  few_partials<NC>(acc, P, row1);
  if constexpr (BOTH) few_partials<NC>(acc2, P, row2);
}

template <int NC, bool H0>
__global__ __launch_bounds__(kLB) void k_lb_few_ya(int64_t n, int64_t tiles,
                                                   const double* __restrict__ Y, Ring R,
                                                   const double* __restrict__ g,
                                                   const double* __restrict__ h0,
                                                   const double* __restrict__ red,
                                                   double* __restrict__ a_out,
                                                   double* __restrict__ P) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  double f[NC] = {}, c[NC];
#pragma unroll
  for (int u = 0; u < NC; ++u) c[u] = red[u];
  for (int64_t t = (int64_t)blockIdx.x * kWaves + w; t < tiles; t += (int64_t)gridDim.x * kWaves) {
    const int64_t r = t * kTileRows + 2 * lane;
    const dbl2 gv = load2(g, r, n);
    dbl2 hv = {1.0, 1.0}, y[NC];
    if constexpr (H0) hv = load2(h0, r, n);
#pragma unroll
    for (int u = 0; u < NC; ++u)
      y[u] = load_once(Y + t * R.m * kTileRows + 2 * lane + R.slot(u) * kTileRows);
    dbl2 a = {0.0, 0.0};
#pragma unroll
    for (int u = 0; u < NC; ++u) a += y[u] * c[u];
    a = gv + a;
    if constexpr (H0) a = hv * a;
    a = dbl2{r < n ? a.x : 0.0, r + 1 < n ? a.y : 0.0};
    *reinterpret_cast<dbl2*>(a_out + t * kTileRows + 2 * lane) = a;
#pragma unroll
    for (int u = 0; u < NC; ++u) {
      f[u] += y[u].x * a.x;
      f[u] += y[u].y * a.y;
    }
  }
  few_partials<NC>(f, P, 0);
}

// ------------------------------------------------------------ p = a - S e
// e in red[kMaxHistory ..): a wave per tile, kPU columns' loads in flight; p
// is held in LDS and stored several tiles at a time (658 us against 702
// stored tile by tile).  S e is summed before a, which mostly outweighs it, is
// added.
constexpr int kPU = 8;
template <int NC>
__global__ __launch_bounds__(kLB) void k_lb_p(int64_t n, int64_t tiles, const double* __restrict__ S,
                                              Ring R, const double* __restrict__ a,
                                              const double* __restrict__ red,
                                              double* __restrict__ p) {
  constexpr int kHeld = hold_tiles(NC) / kWaves;
  __shared__ dbl2 hold[kWaves][kHeld][64];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const double* e = red + kMaxHistory;
  const bool wp = is_wide(p);
  const int cnt = R.cnt;
  const int64_t step = (int64_t)gridDim.x * kWaves;
  int64_t first = (int64_t)blockIdx.x * kWaves + w;
  int held = 0;
  for (int64_t t = first; t < tiles; t += step) {
    const double* tile = S + t * R.m * kTileRows + 2 * lane;
    const dbl2 av = *reinterpret_cast<const dbl2*>(a + t * kTileRows + 2 * lane);
    dbl2 v = {0.0, 0.0};
    for (int b = 0; b < cnt; b += kPU) {
      dbl2 c[kPU];
#pragma unroll
      for (int u = 0; u < kPU; ++u) {
        c[u] = dbl2{0.0, 0.0};
        if (b + u < cnt) c[u] = load_once(tile + R.slot(b + u) * kTileRows);
      }
#pragma unroll
      for (int u = 0; u < kPU; ++u) v += c[u] * (b + u < cnt ? e[b + u] : 0.0);
    }
    hold[w][held][lane] = av - v;
    if (++held == kHeld || t + step >= tiles) {
      for (int i = 0; i < held; ++i) {
        const int64_t q = first + i * step;
        store2(p, q * kTileRows + 2 * lane, n, wp && (q + 1) * kTileRows <= n, hold[w][i][lane]);
      }
      first = t + step;
      held = 0;
    }
  }
}

// ------------------------------------------------------ sums and solves
// Row sums of P's rows row .. row + cnt over the G partials, into out (LDS):
// a wave per row, two rows' loads in flight.
__device__ __forceinline__ void row_sums(const double* __restrict__ P, int64_t G, int row, int cnt,
                                         double* out) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  constexpr int U = 12, W = kSolve / 64;
  for (int b = w; b < cnt; b += 2 * W) {
    const int b2 = b + W < cnt ? b + W : b;
    const double* p = P + (row + b) * G;
    const double* p2 = P + (row + b2) * G;
    double s = 0.0, s2 = 0.0;
    for (int64_t i0 = lane; i0 < G; i0 += 64 * U) {
      double v[U], v2[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t i = i0 + 64 * u < G ? i0 + 64 * u : 0;
        v[u] = p[i];
        v2[u] = p2[i];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (i0 + 64 * u < G) {
          s += v[u];
          s2 += v2[u];
        }
      }
    }
    s = wave_sum(s);
    s2 = wave_sum(s2);
    if (lane == 0) {
      out[b] = s;
      out[b2] = s2;
    }
  }
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), lane);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// One triangular solve in a wave: lane x holds row x's right-hand side t and
// diagonal entry d; the unknowns are finished from lane cnt - 1 down (UP
// false) or from lane 0 up, and step y takes r[y * step] times the finished
// unknown from the lanes still open.  Returns unknown x.  The quotients are
// those of the reciprocal, taken beforehand, corrected by their remainder;
// EXACT divides, and is for the systems where that is not finite.
template <bool UP, bool EXACT>
__device__ __forceinline__ double tri_solve(double t, double d, const double* r, int step, int cnt) {
  const int x = threadIdx.x;
  const double inv = 1.0 / d;
  auto unknown = [&]() {
    if constexpr (EXACT) return t / d;
    const double q = t * inv;
    return fma(fma(-q, d, t), inv, q);
  };
  int y = UP ? 0 : cnt - 1;
  double a = r[y * step];
  for (int i = 0; i < cnt; ++i) {
    const int ny = UP ? min(y + 1, cnt - 1) : max(y - 1, 0);
    const double next = r[ny * step];
    const double uy = lane_value(unknown(), y);
    const double u = t - a * uy;
    if (UP ? x > y : x < y) t = u;
    a = next;
    y = ny;
  }
  return unknown();
}

// Adds a pass's partials and does what follows, R = triu(S^T Y) in the
// ring's logical order:
//   UPDATE: the new slot's column of SY from rows kMaxHistory + b;
//   SOLVE 1: q from rows q_row + b, then c = -R^-1 q into red[0 ..);
//   SOLVE 2: f from rows b, then e = R^-T (f + D c) into red[kMaxHistory ..).
// One workgroup stages R in LDS; one wave then sweeps the columns: lane x
// holds row x's running sum, and at step y every lane takes the finished
// unknown y and lanes still open subtract their entry of column y times it
// (cnt <= 64 lanes).
template <bool UPDATE, int SOLVE>
__global__ __launch_bounds__(kSolve) void k_lb_solve(const double* __restrict__ P, int64_t G, Ring R,
                                                     int q_row, double* __restrict__ SY,
                                                     double* __restrict__ red) {
  __shared__ double rl[kMaxHistory * kRStride];
  __shared__ double v[kMaxHistory];
  __shared__ double q[kMaxHistory];
  const int cnt = R.cnt, tid = threadIdx.x;
  // entries (a0 + i kSolve / 64, b) of R and, for SOLVE 2, c_b
  const int a0 = tid >> 6, b = tid & 63;
  constexpr int kA = SOLVE == 0 ? 1 : kMaxHistory / (kSolve / 64);
  double sy[kA], cb = 0.0;
  if constexpr (SOLVE != 0) {
#pragma unroll
    for (int i = 0; i < kA; ++i) {
      const int a = min(a0 + i * (kSolve / 64), cnt - 1);
      sy[i] = SY[R.slot(a) * R.m + R.slot(min(b, cnt - 1))];
    }
    if constexpr (SOLVE == 2) cb = red[min(b, cnt - 1)];
  }
  if constexpr (UPDATE) row_sums(P, G, kMaxHistory, cnt, v);
  if constexpr (SOLVE != 0) {
    row_sums(P, G, q_row, cnt, q);
#pragma unroll
    for (int i = 0; i < kA; ++i) {
      const int a = a0 + i * (kSolve / 64);
      // the new column comes from v
      if (a <= b && b < cnt && !(UPDATE && b == cnt - 1)) rl[a * kRStride + b] = sy[i];
    }
  }
  __syncthreads();
  if constexpr (UPDATE) {
    if (tid < cnt) {
      SY[R.slot(tid) * R.m + R.slot(cnt - 1)] = v[tid];
      if constexpr (SOLVE != 0) rl[tid * kRStride + cnt - 1] = v[tid];
    }
    __syncthreads();
  }
  if (SOLVE == 0 || tid >= 64) return;
  const int x = tid;
  const double d = x < cnt ? rl[x * kRStride + x] : 1.0;
  if constexpr (SOLVE == 1) {
    const double t = x < cnt ? -q[x] : 0.0;
    double u = tri_solve<false, false>(t, d, rl + x * kRStride, 1, cnt);
    if (__ballot(x < cnt && !__builtin_isfinite(u)))
      u = tri_solve<false, true>(t, d, rl + x * kRStride, 1, cnt);
    if (x < cnt) red[x] = u;
  } else {
    const double t = x < cnt ? q[x] + d * cb : 0.0;
    double u = tri_solve<true, false>(t, d, rl + x, kRStride, cnt);
    if (__ballot(x < cnt && !__builtin_isfinite(u)))
      u = tri_solve<true, true>(t, d, rl + x, kRStride, cnt);
    if (x < cnt) red[kMaxHistory + x] = u;
  }
}

__global__ void k_lb_scale(int64_t n, const double* __restrict__ g, const double* __restrict__ h0,
                           double* __restrict__ p) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = (h0 ? h0[i] : 1.0) * g[i];
}

// Workgroups of the passes over cnt columns.  Two per CU: at m = 50 their
// loads in flight (12 KB a wave) cover the memory's latency, and more make the
// sums longer for nothing (the solves 11 and 17 us against 16 and 22 with
// four; m = 16, n = 10^7, a step of 844 us against 888 with eight).  Up to 8
// columns are too few bytes in flight for that, where the pass is long enough
// for the sums not to matter: m = 3, n = 10^7 413 us with two per CU and 310
// with eight (370 with whole columns), n = 10^6 54 and 46; n = 10^5 22 and 24.
unsigned blocks(const spx_lbfgs* h, int cnt) {
  const int64_t per_cu = cnt <= 2 * kWaves && h->tiles >= 4096 ? 8 : 2;
  return (unsigned)std::min<int64_t>(h->tiles, per_cu * cu_count());
}

// Calls f with the smallest of 2, 4, 8, 12 and 16 columns per wave that hold a
// quarter of cnt.
template <typename F>
void with_cols(int cnt, F&& f) {
  const int nc = (cnt + kWaves - 1) / kWaves;
  if (nc <= 2)
    f(std::integral_constant<int, 2>());
  else if (nc <= 4)
    f(std::integral_constant<int, 4>());
  else if (nc <= 8)
    f(std::integral_constant<int, 8>());
  else if (nc <= 12)
    f(std::integral_constant<int, 12>());
  else
    f(std::integral_constant<int, kWaveCols>());
}

}  // namespace
}  // namespace spx

using namespace spx;

namespace {
// The apply.  With have_q the partials of S^T g are already in rows 2
// kMaxHistory + b of the workspace, and those of the new column of SY in
// rows kMaxHistory + b (left there by the update's pass).
int apply_passes(spx_lbfgs* h, const double* g, const double* h0, double* p, hipStream_t st,
                 bool have_q) {
  const int64_t n = h->n;
  const unsigned G = blocks(h, h->count);
  const Ring R{h->m, h->start, h->count};
  const double* none = nullptr;
  if (have_q) {
    hipLaunchKernelGGL((k_lb_solve<true, 1>), dim3(1), dim3(kSolve), 0, st, h->P, (int64_t)G, R,
                       2 * kMaxHistory, h->SY, h->red);
  } else {
    auto dots = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(G), dim3(kLB), 0, st, n, h->tiles, h->S, h->Y, R, none, g, none,
                         h->P, 0, 0);
    };
    if (R.cnt == 1)
      dots(k_lb_few_dots<1, false, false>);
    else if (R.cnt == 2)
      dots(k_lb_few_dots<2, false, false>);
    else
      with_cols(R.cnt, [&](auto nc) { dots(k_lb_dots<decltype(nc)::value, false, false>); });
    hipLaunchKernelGGL((k_lb_solve<false, 1>), dim3(1), dim3(kSolve), 0, st, h->P, (int64_t)G, R, 0,
                       h->SY, h->red);
  }
  auto ya = [&](auto with_h0, auto without) {
    hipLaunchKernelGGL(h0 ? with_h0 : without, dim3(G), dim3(kLB), 0, st, n, h->tiles, h->Y, R, g, h0,
                       h->red, h->a, h->P);
  };
  if (R.cnt == 1)
    ya(k_lb_few_ya<1, true>, k_lb_few_ya<1, false>);
  else if (R.cnt == 2)
    ya(k_lb_few_ya<2, true>, k_lb_few_ya<2, false>);
  else
    with_cols(R.cnt, [&](auto nc) {
      constexpr int NC = decltype(nc)::value;
      ya(k_lb_ya<NC, true>, k_lb_ya<NC, false>);
    });
  hipLaunchKernelGGL((k_lb_solve<false, 2>), dim3(1), dim3(kSolve), 0, st, h->P, (int64_t)G, R, 0,
                     h->SY, h->red);
  with_cols(R.cnt, [&](auto nc) {
    hipLaunchKernelGGL(k_lb_p<decltype(nc)::value>, dim3(G), dim3(kLB), 0, st, n, h->tiles, h->S, R,
                       h->a, h->red, p);
  });
  return SPX_OK;
}
}  // namespace

extern "C" int spx_lbfgs_create(int64_t n, int32_t m, void* stream, spx_lbfgs_handle* out) {
  clear_error();
  if (!out) return set_error(SPX_INVALID_ARG, "lbfgs_create: out is NULL");
  *out = nullptr;
  if (n <= 0 || m < 1 || m > kMaxHistory)
    return set_error(SPX_INVALID_ARG, "lbfgs_create: need n > 0 and 1 <= m <= %d", kMaxHistory);
  (void)stream;
  spx_lbfgs* h = new (std::nothrow) spx_lbfgs();
  if (!h) return set_error(SPX_OUT_OF_MEMORY, "lbfgs_create: host allocation failed");
  (void)hipGetDevice(&h->device);
  h->n = n;
  h->m = m;
  h->tiles = ceil_div(n, kTileRows);
  const size_t rows = (size_t)h->tiles * kTileRows;
  int st = SPX_OK;
  do {
    if ((st = dalloc_n(&h->S, rows * m)) != SPX_OK) break;
    if ((st = dalloc_n(&h->Y, rows * m)) != SPX_OK) break;
    if ((st = dalloc_n(&h->SY, (size_t)m * m)) != SPX_OK) break;
    if ((st = dalloc_n(&h->P, (size_t)3 * kMaxHistory * blocks(h, 1))) != SPX_OK) break;
    if ((st = dalloc_n(&h->red, (size_t)2 * kMaxHistory)) != SPX_OK) break;
    if ((st = dalloc_n(&h->a, rows)) != SPX_OK) break;
  } while (false);
  if (st != SPX_OK) {
    spx_lbfgs_destroy(h);
    return st;
  }
  *out = h;
  return SPX_OK;
}

extern "C" int spx_lbfgs_destroy(spx_lbfgs_handle h) {
  clear_error();
  if (!h) return SPX_OK;
  dfree(h->S);
  dfree(h->Y);
  dfree(h->SY);
  dfree(h->P);
  dfree(h->red);
  dfree(h->a);
  delete h;
  return SPX_OK;
}

extern "C" int spx_lbfgs_reset(spx_lbfgs_handle h) {
  clear_error();
  if (!h) return set_error(SPX_INVALID_ARG, "lbfgs_reset: NULL handle");
  h->count = 0;
  h->start = 0;
  return SPX_OK;
}

extern "C" int spx_lbfgs_get_info(spx_lbfgs_handle h, int64_t* n, int32_t* m, int32_t* count) {
  clear_error();
  if (!h) return set_error(SPX_INVALID_ARG, "lbfgs_get_info: NULL handle");
  if (n) *n = h->n;
  if (m) *m = h->m;
  if (count) *count = h->count;
  return SPX_OK;
}

namespace {
// The update's pass; with g (non-NULL) it also leaves the partials of S^T g
// for the apply that follows, and the new column of SY to that apply.
int update_impl(spx_lbfgs* h, const double* s, const double* y, const double* g,
                hipStream_t st) {
  int slot, start, cnt;
  if (h->count < h->m) {
    slot = (h->start + h->count) % h->m;
    start = h->start;
    cnt = h->count + 1;
  } else {
    slot = h->start;  // the oldest pair leaves
    start = (h->start + 1) % h->m;
    cnt = h->m;
  }
  const unsigned G = blocks(h, cnt);
  const Ring R{h->m, start, cnt};
  const bool put = cnt > kPutInPass;
  if (put)
    hipLaunchKernelGGL(k_lb_put, dim3((unsigned)ceil_div(h->tiles, kWaves)), dim3(kLB), 0, st, h->n,
                       h->tiles, h->m, slot, s, y, h->S, h->Y);
  auto dots = [&](auto kernel, int row2) {
    hipLaunchKernelGGL(kernel, dim3(G), dim3(kLB), 0, st, h->n, h->tiles, h->S, h->Y, R, s, y, g, h->P,
                       kMaxHistory, row2);
  };
  if (put) {
    with_cols(cnt, [&](auto nc) {
      constexpr int NC = decltype(nc)::value;
      if (g)
        dots(k_lb_dots<NC, true, false>, 2 * kMaxHistory);
      else
        dots(k_lb_dots<NC, false, false>, 0);
    });
  } else {
    auto either = [&](auto both, auto alone) {
      if (g)
        dots(both, 2 * kMaxHistory);
      else
        dots(alone, 0);
    };
    if (cnt == 1)
      either(k_lb_few_dots<1, true, true>, k_lb_few_dots<1, false, true>);
    else if (cnt == 2)
      either(k_lb_few_dots<2, true, true>, k_lb_few_dots<2, false, true>);
    else
      either(k_lb_dots<2, true, true>, k_lb_dots<2, false, true>);
  }
  if (!g)
    hipLaunchKernelGGL((k_lb_solve<true, 0>), dim3(1), dim3(kSolve), 0, st, h->P, (int64_t)G, R, 0,
                       h->SY, h->red);
  SPX_CHECK_HIP(hipGetLastError());
  h->start = start;
  h->count = cnt;
  return SPX_OK;
}
}  // namespace

extern "C" int spx_lbfgs_update(spx_lbfgs_handle h, const double* s, const double* y,
                                void* stream) {
  clear_error();
  if (!h || !s || !y) return set_error(SPX_INVALID_ARG, "lbfgs_update: NULL argument");
  return update_impl(h, s, y, nullptr, static_cast<hipStream_t>(stream));
}

extern "C" int spx_lbfgs_update_apply(spx_lbfgs_handle h, const double* s, const double* y,
                                      const double* g, const double* h0, double* p,
                                      void* stream) {
  clear_error();
  if (!h || !s || !y || !g || !p)
    return set_error(SPX_INVALID_ARG, "lbfgs_update_apply: NULL argument");
  if (p == g) return set_error(SPX_INVALID_ARG, "lbfgs_update_apply: p must not alias g");
  hipStream_t st = static_cast<hipStream_t>(stream);
  SPX_TRY(update_impl(h, s, y, g, st));
  SPX_TRY(apply_passes(h, g, h0, p, st, true));
  SPX_CHECK_HIP(hipGetLastError());
  return SPX_OK;
}

extern "C" int spx_lbfgs_apply(spx_lbfgs_handle h, const double* g, const double* h0, double* p,
                               void* stream) {
  clear_error();
  if (!h || !g || !p) return set_error(SPX_INVALID_ARG, "lbfgs_apply: NULL argument");
  if (p == g) return set_error(SPX_INVALID_ARG, "lbfgs_apply: p must not alias g");
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int64_t n = h->n;
  const int cnt = h->count;
  if (cnt == 0) {
    hipLaunchKernelGGL(k_lb_scale, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, n, g, h0, p);
    SPX_CHECK_HIP(hipGetLastError());
    return SPX_OK;
  }
  SPX_TRY(apply_passes(h, g, h0, p, st, false));
  SPX_CHECK_HIP(hipGetLastError());
  return SPX_OK;
}
