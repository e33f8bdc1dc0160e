// COO -> CSR assembly on the device (paper Sec. 5, "Portable matrix assembly
// on GPUs"): a symbolic stage that turns the index arrays into a CSR pattern
// plus the jmap/perm maps, and a numeric stage in which one thread owns one
// stored entry and sums its contributions in input order (no atomics).
#include <algorithm>
#include <new>

#include "common.hpp"
#include "device.hpp"

namespace spx {

namespace {

constexpr int kBlock = 256;
constexpr int kIpt = 8;
constexpr int64_t kTile = kBlock * kIpt;
// Tile of the row stage: the items it starts from and the most it holds.
constexpr int64_t kRowTile = 512;  // 1024 measured slower (5.55 vs 5.3 ms at 131M items)
constexpr int kRowCap = 1024;

__device__ __forceinline__ uint32_t block_exscan(uint32_t v, uint32_t* lds_wave, uint32_t* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t inc = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    uint32_t t = __shfl_up(inc, off, 64);
    if (lane >= off) inc += t;
  }
  if (lane == 63) lds_wave[w] = inc;
  __syncthreads();
  uint32_t wave_off = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < kBlock / 64; ++i) {
    uint32_t c = lds_wave[i];
    if (i < w) wave_off += c;
    tot += c;
  }
  __syncthreads();
  if (total) *total = tot;
  return wave_off + inc - v;
}

__global__ void k_fill_i32(int32_t* p, int64_t count, int32_t value) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < count) p[t] = value;
}

__global__ void k_fill_f64(double* p, int64_t count, double value) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < count) p[t] = value;
}

// Triplets k .. k + kIpt of p (those at ncoo and beyond -1): two 16-byte
// loads where p is aligned and the range whole.
typedef int32_t int4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void load_ipt(const int32_t* __restrict__ p, int64_t k, int64_t ncoo,
                                         bool aligned, int32_t (&a)[kIpt]) {
  static_assert(kIpt == 8, "two vectors");
  if (aligned && k + kIpt <= ncoo) {
    const int4v x = *reinterpret_cast<const int4v*>(p + k);
    const int4v y = *reinterpret_cast<const int4v*>(p + k + 4);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a[u] = x[u];
      a[4 + u] = y[u];
    }
  } else {
#pragma unroll
    for (int u = 0; u < kIpt; ++u) a[u] = k + u < ncoo ? p[k + u] : -1;
  }
}

// The row before triplet k, given this thread's rows from k on (k a
// multiple of kIpt, threads in order): the lane before has it.
__device__ __forceinline__ int32_t row_before(const int32_t* __restrict__ i, int64_t k,
                                              int64_t ncoo, const int32_t (&a)[kIpt]) {
  const int32_t up = __shfl_up(a[kIpt - 1], 1, 64);
  return (threadIdx.x & 63) != 0 ? up : k > 0 && k < ncoo ? i[k - 1] : -1;
}

// Per tile of kTile triplets: number of kept triplets in cnt[tile] and of
// triplets whose row differs from the one before in cnt[ntiles + tile] (the
// runs of equal rows, when every triplet is kept); flags indices >= n.
__global__ __launch_bounds__(kBlock) void k_coo_count(const int32_t* __restrict__ i,
                                                      const int32_t* __restrict__ j,
                                                      int64_t ncoo, int64_t n, int64_t ntiles,
                                                      uint32_t* __restrict__ cnt,
                                                      int32_t* __restrict__ err) {
  __shared__ uint32_t lds[kBlock / 64];
  const int64_t k = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * kIpt;
  const bool aligned = ((reinterpret_cast<uintptr_t>(i) | reinterpret_cast<uintptr_t>(j)) & 15) == 0;
  int32_t a[kIpt], b[kIpt];
  load_ipt(i, k, ncoo, aligned, a);
  load_ipt(j, k, ncoo, aligned, b);
  int32_t prev = row_before(i, k, ncoo, a);
  uint32_t c = 0;  // kept in the low half, run starts in the high one
  bool bad = false;
#pragma unroll
  for (int u = 0; u < kIpt; ++u) {
    if (a[u] >= 0 && b[u] >= 0) {
      if (a[u] >= n || b[u] >= n)
        bad = true;
      else
        ++c;
    }
    if (k + u < ncoo && (k + u == 0 || prev != a[u])) c += 1u << 16;
    prev = a[u];
  }
  if (bad) atomicOr(err, 1);
  static_assert(kTile < (1 << 16), "both counts in one word");
  uint32_t tot;
  (void)block_exscan(c, lds, &tot);
  if (threadIdx.x == 0) {
    cnt[blockIdx.x] = tot & 0xffffu;
    cnt[ntiles + blockIdx.x] = tot >> 16;
  }
}

// The runs of equal rows in order: run r's row and first triplet (every
// triplet kept).  off: the tiles' run starts, less base.
__global__ __launch_bounds__(kBlock) void k_seg_emit(const int32_t* __restrict__ i, int64_t ncoo,
                                                     const uint32_t* __restrict__ off,
                                                     uint32_t base, uint32_t* __restrict__ row,
                                                     uint32_t* __restrict__ start, int64_t nseg) {
  __shared__ uint32_t lds[kBlock / 64];
  const int64_t k = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * kIpt;
  int32_t a[kIpt];
  load_ipt(i, k, ncoo, (reinterpret_cast<uintptr_t>(i) & 15) == 0, a);
  const int32_t before = row_before(i, k, ncoo, a);
  uint32_t heads = 0;
#pragma unroll
  for (int u = 0; u < kIpt; ++u) {
    const int32_t prev = u == 0 ? before : a[u > 0 ? u - 1 : 0];
    if (k + u < ncoo && (k + u == 0 || prev != a[u])) heads |= 1u << u;
  }
  uint32_t at = off[blockIdx.x] - base + block_exscan(__popc(heads), lds, nullptr);
#pragma unroll
  for (int u = 0; u < kIpt; ++u) {
    if (heads >> u & 1u) {
      row[at] = (uint32_t)a[u];
      start[at] = (uint32_t)(k + u);
      ++at;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) start[nseg] = (uint32_t)ncoo;
}

// Runs in sorted order: their first triplets and lengths.
__global__ void k_seg_lengths(const uint32_t* __restrict__ order, const uint32_t* __restrict__ start,
                              int64_t nseg, uint32_t* __restrict__ first,
                              uint32_t* __restrict__ len) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nseg) return;
  const uint32_t r = order[e], a = start[r];
  first[e] = a;
  len[e] = start[r + 1] - a;
}

// The first run from e on, up to lim, that is not of run e - 1's row.  Galloped
// for: most rows end within a few runs, and one step after the other was a
// chain of 1024 loads for rows that exceed a tile (158 us).
__device__ __forceinline__ int64_t row_end(const uint32_t* __restrict__ row, int64_t e,
                                           int64_t lim) {
  if (e == 0 || e >= lim) return e < lim ? e : lim;
  const uint32_t r = row[e - 1];
  if (row[e] != r) return e;
  int64_t step = 1;  // row[e] is r
  while (e + step < lim && row[e + step] == r) {
    e += step;
    step *= 2;
  }
  int64_t hi = e + step < lim ? e + step : lim;  // another row, or the limit
  while (hi - e > 1) {
    const int64_t mid = e + (hi - e) / 2;
    if (row[mid] == r)
      e = mid;
    else
      hi = mid;
  }
  return hi;
}

// tile[b] = the first run that starts a row and whose first item is at b
// kRowTile or later, for b = 0 .. tiles (row: the runs' rows in order; SEG:
// pos their first items, pos[count] the item count; else every item is a
// run), with that run's first item.  The search stops kRowCap + 1 runs on: the
// rows of the tile before then exceed a tile's capacity, wherever the next
// row starts.  *longrow is set where the items passed over do already, which
// spares the stage that follows its work for nothing.
template <bool SEG>
__global__ void k_row_tiles(const uint32_t* __restrict__ row, const uint32_t* __restrict__ pos,
                            int64_t count, int64_t tiles, uint2* __restrict__ tile,
                            uint32_t* __restrict__ longrow) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t lo, hi, e = t;
  uint64_t heads = 0;
  if constexpr (SEG) {  // a thread per run, the one past the last included
    heads = __ballot(t >= count || t == 0 || row[t] != row[t - 1]);
    if (t > count) return;
    lo = t == 0 ? 0 : (int64_t)pos[t - 1] / kRowTile + 1;
    hi = t == count ? tiles : (int64_t)pos[t] / kRowTile;
    if (lo > hi) return;
  } else {  // a thread per tile
    if (t > tiles) return;
    lo = hi = t;
    e = t * kRowTile < count ? t * kRowTile : count;
  }
  const int64_t lim = e + kRowCap + 1 < count ? e + kRowCap + 1 : count;
  if constexpr (SEG) {
    // the next row start among this wave's runs, where there is one
    const int lane = threadIdx.x & 63;
    const uint64_t m = heads >> lane;
    e += m ? __ffsll((unsigned long long)m) - 1 : 64 - lane;
  }
  const int64_t from = SEG ? t : e;
  e = row_end(row, e, lim);
  const uint2 v = make_uint2((uint32_t)e, SEG ? pos[e] : (uint32_t)e);
  // (runs from .. e are one row's, the row of run from - 1)
  if (e > from && v.y - (SEG ? pos[from] : (uint32_t)from) > (uint32_t)kRowCap) *longrow = 1;
  for (int64_t b = lo; b <= hi; ++b) tile[b] = v;
}

// Stable compaction of the kept triplets into (key, k) pairs with
// key = row << cb | col (ROW_ONLY: key = row).  Wave w of a tile owns the contiguous items
// [w*512, (w+1)*512) and walks them in 64-item steps (coalesced loads); the
// write position of an item is its wave's offset plus the number of kept
// items before it, counted with ballots, so input order is preserved.
template <typename K, bool ROW_ONLY = false>
__global__ __launch_bounds__(kBlock) void k_coo_compact(const int32_t* __restrict__ i,
                                                        const int32_t* __restrict__ j,
                                                        int64_t ncoo, int64_t n, int cb,
                                                        const uint32_t* __restrict__ tileoff,
                                                        K* __restrict__ keys,
                                                        uint32_t* __restrict__ vals) {
  __shared__ uint32_t wcount[kBlock / 64];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)w * (kIpt * 64);
  const uint64_t lt = (1ull << lane) - 1ull;
  int32_t a[kIpt], b[kIpt];
  bool keep[kIpt];
  uint32_t cnt = 0;
#pragma unroll
  for (int s = 0; s < kIpt; ++s) {
    const int64_t k = base + s * 64 + lane;
    a[s] = k < ncoo ? i[k] : -1;
    b[s] = k < ncoo ? j[k] : -1;
    keep[s] = a[s] >= 0 && b[s] >= 0 && a[s] < n && b[s] < n;
    cnt += (uint32_t)__popcll(__ballot(keep[s]));
  }
  if (lane == 0) wcount[w] = cnt;
  __syncthreads();
  uint32_t pos = tileoff[blockIdx.x];
  for (int ww = 0; ww < w; ++ww) pos += wcount[ww];
#pragma unroll
  for (int s = 0; s < kIpt; ++s) {
    const uint64_t m = __ballot(keep[s]);
    if (keep[s]) {
      const uint32_t at = pos + (uint32_t)__popcll(m & lt);
      if constexpr (ROW_ONLY)
        keys[at] = (K)(uint32_t)a[s];
      else
        keys[at] = ((K)(uint32_t)a[s] << cb) | (K)(uint32_t)b[s];
      vals[at] = (uint32_t)(base + s * 64 + lane);
    }
    pos += (uint32_t)__popcll(m);
  }
}

// Second stage of the two-stage order: runs of items sorted stably by row
// alone (increasing k within a row) are re-sorted by column inside each row
// in LDS, ties keeping their order, which gives the (row, column, k) order
// of the full sort.  Tile b takes the whole rows whose first run is one of
// its runs (those that start in items [b kRowTile, (b + 1) kRowTile)); when
// those rows hold more than kRowCap items, *overflow is set and the caller
// sorts the full keys instead.
constexpr int kRowPosBits = 10;  // positions in a tile, in the rank key
static_assert(kRowCap <= (1 << kRowPosBits), "tile positions must fit the rank key");
constexpr int kRowColBits = 32 - kRowPosBits;  // columns of the rank key (n up to 2^22)
constexpr int kRowIpt = kRowCap / kBlock;  // items per thread
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

// What the row-tile stage reads and writes.  Runs in sorted order: row, the
// first triplet (SEG) or the triplet itself (first), each tile's first run
// and item (tile), and with SEG the runs' first items (pos, the item count
// after the last).
struct RowTiles {
  const uint32_t* row;
  const uint32_t* first;
  const uint32_t* pos;
  const uint2* tile;
  const int32_t* j;
  int32_t* perm;
  // per tile, at its first item: its distinct entries' columns and first
  // items, compact; how many, and where
  uint32_t* ecol;
  uint32_t* eq;
  uint32_t* ecount;
  uint32_t* eat;
  // per row: its first entry in its tile, that tile, its diagonal entry
  uint32_t* rent;
  uint32_t* rtile;
  int32_t* rdiag;
  const uint32_t* longrow;  // a tile will overflow
  uint32_t* overflow;
};

// The tile's rows and, once ranked, its distinct entries are numbered with
// wave ballots.  An item's rank in its row is the number of the row's items
// with a smaller column, or an equal column and a smaller position (the row
// sort left equal columns in increasing k): one compare of col <<
// kRowPosBits | position against every item of the row, 16 keys of LDS per
// step.  These compares bound the kernel: 64 per item on the 3-D operator,
// whose rows hold eight runs of eight.  SEG: the runs are longer than one
// triplet, so the stage reads a few words per run and the columns of a run
// as one piece; without it every item is its own run.
template <bool SEG>
__global__ __launch_bounds__(kBlock) void k_rowtile_sort(RowTiles t) {
  constexpr int W = kBlock / 64;
  // 16.5 KB: eight workgroups per CU, so that their chains of loads (tile,
  // runs, columns) hide each other
  __shared__ uint32_t first[kRowCap];              // run -> first triplet
  __shared__ __align__(16) uint32_t key[kRowCap];  // item -> rank key, then in order
  __shared__ uint16_t pre[SEG ? kRowCap : 1];      // run -> first item
  __shared__ uint16_t run[SEG ? kRowCap : 1];      // item -> run
  __shared__ uint16_t rid[kRowCap];                // run -> row of the tile
  __shared__ uint16_t start[kRowCap + 1];          // row of the tile -> first item
  __shared__ uint32_t count[2][kRowIpt * W];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const uint64_t below = (1ull << lane) - 1ull;
  const int64_t b = blockIdx.x;
  const uint2 ta = t.tile[b], tb = t.tile[b + 1];
  const int64_t s0 = ta.x, s1 = tb.x, q0 = ta.y, items = (int64_t)tb.y - q0;
  // no row starts here, or nothing will be built (longrow was set before this
  // kernel, so it is the same for every thread)
  const bool none = *t.longrow != 0;
  if (s0 >= s1 || none) {
    if (tid == 0) {
      t.ecount[b] = 0;
      if (none && b == 0) atomicOr(t.overflow, 1u);  // (one for all: they take turns)
    }
    return;
  }
  if (s1 - s0 > kRowCap || items > kRowCap) {
    if (tid == 0) {
      t.ecount[b] = 0;
      atomicOr(t.overflow, 1u);
    }
    return;
  }
  const int S = (int)(s1 - s0), L = (int)items;
  // the runs, kBlock at a time: their rows numbered in order
  int rows = 0;
  for (int c = 0; c < S; c += kBlock) {
    const int e = c + tid;
    const bool in = e < S;
    uint32_t row = 0, prev = 0, p = (uint32_t)e, q = (uint32_t)e + 1;
    if (in) {
      row = t.row[s0 + e];
      prev = e > 0 ? t.row[s0 + e - 1] : 0;
      first[e] = t.first[s0 + e];
      if constexpr (SEG) {
        p = (uint32_t)((int64_t)t.pos[s0 + e] - q0);
        q = (uint32_t)((int64_t)t.pos[s0 + e + 1] - q0);
      }
    }
    const bool head = in && (e == 0 || row != prev);
    const uint64_t m = __ballot(head);
    uint32_t* slot = count[(c / kBlock) & 1];
    if (lane == 0) slot[w] = (uint32_t)__popcll(m);
    __syncthreads();
    int r = rows + (int)__popcll(m & below);
#pragma unroll
    for (int ww = 0; ww < W; ++ww) {
      if (ww < w) r += (int)slot[ww];
      rows += (int)slot[ww];
    }
    if (in) {
      if (head) start[r] = (uint16_t)p;
      rid[e] = (uint16_t)(head ? r : r - 1);
      if constexpr (SEG) {
        pre[e] = (uint16_t)p;
        for (uint32_t l = p; l < q; ++l) run[l] = (uint16_t)e;
      }
    }
  }
  if (tid == 0) start[rows] = (uint16_t)L;
  __syncthreads();
  // the triplet of item l
  auto triplet = [&](int l) -> uint32_t {
    if constexpr (SEG) {
      const int e = run[l];
      return first[e] + (uint32_t)(l - pre[e]);
    } else {
      return first[l];
    }
  };
#pragma unroll
  for (int u = 0; u < kRowIpt; ++u) {
    const int l = tid + u * kBlock;
    if (l < L) key[l] = ((uint32_t)t.j[triplet(l)] << kRowPosBits) | (uint32_t)l;
  }
  __syncthreads();
  uint32_t k4[kRowIpt];
  int at4[kRowIpt];
#pragma unroll
  for (int u = 0; u < kRowIpt; ++u) {
    const int l = tid + u * kBlock;
    k4[u] = 0;
    at4[u] = 0;
    if (l < L) {
      const int row = rid[SEG ? run[l] : l];
      const int rs = start[row], re = start[row + 1];
      const uint32_t k = key[l];
      int at = rs, m = rs;
      for (; m < re && (m & 3); ++m) at += key[m] < k ? 1 : 0;
      for (; m + 16 <= re; m += 16) {
        uint4v km[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) km[v] = *reinterpret_cast<const uint4v*>(key + m + 4 * v);
#pragma unroll
        for (int v = 0; v < 16; ++v) at += km[v / 4][v % 4] < k ? 1 : 0;
      }
      for (; m < re; ++m) at += key[m] < k ? 1 : 0;
      k4[u] = k;
      at4[u] = at;
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kRowIpt; ++u)
    if (tid + u * kBlock < L) key[at4[u]] = k4[u];
  __syncthreads();
  // in order: the items' triplets, and the distinct entries numbered
  uint64_t m4[kRowIpt];
  bool first4[kRowIpt];
#pragma unroll
  for (int u = 0; u < kRowIpt; ++u) {
    const int l = tid + u * kBlock;
    bool head = false;
    first4[u] = false;
    if (l < L) {
      const uint32_t k = key[l];
      t.perm[q0 + l] = (int32_t)triplet((int)(k & (kRowCap - 1)));
      first4[u] = l == start[rid[SEG ? run[l] : l]];
      head = first4[u] || (key[l - 1] >> kRowPosBits) != (k >> kRowPosBits);
    }
    m4[u] = __ballot(head);
    if (lane == 0) count[0][u * W + w] = (uint32_t)__popcll(m4[u]);
  }
  __syncthreads();
  uint32_t before = 0;
#pragma unroll
  for (int u = 0; u < kRowIpt; ++u) {
    uint32_t e = before + (uint32_t)__popcll(m4[u] & below);
#pragma unroll
    for (int ww = 0; ww < W; ++ww) {
      const uint32_t x = count[0][u * W + ww];
      if (ww < w) e += x;
      before += x;
    }
    if (m4[u] >> lane & 1ull) {
      const int l = tid + u * kBlock;
      const int64_t r = s0 + (SEG ? run[l] : l);  // of the item's row: its first when first4
      const uint32_t c = key[l] >> kRowPosBits, row = t.row[r];
      t.ecol[q0 + e] = c;
      t.eq[q0 + e] = (uint32_t)(q0 + l);
      if (first4[u]) {
        // this row, and the empty rows before it, start here
        for (uint32_t rr = r > 0 ? t.row[r - 1] + 1 : 0; rr <= row; ++rr) {
          t.rent[rr] = e;
          t.rtile[rr] = (uint32_t)b;
        }
      }
      if (c == row) t.rdiag[row] = (int32_t)e;
    }
  }
  if (tid == 0) {
    t.ecount[b] = before;
    t.eat[b] = (uint32_t)q0;
  }
}

// The tiles' entries to their final places: a wave per tile.
__global__ __launch_bounds__(kBlock) void k_entries(const uint32_t* __restrict__ ecol,
                                                    const uint32_t* __restrict__ eq,
                                                    const uint32_t* __restrict__ off,
                                                    const uint32_t* __restrict__ eat,
                                                    int64_t tiles, int32_t* __restrict__ col,
                                                    int32_t* __restrict__ jmap) {
  const int64_t b = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  if (b >= tiles) return;
  const uint32_t to = off[b], cnt = off[b + 1] - to;
  if (cnt == 0) return;
  const uint32_t from = eat[b];
  constexpr int U = 4;  // loads in flight together
  for (uint32_t e0 = threadIdx.x & 63; e0 < cnt; e0 += 64 * U) {
    uint32_t c[U], q[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t e = e0 + 64 * u < cnt ? e0 + 64 * u : cnt - 1;
      c[u] = ecol[from + e];
      q[u] = eq[from + e];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t e = e0 + 64 * u;
      if (e < cnt) {
        col[to + e] = (int32_t)c[u];
        jmap[to + e] = (int32_t)q[u];
      }
    }
  }
}

// Per-row words of a new pattern: no entry, past the last tile, no diagonal;
// and no entries past the last tile.
__global__ void k_row_init(uint32_t* rent, uint32_t* rtile, int32_t* rdiag, int64_t n,
                           uint32_t tiles, uint32_t* ecount) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r == 0) ecount[tiles] = 0;
  if (r >= n) return;
  rent[r] = 0;
  rtile[r] = tiles;
  rdiag[r] = -1;
}

// rowptr and dpos from the rows' tiles; the closing jmap entry.
__global__ void k_row_emit(const uint32_t* __restrict__ rent, const uint32_t* __restrict__ rtile,
                           const int32_t* __restrict__ rdiag, const uint32_t* __restrict__ off,
                           int64_t n, int64_t tiles, int64_t nvalid, int32_t* __restrict__ rowptr,
                           int32_t* __restrict__ dpos, int32_t* __restrict__ jmap) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r > n) return;
  if (r == n) {
    rowptr[n] = (int32_t)off[tiles];
    jmap[off[tiles]] = (int32_t)nvalid;
    return;
  }
  const uint32_t o = off[rtile[r]];
  const int32_t d = rdiag[r];
  rowptr[r] = (int32_t)(o + rent[r]);
  dpos[r] = d >= 0 ? (int32_t)o + d : -1;
}

// Number of run heads (first element of each distinct key) per tile.
template <typename K>
__global__ __launch_bounds__(kBlock) void k_heads_count(const K* __restrict__ keys,
                                                        int64_t count,
                                                        uint32_t* __restrict__ tilecnt) {
  __shared__ uint32_t lds[kBlock / 64];
  const int64_t base = (int64_t)blockIdx.x * kTile;
  uint32_t c = 0;
#pragma unroll
  for (int s = 0; s < kIpt; ++s) {
    const int64_t q = base + (int64_t)s * kBlock + threadIdx.x;
    if (q < count && (q == 0 || keys[q] != keys[q - 1])) ++c;
  }
  uint32_t tot;
  (void)block_exscan(c, lds, &tot);
  if (threadIdx.x == 0) tilecnt[blockIdx.x] = tot;
}

// For each run head q (entry t): jmap[t] = q, col[t], diagonal position,
// and rowptr for every row that starts at t (empty rows included).  Same
// wave-ordered walk as the compaction: entry numbers are the tile offset
// plus the heads before q, counted with ballots.
template <typename K>
__global__ __launch_bounds__(kBlock) void k_heads_emit(const K* __restrict__ keys, int64_t count,
                                                       int cb, const uint32_t* __restrict__ tileoff,
                                                       int32_t* __restrict__ jmap,
                                                       int32_t* __restrict__ col,
                                                       int32_t* __restrict__ rowptr,
                                                       int32_t* __restrict__ dpos) {
  __shared__ uint32_t wcount[kBlock / 64];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)w * (kIpt * 64);
  const K cmask = cb >= (int)(8 * sizeof(K)) ? ~K(0) : ((K(1) << cb) - K(1));
  const uint64_t lt = (1ull << lane) - 1ull;
  K cur[kIpt], prev[kIpt];
  bool head[kIpt];
  uint32_t cnt = 0;
#pragma unroll
  for (int s = 0; s < kIpt; ++s) {
    const int64_t q = base + s * 64 + lane;
    cur[s] = q < count ? keys[q] : K(0);
    prev[s] = (q > 0 && q < count) ? keys[q - 1] : K(0);
    head[s] = q < count && (q == 0 || cur[s] != prev[s]);
    cnt += (uint32_t)__popcll(__ballot(head[s]));
  }
  if (lane == 0) wcount[w] = cnt;
  __syncthreads();
  uint32_t pos = tileoff[blockIdx.x];
  for (int ww = 0; ww < w; ++ww) pos += wcount[ww];
#pragma unroll
  for (int s = 0; s < kIpt; ++s) {
    const uint64_t m = __ballot(head[s]);
    if (head[s]) {
      const int64_t q = base + s * 64 + lane;
      const uint32_t t = pos + (uint32_t)__popcll(m & lt);
      const int64_t r = (int64_t)(cur[s] >> cb);
      const int32_t cc = (int32_t)(cur[s] & cmask);
      jmap[t] = (int32_t)q;
      col[t] = cc;
      if (r == cc) dpos[r] = (int32_t)t;
      const int64_t pr = q == 0 ? -1 : (int64_t)(prev[s] >> cb);
      for (int64_t rr = pr + 1; rr <= r; ++rr) rowptr[rr] = (int32_t)t;
    }
    pos += (uint32_t)__popcll(m);
  }
}

// rowptr of the rows after the last stored row, and the closing jmap entry.
template <typename K>
__global__ void k_rowptr_tail(const K* __restrict__ keys, int64_t count, int cb, int64_t n,
                              const uint32_t* __restrict__ nnz_dev, int32_t* __restrict__ rowptr,
                              int32_t* __restrict__ jmap) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t last = count > 0 ? (int64_t)(keys[count - 1] >> cb) : -1;
  const int32_t nnz = (int32_t)*nnz_dev;
  if (r <= n && r > last) rowptr[r] = nnz;
  if (r == 0 && jmap) jmap[nnz] = (int32_t)count;
}

// out[0] = longest row, out[1 + k] = most entries in a block of 32 << k
// consecutive rows (k < 4).  At most kStatBlocks workgroups, each with its
// own maxima before its atomics: one address for all of them (one atomic per
// 256 rows took 96 us for 2M rows).
constexpr int kStatBlocks = 256;
__global__ __launch_bounds__(256) void k_row_stats(const int32_t* __restrict__ rowptr, int64_t n,
                                                   int32_t* __restrict__ out) {
  __shared__ int32_t lds[4][5];
  int32_t m[5] = {0, 0, 0, 0, 0};
  for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < n; r += (int64_t)gridDim.x * 256) {
    const int32_t p = rowptr[r];
    m[0] = max(m[0], rowptr[r + 1] - p);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t R = 32 << k;
      if (r % R == 0) m[1 + k] = max(m[1 + k], rowptr[r + R < n ? r + R : n] - p);
    }
  }
#pragma unroll
  for (int k = 0; k < 5; ++k) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m[k] = max(m[k], __shfl_xor(m[k], off, 64));
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6][k] = m[k];
  }
  __syncthreads();
  if (threadIdx.x < 5) {
    const int k = threadIdx.x;
    atomicMax(out + k, max(max(lds[0][k], lds[1][k]), max(lds[2][k], lds[3][k])));
  }
}

void launch_row_stats(const Csr& M, int64_t n, int32_t* out, hipStream_t s) {
  const int64_t g = std::min<int64_t>(ceil_div(n, 256), kStatBlocks);
  hipLaunchKernelGGL(k_row_stats, dim3((unsigned)std::max<int64_t>(g, 1)), dim3(256), 0, s, M.rowptr,
                     n, out);
}

// Tiled numeric stage: a workgroup owns `ents` consecutive entries.
// Their contributions form one contiguous run of perm, which the workgroup
// reads coalesced while gathering v into LDS, kSvBatch values per thread at
// a time with all of a batch's gathers in flight before any is stored; then
// each thread adds its entries' contributions from LDS in order, from +0.0
// (bitwise the same sums as one thread walking perm).  The gather is bound
// by latency, not bytes, so the batches and a small LDS footprint (more
// workgroups per CU) are what set the rate.  A tile whose run exceeds kSvCap
// values is summed straight from memory, each thread issuing up to kSvBatch
// gathers of its own run before adding them in order.
constexpr int kSvBatch = 4;
constexpr int kSvCap = 2048;

// Entries per workgroup: the largest of 512, 256 and 128 whose tiles
// typically (1.5x the mean contributions per entry) fit in kSvCap values.
int sv_entries(int64_t nvalid, int64_t nnz) {
  const double per = nnz > 0 ? (double)nvalid / (double)nnz : 0.0;
  for (int e : {512, 256, 128})
    if (1.5 * per * e <= kSvCap) return e;
  return 64;
}

__global__ __launch_bounds__(256) void k_set_values_tiled(const int32_t* __restrict__ jmap,
                                                          const int32_t* __restrict__ perm,
                                                          const double* __restrict__ v,
                                                          int64_t nnz, int mode, int ents,
                                                          double* __restrict__ val) {
  __shared__ double lv[kSvCap];
  const int64_t e0 = (int64_t)blockIdx.x * ents;
  const int64_t e1 = e0 + ents < nnz ? e0 + ents : nnz;
  const int32_t q0 = jmap[e0], q1 = jmap[e1];
  if (q1 - q0 > kSvCap) {
    for (int64_t t = e0 + threadIdx.x; t < e1; t += 256) {
      const int32_t qe = jmap[t + 1];
      double s = 0.0;
      for (int32_t q = jmap[t]; q < qe; q += kSvBatch) {
        double x[kSvBatch];
#pragma unroll
        for (int k = 0; k < kSvBatch; ++k) x[k] = q + k < qe ? v[perm[q + k]] : 0.0;
#pragma unroll
        for (int k = 0; k < kSvBatch; ++k)
          if (q + k < qe) s += x[k];
      }
      val[t] = mode ? val[t] + s : s;
    }
    return;
  }
  for (int32_t base = q0; base < q1; base += 256 * kSvBatch) {
    int32_t p[kSvBatch];
#pragma unroll
    for (int k = 0; k < kSvBatch; ++k) {
      const int32_t q = base + k * 256 + (int32_t)threadIdx.x;
      p[k] = q < q1 ? perm[q] : -1;
    }
    double x[kSvBatch];
#pragma unroll
    for (int k = 0; k < kSvBatch; ++k) x[k] = p[k] >= 0 ? v[p[k]] : 0.0;
#pragma unroll
    for (int k = 0; k < kSvBatch; ++k) {
      const int32_t q = base + k * 256 + (int32_t)threadIdx.x;
      if (q < q1) lv[q - q0] = x[k];
    }
  }
  __syncthreads();
  for (int64_t t = e0 + threadIdx.x; t < e1; t += 256) {
    double s = 0.0;
    for (int32_t q = jmap[t]; q < jmap[t + 1]; ++q) s += lv[q - q0];
    val[t] = mode ? val[t] + s : s;
  }
}

__global__ void k_expand_rows(const int32_t* __restrict__ rowptr, int64_t n,
                              int32_t* __restrict__ rowidx) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  for (int32_t t = rowptr[r]; t < rowptr[r + 1]; ++t) rowidx[t] = (int32_t)r;
}

// Explicit transpose from the column-sorted entries: tmap[tt] = entry of A.
__global__ void k_transpose_emit(const uint32_t* __restrict__ ckeys,
                                 const uint32_t* __restrict__ tmap, const int32_t* __restrict__ rowidx,
                                 int64_t nnz, int32_t* __restrict__ rowptrT,
                                 int32_t* __restrict__ colT, int32_t* __restrict__ dposT) {
  const int64_t tt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tt >= nnz) return;
  const int64_t c = ckeys[tt];
  const int32_t r = rowidx[tmap[tt]];
  colT[tt] = r;
  if (r == c) dposT[c] = (int32_t)tt;
  const int64_t pc = tt == 0 ? -1 : (int64_t)ckeys[tt - 1];
  for (int64_t cc = pc + 1; cc <= c; ++cc) rowptrT[cc] = (int32_t)tt;
}

__global__ void k_transpose_tail(const uint32_t* __restrict__ ckeys, int64_t nnz, int64_t n,
                                 int32_t* __restrict__ rowptrT) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t last = nnz > 0 ? (int64_t)ckeys[nnz - 1] : -1;
  if (r <= n && r > last) rowptrT[r] = (int32_t)nnz;
}

__global__ void k_gather_vals(const int32_t* __restrict__ tmap, const double* __restrict__ val,
                              int64_t nnz, double* __restrict__ valT) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < nnz) valT[t] = val[tmap[t]];
}

__global__ void k_to_f32(const double* __restrict__ a, int64_t count, float* __restrict__ b) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < count) b[t] = (float)a[t];
}

__global__ void k_kslot(const int32_t* __restrict__ jmap, const int32_t* __restrict__ perm,
                        int64_t nnz, int32_t* __restrict__ kslot) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nnz) return;
  for (int32_t q = jmap[t]; q < jmap[t + 1]; ++q) kslot[perm[q]] = (int32_t)t;
}

__global__ void k_coo_gather(const int32_t* __restrict__ kslot, const double* __restrict__ G,
                             int64_t ncoo, double* __restrict__ gv) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= ncoo) return;
  const int32_t t = kslot[k];
  gv[k] = t >= 0 ? G[t] : 0.0;
}

__global__ void k_coo_gather_blocks(const int32_t* __restrict__ kslot,
                                    const double* __restrict__ G, const double* __restrict__ w,
                                    int64_t nblocks, int64_t block, double* __restrict__ ge) {
#pragma clang fp contract(off)
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nblocks) return;
  double s = 0.0;
  for (int64_t k = e * block; k < (e + 1) * block; ++k) {
    const int32_t t = kslot[k];
    const double g = t >= 0 ? G[t] : 0.0;
    s += g * w[k];
  }
  ge[e] = s;
}

inline unsigned grid_for(int64_t count, int block) {
  return (unsigned)std::max<int64_t>(1, ceil_div(count, block));
}

void set_row_stats(Csr& M, const int32_t* v) {
  M.max_row = v[0];
  for (int k = 0; k < 4; ++k) M.tile_nnz[k] = v[1 + k];
}

// Device buffers of one preallocation, freed once the stream has passed it.
struct Scratch {
  hipStream_t s;
  void* p[4] = {};
  int n = 0;
  explicit Scratch(hipStream_t stream) : s(stream) {}
  Scratch(const Scratch&) = delete;
  Scratch& operator=(const Scratch&) = delete;
  template <typename T>
  int get(T** out, size_t count) {
    if (n == 4) return set_error(SPX_HIP_ERROR, "coo_preallocate: too many buffers");
    SPX_TRY(dalloc_n(out, count));
    p[n++] = *out;
    return SPX_OK;
  }
  ~Scratch() {
    if (n > 0) (void)hipStreamSynchronize(s);
    for (int k = 0; k < n; ++k) dfree(p[k]);
  }
};

// Parts of one buffer of 32-bit words, each aligned for 16-byte loads.
struct Parts {
  int64_t words = 0;
  int64_t take(int64_t count) {
    const int64_t at = words;
    words += (count + 15) & ~int64_t(15);
    return at;
  }
};

// The counts' words in misc: an index out of range, kept triplets, kept
// triplets and runs of equal rows together, a row tile that overflowed,
// entries, the row statistics, the window index's statistics, a row found to
// exceed a tile beforehand.
enum {
  kErr = 0,
  kKept = 1,
  kBoth = 2,
  kOver = 3,
  kNnz = 4,
  kStats = 5,
  kWin = 10,
  kLong = 16,
  kMisc = 18
};
static_assert(kWin % 2 == 0 && kWin + kWinStats <= kLong, "misc holds the statistics");

struct CooIn {
  const int32_t* i;
  const int32_t* j;
  int64_t ntiles, nvalid, nruns;
  uint32_t* misc;
  const uint32_t* tileoff;  // kept triplets before each tile, then runs (less nvalid)
};

int read_misc(const uint32_t* misc, uint32_t* host, hipStream_t s) {
  SPX_CHECK_HIP(hipMemcpyAsync(host, misc, kMisc * sizeof(uint32_t), hipMemcpyDeviceToHost, s));
  SPX_CHECK_HIP(hipStreamSynchronize(s));
  return SPX_OK;
}

// The pattern's arrays, in one block, for at most `most` entries, values 0;
// every array has its 64 bytes of tail padding.
int alloc_pattern(spx_matrix* h, int64_t most, hipStream_t s) {
  const int64_t n = h->n;
  Parts parts;
  const int64_t pad = 16;
  const int64_t o_val = parts.take(2 * most + pad), o_col = parts.take(most + pad),
                o_jmap = parts.take(most + 1 + pad), o_row = parts.take(n + 1 + pad),
                o_dpos = parts.take(n + pad);
  int32_t* w = nullptr;
  SPX_TRY(dalloc_n(&w, (size_t)parts.words));
  h->A.block = w;
  h->A.n = n;
  h->A.val = reinterpret_cast<double*>(w + o_val);
  h->A.col = w + o_col;
  h->A.rowptr = w + o_row;
  h->A.dpos = w + o_dpos;
  h->jmap = w + o_jmap;
  hipLaunchKernelGGL(k_fill_f64, dim3(grid_for(most, 256)), dim3(256), 0, s, h->A.val, most, 0.0);
  return SPX_OK;
}

// The row statistics and the window index of the pattern in place (at most
// `most` entries, unless misc's overflow is set), and misc read back.
// scratch: window_scratch(n) words.  Waits for the stream.
int finish_pattern(spx_matrix* h, int64_t most, uint32_t* misc, uint32_t* scratch, uint32_t* host,
                   hipStream_t s) {
  launch_row_stats(h->A, h->n, (int32_t*)(misc + kStats), s);
  Window win;
  int st = window_enqueue(h->A, most, misc + kOver, scratch, misc + kWin, s, &win);
  if (st == SPX_OK) st = read_misc(misc, host, s);
  if (st != SPX_OK || host[kOver]) {
    window_release(&win);
    return st;
  }
  h->A.nnz = host[kNnz];
  set_row_stats(h->A, (const int32_t*)(host + kStats));
  window_keep(h->A, host + kWin, &win);
  return SPX_OK;
}

// The two-stage order (n up to 2^22): a stable sort by row alone (32-bit
// keys, few passes), then each tile's whole rows ranked by column in LDS.
// Finite-element and edge streams name the same row several times in a row;
// when every triplet is kept and those runs are at least kSegRun long on
// average, the runs are sorted instead of the triplets (the 3-D operator's
// 131M triplets are 16.4M runs: 0.25 ms of sorting instead of 1.9).
// *overflow: a tile's rows exceed it, and nothing was built.
constexpr int64_t kSegRun = 2;
// Up to here the pattern's block holds an entry per triplet (20 bytes each,
// 5 MB at most), and the host waits for the device twice instead of three
// times.
constexpr int64_t kCountTriplets = 1 << 18;
int symbolic_rows(spx_matrix* h, const CooIn& in, hipStream_t s, bool* overflow) {
  const int64_t n = h->n, ncoo = h->ncoo, nvalid = in.nvalid;
  const int cb = h->colbits;
  const bool all_kept = nvalid == ncoo;
  const bool seg = all_kept && nvalid > 0 && nvalid >= kSegRun * in.nruns;
  const int64_t count = seg ? in.nruns : nvalid;
  const int64_t tiles = std::max<int64_t>(1, ceil_div(nvalid, kRowTile));
  Scratch mem(s);
  Parts parts;
  const int64_t o_key = parts.take(count), o_key2 = parts.take(count), o_val = parts.take(count),
                o_val2 = parts.take(count);
  const int64_t o_start = parts.take(seg ? count + 1 : 0), o_first = parts.take(seg ? count : 0),
                o_pos = parts.take(seg ? count + 1 : 0), o_tile = parts.take(2 * (tiles + 1));
  const int64_t o_ecol = parts.take(nvalid), o_eq = parts.take(nvalid);
  const int64_t o_ecount = parts.take(tiles + 1), o_eat = parts.take(tiles);
  const int64_t o_rent = parts.take(n), o_rtile = parts.take(n), o_rdiag = parts.take(n);
  const int64_t o_work = parts.take(std::max({radix_sort_work(count, cb), scan_scratch_elems(count),
                                              scan_scratch_elems(tiles + 1), window_scratch(n)}));
  uint32_t* w = nullptr;
  SPX_TRY(mem.get(&w, (size_t)parts.words));
  int32_t* perm = nullptr;
  SPX_TRY(mem.get(&perm, (size_t)std::max<int64_t>(nvalid, 1)));
  uint32_t *work = w + o_work, *ecount = w + o_ecount;

  RowTiles t{};
  t.j = in.j;
  t.perm = perm;
  t.ecol = w + o_ecol;
  t.eq = w + o_eq;
  t.ecount = ecount;
  t.eat = w + o_eat;
  t.rent = w + o_rent;
  t.rtile = w + o_rtile;
  t.rdiag = (int32_t*)(w + o_rdiag);
  t.overflow = in.misc + kOver;
  t.longrow = in.misc + kLong;
  uint2* tile = reinterpret_cast<uint2*>(w + o_tile);
  t.tile = tile;
  hipLaunchKernelGGL(k_row_init, dim3(grid_for(n, 256)), dim3(256), 0, s, t.rent, t.rtile, t.rdiag,
                     n, (uint32_t)tiles, ecount);
  uint32_t *row = nullptr, *order = nullptr;
  if (seg) {
    hipLaunchKernelGGL(k_seg_emit, dim3((unsigned)in.ntiles), dim3(kBlock), 0, s, in.i, ncoo,
                       in.tileoff + in.ntiles, (uint32_t)nvalid, w + o_key, w + o_start, count);
    SPX_TRY(radix_sort_pairs_u32(w + o_key, w + o_key2, w + o_val, w + o_val2, count, cb, work, s,
                                 &row, &order, nullptr, true));
    hipLaunchKernelGGL(k_seg_lengths, dim3(grid_for(count, 256)), dim3(256), 0, s, order,
                       w + o_start, count, w + o_first, w + o_pos);
    SPX_TRY(exclusive_scan_u32(w + o_pos, w + o_pos, count, w + o_pos + count, work, s));
    hipLaunchKernelGGL(k_row_tiles<true>, dim3(grid_for(count + 1, 256)), dim3(256), 0, s, row,
                       w + o_pos, count, tiles, tile, in.misc + kLong);
    t.row = row;
    t.first = w + o_first;
    t.pos = w + o_pos;
    hipLaunchKernelGGL(k_rowtile_sort<true>, dim3((unsigned)tiles), dim3(kBlock), 0, s, t);
  } else {
    // with every triplet kept the sort reads the caller's rows and takes the
    // triplet numbers as its values: no compaction
    if (!all_kept)
      hipLaunchKernelGGL((k_coo_compact<uint32_t, true>), dim3((unsigned)in.ntiles), dim3(kBlock), 0,
                         s, in.i, in.j, ncoo, n, cb, in.tileoff, w + o_key, w + o_val);
    SPX_TRY(radix_sort_pairs_u32(w + o_key, w + o_key2, w + o_val, w + o_val2, count, cb, work, s,
                                 &row, &order,
                                 all_kept ? reinterpret_cast<const uint32_t*>(in.i) : nullptr,
                                 all_kept));
    hipLaunchKernelGGL(k_row_tiles<false>, dim3(grid_for(tiles + 1, 256)), dim3(256), 0, s, row,
                       (const uint32_t*)nullptr, count, tiles, tile, in.misc + kLong);
    t.row = row;
    t.first = order;
    hipLaunchKernelGGL(k_rowtile_sort<false>, dim3((unsigned)tiles), dim3(kBlock), 0, s, t);
  }
  SPX_TRY(exclusive_scan_u32(ecount, ecount, tiles + 1, in.misc + kNnz, work, s));
  // small patterns take room for as many entries as triplets instead of
  // waiting for the count
  uint32_t host[kMisc];
  int64_t most = nvalid;
  if (nvalid > kCountTriplets) {
    SPX_TRY(read_misc(in.misc, host, s));
    *overflow = host[kOver] != 0;
    if (*overflow) return SPX_OK;
    most = host[kNnz];
  }
  SPX_TRY(alloc_pattern(h, most, s));
  hipLaunchKernelGGL(k_entries, dim3(grid_for(tiles, kBlock / 64)), dim3(kBlock), 0, s, t.ecol, t.eq,
                     ecount, t.eat, tiles, h->A.col, h->jmap);
  hipLaunchKernelGGL(k_row_emit, dim3(grid_for(n + 1, 256)), dim3(256), 0, s, t.rent, t.rtile,
                     t.rdiag, ecount, n, tiles, nvalid, h->A.rowptr, h->A.dpos, h->jmap);
  SPX_TRY(finish_pattern(h, most, in.misc, work, host, s));
  *overflow = host[kOver] != 0;
  if (*overflow) {
    dfree(h->A.block);
    h->A = Csr();
    h->jmap = nullptr;
    return SPX_OK;
  }
  mem.n = 1;  // perm stays
  h->perm = perm;
  return SPX_OK;
}

// One sort on the full (row, column) keys.
template <typename K>
int symbolic_full(spx_matrix* h, const CooIn& in, hipStream_t s) {
  const int64_t n = h->n, ncoo = h->ncoo, nvalid = in.nvalid;
  const int cb = h->colbits;
  const int64_t cap = std::max<int64_t>(nvalid, 1);
  const int64_t vt = std::max<int64_t>(1, ceil_div(nvalid, kTile));
  Scratch mem(s);
  K* keys = nullptr;
  uint32_t *vals = nullptr, *vals_alt = nullptr, *work = nullptr;
  SPX_TRY(mem.get(&keys, (size_t)cap * 2));
  SPX_TRY(mem.get(&work, (size_t)(vt + std::max({radix_sort_work(nvalid, 2 * cb),
                                                 scan_scratch_elems(vt), window_scratch(n)}))));
  SPX_TRY(mem.get(&vals, (size_t)cap));
  SPX_TRY(mem.get(&vals_alt, (size_t)cap));
  uint32_t* tilecnt = work;
  work += vt;
  K* skeys = keys;
  uint32_t* svals = vals;
  // (after an overflow misc holds the first attempt's counts)
  hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, s, (int32_t*)in.misc + kOver,
                     (int64_t)(kMisc - kOver), 0);
  hipLaunchKernelGGL(k_coo_compact<K>, dim3((unsigned)in.ntiles), dim3(kBlock), 0, s, in.i, in.j,
                     ncoo, n, cb, in.tileoff, keys, vals);
  if constexpr (sizeof(K) == 8)
    SPX_TRY(radix_sort_pairs_u64(keys, keys + cap, vals, vals_alt, nvalid, 2 * cb, work, s, &skeys,
                                 &svals));
  else
    SPX_TRY(radix_sort_pairs_u32(keys, keys + cap, vals, vals_alt, nvalid, 2 * cb, work, s, &skeys,
                                 &svals));
  hipLaunchKernelGGL(k_heads_count<K>, dim3((unsigned)vt), dim3(kBlock), 0, s, skeys, nvalid,
                     tilecnt);
  SPX_TRY(exclusive_scan_u32(tilecnt, tilecnt, vt, in.misc + kNnz, work, s));
  uint32_t host[kMisc];
  SPX_TRY(read_misc(in.misc, host, s));
  SPX_TRY(alloc_pattern(h, host[kNnz], s));
  hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, 256)), dim3(256), 0, s, h->A.dpos, n, -1);
  hipLaunchKernelGGL(k_heads_emit<K>, dim3((unsigned)vt), dim3(kBlock), 0, s, skeys, nvalid, cb,
                     tilecnt, h->jmap, h->A.col, h->A.rowptr, h->A.dpos);
  hipLaunchKernelGGL(k_rowptr_tail<K>, dim3(grid_for(n + 1, 256)), dim3(256), 0, s, skeys, nvalid,
                     cb, n, in.misc + kNnz, h->A.rowptr, h->jmap);
  SPX_TRY(finish_pattern(h, host[kNnz], in.misc, work, host, s));
  // the sorted values are perm: that buffer stays
  mem.n = 3;
  if (svals == vals) mem.p[2] = vals_alt;
  h->perm = reinterpret_cast<int32_t*>(svals);
  return SPX_OK;
}

int symbolic(spx_matrix* h, const int32_t* i, const int32_t* j, hipStream_t s) {
  const int64_t n = h->n, ncoo = h->ncoo;
  const int64_t ntiles = std::max<int64_t>(1, ceil_div(ncoo, kTile));
  Scratch mem(s);
  uint32_t* misc = nullptr;
  SPX_TRY(mem.get(&misc, (size_t)(kMisc + 2 * ntiles + scan_scratch_elems(2 * ntiles))));
  uint32_t* cnt = misc + kMisc;
  hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, s, (int32_t*)misc, (int64_t)kMisc, 0);
  hipLaunchKernelGGL(k_coo_count, dim3((unsigned)ntiles), dim3(kBlock), 0, s, i, j, ncoo, n, ntiles,
                     cnt, (int32_t*)misc + kErr);
  SPX_TRY(exclusive_scan_u32(cnt, cnt, 2 * ntiles, misc + kBoth, cnt + 2 * ntiles, s, ntiles,
                             misc + kKept));
  uint32_t host[kMisc];
  SPX_TRY(read_misc(misc, host, s));
  if (host[kErr])
    return set_error(SPX_INDEX_OUT_OF_RANGE, "coo_preallocate: a COO index is >= n (%lld)",
                     (long long)n);
  const CooIn in{i, j, ntiles, host[kKept], (int64_t)host[kBoth] - host[kKept], misc, cnt};
  h->nvalid = in.nvalid;
  // (with more triplets than all rows' tiles hold, one of them overflows)
  if (h->colbits <= kRowColBits && in.nvalid <= kRowCap * n) {
    bool overflow = false;
    SPX_TRY(symbolic_rows(h, in, s, &overflow));
    if (!overflow) return SPX_OK;
  }
  return 2 * h->colbits <= 32 ? symbolic_full<uint32_t>(h, in, s)
                              : symbolic_full<uint64_t>(h, in, s);
}

}  // namespace

int ensure_transpose(spx_matrix* h, hipStream_t s) {
  const int64_t n = h->n, nnz = h->A.nnz;
  if (!h->has_t) {
    const int64_t cap = std::max<int64_t>(nnz, 1);
    {
      Scratch mem(s);
      Parts parts;
      const int64_t o_key = parts.take(cap), o_key2 = parts.take(cap), o_val = parts.take(cap),
                    o_val2 = parts.take(cap), o_row = parts.take(cap), o_stat = parts.take(kMisc),
                    o_work = parts.take(std::max(radix_sort_work(nnz, h->colbits),
                                                 window_scratch(n)));
      uint32_t* w = nullptr;
      SPX_TRY(mem.get(&w, (size_t)parts.words));
      int32_t *rowidx = (int32_t*)(w + o_row), *stat = (int32_t*)(w + o_stat);
      SPX_TRY(dalloc_n(&h->At.rowptr, (size_t)n + 1));
      SPX_TRY(dalloc_n(&h->At.col, (size_t)cap));
      SPX_TRY(dalloc_n(&h->At.val, (size_t)cap));
      SPX_TRY(dalloc_n(&h->At.dpos, (size_t)n));
      SPX_TRY(dalloc_n(&h->tmap, (size_t)cap));
      hipLaunchKernelGGL(k_expand_rows, dim3(grid_for(n, 256)), dim3(256), 0, s, h->A.rowptr, n,
                         rowidx);
      uint32_t *sk = nullptr, *sv = nullptr;
      SPX_TRY(radix_sort_pairs_u32(w + o_key, w + o_key2, w + o_val, w + o_val2, nnz, h->colbits,
                                   w + o_work, s, &sk, &sv,
                                   reinterpret_cast<const uint32_t*>(h->A.col), true));
      hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, 256)), dim3(256), 0, s, h->At.dpos, n, -1);
      hipLaunchKernelGGL(k_transpose_emit, dim3(grid_for(nnz, 256)), dim3(256), 0, s, sk, sv,
                         rowidx, nnz, h->At.rowptr, h->At.col, h->At.dpos);
      hipLaunchKernelGGL(k_transpose_tail, dim3(grid_for(n + 1, 256)), dim3(256), 0, s, sk, nnz, n,
                         h->At.rowptr);
      if (nnz > 0)
        SPX_CHECK_HIP(hipMemcpyAsync(h->tmap, sv, sizeof(int32_t) * (size_t)nnz,
                                     hipMemcpyDeviceToDevice, s));
      hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, s, stat, (int64_t)kMisc, 0);
      h->At.n = n;
      h->At.nnz = nnz;
      launch_row_stats(h->At, n, stat + kStats, s);
      Window win;
      uint32_t host[kMisc];
      int st = window_enqueue(h->At, nnz, nullptr, w + o_work, (uint32_t*)stat + kWin, s, &win);
      if (st == SPX_OK) st = read_misc((const uint32_t*)stat, host, s);
      if (st != SPX_OK) {
        window_release(&win);
        return st;
      }
      set_row_stats(h->At, (const int32_t*)(host + kStats));
      window_keep(h->At, host + kWin, &win);
    }
    h->has_t = true;
    h->valT_fresh = false;
  }
  if (!h->valT_fresh) {
    hipLaunchKernelGGL(k_gather_vals, dim3(grid_for(nnz, 256)), dim3(256), 0, s, h->tmap, h->A.val,
                       nnz, h->At.val);
    h->valT_fresh = true;
    h->valT32_fresh = false;
  }
  return SPX_OK;
}

int ensure_val32(spx_matrix* h, hipStream_t s) {
  if (!h->A.val32) SPX_TRY(dalloc_n(&h->A.val32, (size_t)std::max<int64_t>(h->A.nnz, 1)));
  if (!h->val32_fresh) {
    hipLaunchKernelGGL(k_to_f32, dim3(grid_for(h->A.nnz, 256)), dim3(256), 0, s, h->A.val,
                       h->A.nnz, h->A.val32);
    h->val32_fresh = true;
  }
  return SPX_OK;
}

int ensure_kslot(spx_matrix* h, hipStream_t s) {
  if (h->kslot) return SPX_OK;
  SPX_TRY(dalloc_n(&h->kslot, (size_t)std::max<int64_t>(h->ncoo, 1)));
  hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(h->ncoo, 256)), dim3(256), 0, s, h->kslot, h->ncoo,
                     -1);
  hipLaunchKernelGGL(k_kslot, dim3(grid_for(h->A.nnz, 256)), dim3(256), 0, s, h->jmap, h->perm,
                     h->A.nnz, h->kslot);
  return SPX_OK;
}

}  // namespace spx

using namespace spx;

extern "C" int spx_coo_preallocate(int64_t n, int64_t ncoo, const int32_t* i, const int32_t* j,
                                   void* stream, spx_handle* out) {
  clear_error();
  if (!out) return set_error(SPX_INVALID_ARG, "coo_preallocate: out is NULL");
  *out = nullptr;
  if (n <= 0 || n > INT32_MAX - 1)
    return set_error(SPX_INVALID_ARG, "coo_preallocate: n = %lld out of [1, 2^31-2]", (long long)n);
  if (ncoo < 0 || ncoo > INT32_MAX - 1)
    return set_error(SPX_INVALID_ARG, "coo_preallocate: ncoo = %lld out of [0, 2^31-2]",
                     (long long)ncoo);
  if (ncoo > 0 && (!i || !j)) return set_error(SPX_INVALID_ARG, "coo_preallocate: i or j is NULL");
  hipStream_t s = static_cast<hipStream_t>(stream);
  spx_matrix* h = new (std::nothrow) spx_matrix();
  if (!h) return set_error(SPX_OUT_OF_MEMORY, "coo_preallocate: host allocation failed");
  SPX_CHECK_HIP(hipGetDevice(&h->device));
  h->n = n;
  h->ncoo = ncoo;
  int cb = 0;
  while (cb < 31 && ((int64_t)1 << cb) < n) ++cb;  // bits of n-1
  h->colbits = cb;
  const int st = symbolic(h, i, j, s);
  if (st != SPX_OK) {
    spx_destroy(h);
    return st;
  }
  *out = h;
  return SPX_OK;
}

namespace spx {
int set_values_into(spx_handle h, const double* v, int mode, double* out, hipStream_t s) {
  const int64_t nnz = h->A.nnz;
  if (nnz > 0) {
    const int ents = sv_entries(h->nvalid, nnz);
    hipLaunchKernelGGL(k_set_values_tiled, dim3(grid_for(nnz, ents)), dim3(256), 0, s, h->jmap,
                       h->perm, v, nnz, mode, ents, out);
  }
  SPX_CHECK_HIP(hipGetLastError());
  return SPX_OK;
}
}  // namespace spx

extern "C" int spx_set_values_coo(spx_handle h, const double* v, int mode, void* stream) {
  clear_error();
  if (!h) return set_error(SPX_INVALID_ARG, "set_values_coo: NULL handle");
  if (mode != SPX_INSERT_VALUES && mode != SPX_ADD_VALUES)
    return set_error(SPX_INVALID_ARG, "set_values_coo: mode %d is not INSERT(0) or ADD(1)", mode);
  if (h->nvalid > 0 && !v) return set_error(SPX_INVALID_ARG, "set_values_coo: v is NULL");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int64_t nnz = h->A.nnz;
  if (nnz > 0) {
    const int ents = sv_entries(h->nvalid, nnz);
    hipLaunchKernelGGL(k_set_values_tiled, dim3(grid_for(nnz, ents)), dim3(256), 0, s, h->jmap,
                       h->perm, v, nnz, mode, ents, h->A.val);
  }
  h->valT_fresh = false;
  h->val32_fresh = false;
  h->valT32_fresh = false;
  SPX_CHECK_HIP(hipGetLastError());
  return SPX_OK;
}

extern "C" int spx_get_info(spx_handle h, int64_t* n, int64_t* nnz, int64_t* nvalid,
                            int64_t* ncoo) {
  clear_error();
  if (!h) return set_error(SPX_INVALID_ARG, "get_info: NULL handle");
  if (n) *n = h->n;
  if (nnz) *nnz = h->A.nnz;
  if (nvalid) *nvalid = h->nvalid;
  if (ncoo) *ncoo = h->ncoo;
  return SPX_OK;
}

extern "C" int spx_get_csr(spx_handle h, int32_t transpose, int32_t* rowptr, int32_t* col,
                           double* val, void* stream) {
  clear_error();
  if (!h) return set_error(SPX_INVALID_ARG, "get_csr: NULL handle");
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (transpose) SPX_TRY(ensure_transpose(h, s));
  const Csr& M = transpose ? h->At : h->A;
  if (rowptr)
    SPX_CHECK_HIP(hipMemcpyAsync(rowptr, M.rowptr, sizeof(int32_t) * (size_t)(h->n + 1),
                                 hipMemcpyDeviceToDevice, s));
  if (col && M.nnz)
    SPX_CHECK_HIP(hipMemcpyAsync(col, M.col, sizeof(int32_t) * (size_t)M.nnz,
                                 hipMemcpyDeviceToDevice, s));
  if (val && M.nnz)
    SPX_CHECK_HIP(hipMemcpyAsync(val, M.val, sizeof(double) * (size_t)M.nnz,
                                 hipMemcpyDeviceToDevice, s));
  return SPX_OK;
}

extern "C" int spx_get_coo_maps(spx_handle h, int32_t* jmap, int32_t* perm, void* stream) {
  clear_error();
  if (!h) return set_error(SPX_INVALID_ARG, "get_coo_maps: NULL handle");
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (jmap)
    SPX_CHECK_HIP(hipMemcpyAsync(jmap, h->jmap, sizeof(int32_t) * (size_t)(h->A.nnz + 1),
                                 hipMemcpyDeviceToDevice, s));
  if (perm && h->nvalid)
    SPX_CHECK_HIP(hipMemcpyAsync(perm, h->perm, sizeof(int32_t) * (size_t)h->nvalid,
                                 hipMemcpyDeviceToDevice, s));
  return SPX_OK;
}

extern "C" int spx_coo_gather(spx_handle h, const double* G, double* grad_v, void* stream) {
  clear_error();
  if (!h || (h->ncoo > 0 && (!G || !grad_v)))
    return set_error(SPX_INVALID_ARG, "coo_gather: NULL argument");
  hipStream_t s = static_cast<hipStream_t>(stream);
  SPX_TRY(ensure_kslot(h, s));
  if (h->ncoo > 0)
    hipLaunchKernelGGL(k_coo_gather, dim3(grid_for(h->ncoo, 256)), dim3(256), 0, s, h->kslot, G,
                       h->ncoo, grad_v);
  SPX_CHECK_HIP(hipGetLastError());
  return SPX_OK;
}

extern "C" int spx_coo_gather_blocks(spx_handle h, const double* G, const double* w,
                                     int64_t block, double* grad_e, void* stream) {
  clear_error();
  if (!h || block <= 0 || (h->ncoo > 0 && (!G || !w || !grad_e)))
    return set_error(SPX_INVALID_ARG, "coo_gather_blocks: bad argument");
  if (h->ncoo % block != 0)
    return set_error(SPX_INVALID_ARG, "coo_gather_blocks: ncoo %lld is not a multiple of %lld",
                     (long long)h->ncoo, (long long)block);
  hipStream_t s = static_cast<hipStream_t>(stream);
  SPX_TRY(ensure_kslot(h, s));
  const int64_t nb = h->ncoo / block;
  if (nb > 0)
    hipLaunchKernelGGL(k_coo_gather_blocks, dim3(grid_for(nb, 256)), dim3(256), 0, s, h->kslot, G,
                       w, nb, block, grad_e);
  SPX_CHECK_HIP(hipGetLastError());
  return SPX_OK;
}
