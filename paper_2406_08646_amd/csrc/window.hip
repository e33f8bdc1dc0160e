// Window index of a CSR pattern for the window walk of the products: per
// tile of kWinRows rows, the ascending list of the kWinBlock-entry blocks of
// x that its columns fall in, and each entry's position in that list.
// Also, where every tile's rows repeat a few patterns, each row's pattern, so
// that the products need not read the columns.
// Built on the device once per pattern (after the symbolic assembly, and for
// the explicit transpose when it is built): one kernel marks each tile's
// blocks in an LDS bitmap, numbers them and writes the tile's list and its
// 16-bit window columns; a scan of the lists' lengths and a small copy then
// put the lists back to back.  The host reads only the statistics, and
// drops the index where it would not pay.  Values are never touched, so
// set_values_coo keeps it valid.
#include <algorithm>
#include <climits>

#include "common.hpp"
#include "device.hpp"

namespace spx {

namespace {

constexpr int kPatTry = 8;
constexpr int kWinWords = kWinSpan / 32;  // bitmap words of one tile
static_assert(kWinWords == kWinRows, "one bitmap word per thread");
static_assert(kWinMaxBlocks * kWinBlock <= 65536, "window columns fit in 16 bits");

__device__ __forceinline__ int32_t wg_min(int32_t v, int32_t* red) {
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
  __syncthreads();  // earlier readers of red are done
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return min(min(red[0], red[1]), min(red[2], red[3]));
}

__device__ __forceinline__ int32_t wg_max(int32_t v, int32_t* red) {
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return max(max(red[0], red[1]), max(red[2], red[3]));
}

// Per tile: cnt[t] blocks in its window (0 if it gets none), their numbers
// ascending in list[t kWinMaxBlocks ..], and lcol[e] = (rank of e's block) *
// kWinBlock + col[e] % kWinBlock.  stats[0] += entries of tiles without a
// window; stats[1] = largest window.  Once *off is set (the pattern is then
// not the final one) every cnt is 0, so that their scan names no place, and
// nothing else is written.  The tile's columns are read three times, the
// later ones from the caches.
// Also the tile's row patterns (row and pat, see Window): the lists are
// found one after the other, each the first row's that has none yet, and
// compared with every such row's in LDS.  A mesh tile has 1 to about 12; a
// tile whose first kPatTry lists hold less than a quarter of its rows is
// given up.  *nopat is set where a tile with a window has no patterns, and no
// further tile looks for any; one without a window shows in stats[0] (a store
// to one address by each of them took 1.2 ms instead of 0.24 on 5M rows of
// random columns).  No patterns are looked for without row.
__global__ __launch_bounds__(kWinRows) void k_win_tiles(int64_t n, const int32_t* __restrict__ rowptr,
                                                        const int32_t* __restrict__ col,
                                                        const uint32_t* __restrict__ off,
                                                        uint32_t* __restrict__ cnt,
                                                        int32_t* __restrict__ list,
                                                        uint16_t* __restrict__ lcol,
                                                        unsigned long long* __restrict__ stats,
                                                        uint32_t* __restrict__ row,
                                                        uint16_t* __restrict__ pat,
                                                        uint32_t* __restrict__ nopat) {
  __shared__ uint16_t lc[kPatLen * kWinRows];
  __shared__ uint32_t bits[kWinWords];
  __shared__ uint32_t incl[kWinWords];
  __shared__ int32_t red[kWinRows / 64];
  __shared__ int32_t range[2];
  const int64_t t = blockIdx.x;
  if (off && *off) {
    if (threadIdx.x == 0) cnt[t] = 0;
    return;
  }
  const int64_t r0 = t * kWinRows;
  const int64_t r1 = r0 + kWinRows < n ? r0 + kWinRows : n;
  const int32_t t0 = rowptr[r0], t1 = rowptr[r1];
  const int tid = threadIdx.x;
  if (t0 == t1) {
    if (tid == 0) cnt[t] = 0;
    if (row && tid < r1 - r0) row[r0 + tid] = 0;
    return;
  }
  int32_t lo = INT_MAX, hi = -1;
  for (int32_t e = t0 + tid; e < t1; e += kWinRows) {
    const int32_t b = col[e] / kWinBlock;
    lo = min(lo, b);
    hi = max(hi, b);
  }
  lo = wg_min(lo, red);
  hi = wg_max(hi, red);
  int32_t c = 0;
  uint32_t word = 0;
  if (hi - lo < kWinSpan) {
    bits[tid] = 0;
    __syncthreads();
    // most entries find their block marked: a read shared by the wave
    // instead of one atomic after the other on the same word
    for (int32_t e = t0 + tid; e < t1; e += kWinRows) {
      const int32_t d = col[e] / kWinBlock - lo;
      const uint32_t m = 1u << (d & 31);
      if (!(__hip_atomic_load(&bits[d >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & m))
        atomicOr(&bits[d >> 5], m);
    }
    __syncthreads();
    // inclusive counts of the bitmap's words
    word = bits[tid];
    int32_t inc = __popc(word);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t v = __shfl_up(inc, o, 64);
      if ((tid & 63) >= o) inc += v;
    }
    if ((tid & 63) == 63) red[tid >> 6] = inc;
    __syncthreads();
    for (int k = 0; k < kWinRows / 64; ++k) {
      if (k < (tid >> 6)) inc += red[k];
      c += red[k];
    }
    incl[tid] = (uint32_t)inc;
    if (c > kWinMaxBlocks) c = 0;
  }
  if (tid == 0) {
    cnt[t] = (uint32_t)c;
    // one address for every tile: an atomic only where it changes something
    if (c == 0)
      atomicAdd(&stats[0], (unsigned long long)(t1 - t0));
    else if ((unsigned long long)c >
             __hip_atomic_load(&stats[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(&stats[1], (unsigned long long)c);
  }
  if (c == 0) return;
  const int32_t rs = tid < r1 - r0 ? rowptr[r0 + tid] - t0 : 0;
  const int32_t len = tid < r1 - r0 ? rowptr[r0 + tid + 1] - t0 - rs : 0;
  const bool fit = __syncthreads_and(len <= kPatLen) && row;
  uint32_t rank = incl[tid] - __popc(word);
  for (uint32_t m = word; m != 0; m &= m - 1)
    list[t * kWinMaxBlocks + rank++] = lo + tid * 32 + (__ffs(m) - 1);
  __syncthreads();
  for (int32_t e = t0 + tid; e < t1; e += kWinRows) {
    const int32_t cc = col[e];
    const int32_t d = cc / kWinBlock - lo;
    const uint32_t w = bits[d >> 5];
    const uint32_t r = incl[d >> 5] - __popc(w) + __popc(w & ((1u << (d & 31)) - 1u));
    const uint16_t v = (uint16_t)(r * kWinBlock + cc % kWinBlock);
    lcol[e] = v;
    if (fit) lc[e - t0] = v;
  }
  if (!row) return;
  __shared__ uint32_t quit;
  if (tid == 0)
    quit = __hip_atomic_load(nopat, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) |
           (__hip_atomic_load(&stats[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0);
  __syncthreads();
  if (quit) return;
  int id = len > 0 ? -1 : 0;
  bool found = fit;
  for (int p = 0; found; ++p) {
    const int32_t lead = wg_min(id < 0 ? tid : INT_MAX, red);
    if (lead == INT_MAX) break;
    if (tid == lead) {
      range[0] = rs;
      range[1] = len;
    }
    __syncthreads();
    found = p < kPats;
    if (!found) break;
    const int32_t ls = range[0], ll = range[1];
    if (id < 0 && len == ll) {
      bool same = true;
      for (int k = 1; same && k < len; ++k)
        same = (uint16_t)(lc[rs + k] - lc[rs]) == (uint16_t)(lc[ls + k] - lc[ls]);
      if (same) id = p;
    }
    if (tid < kPatLen)
      pat[(t * kPats + p) * kPatLen + tid] = tid < ll ? (uint16_t)(lc[ls + tid] - lc[ls]) : 0;
    if (p == kPatTry - 1) found = 4 * __syncthreads_count(id >= 0) >= kWinRows;
  }
  if (!found) {
    if (tid == 0) *nopat = 1;
    return;
  }
  if (tid < r1 - r0) row[r0 + tid] = (len > 0 ? lc[rs] : 0) | (uint32_t)id << 16;
}

// The lists back to back at ptr (a wave per tile), unless *off is set or they
// exceed cap (the index is then dropped).
__global__ __launch_bounds__(kWinRows) void k_win_lists(int64_t tiles, const int32_t* __restrict__ ptr,
                                                        const int32_t* __restrict__ list,
                                                        const uint32_t* __restrict__ off,
                                                        int64_t cap, int32_t* __restrict__ blk) {
  const int64_t t = (int64_t)blockIdx.x * (kWinRows / 64) + (threadIdx.x >> 6);
  if (t >= tiles || (off && *off) || (int64_t)(uint32_t)ptr[tiles] > cap) return;
  const int32_t k0 = ptr[t], c = ptr[t + 1] - k0;
  const int i = threadIdx.x & 63;
  static_assert(kWinMaxBlocks <= 64, "a lane per block");
  if (i < c) blk[k0 + i] = list[t * kWinMaxBlocks + i];
}

// An index that pays holds at most two x entries per matrix entry.
int64_t most_blocks(int64_t nnz) { return 2 * nnz / kWinBlock; }

}  // namespace

int64_t window_scratch(int64_t n) {
  const int64_t tiles = ceil_div(n, kWinRows);
  return tiles + tiles * kWinMaxBlocks + scan_scratch_elems(tiles);
}

int window_enqueue(const Csr& A, int64_t most, const uint32_t* off, uint32_t* scratch,
                   uint32_t* stats, hipStream_t s, Window* w) {
  *w = Window();
  if (A.n == 0 || most == 0) return SPX_OK;
  const int64_t tiles = ceil_div(A.n, kWinRows), cap = most_blocks(most);
  // products walk by patterns from 1.5 entries a row on; they are 8 bytes a row
  const bool patterns = 2 * most > 3 * A.n;
  const int64_t words = tiles + 1 + cap, row = (words + 15) & ~int64_t(15);
  const int64_t pat = patterns ? (row + A.n + 15) & ~int64_t(15) : row;
  const int64_t lcol = patterns ? pat + tiles * (kPats * kPatLen / 2) : row;
  int32_t* block = nullptr;
  const int st = dalloc(reinterpret_cast<void**>(&block),
                        (size_t)(lcol * 4 + most * (int64_t)sizeof(uint16_t) + 128));
  if (st == SPX_OUT_OF_MEMORY) {
    clear_error();
    return SPX_OK;
  }
  SPX_TRY(st);
  w->block = block;
  w->ptr = block;
  w->blk = block + tiles + 1;
  w->row = patterns ? reinterpret_cast<uint32_t*>(block + row) : nullptr;
  w->pat = patterns ? reinterpret_cast<uint16_t*>(block + pat) : nullptr;
  w->lcol = reinterpret_cast<uint16_t*>(block + lcol);
  uint32_t* cnt = scratch;
  int32_t* list = reinterpret_cast<int32_t*>(scratch + tiles);
  uint32_t* work = scratch + tiles + tiles * kWinMaxBlocks;
  uint32_t* ptr = reinterpret_cast<uint32_t*>(w->ptr);
  hipLaunchKernelGGL(k_win_tiles, dim3((unsigned)tiles), dim3(kWinRows), 0, s, A.n, A.rowptr, A.col,
                     off, cnt, list, w->lcol, reinterpret_cast<unsigned long long*>(stats), w->row, w->pat, stats + 5);
  SPX_TRY(exclusive_scan_u32(cnt, ptr, tiles, ptr + tiles, work, s, 0, nullptr));
  hipLaunchKernelGGL(k_win_lists, dim3((unsigned)ceil_div(tiles, kWinRows / 64)), dim3(kWinRows), 0,
                     s, tiles, w->ptr, list, off, cap, w->blk);
  SPX_CHECK_HIP(hipMemcpyAsync(stats + 4, ptr + tiles, sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
  SPX_CHECK_HIP(hipGetLastError());
  return SPX_OK;
}

void window_release(Window* w) {
  dfree(w->block);
  *w = Window();
}

// Keeps w as A's index, or drops it when the window walk would not pay: the
// staged windows would hold more than two x entries per matrix entry, or
// more than one entry in eight would sit in tiles without a window.
void window_keep(Csr& A, const uint32_t* stats, Window* w) {
  window_release(&A.win);
  const int64_t gather = (int64_t)(stats[0] | (uint64_t)stats[1] << 32);
  const int64_t largest = (int64_t)(stats[2] | (uint64_t)stats[3] << 32);
  const int64_t total = stats[4];
  if (w->block && largest > 0 && total <= most_blocks(A.nnz) && gather * 8 <= A.nnz) {
    A.win = *w;
    A.win.max_blocks = largest;
    A.win.total_blocks = total;
    A.win.gather_entries = gather;
    A.win.patterned = w->row && stats[5] == 0 && gather == 0;
    *w = Window();
  } else {
    window_release(w);
  }
}

}  // namespace spx

using namespace spx;

extern "C" int spx_get_window(spx_handle h, int32_t transpose, int64_t* stats, int32_t* ptr,
                              int32_t* blk, uint16_t* lcol, void* stream) {
  clear_error();
  if (!h || !stats) return set_error(SPX_INVALID_ARG, "get_window: NULL handle or stats");
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (transpose) SPX_TRY(ensure_transpose(h, s));
  const Csr& M = transpose ? h->At : h->A;
  const Window& w = M.win;
  stats[0] = w.lcol ? 1 : 0;
  stats[1] = w.max_blocks;
  stats[2] = w.total_blocks;
  stats[3] = w.gather_entries;
  if (!w.lcol) return SPX_OK;
  const int64_t tiles = ceil_div(M.n, kWinRows);
  if (ptr)
    SPX_CHECK_HIP(hipMemcpyAsync(ptr, w.ptr, sizeof(int32_t) * (size_t)(tiles + 1),
                                 hipMemcpyDeviceToDevice, s));
  if (blk && w.total_blocks)
    SPX_CHECK_HIP(hipMemcpyAsync(blk, w.blk, sizeof(int32_t) * (size_t)w.total_blocks,
                                 hipMemcpyDeviceToDevice, s));
  if (lcol && M.nnz)
    SPX_CHECK_HIP(hipMemcpyAsync(lcol, w.lcol, sizeof(uint16_t) * (size_t)M.nnz,
                                 hipMemcpyDeviceToDevice, s));
  return SPX_OK;
}
