// Reduce stage (Sec. 3.1 / 3.3 / 3.4): one output token per cluster = mean of its member tokens, rows in
// ascending cluster id. Integer plumbing: rank of every root (prefix sum over tiles), member lists (stable
// LSD radix sort of the list elements by cluster id), then the one feature pass that gathers and averages.
//
// A list element is a cell, or -- when the caller hands over the stage-1 partition -- a whole node at level
// >= 3, represented by its top-left cell: its per-channel sum was stored by the spatial pass, so its up to
// 4^level cells are not read again; the other cells of such a node take no part in the list ("dropped", key -1).
#include "sttm_dev.h"

namespace sttm {

constexpr int kSortTile = 2048;  // elements per workgroup of the sort kernels
// The sort kernels run a few microseconds on a handful of workgroups each, and what a workgroup spends there is mostly
// the first fetch of its instructions (about 40 ns per 64 bytes of straight-line code: a one-workgroup scatter pass of
// 16 KB took 11 us). So a tile is spread over many wavefronts with few elements each instead of being unrolled eight
// deep in four of them, and nothing is inlined more than once.
constexpr int kPrepThreads = 1024;
constexpr int kPrepPer = kSortTile / kPrepThreads;
constexpr int kSortThreads = 512;
constexpr int kSortPer = kSortTile / kSortThreads;
constexpr int kSortWaves = kSortThreads / kWave;
constexpr int kMaxDigitBits = 11;
// The list of an input of up to this many cells is made by one launch (k_list_small); beyond it the sort passes are as fast:
// the reduce stage of 47,000 to 50,700 cells 40-54 us either way, of 63,488 61 by one launch and 54.
// (The host-thread build of the tests that takes the large inputs' kernels takes the sort passes as well.)
#ifndef STTM_LIST_MAX
#if defined(STTM_PYR_TILES_MAX) && STTM_PYR_TILES_MAX == 0
#define STTM_LIST_MAX 0
#else
#define STTM_LIST_MAX 49152
#endif
#endif
constexpr int kListMax = STTM_LIST_MAX;
static_assert(kListMax < 65536, "cells and counts in 16 bits");
constexpr int kListThreads = 1024;
constexpr int kListTiny = 1024, kListThreadsTiny = 256;  // of up to this many cells: 576 cells 16.9 us by 1024 threads, 16.4;
                                                         // 2304 cells 26 and 28
// Cells up to which the count has a word for every id: 10,816 cells 9.5 us and 9.9 by half words, 512 cells 4.6 and 4.8; 16,384
// 12.8 and 11.7, 35,280 20.6 and 18.3 (twice the LDS to clear and to add up).
constexpr int kListWide = kListMax < 12288 ? kListMax : 12288;
constexpr int kListSlice = 256;  // cells that a workgroup puts into the list
constexpr int kListBatch = 4;    // cells per lane whose loads are in flight together
constexpr int kListPieces = 3;   // pieces of the count per lane whose loads are
constexpr int kListRuns = kListMax / 128 * 2 + 2;  // runs of 64 ids, at most
static_assert(kListMax == 0 || (kListRuns <= kListThreads && kListTiny / 128 * 2 + 2 <= kListThreadsTiny), "a thread per run");
static_assert(kListSlice <= kListThreadsTiny, "a thread per cell");
constexpr int kItem = 16;  // list positions per gather item
constexpr int kBig = 64;   // clusters with more list slots than this are summed item by item, then combined
constexpr int kMaxDigits = 1 << kMaxDigitBits;
// How a scatter workgroup gets its start offsets from hist[tile][digit]: up to kDirectTiles tiles it adds up all
// rows itself; up to kGroupTiles * kMaxGroups tiles a small kernel first adds the rows in groups of kGroupTiles
// and the workgroup adds the group sums and the rows of its own group; beyond that k_sort_colscan turns the
// columns into running sums in place.
constexpr int kDirectTiles = 64;
constexpr int kGroupTiles = 32;
constexpr int kMaxGroups = 256;

struct SortPlan {
  int passes, dbits, nb;
  int mode;  // 0 = direct, 1 = grouped, 2 = column scan
};

static SortPlan sort_plan(int N) {
  SortPlan p;
  int bits = 1;
  while ((1ll << bits) < (long long)N) ++bits;  // keys 0..N-1
  p.passes = max(2, (bits + kMaxDigitBits - 1) / kMaxDigitBits);
  p.dbits = (bits + p.passes - 1) / p.passes;
  if (p.dbits < 2) p.dbits = 2;  // a histogram row is read in pieces of four digits
  p.nb = (N + kSortTile - 1) / kSortTile;
  p.mode = p.nb <= kDirectTiles ? 0 : (p.nb <= kGroupTiles * kMaxGroups ? 1 : 2);
  return p;
}

size_t reduce_tiles(int N) { return (size_t)(N + kSortTile - 1) / kSortTile; }
size_t reduce_gsum_entries() { return (size_t)kMaxGroups * kMaxDigits; }
size_t reduce_hist_entries(int N) { return (size_t)kMaxDigits * reduce_tiles(N); }

// Exclusive prefix of v over the threads of a workgroup of WAVES wavefronts; *total = sum over all threads.
template <int WAVES>
__device__ inline int block_exclusive_scan(int v, int* total) {
  __shared__ int wsum[WAVES];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  int base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    if (w < wave) base += wsum[w];
    tot += wsum[w];
  }
  __syncthreads();
  *total = tot;
  return base + inc - v;
}

__device__ inline int node_cells(const Geo& g, int cell_in_frame, int lvl) {
  const int y = cell_in_frame / g.W, x = cell_in_frame - y * g.W, s = 1 << lvl;
  return (min(y + s, g.H) - y) * (min(x + s, g.W) - x);
}
// True when the node with top-left cell c (in-frame index) at level lv is represented by its stored sum.
__device__ inline bool node_is_summed(const Geo& g, int c, int lv) { return lv >= 3 && node_cells(g, c, lv) >= 2; }
// The cell that stands for the second half of a summed node: the next valid cell of the node in raster order.
__device__ inline int node_second_cell(const Geo& g, int c) { return (c % g.W) + 1 < g.W ? c + 1 : c + g.W; }

// ------------------------------------------------------------------------------------------------
// k_reduce_prep: one workgroup per tile of 2048 cells. Sort keys (cluster id, or -1 for a cell covered by a
// stored node sum), tile-local exclusive ranks of the roots (cells that are their own cluster id), the
// tile's number of roots, and the tile's digit histogram of the first sort pass.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kPrepThreads) void k_reduce_prep(Geo g, const int32_t* __restrict__ cluster_ids,
                                                              const int32_t* __restrict__ node_map,
                                                              const uint8_t* __restrict__ node_level, int dbits,
                                                              int32_t* __restrict__ keys, int32_t* __restrict__ rank,
                                                              int32_t* __restrict__ tile_roots,
                                                              int32_t* __restrict__ hist,
                                                              int32_t* __restrict__ bigcount) {
  constexpr int kWaves = kPrepThreads / kWave;
  __shared__ int cnt[kMaxDigits];
  __shared__ int wroots[kWaves];
  const int DIG = 1 << dbits, b = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int e0 = b * kSortTile + wave * (kPrepPer * kWave) + lane;  // a wavefront takes consecutive cells
  int cid[kPrepPer], rep[kPrepPer], lv[kPrepPer];
#pragma unroll
  for (int r = 0; r < kPrepPer; ++r) {  // all loads first: they do not depend on one another
    const int i = min(e0 + r * kWave, g.N - 1);
    cid[r] = cluster_ids[i];
    rep[r] = lv[r] = 0;
    if (node_map) {
      rep[r] = node_map[i];
      lv[r] = node_level[i];
    }
  }
  for (int d = tid; d < DIG; d += kPrepThreads) cnt[d] = 0;
  if (b == 0 && tid == 0) *bigcount = 0;  // the list of big clusters starts empty
  __syncthreads();
  int before[kPrepPer], nroot = 0;  // roots of the wavefront before this cell
#pragma unroll
  for (int r = 0; r < kPrepPer; ++r) {
    const int i = e0 + r * kWave;
    const bool in = i < g.N;
    const unsigned long long roots = __ballot(in && cid[r] == i);
    before[r] = nroot + __popcll(roots & ((1ull << lane) - 1ull));
    nroot += __popcll(roots);
    if (in) {
      bool live = true;
      if (lv[r] >= 3) {  // a node with a stored sum: only the cells standing for it stay
        const int c = rep[r] % g.HW;
        if (node_is_summed(g, c, lv[r]))
          live = i == rep[r] || (g.vec == 8 && i == rep[r] - c + node_second_cell(g, c));
      }
      keys[i] = live ? cid[r] : -1;
      if (live) atomicAdd(&cnt[cid[r] & (DIG - 1)], 1);
    }
  }
  if (lane == 0) wroots[wave] = nroot;
  __syncthreads();
  int base = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    if (w < wave) base += wroots[w];
    total += wroots[w];
  }
#pragma unroll
  for (int r = 0; r < kPrepPer; ++r)
    if (e0 + r * kWave < g.N) rank[e0 + r * kWave] = base + before[r];
  if (tid == 0) tile_roots[b] = total;
  for (int d = tid; d < DIG; d += kPrepThreads) hist[(size_t)b * DIG + d] = cnt[d];
}

// Digit histogram per tile of the (compacted) keys of a later pass; tiles beyond the list write zeros.
__global__ __launch_bounds__(kSortThreads) void k_sort_hist(const int32_t* __restrict__ kdev, int shift, int dbits,
                                                            const uint2* __restrict__ pairs,
                                                            int32_t* __restrict__ hist) {
  __shared__ int cnt[kMaxDigits];
  const int DIG = 1 << dbits, b = blockIdx.x, tid = threadIdx.x, n = kdev[1];
  for (int d = tid; d < DIG; d += kSortThreads) cnt[d] = 0;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSortPer; ++j) {
    const int i = b * kSortTile + j * kSortThreads + tid;
    if (i < n) atomicAdd(&cnt[((int)pairs[i].x >> shift) & (DIG - 1)], 1);
  }
  __syncthreads();
  for (int d = tid; d < DIG; d += kSortThreads) hist[(size_t)b * DIG + d] = cnt[d];
}

// Large inputs only: turns every column (digit) of hist[tile][digit] into its exclusive prefix over the
// tiles and leaves the column total in tot[digit].
__global__ __launch_bounds__(256) void k_sort_colscan(int nb, int DIG, int32_t* __restrict__ hist,
                                                      int32_t* __restrict__ tot) {
  const int d = blockIdx.x * blockDim.x + threadIdx.x;
  if (d >= DIG) return;
  int run = 0;
  for (int t = 0; t < nb; ++t) {
    const int v = hist[(size_t)t * DIG + d];
    hist[(size_t)t * DIG + d] = run;
    run += v;
  }
  tot[d] = run;
}

// Medium inputs: gsum[group][digit] = sum of the group's rows of hist[tile][digit]; one thread per digit, the
// group's rows in two batches of loads.
__global__ __launch_bounds__(256) void k_sort_groupsum(int nb, int DIG, const int32_t* __restrict__ hist,
                                                       int32_t* __restrict__ gsum) {
  const int d = blockIdx.x * blockDim.x + threadIdx.x, grp = blockIdx.y;
  if (d >= DIG) return;
  const int t0 = grp * kGroupTiles;
  int run = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    int v[kGroupTiles / 2];
#pragma unroll
    for (int u = 0; u < kGroupTiles / 2; ++u) {
      const int t = t0 + h * (kGroupTiles / 2) + u;
      v[u] = t < nb ? hist[(size_t)t * DIG + d] : 0;
    }
#pragma unroll
    for (int u = 0; u < kGroupTiles / 2; ++u) run += v[u];
  }
  gsum[(size_t)grp * DIG + d] = run;
}

// Adds rows [r0, r1) of a table of 2^dbits-int rows to at[] (if to_total) and, for the rows below `limit`, to
// am[]. The table is read as 16-byte pieces, consecutive threads next to each other, eight loads in flight per
// thread; the four digits a thread sees do not change from load to load (a row has at most as many pieces as the
// workgroup has threads).
__device__ inline void sort_add_rows(const int32_t* __restrict__ table, int r0, int r1, int dbits, int limit,
                                     bool to_total, int (&at)[4], int (&am)[4]) {
  constexpr int kBatch = 8;
  static_assert(kMaxDigits / 4 <= kSortThreads, "one digit piece per thread");
  const int vshift = dbits - 2;  // log2 of the 16-byte pieces per row
  const int first = r0 << vshift, last = r1 << vshift;
  const int4* h4 = reinterpret_cast<const int4*>(table);
  const int take_total = to_total ? -1 : 0;
#pragma unroll 1
  for (int q0 = first + (int)threadIdx.x; q0 < last; q0 += kBatch * kSortThreads) {
    int4 v[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) v[u] = h4[min(q0 + u * kSortThreads, last - 1)];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int q = q0 + u * kSortThreads;
      const int in = q < last ? -1 : 0, mb = (q >> vshift) < limit ? in : 0, mt = in & take_total;
      at[0] += v[u].x & mt; at[1] += v[u].y & mt; at[2] += v[u].z & mt; at[3] += v[u].w & mt;
      am[0] += v[u].x & mb; am[1] += v[u].y & mb; am[2] += v[u].z & mb; am[3] += v[u].w & mb;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// k_sort_pass: one stable scatter pass, one workgroup per tile of 2048 elements. The workgroup first turns
// the histogram into its own start offset for every digit (summing the columns over the tiles before it
// unless k_sort_colscan did so), then every wavefront ranks its 256 consecutive elements 64 at a time in
// index order (ballot matching), so the order of equal keys is kept.
//   FIRST: elements are the cells themselves (value = index), dropped cells (key < 0) stay behind, so the
//          output is compact. Also makes the root ranks global, and writes out_ids, the per-video offsets
//          and the totals (K, list length).
//   LAST:  writes the sorted element list, the output row of every list position and the first list
//          position of every row (the root is the smallest index of its cluster, hence first in its list).
// A wavefront's cursors are counts inside the tile (at most 2048) and are kept as 16-bit halves, two digits to a word.
// ------------------------------------------------------------------------------------------------
struct SortArgs {
  int n, shift, dbits, nb, mode;  // mode: how the start offsets are found (see kDirectTiles)
  const int32_t* gsum;
  const int32_t* keys;  // FIRST
  const uint2* in;      // else: (key, cell)
  uint2* out;           // LAST: the sorted element list, (cell, output row)
  const int32_t* hist;
  const int32_t* tot;
  // FIRST
  const int32_t* cluster_ids;
  int32_t* rank;
  const int32_t* tile_roots;
  int32_t* kdev;  // [0] = K, [1] = list length
  int32_t* host_k;  // K once more, in host memory (or NULL)
  int32_t* out_ids;
  int64_t* offsets;
  int64_t capacity;
  int per_video, B;
  // LAST
  int32_t* seg;
};

template <bool FIRST, bool LAST>
__global__ __launch_bounds__(kSortThreads) void k_sort_pass(SortArgs a) {
  __shared__ int s_base[kMaxDigits];                  // first list position of every digit for this tile
  __shared__ unsigned cur[kSortWaves * kMaxDigits / 2];  // [wavefront][two digits to a word]
  __shared__ int s_roots[2];                          // roots in the tiles before this one, and in all
  const int DIG = 1 << a.dbits, b = blockIdx.x, tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = FIRST ? a.n : a.kdev[1];

  // ---- everything this tile reads per element is requested first, so that it arrives while the offsets
  //      are worked out (a position beyond the list reads something stale that is not used)
  const int e0 = b * kSortTile + wave * (kSortTile / kSortWaves);
  int key[kSortPer], val[kSortPer], aux[kSortPer];
  int rk0[kSortPer], cid[kSortPer];
#pragma unroll
  for (int r = 0; r < kSortPer; ++r) {
    const int i = e0 + r * 64 + lane, j = min(i, a.n - 1);
    if (FIRST) {
      key[r] = a.keys[j];
      val[r] = i;
    } else {
      const uint2 e = a.in[j];
      key[r] = (int)e.x;
      val[r] = (int)e.y;
    }
    rk0[r] = FIRST ? a.rank[j] : 0;
    cid[r] = FIRST ? a.cluster_ids[j] : 0;
  }
  int roots_before = 0, roots_all = 0;
  if (FIRST) {
    for (int t = tid; t < a.nb; t += kSortThreads) {
      const int v = a.tile_roots[t];
      roots_all += v;
      if (t < b) roots_before += v;
    }
  }

  // ---- start offset of every digit for this tile
  int* tot = reinterpret_cast<int*>(cur);  // column totals and the part of them that lies in the tiles before this one
  int* mine = tot + kMaxDigits;            // (the cursors are not in use yet)
  static_assert(kSortWaves >= 4, "the two column tables fit the cursors' place");
  if (tid < 2) s_roots[tid] = 0;
  for (int d = tid; d < DIG; d += kSortThreads) tot[d] = mine[d] = 0;
  __syncthreads();
  if (FIRST) {
    if (roots_before) atomicAdd(&s_roots[0], roots_before);
    if (roots_all) atomicAdd(&s_roots[1], roots_all);
  }
  if (a.mode != 2) {
    int at[4] = {0, 0, 0, 0}, am[4] = {0, 0, 0, 0};
    const int grp = b / kGroupTiles, ngrp = (a.nb + kGroupTiles - 1) / kGroupTiles;
#pragma unroll 1
    for (int part = 0; part <= a.mode; ++part) {
      // mode 0: all rows of all tiles; mode 1: the sums of all groups, then the rows of this tile's own group
      const bool sums = a.mode == 1 && part == 0, own = part == 1;
      sort_add_rows(sums ? a.gsum : a.hist, own ? grp * kGroupTiles : 0,
                    sums ? ngrp : (own ? min(a.nb, (grp + 1) * kGroupTiles) : a.nb), a.dbits, sums ? grp : b, !own, at, am);
    }
    const int vc = tid & ((1 << (a.dbits - 2)) - 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (at[i]) atomicAdd(&tot[vc * 4 + i], at[i]);
      if (am[i]) atomicAdd(&mine[vc * 4 + i], am[i]);
    }
  } else {
    for (int d = tid; d < DIG; d += kSortThreads) {
      tot[d] = a.tot[d];
      mine[d] = a.hist[(size_t)b * DIG + d];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortPer; ++r) {
    if (e0 + r * 64 + lane >= n) key[r] = -1;
    aux[r] = 0;
    if (LAST && key[r] >= 0) aux[r] = a.rank[key[r]];  // output row of the element's cluster (arrives during the scan)
  }
  {
    constexpr int kDpt = kMaxDigits / kSortThreads;
    const int dpt = DIG >= kSortThreads ? DIG / kSortThreads : 1;
    int tv[kDpt], cv[kDpt], s = 0;
#pragma unroll
    for (int j = 0; j < kDpt; ++j) {
      const int d = tid * dpt + j;
      const bool in = j < dpt && d < DIG;
      tv[j] = in ? tot[d] : 0;
      cv[j] = in ? mine[d] : 0;
      s += tv[j];
    }
    int live;  // all elements of the list
    int ex = block_exclusive_scan<kSortWaves>(s, &live);  // (its barriers also fence the reads above from the clearing below)
#pragma unroll
    for (int j = 0; j < kDpt; ++j) {
      const int d = tid * dpt + j;
      if (j < dpt && d < DIG) s_base[d] = ex + cv[j];
      ex += tv[j];
    }
    if (b == 0 && tid == 0) {
      if (FIRST) {
        const int all = s_roots[1];
        a.kdev[0] = all;
        if (a.host_k) *a.host_k = all;
        a.kdev[1] = live;
        a.offsets[a.B] = all;
      } else if (LAST) {
        a.seg[a.kdev[0]] = n;
      }
    }
  }
  const int hd = DIG >> 1;
  for (int d = tid; d < kSortWaves * hd; d += kSortThreads) cur[d] = 0;
  __syncthreads();

  // ---- per-wavefront digit counts of its 256 elements
  unsigned* mycur = cur + wave * hd;
#pragma unroll
  for (int r = 0; r < kSortPer; ++r) {
    const int digit = (key[r] >> a.shift) & (DIG - 1);
    if (key[r] >= 0) atomicAdd(&mycur[digit >> 1], 1u << ((digit & 1) * 16));
  }
  if (FIRST) {
    // bookkeeping outputs of the cells themselves; the wavefront's first video start at or after its first cell
    const int root_prefix = s_roots[0];
    int video = (e0 + a.per_video - 1) / a.per_video;
    long long start = (long long)video * a.per_video;
#pragma unroll
    for (int r = 0; r < kSortPer; ++r) {
      const int i = e0 + r * 64 + lane;
      const int rk = rk0[r] + root_prefix;
      if (i < n) {
        if (b != 0) a.rank[i] = rk;
        if (cid[r] == i && a.out_ids && rk < a.capacity) a.out_ids[rk] = i;
      }
      for (; start < e0 + (r + 1) * 64 && start < n; start += a.per_video, ++video)
        if (i == start) a.offsets[video] = rk;
    }
  }
  __syncthreads();
  for (int d = tid; d < hd; d += kSortThreads) {
    unsigned run = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
      const unsigned c = cur[w * hd + d];
      cur[w * hd + d] = run;
      run += c;
    }
  }
  __syncthreads();

  // ---- ranked scatter, 64 elements at a time in index order: first which lanes hold the same digit (no
  //      memory involved), then the cursors
  const unsigned long long below = (1ull << lane) - 1ull;
  unsigned long long same[kSortPer];
#pragma unroll
  for (int r = 0; r < kSortPer; ++r) same[r] = __ballot(key[r] >= 0);
#pragma unroll 1
  for (int bit = 0; bit < a.dbits; ++bit) {
#pragma unroll
    for (int r = 0; r < kSortPer; ++r) {
      const bool one = (key[r] >> (a.shift + bit)) & 1;
      const unsigned long long m = __ballot(one);
      same[r] &= one ? m : ~m;
    }
  }
#pragma unroll
  for (int r = 0; r < kSortPer; ++r) {  // the stores of one round travel while the next round's cursors are read
    const int digit = (key[r] >> a.shift) & (DIG - 1), half = (digit & 1) * 16;
    if (key[r] >= 0) {
      const int dst = s_base[digit] + (int)((mycur[digit >> 1] >> half) & 0xffffu) + __popcll(same[r] & below);
      // (in one piece: what bounds this pass on a large input is lines that are written eight bytes at a time)
      a.out[dst] = LAST ? make_uint2((unsigned)val[r], (unsigned)aux[r]) : make_uint2((unsigned)key[r], (unsigned)val[r]);
      if (LAST && key[r] == val[r]) a.seg[aux[r]] = dst;
    }
    wave_lds_fence();
    if (r + 1 < kSortPer && key[r] >= 0 && ((same[r] >> lane) >> 1) == 0)  // highest lane of its digit group advances the cursor
      atomicAdd(&mycur[digit >> 1], (unsigned)__popcll(same[r]) << half);
    wave_lds_fence();
  }
}

// The value of the lane before (the first one: 0), and this lane's bit of a mask.
#ifndef STTM_HOST_EMULATION
__device__ inline int lane_before(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xF, 0xF, true); }  // wave_shr:1
__device__ inline bool from_mask(unsigned long long m, int) { return __builtin_amdgcn_inverse_ballot_w64(m); }
#else
inline int lane_before(int v) { const int r = __shfl_up(v, 1, 64); return (threadIdx.x & 63) ? r : 0; }
inline bool from_mask(unsigned long long m, int lane) { return (m >> lane) & 1ull; }
#endif

// ------------------------------------------------------------------------------------------------
// k_list_small: all of the integer plumbing of a small input in one launch. A workgroup puts kListSlice consecutive cells
// into the list. The place of an element is the number of elements with a smaller id plus that of earlier ones with the
// same id; both come from a count of every id, which each workgroup keeps in LDS and makes by itself from all cells of the
// input. For the earlier ones of an id it either counts the cells before its own beside all of them, 32 bits an id (WIDE),
// or counts those before its own first, then its own, then the rest, 16 bits an id. Its own cells take their turns, a
// wavefront after the other. Ranks come from a bit per cell, "is a root". No workgroup waits for another: what they would
// have to tell each other every one finds out by itself, at 4 bytes a cell (9 with the partition) from the caches.
// Writes what the sort passes write (rank, list, output row of every position, first position of every row, out_ids,
// offsets, totals).
// What bounds it: the look over all cells by every workgroup, by its instructions (about 25 vector ones for 64 cells, 16
// wavefronts a workgroup) and the LDS atomics; by time stamps, 45,000 cells: 11 us of 18 with 3 for the sums over the count.
// The work does not depend on the labelling: a workgroup for 256 ids that found and sorted their cells did all the work
// alone where a still scene leaves the cells of all frames to the first frame's ids. Whole reduce stage at D = 256, us, that
// kernel and this one: 300 still frames of 13x13 130 -> 42, 64 of them 49 -> 32; moving scenes of 92 frames of 13x13 44 -> 37,
// 64 of 16x16 45 -> 37, 512 of 8x8 45 -> 47; the launch alone in passes of the package's workloads 9.0 -> 9.5 (10,816 cells),
// 11.1 -> 11.7 (16,384), 14.1 -> 13.1 (20,064), 15.8 -> 18.3 (35,280), 20.4 -> 20.3 (45,000).
// ------------------------------------------------------------------------------------------------
struct ListArgs {
  int n, W;
  int both_halves;        // both_halves: a stored node sum takes two list elements (16-bit input)
  unsigned inv_w;         // where a node may be one column wide (W = 9, 17, 25): 2^32 / W rounded up, exact for 16-bit numerators
  int words;                  // of the count
  int id_bits;
  const int32_t* cluster_ids;
  const int32_t* node_map;    // the stage-1 partition, or both NULL
  const uint8_t* node_level;
  int32_t* rank;
  int32_t* kdev;
  int32_t* host_k;
  int32_t* out_ids;
  int64_t* offsets;
  int64_t capacity;
  int per_video, B;
  uint2* list;
  int32_t* seg;
};

// The count's words for n ids, whole runs of 64: WIDE one for every id, with the cells before the workgroup's own in its low
// half and all of them in its high one; otherwise id j is in the low half of word j, id words + j in the high one. (Neighbouring
// ids are in different words: the cells of a row of lanes mostly have ids in a row, and two atomics on one word would take
// their turns.)
static int list_words(int n, bool wide) { return wide ? (n + 63) / 64 * 64 : (n + 127) / 128 * 64; }

template <int THREADS, bool WIDE>
__global__ __launch_bounds__(THREADS) void k_list_small(ListArgs a) {
  constexpr int WAVES = THREADS / kWave;
  STTM_DYNAMIC_LDS(unsigned, count);                 // [words]
  __shared__ __attribute__((aligned(16))) unsigned long long s_roots[kListRuns + 2];  // a bit per cell; whole batches of rows
  __shared__ unsigned s_first[kListRuns];            // per run of 64 ids: elements (low half) and roots in the runs before it
  __shared__ unsigned s_none[64];                    // where additions of nothing go
  __shared__ unsigned s_wave[WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lo = blockIdx.x * kListSlice, hi = min(a.n, lo + kListSlice), rows = (a.n + 63) >> 6;
  const unsigned long long before = (1ull << lane) - 1ull;

  // the id of cell i, whose node's top-left cell is rep and level lv; -1 if the cell is not an element of the list
  auto element_id = [&](int i, int cid, int rep, int lv) {
    // of a node with a stored sum only its top-left cell stays and, where that takes two elements, its next cell in
    // raster order: the one to the right, or in a node of one column the one below
    const int past = i - rep;
    bool dropped = (lv >= 3) & ((unsigned)past > (unsigned)a.both_halves);
    if (a.inv_w && a.both_halves) {
      const int col = i - (int)((unsigned long long)(unsigned)i * a.inv_w >> 32) * a.W;
      dropped &= (past != a.W) | (col != a.W - 1);
    }
    return (!dropped & ((unsigned)cid < (unsigned)a.n)) ? cid : -1;
  };
  auto word = [&](int id) { return count + (WIDE ? (unsigned)id : min((unsigned)id, (unsigned)id - (unsigned)a.words)); };
  auto low = [&](int id) { return WIDE || id < a.words; };

  const int own = lo + tid;  // the cell that this thread places (of the first kListSlice threads)
  const bool mine = tid < kListSlice && own < hi;
  int own_cid = -1, own_rep = 0, own_lv = 0;
  if (mine) {
    own_cid = a.cluster_ids[own];
    if (a.node_map) {
      own_rep = a.node_map[own];
      own_lv = a.node_level[own];
    }
  }
  for (int d = tid; d < a.words >> 2; d += THREADS) reinterpret_cast<uint4*>(count)[d] = make_uint4(0u, 0u, 0u, 0u);
  const int per = a.words >> 6, runs = WIDE ? per : 2 * per;
  if (tid < runs) s_roots[tid] = 0;
  __syncthreads();
  const int id = mine ? element_id(own, own_cid, own_rep, own_lv) : -1;
  int place = 0;  // of the own element among those with its id
  unsigned long long same = 0;  // the wavefront's own cells with that id
  const Window ids = make_window(a.cluster_ids, (unsigned)a.n * 4u), reps = make_window(a.node_map, a.node_map ? (unsigned)a.n * 4u : 0u),
               levels = make_window(a.node_level, a.node_map ? (unsigned)a.n : 0u);
  struct Rows { int cid[kListBatch], rep[kListBatch], lv[kListBatch]; };
  auto load = [&](Rows& q, int r0) {  // (zeros behind the last cell)
#pragma unroll
    for (int u = 0; u < kListBatch; ++u) {
      q.cid[u] = window_load_i32(ids, (unsigned)(lane * 4 + u * 256), (unsigned)r0 * 256u);
      q.rep[u] = q.lv[u] = 0;
      if (a.node_map) {
        q.rep[u] = window_load_i32(reps, (unsigned)(lane * 4 + u * 256), (unsigned)r0 * 256u);
        q.lv[u] = window_load_u8(levels, (unsigned)(lane + u * 64), (unsigned)r0 * 64u);
      }
    }
  };
  // WIDE: all rows of 64 cells. Otherwise those before the own ones, then those behind.
#pragma unroll 1
  for (int part = 0; part < (WIDE ? 1 : 2); ++part) {
    const int rb = part ? (hi + 63) >> 6 : 0, r1 = WIDE || part ? rows : lo >> 6, end = min(a.n, r1 * 64);
    // Batches of rows; workgroups of one die (they are dealt to the eight in turn) begin at different places, so that not all of
    // them wait for the same lines to reach the die's L2.
    const int batches = (max(0, r1 - rb) + kListBatch - 1) / kListBatch, skip = batches * (int)(blockIdx.x >> 3 & 15) >> 4;
    auto row_of = [&](int j) { return rb + (j + skip < batches ? j + skip : j + skip - batches) * kListBatch; };
    Rows next;
    if (wave < batches) load(next, row_of(wave));
    if (part == 0 && wave < kListSlice / 64) {  // (while these are on their way)
      const unsigned long long roots = __ballot(mine && own_cid == own);
      if (lane == 0 && (lo >> 6) + wave < rows) s_roots[(lo >> 6) + wave] = roots;
      same = __ballot(id >= 0);
#pragma unroll 1
      for (int bit = 0; bit < a.id_bits; ++bit) {
        const bool set = (id >> bit) & 1;
        const unsigned long long m = __ballot(set);
        same &= set ? m : ~m;
      }
    }
#pragma unroll 1
    for (int j = wave; j < batches; j += WAVES) {
      const int r0 = row_of(j);
      const Rows now = next;  // the next rows are on their way while these are counted
      if (j + WAVES < batches) load(next, row_of(j + WAVES));
      unsigned long long roots[kListBatch];
      int e[kListBatch];
#pragma unroll
      for (int u = 0; u < kListBatch; ++u) {
        const int i = (r0 + u) * 64 + lane;
        roots[u] = __ballot(now.cid[u] == i);
        e[u] = a.node_map ? element_id(i, now.cid[u], now.rep[u], now.lv[u]) : ((unsigned)now.cid[u] < (unsigned)a.n ? now.cid[u] : -1);
      }
      if ((r0 + kListBatch) * 64 > end) {
#pragma unroll
        for (int u = 0; u < kListBatch; ++u) e[u] = (r0 + u) * 64 + lane < end ? e[u] : -1;
      }
      const int twice = r0 * 64 < lo ? -1 : 0;
#pragma unroll
      for (int u = 0; u < kListBatch; ++u) {
        // Neighbours with the same id (a merged node's cells; their atomics would take their turns) are counted as one run:
        // its first lane takes its number off, its last one adds its own and one. Whoever has nothing to add does so in a
        // word of its own: a branch around the atomic costs more.
        const unsigned long long heads = __ballot(e[u] != lane_before(e[u])) | 1ull, tails = heads >> 1 | 1ull << 63;
        const unsigned long long act = __ballot(e[u] >= 0) & (heads | tails);
        const unsigned add = (unsigned)((from_mask(tails, lane) ? lane + 1 : 0) - (from_mask(heads, lane) ? lane : 0));
        const unsigned sum = WIDE ? (add << 16) + (add & (unsigned)twice) : add << (low(e[u]) ? 0 : 16);
        atomicAdd(from_mask(act, lane) ? word(e[u]) : s_none + lane, sum);
      }
      if (lane == 0) {
#pragma unroll
        for (int u = 0; u < kListBatch; ++u) s_roots[r0 + u] = roots[u];
      }
    }
    if (part) break;
    // the own cells, a wavefront after the other
#pragma unroll 1
    for (int w = 0; w < kListSlice / 64; ++w) {
      __syncthreads();
      if (wave != w) continue;
      if (id >= 0) place = (int)(low(id) ? *word(id) & 0xffffu : *word(id) >> 16) + __popcll(same & before);
      wave_lds_fence();
      if (id >= 0 && ((same >> lane) >> 1) == 0)  // the highest lane of an id's group counts them all
        atomicAdd(word(id), (unsigned)__popcll(same) << (low(id) ? 0 : 16));
    }
    __syncthreads();  // (nobody counts the cells behind before the last of these has its place)
  }
  if (!WIDE) __syncthreads();
  // the count of every id -> that of the ids before it in its run of 64, and the runs' totals (both halves side by side:
  // all totals together fit 16 bits)
#pragma unroll 1
  for (int d0 = wave * 256; d0 < a.words; d0 += WAVES * 256 * kListPieces) {  // 16 lanes, four words each, to a run
    uint4 c[kListPieces];
#pragma unroll
    for (int k = 0; k < kListPieces; ++k) {
      const int d = d0 + k * WAVES * 256 + lane * 4;
      c[k] = make_uint4(0u, 0u, 0u, 0u);
      if (d < a.words) c[k] = *reinterpret_cast<const uint4*>(count + d);
    }
#pragma unroll
    for (int k = 0; k < kListPieces; ++k) {
      const int d = d0 + k * WAVES * 256 + lane * 4;
      if (WIDE) { c[k].x >>= 16; c[k].y >>= 16; c[k].z >>= 16; c[k].w >>= 16; }
      c[k].y += c[k].x; c[k].z += c[k].y; c[k].w += c[k].z;
      const unsigned upto = row16_inclusive(c[k].w, lane), ex = upto - c[k].w;
      if (d < a.words) {
        *reinterpret_cast<uint4*>(count + d) = make_uint4(ex, ex + c[k].x, ex + c[k].y, ex + c[k].z);
        if ((lane & 15) == 15) {
          s_first[d >> 6] = upto & 0xffffu;
          if (!WIDE) s_first[per + (d >> 6)] = upto >> 16;
        }
      }
    }
  }
  __syncthreads();
  const unsigned run = tid < runs ? s_first[tid] | (unsigned)__popcll(s_roots[tid]) << 16 : 0u;
  const unsigned upto = wave_inclusive(run, lane);
  if (lane == 63) s_wave[wave] = upto;
  __syncthreads();
  const int waves = (int)row16_inclusive(lane < WAVES ? s_wave[lane] : 0u, lane);
  const unsigned all = (unsigned)lane_value(waves, WAVES - 1);
  const unsigned earlier = wave ? (unsigned)lane_value(waves, wave - 1) : 0u;  // (by all lanes of the wavefront)
  if (tid < runs) s_first[tid] = earlier + upto - run;
  __syncthreads();
  auto rank_of = [&](int i) {
    return (int)(s_first[i >> 6] >> 16) + __popcll(s_roots[i >> 6] & ((1ull << (i & 63)) - 1ull));
  };
  if (mine) {
    const int rk = rank_of(own);
    a.rank[own] = rk;
    if (own_cid == own && a.out_ids && rk < a.capacity) a.out_ids[rk] = own;
    if (own % a.per_video == 0) a.offsets[own / a.per_video] = rk;
    if (id >= 0) {
      const unsigned ex = *word(id);
      const int dst = (int)((s_first[id >> 6] & 0xffffu) + (low(id) ? ex & 0xffffu : ex >> 16)) + place;
      a.list[dst] = make_uint2((unsigned)own, (unsigned)rank_of(id));
      if (id == own) a.seg[rk] = dst;
    }
  }
  if (tid == 0) {
    if (blockIdx.x == 0) a.kdev[2] = 0;  // the list of big clusters starts empty
    if (hi == a.n) {
      const int k = (int)(all >> 16), live = (int)(all & 0xffffu);
      a.kdev[0] = k;
      if (a.host_k) *a.host_k = k;
      a.kdev[1] = live;
      a.offsets[a.B] = k;
      a.seg[k] = live;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// The gather/average pass. Every list slot is one 16-byte load per lane: a cell's row (VEC channels of the
// input type), or four fp32 channels of a stored node sum -- with bf16 input a lane owns eight channels, so
// such a node takes two slots (its top-left cell and the next cell of the node stand for the two halves).
// The list is cut into items of kItem consecutive slots; an item owns the clusters whose list starts
// inside it. One wavefront per (item, chunk of the row). All index look-ups of the item are done
// lane-parallel first, then all loads are issued, then the slots are added up in list order (fp32) with the
// cluster boundaries handled as wave-uniform control flow. A cluster with more than kBig slots is not
// followed past the item: every item adds up the slots of such a cluster that lie inside it and leaves the
// partial sum in the workspace (at most two per item: the cluster running in from the left and the one
// starting inside), the item in which the cluster starts puts it on a list, and k_reduce_big_combine adds
// the partial sums up in item order -- so the summation order does not depend on scheduling.
// ------------------------------------------------------------------------------------------------

// Where a list slot's data lives.
struct Slot {
  int kind;    // 0 = cell row, 1 / 2 = first / second four channels of a lane's share of a node sum
  int idx;     // flat cell index, or row of the node-sum table
  int weight;  // member cells it stands for
};

template <int DT>
__device__ inline Slot describe(const Geo& g, const int32_t* __restrict__ node_map,
                                const uint8_t* __restrict__ lvl, int cell) {
  Slot e;
  e.kind = 0;
  e.idx = cell;
  e.weight = 1;
  if (lvl) {
    const int lv = lvl[cell];
    if (lv >= 3) {
      const int rep = node_map[cell];
      const int f = rep / g.HW, c = rep - f * g.HW;
      if (node_is_summed(g, c, lv)) {
        const int y = c / g.W, x = c - y * g.W;
        e.idx = f * (g.NN - g.lvl_base[3]) + node_index(g, lv, y >> lv, x >> lv) - g.lvl_base[3];
        e.kind = cell == rep ? 1 : 2;
        e.weight = cell == rep ? node_cells(g, c, lv) : 0;
      }
    }
  }
  return e;
}

// Where a slot's row, or its half of the channels of a node's sum, begins.
template <int DT>
__device__ inline uint64_t slot_address(const void* feats, const float* nsum, int D, const Slot& e) {
  const size_t first = (size_t)e.idx * D;
  return e.kind == 0 ? reinterpret_cast<uint64_t>(static_cast<const typename Row<DT>::Elem*>(feats) + first)
                     : reinterpret_cast<uint64_t>(nsum + first + (e.kind - 1) * 4);
}
// The address that lane `src` holds in two halves, in scalar registers; said to be one of global memory (a load from an
// address of any kind counts as one from LDS too, and is waited for as such).
#ifndef STTM_HOST_EMULATION
#define STTM_GLOBAL __attribute__((address_space(1)))
#else
#define STTM_GLOBAL
#endif
__device__ inline char* lane_address(uint2 v, int src) {
  const uint64_t a = (uint64_t)(unsigned)lane_value((int)v.y, src) << 32 | (unsigned)lane_value((int)v.x, src);
  return (char*)(STTM_GLOBAL char*)a;
}
__device__ inline uint2 halves(uint64_t a) { return make_uint2((unsigned)a, (unsigned)(a >> 32)); }

// (fp32 rows and node sums share a layout)
template <int DT>
__device__ inline void acc_slot(const float4& r, unsigned, unsigned, float (&acc)[4]) {
  acc[0] += r.x; acc[1] += r.y; acc[2] += r.z; acc[3] += r.w;
}
// (Three steps, each skipped or not: as one choice of three the sums came out of it in three sets of registers and were
// moved back into one, eight moves a slot. The node sum's two halves add to different channels, so their order is free.)
template <int DT>
__device__ inline void acc_slot(const uint4& r, unsigned half1, unsigned half2, float (&acc)[8]) {
  if (!(half1 | half2)) Row<DT>::add_row(r, acc);
  const float f0 = __uint_as_float(r.x), f1 = __uint_as_float(r.y);
  const float f2 = __uint_as_float(r.z), f3 = __uint_as_float(r.w);
  if (half1) {
    STTM_OPAQUE_S(half1);  // (keeps this a branch; the additions are not made by every slot and dropped)
    acc[0] += f0; acc[1] += f1; acc[2] += f2; acc[3] += f3;
  }
  if (half2) {
    STTM_OPAQUE_S(half2);
    acc[4] += f0; acc[5] += f1; acc[6] += f2; acc[7] += f3;
  }
}

// A lane's channels of a row's mean, written at `to`.
template <int DT, int ODT>
__device__ inline void store_mean(void* to, const float (&acc)[Row<DT>::VEC], float inv) {
  constexpr int VEC = Row<DT>::VEC;
  if (ODT == 0) {
    float* o = static_cast<float*>(to);
#pragma unroll
    for (int v = 0; v < VEC; v += 4)
      store_once(reinterpret_cast<float4*>(o + v),
                 make_float4(acc[v] * inv, acc[v + 1] * inv, acc[v + 2] * inv, acc[v + 3] * inv));
  } else {
    uint32_t w[VEC / 2];
#pragma unroll
    for (int v = 0; v < VEC; v += 2)
      w[v / 2] = ODT == 1 ? pack2_bf16(acc[v] * inv, acc[v + 1] * inv) : pack2_f16(acc[v] * inv, acc[v + 1] * inv);
    if (VEC == 8)
      store_once(static_cast<uint4*>(to), make_uint4(w[0], w[1], w[2 % (VEC / 2)], w[3 % (VEC / 2)]));
    else
      *static_cast<uint2*>(to) = make_uint2(w[0], w[1]);
  }
}

struct GatherArgs {
  const void* feats;
  const float* nsum;
  const int32_t* node_map;  // the stage-1 partition, or both NULL when every slot is a cell
  const uint8_t* lvl;
  const uint2* list;
  const int32_t* seg;
  const int32_t* kdev;
  int64_t capacity;
  void* merged;
  int32_t* counts;
  float* bigpart;     // [items][2][D] partial sums of big clusters
  int32_t* bigw;      // [items][2] member cells behind them
  int4* biglist;      // one entry per big cluster: output row, first list position, end of its list
  int32_t* bigcount;  // length of that list
  const int32_t* zpos;  // output row of every cluster rank when the rows follow the Z-shaped scan, else NULL
};

template <int VEC>
__device__ inline void store_partial(float* o, const float (&acc)[VEC]) {
#pragma unroll
  for (int v = 0; v < VEC; v += 4) *reinterpret_cast<float4*>(o + v) = make_float4(acc[v], acc[v + 1], acc[v + 2], acc[v + 3]);
}

// What a slot asks for is decided for all slots at once, a lane each, and kept as bit masks in scalar registers: per
// slot only its loads, additions and row stores are left, on scalar branches and addresses. The counts, and which
// items hold shares of a big cluster, are written by the lanes together. (Read from lane to lane per slot, by masked
// branches, the kernel was 31 KB of code, now 13: 8 frames of 8x8 tokens 13.1 -> 8.8 us, 96 of 11x19 in fp32 33 -> 26; and it
// issues less: 1024 frames of 27x27 at D = 1152 306 -> 266 us (1.72 GB, 6.5 TB/s), 512 of 13x13 at D = 3584 140 -> 134.)
template <int DT, int ODT>
__global__ __launch_bounds__(64) void k_reduce(Geo g, GatherArgs a) {
  typedef Row<DT> R;
  typedef typename R::Raw Raw;
  constexpr int VEC = R::VEC;
  // one-wavefront workgroups; consecutive ones take the chunks of one item
  const int chunk = blockIdx.x % g.nC, item = blockIdx.x / g.nC, lane = threadIdx.x;
  // Lane j describes list position p0 + j: the item's first, those after it only where its last cluster runs past it. The
  // list entries are requested together with the list's length: entries at or beyond the end are stale and are not used.
  const int p0 = item * kItem, pl = p0 + lane;
  int cell_l = 0, rank_l = 0;
  if (pl < g.N) {
    const uint2 e = a.list[pl];
    cell_l = (int)e.x;
    rank_l = (int)e.y;  // clusters are listed in ascending id; the output row may differ
  }
  const int M = a.kdev[1];
  const int p1 = min(p0 + kItem, M);
  if (p0 >= M) return;
  Slot sv = {0, 0, 0};
  int row_v = -1, beg_v = 0, end_v = 0;
  if (lane < kItem && pl < M) {
    sv = describe<DT>(g, a.node_map, a.lvl, cell_l);
    beg_v = a.seg[rank_l];
    end_v = a.seg[rank_l + 1];
    row_v = a.zpos ? a.zpos[rank_l] : rank_l;
  }
  const bool big = end_v - beg_v > kBig;
  const bool use = pl < p1 && (beg_v >= p0 || big);  // (else the tail of a cluster that an earlier item finishes)
  // a cluster of one cell whose row is written in the type it came in: the mean is the row itself
  const bool one = DT == ODT && use && end_v - beg_v == 1 && sv.kind == 0;
  const bool closes = use && !one && !big && pl + 1 == end_v;
  const bool share = use && big && (pl + 1 == end_v || pl + 1 == p1);  // ends this item's share of a big cluster
  const bool fits = row_v < a.capacity;
  // member cells of the slot's cluster from its first slot in this item up to the slot
  int members = use ? sv.weight : 0;
#pragma unroll
  for (int o = 1; o < kItem; o <<= 1) {
    const int t = __shfl_up(members, o, 64);
    if (lane >= o) members += t;
  }
  members -= __shfl(members, max(beg_v - p0, 0) - 1, 64) * (beg_v > p0);
  unsigned use_m = (unsigned)__ballot(use), one_m = (unsigned)__ballot(one && fits);
  unsigned add_m = (unsigned)__ballot(use && !one), mean_m = (unsigned)__ballot(closes && fits);
  unsigned share_m = (unsigned)__ballot(share), end_m = share_m | (unsigned)__ballot(closes);
  int inv_v = (int)__float_as_uint(1.f / (float)members);
  const int part_slot = beg_v < p0 ? 0 : 1;  // of a big cluster's share: which of the item's two
  if (chunk == 0) {
    if ((one || closes) && fits && a.counts) a.counts[row_v] = members;
    if (share) {
      a.bigw[item * 2 + part_slot] = members;
      if (part_slot == 1) a.biglist[atomicAdd(a.bigcount, 1)] = make_int4(row_v, beg_v, end_v, 0);
    }
  }
  // The cluster still open after the item's last position (the item is full then) is followed to its end, kItem positions at
  // a time. All of these are described at once: the lanes after the item's, and the first ones once more for what lies
  // beyond the last lane.
  constexpr size_t kOutBytes = ODT == 0 ? 4 : 2;
  char* const merged = static_cast<char*>(a.merged);
  const int lastj = p1 - 1 - p0;
  const bool open = (add_m >> lastj & 1u) && !(end_m >> lastj & 1u);
  static_assert(kBig + kItem <= 2 * kWave, "an open cluster's positions");
  int open_row = 0, open_end = 0, open_inv = 0;
  Slot beyond = {0, 0, 0};
  if (open) {
    open_row = lane_value(row_v, kItem - 1);
    open_end = lane_value(end_v, kItem - 1);
    if (lane >= kItem && pl < open_end) sv = describe<DT>(g, a.node_map, a.lvl, cell_l);
    if (pl + kWave < open_end) beyond = describe<DT>(g, a.node_map, a.lvl, (int)a.list[pl + kWave].x);
    const unsigned later = wave_inclusive((unsigned)((lane >= kItem ? sv.weight : 0) + beyond.weight), lane);
    const int total = lane_value(members, kItem - 1) + lane_value((int)later, kWave - 1);
    open_inv = (int)__float_as_uint(1.f / (float)total);
    if (chunk == 0 && lane == 0 && open_row < a.capacity && a.counts) a.counts[open_row] = total;
  }
  // Where each slot's data is and where its result goes, a lane each: per slot two scalar reads are left of either.
  uint2 src = halves(slot_address<DT>(a.feats, a.nsum, g.D, sv));
  uint2 dst = halves(share ? reinterpret_cast<uint64_t>(a.bigpart + ((size_t)item * 2 + part_slot) * g.D)
                           : reinterpret_cast<uint64_t>(merged + (size_t)row_v * g.D * kOutBytes));
  unsigned long long half1_m = __ballot(sv.kind == 1), half2_m = __ballot(sv.kind == 2);
  const int ch0 = chunk * g.cch + lane * VEC;
  const bool act = ch0 < g.D;
  const unsigned chl = act ? (unsigned)ch0 : 0u;  // (a lane beyond the last channel reads the row's first channels and drops them)
  float acc[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
#pragma unroll 1
  for (int base = p0;;) {
    // (The slots' bits and numbers are taken from these registers where they are used: a copy the compiler cannot look
    // through, or it takes all of them out of the loop and runs out of scalar registers.)
    STTM_OPAQUE_S(use_m); STTM_OPAQUE_S(one_m); STTM_OPAQUE_S(add_m);
    STTM_OPAQUE_S(mean_m); STTM_OPAQUE_S(share_m); STTM_OPAQUE_S(end_m);
    STTM_OPAQUE_V(src.x); STTM_OPAQUE_V(src.y); STTM_OPAQUE_V(dst.x); STTM_OPAQUE_V(dst.y); STTM_OPAQUE_V(inv_v);
    unsigned half1 = (unsigned)half1_m, half2 = (unsigned)half2_m;
    STTM_OPAQUE_S(half1); STTM_OPAQUE_S(half2);
    const unsigned wide = half1 | half2;
    Raw raw[kItem];
#pragma unroll
    for (int j = 0; j < kItem; ++j) {
      raw[j] = R::zero();
      // (this is the last use of a feature row, and node sums are read once as well)
      if (use_m >> j & 1u)
        raw[j] = load_once(reinterpret_cast<const Raw*>(lane_address(src, j) + (DT == 0 ? chl * 4u : chl * 2u << (wide >> j & 1u))));
    }
    // (all of them are waited for here: at each slot, behind a branch that may have stored a row, the compiler would wait
    // for that store as well)
#pragma unroll
    for (int j = 0; j < kItem; ++j) {
      STTM_OPAQUE_V(raw[j].x); STTM_OPAQUE_V(raw[j].y); STTM_OPAQUE_V(raw[j].z); STTM_OPAQUE_V(raw[j].w);
    }
#pragma unroll
    for (int j = 0; j < kItem; ++j) {
      // (every lane takes part where another lane's address is read, also those beyond the last channel)
      if (one_m >> j & 1u) {
        char* const to = lane_address(dst, j);
        if (act) store_once(reinterpret_cast<Raw*>(to + chl * (unsigned)kOutBytes), raw[j]);
      }
      if (add_m >> j & 1u) acc_slot<DT>(raw[j], half1 >> j & 1u, half2 >> j & 1u, acc);
      if (end_m >> j & 1u) {
        char* const to = lane_address(dst, j);
        if (mean_m >> j & 1u) {
          const float inv = __uint_as_float((unsigned)lane_value(inv_v, j));
          if (act) store_mean<DT, ODT>(to + chl * (unsigned)kOutBytes, acc, inv);
        } else if (share_m >> j & 1u) {
          if (act) store_partial<VEC>(reinterpret_cast<float*>(to) + chl, acc);
        }
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
      }
    }
    base += kItem;
    if (!open || base >= open_end) break;
    const int left = open_end - base;
    use_m = add_m = left < kItem ? (1u << left) - 1u : (1u << kItem) - 1u;
    end_m = left <= kItem ? 1u << (left - 1) : 0u;
    mean_m = open_row < a.capacity ? end_m : 0u;
    one_m = share_m = 0u;
    dst = halves(reinterpret_cast<uint64_t>(merged + (size_t)open_row * g.D * kOutBytes));
    inv_v = open_inv;
    if (base - p0 == kWave) {  // (at most once: kBig + kItem positions)
      src = halves(slot_address<DT>(a.feats, a.nsum, g.D, beyond));
      half1_m = __ballot(beyond.kind == 1);
      half2_m = __ballot(beyond.kind == 2);
    } else {
      src = make_uint2((unsigned)__shfl_down((int)src.x, kItem, 64), (unsigned)__shfl_down((int)src.y, kItem, 64));
      half1_m >>= kItem;
      half2_m >>= kItem;
    }
  }
}

// A number of workgroups per chunk that follows from the sizes walks the list of big clusters. A cluster's partial sums are added up
// in item order (the starting item's own, then the left-hand shares of the items after it): the run of items is
// cut into kBigSeg contiguous segments, one wavefront each, eight loads in flight, and the segment sums are
// added in segment order through LDS -- an order that depends on the list alone. The workgroups of a chunk: one for every
// kBigPer clusters that the list has room for, but kBigMost at most and at least as many as it takes for two to a compute unit
// in all; and an odd number of them: workgroups go to the eight dies in turn, and by an even number the chunks of a cluster,
// which lie side by side in memory, mostly meet on one. us by 64, by 256, and by this rule:
//   six clips of 25 frames of 15x20, fp32 rows (three chunks; room for 693, few are there)         7.7   12.9    8.1
//   five videos of 115 frames of 17x17, two chunks                                               11.1   13.8    9.9
//   64 frames of 14x16, fp32 rows, seven chunks (room for 221; 73 and 221 alike)                  19.9   12.2   12.0
//   1152 clusters of 100 cells, one chunk                                                        36.5   12.8   12.9
//   2048 clusters of 70 cells, two chunks (nothing but still scenes: an odd number costs here)    60.8   22.1   23.4
//   576 of 90, four chunks                                                                       20.1   15.4   17.3
//   32 videos of 32 frames of 27x27, three chunks                                                11.3    8.5    8.2
constexpr int kBigGrid = 65, kBigMost = 255, kBigPer = 4;
constexpr int kBigBatch = 8;
constexpr int kBigSeg = 8;

template <int DT, int ODT>
__global__ __launch_bounds__(64 * kBigSeg) void k_reduce_big_combine(Geo g, GatherArgs a) {
  constexpr int VEC = Row<DT>::VEC;
  __shared__ float segsum[kBigSeg - 1][64][VEC];
  __shared__ int segmem[kBigSeg];
  const int seg = threadIdx.x >> 6, lane = threadIdx.x & 63, chunk = blockIdx.y;
  const int ch0 = chunk * g.cch + lane * VEC;
  const bool act = ch0 < g.D;
  // (the first entry is requested with the list's length: behind the list's end it is stale and not used)
  int4 en = a.biglist[blockIdx.x];
  const int nbig = *a.bigcount;
  for (int e = blockIdx.x; e < nbig; e += gridDim.x) {  // uniform over the workgroup
    if (e != (int)blockIdx.x) en = a.biglist[e];
    const int k = en.x, it0 = en.y / kItem, it1 = (en.z - 1) / kItem;
    // the partial sums of the cluster: number 0 is the starting item's (slot 1), number j > 0 item it0 + j's (slot 0)
    const int np = it1 - it0 + 1, per = (np + kBigSeg - 1) / kBigSeg;
    const int j0 = min(np, seg * per), j1 = min(np, j0 + per);
    float acc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
    int members = 0;
    for (int j = j0; j < j1; j += kBigBatch) {
      float4 r[kBigBatch][VEC / 4];
#pragma unroll
      for (int u = 0; u < kBigBatch; ++u) {
        const int jj = min(j + u, j1 - 1);
        const float4* q =
            reinterpret_cast<const float4*>(a.bigpart + ((size_t)(it0 + jj) * 2 + (jj == 0 ? 1 : 0)) * g.D + (act ? ch0 : 0));
#pragma unroll
        for (int v = 0; v < VEC / 4; ++v) r[u][v] = q[v];
      }
#pragma unroll
      for (int u = 0; u < kBigBatch; ++u) {
        if (j + u >= j1) continue;
#pragma unroll
        for (int v = 0; v < VEC / 4; ++v) {
          acc[4 * v] += r[u][v].x; acc[4 * v + 1] += r[u][v].y;
          acc[4 * v + 2] += r[u][v].z; acc[4 * v + 3] += r[u][v].w;
        }
      }
    }
    for (int j = j0 + lane; j < j1; j += 64) members += a.bigw[(it0 + j) * 2 + (j == 0 ? 1 : 0)];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) members += __shfl_xor(members, o, 64);
    if (seg > 0) {
#pragma unroll
      for (int v = 0; v < VEC; ++v) segsum[seg - 1][lane][v] = acc[v];
    }
    if (lane == 0) segmem[seg] = members;
    __syncthreads();
    if (seg == 0 && k < a.capacity) {
      int total = 0;
#pragma unroll
      for (int u = 0; u < kBigSeg; ++u) total += segmem[u];
#pragma unroll
      for (int u = 1; u < kBigSeg; ++u)
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] += segsum[u - 1][lane][v];
      if (chunk == 0 && lane == 0 && a.counts) a.counts[k] = total;
      if (act) store_mean<DT, ODT>(static_cast<char*>(a.merged) + ((size_t)k * g.D + ch0) * (ODT == 0 ? 4 : 2), acc, 1.f / (float)total);
    }
    __syncthreads();
  }
}

size_t reduce_items(const Geo& g) { return (size_t)(g.N + kItem - 1) / kItem; }
size_t reduce_bigpart_floats(const Geo& g) { return reduce_items(g) * 2 * g.D; }
size_t reduce_bigw_entries(const Geo& g) { return reduce_items(g) * 2; }
size_t reduce_biglist_entries(const Geo& g) { return (size_t)g.N / (kBig + 1) + 1; }  // a big cluster has > kBig slots

// ------------------------------------------------------------------------------------------------
// Z-shaped scan (Sec. 3.4): inside a frame the rows follow the Morton rank of the root's top-left cell
// instead of its raster index. The clusters stay listed by ascending id (rank); this kernel, one workgroup per
// frame, gives every rank of the frame its output row: the frame's rows are the same range either way, only
// permuted. Needs the global ranks (after the first sort pass). Also writes out_ids in the new order.
// ------------------------------------------------------------------------------------------------
__device__ inline int morton_rank(int y, int x) {
  int z = 0;
#pragma unroll
  for (int b = 0; b < kMaxLevels; ++b) z |= (((x >> b) & 1) << (2 * b)) | (((y >> b) & 1) << (2 * b + 1));
  return z;
}

__global__ __launch_bounds__(256) void k_zorder(Geo g, const int32_t* __restrict__ cluster_ids,
                                                const int32_t* __restrict__ rank, int64_t capacity,
                                                int32_t* __restrict__ zpos, int32_t* __restrict__ out_ids) {
  __shared__ int flag[1024];  // root cells of the frame at their Morton slot, then their exclusive count
  const int f = blockIdx.x, tid = threadIdx.x, PP = g.P * g.P;
  for (int z = tid; z < 1024; z += 256) flag[z] = 0;
  __syncthreads();
  for (int c = tid; c < g.HW; c += 256) {
    const int i = f * g.HW + c;
    if (cluster_ids[i] == i) flag[morton_rank(c / g.W, c % g.W)] = 1;
  }
  __syncthreads();
  // exclusive scan over the (up to 1024) Morton slots: four consecutive slots per thread
  int v[4], sum = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    v[j] = tid * 4 + j < PP ? flag[tid * 4 + j] : 0;
    sum += v[j];
  }
  int total;
  int ex = block_exclusive_scan<256 / kWave>(sum, &total);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (tid * 4 + j < PP) flag[tid * 4 + j] = ex;
    ex += v[j];
  }
  __syncthreads();
  const int r0 = rank[f * g.HW];  // roots before this frame
  for (int c = tid; c < g.HW; c += 256) {
    const int i = f * g.HW + c;
    if (cluster_ids[i] != i) continue;
    const int row = r0 + flag[morton_rank(c / g.W, c % g.W)];
    zpos[rank[i]] = row;
    if (out_ids && row < capacity) out_ids[row] = i;
  }
}

// ------------------------------------------------------------------------------------------------
// Position indices of the output rows (Sec. 3.4). k_positions_cells adds every cell's original index (within
// its video) to its row's integer sum; k_positions_rows turns the sums into means and writes the root's
// own index, the row's index in its video's output, and the root's (t, y0, x0, level).
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_positions_clear(int n, unsigned long long* __restrict__ possum,
                                                         unsigned* __restrict__ poscnt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    possum[i] = 0ull;
    poscnt[i] = 0u;
  }
}

// With the stage-1 partition at hand a whole node is added at once, by its top-left cell: the sum of the indices
// of its valid cells has a closed form, and a cluster made of a few large nodes costs a few atomics instead of
// hundreds on one address.
__global__ __launch_bounds__(256) void k_positions_cells(Geo g, const int32_t* __restrict__ cluster_ids,
                                                         const int32_t* __restrict__ node_map,
                                                         const uint8_t* __restrict__ node_level,
                                                         const int32_t* __restrict__ rank,
                                                         unsigned long long* __restrict__ possum,
                                                         unsigned* __restrict__ poscnt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.N) return;
  const int loc = i % (g.T * g.HW);
  unsigned long long sum = (unsigned long long)loc;
  unsigned cnt = 1u;
  if (node_map) {
    if (node_map[i] != i) return;
    const int c = loc % g.HW, y0 = c / g.W, x0 = c - y0 * g.W, s = 1 << node_level[i];
    const int ny = min(y0 + s, g.H) - y0, nx = min(x0 + s, g.W) - x0;
    // sum over y0 <= y < y0+ny, x0 <= x < x0+nx of (loc + (y - y0) * W + (x - x0))
    cnt = (unsigned)(ny * nx);
    sum = (unsigned long long)cnt * loc + (unsigned long long)nx * g.W * (ny * (ny - 1) / 2) +
          (unsigned long long)ny * (nx * (nx - 1) / 2);
  }
  const int r = rank[cluster_ids[i]];
  atomicAdd(&possum[r], sum);
  atomicAdd(&poscnt[r], cnt);
}

__global__ __launch_bounds__(256) void k_positions_rows(Geo g, const int32_t* __restrict__ kdev,
                                                        const uint2* __restrict__ list,
                                                        const int32_t* __restrict__ seg,
                                                        const int32_t* __restrict__ zpos,
                                                        const uint8_t* __restrict__ node_level,
                                                        const int64_t* __restrict__ offsets,
                                                        const unsigned long long* __restrict__ possum,
                                                        const unsigned* __restrict__ poscnt, int64_t capacity,
                                                        int32_t* __restrict__ survived,
                                                        int32_t* __restrict__ reassigned,
                                                        float* __restrict__ merged_pos,
                                                        int32_t* __restrict__ root_tyxl) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;  // cluster rank (ascending id)
  if (r >= kdev[0]) return;
  const int root = (int)list[seg[r]].x;  // the root is the first element of its cluster's list
  const int row = zpos ? zpos[r] : r;
  if (row >= capacity) return;
  const int per_video = g.T * g.HW, b = root / per_video, loc = root - b * per_video;
  if (survived) survived[row] = loc;
  if (reassigned) reassigned[row] = row - (int)offsets[b];
  if (merged_pos) merged_pos[row] = (float)((double)possum[r] / (double)poscnt[r]);
  if (root_tyxl) {
    const int t = loc / g.HW, c = loc - t * g.HW;
    root_tyxl[4 * row + 0] = t;
    root_tyxl[4 * row + 1] = c / g.W;
    root_tyxl[4 * row + 2] = c % g.W;
    root_tyxl[4 * row + 3] = node_level ? (int)node_level[root] : -1;
  }
}

void launch_positions(const Geo& g, const int32_t* cluster_ids, const int32_t* node_map, const uint8_t* node_level,
                      const int64_t* offsets,
                      int64_t capacity, const ReduceBuffers& rb, bool zscan, unsigned long long* possum,
                      unsigned* poscnt, int32_t* survived, int32_t* reassigned, float* merged_pos,
                      int32_t* root_tyxl, hipStream_t s) {
  const dim3 grid((g.N + 255) / 256), block(256);
  if (merged_pos) {
    hipLaunchKernelGGL(k_positions_clear, grid, block, 0, s, g.N, possum, poscnt);
    hipLaunchKernelGGL(k_positions_cells, grid, block, 0, s, g, cluster_ids, node_level ? node_map : nullptr,
                       node_level, rb.rank, possum, poscnt);
  }
  hipLaunchKernelGGL(k_positions_rows, grid, block, 0, s, g, rb.kdev, rb.list, rb.seg, zscan ? rb.zpos : nullptr,
                     node_level, offsets, possum, poscnt, capacity, survived, reassigned, merged_pos, root_tyxl);
}

// Integer plumbing of the reduce stage: sorted element list, row of every list position, row starts.
void launch_reduce_prepare(const Geo& g, const int32_t* cluster_ids, const int32_t* node_map,
                           const uint8_t* node_level, int64_t capacity, int32_t* out_ids, int64_t* offsets,
                           const ReduceBuffers& rb, bool zscan, hipStream_t s) {
  const int N = g.N;
  if (N <= kListMax) {
    ListArgs a;
    a.n = N; a.W = g.W; a.both_halves = g.vec == 8;
    a.inv_w = (g.W & 7) == 1 && g.W > 1 ? 0xffffffffu / (unsigned)g.W + 1u : 0u;
    a.words = list_words(N, N <= kListWide);
    a.id_bits = 1;
    while ((N - 1) >> a.id_bits) ++a.id_bits;
    a.cluster_ids = cluster_ids; a.node_map = node_map; a.node_level = node_level;
    a.rank = rb.rank; a.kdev = rb.kdev; a.host_k = rb.host_k;
    a.out_ids = zscan ? nullptr : out_ids; a.offsets = offsets; a.capacity = capacity;
    a.per_video = g.T * g.HW; a.B = g.B;
    a.list = rb.list; a.seg = rb.seg;
    const dim3 slices((N + kListSlice - 1) / kListSlice);
    const size_t lds = (size_t)a.words * sizeof(unsigned);
    if (N <= kListTiny)
      hipLaunchKernelGGL((k_list_small<kListThreadsTiny, true>), slices, dim3(kListThreadsTiny), lds, s, a);
    else if (N <= kListWide)
      hipLaunchKernelGGL((k_list_small<kListThreads, true>), slices, dim3(kListThreads), lds, s, a);
    else
      hipLaunchKernelGGL((k_list_small<kListThreads, false>), slices, dim3(kListThreads), lds, s, a);
    if (zscan)
      hipLaunchKernelGGL(k_zorder, dim3(g.F), dim3(256), 0, s, g, cluster_ids, rb.rank, capacity, rb.zpos, out_ids);
    return;
  }
  const SortPlan pl = sort_plan(N);
  const int DIG = 1 << pl.dbits;
  const dim3 grid(pl.nb), block(kSortThreads);
  hipLaunchKernelGGL(k_reduce_prep, grid, dim3(kPrepThreads), 0, s, g, cluster_ids, node_map, node_level, pl.dbits,
                     rb.key, rb.rank, rb.tile_roots, rb.hist, rb.kdev + 2);
  const uint2* in = nullptr;
  uint2* out = rb.pair_b;
  for (int pass = 0; pass < pl.passes; ++pass) {
    const bool first = pass == 0, last = pass == pl.passes - 1;
    if (!first)
      hipLaunchKernelGGL(k_sort_hist, grid, block, 0, s, rb.kdev, pass * pl.dbits, pl.dbits, in, rb.hist);
    if (pl.mode == 2)
      hipLaunchKernelGGL(k_sort_colscan, dim3((DIG + 255) / 256), dim3(256), 0, s, pl.nb, DIG, rb.hist, rb.tot);
    else if (pl.mode == 1)
      hipLaunchKernelGGL(k_sort_groupsum, dim3((DIG + 255) / 256, (pl.nb + kGroupTiles - 1) / kGroupTiles), dim3(256), 0,
                         s, pl.nb, DIG, rb.hist, rb.gsum);
    SortArgs a;
    a.n = N; a.shift = pass * pl.dbits; a.dbits = pl.dbits; a.nb = pl.nb; a.mode = pl.mode; a.gsum = rb.gsum;
    a.keys = rb.key; a.in = in; a.out = last ? rb.list : out;
    a.hist = rb.hist; a.tot = rb.tot;
    a.cluster_ids = cluster_ids; a.rank = rb.rank; a.tile_roots = rb.tile_roots;
    a.kdev = rb.kdev; a.host_k = rb.host_k; a.out_ids = zscan ? nullptr : out_ids; a.offsets = offsets; a.capacity = capacity;
    a.per_video = g.T * g.HW; a.B = g.B;
    a.seg = rb.seg;
    if (first) hipLaunchKernelGGL((k_sort_pass<true, false>), grid, block, 0, s, a);
    else if (last) hipLaunchKernelGGL((k_sort_pass<false, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_sort_pass<false, false>), grid, block, 0, s, a);
    in = out;
    out = out == rb.pair_b ? rb.pair_a : rb.pair_b;
  }
  if (zscan)
    hipLaunchKernelGGL(k_zorder, dim3(g.F), dim3(256), 0, s, g, cluster_ids, rb.rank, capacity, rb.zpos, out_ids);
}

static GatherArgs gather_args(const void* feats, const float* nsum, const int32_t* node_map,
                              const uint8_t* node_level, int64_t capacity, void* merged, int32_t* counts,
                              const ReduceBuffers& rb, bool zscan) {
  GatherArgs a;
  a.feats = feats; a.nsum = nsum; a.node_map = node_map; a.lvl = node_level; a.list = rb.list;
  a.seg = rb.seg; a.kdev = rb.kdev; a.capacity = capacity; a.merged = merged; a.counts = counts;
  a.bigpart = rb.bigpart; a.bigw = rb.bigw;
  a.biglist = reinterpret_cast<int4*>(rb.biglist); a.bigcount = rb.kdev + 2;
  a.zpos = zscan ? rb.zpos : nullptr;
  return a;
}

// Input / output element types a gather kernel is built for: fp32 in with any output type; a 16-bit input with
// the same type or fp32 out (reduce_io_supported() says which pairs exist).
#define STTM_DISPATCH_IO(KERNEL, IN, OUT, GRID, BLOCK, STREAM, ...)                                      \
  do {                                                                                                   \
    const int io_ = (IN) * 3 + (OUT);                                                                    \
    if (io_ == 0) hipLaunchKernelGGL((KERNEL<0, 0>), GRID, BLOCK, 0, STREAM, __VA_ARGS__);               \
    else if (io_ == 1) hipLaunchKernelGGL((KERNEL<0, 1>), GRID, BLOCK, 0, STREAM, __VA_ARGS__);          \
    else if (io_ == 2) hipLaunchKernelGGL((KERNEL<0, 2>), GRID, BLOCK, 0, STREAM, __VA_ARGS__);          \
    else if (io_ == 3) hipLaunchKernelGGL((KERNEL<1, 0>), GRID, BLOCK, 0, STREAM, __VA_ARGS__);          \
    else if (io_ == 4) hipLaunchKernelGGL((KERNEL<1, 1>), GRID, BLOCK, 0, STREAM, __VA_ARGS__);          \
    else if (io_ == 6) hipLaunchKernelGGL((KERNEL<2, 0>), GRID, BLOCK, 0, STREAM, __VA_ARGS__);          \
    else if (io_ == 8) hipLaunchKernelGGL((KERNEL<2, 2>), GRID, BLOCK, 0, STREAM, __VA_ARGS__);          \
  } while (0)

bool reduce_io_supported(int in_dtype, int out_dtype) {
  if (in_dtype < 0 || in_dtype > 2 || out_dtype < 0 || out_dtype > 2) return false;
  return in_dtype == 0 || out_dtype == 0 || out_dtype == in_dtype;
}

// The feature pass of the reduce stage: the gather over the whole list (clusters of up to kBig slots) ...
void launch_reduce_gather(const Geo& g, const void* feats, const float* nsum, const int32_t* node_map,
                          const uint8_t* node_level, int out_dtype, int64_t capacity, void* merged, int32_t* counts,
                          const ReduceBuffers& rb, bool zscan, hipStream_t s) {
  const int nitems = (g.N + kItem - 1) / kItem;
  const dim3 grid((unsigned)nitems * (unsigned)g.nC), block(64);  // (16 KB of features each: fewer than 2^32 threads)
  const GatherArgs a = gather_args(feats, nsum, node_map, node_level, capacity, merged, counts, rb, zscan);
  STTM_DISPATCH_IO(k_reduce, g.dtype, out_dtype, grid, block, s, g, a);
}

// ... and the means of the clusters with more than kBig slots from the partial sums the gather left behind.
void launch_reduce_big(const Geo& g, const void* feats, const float* nsum, const int32_t* node_map,
                       const uint8_t* node_level, int out_dtype, int64_t capacity, void* merged, int32_t* counts,
                       const ReduceBuffers& rb, bool zscan, hipStream_t s) {
  const int nmax = (int)reduce_biglist_entries(g);
  int n = min(nmax, min(kBigMost, max(max(kBigGrid, 2 * kBigMost / g.nC), nmax / kBigPer)));
  n -= n > 1 && n % 2 == 0;
  const dim3 grid(n, g.nC), block(64 * kBigSeg);
  const GatherArgs a = gather_args(feats, nsum, node_map, node_level, capacity, merged, counts, rb, zscan);
  STTM_DISPATCH_IO(k_reduce_big_combine, g.dtype, out_dtype, grid, block, s, g, a);
}

}  // namespace sttm
