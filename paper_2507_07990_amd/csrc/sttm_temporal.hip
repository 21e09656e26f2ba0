// Temporal stage (Sec. 3.3): similarities between every kept node of frame t and the kept nodes of
// frame t-1 it overlaps, directed edges with top-left priority, and the common root of every chain.
#include "sttm_dev.h"

namespace sttm {

// Sum of the valid cells of a block of at most 4x4 cells (h x w of them valid, h, w >= 1) with top-left cell
// (y0, x0), for this lane's channels: all row loads are issued before the first one is used.
template <int DT>
__device__ inline void block_sum16(const typename Row<DT>::Elem* fb, int D, int W, int y0, int x0, int h, int w,
                                   float (&S)[Row<DT>::VEC]) {
  typedef Row<DT> R;
  constexpr int VEC = R::VEC;
  typename R::Raw r[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int dy = i >> 2, dx = i & 3;
    r[i] = R::zero();
    if (dy < h && dx < w) r[i] = *reinterpret_cast<const typename R::Raw*>(fb + (size_t)((y0 + dy) * W + x0 + dx) * D);
  }
#pragma unroll
  for (int v = 0; v < VEC; ++v) S[v] = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    float t[VEC];
    R::unpack(r[i], t);
#pragma unroll
    for (int v = 0; v < VEC; ++v) S[v] += t[v];
  }
}

// ------------------------------------------------------------------------------------------------
// The feature pass of the temporal stage, in two kernels, or for small inputs in one (k_temporal_tiles).
// The two frames' partitions are both quadtree cuts, so any two overlapping nodes are nested; a pair is named by
// the top-left cell q of its finer node, and its "join" block is the coarser node.
//
// k_temporal_plan, one workgroup per frame t >= 1, looks at the node levels of frames t and t-1 only and cuts the
// pair's work into items of about equal size, by join level J:
//  * J <= 1 ("fast"): aligned 2x2 regions in which both frames' nodes are single cells or the 2x2 block; four
//    regions per item.
//  * J == 2 ("mid"): one 4x4 block per item.
//    With `skip_same` the regions (of single cells, 2x2 and 4x4 blocks) that are the same node
//    in both frames are left out: the spatial pass has already formed those dot products (k_temporal_resolve
//    reads them from its table).
//  * J >= 3 ("big"): the coarse sum is not recomputed: the spatial pass left the per-channel sums of all nodes
//    at levels >= 3 in `nsum`. Pairs whose finer node is a single cell go sixteen to an item (all under the same
//    join block), every other finer node is an item of its own.
// The items go into kTQueues queues, each of a run of consecutive frames (a workgroup reserves its stretch with one
// atomic on the queue's counter; with one counter for all, the five hundred atomics of a long video queued up
// behind one another). The order of the stretches varies from run to run, what is computed for an item does not.
//
// k_temporal_dots, a fixed grid of four-wavefront workgroups. The queues one after the other are one list in frame
// order; each of the eight dies takes an eighth of it, and wavefront w of the die's W the (item, chunk) tasks w, w + W,
// w + 2W, ... of that part (a trip count known on entry): every wavefront has the same number of tasks, however unevenly
// the work is spread over the frames (scene cuts concentrate it in a few of them), and the frame pairs that need the
// same rows meet in one die's L2. A wavefront reads its next item while it works on the present one, loads the rows the
// item names, and reduces its lanes' partial dot products through LDS ([scalar][lane] rows).
// Output: pd_part[f][chunk][q].
// ------------------------------------------------------------------------------------------------
struct TItem {
  int32_t f;     // frame t of the pair (the first two of the item's 24 16-bit words)
  int16_t type;  // 0 fast, 1 mid, 2 cells under a big block, 3 one finer node under a big block
  int16_t n;     // fast: regions (1..4); cells: cells (1..16)
  int16_t a;     // mid: top-left cell of the block; big: join block's node index counted from the first level-3 node
  int16_t b;     // mid, big: 1 when the join block is frame t's node (else frame t-1's)
  // fast: region's top-left cell | (frame t holds the 2x2 block) << 10 | (frame t-1 does) << 11
  // mid:  level (0..2) of the other frame's node at each of the block's 16 cells
  // cells: the cells; node: top-left cell of the finer node, its level
  int16_t e[18];
};
static_assert(sizeof(TItem) == 48, "three 16-byte pieces");

__host__ __device__ inline int temporal_items_per_pair(const Geo& g) { return g.P * g.P / 4 + g.P * g.P / 64 + 4; }
constexpr int kFastRows = 16;
constexpr int kBigNodes = 24;  // nodes at levels >= 3 of a 32x32 grid: 16 + 4 + 1
constexpr int kTItemWords = 24, kTItemE = 6;  // 16-bit words of an item; the first of the e[]
// Workgroups of the feature pass at most: what the chip holds at three wavefronts per SIMD, so that all start at once
// and share the list evenly. (The statistics call -- the planner, this pass and k_temporal_resolve -- with 512, 768 and 1536
// workgroups, us: 512 frames of 13x13 at D = 3584, half the tokens kept, 29.8, 27.7, 29.9, a third kept 38.0, 36.8, 36.4;
// 1024 frames of 27x27 at D = 1152 82.4, 72.6, 72.1. Three wavefronts per SIMD hold 168 registers, which the 16-bit instances
// use to the last one; none of them spills, at four per SIMD they do.)
constexpr int kTBlocks = 768;

__host__ __device__ inline int temporal_queue_items(const Geo& g) {
  return ((g.F + kTQueues - 1) / kTQueues) * temporal_items_per_pair(g);
}
__device__ inline int temporal_queue_of(const Geo& g, int f) { return f / ((g.F + kTQueues - 1) / kTQueues); }


__global__ __launch_bounds__(256) void k_temporal_plan(Geo g, const uint8_t* __restrict__ node_level, bool skip_same,
                                                       TItem* __restrict__ items, int* __restrict__ count,
                                                       SelState* __restrict__ sel) {
  __shared__ uint8_t lvl_t[1024], lvl_p[1024];
  __shared__ int16_t fast[256], mid[64], pairs0[1024], pairsX[256];
  __shared__ int nfast, nmid, nX, s_base;
  __shared__ int cnt0[kBigNodes], fill0[kBigNodes], off0[kBigNodes + 1], ioff0[kBigNodes + 1];
  __shared__ uint8_t coarse_t[kBigNodes];
  const int f = blockIdx.x, t = f % g.T, b = f / g.T;
  const int H = g.H, W = g.W, HW = g.HW, tid = threadIdx.x;
  if (t == 0) {  // no pair ends here; the temporal budget search of this video starts afresh
    sel_clear(sel + b, g.T * g.HW);
    return;
  }
  if (tid == 0) { nfast = nmid = nX = 0; }
  if (tid < kBigNodes) cnt0[tid] = fill0[tid] = 0;
  for (int c = tid; c < HW; c += blockDim.x) {
    lvl_t[c] = node_level[(size_t)f * HW + c];
    lvl_p[c] = node_level[(size_t)(f - 1) * HW + c];
  }
  __syncthreads();
  for (int c = tid; c < HW; c += blockDim.x) {
    const int a = lvl_t[c], bb = lvl_p[c];
    const int J = max(a, bb), lf = min(a, bb);
    const int y = c / W, x = c - y * W;
    const bool join_head = !(y & ((1 << J) - 1)) && !(x & ((1 << J) - 1));
    // (where both frames keep the same node at a level <= 2 there is nothing to do when the spatial pass left
    // those dot products)
    const bool same_done = skip_same && a == bb;
    if (J <= 1) {
      if (!(y & 1) && !(x & 1) && !same_done) fast[atomicAdd(&nfast, 1)] = (int16_t)c;
    } else if (J == 2) {
      if (join_head && !same_done) mid[atomicAdd(&nmid, 1)] = (int16_t)c;
    } else {
      const int nid = node_index(g, J, y >> J, x >> J) - g.lvl_base[3];
      if (join_head) coarse_t[nid] = a >= bb ? 1 : 0;
      if (!(y & ((1 << lf) - 1)) && !(x & ((1 << lf) - 1))) {  // top-left cell of the finer node
        if (lf == 0) atomicAdd(&cnt0[nid], 1);
        else pairsX[atomicAdd(&nX, 1)] = (int16_t)c;
      }
    }
  }
  __syncthreads();
  if (tid <= kBigNodes) {  // where each join block's cells start in pairs0, and where its items start among the cell items
    int o = 0, io = 0;
    for (int s = 0; s < tid; ++s) {
      o += cnt0[s];
      io += (cnt0[s] + 15) >> 4;
    }
    off0[tid] = o;
    ioff0[tid] = io;
    if (tid == kBigNodes) {
      const int total = ((nfast + 3) >> 2) + nmid + io + nX;
      s_base = total ? atomicAdd(count + temporal_queue_of(g, f) * kTCountStride, total) : 0;
    }
  }
  __syncthreads();
  for (int c = tid; c < HW; c += blockDim.x) {
    const int a = lvl_t[c], bb = lvl_p[c];
    if (max(a, bb) >= 3 && min(a, bb) == 0) {
      const int J = max(a, bb), y = c / W, x = c - y * W;
      const int nid = node_index(g, J, y >> J, x >> J) - g.lvl_base[3];
      pairs0[off0[nid] + atomicAdd(&fill0[nid], 1)] = (int16_t)c;
    }
  }
  __syncthreads();
  // The items are written piecemeal, one thread per header and one per entry (an item assembled in registers and
  // stored in one piece needs its entry array indexed at run time, which cost more than everything else here).
  const int nfi = (nfast + 3) >> 2, nmi = nmid, n0i = ioff0[kBigNodes], nxi = nX;
  const int ntot = nfi + nmi + n0i + nxi;
  TItem* out = items + (size_t)temporal_queue_of(g, f) * temporal_queue_items(g) + s_base;
  for (int idx = tid; idx < ntot * 19; idx += blockDim.x) {
    const int i = idx / 19, j = idx - i * 19 - 1;  // j = -1: the header
    int type, n = 0, a = 0, bflag = 0, ev = 0;
    if (i < nfi) {
      type = 0;
      n = min(4, nfast - 4 * i);
      if (j >= 0 && j < n) {
        const int c0 = fast[4 * i + j];
        ev = c0 | ((lvl_t[c0] == 1 ? 1 : 0) << 10) | ((lvl_p[c0] == 1 ? 1 : 0) << 11);
      }
    } else if (i < nfi + nmi) {
      const int c = mid[i - nfi];
      const bool coarse_is_t = lvl_t[c] >= lvl_p[c];
      type = 1;
      a = c;
      bflag = coarse_is_t ? 1 : 0;
      if (j >= 0 && j < 16) {
        const int y = c / W + (j >> 2), x = c % W + (j & 3);
        if (y < H && x < W) ev = min((int)(coarse_is_t ? lvl_p : lvl_t)[y * W + x], 2);
      }
    } else if (i < nfi + nmi + n0i) {
      const int k = i - nfi - nmi;
      int sl = 0;
      while (ioff0[sl + 1] <= k) ++sl;  // the join block this item belongs to (at most kBigNodes steps)
      const int first = off0[sl] + 16 * (k - ioff0[sl]);
      type = 2;
      n = min(16, off0[sl + 1] - first);
      a = sl;
      bflag = coarse_t[sl];
      if (j >= 0 && j < n) ev = pairs0[first + j];
    } else {
      const int q = pairsX[i - nfi - nmi - n0i];
      const int la = lvl_t[q], lb = lvl_p[q], J = max(la, lb), y = q / W, x = q - y * W;
      type = 3;
      a = node_index(g, J, y >> J, x >> J) - g.lvl_base[3];
      bflag = la >= lb ? 1 : 0;
      ev = j == 0 ? q : min(la, lb);
    }
    if (j < 0) {
      out[i].f = f;
      out[i].type = (int16_t)type;
      out[i].n = (int16_t)n;
      out[i].a = (int16_t)a;
      out[i].b = (int16_t)bflag;
    } else if (j < 18) {
      out[i].e[j] = (int16_t)ev;
    }
  }
}

// Sums the 16 rows [row][lane] of a wavefront's LDS staging area: lane r < 16 returns the sum of row r.
__device__ inline float rows16_sum(const float* tb, int lane) {
  float acc = 0.f;
  if (lane < 16) {
    const float4* row = reinterpret_cast<const float4*>(tb + lane * 68);
#pragma unroll
    for (int jj = 0; jj < 16; ++jj) {
      const float4 q = row[jj];
      acc += (q.x + q.y) + (q.z + q.w);
    }
  }
  return acc;
}

// One item for one chunk of the channels, by a wavefront: `words` holds the item's 16-bit words, one per lane; `tb` is a staging
// area of kFastRows rows of 68 floats in LDS.
template <int DT>
__device__ __forceinline__ void temporal_item(const Geo& g, const void* __restrict__ feats_v, const float* __restrict__ nsum,
                                              float* __restrict__ pd_part, int words, int chunk, float* tb, int lane) {
  typedef Row<DT> R;
  typedef typename R::Raw Raw;
  constexpr int VEC = R::VEC;
  const int H = g.H, W = g.W, HW = g.HW, NB = g.NN - g.lvl_base[3];
  auto e = [&](int j) { return lane_value(words, kTItemE + j); };
  const int f = (lane_value(words, 0) & 0xffff) | (lane_value(words, 1) << 16), type = lane_value(words, 2);
  const int it_n = lane_value(words, 3), it_a = lane_value(words, 4);
  const bool coarse_is_t = lane_value(words, 5) != 0;
  const int ch0 = chunk * g.cch + lane * VEC;
  const bool act = ch0 < g.D;
  const int chl = act ? ch0 : 0;  // (a lane beyond the last channel reads the first ones; its share is dropped below)
  const typename R::Elem* ft = reinterpret_cast<const typename R::Elem*>(feats_v) + (size_t)f * HW * g.D;
  const typename R::Elem* fp = ft - (size_t)HW * g.D;
  auto row = [&](const typename R::Elem* frame, int cell) {
    return *reinterpret_cast<const Raw*>(frame + (size_t)cell * g.D + chl);
  };
  float* out = pd_part + (size_t)(f * g.nC + chunk) * HW;
  if (type == 0) {
    // ---- up to four 2x2 regions, two at a time (16 rows in flight)
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
      if (half * 2 >= it_n) break;
      Raw rt[2][4], rp[2][4];
#pragma unroll
      for (int rr = 0; rr < 2; ++rr) {
        const int ri = half * 2 + rr;
        const int c0 = ri < it_n ? (e(ri) & 1023) : HW;  // (HW: no such row)
        const int y0 = c0 / W, x0 = c0 - y0 * W;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int y = y0 + (k >> 1), x = x0 + (k & 1);
          rt[rr][k] = R::zero();
          rp[rr][k] = R::zero();
          if (y < H && x < W) {
            rt[rr][k] = row(ft, y * W + x);
            rp[rr][k] = row(fp, y * W + x);
          }
        }
      }
#pragma unroll
      for (int rr = 0; rr < 2; ++rr) {
        const int ri = half * 2 + rr;
        const int ee = ri < it_n ? e(ri) : 0;
        const bool t_block = (ee >> 10) & 1, p_block = (ee >> 11) & 1;  // wave-uniform
        if (!t_block && !p_block) {  // four cells against four cells: no sums needed
#pragma unroll
          for (int k = 0; k < 4; ++k) tb[(ri * 4 + k) * 68 + lane] = act ? R::dot(rt[rr][k], rp[rr][k]) : 0.f;
          continue;
        }
        // a frame that holds the 2x2 block takes part with the sum of its four cells
        float st[VEC], sp[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) st[v] = sp[v] = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float xv[VEC];
          if (t_block) {
            R::unpack(rt[rr][k], xv);
#pragma unroll
            for (int v = 0; v < VEC; ++v) st[v] += xv[v];
          }
          if (p_block) {
            R::unpack(rp[rr][k], xv);
#pragma unroll
            for (int v = 0; v < VEC; ++v) sp[v] += xv[v];
          }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float xa[VEC], xb[VEC];
          if (t_block) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) xa[v] = st[v];
          } else {
            R::unpack(rt[rr][k], xa);
          }
          if (p_block) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) xb[v] = sp[v];
          } else {
            R::unpack(rp[rr][k], xb);
          }
          float d = 0.f;
#pragma unroll
          for (int v = 0; v < VEC; ++v) d = fmaf(xa[v], xb[v], d);
          tb[(ri * 4 + k) * 68 + lane] = act ? d : 0.f;
        }
      }
    }
    wave_lds_fence();
    const float acc = rows16_sum(tb, lane);
    int row_l = lane;  // (what is derived from it is worked out here: kept through the loop it does not fit the registers)
    STTM_OPAQUE_V(row_l);
    const int ri = (row_l >> 2) & 3, k = row_l & 3, ee = __shfl(words, kTItemE + ri, 64);
    if (row_l < kFastRows && ri < it_n) {
      const int c0 = ee & 1023, y = c0 / W + (k >> 1), x = c0 % W + (k & 1);
      const bool both_block = ((ee >> 10) & 3) == 3;
      if (y < H && x < W && (k == 0 || !both_block)) out[y * W + x] = acc;
    }
    wave_lds_fence();
  } else if (type == 1) {
    // ---- a 4x4 join block: its sum in the frame where it is one node, then every cell of the other frame dotted
    //      with it; the dot product of a finer node is the sum over its cells
    const int y0 = it_a / W, x0 = it_a - y0 * W;
    const typename R::Elem* coarse = coarse_is_t ? ft : fp;
    const typename R::Elem* fine = coarse_is_t ? fp : ft;
    float SA[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) SA[v] = 0.f;
    {
      Raw rc[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int y = y0 + (j >> 2), x = x0 + (j & 3);
        rc[j] = R::zero();
        if (y < H && x < W) rc[j] = row(coarse, y * W + x);
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        float tv[VEC];
        R::unpack(rc[j], tv);
#pragma unroll
        for (int v = 0; v < VEC; ++v) SA[v] += tv[v];
      }
    }
    // (the compiler asks for these sixteen rows before it adds up the first sixteen: all 32 are in flight, and fit)
    {
      Raw rf[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int y = y0 + (j >> 2), x = x0 + (j & 3);
        rf[j] = R::zero();
        if (y < H && x < W) rf[j] = row(fine, y * W + x);
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        float tv[VEC];
        R::unpack(rf[j], tv);
        float d = 0.f;
#pragma unroll
        for (int v = 0; v < VEC; ++v) d = fmaf(tv[v], SA[v], d);
        tb[j * 68 + lane] = act ? d : 0.f;
      }
    }
    wave_lds_fence();
    const float cd = rows16_sum(tb, lane);  // lane i < 16: cell (i / 4, i % 4) of the block against the coarse sum
    wave_lds_fence();
    const float s4 = (cd + __shfl_down(cd, 1, 64)) + (__shfl_down(cd, 4, 64) + __shfl_down(cd, 5, 64));  // 2x2 at lane
    float s16 = s4;  // lanes 0, 2, 8, 10 hold the four 2x2 sums
    s16 = (s16 + __shfl_down(s16, 2, 64)) + (__shfl_down(s16, 8, 64) + __shfl_down(s16, 10, 64));
    const int lf = __shfl_down(words, kTItemE, 64);  // level of the other frame's node at the lane's cell
    int cell_l = lane;  // (as above)
    STTM_OPAQUE_V(cell_l);
    if (cell_l < 16) {
      const int dy = cell_l >> 2, dx = cell_l & 3, y = y0 + dy, x = x0 + dx;
      if (y < H && x < W) {
        const int cb = y * W + x;
        if (lf == 0) out[cb] = cd;
        else if (lf == 1 && !(dy & 1) && !(dx & 1)) out[cb] = s4;
        else if (lf == 2 && lane == 0) out[cb] = s16;
      }
    }
  } else {
    // ---- under a join block at a level >= 3: its stored sum against single cells (sixteen at a time) or against
    //      one finer node
    const int fc = coarse_is_t ? f : f - 1;  // frame in which the join block is one node
    const typename R::Elem* fine = coarse_is_t ? fp : ft;
    const float* srow = nsum + ((size_t)fc * NB + it_a) * g.D + chl;
    float S[VEC];
#pragma unroll
    for (int v = 0; v < VEC; v += 4) {
      const float4 q = *reinterpret_cast<const float4*>(srow + v);
      S[v] = q.x; S[v + 1] = q.y; S[v + 2] = q.z; S[v + 3] = q.w;
    }
    if (type == 2) {
      Raw r[16];
#pragma unroll
      for (int jj = 0; jj < 16; ++jj) {
        r[jj] = R::zero();
        if (jj < it_n) r[jj] = row(fine, e(jj));
      }
#pragma unroll
      for (int jj = 0; jj < 16; ++jj) {
        float xv[VEC];
        R::unpack(r[jj], xv);
        float d = 0.f;
#pragma unroll
        for (int v = 0; v < VEC; ++v) d = fmaf(xv[v], S[v], d);
        tb[jj * 68 + lane] = act ? d : 0.f;
      }
      wave_lds_fence();
      const float acc = rows16_sum(tb, lane);
      const int cell = __shfl_down(words, kTItemE, 64);
      if (lane < it_n) out[cell] = acc;
      wave_lds_fence();
    } else {
      const int q = e(0), lf = e(1);
      const int y = q / W, x = q - y * W;
      float SB[VEC];
      if (lf >= 3) {
        const int ff = coarse_is_t ? f - 1 : f;
        const float* brow = nsum + ((size_t)ff * NB + node_index(g, lf, y >> lf, x >> lf) - g.lvl_base[3]) * g.D + chl;
#pragma unroll
        for (int v = 0; v < VEC; v += 4) {
          const float4 t = *reinterpret_cast<const float4*>(brow + v);
          SB[v] = t.x; SB[v + 1] = t.y; SB[v + 2] = t.z; SB[v + 3] = t.w;
        }
      } else {
        const int s = 1 << lf;
        block_sum16<DT>(fine + chl, g.D, W, y, x, min(s, H - y), min(s, W - x), SB);
      }
      float d = 0.f;
#pragma unroll
      for (int v = 0; v < VEC; ++v) d = fmaf(SB[v], S[v], d);
      if (!act) d = 0.f;
      d = wave_sum(d);
      if (lane == 0) out[q] = d;
    }
  }
}

template <int DT>
__global__ __launch_bounds__(256, 3) void k_temporal_dots(Geo g, const void* __restrict__ feats_v,
                                                       const float* __restrict__ nsum,
                                                       const TItem* __restrict__ items,
                                                       const int* __restrict__ count, float* __restrict__ pd_part) {
  __shared__ float tbuf[4][kFastRows * 68];
  // (the wavefront's number is the same in all its lanes: said explicitly, so that everything derived from it --
  // the task, the item and the row addresses -- is kept in scalar registers)
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  // where each queue's items lie in the list: lane q holds the number of items up to and including queue q's
  static_assert(kTQueues == kWave, "a lane per queue");
  const int mine = count[lane * kTCountStride];
  int upto = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(upto, o, 64);
    if (lane >= o) upto += t;
  }
  const int total = lane_value(upto, 63);
  // Workgroups go to the eight dies round-robin by their index.
  const int die = blockIdx.x & 7;
  const int first = (int)((long long)total * die / 8), nitems = (int)((long long)total * (die + 1) / 8) - first;
  const int ntasks = nitems * g.nC, stride = (int)(gridDim.x >> 3) * 4;
  const int qitems = temporal_queue_items(g);
  // the 16-bit words of the item of task t, one per lane
  auto fetch = [&](int t) {
    const int i = first + t / g.nC;
    const int q = __popcll(__ballot(upto <= i));  // the queue that holds it
    const int at = i - (lane_value(upto, q) - lane_value(mine, q));
    const int16_t* w = reinterpret_cast<const int16_t*>(items + (size_t)q * qitems + at);
    return (int)w[min(lane, kTItemWords - 1)];
  };
  int task = (int)(blockIdx.x >> 3) * 4 + wave;
  if (task >= ntasks) return;  // (the wavefronts of a workgroup share nothing)
  int next_words = fetch(task);
#pragma unroll 1
  for (; task < ntasks; task += stride) {
    const int words = next_words, chunk = task % g.nC;
    if (task + stride < ntasks) next_words = fetch(task + stride);
    temporal_item<DT>(g, feats_v, nsum, pd_part, words, chunk, tbuf[wave], lane);
  }
}

// ------------------------------------------------------------------------------------------------
// k_temporal_tiles: the same for small inputs, without a plan: a wavefront takes a 4x4 tile of a frame pair for one chunk of
// the channels, finds out from the two frames' levels there what it has to do, and does it item by item, the same arithmetic
// on the same rows (`share` wavefronts take turns at the items of one). What a plan costs is a launch, two trips to memory for
// making its items and one for reading them; what it gives is an even share of the work for every wavefront, which matters
// once there are many more tiles than wavefronts. Both are bound by the latency of the rows a single item waits for.
// ------------------------------------------------------------------------------------------------
template <int DT>
__global__ __launch_bounds__(256, 3) void k_temporal_tiles(Geo g, const void* __restrict__ feats_v,
                                                        const float* __restrict__ nsum,
                                                        const uint8_t* __restrict__ node_level, bool skip_same,
                                                        float* __restrict__ pd_part, SelState* __restrict__ sel, int share) {
  __shared__ float tbuf[4][kFastRows * 68];
  __shared__ int item[4][kTItemWords];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int H = g.H, W = g.W, TX = (W + 3) >> 2, tiles = TX * ((H + 3) >> 2);
  sel_clear_all(sel, g.B, g.T * g.HW);  // the temporal budget searches start afresh
  // Workgroups go to the eight dies round-robin by their index; each die has an eighth of the frames, so that both pairs
  // that need a frame's rows mostly meet in its L2.
  const long long tasks = (long long)g.F * tiles * g.nC;
  const int die = blockIdx.x & 7, first = (int)(tasks * die / 8), last = (int)(tasks * (die + 1) / 8);
  const int slot = (int)(blockIdx.x >> 3) * 4 + wave, task = first + slot / share, turn = slot % share;
  if (task >= last) return;  // (the wavefronts of a workgroup share nothing from here on)
  const int chunk = task % g.nC, tile = task / g.nC % tiles, f = task / g.nC / tiles;
  if (f % g.T == 0) return;
  const int y0 = tile / TX * 4, x0 = (tile - tile / TX * TX) * 4, head = y0 * W + x0;
  // lane i < 16: cell (i / 4, i % 4) of the tile, if there is one
  const int dy = lane >> 2 & 3, dx = lane & 3, cell = head + dy * W + dx;
  const bool in = lane < 16 && y0 + dy < H && x0 + dx < W;
  const size_t at = (size_t)f * g.HW + (in ? cell : head);
  const int a = node_level[at], b = node_level[at - g.HW];
  // a node above level 1 covers the tile: the first cell speaks for it
  const int a0 = lane_value(a, 0), b0 = lane_value(b, 0), J = max(a0, b0), lf = min(a0, b0);
  const bool coarse_is_t = a0 >= b0, corner = !(dy & 1) && !(dx & 1);
  // What there is to do: one item of the lanes in `heads`, then an item for each lane in `blocks` (2x2 blocks under a node
  // of level 3 or more).
  int type, aa = 0;
  unsigned heads, blocks = 0;
  if (J <= 1) {
    type = 0;
    heads = (unsigned)__ballot(in && corner && !(skip_same && a == b));
  } else if (J == 2) {
    type = 1;
    heads = skip_same && a0 == b0 ? 0u : 0xffffu;
    aa = head;
  } else {
    aa = node_index(g, J, y0 >> J, x0 >> J) - g.lvl_base[3];
    type = lf >= 2 ? 3 : 2;
    heads = lf >= 2 ? ((y0 | x0) & ((1 << lf) - 1) ? 0u : 1u) : (unsigned)__ballot(in && min(a, b) == 0);
    if (lf < 2) blocks = (unsigned)__ballot(in && corner && min(a, b) == 1);
  }
  int* w = item[wave];
#pragma unroll 1
  for (int left = (heads != 0) + (int)__popcll((unsigned long long)blocks); left > 0; --left) {
    const bool whole = heads != 0;
    if (!whole) type = 3;
    const unsigned mine = whole ? heads : blocks & (0u - blocks);
    if (whole) heads = 0;
    else blocks &= blocks - 1u;
    if (left % share != turn) continue;
    if (mine >> (lane & 31) & (unsigned)(lane < 16)) {
      const int to = kTItemE + (int)__popcll((unsigned long long)(mine & ((1u << (lane & 15)) - 1u)));
      w[to] = type == 0 ? cell | (a == 1 ? 1 << 10 : 0) | (b == 1 ? 1 << 11 : 0) : type == 1 ? (in ? min(coarse_is_t ? b : a, 2) : 0) : cell;
      if (type == 3) w[to + 1] = min(a, b);
    }
    if (lane < kTItemE)
      w[lane] = lane == 0 ? f & 0xffff : lane == 1 ? f >> 16 : lane == 2 ? type : lane == 3 ? (int)__popcll((unsigned long long)mine) : lane == 4 ? aa : (int)coarse_is_t;
    wave_lds_fence();
    const int words = w[min(lane, kTItemWords - 1)];
    temporal_item<DT>(g, feats_v, nsum, pd_part, words, chunk, tbuf[wave], lane);
    wave_lds_fence();
  }
}

// Up to this many (frame, tile, chunk) triples take the kernel without a plan. A pass with the plan and without, us: 7168
// triples (64 frames of 13x13 at D = 3584) 108.5 and 105.4, 5760 (96 of 11x19, fp32, D = 1000) 160.3 and 154.9, 9000 (150 of
// 15x20 at D = 1280) 157.8 and 156.9, 20,160 (180 of 14x14 at D = 3584) 220.6 and 223.7, 57,344 401 and 420.
// (The host-thread build of the tests that takes the large inputs' kernels takes the plan.)
#ifndef STTM_TEMPORAL_TILES_MAX
#define STTM_TEMPORAL_TILES_MAX 12288
#endif
constexpr long long kTilesMax = STTM_TEMPORAL_TILES_MAX;
// Of few triples the items of one are shared out among four or two wavefronts (8 frames of 8x8: 49.4 and 45.9 us a pass; 37 of
// 16x5 108.1 and 106.4; four wavefronts for 7168 triples: 106.4 and 109.8).
constexpr long long kTilesFour = 1024, kTilesTwo = 3072;
static long long temporal_tasks(const Geo& g) { return (long long)g.F * ((g.H + 3) / 4) * ((g.W + 3) / 4) * g.nC; }

size_t temporal_items_bytes(const Geo& g) { return (size_t)kTQueues * temporal_queue_items(g) * sizeof(TItem); }
size_t temporal_count_bytes() { return (size_t)kTQueues * kTCountStride * sizeof(int); }

void launch_temporal_dots(const Geo& g, const void* feats, const uint8_t* node_level, const float* nsum,
                          bool skip_same, float* pd_part, SelState* sel, void* items, int* item_count,
                          hipStream_t s) {
  if (g.T == 1) return;  // no pairs
  if (const long long tasks = temporal_tasks(g); tasks <= kTilesMax) {
    const int share = tasks <= kTilesFour ? 4 : tasks <= kTilesTwo ? 2 : 1;
    const dim3 grid(8u * (unsigned)(((tasks / 8 + 1) * share + 3) / 4)), block(256);  // a die has at most tasks / 8 + 1 of them
    if (g.dtype == 1)
      hipLaunchKernelGGL(k_temporal_tiles<1>, grid, block, 0, s, g, feats, nsum, node_level, skip_same, pd_part, sel, share);
    else if (g.dtype == 2)
      hipLaunchKernelGGL(k_temporal_tiles<2>, grid, block, 0, s, g, feats, nsum, node_level, skip_same, pd_part, sel, share);
    else
      hipLaunchKernelGGL(k_temporal_tiles<0>, grid, block, 0, s, g, feats, nsum, node_level, skip_same, pd_part, sel, share);
    return;
  }
  TItem* q = reinterpret_cast<TItem*>(items);
  hipLaunchKernelGGL(k_temporal_plan, dim3(g.F), dim3(256), 0, s, g, node_level, skip_same, q, item_count, sel);
  // enough wavefronts for about four tasks each if every pair came with all the items it can have; whole rounds of dies
  const long long worst = (long long)g.F * temporal_items_per_pair(g) * g.nC;
  long long blocks = (worst + 15) / 16;
  blocks = blocks < kTBlocks ? (blocks + 7) / 8 * 8 : kTBlocks;
  const dim3 grid((unsigned)blocks), block(256);
  if (g.dtype == 1)
    hipLaunchKernelGGL(k_temporal_dots<1>, grid, block, 0, s, g, feats, nsum, q, item_count, pd_part);
  else if (g.dtype == 2)
    hipLaunchKernelGGL(k_temporal_dots<2>, grid, block, 0, s, g, feats, nsum, q, item_count, pd_part);
  else
    hipLaunchKernelGGL(k_temporal_dots<0>, grid, block, 0, s, g, feats, nsum, q, item_count, pd_part);
}

__device__ inline int node_idx_of(const Geo& g, int lvl, int y0, int x0) {
  return node_index(g, lvl, y0 >> lvl, x0 >> lvl);
}

// Per-frame view of the two partitions in LDS.
struct PairFrame {
  uint8_t lvl_t[1024], lvl_p[1024];
  int16_t rep_t[1024], rep_p[1024];
};

__device__ inline void load_pair_frame(const Geo& g, int f, const int32_t* node_map, const uint8_t* node_level,
                                       PairFrame& pf) {
  const int HW = g.HW;
  for (int c = threadIdx.x; c < HW; c += blockDim.x) {
    pf.lvl_t[c] = node_level[(size_t)f * HW + c];
    pf.lvl_p[c] = node_level[(size_t)(f - 1) * HW + c];
    pf.rep_t[c] = (int16_t)(node_map[(size_t)f * HW + c] - f * HW);
    pf.rep_p[c] = (int16_t)(node_map[(size_t)(f - 1) * HW + c] - (f - 1) * HW);
  }
}

// ------------------------------------------------------------------------------------------------
// k_temporal_resolve: one workgroup per frame. Every overlapping (source n in frame t, destination d in
// frame t-1) pair lives at the top-left cell of the finer of the two nodes: the thread of that cell sums
// the per-chunk partial dots in chunk order, divides by the norms from the spatial stage and stores the
// similarity; e_n = max over n's destinations is collected with an integer max in LDS (order-free).
// Also writes the order-preserving integer image of e_n for the budget search (0 = not a candidate).
// match = 1 (only the destination under n's top-left cell counts): that pair always lives at n's own top-left
// cell -- n is the finer node, or the destination there is and shares the corner -- so e_n is that one entry.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_temporal_resolve(Geo g, int match,
                                                          const int32_t* __restrict__ node_map,
                                                          const uint8_t* __restrict__ node_level,
                                                          const float* __restrict__ pd_part,
                                                          const float* __restrict__ cell_part,
                                                          const float* __restrict__ nrm2,
                                                          float* __restrict__ sig, float* __restrict__ e,
                                                          uint32_t* __restrict__ sel_key,
                                                          SelState* __restrict__ sel, int* __restrict__ item_count) {
  __shared__ PairFrame pf;
  __shared__ unsigned ekey[1024];
  __shared__ unsigned h0[kSelBins];
  const int f = blockIdx.x, HW = g.HW, W = g.W;
  if (f == 0) temporal_clear(item_count, threadIdx.x);  // the feature pass is over: its queues are empty for the next one
  if (f % g.T == 0) {
    if (g.T == 1) sel_clear(sel + f, HW);  // (the feature pass over frame pairs, which does so, is left out)
    for (int c = threadIdx.x; c < HW; c += blockDim.x) sel_key[(size_t)f * HW + c] = 0;
    return;
  }
  load_pair_frame(g, f, node_map, node_level, pf);
  for (int c = threadIdx.x; c < HW; c += blockDim.x) ekey[c] = 0;
  for (int j = threadIdx.x; j < kSelBins; j += blockDim.x) h0[j] = 0;
  __syncthreads();
  for (int c = threadIdx.x; c < HW; c += blockDim.x) {
    const int a = pf.lvl_t[c], b = pf.lvl_p[c];
    const int n = pf.rep_t[c], d = pf.rep_p[c];
    if ((a <= b ? n : d) != c) continue;  // not the top-left cell of the finer node
    // the two norms and the per-chunk partial dot products, eight chunks in flight, added in chunk order
    const float nn = nrm2[(size_t)f * g.NN + node_idx_of(g, a, n / W, n % W)];
    const float nd = nrm2[(size_t)(f - 1) * g.NN + node_idx_of(g, b, d / W, d % W)];
    float dot = 0.f;
    const float* pp = pd_part + (size_t)f * g.nC * HW + c;
    size_t cstride = HW;  // from one chunk's partial to the next
    if (cell_part && a == b && a <= 2) {
      // the same node (a cell, a 2x2 or a 4x4 block) in both frames: the spatial pass of frame t-1 left the dot
      // product of its sum with the same node's sum in frame t
      const int y = c / W, x = c - y * W, NU = unit_cols(g) * unit_rows(g);
      cstride = (size_t)NU * kUnitScalars;
      pp = cell_part + ((size_t)(f - 1) * g.nC * NU + (y >> 3) * unit_cols(g) + (x >> 3)) * kUnitScalars +
           (a == 0 ? unit_cell_dot_slot(y, x) : unit_node_dot_slot(a, y, x));
    }
    for (int k0 = 0; k0 < g.nC; k0 += 8) {
      float pv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) pv[u] = k0 + u < g.nC ? pp[(size_t)(k0 + u) * cstride] : 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u) dot += pv[u];
    }
    const float v = cosine_from(dot, nn, nd);
    sig[(size_t)f * HW + c] = v;
    if (v == v && (match != 1 || c == n)) atomicMax(&ekey[n], float_key(v));
  }
  __syncthreads();
  for (int c0 = 0; c0 < HW; c0 += blockDim.x) {  // uniform trip count: the histogram update is wave-wide
    const int c = c0 + threadIdx.x;
    unsigned key = 0;
    if (c < HW) {
      const size_t i = (size_t)f * HW + c;
      if (pf.rep_t[c] == c) {
        const unsigned k = ekey[c];                 // 0 only if every similarity was NaN
        e[i] = k ? key_float(k) : -2.f;
        key = k ? k : float_key(-2.f);
      }
      sel_key[i] = key;
    }
    wave_hist_add(h0, key != 0, sel_bin(key), 1u);
  }
  __syncthreads();
  sel_flush_bins(sel + f / g.T, h0);
}

void launch_temporal_resolve(const Geo& g, int match, const int32_t* node_map,
                             const uint8_t* node_level,
                             const float* pd_part, const float* cell_part, const float* nrm2, float* sig, float* e,
                             uint32_t* sel_key, SelState* sel, int* item_count, hipStream_t s) {
  hipLaunchKernelGGL(k_temporal_resolve, dim3(g.F), dim3(256), 0, s, g, match, node_map, node_level, pd_part,
                     cell_part,
                     nrm2, sig, e, sel_key, sel, item_count);
}

// ------------------------------------------------------------------------------------------------
// k_temporal_parent: directed edge of every kept node (Sec. 3.3), one workgroup per run of frames of a video. Among the
// destinations whose similarity exceeds tau_T: the one towards the top-left (smallest raster index; integer min in LDS) --
// or, by `match`, only the one under the node's top-left cell, or the most similar one (64-bit integer max in LDS over
// (similarity image, reversed raster index), so ties go towards the top-left). A chain is followed through the run's frames
// in LDS right away, so that the jumps over memory below go from run to run: `ptr` of a node is its root, or the node of
// the frame before the run that its chain leaves the run by.
// (With one frame to a workgroup everywhere, and a launch more for the first 23 hops of every chain, these kernels took, us:
// 64 frames of 13x13 15.3, now 12.8, 32 videos of 32 frames of 27x27 22.0 and 16.7, 96 frames of 11x19 12.6 and 9.7, six
// clips of 25 frames 13.2 and 9.2.)
// ------------------------------------------------------------------------------------------------
constexpr int kParThreads = 1024;  // of a workgroup with more than one frame
constexpr int kParCells = 2048;  // cells of a run of more than one frame at most
constexpr int kHops = 23;        // edges that one launch below follows
// Frames of a run: as many as it takes for the runs of a video to be crossed by one launch, if these are no more cells than
// one workgroup takes at a time and no longer than kRunFrames; else, while they are few cells all the same, a hundred or so
// runs (a chain is followed frame by frame through a run, and few workgroups follow them) and a launch more. Edges and
// roots, us, with as many as needed and by this rule: 1000 frames of 6x6 22.3 and 18.0, 2000 of 4x4 22.6 and 17.0, 512 of 8x8
// 17.9 and 17.1; a pass over 8000 still frames of 2x2 171 and 134. Up to kRunFrames: 300 frames of 3x3 in runs of 14 14.1, of
// 4 15.6; 200 of 9x9 in runs of 9 15.5, of 3 18.7, of one 20.6.
constexpr int kRunFrames = 14, kRuns = 128, kRunLeast = 8;
static int parent_run(const Geo& g) {
  const int needed = (g.T + kHops - 1) / kHops;
  if (needed * g.HW > kParCells) return 1;
  return needed <= kRunFrames ? needed : max(kRunLeast, (g.T + kRuns - 1) / kRuns);
}
static size_t parent_lds(const Geo& g, int run, int match) {
  const size_t cells = (size_t)run * g.HW;
  return cells * (match == 2 ? 8 : 4) + (cells + g.HW) * 3 + 16;
}

template <int THREADS, int KIND>
__global__ __launch_bounds__(THREADS) void k_temporal_parent(Geo g, int match, int run, int runs,
                                                                 const int32_t* __restrict__ node_map,
                                                                 const uint8_t* __restrict__ node_level,
                                                                 const float* __restrict__ sig,
                                                                 float* __restrict__ tau, TauArgs given,
                                                                 SelSearch pending,
                                                                 int32_t* __restrict__ parent, int32_t* __restrict__ ptr) {
  // dynamic: per cell of the run the chosen destination (its place in the frame before; 64 bits wide with its similarity
  // when the most similar one is wanted), then of the frame before the run and of the run's own frames the top-left cell
  // and the level of every cell's node
  STTM_DYNAMIC_LDS(unsigned long long, sm);
  const int HW = g.HW, tid = threadIdx.x, b = blockIdx.x / runs, t0 = (blockIdx.x - b * runs) * run;
  const int frames = min(run, g.T - t0), cells = frames * HW, f0 = b * g.T + t0, i0 = f0 * HW;
  int* par = reinterpret_cast<int*>(sm);
  unsigned long long* best = sm;
  int16_t* rep = reinterpret_cast<int16_t*>(reinterpret_cast<char*>(sm) + (size_t)run * HW * (match == 2 ? 8 : 4));
  uint8_t* lvl = reinterpret_cast<uint8_t*>(rep + (run + 1) * HW);
  // What the frames hold does not depend on the threshold. The similarities are on their way while that is being found; the
  // tables are in LDS before it begins. (Kept in registers until after the search they cost more code and gave nothing: 512
  // frames of 13x13 13.1 us and 13.3 with them, 32 videos of 27x27 6.9 and 6.7, 64 frames of 13x13 9.6 and 9.7.)
  constexpr int kPer = THREADS >= kParThreads ? kParCells / THREADS : (THREADS > kSelThreads ? 1024 : kSelThreads) / THREADS;
  float val[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) val[u] = sig[i0 + min(tid + u * THREADS, cells - 1)];
  for (int q = tid; q < cells + HW; q += THREADS) {  // (cell q of these tables is cell q - HW of the run)
    if (t0 == 0 && q < HW) continue;
    const int i = i0 - HW + q, f = i / HW;
    rep[q] = (int16_t)(node_map[i] - f * HW);
    lvl[q] = node_level[i];
  }
  float th;
  if (KIND != kTauKnown || given.n) {  // the budget search was left to this kernel, or the caller named the threshold
    if constexpr (KIND == kTauKnown) th = given.v[b];
    else th = sel_threshold<THREADS, KIND>(g, pending, b);
    if (t0 == 0 && tid == 0) tau[b] = th;
  } else {
    th = tau[b];
  }
  for (int q = tid; q < cells; q += THREADS) {
    if (match == 2) best[q] = 0ull;
    else par[q] = 0x7fffffff;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int q = tid + u * THREADS, r = q / HW, c = q - r * HW;
    if (q >= cells || t0 + r == 0) continue;
    const int a = lvl[q + HW], bb = lvl[q], n = rep[q + HW], d = rep[q];
    if ((a <= bb ? n : d) != c) continue;  // not the top-left cell of the finer node
    const float v = val[u];
    if (!(v > th)) continue;
    if (match == 2)
      atomicMax(&best[r * HW + n], ((unsigned long long)float_key(v) << 32) | (unsigned)(0x7fffffff - d));
    else if (match == 0 || c == n)
      atomicMin(&par[r * HW + n], d);
  }
  __syncthreads();
  // the edge a cell's place holds: destination in the frame before, or -1
  auto edge = [&](int q) {
    if (match == 2) return best[q] ? 0x7fffffff - (int)(best[q] & 0xffffffffull) : -1;
    return par[q] != 0x7fffffff ? par[q] : -1;
  };
  for (int q = tid; q < cells; q += THREADS) {
    const int r = q / HW, c = q - r * HW;
    int p = -1, end = q;
    if (rep[q + HW] == c) {
      const int d = edge(q);
      if (d >= 0) p = i0 + (r - 1) * HW + d;
      // along the chain until it ends or leaves the run (then `end` is a cell of the frame before the run: negative)
      for (int h = r, e = d; e >= 0; --h) {
        end = (h - 1) * HW + e;
        if (h == 0) break;
        e = edge(end);
      }
    }
    parent[i0 + q] = p;
    ptr[i0 + q] = i0 + end;
  }
}

void launch_temporal_parent(const Geo& g, int match, const int32_t* node_map, const uint8_t* node_level,
                            const float* sig, float* tau, const TauArgs& given, const SelSearch& pending, int32_t* parent,
                            int32_t* ptr, hipStream_t s) {
  const int run = parent_run(g), runs = (g.T + run - 1) / run;
  const dim3 grid(g.B * runs);
  const size_t lds = parent_lds(g, run, match);
  // (64 frames of 32x32: edges and roots 20.9 us by 256 threads a frame, 18.7 by 512)
  const int threads = run > 1 ? kParThreads : g.HW > kSelThreads ? 2 * kSelThreads : kSelThreads;
  with_tau_kind(pending, [&](auto kind) {
    constexpr int KIND = decltype(kind)::value;
    const auto kernel = run > 1              ? k_temporal_parent<kParThreads, KIND>
                        : g.HW > kSelThreads ? k_temporal_parent<2 * kSelThreads, KIND>
                                             : k_temporal_parent<kSelThreads, KIND>;
    hipLaunchKernelGGL(kernel, grid, dim3(threads), lds, s, g, match, run, runs, node_map, node_level, sig, tau, given,
                       pending, parent, ptr);
  });
}

// ------------------------------------------------------------------------------------------------
// Common root of every chain by pointer jumping (root finding of Sec. 3.3): every pointer is a root or leads to the run of
// frames before; each launch multiplies the reach by kHops.
// ------------------------------------------------------------------------------------------------
// One launch follows up to kHops edges of the previous array, i.e. multiplies the reach by kHops; a walk stops at a
// root (an entry that points to itself), so short chains cost a load or two.
__global__ __launch_bounds__(256) void k_root_jump(int n, const int32_t* __restrict__ src,
                                                   int32_t* __restrict__ dst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int p = i;
  for (int h = 0; h < kHops; ++h) {
    const int q = src[p];
    if (q == p) break;
    p = q;
  }
  dst[i] = p;
}

// Last round, taken from every cell's node: cluster id = root of the node covering the cell.
__global__ __launch_bounds__(256) void k_root_jump_cells(int n, int hops, const int32_t* __restrict__ src,
                                                         const int32_t* __restrict__ node_map,
                                                         int32_t* __restrict__ cluster_ids) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int p = node_map[i];
  for (int h = 0; h < hops; ++h) {
    const int q = src[p];
    if (q == p) break;
    p = q;
  }
  cluster_ids[i] = p;
}

void launch_roots(const Geo& g, int32_t* ptr_a, int32_t* ptr_b, const int32_t* node_map, int32_t* cluster_ids,
                  hipStream_t s) {
  const int run = parent_run(g), runs = (g.T + run - 1) / run;
  // a chain crosses every run but the first, where one more step may lead to the root
  const long long steps = g.T == 1 ? 0 : runs;
  int rounds = steps > 0;
  for (long long reach = kHops; reach < steps; reach *= kHops) ++rounds;
  dim3 grid((g.N + 255) / 256), block(256);
  int32_t* src = ptr_a;
  int32_t* dst = ptr_b;
  for (int r = 0; r + 1 < rounds; ++r) {
    hipLaunchKernelGGL(k_root_jump, grid, block, 0, s, g.N, src, dst);
    int32_t* tmp = src; src = dst; dst = tmp;
  }
  hipLaunchKernelGGL(k_root_jump_cells, grid, block, 0, s, g.N, rounds > 0 ? kHops : 0, src, node_map,
                     cluster_ids);
}

}  // namespace sttm
