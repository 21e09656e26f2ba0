// Spatial stage (Sec. 3.2): pyramid sums, squared norms, parent-child cosine similarities, the
// coarse-to-fine decision, and the budget-driven threshold for it.
#include "sttm_dev.h"

namespace sttm {

constexpr int kTileRows = 36;    // 16 n0 + 16 d0 + 4 d1
// Rows of the staging area per tile, in batches of eight: four batches of the 2x2 blocks' statistics, one of the
// blocks' dot products with the tile (4) and with the next frame (4), two of the cell-to-cell dot products, one for
// the tile with the next frame.
constexpr int kStageRows = 64;
constexpr int kStageStride = 8;  // floats per staging row: one per group of eight lanes

// Issues the row loads of the tile whose top-left cell is (ty, tx); th x tw of its 4x4 cells are valid
// (th, tw >= 1). Every one of the 16 loads is issued, without a condition: a cell beyond the edge, or a lane
// beyond the last channel, reads a valid cell of the tile again (a cache hit) and tile_mask() discards it. The
// number of loads in flight is then known at compile time, and the wavefront can wait for this tile's rows
// while the partner tile's are still on their way.
template <int DT>
__device__ __forceinline__ void tile_load(typename Row<DT>::Raw (&raw)[16], const typename Row<DT>::Elem* fbase,
                                          int W, int D, int ty, int tx, int th, int tw) {
  typedef Row<DT> R;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int q1 = i >> 2, k = i & 3;
    const int dy = min((q1 >> 1) * 2 + (k >> 1), th - 1), dx = min((q1 & 1) * 2 + (k & 1), tw - 1);
    raw[i] = *reinterpret_cast<const typename R::Raw*>(fbase + (size_t)((ty + dy) * W + tx + dx) * D);
  }
}

// The same for one 2x2 block (q1) of the tile.
template <int DT>
__device__ __forceinline__ void block_load(typename Row<DT>::Raw (&raw)[4], const typename Row<DT>::Elem* fbase,
                                           int W, int D, int ty, int tx, int th, int tw, int q1) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int dy = min((q1 >> 1) * 2 + (k >> 1), th - 1), dx = min((q1 & 1) * 2 + (k & 1), tw - 1);
    raw[k] = *reinterpret_cast<const typename Row<DT>::Raw*>(fbase + (size_t)((ty + dy) * W + tx + dx) * D);
  }
}

// Zeroes what tile_load fetched for cells beyond the edge and for lanes beyond the last channel.
template <int DT>
__device__ __forceinline__ void tile_mask(typename Row<DT>::Raw (&raw)[16], int th, int tw, bool act) {
  typedef Row<DT> R;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int q1 = i >> 2, k = i & 3;
    const int dy = (q1 >> 1) * 2 + (k >> 1), dx = (q1 & 1) * 2 + (k & 1);
    if (!(dy < th && dx < tw && act)) raw[i] = R::zero();
  }
}

// Eight scalars of the wavefront at once (v[i] = this lane's share of scalar i): returns, in lane l, the sum of
// scalar (l & 7) over the eight lanes of l's group (l >> 3). Three exchanges, each halving the scalars a lane
// carries: with the neighbour (lane ^ 1), across the quad (^ 2), across the two quads (^ 4).
__device__ __forceinline__ float group_sums8(const float (&v)[8], int lane) {
  const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
  float a[4], c[2];
#ifndef STTM_HOST_EMULATION
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float keep = b0 ? v[2 * i + 1] : v[2 * i], give = b0 ? v[2 * i] : v[2 * i + 1];
    a[i] = keep + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(give), 0xB1, 0xF, 0xF, true));  // quad_perm [1,0,3,2]
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float keep = b1 ? a[2 * i + 1] : a[2 * i], give = b1 ? a[2 * i] : a[2 * i + 1];
    c[i] = keep + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(give), 0x4E, 0xF, 0xF, true));  // quad_perm [2,3,0,1]
  }
  const float keep = b2 ? c[1] : c[0], give = b2 ? c[0] : c[1];
  int r = __builtin_amdgcn_update_dpp(0, __float_as_int(give), 0x104, 0xF, 0x5, true);  // lanes 0-3, 8-11 of a row: from lane + 4
  r = __builtin_amdgcn_update_dpp(r, __float_as_int(give), 0x114, 0xF, 0xA, true);      // lanes 4-7, 12-15: from lane - 4
  return keep + __int_as_float(r);
#else
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float keep = b0 ? v[2 * i + 1] : v[2 * i], give = b0 ? v[2 * i] : v[2 * i + 1];
    a[i] = keep + __shfl_xor(give, 1, 64);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float keep = b1 ? a[2 * i + 1] : a[2 * i], give = b1 ? a[2 * i] : a[2 * i + 1];
    c[i] = keep + __shfl_xor(give, 2, 64);
  }
  const float keep = b2 ? c[1] : c[0], give = b2 ? c[0] : c[1];
  return keep + __shfl_xor(give, 4, 64);
#endif
}

// Eight scalars go into the staging area as rows 8 * batch .. 8 * batch + 7, each row the eight partial sums of one
// scalar over the groups of eight lanes: one store per lane, all to different words. (Every lane calls it.)
__device__ __forceinline__ void stage8(float* tbs, int batch, int lane, const float (&v)[8]) {
  tbs[(batch * 8 + (lane & 7)) * kStageStride + (lane >> 3)] = group_sums8(v, lane);
}

// Adds row `row` of the staging area up (a fixed order).
__device__ __forceinline__ float staged_row_sum(const float* tbs, int row) {
  const float4* p = reinterpret_cast<const float4*>(tbs + row * kStageStride);
  const float4 a = p[0], b = p[1];
  return ((a.x + a.y) + (a.z + a.w)) + ((b.x + b.y) + (b.z + b.w));
}

// Sum and per-lane scalars of one 2x2 block: its per-channel sum in S1, and nd = squared norms of its four cells, then
// each cell . the block's sum. A cell's dot product with the sum is the sum of its dot products with the block's four
// cells, which come straight from the packed rows (no element is widened for them). Rows of cells beyond the edge and
// lanes beyond the last channel must be zero (tile_mask).
template <int DT>
__device__ __forceinline__ void block_stats(uint2 ident, const typename Row<DT>::Raw* raw, float (&S1)[Row<DT>::VEC],
                                            float (&nd)[8]) {
  typedef Row<DT> R;
  R::sum4(ident, raw, S1);
#pragma unroll
  for (int k = 0; k < 4; ++k) nd[k] = R::dot(raw[k], raw[k]);  // (zero rows give zero)
  const float p01 = R::dot(raw[0], raw[1]), p02 = R::dot(raw[0], raw[2]), p03 = R::dot(raw[0], raw[3]);
  const float p12 = R::dot(raw[1], raw[2]), p13 = R::dot(raw[1], raw[3]), p23 = R::dot(raw[2], raw[3]);
  nd[4] = (nd[0] + p01) + (p02 + p03);
  nd[5] = (nd[1] + p01) + (p12 + p13);
  nd[6] = (nd[2] + p02) + (p12 + p23);
  nd[7] = (nd[3] + p03) + (p13 + p23);
}

// The sums over a unit of N channels from `ch` on (N and ch even), by the packed dot product and in the order of the
// pyramid kernels: for a sum that came out as no finite number. There one broken value takes three more channels with it,
// here at most the other one of its pair, as where the rows themselves are added up for the output.
template <int DT, int N>
__device__ inline void unit_pair_sums(const Geo& g, const void* frame, int y3, int x3, int ch, float (&sum)[N]) {
  uint32_t klo, khi;
  if (DT == 1) opaque_pairs<0x3f80u, 0x3f800000u>(klo, khi);
  else opaque_pairs<0x3c00u, 0x3c000000u>(klo, khi);
#pragma unroll
  for (int n = 0; n < N; n += 2) {
    const uint16_t* rows = static_cast<const uint16_t*>(frame) + ch + n;
    float s3[2];
#pragma unroll 1
    for (int q2 = 0; q2 < 4; ++q2) {
      float s2[2] = {0.f, 0.f};
#pragma unroll 1
      for (int q1 = 0; q1 < 4; ++q1) {
        float s1[2] = {0.f, 0.f};
#pragma unroll 1
        for (int k = 0; k < 4; ++k) {
          const int y = y3 + (q2 >> 1) * 4 + (q1 >> 1) * 2 + (k >> 1), x = x3 + (q2 & 1) * 4 + (q1 & 1) * 2 + (k & 1);
          if (y >= g.H || x >= g.W) continue;
          const uint32_t w = *reinterpret_cast<const uint32_t*>(rows + (size_t)(y * g.W + x) * g.D);
          s1[0] = DT == 1 ? dot2_bf16(w, klo, s1[0]) : dot2_f16(w, klo, s1[0]);
          s1[1] = DT == 1 ? dot2_bf16(w, khi, s1[1]) : dot2_f16(w, khi, s1[1]);
        }
        s2[0] += s1[0];
        s2[1] += s1[1];
      }
      s3[0] = q2 ? s3[0] + s2[0] : s2[0];
      s3[1] = q2 ? s3[1] + s2[1] : s2[1];
    }
    sum[n] = s3[0];
    sum[n + 1] = s3[1];
  }
}
__device__ inline bool finite(float v) { return (__float_as_uint(v) & 0x7f800000u) != 0x7f800000u; }

// Which (frame, unit, chunk) a workgroup of a 1-D grid works on; false = none. With the frame-to-frame dot products a
// tile is asked for by two workgroups: its own frame's and the one of the frame before. Workgroups go to the eight dies
// round-robin by their index; each die gets a contiguous range of frames and walks it in order, two frames at a time
// with the same (unit, chunk) of both next to each other, so that the two requests come from the same die within a few
// microseconds of each other and the second one is served by that die's L2. (The statistics call, frame after frame and in
// pairs: 25 frames of 18x24 tokens at D = 8192, 144 workgroups a frame, 81.3 and 69.6 us; 64 of 13x13 at D = 3584 30.6 and
// 29.7; 140 of those and 64 of 16x16 at D = 1152 the same; 150 of 15x20 at D = 1280 41.6 and 42.1.)
constexpr int kPyrGroup = 2;
__device__ __forceinline__ bool pyramid_place(const Geo& g, int NU, int& f, int& u, int& chunk) {
  const int per_die = (g.F + 7) / 8, die = blockIdx.x & 7;
  int slot = blockIdx.x >> 3;
  const int fi = slot % kPyrGroup;
  slot /= kPyrGroup;
  chunk = slot % g.nC;
  slot /= g.nC;
  u = slot % NU;
  const int fl = (slot / NU) * kPyrGroup + fi;
  f = die * per_die + fl;
  return fl < per_die && f < g.F;
}
static unsigned pyramid_grid(const Geo& g) {
  const unsigned pairs = ((g.F + 7) / 8 + kPyrGroup - 1) / kPyrGroup;  // per die
  return 8u * pairs * kPyrGroup * (unsigned)(unit_cols(g) * unit_rows(g) * g.nC);
}

// ------------------------------------------------------------------------------------------------
// k_pyramid_tiles: the same pass with a workgroup for every frame, the same results bit for bit: for small inputs, and
// where no frame-to-frame products are wanted. The four tiles of a unit are four wavefronts: each reads its tile and, four
// rows at a time, the partner tile (the same tile of the next frame), the first eight partner rows requested with the
// tile's own; the tiles' sums meet in LDS for the unit's sum. Three wavefronts per SIMD.
// (8 frames of 8x8 tokens, D = 64, fp32: 7.9 us; one image of 24x24, D = 1152: 5.9; 64 frames of 16x16, D = 1152: 15.6,
// of 13x13, D = 3584: 23.6 and 28.2 by k_pyramid_stats.)
// ------------------------------------------------------------------------------------------------
template <int DT, bool CC>  // CC: with the frame-to-frame dot products of cells, 2x2 blocks and tiles
__global__ __launch_bounds__(256, 3) void k_pyramid_tiles(Geo g, const void* __restrict__ feats_v,
                                                          float* __restrict__ part, float* __restrict__ nsum,
                                                          SelState* __restrict__ sel) {
  typedef Row<DT> R;
  typedef typename R::Raw Raw;
  constexpr int VEC = R::VEC;
  __shared__ __attribute__((aligned(16))) float stage[4][kStageRows * kStageStride];
  __shared__ __attribute__((aligned(16))) float st[kUnitScalars];
  __shared__ float4 tsum[4][VEC / 4][64];  // the four tiles' sums
  const int UX = unit_cols(g), NU = UX * unit_rows(g), lane = threadIdx.x & 63;
  int f, u, chunk;
  if (CC) {
    if (!pyramid_place(g, NU, f, u, chunk)) return;  // (the whole workgroup)
  } else {
    chunk = blockIdx.x;
    u = blockIdx.y;
    f = blockIdx.z;
  }
  // (which wavefront -- and so which SIMD -- gets which tile rotates: in a ragged unit the first tile is the fullest)
  const int q2 = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6) + u + f + chunk) & 3;
  float* tbs = stage[q2];
  const int ch0 = chunk * g.cch + lane * VEC;
  const bool act = ch0 < g.D;
  const int H = g.H, W = g.W, L = g.L;
  const int y3 = (u / UX) * 8, x3 = (u % UX) * 8;
  const int ty = y3 + (q2 >> 1) * 4, tx = x3 + (q2 & 1) * 4;
  const int th = max(0, min(4, H - ty)), tw = max(0, min(4, W - tx));  // valid rows / columns of the tile
  const bool has_next = CC && f % g.T != g.T - 1;
  if (chunk == 0 && u == 0 && f % g.T == 0) sel_clear(sel + f / g.T, g.T * (g.NN - g.lvl_base[1]));  // this video's budget search starts afresh
  float S2[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) S2[v] = 0.f;
  if (th > 0 && tw > 0) {
    const typename R::Elem* fbase =
        reinterpret_cast<const typename R::Elem*>(feats_v) + (size_t)f * g.HW * g.D + (act ? ch0 : 0);
    const typename R::Elem* nbase = fbase + (size_t)g.HW * g.D;
    Raw raw[16];
    tile_load<DT>(raw, fbase, W, g.D, ty, tx, th, tw);
    Raw pr[2][4];  // rows of the partner tile, two 2x2 blocks at a time
    if (CC && has_next) {
      block_load<DT>(pr[0], nbase, W, g.D, ty, tx, th, tw, 0);
      block_load<DT>(pr[1], nbase, W, g.D, ty, tx, th, tw, 1);
    }
    // a full tile of a full chunk needs no masking
    const bool ragged = th < 4 || tw < 4 || (chunk + 1) * g.cch > g.D;
    if (ragged) tile_mask<DT>(raw, th, tw, act);
    const uint2 ident = R::ident();
    float S1[4][VEC];  // the tile's 2x2 block sums
    float b4[8];  // the blocks' dot products with the tile, then with the same blocks of the next frame
    float SN2[VEC], cd[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) b4[i] = 0.f;
#pragma unroll
    for (int v = 0; v < VEC; ++v) SN2[v] = 0.f;
    // Block by block, so that a block's rows are done with before the next one's sums need their registers.
#pragma unroll
    for (int q1 = 0; q1 < 4; ++q1) {
      const bool live = (q1 >> 1) * 2 < th && (q1 & 1) * 2 < tw;  // (wave-uniform)
#pragma unroll
      for (int v = 0; v < VEC; ++v) S1[q1][v] = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) cd[(q1 & 1) * 4 + k] = 0.f;
      if (live) {
        float nd[8];
        block_stats<DT>(ident, raw + q1 * 4, S1[q1], nd);
        stage8(tbs, q1, lane, nd);
#pragma unroll
        for (int v = 0; v < VEC; ++v) S2[v] += S1[q1][v];
        if (CC && has_next) {
          // x_c(t) . x_c(t+1) for the block's cells: where both frames keep single cells the temporal stage needs
          // nothing else (Sec. 3.3 compares node features; a cell's feature is its own row).
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            if (ragged) {  // (a clamped request repeated another cell; a lane beyond the last channel read channel 0)
              const bool in = (q1 >> 1) * 2 + (k >> 1) < th && (q1 & 1) * 2 + (k & 1) < tw && act;
              if (!in) pr[q1 & 1][k] = R::zero();
            }
            cd[(q1 & 1) * 4 + k] = R::dot(raw[q1 * 4 + k], pr[q1 & 1][k]);
          }
          // The same for the tile's 2x2 blocks and for the tile itself: S_n(t) . S_n(t+1), what the temporal
          // stage needs where both frames keep the same node n at level 1 or 2: the block's sum with the sum of the
          // partner block's four rows, the tile's sum with the sum of the partner blocks.
          float SN1[VEC], d1 = 0.f;
          R::sum4(ident, pr[q1 & 1], SN1);
#pragma unroll
          for (int v = 0; v < VEC; ++v) {
            d1 = fmaf(S1[q1][v], SN1[v], d1);
            SN2[v] += SN1[v];
          }
          b4[4 + q1] = d1;
        }
      }
      if (CC && has_next) {
        if (q1 < 2) block_load<DT>(pr[q1], nbase, W, g.D, ty, tx, th, tw, 2 + q1);
        if (q1 & 1) stage8(tbs, 5 + (q1 >> 1), lane, cd);
      }
    }
#pragma unroll
    for (int q1 = 0; q1 < 4; ++q1) {
#pragma unroll
      for (int v = 0; v < VEC; ++v) b4[q1] = fmaf(S1[q1][v], S2[v], b4[q1]);
    }
    if (CC && has_next) {
      float t8[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) t8[i] = 0.f;
#pragma unroll
      for (int v = 0; v < VEC; ++v) t8[0] = fmaf(S2[v], SN2[v], t8[0]);
      stage8(tbs, 7, lane, t8);
    }
#pragma unroll
    for (int v = 0; v < VEC; v += 4) tsum[q2][v / 4][lane] = make_float4(S2[v], S2[v + 1], S2[v + 2], S2[v + 3]);
    stage8(tbs, 4, lane, b4);
    // row r of the staging area is added up by lane r and goes to its place in the unit's block (zero where the
    // row stands for nothing: beyond the edge, above the root level, no next frame)
    wave_lds_fence();
    if (lane < 57) {
      const int r = lane;
      bool live;
      int dst;
      if (r < 32 || (r >= 40 && r < 56)) {  // a cell's row: norm, dot with its block, or with the next frame
        const int q1 = r < 32 ? r >> 3 : (r - 40) >> 2, k = r & 3;
        live = (q1 >> 1) * 2 + (k >> 1) < th && (q1 & 1) * 2 + (k & 1) < tw;
        if (r < 32 && (r & 4)) live = live && 0 < L;
        if (r >= 40) live = live && has_next;
        dst = r < 32 ? q2 * kTileRows + ((r & 4) ? 16 : 0) + q1 * 4 + k : kUnitCellDots + q2 * 16 + (r - 40);
      } else if (r < 40) {  // a 2x2 block's row: dot with the tile, or with the next frame
        const int q1 = r & 3;
        live = (q1 >> 1) * 2 < th && (q1 & 1) * 2 < tw;
        live = live && (r < 36 ? 1 < L : has_next);
        dst = r < 36 ? q2 * kTileRows + 32 + q1 : kUnitNodeDots + q2 * 8 + q1;
      } else {  // the tile with the next frame's
        live = has_next;
        dst = kUnitNodeDots + q2 * 8 + 4;
      }
      st[dst] = live ? staged_row_sum(tbs, r) : 0.f;
    }
  } else {
#pragma unroll
    for (int v = 0; v < VEC; v += 4) tsum[q2][v / 4][lane] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (lane < kTileRows) st[q2 * kTileRows + lane] = 0.f;
    if (lane < 16) st[kUnitCellDots + q2 * 16 + lane] = 0.f;
    if (lane < 5) st[kUnitNodeDots + q2 * 8 + lane] = 0.f;
  }
  if (lane >= 5 && lane < 8) st[kUnitNodeDots + q2 * 8 + lane] = 0.f;
  if (q2 == 0 && lane < kUnitCellDots - 4 * kTileRows - 4) st[4 * kTileRows + 4 + lane] = 0.f;
  __syncthreads();
  // level-2 dot products of the four tiles with the unit's sum
  float d2 = 0.f;
  if (L >= 3) {
    float S3[VEC];
#pragma unroll
    for (int v = 0; v < VEC; v += 4) {
      float4 s = tsum[0][v / 4][lane];
#pragma unroll
      for (int q = 1; q < 4; ++q) {
        const float4 t = tsum[q][v / 4][lane];
        s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
      }
      S3[v] = s.x; S3[v + 1] = s.y; S3[v + 2] = s.z; S3[v + 3] = s.w;
      if (q2 == v / 4 && act) {  // a wavefront per four channels of the lanes stores the unit's sum
        if constexpr (DT != 0) {
          if (!(finite(s.x) && finite(s.y) && finite(s.z) && finite(s.w))) {
            float again[4];
            unit_pair_sums<DT>(g, reinterpret_cast<const typename R::Elem*>(feats_v) + (size_t)f * g.HW * g.D, y3, x3, ch0 + v, again);
            s = make_float4(again[0], again[1], again[2], again[3]);
          }
        }
        *reinterpret_cast<float4*>(nsum + ((size_t)f * (g.NN - g.lvl_base[3]) + (y3 >> 3) * (g.P >> 3) + (x3 >> 3)) * g.D + ch0 + v) = s;
      }
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) d2 = fmaf(S2[v], S3[v], d2);
    const float one[8] = {d2, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    stage8(tbs, 0, lane, one);
    wave_lds_fence();
    if (lane == 0) d2 = staged_row_sum(tbs, 0);
  }
  if (lane == 0) st[4 * kTileRows + q2] = d2;
  // the workgroup's scalars leave in one piece: whole, aligned 128-byte lines that no other workgroup touches
  __syncthreads();
  if (threadIdx.x < kUnitScalars / 4)
    reinterpret_cast<float4*>(part + ((size_t)(f * g.nC + chunk) * NU + u) * kUnitScalars)[threadIdx.x] =
        reinterpret_cast<const float4*>(st)[threadIdx.x];
}

// ------------------------------------------------------------------------------------------------
// k_pyramid_stats: the one pass over the features of the spatial stage, for videos that fill the chip.
//
// A workgroup owns a "unit" = an 8x8 cell block (level 3) for one chunk of the token rows, and walks through a run of
// frames; its four wavefronts own the unit's four 4x4 tiles (level 2). A lane owns VEC consecutive channels, so all
// pyramid sums are private to the lane and only scalars are reduced across lanes: three exchanges between lanes leave
// eight partial sums per scalar, which go through a small LDS area ([scalar][8]) to the lane that adds them up.
// Scalars: the squared norm of every cell, and for every node below the root the dot product of its sum
// with its parent's sum. (The squared norm of a parent is the sum of its children's dot products with it,
// which the finalize kernel adds up.) With CC also x_c(t) . x_c(t+1) of the cells and the same of the 2x2 blocks and the
// tiles: what the temporal stage needs where both frames keep the same node.
// A row is read once: the next frame's rows, wanted for those products, are the next step's own. Six places of four rows
// (one 2x2 block each) hold the frame's blocks and, two blocks ahead of the arithmetic, the next frame's; a block that is
// done with gives its place to the one six further on, so that the places' roles come round every three frames, which are
// written out one after the other. A cell beyond the edge, or a lane beyond the last channel, is beyond the window its
// load is checked against and reads as zero without a request to memory; no load or store of the walk is under a
// condition, so what is in flight is a compile-time fact and only the block that is needed is waited for. The tiles' sums
// meet in LDS, two frames' worth of places: one barrier a frame.
// Output: part[f][chunk][unit][kUnitScalars] = the workgroup's scalars, partial over this chunk's channels: per tile 16
//         squared norms, 16 cell and 4 level-1 dot products (child sum . parent sum), then the 4 level-2 dot products,
//         then per tile the 16 cell-to-cell dot products and the 4 + 1 of its blocks and itself (zeros without CC); the
//         levels from 3 up are the finalize kernel's when the pyramid is taller than a unit;
//         nsum[f][node - first level-3 node][D] = the per-channel sums of the level-3 nodes (fp32), which
//         the later stages read instead of re-adding up to 64 token rows.
// What bounds it: memory. 512 frames of 13x13 at D = 3584 in bf16, 653 MB read and 44 MB written in 145 us: 138 without
// the arithmetic, 124 without the stores, 111 without either. 180 frames of 18x24 at D = 8192: 1.31 GB and 79 MB in 290 us
// (4.8 TB/s). (A wavefront that took a unit's tiles one after the other and asked for the next frame's rows as well, from
// the cache its neighbour had just filled: 172 and 328 us.) The loads are marked non-temporal: the 512 frames in 158 us
// without. Eight places and two wavefronts per SIMD: 147. Two or three rounds of workgroups with shorter runs read more rows
// of them twice: 154 and 161 us.
// ------------------------------------------------------------------------------------------------
constexpr int kWalkSlots = 6, kWalkPeriod = 3;  // places of a block's rows; frames after which their roles are the same again
// Workgroups of one round: three wavefronts per SIMD. While a run stays this many frames long (3 % of the rows read twice)
// there are more rounds, up to three, which even out what ragged units need. The statistics call (this kernel and the next)
// with at most one, two and three rounds, us: 2000 frames of 13x13 at D = 3584 598, 595, 570; 600 of 18x24 at D = 8192 1052,
// 1001, 977; 2048 of 27x27 at D = 1152 938, 925, 919; 1024 of those (long enough for two) 465, 463, 462.
// (The host-thread build of the tests asks for few, so that it has runs of more than one frame.)
#ifndef STTM_WALK_GROUPS
#ifdef STTM_HOST_EMULATION
#define STTM_WALK_GROUPS 2
#else
#define STTM_WALK_GROUPS 768
#endif
#endif
constexpr int kWalkGroups = STTM_WALK_GROUPS, kWalkRounds = 3, kWalkLongRun = 32;
static int walk_segments(const Geo& g) {
  const long long columns = (long long)unit_cols(g) * unit_rows(g) * g.nC;
  long long s = max(kWalkGroups / columns, min(kWalkRounds * kWalkGroups / columns, (long long)(g.F / kWalkLongRun)));
  return (int)max(1ll, min(s, (long long)g.F));
}

// One scalar of the wavefront: row `row` of the staging area gets its eight partial sums, added up as group_sums8 does.
__device__ __forceinline__ void stage1(float* tbs, int row, int lane, float v) {
#ifndef STTM_HOST_EMULATION
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));  // quad_perm [1,0,3,2]
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true));  // quad_perm [2,3,0,1]
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, true)); // row_half_mirror
#else
  v += __shfl_xor(v, 1, 64);
  v += __shfl_xor(v, 2, 64);
  v += __shfl_xor(v, 4, 64);
#endif
  if ((lane & 7) == 0) tbs[row * kStageStride + (lane >> 3)] = v;
}

template <int DT, bool CC>  // CC: with the frame-to-frame dot products of cells, 2x2 blocks and tiles
__global__ __launch_bounds__(256, 3) void k_pyramid_stats(Geo g, const void* __restrict__ feats_v,
                                                          float* __restrict__ part, float* __restrict__ nsum,
                                                          SelState* __restrict__ sel, int segs) {
  typedef Row<DT> R;
  typedef typename R::Raw Raw;
  constexpr int VEC = R::VEC;
  __shared__ __attribute__((aligned(16))) float stage[4][kStageRows * kStageStride];
  __shared__ __attribute__((aligned(16))) float st[3][kUnitScalars];
  __shared__ __attribute__((aligned(16))) float4 tsum[2][4][VEC / 4][64];  // the four tiles' sums
  __shared__ float4 early[CC ? 4 : 1][2][VEC / 4][64];  // sums of a tile's first two blocks, when registers are short
  const int H = g.H, W = g.W, L = g.L;
  const int UX = unit_cols(g), NU = UX * unit_rows(g), tid = threadIdx.x, lane = tid & 63;
  int rest = blockIdx.x;
  const int chunk = rest % g.nC;
  rest /= g.nC;
  const int u = rest % NU, seg = rest / NU;
  const int f0 = (int)((long long)g.F * seg / segs), f1 = (int)((long long)g.F * (seg + 1) / segs);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // (which wavefront -- and so which SIMD -- gets which tile rotates: in a ragged unit the first tile is the fullest)
  const int q2 = __builtin_amdgcn_readfirstlane(wave + u + seg + chunk) & 3;
  float* tbs = stage[q2];
  const int ch0 = chunk * g.cch + lane * VEC;
  const int y3 = (u / UX) * 8, x3 = (u % UX) * 8;
  const int ty = y3 + (q2 >> 1) * 4, tx = x3 + (q2 & 1) * 4;
  const int th = max(0, min(4, H - ty)), tw = max(0, min(4, W - tx));  // valid rows / columns of the tile
  if (chunk == 0 && u == 0)  // the budget searches of the videos that begin here start afresh
    for (int b = (f0 + g.T - 1) / g.T; b * g.T < f1; ++b) sel_clear(sel + b, g.T * (g.NN - g.lvl_base[1]));
  for (int i = tid; i < 3 * kUnitScalars; i += 256) (&st[0][0])[i] = 0.f;
  for (int i = tid; i < 2 * 4 * (VEC / 4) * 64; i += 256) (&tsum[0][0][0][0])[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  __syncthreads();

  const unsigned row_bytes = (unsigned)g.D * (unsigned)sizeof(typename R::Elem), frame_bytes = row_bytes * (unsigned)g.HW;
  const unsigned voff = ch0 < g.D ? (unsigned)ch0 * (unsigned)sizeof(typename R::Elem) : frame_bytes;
  // the channels of the unit's sum that this lane stores, and the first one's place in a tile's sum in LDS
  const int own = (wave * 64 + lane) * (VEC / 4), pick = VEC == 4 ? own : ((own >> 2) & 1) * 256 + (own >> 3) * 4 + (own & 3);
  const unsigned noff = (unsigned)(chunk * g.cch + own) * 4u;
  unsigned soff[16];  // rows of the tile, wave-uniform; beyond the edge: past the window
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int q1 = i >> 2, k = i & 3, dy = (q1 >> 1) * 2 + (k >> 1), dx = (q1 & 1) * 2 + (k & 1);
    soff[i] = dy < th && dx < tw ? (unsigned)((ty + dy) * W + tx + dx) * row_bytes : frame_bytes;
  }
  // the last frame whose rows are needed: one past the run, if it belongs to the same video
  const int flast = CC && f1 < g.F && f1 % g.T != 0 ? f1 : f1 - 1;
  // where the frame being worked on is: its scalars and its unit's sum; the next frame's rows, those of the one after it
  // (never beyond flast: the loads are issued whatever they are for); how many frames of the video come after it
  float* part_f = part + ((size_t)(f0 * g.nC + chunk) * NU + u) * kUnitScalars;
  const size_t part_step = (size_t)g.nC * NU * kUnitScalars, nsum_step = (size_t)(g.NN - g.lvl_base[3]) * g.D;
  float* nsum_f = nsum + (size_t)f0 * nsum_step + (size_t)((y3 >> 3) * (g.P >> 3) + (x3 >> 3)) * g.D;
  const char* rows0 = reinterpret_cast<const char*>(feats_v) + (size_t)f0 * frame_bytes;
  const char* rows1 = rows0 + (f0 + 1 <= flast ? frame_bytes : 0u);
  const char* rows2 = rows1 + (f0 + 2 <= flast ? frame_bytes : 0u);
  int after = g.T - 1 - f0 % g.T;
  auto load_block = [&](Raw (&dst)[4], const Window& w, int q1) {
#pragma unroll
    for (int k = 0; k < 4; ++k) dst[k] = window_load_once<Raw>(w, voff, soff[q1 * 4 + k]);
  };
  // what lane r < 57 adds up: row r of the staging area, and where it goes
  const int r = lane;
  bool live = false;
  int dst = kUnitNodeDots + q2 * 8 + 4;
  if (r < 32 || (r >= 40 && r < 56)) {  // a cell's row: norm, dot with its block, or with the next frame
    const int q1 = r < 32 ? r >> 3 : (r - 40) >> 2, k = r & 3;
    live = (q1 >> 1) * 2 + (k >> 1) < th && (q1 & 1) * 2 + (k & 1) < tw;
    if (r < 32 && (r & 4)) live = live && 0 < L;
    dst = r < 32 ? q2 * kTileRows + ((r & 4) ? 16 : 0) + q1 * 4 + k : kUnitCellDots + q2 * 16 + (r - 40);
  } else if (r < 40) {  // a 2x2 block's row: dot with the tile, or with the next frame
    const int q1 = r & 3;
    live = (q1 >> 1) * 2 < th && (q1 & 1) * 2 < tw;
    live = live && (r < 36 ? 1 < L : CC);
    dst = r < 36 ? q2 * kTileRows + 32 + q1 : kUnitNodeDots + q2 * 8 + q1;
  } else {  // the tile with the next frame's
    live = CC;
  }

  // The second half of a frame, by all four wavefronts: the unit's sum, the tiles' dot products with it.
  auto unit_half = [&](int f, int buf3, int buf2, const float (&S2)[VEC], bool some) {
    __syncthreads();
    // what the frame before left, its last entries made before this barrier
    {
      const Window w = make_window(f > f0 ? part_f - part_step : part_f, f > f0 ? kUnitScalars * 4u : 0u);
      const float v[1] = {st[buf3 == 0 ? 2 : buf3 - 1][tid]};
      window_store(w, (unsigned)(tid * 4), 0u, v);
    }
    if (L >= 3) {
      float S3[VEC];
#pragma unroll
      for (int v = 0; v < VEC; v += 4) {
        float4 s = tsum[buf2][0][v / 4][lane];
#pragma unroll
        for (int q = 1; q < 4; ++q) {
          const float4 t = tsum[buf2][q][v / 4][lane];
          s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
        }
        S3[v] = s.x; S3[v + 1] = s.y; S3[v + 2] = s.z; S3[v + 3] = s.w;
      }
      if (some) {
        float d2 = 0.f;
#pragma unroll
        for (int v = 0; v < VEC; ++v) d2 = fmaf(S2[v], S3[v], d2);
        stage1(tbs, 0, lane, d2);
        wave_lds_fence();
        if (lane == 0) st[buf3][4 * kTileRows + q2] = staged_row_sum(tbs, 0);
        wave_lds_fence();
      }
      // a quarter of the sum's channels each
      const Window w = make_window(nsum_f, (unsigned)g.D * (unsigned)sizeof(float));
      float v[VEC / 4];
      const float* t = reinterpret_cast<const float*>(&tsum[buf2][0][0][0]) + pick;
#pragma unroll
      for (int i = 0; i < VEC / 4; ++i)
        v[i] = ((t[i] + t[VEC * 64 + i]) + t[2 * VEC * 64 + i]) + t[3 * VEC * 64 + i];
      if constexpr (DT != 0) {  // (a lane beyond the last channel holds zeros)
        if (!(finite(v[0]) && finite(v[1])))
          unit_pair_sums<DT>(g, reinterpret_cast<const typename R::Elem*>(feats_v) + (size_t)f * g.HW * g.D, y3, x3,
                             chunk * g.cch + own, v);
      }
      window_store(w, noff, 0u, v);
    }
    part_f += part_step;
    nsum_f += nsum_step;
  };

  if (th > 0 && tw > 0) {
    const uint2 ident = R::ident();
    Raw s[kWalkSlots][4];  // rows of a 2x2 block each: the frame's own blocks, those of the next one as they arrive
    {
      const Window w0 = make_window(rows0, frame_bytes), w1 = make_window(rows1, frame_bytes);
#pragma unroll
      for (int n = 0; n < kWalkSlots; ++n) load_block(s[n], n < 4 ? w0 : w1, n & 3);
    }
    auto frame = [&](auto phase, int f, int buf3, int buf2) {
      constexpr int P = decltype(phase)::value;
      const bool has_next = CC && after > 0;
      const Window w1 = make_window(rows1, frame_bytes), w2 = make_window(rows2, frame_bytes);
      float S1[4][VEC], S2[VEC];  // the tile's 2x2 block sums, its sum
      float b4[8];  // the blocks' dot products with the tile, then with the same blocks of the next frame
      float SN2[VEC], cd[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) b4[i] = 0.f;
#pragma unroll
      for (int v = 0; v < VEC; ++v) S2[v] = SN2[v] = 0.f;
#pragma unroll
      for (int q1 = 0; q1 < 4; ++q1) {
        Raw(&own)[4] = s[(4 * P + q1) % kWalkSlots];
        Raw(&nxt)[4] = s[(4 * P + q1 + 4) % kWalkSlots];
        const bool in = (q1 >> 1) * 2 < th && (q1 & 1) * 2 < tw;  // (wave-uniform)
#pragma unroll
        for (int v = 0; v < VEC; ++v) S1[q1][v] = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) cd[(q1 & 1) * 4 + k] = 0.f;
        if (in) {
          float nd[8];
          block_stats<DT>(ident, own, S1[q1], nd);
          stage8(tbs, q1, lane, nd);
#pragma unroll
          for (int v = 0; v < VEC; ++v) S2[v] += S1[q1][v];
          if (CC && q1 < 2) {
#pragma unroll
            for (int v = 0; v < VEC; v += 4)
              early[q2][q1][v / 4][lane] = make_float4(S1[q1][v], S1[q1][v + 1], S1[q1][v + 2], S1[q1][v + 3]);
          }
          if (CC && has_next) {
#pragma unroll
            for (int k = 0; k < 4; ++k) cd[(q1 & 1) * 4 + k] = R::dot(own[k], nxt[k]);
            float SN1[VEC], d1 = 0.f;
            R::sum4(ident, nxt, SN1);
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
              d1 = fmaf(S1[q1][v], SN1[v], d1);
              SN2[v] += SN1[v];
            }
            b4[4 + q1] = d1;
          }
        }
        // the block's rows are done with: their place goes to the block kWalkSlots further on
        load_block(own, q1 + kWalkSlots - 4 < 4 ? w1 : w2, (q1 + kWalkSlots) & 3);
        if (CC && (q1 & 1) && has_next) stage8(tbs, 5 + (q1 >> 1), lane, cd);
      }
#pragma unroll
      for (int q1 = 0; q1 < 4; ++q1) {
        if (CC && q1 < 2) {
          if ((q1 & 1) * 2 >= tw) continue;  // (no such block, nothing was kept)
#pragma unroll
          for (int v = 0; v < VEC; v += 4) {
            const float4 k = early[q2][q1][v / 4][lane];
            b4[q1] = fmaf(k.w, S2[v + 3], fmaf(k.z, S2[v + 2], fmaf(k.y, S2[v + 1], fmaf(k.x, S2[v], b4[q1]))));
          }
        } else {
#pragma unroll
          for (int v = 0; v < VEC; ++v) b4[q1] = fmaf(S1[q1][v], S2[v], b4[q1]);
        }
      }
      if (CC && has_next) {
        float t = 0.f;
#pragma unroll
        for (int v = 0; v < VEC; ++v) t = fmaf(S2[v], SN2[v], t);
        stage1(tbs, 56, lane, t);
      }
#pragma unroll
      for (int v = 0; v < VEC; v += 4) tsum[buf2][q2][v / 4][lane] = make_float4(S2[v], S2[v + 1], S2[v + 2], S2[v + 3]);
      stage8(tbs, 4, lane, b4);
      wave_lds_fence();
      if (lane < 57) st[buf3][dst] = live && (lane < 36 || has_next) ? staged_row_sum(tbs, lane) : 0.f;
      wave_lds_fence();
      unit_half(f, buf3, buf2, S2, true);
      rows1 = rows2;
      rows2 += f + 3 <= flast ? frame_bytes : 0u;
      after = after ? after - 1 : g.T - 1;
    };
    static_assert(kWalkPeriod * 4 % kWalkSlots == 0, "the places' roles come round");
    int f = f0, buf3 = 0;
#pragma unroll 1
    while (true) {
      auto next = [&] { buf3 = buf3 == 2 ? 0 : buf3 + 1; return ++f == f1; };
      frame(std::integral_constant<int, 0>(), f, buf3, (f - f0) & 1);
      if (next()) break;
      frame(std::integral_constant<int, 1>(), f, buf3, (f - f0) & 1);
      if (next()) break;
      frame(std::integral_constant<int, 2>(), f, buf3, (f - f0) & 1);
      if (next()) break;
    }
  } else {
    float none[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) none[v] = 0.f;
#pragma unroll 1
    for (int f = f0; f < f1; ++f) unit_half(f, (f - f0) % 3, (f - f0) & 1, none, false);
  }
  __syncthreads();
  (part_f - part_step)[tid] = st[(f1 - 1 - f0) % 3][tid];
}

// Up to this many (unit, chunk, frame) triples the pass is given to k_pyramid_tiles, beyond it to k_pyramid_stats, whose
// runs get too short below: 2800 triples (100 frames of 13x13, D = 3584) 34 against 38 us, 3072 (256 of 16x16, D = 1152)
// 43 and 43, 4200 (150 of 13x13) 54 and 53, 5600 69 and 66, 9600 (800 of 16x16) 125 and 110.
// Without frame-to-frame products nothing is read twice, and k_pyramid_tiles needs 95 registers, for five wavefronts per
// SIMD: it takes all (128 images of 24x24, D = 1152: 40 against 54 us; 512 frames of 13x13, D = 3584: 127 and 146).
// (The host-thread build of the tests sets 0, for k_pyramid_stats on inputs that are small enough for it.)
#ifndef STTM_PYR_TILES_MAX
#define STTM_PYR_TILES_MAX 4096
#endif
constexpr long long kPyrTilesMax = STTM_PYR_TILES_MAX;

template <int DT, bool CC>
static void launch_pyramid_dt(const Geo& g, const void* feats, float* part, float* nsum, SelState* sel, hipStream_t s) {
  const int NU = unit_cols(g) * unit_rows(g);
  // Without the frame-to-frame products no two workgroups share rows: a plain grid, dealt to all dies in turn. (In ranges
  // of frames per die one image is one die's work: 32x32 tokens at D = 8192, fp32, 34.8 against 11.0 us.)
  const dim3 grid = CC ? dim3(pyramid_grid(g)) : dim3(g.nC, NU, g.F);
  if constexpr (CC || kPyrTilesMax == 0) {
    const long long frame_bytes = (long long)g.HW * g.D * (g.dtype == 0 ? 4 : 2);  // (a window's offsets are 32 bits wide)
    if ((long long)NU * g.F * g.nC > kPyrTilesMax && frame_bytes < 1ll << 31) {
      const int segs = walk_segments(g);
      hipLaunchKernelGGL((k_pyramid_stats<DT, CC>), dim3((unsigned)(segs * NU * g.nC)), dim3(256), 0, s, g, feats, part,
                         nsum, sel, segs);
      return;
    }
  }
  hipLaunchKernelGGL((k_pyramid_tiles<DT, CC>), grid, dim3(256), 0, s, g, feats, part, nsum, sel);
}

template <bool CC>
static void launch_pyramid_cc(const Geo& g, const void* feats, float* part, float* nsum, SelState* sel, hipStream_t s) {
  if (g.dtype == 1) launch_pyramid_dt<1, CC>(g, feats, part, nsum, sel, s);
  else if (g.dtype == 2) launch_pyramid_dt<2, CC>(g, feats, part, nsum, sel, s);
  else launch_pyramid_dt<0, CC>(g, feats, part, nsum, sel, s);
}

void launch_pyramid_stats(const Geo& g, const void* feats, bool pairs, float* part, float* nsum, SelState* sel,
                          hipStream_t s) {
  if (pairs) launch_pyramid_cc<true>(g, feats, part, nsum, sel, s);
  else launch_pyramid_cc<false>(g, feats, part, nsum, sel, s);
}

// ------------------------------------------------------------------------------------------------
// k_spatial_finalize: one workgroup per frame. First the levels above the 8x8 units (UP = 1: a 16x16 grid, one node of
// level 4; UP = 2: a 32x32 grid, four of level 4 and, if the root is one node, the one of level 5): a lane owns four
// channels, loads them from all level-3 sums of the frame at once, adds the levels up in registers, stores the sums
// next to the level-3 ones and keeps its share of the dot products child . parent, which are added up over the
// wavefront and the chunks at the end. (One wavefront per node and chunk, level by level, paid the memory latency once per node, chunk
// and level: 44 us of 180 frames of 18x24 tokens at D = 8192, 50 us of 1024 frames of 27x27 at D = 1152.)
// Then it sums the per-chunk partials of the lower levels in chunk order, 16 bytes per thread into LDS, turns
// them into sigma(parent, child) (Sec. 3.2: cosine between a level's nodes and their children),
// m_n = min over existing children, and the split score s_n = max of m along the path from the root.
// ------------------------------------------------------------------------------------------------
constexpr int kUnitStats = 4 * kTileRows + 4;  // the scalars of a unit's block that this kernel reads
static_assert(kUnitStats % 4 == 0, "whole 16-byte pieces");
constexpr int kUpRows = 24;                    // dot products with a parent at level 4 (16) or 5 (4), whole batches of 8
// Threads of the kernel. With a 32x32 grid (1365 nodes) and no more frames than CUs, twice as many.
constexpr int kFinThreads = 512, kFinThreadsWide = 1024, kFinWaves = kFinThreadsWide / kWave;
constexpr int kFinWideFrames = 256;

__device__ inline float dot4(const float4& a, const float4& b, float c) {
  return fmaf(a.x, b.x, fmaf(a.y, b.y, fmaf(a.z, b.z, fmaf(a.w, b.w, c))));
}
__device__ inline float4 add4(const float4& a, const float4& b) {
  return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

// Eight sums over the wavefront at once, each by the tree of wave_sum (lane distances 32, 16, 8, 4, 2, 1): lane 8 i
// returns the sum of scalar i. Three exchanges halve the scalars a lane carries.
__device__ __forceinline__ float wave_sums8(const float (&v)[8], int lane) {
  const bool b5 = lane & 32, b4 = lane & 16, b3 = lane & 8;
  float a[4], c[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = (b5 ? v[i + 4] : v[i]) + __shfl_xor(b5 ? v[i] : v[i + 4], 32, 64);
#pragma unroll
  for (int i = 0; i < 2; ++i) c[i] = (b4 ? a[i + 2] : a[i]) + __shfl_xor(b4 ? a[i] : a[i + 2], 16, 64);
  float r = (b3 ? c[1] : c[0]) + __shfl_xor(b3 ? c[0] : c[1], 8, 64);
#pragma unroll
  for (int o = 4; o > 0; o >>= 1) r += __shfl_xor(r, o, 64);
  return r;
}

// The upper levels of frame f by the whole workgroup; leaves the dot product of level-3 node
// (2 py + ky, 2 px + kx) with its parent p = (py, px) in up[4 p + 2 ky + kx], that of level-4 node p with its parent in
// up[16 + p] (call a barrier before reading them). A wavefront takes a chunk of the channels at a time; the chunks'
// sums are added in chunk order. `red` is kUpRows * kFinWaves floats of LDS.
template <int UP>
__device__ inline void upper_levels(const Geo& g, float* nsum, int f, float* red, float* up) {
  constexpr int S4 = UP == 1 ? 1 : 2, N4 = S4 * S4;
  constexpr int kBatches = UP == 1 ? 1 : kUpRows / 8;
  const int NB = g.NN - g.lvl_base[3], D4 = g.D >> 2, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nwaves = blockDim.x >> 6;
  float4* rows = reinterpret_cast<float4*>(nsum + (size_t)f * NB * g.D);
  const int base4 = 4 * N4;  // nodes of level 3 come first, then level 4, then level 5
  float all = 0.f;           // thread i < 8 kBatches: dot product i over the chunks so far
#pragma unroll 1
  for (int c0 = 0; c0 < g.nC; c0 += nwaves) {
    const int chunk = c0 + wave;
    float tot[8 * kBatches];
#pragma unroll
    for (int i = 0; i < 8 * kBatches; ++i) tot[i] = 0.f;
    const int last = min(D4, (chunk + 1) * (g.cch >> 2));
#pragma unroll 1
    for (int c = chunk * (g.cch >> 2) + lane; c < last; c += kWave) {
      float4 a[4 * N4], s4[N4];
#pragma unroll
      for (int i = 0; i < 4 * N4; ++i) {  // i = 4 p + k
        const int p = i >> 2, k = i & 3, y = 2 * (p / S4) + (k >> 1), x = 2 * (p % S4) + (k & 1);
        a[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (node_exists(g, 3, y, x)) a[i] = rows[(size_t)(y * 2 * S4 + x) * D4 + c];
      }
#pragma unroll
      for (int p = 0; p < N4; ++p) {
        s4[p] = add4(add4(a[4 * p], a[4 * p + 1]), add4(a[4 * p + 2], a[4 * p + 3]));
        if (node_exists(g, 4, p / S4, p % S4)) rows[(size_t)(base4 + p) * D4 + c] = s4[p];
#pragma unroll
        for (int k = 0; k < 4; ++k) tot[4 * p + k] = dot4(a[4 * p + k], s4[p], tot[4 * p + k]);
      }
      if (UP == 2 && g.L >= 5) {
        const float4 s5 = add4(add4(s4[0], s4[1 % N4]), add4(s4[2 % N4], s4[3 % N4]));
        rows[(size_t)(base4 + N4) * D4 + c] = s5;
#pragma unroll
        for (int p = 0; p < N4; ++p) tot[(16 + p) % (8 * kBatches)] = dot4(s4[p], s5, tot[(16 + p) % (8 * kBatches)]);
      }
    }
#pragma unroll
    for (int i = 0; i < kBatches; ++i) {
      const float v[8] = {tot[8 * i], tot[8 * i + 1], tot[8 * i + 2], tot[8 * i + 3],
                          tot[8 * i + 4], tot[8 * i + 5], tot[8 * i + 6], tot[8 * i + 7]};
      const float r = wave_sums8(v, lane);
      if ((lane & 7) == 0) red[(8 * i + (lane >> 3)) * kFinWaves + wave] = r;
    }
    __syncthreads();
    if ((int)threadIdx.x < 8 * kBatches) {
      for (int w = 0; w < nwaves; ++w) all += red[threadIdx.x * kFinWaves + w];  // (zero beyond the last chunk)
    }
    __syncthreads();
  }
  if ((int)threadIdx.x < 8 * kBatches) up[threadIdx.x] = all;
}

template <int UP>
__global__ __launch_bounds__(UP == 2 ? kFinThreadsWide : kFinThreads) void k_spatial_finalize(Geo g, const float* __restrict__ part,
                                                                  float* __restrict__ nsum, float* __restrict__ nrm2,
                                                                  float* __restrict__ sim, float* __restrict__ m,
                                                                  uint32_t* __restrict__ sel_key,
                                                                  uint8_t* __restrict__ sel_w,
                                                                  SelState* __restrict__ sel, int* __restrict__ item_count,
                                                                  DecideArgs decide) {
  STTM_DYNAMIC_LDS(float, sm);
  __shared__ unsigned h0[kSelBins];
  __shared__ __attribute__((aligned(16))) float red[UP ? kUpRows * kFinWaves : 1];
  __shared__ float up[kUpRows];
  // dynamic: the units' scalars, then per node squared norm, similarity to the parent, m, and (level, row, column)
  const int NU = unit_cols(g) * unit_rows(g), UC = unit_cols(g), tid = threadIdx.x, nthr = blockDim.x;
  float* s_part = sm;
  float* s_n = sm + NU * kUnitStats;
  float* s_sim = s_n + g.NN;
  float* s_m = s_sim + g.NN;
  int* s_pos = reinterpret_cast<int*>(s_m + g.NN);
  const int f = blockIdx.x;
  const size_t fo = (size_t)f * g.NN;
  if (f == 0) temporal_clear(item_count, tid);
  {
    constexpr int kPieces = kUnitStats / 4;
    const float4* p4 = reinterpret_cast<const float4*>(part) + (size_t)f * g.nC * NU * (kUnitScalars / 4);
    const size_t cstride = (size_t)NU * (kUnitScalars / 4);  // from one chunk's block to the next
#pragma unroll 1
    for (int j = tid; j < NU * kPieces; j += nthr) {
      const int u = j / kPieces;
      const float4* p = p4 + u * (kUnitScalars / 4) + (j - u * kPieces);
      float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 1
      for (int c0 = 0; c0 < g.nC; c0 += 8) {  // eight chunks' partials in flight, added in chunk order
        float4 v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = p[(size_t)min(c0 + i, g.nC - 1) * cstride];
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (c0 + i < g.nC) s = add4(s, v[i]);
      }
      reinterpret_cast<float4*>(s_part)[j] = s;
    }
  }
  if constexpr (UP > 0) upper_levels<UP>(g, nsum, f, red, up);
  for (int j = tid; j < kSelBins; j += nthr) h0[j] = 0;
  for (int idx = tid; idx < g.NN; idx += nthr) {
    int lvl, by, bx;
    node_decode(g, idx, lvl, by, bx);
    s_pos[idx] = node_exists(g, lvl, by, bx) ? (lvl << 16) | (by << 8) | bx : -1;
  }
  __syncthreads();
  // dot product of every node's sum with its parent's; the squared norm of a cell
  for (int idx = tid; idx < g.NN; idx += nthr) {
    const int pos = s_pos[idx], lvl = pos >> 16, by = (pos >> 8) & 255, bx = pos & 255;
    float n = 0.f, d = 0.f;
    if (pos >= 0) {
      if (lvl <= 2) {
        const int y = by << lvl, x = bx << lvl;
        const int q2 = ((y >> 2) & 1) * 2 + ((x >> 2) & 1), q1 = ((y >> 1) & 1) * 2 + ((x >> 1) & 1);
        const int slot = lvl == 2 ? 4 * kTileRows + q2
                                  : q2 * kTileRows + (lvl == 1 ? 32 + q1 : 16 + q1 * 4 + (y & 1) * 2 + (x & 1));
        const float* q = s_part + ((y >> 3) * UC + (x >> 3)) * kUnitStats + slot;
        if (lvl < g.L) d = q[0];
        if (lvl == 0) n = q[-16];
      } else if (UP && lvl < g.L) {
        d = lvl == 3 ? up[((by >> 1) * UP + (bx >> 1)) * 4 + (by & 1) * 2 + (bx & 1)] : up[16 + by * 2 + bx];
      }
    }
    s_n[idx] = n;
    s_sim[idx] = d;
  }
  __syncthreads();
  // squared norm of a node above the cells = sum over its children of (child sum) . (node sum)
  for (int idx = tid; idx < g.NN; idx += nthr) {
    const int pos = s_pos[idx], lvl = pos >> 16, by = (pos >> 8) & 255, bx = pos & 255;
    float n = s_n[idx];
    if (pos >= 0 && lvl >= 1) {
      const int c = node_index(g, lvl - 1, 2 * by, 2 * bx), side = g.P >> (lvl - 1);
      n = ((s_sim[c] + s_sim[c + 1]) + s_sim[c + side]) + s_sim[c + side + 1];  // (zero where there is no child)
      s_n[idx] = n;
    }
    nrm2[fo + idx] = n;
  }
  __syncthreads();
  for (int idx = tid; idx < g.NN; idx += nthr) {
    const int pos = s_pos[idx], lvl = pos >> 16, by = (pos >> 8) & 255, bx = pos & 255;
    float v = 0.f;
    if (pos >= 0 && lvl < g.L) v = cosine_from(s_sim[idx], s_n[idx], s_n[node_index(g, lvl + 1, by >> 1, bx >> 1)]);
    sim[fo + idx] = v;
    s_m[idx] = v;  // the similarities, until the next step has read them
  }
  __syncthreads();
  for (int idx = tid; idx < g.NN; idx += nthr) {
    const int pos = s_pos[idx], lvl = pos >> 16, by = (pos >> 8) & 255, bx = pos & 255;
    float mv = 2.f;
    if (pos >= 0 && lvl >= 1) {
      const int c = node_index(g, lvl - 1, 2 * by, 2 * bx), side = g.P >> (lvl - 1);
      bool nan = false;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int ci = c + (k >> 1) * side + (k & 1);
        if (s_pos[ci] < 0) continue;
        const float v = s_m[ci];
        if (v != v) nan = true;
        mv = fminf(mv, v);
      }
      if (nan) mv = __uint_as_float(0x7fc00000u);
    }
    s_sim[idx] = mv;  // m in LDS
    m[fo + idx] = mv;
  }
  __syncthreads();
  if (decide.node_map) {  // the caller has named the threshold: the frame's partition (see k_spatial_decide)
    const int b = f / g.T;
    const float t = decide.given.n ? decide.given.v[b] : decide.tau[b];
    if (decide.given.n && f % g.T == 0 && tid == 0) decide.tau[b] = t;
    for (int c = tid; c < g.HW; c += nthr) {
      const int y = c / g.W, x = c - y * g.W;
      int l = g.L;
      while (l >= 1 && !(s_sim[node_index(g, l, y >> l, x >> l)] > t)) --l;
      decide.node_map[f * g.HW + c] = f * g.HW + (y >> l << l) * g.W + (x >> l << l);
      if (decide.node_level) decide.node_level[f * g.HW + c] = (uint8_t)l;
    }
  }
#pragma unroll 1
  for (int i0 = g.lvl_base[1]; i0 < g.NN; i0 += nthr) {  // uniform trip count: the histogram update is wave-wide
    const int idx = i0 + tid;
    uint32_t key = 0;
    unsigned wgt = 0;
    if (idx < g.NN) {
      const int pos = s_pos[idx], lvl = pos >> 16, by = (pos >> 8) & 255, bx = pos & 255;
      // compact (value, weight) element of the budget search: upper-level nodes with >= 2 children
      if (pos >= 0) {
        float s = -2.f;
        for (int l = lvl, y = by, x = bx; l <= g.L; ++l, y >>= 1, x >>= 1) {
          const float v = s_sim[node_index(g, l, y, x)];
          s = fmaxf(s, (v != v) ? -2.f : v);  // NaN always splits
        }
        const int h = ((2 * by + 1) << (lvl - 1)) < g.H, w = ((2 * bx + 1) << (lvl - 1)) < g.W;
        wgt = (unsigned)((1 + h) * (1 + w) - 1);  // children beyond the first
        if (wgt) key = float_key(s);
      }
      const size_t o = (size_t)f * (g.NN - g.lvl_base[1]) + (idx - g.lvl_base[1]);
      sel_key[o] = key;
      sel_w[o] = (uint8_t)wgt;
    }
    wave_hist_add(h0, wgt != 0, sel_bin(key), wgt);
  }
  __syncthreads();
  sel_flush_bins(sel + f / g.T, h0);
}

void launch_spatial_finalize(const Geo& g, const float* part, float* nsum, float* nrm2, float* sim, float* m,
                             uint32_t* sel_key, uint8_t* sel_w, SelState* sel, int* item_count, const DecideArgs& decide,
                             hipStream_t s) {
  const int up = g.L < 4 ? 0 : (g.P == 16 ? 1 : 2);
  const int threads = up == 2 && g.F <= kFinWideFrames ? kFinThreadsWide : (g.NN <= 256 && !up ? 256 : kFinThreads);  // one node per thread where it fits
  const size_t lds = ((size_t)unit_cols(g) * unit_rows(g) * kUnitStats + 4 * (size_t)g.NN) * sizeof(float);
  if (up == 0)
    hipLaunchKernelGGL(k_spatial_finalize<0>, dim3(g.F), dim3(threads), lds, s, g, part, nsum, nrm2, sim, m, sel_key, sel_w, sel, item_count, decide);
  else if (up == 1)
    hipLaunchKernelGGL(k_spatial_finalize<1>, dim3(g.F), dim3(threads), lds, s, g, part, nsum, nrm2, sim, m, sel_key, sel_w, sel, item_count, decide);
  else
    hipLaunchKernelGGL(k_spatial_finalize<2>, dim3(g.F), dim3(threads), lds, s, g, part, nsum, nrm2, sim, m, sel_key, sel_w, sel, item_count, decide);
}

// ------------------------------------------------------------------------------------------------
// k_spatial_decide: coarse-to-fine search (Sec. 3.2). Grid (cells of a video / threads, videos); one thread per cell
// walks down from its root: the first node on the path whose smallest child similarity exceeds tau_S is kept. (Where the caller
// has named the threshold k_spatial_finalize does so itself: 8 frames of 8x8 45.0 -> 43.9 us a pass, six clips of 25 frames of
// 15x20 156.3 -> 155.2, 85 frames of 31x31 379.7 -> 377.8.)
// Large videos, and searches through many keys, take fewer and larger workgroups, since each carries the search out (512 frames
// of 13x13 random vectors 19.8 -> 16.3 us, moving scenes of that size 10.9 and 11.1, of 46 frames of 27x27 9.9 and 10.4; 1024
// threads 16.8, 12.3, 11.8).
// ------------------------------------------------------------------------------------------------
constexpr int kDecideWide = 65536, kDecideThreads = 512;
// A search that looks through more keys than this has larger workgroups as well.
constexpr int kSelFewKeys = 2048;
template <int THREADS, int KIND>
__global__ __launch_bounds__(THREADS) void k_spatial_decide(Geo g, const float* __restrict__ m,
                                                                float* __restrict__ tau, SelSearch pending,
                                                                int32_t* __restrict__ node_map,
                                                                uint8_t* __restrict__ node_level) {
  const int b = blockIdx.y, per_video = g.T * g.HW;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int i = b * per_video + min(j, per_video - 1);
  const int f = i / g.HW, c = i - f * g.HW;
  const int y = c / g.W, x = c - y * g.W;
  // the path's nodes do not depend on the threshold: they are on their way while it is being found
  float path[kMaxLevels];
#pragma unroll
  for (int l = 1; l < kMaxLevels; ++l)  // (no branches: of a level above the roots the roots are read again)
    path[l] = m[(size_t)f * g.NN + node_index(g, min(l, g.L), y >> min(l, g.L), x >> min(l, g.L))];
  float t;
  if constexpr (KIND != kTauKnown) {  // the budget search was left to this kernel
    t = sel_threshold<THREADS, KIND>(g, pending, b);
    if (blockIdx.x == 0 && threadIdx.x == 0) tau[b] = t;
  } else {
    t = tau[b];
  }
  if (j >= per_video) return;
  int lvl = 0;
#pragma unroll
  for (int l = 1; l < kMaxLevels; ++l)
    if (l <= g.L && path[l] > t) lvl = l;  // (the last one that passes is the coarsest)
  const int y0 = (y >> lvl) << lvl, x0 = (x >> lvl) << lvl;
  node_map[i] = f * g.HW + y0 * g.W + x0;
  if (node_level) node_level[i] = (uint8_t)lvl;
}

void launch_spatial_decide(const Geo& g, const float* m, float* tau, const SelSearch& pending, int32_t* node_map, uint8_t* node_level, hipStream_t s) {
  const int per_video = g.T * g.HW;
  const bool look = tau_kind(pending) == kTauLook && pending.per_video > kSelFewKeys;  // through all keys
  const bool wide = per_video > kDecideWide || look;
  with_tau_kind(pending, [&](auto kind) {
    constexpr int KIND = decltype(kind)::value;
    const int threads = wide ? kDecideThreads : kSelThreads;
    const auto kernel = wide ? k_spatial_decide<kDecideThreads, KIND> : k_spatial_decide<kSelThreads, KIND>;
    hipLaunchKernelGGL(kernel, dim3((per_video + threads - 1) / threads, g.B), dim3(threads), 0, s, g, m, tau, pending,
                       node_map, node_level);
  });
}

// Recovers node levels from a node map (callers may pass node_level == NULL to the temporal stage).
__global__ __launch_bounds__(256) void k_node_levels(Geo g, const int32_t* __restrict__ node_map,
                                                     uint8_t* __restrict__ node_level) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.N) return;
  const int f = i / g.HW, c = i - f * g.HW;
  const int y = c / g.W, x = c - y * g.W;
  const int r = node_map[i] - f * g.HW;
  const int y0 = r / g.W, x0 = r - y0 * g.W;
  // smallest level whose block at (y0, x0) contains (y, x) and is aligned; the partition's block is
  // the largest aligned block rooted at (y0,x0) in which every valid cell maps to it -- found by growing.
  int lvl = 0;
  while (lvl < g.L) {
    const int s2 = 2 << lvl;
    if ((y0 & (s2 - 1)) || (x0 & (s2 - 1))) break;
    // the candidate block [y0, y0+s2) x [x0, x0+s2): its bottom-right valid corner must map to r as well
    const int yy = min(y0 + s2 - 1, g.H - 1), xx = min(x0 + s2 - 1, g.W - 1);
    if (node_map[f * g.HW + yy * g.W + xx] - f * g.HW != r) break;
    ++lvl;
  }
  (void)y; (void)x;
  node_level[i] = (uint8_t)lvl;
}

void launch_node_levels(const Geo& g, const int32_t* node_map, uint8_t* node_level, hipStream_t s) {
  hipLaunchKernelGGL(k_node_levels, dim3((g.N + 255) / 256), dim3(256), 0, s, g, node_map, node_level);
}

// ------------------------------------------------------------------------------------------------
// Budget-driven thresholds (see SelState). The statistics pass of the stage has filled the histogram of bins;
// k_select_list, grid (slices, videos), picks the bin and lists its elements, and every workgroup of the kernel that uses
// the threshold finds the value among those (sel_threshold). Of a video of up to kSelWhole elements such a workgroup picks the
// bin and looks through all keys by itself, and no launch is made for the search: passes of 64 frames of 13x13 (5440 and 10,816
// elements) 116.8 us with the list and 112.6 without, of 16x16 (16,384) 105.7 and 101.4; 180 of 14x14 (14,400 and 35,280)
// 227.4 with the list for both, 223.4 without the smaller one's, 225.4 without both; 512 of 13x13 (43,520) 402 and 409.
// Every workgroup of every video looks through its video's keys, so in a batch the elements of all videos count as well, up to
// kSelWholeAll of them. Passes over B videos of 13x13 at D = 512 with the list and without (temporal elements in all): 32 of
// 16 frames (86,528) 140.8 and 139.8 us, 8 of 64 (86,528) 139.6 and 135.7, 12 of 64 (129,792) 172.0 and 173.0, 8 of 100
// (135,200) 180.2 and 179.7, 16 of 64 (173,056) 198.5 and 201.9, 16 of 100 (270,400) 267.8 and 274.7; 8 of 64 frames of 16x16
// (131,072) 157.6 and 154.5, 64 of 40 of 8x8 (163,840) 199.4 and 211.3. Where the thresholds are handed back one workgroup a
// video looks, whatever B is: 16 of 64 frames of 13x13 247 and 242, 16 of 100 317 and 314.
// Input: keys[video][per_video] (0 = not an element), weights (NULL = 1 for every element).
// What it costs is launches and dependent loads. Against a radix search of 11 + 11 + 10 bits, two launches and the last
// digit in the kernel that uses the threshold (the first bits of a float tell similarities apart badly: four bins from a
// half to one), both searches of a pass with those kernels, us: 64 frames of 13x13 35 -> 27, 512 of 13x13 39 -> 27, 180 of
// 18x24 40 -> 28; one image with the value handed back 21 -> 13. (One workgroup for every video up to 16384 elements instead
// of the list: 15 us more at 64 frames.)
// ------------------------------------------------------------------------------------------------
// (The host-thread build of the tests that takes the large inputs' kernels lists the elements of every search.)
#ifndef STTM_SEL_WHOLE
#define STTM_SEL_WHOLE 20480
#endif
constexpr int kSelWhole = STTM_SEL_WHOLE, kSelWholeAll = 131072;
constexpr int kSelThreadsWhole = 1024;
// Threads of the listing pass, and elements per thread. (Fewer in the host-thread build: a small input has several workgroups.)
#ifndef STTM_SEL_THREADS
#define STTM_SEL_THREADS 512
#endif
constexpr int kPassThreads = STTM_SEL_THREADS, kSelPer = 4;
// A bin of more weight than this is crowded.
#ifndef STTM_SEL_CROWD
#define STTM_SEL_CROWD 4096
#endif
constexpr unsigned kSelCrowd = STTM_SEL_CROWD;

// A workgroup's slice of the elements, kSelPer to a thread.
struct SelSlice {
  uint32_t key[kSelPer];
  unsigned w[kSelPer];
};
__device__ inline SelSlice sel_load(const uint32_t* keys, const uint8_t* weights, int per_video, int b) {
  SelSlice q;
#pragma unroll
  for (int u = 0; u < kSelPer; ++u) {
    const int j = (blockIdx.x * kSelPer + u) * kPassThreads + threadIdx.x;
    const size_t at = (size_t)b * per_video + j;
    q.key[u] = j < per_video ? keys[at] : 0u;
    q.w[u] = weights && j < per_video ? weights[at] : 1u;
  }
  return q;
}

// Appends the elements of the slice whose `where` (a bin, or a piece of one) is `picked` to the list, and notes the largest key
// with a smaller one.
template <class Where>
__device__ inline void sel_append(SelSlice& q, Where where, unsigned picked, SelList* l, int per_video, int b,
                                  uint32_t* __restrict__ list_key, uint8_t* __restrict__ list_w) {
  __shared__ unsigned s_lo, s_n, s_at;
  const int tid = threadIdx.x, lane = tid & 63;
  if (tid == 0) s_lo = s_n = 0;
  __syncthreads();
  unsigned lo = 0, place[kSelPer];  // key 0 is below every real value
#pragma unroll
  for (int u = 0; u < kSelPer; ++u) {
    const unsigned at = q.key[u] ? where(q.key[u]) : 0xffffffffu;
    if (at < picked) lo = max(lo, q.key[u]);
    place[u] = 0xffffffffu;
    // Equal keys of the wavefront's 64 become one element (for the two most frequent of them): still scenes are full of
    // them, and so are the scores of a node's descendants, which are the node's.
    unsigned long long todo = __ballot(at == picked);
#pragma unroll 1
    for (int it = 0; it < 2 && __popcll(todo) > 8; ++it) {
      const int leader = __ffsll((long long)todo) - 1;
      const uint32_t leads = (uint32_t)__shfl((int)q.key[u], leader, 64);  // (by all lanes, whatever their own key)
      const bool mine = at == picked && q.key[u] == leads;
      const unsigned long long m = __ballot(mine);
      const unsigned sum = __popcll(__ballot(mine && (q.w[u] & 1))) + 2u * __popcll(__ballot(mine && (q.w[u] & 2)));
      if (lane == leader) {
        place[u] = atomicAdd(&s_n, 1u);
        q.w[u] = sum;
      }
      todo &= ~m;
    }
    if ((todo >> lane) & 1ull) place[u] = atomicAdd(&s_n, 1u);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) lo = max(lo, (unsigned)__shfl_xor((int)lo, o, 64));
  if (lane == 0 && lo) atomicMax(&s_lo, lo);
  __syncthreads();
  if (tid == 0) {
    if (s_lo) atomicMax(&l->lo, s_lo);
    s_at = s_n ? atomicAdd(&l->count, s_n) : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kSelPer; ++u) {
    if (place[u] == 0xffffffffu || s_at + place[u] >= (unsigned)per_video) continue;  // (never beyond the list's room)
    const size_t o = (size_t)b * per_video + s_at + place[u];
    list_key[o] = q.key[u];
    list_w[o] = (uint8_t)q.w[u];  // (at most 64 elements of weight 3)
  }
}

// REFINE: a crowded bin is not listed, its pieces' weights are counted for k_select_piece.
template <bool REFINE>
__global__ __launch_bounds__(kPassThreads) void k_select_list(Geo g, const uint32_t* __restrict__ keys,
                                                             const uint8_t* __restrict__ weights, int per_video,
                                                             const int* __restrict__ target, int base_const,
                                                             const int32_t* __restrict__ node_map,
                                                             SelState* __restrict__ states,
                                                             uint32_t* __restrict__ list_key,
                                                             uint8_t* __restrict__ list_w) {
  __shared__ unsigned s_list;
  const int b = blockIdx.y, tid = threadIdx.x;
  SelState* st = states + b;
  // the slice's keys do not depend on the search: their loads fly while the bin is being found
  SelSlice q = sel_load(keys, weights, per_video, b);
  unsigned turn = 0, weight = 0;
  if (tid == 0) turn = atomicAdd(&st->begun, 1u);
  SelFound fd = {};
  sel_pick<kSelCopies, kPassThreads>(g, b, st->hist0[0], target, base_const, node_map, fd, weight);
  fd.crowded = REFINE && fd.rc == 0 && weight > kSelCrowd;
  if (tid == 0) {
    fd.list = turn >= gridDim.x;
    if (turn == 2 * gridDim.x - 1) atomicExch(&st->begun, 0u);  // (every workgroup of both searches has its number)
    if (blockIdx.x == 0) {
      st->found[0] = fd;
      st->list[1 - fd.list] = {0u, 0u};  // for the next search
    }
    s_list = fd.list;
  }
  if (!REFINE && fd.rc) return;  // uniform over the workgroup
  __syncthreads();
  const unsigned list = s_list;
  if constexpr (REFINE) {
    if (blockIdx.x == 0)
      for (int j = tid; j < kSelBins; j += kPassThreads) st->pieces[1 - list][j] = 0;
    if (fd.rc) return;
    if (fd.crowded) {
      __shared__ unsigned h[kSelBins];
      for (int j = tid; j < kSelBins; j += kPassThreads) h[j] = 0;
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kSelPer; ++u)
        wave_hist_add(h, q.key[u] && sel_bin(q.key[u]) == fd.bin, sel_piece(q.key[u]) & (kSelBins - 1), q.w[u]);
      __syncthreads();
      for (int j = tid; j < kSelBins; j += kPassThreads)
        if (h[j]) atomicAdd(&st->pieces[list][j], h[j]);
      return;
    }
  }
  sel_append(q, [](uint32_t key) { return sel_bin(key); }, fd.bin, &st->list[list], per_video, b, list_key, list_w);
}

// The second pass over a video whose picked bin is crowded: lists one piece of it.
__global__ __launch_bounds__(kPassThreads) void k_select_piece(Geo g, const uint32_t* __restrict__ keys,
                                                              const uint8_t* __restrict__ weights, int per_video,
                                                              SelState* __restrict__ states,
                                                              uint32_t* __restrict__ list_key,
                                                              uint8_t* __restrict__ list_w) {
  const int b = blockIdx.y;
  SelState* st = states + b;
  SelFound fd = st->found[0];
  if (!fd.crowded) return;  // uniform over the workgroup, as everywhere
  SelSlice q = sel_load(keys, weights, per_video, b);
  const unsigned bin = fd.bin;
  unsigned weight;
  sel_pick<1, kPassThreads>(g, b, st->pieces[fd.list], nullptr, 0, nullptr, fd, weight);
  if (fd.rc) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) st->found[1] = fd;
  sel_append(q, [](uint32_t key) { return sel_piece(key); }, bin * kSelBins + fd.bin, &st->list[fd.list], per_video, b,
             list_key, list_w);
}

// The whole search as a launch of its own (when the caller wants the threshold back).
template <int THREADS, int KIND>
__global__ __launch_bounds__(THREADS) void k_select_tau(Geo g, SelSearch search, float* __restrict__ tau,
                                                        float* __restrict__ host_tau) {
  const float t = sel_threshold<THREADS, KIND>(g, search, blockIdx.x);
  if (threadIdx.x == 0) {
    tau[blockIdx.x] = t;
    if (host_tau) host_tau[blockIdx.x] = t;
  }
}

static SelSearch launch_select(const Geo& g, const uint32_t* keys, const uint8_t* weights, int per_video,
                               const int* target, int base_const, const int32_t* node_map, SelState* st,
                               uint32_t* list_key, uint8_t* list_w, bool handed_back, hipStream_t s) {
  SelSearch q = {st, keys, weights, per_video, false, target, base_const, node_map};
  const bool few = handed_back || per_video <= kSelFewKeys || (long long)g.B * per_video <= kSelWholeAll;
  if (per_video <= kSelWhole && few) return q;
  const dim3 grid((per_video + kPassThreads * kSelPer - 1) / (kPassThreads * kSelPer), g.B), block(kPassThreads);
  if (per_video > kSelRefine) {
    hipLaunchKernelGGL(k_select_list<true>, grid, block, 0, s, g, keys, weights, per_video, target, base_const, node_map, st,
                       list_key, list_w);
    hipLaunchKernelGGL(k_select_piece, grid, block, 0, s, g, keys, weights, per_video, st, list_key, list_w);
  } else {
    hipLaunchKernelGGL(k_select_list<false>, grid, block, 0, s, g, keys, weights, per_video, target, base_const, node_map, st,
                       list_key, list_w);
  }
  q.keys = list_key;
  q.weights = list_w;
  q.listed = true;
  return q;
}

int select_elements(const Geo& g, bool spatial) { return g.T * (spatial ? g.NN - g.lvl_base[1] : g.HW); }

SelSearch launch_select_spatial(const Geo& g, const uint32_t* keys, const uint8_t* weights, const int* target,
                                SelState* state, uint32_t* list_key, uint8_t* list_w, bool handed_back,
                                hipStream_t s) {
  int roots = 0;
  for (int ry = 0; ry < g.R; ++ry)
    for (int rx = 0; rx < g.R; ++rx) roots += node_exists(g, g.L, ry, rx);
  return launch_select(g, keys, weights, select_elements(g, true), target, roots * g.T, nullptr, state, list_key, list_w,
                       handed_back, s);
}

SelSearch launch_select_temporal(const Geo& g, const int32_t* node_map, const uint32_t* keys, const int* target,
                                 SelState* state, uint32_t* list_key, uint8_t* list_w, bool handed_back,
                                 hipStream_t s) {
  return launch_select(g, keys, nullptr, select_elements(g, false), target, 0, node_map, state, list_key, list_w, handed_back,
                       s);
}

void launch_select_tau(const Geo& g, const SelSearch& search, float* tau, float* host_tau, hipStream_t s) {
  const bool whole = !search.listed && search.per_video > kSelFewKeys;
  const int threads = whole ? kSelThreadsWhole : kSelThreads;
  const auto kernel = search.listed ? k_select_tau<kSelThreads, kTauListed>
                      : whole       ? k_select_tau<kSelThreadsWhole, kTauLook>
                                    : k_select_tau<kSelThreads, kTauLook>;
  hipLaunchKernelGGL(kernel, dim3(g.B), dim3(threads), 0, s, g, search, tau, host_tau);
}

}  // namespace sttm
