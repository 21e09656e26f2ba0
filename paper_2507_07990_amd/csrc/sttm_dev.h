// Shared declarations of the HIP kernels behind libsttm (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stddef.h>
#include <stdint.h>
#include <type_traits>

// Dynamic LDS of a kernel. (The second form serves the host-thread build used by the CPU tests.)
#ifndef STTM_HOST_EMULATION
#define STTM_DYNAMIC_LDS(T, name) extern __shared__ T name[]
#else
#define STTM_DYNAMIC_LDS(T, name) T* name = reinterpret_cast<T*>(hip_emul::g_dynamic_lds)
#endif

// A value in a scalar / vector register that the compiler must take as new from here on.
#ifndef STTM_HOST_EMULATION
#define STTM_OPAQUE_S(x) asm volatile("" : "+s"(x))
#define STTM_OPAQUE_V(x) asm volatile("" : "+v"(x))
#else
#define STTM_OPAQUE_S(x) ((void)(x))
#define STTM_OPAQUE_V(x) ((void)(x))
#endif

namespace sttm {

constexpr int kWave = 64;
constexpr int kMaxLevels = 6;  // P <= 32  =>  levels 0..5

// Problem geometry, passed by value to every kernel.
struct Geo {
  int B, T, H, W, D;
  int P;         // padded power-of-two grid side
  int L;         // root level = log2(P / R)
  int R;         // root nodes per side
  int HW;        // valid cells per frame
  int F;         // frames = B*T
  int NN;        // pyramid nodes per frame (levels 0..L of the P x P grid)
  int lvl_base[kMaxLevels + 1];
  int dtype;     // 0 = f32, 1 = bf16, 2 = f16
  int vec;       // channels per lane per 16-byte load: 4 (f32) / 8 (bf16, f16)
  int cch;       // channels per chunk = 64 * vec (one wavefront spans one chunk of a token row)
  int nC;        // chunks per row = ceil(D / cch)
  int N;         // B*T*H*W
};

// First node index of a level: sum over the finer levels k of (P >> k)^2 = 4 (P^2 - (P >> lvl)^2) / 3. Computed, not
// looked up: with a per-lane level the table in the kernel arguments would cost a memory access each time.
__host__ __device__ inline int level_base(const Geo& g, int lvl) {
  const int q = g.P >> lvl;
  return (g.P * g.P - q * q) * 4 / 3;
}

__host__ __device__ inline int node_index(const Geo& g, int lvl, int by, int bx) {
  return level_base(g, lvl) + by * (g.P >> lvl) + bx;
}

__host__ __device__ inline bool node_exists(const Geo& g, int lvl, int by, int bx) {
  return (by << lvl) < g.H && (bx << lvl) < g.W;
}

// Decodes a per-frame node index into (level, by, bx).
__host__ __device__ inline void node_decode(const Geo& g, int idx, int& lvl, int& by, int& bx) {
  lvl = 0;
  while (lvl < g.L && idx >= level_base(g, lvl + 1)) ++lvl;
  const int r = idx - level_base(g, lvl);
  const int sh = __builtin_ctz((unsigned)g.P) - lvl;  // the level's grid side is a power of two
  by = r >> sh;
  bx = r & ((1 << sh) - 1);
}

// ---- the packed dot product of the target -----------------------------------------------------------------
// c + a.lo * b.lo + a.hi * b.hi on the two 16-bit values each register holds (v_dot2c_f32_bf16, v_dot2_f32_f16: the
// products of two 16-bit values are exact in fp32), and a pair of constants handed over as register contents the
// compiler cannot look into: written as literals, the bf16 pair (1, 0) = 0x00003f80 is encoded as the inline operand
// "1.0", which the instruction does not read as this pair. These three are all that differs in the host-thread
// build of the tests; everything built on them is the same code in both.
#ifndef STTM_HOST_EMULATION
__device__ inline float dot2_bf16(uint32_t a, uint32_t b, float c) {
  typedef __bf16 pair __attribute__((ext_vector_type(2)));
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(pair, a), __builtin_bit_cast(pair, b), c, false);
}
__device__ inline float dot2_f16(uint32_t a, uint32_t b, float c) {
  typedef _Float16 pair __attribute__((ext_vector_type(2)));
  return __builtin_amdgcn_fdot2(__builtin_bit_cast(pair, a), __builtin_bit_cast(pair, b), c, false);
}
template <uint32_t LO, uint32_t HI>
__device__ inline void opaque_pairs(uint32_t& lo, uint32_t& hi) {
  asm volatile("s_mov_b32 %0, %2\n\ts_mov_b32 %1, %3" : "=s"(lo), "=s"(hi) : "i"(LO), "i"(HI));
}
#else
inline float dot2_bf16(uint32_t a, uint32_t b, float c) {
  return fmaf(__uint_as_float(a & 0xffff0000u), __uint_as_float(b & 0xffff0000u),
              fmaf(__uint_as_float(a << 16), __uint_as_float(b << 16), c));
}
inline float dot2_f16(uint32_t a, uint32_t b, float c) {
  return fmaf(__half2float(__ushort_as_half((unsigned short)(a >> 16))),
              __half2float(__ushort_as_half((unsigned short)(b >> 16))),
              fmaf(__half2float(__ushort_as_half((unsigned short)(a & 0xffffu))),
                   __half2float(__ushort_as_half((unsigned short)(b & 0xffffu))), c));
}
template <uint32_t LO, uint32_t HI>
inline void opaque_pairs(uint32_t& lo, uint32_t& hi) { lo = LO; hi = HI; }
#endif

// ---- widening sums on the matrix cores ---------------------------------------------------------------------
// S[0..3] += the four 16-bit channels a lane holds in two registers, as a product of the 4x4 identity with the lanes'
// channels (v_mfma_f32_4x4x4_16b: sixteen products side by side, four lanes each; a lane's column is its own channels, and
// row i of the result is its register i). One instruction on an otherwise idle pipe instead of four on the vector one; the
// same bits for every finite input, subnormal ones included (4 x 10^6 random sums compared for either type). Where a value
// is an infinity or a NaN, all four of the lane's sums come out as NaN: similarities are undefined then in any case, but a
// sum that is kept for the rows of the output is formed again by Row::add_row (unit_pair_sums).
// `ident`: this lane's row of the identity (identity_row).
#ifndef STTM_HOST_EMULATION
typedef float sttm_sum4 __attribute__((ext_vector_type(4)));
template <uint32_t ONE>
__device__ inline uint2 identity_row() {
  const unsigned i = threadIdx.x & 3;
  return make_uint2(i == 0 ? ONE : (i == 1 ? ONE << 16 : 0u), i == 2 ? ONE : (i == 3 ? ONE << 16 : 0u));
}
__device__ inline sttm_sum4 widen_add_bf16(uint2 ident, uint32_t lo, uint32_t hi, sttm_sum4 s) {
  typedef short quad __attribute__((ext_vector_type(4)));
  return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(quad, ident), __builtin_bit_cast(quad, make_uint2(lo, hi)), s, 0, 0, 0);
}
__device__ inline sttm_sum4 widen_add_f16(uint2 ident, uint32_t lo, uint32_t hi, sttm_sum4 s) {
  typedef _Float16 quad __attribute__((ext_vector_type(4)));
  return __builtin_amdgcn_mfma_f32_4x4x4f16(__builtin_bit_cast(quad, ident), __builtin_bit_cast(quad, make_uint2(lo, hi)), s, 0, 0, 0);
}
#else
struct sttm_sum4 {
  float v[4];
  float& operator[](int i) { return v[i]; }
};
template <uint32_t ONE>
inline uint2 identity_row() { return make_uint2(0u, 0u); }
inline sttm_sum4 widen_add_bf16(uint2, uint32_t lo, uint32_t hi, sttm_sum4 s) {
  for (int i = 0; i < 4; ++i) s[i] += __uint_as_float((i < 2 ? lo : hi) >> 16 * (i & 1) << 16);
  return s;
}
inline sttm_sum4 widen_add_f16(uint2, uint32_t lo, uint32_t hi, sttm_sum4 s) {
  for (int i = 0; i < 4; ++i) s[i] += __half2float(__ushort_as_half((unsigned short)((i < 2 ? lo : hi) >> 16 * (i & 1))));
  return s;
}
#endif

// ---- feature row access: one lane owns `VEC` consecutive channels ------------------------------------
template <int DT> struct Row;  // DT: 0 = f32, 1 = bf16, 2 = f16

template <> struct Row<0> {
  static constexpr int VEC = 4;
  typedef float4 Raw;
  typedef float Elem;
  __device__ static inline Raw zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
  __device__ static inline void unpack(const Raw& r, float (&x)[4]) {
    x[0] = r.x; x[1] = r.y; x[2] = r.z; x[3] = r.w;
  }
  // this lane's share of the dot product of two rows
  __device__ static inline float dot(const Raw& a, const Raw& b) {
    return fmaf(a.x, b.x, fmaf(a.y, b.y, fmaf(a.z, b.z, a.w * b.w)));
  }
  // S += the row's channels
  __device__ static inline void add_row(const Raw& r, float (&S)[4]) {
    S[0] += r.x; S[1] += r.y; S[2] += r.z; S[3] += r.w;
  }
  // S = the sum of four rows, added up in their order (`ident`: see identity_row; not needed here)
  __device__ static inline uint2 ident() { return make_uint2(0u, 0u); }
  __device__ static inline void sum4(uint2, const Raw* r, float (&S)[4]) {
#pragma unroll
    for (int v = 0; v < 4; ++v) S[v] = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) add_row(r[k], S);
  }
};

template <> struct Row<1> {
  static constexpr int VEC = 8;
  typedef uint4 Raw;
  typedef uint16_t Elem;
  __device__ static inline Raw zero() { return make_uint4(0u, 0u, 0u, 0u); }
  __device__ static inline void unpack(const Raw& r, float (&x)[8]) {
    x[0] = __uint_as_float(r.x << 16); x[1] = __uint_as_float(r.x & 0xffff0000u);
    x[2] = __uint_as_float(r.y << 16); x[3] = __uint_as_float(r.y & 0xffff0000u);
    x[4] = __uint_as_float(r.z << 16); x[5] = __uint_as_float(r.z & 0xffff0000u);
    x[6] = __uint_as_float(r.w << 16); x[7] = __uint_as_float(r.w & 0xffff0000u);
  }
  // Straight from the packed pairs: one instruction multiplies two pairs and adds both products to the running
  // fp32 sum, so nothing has to be unpacked.
  __device__ static inline float dot(const Raw& a, const Raw& b) {
    return dot2_bf16(a.w, b.w, dot2_bf16(a.z, b.z, dot2_bf16(a.y, b.y, dot2_bf16(a.x, b.x, 0.f))));
  }
  // S += the row's channels: the same instruction against the constant pairs (1, 0) and (0, 1) widens a channel and
  // adds it in one step (multiplying the other channel by zero: exact for every finite value, and where a value is an
  // infinity or a NaN in the other element of the pair spills over, into a sum that is undefined then anyway).
  __device__ static inline void add_row(const Raw& r, float (&S)[8]) {
    uint32_t klo, khi;
    opaque_pairs<0x3f80u, 0x3f800000u>(klo, khi);
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      S[2 * j] = dot2_bf16(w[j], klo, S[2 * j]);
      S[2 * j + 1] = dot2_bf16(w[j], khi, S[2 * j + 1]);
    }
  }
  // S = the sum of four rows, added up in their order
  __device__ static inline uint2 ident() { return identity_row<0x3f80u>(); }
  __device__ static inline void sum4(uint2 ident, const Raw* r, float (&S)[8]) {
    sttm_sum4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      lo = widen_add_bf16(ident, r[k].x, r[k].y, lo);
      hi = widen_add_bf16(ident, r[k].z, r[k].w, hi);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      S[v] = lo[v];
      S[v + 4] = hi[v];
    }
  }
};

template <> struct Row<2> {
  static constexpr int VEC = 8;
  typedef uint4 Raw;
  typedef uint16_t Elem;
  __device__ static inline Raw zero() { return make_uint4(0u, 0u, 0u, 0u); }
  __device__ static inline float lo(uint32_t w) { return __half2float(__ushort_as_half((unsigned short)(w & 0xffffu))); }
  __device__ static inline float hi(uint32_t w) { return __half2float(__ushort_as_half((unsigned short)(w >> 16))); }
  __device__ static inline void unpack(const Raw& r, float (&x)[8]) {
    x[0] = lo(r.x); x[1] = hi(r.x); x[2] = lo(r.y); x[3] = hi(r.y);
    x[4] = lo(r.z); x[5] = hi(r.z); x[6] = lo(r.w); x[7] = hi(r.w);
  }
  __device__ static inline float dot(const Raw& a, const Raw& b) {
    return dot2_f16(a.w, b.w, dot2_f16(a.z, b.z, dot2_f16(a.y, b.y, dot2_f16(a.x, b.x, 0.f))));
  }
  // S += the row's channels (see Row<1>::add_row)
  __device__ static inline void add_row(const Raw& r, float (&S)[8]) {
    uint32_t klo, khi;
    opaque_pairs<0x3c00u, 0x3c000000u>(klo, khi);
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      S[2 * j] = dot2_f16(w[j], klo, S[2 * j]);
      S[2 * j + 1] = dot2_f16(w[j], khi, S[2 * j + 1]);
    }
  }
  // S = the sum of four rows, added up in their order
  __device__ static inline uint2 ident() { return identity_row<0x3c00u>(); }
  __device__ static inline void sum4(uint2 ident, const Raw* r, float (&S)[8]) {
    sttm_sum4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      lo = widen_add_f16(ident, r[k].x, r[k].y, lo);
      hi = widen_add_f16(ident, r[k].z, r[k].w, hi);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      S[v] = lo[v];
      S[v + 4] = hi[v];
    }
  }
};

// 16-byte accesses for data that is touched once (the gather's rows and its output): marked non-temporal so that
// they do not displace what later kernels want to find in the caches.
#ifndef STTM_HOST_EMULATION
typedef unsigned int sttm_u32x4 __attribute__((ext_vector_type(4)));
typedef float sttm_f32x4 __attribute__((ext_vector_type(4)));
__device__ inline uint4 load_once(const uint4* p) {
  const sttm_u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const sttm_u32x4*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ inline float4 load_once(const float4* p) {
  const sttm_f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const sttm_f32x4*>(p));
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ inline void store_once(uint4* p, const uint4& v) {
  sttm_u32x4 w = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(w, reinterpret_cast<sttm_u32x4*>(p));
}
__device__ inline void store_once(float4* p, const float4& v) {
  sttm_f32x4 w = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(w, reinterpret_cast<sttm_f32x4*>(p));
}
#else
template <class T> inline T load_once(const T* p) { return *p; }
template <class T> inline void store_once(T* p, const T& v) { *p = v; }
#endif

// A stretch of global memory with its length: a load beyond it gives zeros and fetches nothing, a store beyond it is
// dropped, by the hardware's own check of every access against the length. Address = base + uniform + lane.
#ifndef STTM_HOST_EMULATION
typedef __amdgpu_buffer_rsrc_t Window;
__device__ __forceinline__ Window make_window(const void* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
template <class Raw>
__device__ __forceinline__ Raw window_load_once(Window w, unsigned lane_off, unsigned uniform_off) {
  return __builtin_bit_cast(Raw, __builtin_amdgcn_raw_buffer_load_b128(w, (int)lane_off, (int)uniform_off, 2));  // (2: non-temporal)
}
__device__ __forceinline__ int window_load_i32(Window w, unsigned lane_off, unsigned uniform_off) {
  return (int)__builtin_amdgcn_raw_buffer_load_b32(w, (int)lane_off, (int)uniform_off, 0);
}
__device__ __forceinline__ int window_load_u8(Window w, unsigned lane_off, unsigned uniform_off) {
  return (int)__builtin_amdgcn_raw_buffer_load_b8(w, (int)lane_off, (int)uniform_off, 0);
}
__device__ __forceinline__ void window_store(Window w, unsigned lane_off, unsigned uniform_off, const float (&v)[1]) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[0]), w, (int)lane_off, (int)uniform_off, 0);
}
__device__ __forceinline__ void window_store(Window w, unsigned lane_off, unsigned uniform_off, const float (&v)[2]) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 d = {__float_as_uint(v[0]), __float_as_uint(v[1])};
  __builtin_amdgcn_raw_buffer_store_b64(d, w, (int)lane_off, (int)uniform_off, 0);
}
#else
struct Window { char* base; unsigned bytes; };
inline Window make_window(const void* base, unsigned bytes) {
  if (base && reinterpret_cast<uintptr_t>(base) < 65536) hip_emul::g_off_null = true;  // (no memory there: NULL and an offset)
  return {static_cast<char*>(const_cast<void*>(base)), bytes};
}
template <class Raw>
inline Raw window_load_once(const Window& w, unsigned lane_off, unsigned uniform_off) {
  Raw r;
  memset(&r, 0, sizeof r);
  if ((uint64_t)lane_off + uniform_off + sizeof r <= w.bytes) memcpy(&r, w.base + uniform_off + lane_off, sizeof r);
  return r;
}
inline int window_load_i32(const Window& w, unsigned lane_off, unsigned uniform_off) {
  int r = 0;
  if ((uint64_t)lane_off + uniform_off + sizeof r <= w.bytes) memcpy(&r, w.base + uniform_off + lane_off, sizeof r);
  return r;
}
inline int window_load_u8(const Window& w, unsigned lane_off, unsigned uniform_off) {
  return (uint64_t)lane_off + uniform_off < w.bytes ? (int)(uint8_t)w.base[uniform_off + lane_off] : 0;
}
template <int N>
inline void window_store(const Window& w, unsigned lane_off, unsigned uniform_off, const float (&v)[N]) {
  if ((uint64_t)lane_off + uniform_off + sizeof v <= w.bytes) memcpy(w.base + uniform_off + lane_off, v, sizeof v);
}
#endif

__device__ inline uint32_t f32_to_f16_rne(float f) { return (uint32_t)__half_as_ushort(__float2half_rn(f)); }

__device__ inline uint32_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;  // NaN stays NaN
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// Two fp32 values rounded to nearest even and packed into one register (a in the low half): one conversion
// instruction of the target per pair (v_cvt_pk_bf16_f32 / v_cvt_pk_f16_f32); the host-thread build of the tests
// rounds in integer arithmetic.
#ifndef STTM_HOST_EMULATION
__device__ inline uint32_t pack2_bf16(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ inline uint32_t pack2_f16(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
}
#else
inline uint32_t pack2_bf16(float a, float b) { return f32_to_bf16_rne(a) | (f32_to_bf16_rne(b) << 16); }
inline uint32_t pack2_f16(float a, float b) { return f32_to_f16_rne(a) | (f32_to_f16_rne(b) << 16); }
#endif

// cos(a, b) from the dot product and the two squared norms: clamped to <= 1, 0 for a zero norm.
__device__ inline float cosine_from(float dot, float na2, float nb2) {
  if (na2 == 0.f || nb2 == 0.f) return 0.f;
  float v = dot / (sqrtf(na2) * sqrtf(nb2));
  return v > 1.f ? 1.f : v;
}

// Monotone map float -> uint32 (order preserving for all non-NaN values).
__device__ inline uint32_t float_key(float v) {
  uint32_t u = __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float key_float(uint32_t k) {
  uint32_t u = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
  return __uint_as_float(u);
}

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// The value lane `src` holds, in a scalar register (`src` is the same in all lanes). What is derived from it is known to
// be the same in all lanes: scalar branches and scalar addresses, where a __shfl would give a vector and masked branches.
__device__ inline int lane_value(int v, int src) {
#ifndef STTM_HOST_EMULATION
  return __builtin_amdgcn_readlane(v, src);
#else
  return __shfl(v, src, 64);
#endif
}

// Running sum over the lanes of each row of sixteen, and over the wavefront; the largest value.
#ifndef STTM_HOST_EMULATION
__device__ inline unsigned row16_inclusive(unsigned v, int) {
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);  // row_shr:1 (zero from beyond the row)
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);
  return v;
}
__device__ inline unsigned wave_inclusive(unsigned v, int lane) {
  v = row16_inclusive(v, lane);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast:15, to the second and fourth row
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);  // row_bcast:31, to the third and fourth
  return v;
}
__device__ inline unsigned wave_max(unsigned v) {
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false));
  return (unsigned)lane_value((int)v, 63);
}
#else
inline unsigned wave_max(unsigned v) {
  for (int o = 32; o > 0; o >>= 1) v = max(v, (unsigned)__shfl_xor((int)v, o, 64));
  return v;
}
inline unsigned lanes_inclusive(unsigned v, int lane, int width) {
  for (int o = 1; o < width; o <<= 1) {
    const unsigned t = __shfl_up(v, o, 64);
    if ((lane & (width - 1)) >= o) v += t;
  }
  return v;
}
inline unsigned row16_inclusive(unsigned v, int lane) { return lanes_inclusive(v, lane, 16); }
inline unsigned wave_inclusive(unsigned v, int lane) { return lanes_inclusive(v, lane, 64); }
#endif

// Orders LDS traffic between the lanes of one wavefront (no cross-wave synchronisation).
__device__ inline void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- budget search state (one per video and stage) ---------------------------------------------------
// Token count as a function of the threshold is K(tau) = base + sum_j w_j [v_j <= tau]. The search is for the smallest v at
// which K exceeds the target and for the largest v below it. The kernels that make the values count their weight in a
// histogram of kSelBins bins (sel_bin); the bin in which K exceeds the target is picked from that, and of the few values
// in that bin the one is found exactly.
constexpr int kSelBins = 2048;
// The bin of a value, by its key: any function that never decreases would do. Equal steps in the logarithm of
// 1 + 2^-14 - v, 128 to the octave: 5e-7 wide at v = 1, where the similarities of still scenes crowd, 6e-5 at 0.99, 4e-3 at
// a half, 8e-3 below zero.
__device__ inline unsigned sel_bin(uint32_t key);
// The bin again, in its upper bits, with the piece of the bin that the value is in (2048 to a bin) in the lower 11.
__device__ inline unsigned sel_piece(uint32_t key);
// What a pass over a large input found.
struct SelFound {
  unsigned long long budget;  // target - base
  unsigned long long acc;     // weight of the keys in the bins (and pieces) before the picked one
  int rc;                     // 0 = searching, 1 = everything fits (tau = 1), 2 = the base alone exceeds the target
  int list;                   // which of the state's two lists holds the elements
  unsigned bin;
  int crowded;                // the picked bin holds too much to be listed: a second pass lists one of its pieces
};
// The list that such a pass makes of the picked bin; the elements themselves lie beside the state.
struct SelList {
  unsigned count;
  unsigned lo;                // the largest key in the bins before the picked one (0 = none)
};
// The histogram is fed by hundreds of workgroups whose values may crowd in a few bins; it is kept
// in kSelCopies copies, one per accelerator die (workgroups go to the dies round-robin by their index), so that
// the hot counters stay in one die's L2 instead of travelling between the dies with every atomic.
constexpr int kSelCopies = 8;
struct alignas(16) SelState {
  unsigned hist0[kSelCopies][kSelBins];  // weight per bin over all elements; the copies add up
  // Large inputs. Every search appends to an empty list, however often it is made on the same statistics, also where it is
  // replayed from a graph that was recorded without them: the searches take the two lists in turn, and each empties the
  // other's. Whose turn it is follows from `begun`, which every workgroup of the listing pass counts up as it begins; the
  // last one of the second search puts it back to zero.
  SelList list[2];
  unsigned begun;
  unsigned pad0;
  SelFound found[2];           // by the first pass, by the second one
  unsigned pad[10];
  unsigned pieces[2][kSelBins];  // weight per piece of the picked bin where that is crowded; taken in turn like the lists
};
static_assert(sizeof(SelState) % 128 == 0, "whole lines");

// Videos of more elements than this have a crowded bin searched piece by piece. Every workgroup of the kernel that uses the
// threshold looks at all listed elements, so what that costs grows with the square of a video's size where similarities
// crowd. 512 frames of 32x32, the searches and the kernels that use them, us, without and with the second pass: similarities
// within 10^-4 of one 112 and 73, unrelated vectors 102 and 69, moving blocks 72 and 68; 128 frames of 32x32 (within 10^-4) 54
// by one pass.
#ifndef STTM_SEL_REFINE
#define STTM_SEL_REFINE 131072
#endif
constexpr int kSelRefine = STTM_SEL_REFINE;

// One workgroup zeroes a state (of a video of `elements` elements).
__device__ inline void sel_clear(SelState* st, int elements) {
  unsigned* p = reinterpret_cast<unsigned*>(st);
  const int words = (int)((elements > kSelRefine ? sizeof(SelState) : offsetof(SelState, pieces)) / 4);
  for (int j = threadIdx.x; j < words; j += blockDim.x) p[j] = 0;
}

// The whole grid zeroes the states of `videos` videos.
__device__ inline void sel_clear_all(SelState* st, int videos, int elements) {
  constexpr int kWords = (int)(sizeof(SelState) / 4);
  const int words = elements > kSelRefine ? kWords : (int)(offsetof(SelState, pieces) / 4);
  const long long all = (long long)videos * words, step = (long long)gridDim.x * blockDim.x;
  for (long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x; j < all; j += step)
    reinterpret_cast<unsigned*>(st + j / words)[j % words] = 0;
}

// Adds w to hist[digit] for the lanes with valid set; every lane of the wavefront must call it. The two
// most frequent digits of the wavefront are combined before the atomic (real similarities sit in
// tight clusters, which would otherwise serialise on one LDS word); whatever is left goes through plain
// LDS atomics.
__device__ inline void wave_hist_add(unsigned* hist, bool valid, unsigned digit, unsigned w) {
  unsigned long long todo = __ballot(valid);
#pragma unroll 1
  for (int it = 0; it < 2 && todo; ++it) {
    const int leader = __ffsll((long long)todo) - 1;
    const unsigned d = __shfl(digit, leader, 64);
    const bool mine = valid && digit == d;
    const unsigned long long m = __ballot(mine);
    const unsigned sum = __popcll(__ballot(mine && (w & 1))) + 2u * __popcll(__ballot(mine && (w & 2)));
    if ((int)(threadIdx.x & 63) == leader) atomicAdd(&hist[d], sum);
    todo &= ~m;
  }
  if ((todo >> (threadIdx.x & 63)) & 1ull) atomicAdd(&hist[digit], w);
}

// Adds a workgroup's LDS histogram of bins to the state's (call after a barrier).
__device__ inline void sel_flush_bins(SelState* st, const unsigned* lds_hist) {
  unsigned* dst = st->hist0[blockIdx.x % kSelCopies];
  for (int j = threadIdx.x; j < kSelBins; j += blockDim.x)
    if (lds_hist[j]) atomicAdd(&dst[j], lds_hist[j]);
}

constexpr int kSelThreads = 256;

// Workgroup-wide (THREADS threads): the first bin of `hist` at which fd.acc + running weight exceeds the budget; fd.bin and
// fd.acc become that bin and the weight before it, `weight` its own, fd.rc 1 where the whole histogram fits. All threads get
// the same answer. The histogram is the sum of COPIES arrays of kSelBins counters. With `target` the budget is worked out
// here as well: the target less the base, which is base_const or, with a node map, the kept nodes of the video's first frame
// (fd.rc 2 where the base alone exceeds the target). The copies are requested at once, with whatever the caller has requested
// before. The base's cells are counted after that, a trip to memory for every THREADS of them, and the target is another: two
// trips for a spatial search, three or more for a temporal one.
template <int COPIES, int THREADS>
__device__ inline void sel_pick(const Geo& g, int b, const unsigned* __restrict__ hist, const int* __restrict__ target,
                                int base_const, const int32_t* __restrict__ node_map, SelFound& fd, unsigned& weight) {
  constexpr int WAVES = THREADS / kWave;
  static_assert(WAVES <= 16, "a row of lanes");
  __shared__ unsigned wsum[WAVES], wbase[WAVES];
  __shared__ unsigned s_digit, s_weight, s_acc;
  __shared__ int s_found;
  constexpr int PER = kSelBins / THREADS < 4 ? 4 : kSelBins / THREADS;  // (of more threads than pieces some have none)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  static_assert(PER % 4 == 0, "whole 16-byte pieces");
  unsigned h[PER], base = 0, tot = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) h[j] = 0;
  if (tid * PER < kSelBins) {
#pragma unroll
    for (int c = 0; c < COPIES; ++c)  // all loads at once
#pragma unroll
      for (int j = 0; j < PER; j += 4) {
        const uint4 v = *reinterpret_cast<const uint4*>(hist + c * kSelBins + tid * PER + j);
        h[j] += v.x; h[j + 1] += v.y; h[j + 2] += v.z; h[j + 3] += v.w;
      }
  }
  if (node_map) {
    for (int j = tid; j < g.HW; j += THREADS) {
      const int i = b * g.T * g.HW + j;
      base += (node_map[i] == i);
    }
  }
  const int want = target ? target[b] : 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) tot += h[j];
  const unsigned inc = wave_inclusive(tot, lane);
  if (node_map) base = wave_inclusive(base, lane);
  if (tid == 0) s_found = 0;
  if (lane == 63) {
    wsum[wave] = inc;
    wbase[wave] = base;
  }
  __syncthreads();
  const int sums = (int)row16_inclusive(lane < WAVES ? wsum[lane] : 0u, lane);
  if (target) {
    const int bases = (int)row16_inclusive(lane < WAVES ? wbase[lane] : 0u, lane);
    const long long budget = (long long)want - (node_map ? lane_value(bases, WAVES - 1) : base_const);
    fd.budget = budget < 0 ? 0ull : (unsigned long long)budget;
    fd.rc = budget < 0 ? 2 : 0;
  }
  if (fd.rc) return;  // uniform over the workgroup
  unsigned long long ex = fd.acc + (inc - tot) + (unsigned)(wave ? lane_value(sums, wave - 1) : 0);
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if (ex <= fd.budget && ex + h[j] > fd.budget) {
      s_found = 1;
      s_digit = (unsigned)(tid * PER + j);
      s_weight = h[j];
      s_acc = (unsigned)ex;
    }
    ex += h[j];
  }
  __syncthreads();
  fd.rc = s_found ? 0 : 1;
  fd.bin = s_digit;
  fd.acc = s_acc;
  weight = s_weight;
}

// What the bins are made from: the bits of a positive float that falls as the value rises.
__device__ inline unsigned sel_distance(uint32_t key) {
  return __float_as_uint(1.00006103515625f - key_float(key));  // (at least 2^-14: similarities are at most 1; key 0: a NaN)
}
__device__ inline unsigned sel_bin(uint32_t key) {
  return 2047u - (unsigned)min(max((int)(sel_distance(key) - 0x38800000u) >> 16, 0), 2047);
}
__device__ inline unsigned sel_piece(uint32_t key) {
  return 0x3fffffu - (unsigned)min(max((int)(sel_distance(key) - 0x38800000u) >> 5, 0), 0x3fffff);
}
// The distances in a bin: from sel_first up to, not with, sel_past (where the bins before it begin).
__device__ inline unsigned sel_first(unsigned bin) { return bin == 2047u ? 0u : 0x38800000u + ((2047u - bin) << 16); }
__device__ inline unsigned sel_past(unsigned bin) { return bin == 0u ? 0x7f800001u : 0x38800000u + ((2048u - bin) << 16); }

// A budget search that the kernel using its threshold carries out.
struct SelSearch {
  const SelState* states;  // [videos]; NULL: no search is pending
  const uint32_t* keys;    // [videos][per_video]: those of the picked bin's elements if they have been listed, else all
  const uint8_t* weights;  // (0 = not an element); weights of the elements (NULL = 1 each)
  int per_video;
  bool listed;             // (a small input is left to the consumer as it is: nothing has been picked yet)
  const int* target;       // [videos]
  int base_const;          // base of the step function: spatial = roots of all frames
  const int32_t* node_map; // temporal: the kept nodes of the video's first frame are counted here
};

// How a kernel comes by its threshold, which the host knows when it launches it: named by the caller or found by an earlier
// launch, by a search among listed elements, or by one that looks through all keys. Each is an instance of its own: with
// all three in one, k_temporal_parent of a frame of 169 cells was 12.8 KB of code and 90 registers, also where nothing was
// searched; now 1.9 KB and 13 registers, 7.9 and 27, 12.2 and 88.
enum { kTauKnown, kTauListed, kTauLook };
inline int tau_kind(const SelSearch& pending) { return !pending.states ? kTauKnown : pending.listed ? kTauListed : kTauLook; }
// f(kind), with the kind as a constant
template <class F>
inline void with_tau_kind(const SelSearch& pending, F f) {
  const int kind = tau_kind(pending);
  if (kind == kTauKnown) f(std::integral_constant<int, kTauKnown>());
  else if (kind == kTauListed) f(std::integral_constant<int, kTauListed>());
  else f(std::integral_constant<int, kTauLook>());
}

// Elements a search keeps in LDS; of more it reads the keys again in every round.
#ifndef STTM_SEL_LIST
#define STTM_SEL_LIST 4096
#endif
constexpr int kSelList = STTM_SEL_LIST;

// tau of video b, by a workgroup of THREADS threads (256 or more): midpoint between the searched key and the largest key below it.
// All threads get the value. Of a small input the right bin is picked here and its elements are taken from among all keys; of
// a large one they have been listed. Up to kSelFew of them are searched by one wavefront, each with each or bit by bit; else
// the range of keys is cut into 256 pieces, of which one is picked, until it is one key (two rounds for the elements of a bin,
// however many of them are equal).
// What bounds it: trips to memory (histogram and first keys are one, then the base's and the target's, see sel_pick), and
// instructions that are fetched for the first time, by time stamps of 64 frames of 13x13 in cycles: 1500 until the first
// requests are out, 3000 until they are answered, 2500 for the bin, 3000 for a look at 8192 keys, 600 to 5000 for the
// elements. So what is executed is kept short, and what the caller reads for its own work is requested before.
constexpr int kSelFew = kSelList < 256 ? kSelList : 256;
template <int THREADS, int KIND>
__device__ inline float sel_threshold(const Geo& g, const SelSearch& q, int b) {
  static_assert(KIND != kTauKnown, "a search");
  __shared__ uint32_t s_key[kSelList + kWave];  // (the last ones: where what is not in the bin goes)
  __shared__ uint8_t s_w[kSelList + kWave];
  constexpr int kPieces = 256, kBatch = 8;
  __shared__ unsigned hist[kPieces];
  __shared__ unsigned wsum[kPieces / 64];
  __shared__ unsigned s_lo, s_not_min, s_max, s_piece, s_acc;  // (s_not_min: the complement of the smallest key)
  __shared__ int s_count;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const Window keys = make_window(q.keys + (size_t)b * q.per_video, (unsigned)q.per_video * 4u);
  const Window weights = make_window(q.weights ? q.weights + (size_t)b * q.per_video : nullptr,
                                     q.weights ? (unsigned)q.per_video : 0u);
  const unsigned plain = q.weights ? 0u : 1u;
  // keys j0 + tid, j0 + tid + THREADS, ... (0 behind the last one) with their weights
  auto load = [&](uint32_t (&k)[kBatch], unsigned (&w)[kBatch], int j0) {
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      k[u] = (uint32_t)window_load_i32(keys, (unsigned)tid * 4u, (unsigned)(j0 + u * THREADS) * 4u);
      w[u] = (unsigned)window_load_u8(weights, (unsigned)tid, (unsigned)(j0 + u * THREADS)) + plain;
    }
  };
  if (tid == 0) {
    s_lo = s_not_min = s_max = 0;
    s_count = 0;
  }
  SelFound fd;
  int n = q.per_video;
  unsigned first = 0, past = 0;  // of all keys, the bin: what it makes of the values in it (see sel_first)
  if constexpr (KIND == kTauListed) {
    // (a list is short as a rule: the first keys are requested with its length)
    uint32_t key = (uint32_t)window_load_i32(keys, (unsigned)tid * 4u, 0u);
    unsigned weight = (unsigned)window_load_u8(weights, (unsigned)tid, 0u);
    fd = q.states[b].found[0];
    const unsigned long long acc = q.states[b].found[1].acc;
    if (fd.crowded) fd.acc = acc;
    const SelList l0 = q.states[b].list[0], l1 = q.states[b].list[1];
    n = min((int)(fd.list ? l1.count : l0.count), q.per_video);
    if (fd.rc) return fd.rc == 1 ? 1.f : -2.f;  // uniform over the workgroup
    __syncthreads();
    if (tid == 0) {
      s_lo = fd.list ? l1.lo : l0.lo;
      s_count = n;
    }
    // (the rest of a long one a batch at a time: of 3442 elements, one trip to memory after the other, k_temporal_parent of 512
    // frames of 13x13 took 13.1 us, so 11.5)
    const int held = min(n, kSelList);
    if (tid < held) {
      s_key[tid] = key;
      s_w[tid] = (uint8_t)weight;
    }
#pragma unroll 1
    for (int j0 = THREADS; j0 < held; j0 += kBatch * THREADS) {
      uint32_t k[kBatch];
      unsigned w[kBatch];
      load(k, w, j0);
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int j = j0 + u * THREADS + tid;
        if (j < held) {
          s_key[j] = k[u];
          s_w[j] = (uint8_t)w[u];
        }
      }
    }
  } else {
    // the first keys do not depend on the search: they are on their way while the bin is being found
    uint32_t k[kBatch];
    unsigned w[kBatch];
    load(k, w, 0);
    unsigned weight;
    fd.acc = 0;
    sel_pick<kSelCopies, THREADS>(g, b, q.states[b].hist0[0], q.target, q.base_const, q.node_map, fd, weight);
    if (fd.rc) return fd.rc == 1 ? 1.f : -2.f;
    first = sel_first(fd.bin);
    past = sel_past(fd.bin);
    // the picked bin's elements into LDS (no branches: they cost more than what they save); the largest key below the bin
    unsigned under = 0;
#pragma unroll 1
    for (int j0 = 0;;) {
      bool in[kBatch];
      int mine = 0;
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const unsigned t = sel_distance(k[u]);
        in[u] = (t - first < past - first) & (k[u] != 0);
        mine += in[u];
        under = max(under, t >= past ? k[u] : 0u);
      }
      const int upto = (int)wave_inclusive((unsigned)mine, lane), all = lane_value(upto, 63);
      int at = 0;
      if (lane == 0 && all) at = atomicAdd(&s_count, all);
      at = lane_value(at, 0) + upto - mine;
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int to = (in[u] & (at < kSelList)) ? at : kSelList + lane;
        s_key[to] = k[u];
        s_w[to] = (uint8_t)w[u];
        at += in[u];
      }
      j0 += kBatch * THREADS;
      if (j0 >= n) break;
      load(k, w, j0);
    }
    under = wave_max(under);
    if (lane == 0 && under) atomicMax(&s_lo, under);
  }
  __syncthreads();
  const int count = s_count;
  unsigned room = (unsigned)(fd.budget - fd.acc);  // weight that still fits before the searched key
  unsigned a, under;                               // that key: the largest one with no more than that before it; the one below
  if (count <= kSelFew) {
    if (wave == 0) {
      if (count <= kWave) {  // each with each
        const unsigned own = lane < count ? s_key[lane] : 0u, weight = lane < count ? s_w[lane] : 0u;
        unsigned before = 0, equal = 0, below = 0;
#pragma unroll 1
        for (int j = 0; j < count; ++j) {
          const unsigned kj = (unsigned)lane_value((int)own, j), wj = (unsigned)lane_value((int)weight, j);
          before += kj < own ? wj : 0u;
          equal += kj == own ? wj : 0u;
          below = max(below, kj < own ? kj : 0u);
        }
        if (before <= room && before + equal > room) {  // (whoever holds this key has found the same)
          s_piece = own;
          s_max = below;
        }
      } else {  // the searched key's distance from the smallest one, bit by bit
        constexpr int kPer = (kSelFew + kWave - 1) / kWave;
        uint32_t k[kPer];
        unsigned w[kPer], kmin = 0xffffffffu, kmax = 0, below = 0, d = 0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
          const int j = u * kWave + lane;
          k[u] = j < count ? s_key[j] : 0xffffffffu;
          w[u] = j < count ? s_w[j] : 0u;
          kmin = min(kmin, k[u]);
          kmax = max(kmax, j < count ? k[u] : 0u);
        }
        kmin = ~wave_max(~kmin);
        kmax = wave_max(kmax);
#pragma unroll 1
        for (int bit = kmax == kmin ? -1 : 31 - __builtin_clz(kmax - kmin); bit >= 0; --bit) {
          const unsigned at = kmin + (d | 1u << bit);
          unsigned before = 0;
#pragma unroll
          for (int u = 0; u < kPer; ++u) before += k[u] < at ? w[u] : 0u;
          if ((unsigned)lane_value((int)wave_inclusive(before, lane), 63) <= room) d |= 1u << bit;
        }
        a = kmin + d;
#pragma unroll
        for (int u = 0; u < kPer; ++u) below = max(below, k[u] < a ? k[u] : 0u);
        below = wave_max(below);
        if (lane == 0) {
          s_piece = a;
          s_max = below;
        }
      }
    }
    __syncthreads();
    a = s_piece;
    under = max(s_max, s_lo);
  } else {
    const bool kept = count <= kSelList;
    auto read = [&](auto use) {  // (of all keys those of the bin)
      if (kept) {
#pragma unroll 1
        for (int j = tid; j < count; j += THREADS) use(s_key[j], (unsigned)s_w[j]);
      } else {
#pragma unroll 1
        for (int j0 = 0; j0 < n; j0 += kBatch * THREADS) {
          uint32_t k[kBatch];
          unsigned w[kBatch];
          load(k, w, j0);
#pragma unroll
          for (int u = 0; u < kBatch; ++u)
            if (j0 + u * THREADS + tid < n && (KIND == kTauListed || (k[u] && sel_distance(k[u]) - first < past - first)))
              use(k[u], w[u]);
        }
      }
    };
    unsigned not_min = 0, kmax = 0;
    read([&](uint32_t key, unsigned) {
      not_min = max(not_min, ~key);
      kmax = max(kmax, key);
    });
    not_min = wave_max(not_min);
    kmax = wave_max(kmax);
    if (lane == 0) {
      atomicMax(&s_not_min, not_min);
      atomicMax(&s_max, kmax);
    }
    __syncthreads();
    a = ~s_not_min;
    unsigned z = s_max;
#pragma unroll 1
    while (a != z) {
      const int shift = max(0, 24 - __builtin_clz(z - a));
      if (tid < kPieces) hist[tid] = 0;
      __syncthreads();
      read([&](uint32_t key, unsigned weight) {
        if (key >= a && key <= z) atomicAdd(&hist[(key - a) >> shift], weight);
      });
      __syncthreads();
      const unsigned h = tid < kPieces ? hist[tid] : 0u, inc = wave_inclusive(h, lane);
      if (lane == 63 && tid < kPieces) wsum[wave] = inc;
      __syncthreads();
      unsigned ex = inc - h;
      for (int v = 0; v < min(wave, kPieces / 64); ++v) ex += wsum[v];
      if (ex <= room && ex + h > room) {
        s_piece = (unsigned)tid;
        s_acc = ex;
      }
      __syncthreads();
      a += s_piece << shift;
      z = min(z, a + ((1u << shift) - 1u));
      room -= s_acc;
    }
    // (an element may still lie below the searched key in its bin)
    under = 0;
    read([&](uint32_t key, unsigned) {
      if (key < a) under = max(under, key);
    });
    under = wave_max(under);
    if (lane == 0 && under) atomicMax(&s_lo, under);
    __syncthreads();
    under = s_lo;
  }
  const float hi = key_float(a);
  const float lof = under ? key_float(under) : -2.f;
  float t = 0.5f * (lof + hi);
  if (!(t < hi)) t = lof;
  return t;
}

// ---- launchers (defined in the .hip files; all asynchronous on `s`) ------------------------------------

// `sel`: the spatial search states [B]; cleared by the statistics pass, the histogram filled by the finalize kernel.
// `pairs`: also leave S_n(t) . S_n(t+1) of every cell, 2x2 and 4x4 block n in `part` (the temporal stage then skips those).
void launch_pyramid_stats(const Geo& g, const void* feats, bool pairs, float* part, float* nsum, SelState* sel,
                          hipStream_t s);
// The counters of the temporal pass's work queues. They are empty when the pass begins: the spatial stage clears them, and
// so does the pass itself when it is over. (Not by a memset when a shape is bound: one recorded into a graph has given
// wrong results on replays, and a graph recorded later would count on memory that another shape may have used since.)
constexpr int kTQueues = 64;
constexpr int kTCountStride = 32;  // ints between two queues' counters: a 128-byte line each
__device__ inline void temporal_clear(int* item_count, int tid) {
  if (tid < kTQueues) item_count[tid * kTCountStride] = 0;
}
// Thresholds a caller has named, handed to the kernels that use them as a launch argument (n = 0: none). A copy from the
// caller's memory to the device is a stream operation of its own: 2.5-5 us there and about as much on the host.
constexpr int kTauArgs = 32;
struct TauArgs {
  int n;
  float v[kTauArgs];
};
// The decision about the partition, where it is made with the statistics: from the thresholds in `given` (which are left in `tau`
// for later readers) or, if there are none, from those in `tau`. node_map NULL: not made.
struct DecideArgs {
  TauArgs given;
  float* tau;
  int32_t* node_map;
  uint8_t* node_level;
};
// Also works out the levels above an 8x8 unit from the stored unit sums (extends `nsum`).
void launch_spatial_finalize(const Geo& g, const float* part, float* nsum, float* nrm2, float* sim, float* m,
                             uint32_t* sel_key, uint8_t* sel_w, SelState* sel, int* item_count, const DecideArgs& decide,
                             hipStream_t s);
// `pending`: a budget search that has not been carried out yet (or states == NULL); the kernel then works the threshold out
// itself (and leaves it in `tau` for later readers) instead of reading `tau`.
void launch_spatial_decide(const Geo& g, const float* m, float* tau, const SelSearch& pending, int32_t* node_map,
                           uint8_t* node_level, hipStream_t s);
// Begins a budget search and says how it goes on. A small input is left to whoever uses the threshold; of a large one the
// elements of the right bin are listed (`list_key`, `list_w`: [videos][select_elements()]). `handed_back`: launch_select_tau
// will carry it out.
SelSearch launch_select_spatial(const Geo& g, const uint32_t* keys, const uint8_t* weights, const int* target,
                                SelState* state, uint32_t* list_key, uint8_t* list_w, bool handed_back, hipStream_t s);
SelSearch launch_select_temporal(const Geo& g, const int32_t* node_map, const uint32_t* keys, const int* target,
                                 SelState* state, uint32_t* list_key, uint8_t* list_w, bool handed_back,
                                 hipStream_t s);
// Carries a search out now, for a caller who wants the thresholds back.
// `host_tau` (may be NULL): host memory the device can write, which receives the thresholds as well.
void launch_select_tau(const Geo& g, const SelSearch& search, float* tau, float* host_tau, hipStream_t s);
// Elements per video of a spatial / temporal search: what its list has room for.
int select_elements(const Geo& g, bool spatial);
inline size_t select_state_bytes(int B) { return (size_t)B * sizeof(SelState); }
// `sel`: the temporal search states [B]; cleared here, the histogram filled by launch_temporal_resolve.
// `skip_same`: pairs of the same cell, 2x2 or 4x4 block in both frames are left out (their dot products are in the
// spatial pass's `part`).
// `items` (temporal_items_bytes() of them) / `item_count`: the work queues of the pass (see temporal_clear).
void launch_temporal_dots(const Geo& g, const void* feats, const uint8_t* node_level, const float* nsum,
                          bool skip_same, float* pd_part, SelState* sel, void* items, int* item_count,
                          hipStream_t s);
size_t temporal_items_bytes(const Geo& g);
size_t temporal_count_bytes();
// The first pass works in 8x8-cell units (one workgroup per unit and chunk) and leaves each unit's scalars
// as one block of kUnitScalars floats: per 4x4 tile 16 squared norms, 16 cell and 4 level-1 dot products, then the
// 4 level-2 dot products (padded to whole 128-byte lines), then per tile the 16 dot products of its cells with the
// same cells of the next frame, then per tile the dot products of its four 2x2 blocks and of the tile itself with the
// same blocks of the next frame (zeros where those products are not formed): part[f][chunk][unit][kUnitScalars].
constexpr int kUnitScalars = 256;
constexpr int kUnitCellDots = 160;
constexpr int kUnitNodeDots = 224;
// Offset of cell (y, x)'s cell-to-cell dot product inside its unit's block.
inline __host__ __device__ int unit_cell_dot_slot(int y, int x) {
  return kUnitCellDots + (((y >> 2) & 1) * 2 + ((x >> 2) & 1)) * 16 + (((y >> 1) & 1) * 2 + ((x >> 1) & 1)) * 4 +
         (y & 1) * 2 + (x & 1);
}
// Offset of the frame-to-frame dot product of the node at level 1 or 2 whose top-left cell is (y, x).
inline __host__ __device__ int unit_node_dot_slot(int lvl, int y, int x) {
  return kUnitNodeDots + (((y >> 2) & 1) * 2 + ((x >> 2) & 1)) * 8 + (lvl == 2 ? 4 : ((y >> 1) & 1) * 2 + ((x >> 1) & 1));
}
inline __host__ __device__ int unit_cols(const Geo& g) { return (g.W + 7) >> 3; }
inline __host__ __device__ int unit_rows(const Geo& g) { return (g.H + 7) >> 3; }
// fp32 sums of the pyramid nodes at levels >= 3: [F][nsum_nodes][D]
inline size_t nsum_nodes(const Geo& g) { return g.L >= 3 ? (size_t)(g.NN - g.lvl_base[3]) : 0; }
// `match`: destination rule (0 = top-left-most passing, 1 = the one under the top-left cell only, 2 = most similar).
// `cell_part`: the spatial pass's `part` when it holds frame-to-frame dot products (else NULL).
void launch_temporal_resolve(const Geo& g, int match, const int32_t* node_map, const uint8_t* node_level,
                             const float* pd_part, const float* cell_part, const float* nrm2, float* sig, float* e,
                             uint32_t* sel_key, SelState* sel, int* item_count, hipStream_t s);
// `given`: if it holds thresholds the kernel takes them from there (and leaves them in `tau` for later readers); `pending` as
// above.
void launch_temporal_parent(const Geo& g, int match, const int32_t* node_map, const uint8_t* node_level,
                            const float* sig, float* tau, const TauArgs& given, const SelSearch& pending, int32_t* parent,
                            int32_t* ptr, hipStream_t s);
void launch_roots(const Geo& g, int32_t* ptr_a, int32_t* ptr_b, const int32_t* node_map, int32_t* cluster_ids,
                  hipStream_t s);
void launch_node_levels(const Geo& g, const int32_t* node_map, uint8_t* node_level, hipStream_t s);

struct ReduceBuffers {
  int32_t* rank;        // [N]   exclusive count of roots before every cell
  int32_t* key;         // [N] keys of the cells, for the first pass
  uint2* pair_a;        // [N] (key, cell): sort ping; `key` is its first half
  uint2* pair_b;        // [N] sort pong
  uint2* list;          // [N] the sorted elements: (cell, output row)
  int32_t* hist;        // [tiles][digits] radix histogram of the running pass
  int32_t* tot;         // [digits] column totals (very large inputs)
  int32_t* gsum;        // [groups of tiles][digits] partial column sums (medium inputs)
  int32_t* tile_roots;  // [tiles]
  int32_t* seg;         // [N+1] first list position of every output row
  int32_t* kdev;        // [4] number of clusters, length of the live list, length of the big-cluster list
  int32_t* zpos;        // [N] output row of every cluster rank under the Z-shaped scan
  int32_t* host_k;      // host memory the device can write, receives the number of clusters (or NULL)
  int32_t* biglist;     // [big clusters][4] output row, first list position, end of the list, unused
  float* bigpart;       // [gather items][2][D] partial sums of clusters with more than 64 list slots
  int32_t* bigw;        // [gather items][2] member cells behind those partial sums
};
// node_map / node_level: the stage-1 partition, or both NULL (every cell is its own list element).
void launch_reduce_prepare(const Geo& g, const int32_t* cluster_ids, const int32_t* node_map,
                           const uint8_t* node_level, int64_t capacity, int32_t* out_ids, int64_t* offsets,
                           const ReduceBuffers& rb, bool zscan, hipStream_t s);
void launch_reduce_gather(const Geo& g, const void* feats, const float* nsum, const int32_t* node_map,
                          const uint8_t* node_level, int out_dtype, int64_t capacity, void* merged, int32_t* counts,
                          const ReduceBuffers& rb, bool zscan, hipStream_t s);
void launch_reduce_big(const Geo& g, const void* feats, const float* nsum, const int32_t* node_map,
                       const uint8_t* node_level, int out_dtype, int64_t capacity, void* merged, int32_t* counts,
                       const ReduceBuffers& rb, bool zscan, hipStream_t s);
// Position indices of the rows of the reduce call that has just run (its list, ranks and row map are still in `rb`).
void launch_positions(const Geo& g, const int32_t* cluster_ids, const int32_t* node_map, const uint8_t* node_level,
                      const int64_t* offsets,
                      int64_t capacity, const ReduceBuffers& rb, bool zscan, unsigned long long* possum,
                      unsigned* poscnt, int32_t* survived, int32_t* reassigned, float* merged_pos,
                      int32_t* root_tyxl, hipStream_t s);
size_t reduce_bigpart_floats(const Geo& g);
size_t reduce_bigw_entries(const Geo& g);
bool reduce_io_supported(int in_dtype, int out_dtype);
size_t reduce_biglist_entries(const Geo& g);
size_t reduce_hist_entries(int N);
size_t reduce_tiles(int N);
size_t reduce_gsum_entries();

}  // namespace sttm
