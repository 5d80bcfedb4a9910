// rmdf_wave.h - wavefront-level helpers shared by the per-pixel kernels: DPP
// lane exchanges within rows of 16 lanes, lane reads, and reductions over a
// group of 32 or 64 lanes of one wavefront that stay off the LDS permute path
// (a chain of ds_bpermute costs an LDS round trip per level; DPP operands
// come from the neighbouring lanes' registers).
#pragma once
#include <hip/hip_runtime.h>

namespace rmdf {

// LDS pointers keep their address space so every access is a ds_* instruction
// with an immediate offset (a generic pointer would become a flat access)
#define RMDF_LDS __attribute__((address_space(3)))
#define RMDF_GLOBAL __attribute__((address_space(1)))
typedef float v2f __attribute__((ext_vector_type(2)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef RMDF_LDS v2f lds_v2;
typedef RMDF_LDS v4f lds_v4;
typedef RMDF_LDS float lds_float;
typedef RMDF_LDS unsigned int lds_u32;
__device__ __forceinline__ float2 ld2(const lds_v2* p) { const v2f v = *p; return make_float2(v.x, v.y); }
__device__ __forceinline__ float4 ld4(const lds_v2* p) {
  const v4f v = *reinterpret_cast<const lds_v4*>(p);
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st2(lds_v2* p, float2 v) { *p = v2f{v.x, v.y}; }
__device__ __forceinline__ void st4(lds_v2* p, float a, float b, float c, float d) {
  *reinterpret_cast<lds_v4*>(p) = v4f{a, b, c, d};
}

// Element at a byte offset from a base that is the same in all lanes: a 32-bit
// offset per lane instead of a 64-bit address.
template <class T>
static __device__ __forceinline__ const T& at(const T* base, unsigned bytes) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + bytes);
}
template <class T>
static __device__ __forceinline__ T& at(T* base, unsigned bytes) {
  return *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + bytes);
}

// Element at a byte offset from an LDS address
static __device__ __forceinline__ lds_v2* lds_at(lds_v2* base, unsigned bytes) {
  return (lds_v2*)((RMDF_LDS char*)base + bytes);
}

// A pointer and an int that all lanes share although the compiler cannot see it
// (arguments of a function that is called, not inlined): held in scalar registers.
template <class T>
static __device__ __forceinline__ T* uniform(T* p) {
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32));
  return reinterpret_cast<T*>((unsigned long long)hi << 32 | lo);
}
static __device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Buffer descriptor of `bytes` bytes at p (the same in all lanes).  Reads past it
// give 0 and writes past it are dropped, so lanes past the end of a run need
// neither a mask nor a clamped index; BUFFER_NONE (with a small constant added)
// lies past every run.  Word 3: untyped 32-bit data.
typedef __amdgpu_buffer_rsrc_t buffer_rsrc;
static __device__ __forceinline__ buffer_rsrc buffer_of(void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00027000);
}
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
static __device__ __forceinline__ float uf(unsigned v) { return __int_as_float((int)v); }
static __device__ __forceinline__ unsigned fu(float v) { return (unsigned)__float_as_int(v); }
static __device__ __forceinline__ float buffer_ld(buffer_rsrc b, unsigned off) {
  return uf(__builtin_amdgcn_raw_buffer_load_b32(b, (int)off, 0, 0));
}
static __device__ __forceinline__ void buffer_st(buffer_rsrc b, float v, unsigned off) {
  __builtin_amdgcn_raw_buffer_store_b32(fu(v), b, (int)off, 0, 0);
}
// (8 and 16 bytes: the observer state, streamed once per frame; non-temporal at every
// size, which takes 2 to 4% off a frame whose state exceeds the chip's last cache, alone
// or with the streams it takes turns with, and costs a lone smaller stream up to 13%:
// the figures are at the generic tile's state accesses)
constexpr int BUFFER_NT = 2;
static __device__ __forceinline__ void buffer_ld(buffer_rsrc b, unsigned off, float2 (&v)[1]) {
  const v2u q = __builtin_amdgcn_raw_buffer_load_b64(b, (int)off, 0, BUFFER_NT);
  v[0] = make_float2(uf(q.x), uf(q.y));
}
static __device__ __forceinline__ void buffer_ld(buffer_rsrc b, unsigned off, float2 (&v)[2]) {
  const v4u q = __builtin_amdgcn_raw_buffer_load_b128(b, (int)off, 0, BUFFER_NT);
  v[0] = make_float2(uf(q.x), uf(q.y));
  v[1] = make_float2(uf(q.z), uf(q.w));
}
static __device__ __forceinline__ void buffer_st(buffer_rsrc b, const float2 (&v)[1], unsigned off) {
  __builtin_amdgcn_raw_buffer_store_b64(v2u{fu(v[0].x), fu(v[0].y)}, b, (int)off, 0, BUFFER_NT);
}
static __device__ __forceinline__ void buffer_st(buffer_rsrc b, const float2 (&v)[2], unsigned off) {
  __builtin_amdgcn_raw_buffer_store_b128(v4u{fu(v[0].x), fu(v[0].y), fu(v[1].x), fu(v[1].y)}, b, (int)off, 0, BUFFER_NT);
}
constexpr unsigned BUFFER_NONE = 0x40000000u;

// The value is computed here, and memory accesses are not moved across (no
// instruction): without it the compiler sinks a pass's arithmetic below the next
// pass's loads and holds both in registers.
static __device__ __forceinline__ void pass_done(float2& v) { asm volatile("" : "+v"(v.x), "+v"(v.y)::"memory"); }

// Orders this wavefront's LDS accesses (lanes of one wavefront exchange
// through LDS without a workgroup barrier).
static __device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// (bound_ctrl: every lane has a source in the patterns below, so no lane needs
// its old value, and the move folds into the instruction that uses it)
template <int CTRL>
static __device__ __forceinline__ float dppf(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
static __device__ __forceinline__ int dppi(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
// row_ror:n -> dst[i] = src[(i - n) mod 16] within each row of 16 lanes;
// row_mirror -> dst[i] = src[15 - i]; quad_perm [1,0,3,2] and [2,3,0,1] ->
// dst[i] = src[i ^ 1] and src[i ^ 2]
constexpr int ROR1 = 0x121, ROR4 = 0x124, ROR8 = 0x128, ROR15 = 0x12F, MIRROR = 0x140, QXOR1 = 0xB1,
              QXOR2 = 0x4E;

static __device__ __forceinline__ float lane_read(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// (value, index) argmax with the first (lowest-index) maximum winning: a
// maximum over a total order, so the shape of a reduction built from it does
// not change its result.
static __device__ __forceinline__ void amax_merge(float& v, int& i, float v2, int i2) {
  const bool take = (v2 > v) | ((v2 == v) & (i2 < i));
  v = take ? v2 : v;
  i = take ? i2 : i;
}

// Reductions over groups of G lanes (G = 32: lanes 0-31 and 32-63 are two
// groups; G = 64: the whole wavefront): within each row of 16 lanes by DPP
// (partners lane ^ 1, lane ^ 2, then rotations by 4 and 8, after which every
// lane holds its row's result), then the rows' results read from lanes 0,
// 16, 32 and 48 and combined per group.  The result is the same in every lane
// of a group.  Every lane of the wavefront must be active.
template <int G>
static __device__ __forceinline__ float group_sum(float v) {
  static_assert(G == 32 || G == 64, "groups of 32 or 64 lanes");
  v += dppf<QXOR1>(v);
  v += dppf<QXOR2>(v);
  v += dppf<ROR4>(v);
  v += dppf<ROR8>(v);
  const float r0 = lane_read(v, 0), r1 = lane_read(v, 16), r2 = lane_read(v, 32), r3 = lane_read(v, 48);
  if (G == 64) return (r0 + r1) + (r2 + r3);
  return (threadIdx.x & 32) ? r2 + r3 : r0 + r1;
}

template <int G>
static __device__ __forceinline__ float group_max(float v) {
  static_assert(G == 32 || G == 64, "groups of 32 or 64 lanes");
  v = fmaxf(v, dppf<QXOR1>(v));
  v = fmaxf(v, dppf<QXOR2>(v));
  v = fmaxf(v, dppf<ROR4>(v));
  v = fmaxf(v, dppf<ROR8>(v));
  const float r0 = lane_read(v, 0), r1 = lane_read(v, 16), r2 = lane_read(v, 32), r3 = lane_read(v, 48);
  if (G == 64) return fmaxf(fmaxf(r0, r1), fmaxf(r2, r3));
  return (threadIdx.x & 32) ? fmaxf(r2, r3) : fmaxf(r0, r1);
}

// group minimum or maximum of an int (the comparison folds the DPP move)
template <int G, bool MAX>
static __device__ __forceinline__ int group_ext(int v) {
  static_assert(G == 32 || G == 64, "groups of 32 or 64 lanes");
  auto ext = [](int a, int b) { return MAX ? max(a, b) : min(a, b); };
  v = ext(v, dppi<QXOR1>(v));
  v = ext(v, dppi<QXOR2>(v));
  v = ext(v, dppi<ROR4>(v));
  v = ext(v, dppi<ROR8>(v));
  const int r0 = __builtin_amdgcn_readlane(v, 0), r1 = __builtin_amdgcn_readlane(v, 16);
  const int r2 = __builtin_amdgcn_readlane(v, 32), r3 = __builtin_amdgcn_readlane(v, 48);
  if (G == 64) return ext(ext(r0, r1), ext(r2, r3));
  return (threadIdx.x & 32) ? ext(r2, r3) : ext(r0, r1);
}
// an order-preserving map of float bits to int and back (its own inverse)
static __device__ __forceinline__ int order_key(int b) { return b ^ ((b >> 31) & 0x7fffffff); }

// The group's maximum v (never NaN: running maxima that began at -infinity)
// and the lowest i that holds it: the maximum first, as an integer key (one DPP
// instruction per level; a float maximum would quiet its operands first), then the
// index from the one lane that equals it, or the lowest where several do.
template <int G>
static __device__ __forceinline__ void group_amax(float& v, int& i) {
  const float m = __int_as_float(order_key(group_ext<G, true>(order_key(__float_as_int(v)))));
  const unsigned long long hold = __ballot(v == m);
  const unsigned lo = (unsigned)hold, hi = (unsigned)(hold >> 32);
  if (G == 64) {
    if ((hold & (hold - 1)) == 0) i = __builtin_amdgcn_readlane(i, __builtin_ctzll(hold));
    else i = group_ext<G, false>(v == m ? i : 0x7fffffff);
  } else {
    if ((lo & (lo - 1)) == 0 && (hi & (hi - 1)) == 0) {
      const int a = __builtin_amdgcn_readlane(i, __builtin_ctz(lo)), b = __builtin_amdgcn_readlane(i, 32 + __builtin_ctz(hi));
      i = (threadIdx.x & 32) ? b : a;
    } else {
      i = group_ext<G, false>(v == m ? i : 0x7fffffff);
    }
  }
  v = m;
}

}  // namespace rmdf
