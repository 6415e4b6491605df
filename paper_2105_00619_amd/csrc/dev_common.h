// Device-side helpers shared by the HIP kernels: storage types, conversions, vector loads.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fastdiv.h"
#include "kernels.h"
#include "launch.h"

namespace oseq {

typedef _Float16 f16_t;
typedef __bf16 bf16_t;

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(f16_t v) { return (float)v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return (float)v; }

template <class T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ f16_t from_f32<f16_t>(float v) { return (f16_t)v; }    // round to nearest even
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v) { return (bf16_t)v; }  // round to nearest even

// Two floats rounded (to nearest even) into a pair of 16-bit values in one register: one packed conversion instead of
// two conversions and a merge.
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
template <class T> struct Pair16;
template <> struct Pair16<f16_t> { typedef __attribute__((ext_vector_type(2))) _Float16 V; };
template <> struct Pair16<bf16_t> { typedef __attribute__((ext_vector_type(2))) __bf16 V; };
template <class T> __device__ __forceinline__ typename Pair16<T>::V from_f32x2(float a, float b) {
  const f32x2_t v = {a, b};
  return __builtin_convertvector(v, typename Pair16<T>::V);
}

// sum of the two products of a pair of 16-bit values, added to c in fp32 (one instruction)
template <class T> struct Dot2;
template <> struct Dot2<bf16_t> {
  typedef __attribute__((ext_vector_type(2))) __bf16 V;
  __device__ static __forceinline__ float run(V a, V b, float c) { return __builtin_amdgcn_fdot2_f32_bf16(a, b, c, false); }
};
template <> struct Dot2<f16_t> {
  typedef __attribute__((ext_vector_type(2))) _Float16 V;
  __device__ static __forceinline__ float run(V a, V b, float c) { return __builtin_amdgcn_fdot2(a, b, c, false); }
};

// V consecutive elements of T, loaded and stored as one access.
template <class T, int V>
struct alignas(sizeof(T) * V) Vec {
  T v[V];
};

// the same as a streaming (non-temporal) load where the V elements are 16 bytes
template <class T, int V>
__device__ __forceinline__ void load_f32_nt(const T* p, float (&out)[V]) {
  if constexpr (sizeof(T) * V == 16) {
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
    const u32x4 c = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    const Vec<T, V> t = __builtin_bit_cast(Vec<T, V>, c);
#pragma unroll
    for (int i = 0; i < V; ++i) out[i] = to_f32(t.v[i]);
  } else {
    Vec<T, V> t = *reinterpret_cast<const Vec<T, V>*>(p);
#pragma unroll
    for (int i = 0; i < V; ++i) out[i] = to_f32(t.v[i]);
  }
}
template <class T, int V>
__device__ __forceinline__ void load_f32(const T* p, float (&out)[V]) {
  Vec<T, V> t = *reinterpret_cast<const Vec<T, V>*>(p);
#pragma unroll
  for (int i = 0; i < V; ++i) out[i] = to_f32(t.v[i]);
}
// V floats rounded to T (16-bit types: pairwise, one packed conversion per pair)
template <class T, int V>
__device__ __forceinline__ Vec<T, V> round_vec(const float (&in)[V]) {
  Vec<T, V> t;
  if constexpr (sizeof(T) == 2 && V % 2 == 0) {
#pragma unroll
    for (int i = 0; i < V; i += 2) {
      const typename Pair16<T>::V q = from_f32x2<T>(in[i], in[i + 1]);
      t.v[i] = q[0]; t.v[i + 1] = q[1];
    }
  } else {
#pragma unroll
    for (int i = 0; i < V; ++i) t.v[i] = from_f32<T>(in[i]);
  }
  return t;
}
template <class T, int V>
__device__ __forceinline__ void store_f32(T* p, const float (&in)[V]) {
  *reinterpret_cast<Vec<T, V>*>(p) = round_vec<T, V>(in);
}

// 16 bytes held in registers between a global load and an LDS store (a plain vector type: arrays of it stay in
// registers across loop back-edges)
typedef __attribute__((ext_vector_type(4))) uint32_t Chunk;
__device__ __forceinline__ Chunk zero_chunk() { Chunk c = {0u, 0u, 0u, 0u}; return c; }

// The BatchNorm affine map; the same instruction sequence in forward and backward so that the
// ReLU mask rebuilt in backward equals the one applied in forward, bit for bit.
__device__ __forceinline__ float bn_affine(float z, float scale, float shift) { return __fmaf_rn(z, scale, shift); }

// The start of a training step, by one whole block before anything else of the step runs: flags[0] = a gradient is not finite
// (set by the optimizer's check), flags[1] = a label lies outside [0, classes).  Either flag makes the update a no-op, and
// flags[1] also keeps the BatchNorm running statistics as they were.  Stream order makes the flags visible to the later kernels.
__device__ __forceinline__ void step_begin(const StepBegin& b) {
  bool bad = false;
  for (int i = threadIdx.x; i < b.n; i += blockDim.x) bad |= b.y[i] < 0 || b.y[i] >= b.classes;
  const int any = __syncthreads_or(bad);
  if (threadIdx.x < 4) b.flags[threadIdx.x] = threadIdx.x == 1 ? (any ? 1 : 0) : 0;
}

// Two transposing 64-bit LDS reads (ds_read_b64_tr_b16).  Within a group of 16 lanes every lane supplies the address
// of 4 consecutive 16-bit elements, and lane l receives element l%4 of the addresses supplied by lanes l/4, l/4 + 4,
// l/4 + 8, l/4 + 12.  With lane r addressing channels [4*(r%4), +4) of row r/4 (of four rows), lane l therefore ends
// up with channel l of the 16 at those four rows.  p0 / p1 address the first / second group of four rows, so the
// result holds 8 consecutive reduction elements (pixels) of one channel: an MFMA operand of type V.
template <class V, class E>
__device__ __forceinline__ V lds_tr_read8(const E* p0, const E* p1) {
  typedef __attribute__((ext_vector_type(4))) short v4s;
  typedef __attribute__((ext_vector_type(8))) short v8s;
  const v4s a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(p0));
  const v4s b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(p1));
  const v8s r = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(V, r);
}

inline int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

}  // namespace oseq
