// Implicit-GEMM convolution on the matrix cores (MFMA 32x32, fp32 accumulate; fp32 operands as three bf16 planes) for gfx950.
//
// Forward and data gradient share one kernel: out[m][n] = sum_kk A[m][kk] * B[n][kk], where
//   m  = output pixel (image, row, col),      n = output channel of this GEMM,
//   kk = (tap r, tap s, source channel) with the source channel fastest,
//   A  is gathered on the fly from the NHWC source tensor (im2col tile staged in LDS, zero outside the image),
//   B  is a [n][R*S*C_src] matrix: the (C_out,kh,kw,C_in) weights for forward, their (C_in,kh,kw,C_out)
//      transpose for the data gradient.
// Forward gathers x[n, p*stride + r - pad, q*stride + s - pad, :]; the data gradient gathers
// dz[n, (h + pad - r)/stride, (w + pad - s)/stride, :] where the division is exact.
// The weight gradient is the transposed problem (reduction over pixels) and has its own kernel.
//
// Tiling: 256 threads = 4 wavefronts of 64 lanes in a 2x2 grid; block tile 128 x BN (BN = 128 or 64), depth BK of
// 64 bytes per row (16 fp32 / 32 half elements, so one depth tile never straddles a filter tap when C_src % BK == 0).
// Each lane keeps 32 bytes of every operand row per depth tile; global loads for tile t+1 are issued before the
// MFMAs of tile t (register prefetch + two LDS buffers, one barrier per tile).
#include <algorithm>
#include <type_traits>

#include "bn_fold.h"
#include "dev_common.h"
#include "epilogue.h"
#include "kernels.h"
#include "patch.h"
#include "split32.h"

namespace oseq {

typedef __attribute__((ext_vector_type(16))) float v16f;
typedef __attribute__((ext_vector_type(8))) __bf16 v8bf;
typedef __attribute__((ext_vector_type(8))) _Float16 v8h;
typedef __attribute__((ext_vector_type(4))) float v4f;

// 16 bytes in flight between global memory and LDS: a first-class vector value, never a stack object

enum { IG_FWD = 0, IG_DGRAD = 1, IG_EVAL = 2 };  // IG_EVAL: forward with the inference-mode BatchNorm in the epilogue

struct IGemmArgs {
  int srcH, srcW, srcC;   // gathered tensor
  int dstH, dstW;         // pixel grid of the result
  int M, Ng, Kg;          // GEMM sizes: rows (pixels), columns (channels), depth (R*S*srcC)
  int R, S, stride, pad, relu;
  int kt_per_split;       // depth tiles per blockIdx.z when the depth is split
  // Data gradient of a stride-2 convolution by parity classes (cls = 1): blockIdx.z is the class (ph, pw) of the
  // output pixel (h, w) = (2*hh + ph, 2*ww + pw); only the taps with (ph + pad - r) and (pw + pad - s) even reach
  // that class, so each class is its own GEMM over its tap list.  dstH / dstW are then the class grid (fullH/2,
  // fullW/2), M its pixel count, taps[c] the list (one byte per tap, r*S + s), ntaps[c] its length.
  int cls, fullH, fullW;
  int taps[4], ntaps[4];
  const uint8_t* amask;   // data gradient with an addend: ReLU bit mask the addend is multiplied by, or null
};

// How operands lie in LDS and the MFMAs that consume them.  E: staged element; BK: depth of a tile; PITCH: staged elements
// per operand row: BK values (Split32: the three bf16 planes of BK values one after the other) and 16 bytes that spread the rows
// over the banks, 80 bytes (Split32: 112).  put: 16 bytes of the tensor, the piece `v` of a row, to LDS.
// A lane holds BK / 2 of a row's values; they are used up in PHASES groups of MFMAs (steps(ph) each), after each of which
// the registers that it was the last to read are loaded with the next tile's (load(ph)).
// ACCS: accumulators per output; depth tile i goes to number i % ACCS.  Split32 has two: the 16-bit MFMA drops what lies eight
// or more bits below the last one of its largest term, towards minus infinity, so that a sum of 400 MFMAs is too low by 6e-8 of
// the results' deviation -- a tenth of its error, but the same for every pixel, so that a sum over pixels behind it keeps it.  The
// second accumulator takes its tiles with the weights negated and is subtracted in the end (6e-9 left of nine taps; a 3x3 layer of
// 128 channels is off by 3.6e-7 of its deviation that way, 5.1e-7 with one accumulator, 6.0e-7 on the fp32 MFMA).
// X: the operands' form: the storage type itself, or for fp32 Split32: the 16-bit MFMAs (split32.h).
struct Split32 {};
template <class X> struct Frag;
template <> struct Frag<float> {
  typedef float E;
  static constexpr int BK = 16, PITCH = BK + 4, ACCS = 1;
  v4f p[2];
  __device__ static __forceinline__ void put(E* row, int v, const Chunk& c, bool zero, bool = false) {
    *reinterpret_cast<Chunk*>(row + v * 4) = zero ? zero_chunk() : c;
  }
  static constexpr int lane_off(int g) { return g * 8; }
  static constexpr int PHASES = 2;
  static constexpr int steps(int) { return 4; }
  __device__ __forceinline__ void load(const E* r, int ph) { p[ph] = *(const v4f*)(r + ph * 4); }
  __device__ static __forceinline__ void mma(const Frag& a, const Frag& b, v16f& c, int ph, int st) {
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.p[ph][st], b.p[ph][st], c, 0, 0, 0);
  }
};
template <> struct Frag<Split32> {
  typedef bf16_t E;
  static constexpr int BK = 16, PITCH = 3 * BK + 8, ACCS = 2;
  v8bf p[3];
  __device__ static __forceinline__ void put(E* row, int v, const Chunk& c, bool zero, bool neg = false) {
    u32x2_t q[3];
    split32(zero ? zero_chunk() : neg ? __builtin_bit_cast(Chunk, -__builtin_bit_cast(v4f, c)) : c, q);
#pragma unroll
    for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x2_t*>(row + k * BK + v * 4) = q[k];
  }
  static constexpr int lane_off(int g) { return g * 8; }
  static constexpr int PHASES = 3;
  static constexpr int steps(int ph) { return 3 - ph; }
  __device__ __forceinline__ void load(const E* r, int ph) { p[2 - ph] = *(const v8bf*)(r + (2 - ph) * BK); }
  // the smallest planes first, so that their registers are free first; the tile begins with the product that does not need
  // the planes which were loaded last
  __device__ static __forceinline__ void mma(const Frag& a, const Frag& b, v16f& c, int ph, int st) {
    constexpr int QA[3][3] = {{1, 2, 0}, {1, 0, 0}, {0, 0, 0}}, QB[3][3] = {{1, 0, 2}, {0, 1, 0}, {0, 0, 0}};
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[QA[ph][st]], b.p[QB[ph][st]], c, 0, 0, 0);
  }
};
template <class T, class V> struct Frag16 {
  typedef T E;
  static constexpr int BK = 32, PITCH = BK + 8, ACCS = 1;
  V p[2];
  __device__ static __forceinline__ void put(E* row, int v, const Chunk& c, bool zero, bool = false) {
    *reinterpret_cast<Chunk*>(row + v * 8) = zero ? zero_chunk() : c;
  }
  static constexpr int lane_off(int g) { return g * 16; }
  static constexpr int PHASES = 2;
  static constexpr int steps(int) { return 1; }
  __device__ __forceinline__ void load(const E* r, int ph) { p[ph] = *(const V*)(r + ph * 8); }
};
template <> struct Frag<bf16_t> : Frag16<bf16_t, v8bf> {
  __device__ static __forceinline__ void mma(const Frag& a, const Frag& b, v16f& c, int ph, int) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[ph], b.p[ph], c, 0, 0, 0);
  }
};
template <> struct Frag<f16_t> : Frag16<f16_t, v8h> {
  __device__ static __forceinline__ void mma(const Frag& a, const Frag& b, v16f& c, int ph, int) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a.p[ph], b.p[ph], c, 0, 0, 0);
  }
};

// fp32: the two accumulators made one; is any of a thread's sums not finite?
template <int MI, int NI>
__device__ __forceinline__ bool sums_not_finite(v16f (&acc)[2][MI][NI]) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[0][i][j] -= acc[1][i][j];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) s = __fmaf_rn(acc[0][i][j][e], 0.f, s);
  return !(s == 0.f);
}
template <int MI, int NI>
__device__ __forceinline__ bool sums_not_finite(v16f (&)[1][MI][NI]) { return false; }  // (16-bit: not asked)
// a lane's products of one depth tile on the fp32 instruction; a, b: its first row of each operand, whose rows lie 32 * pitch apart
template <int MI, int NI>
__device__ __forceinline__ void mma_fp32(const float* a, const float* b, int (&arow)[MI], int bstep, v16f (&acc)[MI][NI]) {
  Frag<float> fa[MI], fb[NI];
#pragma unroll
  for (int ph = 0; ph < 2; ++ph) {
#pragma unroll
    for (int i = 0; i < MI; ++i) fa[i].load(a + arow[i], ph);
#pragma unroll
    for (int j = 0; j < NI; ++j) fb[j].load(b + j * bstep, ph);
  }
#pragma unroll
  for (int ph = 0; ph < 2; ++ph)
#pragma unroll
    for (int st = 0; st < 4; ++st)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) Frag<float>::mma(fa[i], fb[j], acc[i][j], ph, st);
}
template <int MI, int NI>
__device__ __forceinline__ void clear_sums(v16f (&acc)[MI][NI]) {
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
}
// Within a depth tile the two lane groups (lanes 0-31, 32-63) own disjoint halves of the depth range and every MFMA
// pairs the same depth indices of A and B, so any assignment of depth indices to (lane group, step) gives the same sum.

// SPLIT: blockIdx.z owns a fixed range of depth tiles and writes raw fp32 sums to partial[z][M][Ng]; a second
// kernel adds the ranges in order and applies the epilogue (layers with few output pixels, to fill the chip).
// Pipeline: three LDS stages, two register generations.  Iteration j: MFMAs of tile j from operand registers; the
// halves of those registers are reloaded with tile j+1 (LDS stage (j+1)%3) as soon as their MFMAs are issued; the
// global loads of tile j+3 are issued at the top and written to LDS stage j%3 at the end of iteration j+1.
template <int V> struct IC { static constexpr int value = V; };

template <class X, int BM, int BN> constexpr size_t igemm_smem_bytes() {
  constexpr size_t stages = (size_t)3 * (BM + BN) * Frag<X>::PITCH * sizeof(typename Frag<X>::E);
  constexpr size_t epi = (size_t)(BM / 2) * (BN + 4) * 4;
  return stages > epi ? stages : epi;
}

template <class T, class X, int BM, int BN, int MODE, bool SPLIT>
__global__ void __launch_bounds__(256) conv_igemm_kernel(const T* __restrict__ src, const T* __restrict__ wmat,
                                                         const float* __restrict__ bias, const T* __restrict__ addend,
                                                         T* __restrict__ out, float* __restrict__ partial,
                                                         float* __restrict__ stat_partial, IGemmArgs a) {
  constexpr bool S32 = std::is_same_v<X, Split32>;
  constexpr int BK = Frag<X>::BK;
  constexpr int EV = 16 / (int)sizeof(T);   // elements per 16-byte chunk
  typedef typename Frag<X>::E E;
  constexpr int PITCH = Frag<X>::PITCH;     // LDS row pitch in staged elements
  constexpr int MI = BM / 64, NI = BN / 64; // 32x32 MFMA tiles per wavefront
  constexpr int A_CH = BM * 4 / 256;        // 16-byte chunks per thread and depth tile (4 chunks per row)
  constexpr int B_CH = BN * 4 / 256;
  constexpr int STAGE = (BM + BN) * PITCH;  // elements per LDS stage: A rows then B rows
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  E* lds = reinterpret_cast<E*>(smem_raw);

  // kernel arguments used inside the loaders, as plain scalars
  const int srcH = a.srcH, srcW = a.srcW, srcC = a.srcC, S_ = a.S, stride = a.stride, pad = a.pad;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, g = lane >> 5, l32 = lane & 31;
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
  const int vec = tid & 3, row0 = tid >> 2;  // this thread's chunk column and first row

  // This thread's A rows: element offset of the pixel that tap (0, 0) reads and a bit per tap that stays inside the image.
  // Every tap is a fixed distance from there, the same for all pixels (in a strided data gradient also: the taps that meet a
  // pixel have its parity), so a depth tile costs a row one select and one add.  (With the coordinates, three 64-bit
  // products per row and two divisions per depth tile were a serial chain in front of every tile's loads.  3x3 stride-2 layers
  // in fp16, us: forward with 256 x 2 blocks of 72 depth tiles 72 -> 60, 64 x 4 of 144 95 -> 71, data gradient by classes of
  // 32 x 2 blocks, the longest of 64 tiles, 53 -> 36; fp32, 2048 blocks: 368 -> 338 and 462 -> 395.)
  const int cz = a.cls ? blockIdx.z : 0;              // parity class
  const int cph = cz >> 1, cpw = cz & 1;
  const int ctaps = a.cls ? a.taps[cz] : 0;
  int64_t aoff[A_CH];
  unsigned inside[A_CH];
#pragma unroll
  for (int i = 0; i < A_CH; ++i) {
    const int m = m0 + row0 + i * 64;
    const int mm = m < a.M ? m : 0;
    int pb = mm % a.dstW;
    const int t = mm / a.dstW;
    int pa = t % a.dstH;
    const int pn = t / a.dstH;
    if (a.cls) { pa = 2 * pa + cph; pb = 2 * pb + cpw; }
    int y0, x0;
    unsigned rv = 0u, cv = 0u;  // bit r (s): filter row r (column s) stays inside
#pragma unroll
    for (int k = 0; k < 3; ++k) {  // 1x1 and 3x3 filters
      int y, x;
      bool yok = k < a.R, xok = k < S_;
      if (MODE != IG_DGRAD) {
        y = pa * stride + k - pad; x = pb * stride + k - pad;
      } else {
        const int ty = pa + pad - k, tx = pb + pad - k;
        if (stride == 2) { yok = yok && !(ty & 1); xok = xok && !(tx & 1); y = ty >> 1; x = tx >> 1; } else { y = ty; x = tx; }
      }
      rv |= yok && y >= 0 && y < srcH ? 1u << k : 0u;
      cv |= xok && x >= 0 && x < srcW ? 1u << k : 0u;
    }
    if (MODE != IG_DGRAD) { y0 = pa * stride - pad; x0 = pb * stride - pad; }
    else if (stride == 2) { y0 = (pa + pad) >> 1; x0 = (pb + pad) >> 1; }
    else { y0 = pa + pad; x0 = pb + pad; }
    aoff[i] = (((int64_t)pn * srcH + y0) * srcW + x0) * srcC + vec * EV;
    unsigned in = 0u;
#pragma unroll
    for (int r = 0; r < 3; ++r) in |= (rv >> r) & 1u ? cv << (r * S_) : 0u;
    inside[i] = m < a.M ? in : 0u;  // nothing of a row beyond the last pixel
  }
  const T* brow[B_CH];
#pragma unroll
  for (int i = 0; i < B_CH; ++i) brow[i] = wmat + (int64_t)(n0 + row0 + i * 64) * (a.R * a.S * srcC) + vec * EV;

  // Global loads are unconditional (addresses of out-of-image taps are clamped into the tensor) and the zeroing is
  // applied when the chunk is written to LDS: straight-line loads let the hardware keep several generations in flight.
  Chunk ra[2][A_CH], rb[2][B_CH];
  unsigned okm[2] = {0u, 0u};  // per generation: bit i set if A chunk i is inside the image
  const int kt0 = SPLIT ? blockIdx.z * a.kt_per_split : 0;
  int tapi = kt0 * BK / srcC, c0 = kt0 * BK - tapi * srcC;  // next depth tile to load: entry of the tap list, first channel
  int tap = 0;         // its filter tap r * S + s ...
  int64_t tdist = 0;   // ... and how far that lies from tap (0, 0) (two rows of an image may be more than 2^31 elements)
  auto next_tap = [&, srcW, srcC, S_, stride]() {
    tap = a.cls ? (ctaps >> (8 * (tapi & 3))) & 0xff : tapi;
    const int r = S_ == 3 ? (tap * 11) >> 5 : tap;  // tap / S, S being 3 or 1
    const int s = tap - r * S_;
    const int sh = MODE == IG_DGRAD && stride == 2 ? 1 : 0;
    const int64_t d = ((int64_t)(r >> sh) * srcW + (s >> sh)) * srcC;
    tdist = MODE == IG_DGRAD ? -d : d;
  };
  next_tap();
  auto gload = [&, srcC](auto P) {
    constexpr int p = decltype(P)::value;
    const int kkw = tap * srcC + c0;  // depth offset in the weight rows
    const int64_t toff = tdist + c0;
    unsigned m = 0u;
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
      const bool ok = (inside[i] >> tap) & 1u;
      ra[p][i] = *reinterpret_cast<const Chunk*>(src + (ok ? aoff[i] + toff : (int64_t)(vec * EV)));
      m |= ok ? (1u << i) : 0u;
    }
    okm[p] = m;
#pragma unroll
    for (int i = 0; i < B_CH; ++i) rb[p][i] = *reinterpret_cast<const Chunk*>(brow[i] + kkw);
    c0 += BK;
    if (c0 >= srcC) { c0 = 0; ++tapi; next_tap(); }
  };
  auto sstore = [&](auto P, int stage) {  // register generation p -> LDS stage
    constexpr int p = decltype(P)::value;
    E* st = lds + stage * STAGE;
#pragma unroll
    for (int i = 0; i < A_CH; ++i) Frag<X>::put(&st[(row0 + i * 64) * PITCH], vec, ra[p][i], !((okm[p] >> i) & 1u));
#pragma unroll
    for (int i = 0; i < B_CH; ++i) Frag<X>::put(&st[(BM + row0 + i * 64) * PITCH], vec, rb[p][i], false, p % Frag<X>::ACCS != 0);
  };

  constexpr int ACCS = Frag<X>::ACCS;
  v16f acc[ACCS][MI][NI];
#pragma unroll
  for (int h = 0; h < ACCS; ++h)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[h][i][j][e] = 0.f;

  const int nkt = (a.cls ? a.ntaps[cz] * srcC : a.Kg) / BK;  // depth tiles of this GEMM
  const int kt1 = SPLIT ? (kt0 + a.kt_per_split < nkt ? kt0 + a.kt_per_split : nkt) : nkt;
  const int n = kt1 > kt0 ? kt1 - kt0 : 0;
  // prologue: tiles 0 and 1 into LDS stages 0 and 1, tile 2 on its way in generation 0
  if (n > 0) { gload(IC<0>{}); sstore(IC<0>{}, 0); }
  if (n > 1) { gload(IC<1>{}); sstore(IC<1>{}, 1); }
  if (n > 2) gload(IC<0>{});
  __syncthreads();
  const int afrag = (wm * (BM / 2) + l32) * PITCH + Frag<X>::lane_off(g);
  const int bfrag = (BM + wn * (BN / 2) + l32) * PITCH + Frag<X>::lane_off(g);
  Frag<X> fa[MI], fb[NI];
  if (n > 0) {
#pragma unroll
    for (int ph = 0; ph < Frag<X>::PHASES; ++ph) {
#pragma unroll
      for (int i = 0; i < MI; ++i) fa[i].load(lds + afrag + i * 32 * PITCH, ph);
#pragma unroll
      for (int jn = 0; jn < NI; ++jn) fb[jn].load(lds + bfrag + jn * 32 * PITCH, ph);
    }
  }
  // iteration j: generation (j & 1) holds tile j+2 (issued at iteration j-1 or in the prologue)
  // TAIL = 0: steady state, every step unconditional (a branch around the loads would make the compiler wait for
  // the newest loads before each LDS store); TAIL = 1: the last iterations, with the range checks.
  auto body = [&](auto P, auto TAILC, int j, int stage) {
    constexpr int p = decltype(P)::value;  // = j & 1
    constexpr bool TAIL = decltype(TAILC)::value != 0;
    const E* nxt = lds + (stage == 2 ? 0 : stage + 1) * STAGE;
    const bool has_next = TAIL ? j + 1 < n : true;
    if (!TAIL || j + 3 < n) gload(IC<1 - p>{});
#pragma unroll
    for (int ph = 0; ph < Frag<X>::PHASES; ++ph) {
#pragma unroll
      for (int st = 0; st < Frag<X>::steps(ph); ++st)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int jn = 0; jn < NI; ++jn) Frag<X>::mma(fa[i], fb[jn], acc[p % ACCS][i][jn], ph, st);
      __builtin_amdgcn_sched_barrier(0);
      if (has_next) {
#pragma unroll
        for (int i = 0; i < MI; ++i) fa[i].load(nxt + afrag + i * 32 * PITCH, ph);
#pragma unroll
        for (int jn = 0; jn < NI; ++jn) fb[jn].load(nxt + bfrag + jn * 32 * PITCH, ph);
      }
      if (ph + 1 < Frag<X>::PHASES) __builtin_amdgcn_sched_barrier(0);
    }
    if (!TAIL || j + 2 < n) sstore(P, stage == 0 ? 2 : stage - 1);  // tile j+2 -> stage (j+2)%3
    __syncthreads();
  };
  {
    int stage = 0, j = 0;
    for (; j + 4 < n; j += 2) {
      body(IC<0>{}, IC<0>{}, j, stage);
      stage = stage == 2 ? 0 : stage + 1;
      body(IC<1>{}, IC<0>{}, j + 1, stage);
      stage = stage == 2 ? 0 : stage + 1;
    }
    for (; j < n; j += 2) {
      body(IC<0>{}, IC<1>{}, j, stage);
      stage = stage == 2 ? 0 : stage + 1;
      if (j + 1 < n) {
        body(IC<1>{}, IC<1>{}, j + 1, stage);
        stage = stage == 2 ? 0 : stage + 1;
      }
    }
  }

  if constexpr (S32) {
    if (__syncthreads_or(sums_not_finite(acc))) {  // the tile again on the fp32 instruction (split32.h)
      constexpr int FP = Frag<float>::PITCH;
      float* fl = reinterpret_cast<float*>(smem_raw);
      int arow[MI];
#pragma unroll
      for (int i = 0; i < MI; ++i) arow[i] = (wm * (BM / 2) + i * 32 + l32) * FP + Frag<float>::lane_off(g);
      clear_sums(acc[0]);
      tapi = kt0 * BK / srcC; c0 = kt0 * BK - tapi * srcC;
      next_tap();
#pragma unroll 1
      for (int j = 0; j < n; ++j) {
        gload(IC<0>{});
#pragma unroll
        for (int i = 0; i < A_CH; ++i) Frag<float>::put(&fl[(row0 + i * 64) * FP], vec, ra[0][i], !((okm[0] >> i) & 1u));
#pragma unroll
        for (int i = 0; i < B_CH; ++i) Frag<float>::put(&fl[(BM + row0 + i * 64) * FP], vec, rb[0][i], false);
        __syncthreads();
        mma_fp32(fl, fl + (BM + wn * (BN / 2) + l32) * FP + Frag<float>::lane_off(g), arow, 32 * FP, acc[0]);
        __syncthreads();
      }
    }
  }

  // epilogue through LDS, one half of the rows (the two wavefronts with the same wm) at a time, as fp32 [row][BN+4];
  // the store half (bias / addend / ReLU, rounding, stores, BatchNorm sums) is shared with the other kernels
  {
    float* ep = reinterpret_cast<float*>(smem_raw);
    constexpr int EP_PITCH = BN + 4;
    constexpr int HR = BM / 2;  // rows per pass
    constexpr bool STAT = MODE == IG_FWD && !SPLIT;
    float ss[8], qq[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) { ss[k] = 0.f; qq[k] = 0.f; }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      __syncthreads();
      if (wm == u) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int jn = 0; jn < NI; ++jn)
#pragma unroll
            for (int e = 0; e < 16; ++e)
              ep[(i * 32 + 8 * (e >> 2) + 4 * g + (e & 3)) * EP_PITCH + wn * (BN / 2) + jn * 32 + l32] = acc[0][i][jn][e];
      }
      __syncthreads();
      auto rowoff = [&](int row) -> int64_t {
        const int grow = m0 + u * HR + row;
        if (grow >= a.M) return -1;
        int64_t opix = grow;
        if (a.cls) {  // class-local pixel -> pixel of the full grid
          const int ww = grow % a.dstW, t2 = grow / a.dstW;
          const int hh = t2 % a.dstH, nn = t2 / a.dstH;
          opix = ((int64_t)nn * a.fullH + 2 * hh + cph) * a.fullW + 2 * ww + cpw;
        }
        return opix * a.Ng;
      };
      if (SPLIT) {
        epi_store_partial<BN, HR>(ep, tid, n0, partial + (int64_t)blockIdx.z * a.M * a.Ng, rowoff);
      } else if (MODE == IG_EVAL) {
        epi_eval_pass_nt<256, T, BN, HR>(ep, tid, n0, bias, a.Ng, addend, out, a.relu, rowoff);
      } else if (STAT && stat_partial) {
        epi_store_pass<T, BN, HR, MODE == IG_FWD, MODE == IG_DGRAD, true>(ep, tid, n0, bias, addend, a.amask, out, a.relu, rowoff, ss, qq);
      } else {
        epi_store_pass<T, BN, HR, MODE == IG_FWD, MODE == IG_DGRAD, false>(ep, tid, n0, bias, addend, a.amask, out, a.relu, rowoff, ss, qq);
      }
    }
    if (STAT && stat_partial)
      epi_stat_combine<BN>(ep, tid, ss, qq, stat_partial + ((int64_t)blockIdx.x * 2 + 0) * a.Ng + n0,
                           stat_partial + ((int64_t)blockIdx.x * 2 + 1) * a.Ng + n0);
  }
}

// ------------------------------------------------------------------------------------------------------------
// 3x3, stride 1: the input patch of the block's pixels (with its halo and zero border) is staged in LDS once per
// channel chunk and serves all nine filter taps, so the vector-memory path carries every input line once instead
// of nine times; only the 64-byte-deep weight tile changes from tap to tap.
//   block = 256 threads = 4 wavefronts (2 x 2); block tile = 64*MI pixel rows x BN channels; a wavefront owns 32*MI
//   rows and BN/2 channels: MI x (BN/64) MFMA 32x32 tiles.  The rows are SUBT pixel sub-tiles of 64*MI/SUBT pixels
//   (TI images x TR rows x TC columns each, with their own halo).  Instantiated: (MI 2, SUBT 1) with 128 or 64
//   channels and (1, 1) with 64; two blocks share a CU, three with 64 channels (registers capped, patch
//   buffers sized for the layer's tile).
//   LDS: 2 patch buffers [SUBT*256 positions][80 B], 3 weight stages [BN][80 B], address tables.
//   Pipeline (one barrier per tap): the weight tile of (chunk c+1, tap t) is requested before the MFMAs of (c, t)
//   and parked in registers until the end of step (c+1, t-1); the next chunk's patch is requested during taps 0-3
//   and stored during taps 4-7.  All loads are straight-line, so several steps of loads stay in flight.
//   The data gradient of a stride-1 convolution is the same computation on dz with the taps visited in reverse and
//   the border (kh-1-pad).
// ------------------------------------------------------------------------------------------------------------
constexpr int PATCH_MAX_POS = 256;  // positions per sub-tile

// least and most wavefronts per SIMD that the registers are to leave room for
template <class X> constexpr int PATCH_WAVES(int bn, int mi, int most) {
  if (std::is_same_v<X, Split32>) return mi == 1 ? 3 : 2;  // (64 channels per block only)
  return bn == 64 ? 3 : 1 + most;
}

// EVAL: `bias` is the [2][Ng] scale and shift of the inference-mode BatchNorm behind the layer, `addend` its skip connection
// STAT: 1 the sums of the BatchNorm behind the layer, 2 (data gradient) those of the BatchNorm backward in front of it: `bias` is then
// that one's statistics tensor, `addend` its z and a.relu whether a ReLU follows it
template <class T, class X, int BN, int MI, int SUBT, int STAT, bool FOLD = false, bool EVAL = false>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PATCH_WAVES<X>(BN, MI, 0), PATCH_WAVES<X>(BN, MI, 1))))
conv3x3_patch_kernel(const T* __restrict__ src, const T* __restrict__ wmat, const float* __restrict__ bias,
                     const T* __restrict__ addend, T* __restrict__ out, float* __restrict__ partial,
                     float* __restrict__ stat_partial, PatchArgs a) {
  constexpr bool S32 = std::is_same_v<X, Split32>;
  constexpr int ROWS = 64 * MI;              // pixel rows of the block
  constexpr int TPC = ROWS / SUBT;           // rows (pixel capacity) per sub-tile
  constexpr int NSLOT = 4 * SUBT;            // 16-byte patch pieces per thread and channel chunk
  constexpr int SPT = NSLOT / 4;             // pieces requested / stored per tap
  constexpr int CCE = Frag<X>::BK;           // channels per chunk (64 bytes)
  typedef typename Frag<X>::E E;
  constexpr int EV = 16 / (int)sizeof(T);
  constexpr int PITCH = Frag<X>::PITCH;      // staged elements per LDS row
  constexpr int NI = BN / 64;
  constexpr int B_CH = BN * 4 / 256;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int PBUF = a.patch_elems;                                             // one patch buffer, sized for this layer
  E* patch = reinterpret_cast<E*>(smem_raw);                                  // [2][PBUF]
  E* Bs = patch + 2 * PBUF;                                                   // [3][BN][PITCH]
  int64_t* src_off = reinterpret_cast<int64_t*>(Bs + 3 * BN * PITCH);         // [SUBT*PATCH_MAX_POS]
  int64_t* out_off = src_off + SUBT * PATCH_MAX_POS;                          // [256]
  int* apos = reinterpret_cast<int*>(out_off + 256);                          // [256]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, g = lane >> 5, l32 = lane & 31;
  // Block coordinates: (row tile, channel block, depth range).  Workgroups go to the 8 XCDs round-robin by their
  // linear index, and every XCD has an L2 of its own.  With large weights and few pixels the row tiles of one
  // (channel block, depth range) all read the same weight slice: renumbered, they run on one XCD, which then fetches
  // the slice once instead of all eight doing so.  Needs (channel blocks x depth ranges) % 8 == 0 (launcher).
  int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
  if (a.xcd_group == 1) {
    const unsigned lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const unsigned xcd = lin & 7u, slot = lin >> 3;
    const unsigned grp = (slot / gridDim.x) * 8u + xcd;  // index of the (channel block, depth range) pair
    bx = (int)(slot % gridDim.x); by = (int)(grp % gridDim.y); bz = (int)(grp / gridDim.y);
  }
  // Many pixels and two or more channel blocks: the blocks of one row tile all stage the same patches of the source;
  // renumbered onto one XCD in consecutive slots they fetch them from HBM once (256 -> 256 channels at 262 144 pixels,
  // bf16: 293 MB per launch without it for 135 MB of operands).  The grid's x extent is then the number of row tiles
  // rounded up to a multiple of 8.
  if (a.xcd_group == 2) {
    const unsigned lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const unsigned xcd = lin & 7u, slot = lin >> 3;
    const unsigned per = gridDim.y * gridDim.z, idx = slot % per;
    bx = (int)((slot / per) * 8u + xcd); by = (int)(idx % gridDim.y); bz = (int)(idx / gridDim.y);
    if (bx >= a.row_blocks) return;
  }
  const int n0c = by * BN;
  const int npos2 = SUBT * a.NPOS;
  const int srcC = a.srcC, flip = a.flip, SC = a.SC;
  const int RPE = a.row_pitch / (int)sizeof(E);  // elements between staged patch rows

  // ---- address tables ------------------------------------------------------------------------------------------
  for (int e = tid; e < npos2; e += 256) {
    const int u = e / a.NPOS, rem = e - u * a.NPOS;
    const int ti = rem / (a.SR * a.SC), rr = rem - ti * (a.SR * a.SC);
    const int sy = rr / a.SC, sx = rr - sy * a.SC;
    const int tile = SUBT * bx + u;
    int64_t off = -1;
    if (tile < a.NT) {
      const int ci = tile % a.tiles_c, t2 = tile / a.tiles_c;
      const int ri = t2 % a.tiles_r, ii = t2 / a.tiles_r;
      const int n = ii * a.TI + ti, y = ri * a.TR - a.pad + sy, x = ci * a.TC - a.pad + sx;
      if (n < a.N && y >= 0 && y < a.srcH && x >= 0 && x < a.srcW) off = (((int64_t)n * a.srcH + y) * a.srcW + x) * a.srcC;
    }
    src_off[e] = off;
  }
  {
    const int m2 = tid, u = m2 / TPC, m = m2 - u * TPC;
    const int tile = SUBT * bx + u;
    int64_t off = -1;
    int ap = 0;
    if (m2 < ROWS && m < a.TP && tile < a.NT) {
      const int ti = m / (a.TR * a.TC), rr = m - ti * (a.TR * a.TC);
      const int tr = rr / a.TC, tc = rr - tr * a.TC;
      const int ci = tile % a.tiles_c, t2 = tile / a.tiles_c;
      const int ri = t2 % a.tiles_r, ii = t2 / a.tiles_r;
      const int n = ii * a.TI + ti, p = ri * a.TR + tr, q = ci * a.TC + tc;
      ap = ((u * a.TI + ti) * a.SR + tr) * RPE + tc * PITCH;  // LDS element offset of tap (0,0)
      if (n < a.N && p < a.dstH && q < a.dstW) off = (((int64_t)n * a.dstH + p) * a.dstW + q) * a.Ng;
    }
    out_off[m2] = off;
    apos[m2] = ap;
  }
  __syncthreads();

  // channel chunks of this block: all of them, or the range of blockIdx.z (raw sums go to `partial`, a second
  // kernel adds the ranges in order and applies the epilogue)
  const int cb = bz * a.chunks_per_split;
  const int ce = cb + a.chunks_per_split < srcC / CCE ? cb + a.chunks_per_split : srcC / CCE;
  const int Kg = 9 * srcC;

  // ---- loaders ---------------------------------------------------------------------------------------------------
  Chunk PR[NSLOT];  // patch chunks in flight (next channel chunk)
  // weight tiles in flight: one generation per tap, requested a whole channel chunk (nine steps) ahead
  // (a = rows 0-63, b = rows 64-127 of the tile)
  Chunk BRa[9], BRb[9];
  const int bvec = tid & 3, brow0 = tid >> 2;
  // patch pieces of this thread: slot sl covers the 16-byte piece idx = sl*256 + tid.  Loads are unconditional
  // (pieces outside the image read the tensor's first pixel) and are zeroed when written to LDS.
  const T* pptr[NSLOT];
  int pdst[NSLOT];  // LDS element offset of the piece's position within a patch buffer
  unsigned pvalid = 0u, pstore = 0u;
#pragma unroll
  for (int sl = 0; sl < NSLOT; ++sl) {
    const int idx = sl * 256 + tid;
    const int pos = idx >> 2, v = idx & 3;
    int64_t off = 0;
    int dst = 0;
    if (pos < npos2) {
      pstore |= 1u << sl;
      const int64_t o = src_off[pos];
      if (o >= 0) { off = o; pvalid |= 1u << sl; }
      const int prow = pos / SC;
      dst = prow * RPE + (pos - prow * SC) * PITCH;
    }
    pptr[sl] = src + off + v * EV;
    pdst[sl] = dst;
  }
  auto patch_load = [&](int slot, int chunk) { return *reinterpret_cast<const Chunk*>(pptr[slot] + chunk * CCE); };
  // FOLD: all pieces of a thread cover channels [(tid & 3) * EV, + EV) of the chunk; their scale and shift are
  // requested with the first pieces of a chunk and used when the pieces are stored
  float fsc[EV], fsh[EV];
  auto fold_load = [&](int chunk) {
    if (FOLD) {
      const int c = chunk * CCE + (tid & 3) * EV;
      load_f32<float, EV>(a.fold + 2 * srcC + c, fsc);
      load_f32<float, EV>(a.fold + 3 * srcC + c, fsh);
    }
  };
  auto patch_store = [&](int slot, int buf, const Chunk& c) {
    if ((pstore >> slot) & 1u) {
      Chunk v = c;
      if (FOLD) v = bn_fold_chunk<T>(c, fsc, fsh);
      Frag<X>::put(&patch[buf * PBUF + pdst[slot]], tid & 3, v, !((pvalid >> slot) & 1u));
    }
  };
  const T* wrow = wmat + (int64_t)(n0c + brow0) * Kg + bvec * EV;
  // weight tile of global step gs = chunk*9 + tap -> registers REG
  // weight tile of tap slot t_ of channel chunk ch_ -> registers of generation t_
#define B_LOAD(t_, ch_)                                                                                       \
  {                                                                                                           \
    const int tap_ = flip ? 8 - (t_) : (t_);                                                                  \
    const T* wp_ = wrow + tap_ * srcC + (ch_) * CCE;                                                          \
    BRa[t_] = *reinterpret_cast<const Chunk*>(wp_);                                                           \
    if (B_CH > 1) BRb[t_] = *reinterpret_cast<const Chunk*>(wp_ + (int64_t)64 * Kg);                          \
  }
#define B_STORE(t_, stage_)                                                                                   \
  {                                                                                                           \
    Frag<X>::put(&Bs[((stage_) * BN + brow0) * PITCH], bvec, BRa[t_], false, (t_) % Frag<X>::ACCS != 0);      \
    if (B_CH > 1)                                                                                             \
      Frag<X>::put(&Bs[((stage_) * BN + brow0 + 64) * PITCH], bvec, BRb[t_], false, (t_) % Frag<X>::ACCS != 0); \
  }

  // ---- prologue -----------------------------------------------------------------------------------------------
#pragma unroll
  for (int sl = 0; sl < NSLOT; ++sl) PR[sl] = patch_load(sl, cb);
  fold_load(cb);
#pragma unroll
  for (int t = 0; t < 9; ++t) B_LOAD(t, cb);
#pragma unroll
  for (int sl = 0; sl < NSLOT; ++sl) patch_store(sl, 0, PR[sl]);
  B_STORE(0, 0);
  B_STORE(1, 1);
  __syncthreads();

  int arow[MI];  // LDS element offset of tap (0,0) for this lane's 32-row groups
#pragma unroll
  for (int i = 0; i < MI; ++i) arow[i] = apos[wm * (32 * MI) + i * 32 + l32] + Frag<X>::lane_off(g);
  const int bfrag = (wn * (BN / 2) + l32) * PITCH + Frag<X>::lane_off(g);  // this lane's row in a weight stage

  constexpr int ACCS = Frag<X>::ACCS;  // (by the parity of the tap)
  v16f acc[ACCS][MI][NI];
#pragma unroll
  for (int h = 0; h < ACCS; ++h)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[h][i][j][e] = 0.f;

  // Operand fragments live in one set of registers.  Each half (first / second 16 bytes of the 32-byte depth slice) is
  // reloaded for the next step right after the MFMAs that consumed it have been issued, so the LDS reads of step g+1
  // run under the MFMAs of step g and nothing waits on LDS latency.  Weight stage = step % 3; the weight tile of step
  // g+2 is written at the end of step g, the next chunk's patch during taps 4-7, so both are complete one barrier
  // before their first read.
  Frag<X> fa[MI], fb[NI];
#pragma unroll
  for (int ph = 0; ph < Frag<X>::PHASES; ++ph) {
#pragma unroll
    for (int i = 0; i < MI; ++i) fa[i].load(patch + arow[i], ph);
#pragma unroll
    for (int j = 0; j < NI; ++j) fb[j].load(&Bs[bfrag + j * 32 * PITCH], ph);
  }

  // one channel chunk = nine taps; LAST = no chunk follows (no patch prefetch, weight requests stop at the end)
  auto chunk_body = [&](auto LAST, int chunk) {
    constexpr bool last = decltype(LAST)::value != 0;
    const int pbuf = (chunk - cb) & 1;
    const E* pcur = patch + pbuf * PBUF;
    const E* pnxt = patch + (pbuf ^ 1) * PBUF;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      // where the next step reads its operands
      const bool has_next = !last || t + 1 < 9;
      const int tn = (t + 1) % 9;
      const E* pn = t + 1 < 9 ? pcur : pnxt;
      const int tapoff_n = (tn / 3) * RPE + (tn % 3) * PITCH;
      const E* bn_ = &Bs[((t + 1) % 3) * BN * PITCH + bfrag];
      // requests: the weight tile this tap will need in the next chunk, two pieces of the next patch during taps 0-3
      if (!last) B_LOAD(t, chunk + 1);
      if (!last && t < 4) {
#pragma unroll
        for (int q = 0; q < SPT; ++q) PR[SPT * t + q] = patch_load(SPT * t + q, chunk + 1);
        if (t == 0) fold_load(chunk + 1);
      }
#pragma unroll
      for (int ph = 0; ph < Frag<X>::PHASES; ++ph) {
#pragma unroll
        for (int st = 0; st < Frag<X>::steps(ph); ++st)
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) Frag<X>::mma(fa[i], fb[j], acc[t % ACCS][i][j], ph, st);
        __builtin_amdgcn_sched_barrier(0);
        if (has_next) {
#pragma unroll
          for (int i = 0; i < MI; ++i) fa[i].load(pn + arow[i] + tapoff_n, ph);
#pragma unroll
          for (int j = 0; j < NI; ++j) fb[j].load(bn_ + j * 32 * PITCH, ph);
        }
        if (ph + 1 < Frag<X>::PHASES) __builtin_amdgcn_sched_barrier(0);
      }
      // parked data goes to LDS: weight tile of step g+2, patch pieces requested four taps ago
      if (t + 2 < 9) B_STORE(t + 2, (t + 2) % 3) else if (!last) B_STORE(t + 2 - 9, (t + 2) % 3)
      if (!last && t >= 4 && t < 8) {
#pragma unroll
        for (int q = 0; q < SPT; ++q) patch_store(SPT * (t - 4) + q, pbuf ^ 1, PR[SPT * (t - 4) + q]);
      }
      __syncthreads();
    }
  };
  for (int chunk = cb; chunk + 1 < ce; ++chunk) chunk_body(IC<0>{}, chunk);
  chunk_body(IC<1>{}, ce - 1);

  if constexpr (S32) {
    if (__syncthreads_or(sums_not_finite(acc))) {  // the tile again on the fp32 instruction (split32.h), a position's values
      constexpr int FP = PITCH / 2;                // in the place of its planes
      float* fpatch = reinterpret_cast<float*>(patch);
      float* fB = reinterpret_cast<float*>(Bs);
      const float* fb = fB + (wn * (BN / 2) + l32) * FP + Frag<float>::lane_off(g);
      clear_sums(acc[0]);
#pragma unroll
      for (int i = 0; i < MI; ++i) arow[i] = (arow[i] - Frag<X>::lane_off(g)) / 2 + Frag<float>::lane_off(g);
#pragma unroll 1
      for (int chunk = cb; chunk < ce; ++chunk) {
#pragma unroll
        for (int sl = 0; sl < NSLOT; ++sl) {
          const Chunk c = patch_load(sl, chunk);
          if ((pstore >> sl) & 1u) Frag<float>::put(fpatch + pdst[sl] / 2, tid & 3, c, !((pvalid >> sl) & 1u));
        }
#pragma unroll 1
        for (int t = 0; t < 9; ++t) {
          const T* wp = wrow + (flip ? 8 - t : t) * srcC + chunk * CCE;
#pragma unroll
          for (int i = 0; i < B_CH; ++i)
            Frag<float>::put(fB + (brow0 + i * 64) * FP, bvec, *reinterpret_cast<const Chunk*>(wp + (int64_t)(i * 64) * Kg), false);
          __syncthreads();
          mma_fp32(fpatch + (t / 3 * RPE + t % 3 * PITCH) / 2, fb, arow, 32 * FP, acc[0]);
          __syncthreads();
        }
      }
    }
  }

  // ---- epilogue ---------------------------------------------------------------------------------------------------
  // The accumulators go through LDS (the patch buffers are free now), the rows of one wavefront pair at a time, as
  // fp32 [row][BN + 4]; the store half (bias / addend / ReLU, rounding, stores of whole rows, BatchNorm sums of the
  // stored values) is shared with the other kernels.
  {
    float* ep = reinterpret_cast<float*>(smem_raw);
    constexpr int EP_PITCH = BN + 4;
    constexpr int HR = 32 * MI;  // rows per pass
    float ss[8], qq[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) { ss[k] = 0.f; qq[k] = 0.f; }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      __syncthreads();
      if (wm == u) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e)
              ep[(i * 32 + 8 * (e >> 2) + 4 * g + (e & 3)) * EP_PITCH + wn * (BN / 2) + j * 32 + l32] = acc[0][i][j][e];
      }
      __syncthreads();
      auto rowoff = [&](int row) -> int64_t { return out_off[u * HR + row]; };
      if (partial)
        epi_store_partial<BN, HR>(ep, tid, n0c, partial + (int64_t)bz * ((int64_t)a.N * a.dstH * a.dstW * a.Ng), rowoff);
      else if (EVAL)
        epi_eval_pass_nt<256, T, BN, HR>(ep, tid, n0c, bias, a.Ng, addend, out, a.relu, rowoff);
      else if constexpr (STAT == 2)
        epi_bn_sums_rows_nt<256, T, BN, HR>(ep, tid, n0c, bias, a.Ng, addend, out, a.relu, rowoff, ss, qq);
      else
        epi_store_pass<T, BN, HR, true, STAT == 0, STAT == 1>(ep, tid, n0c, bias, addend, a.amask, out, a.relu, rowoff, ss, qq);
    }
    if (STAT)
      epi_stat_combine<BN>(ep, tid, ss, qq, stat_partial + ((int64_t)bx * 2 + 0) * a.Ng + n0c,
                           stat_partial + ((int64_t)bx * 2 + 1) * a.Ng + n0c);
  }
}

#undef B_LOAD
#undef B_STORE

// Sum of the depth ranges in order, then bias / residual addend / ReLU, one rounding, store.  A block covers ROWS rows
// x 64 channels (thread = 4 channels of every 16th row), so that it can also produce the per-channel sums of the
// stored values for the BatchNorm that follows: stat_partial [ceil(M / ROWS)][2][Ng], or null.  Bound by latency at the
// few pixels this is for: the loads of eight ranges are issued before the first is added, and with 64 rows per block a
// layer of 256 pixels and 512 channels left 224 CUs idle (12 us for its 32 ranges); 16 rows where 64 give under 512 blocks.
static int split_epi_rows(int64_t M, int Ng) { return (int64_t)((M + 63) / 64) * (Ng / 64) >= 512 ? 64 : 16; }
template <class T, int ROWS>
__global__ void __launch_bounds__(256) splitk_epilogue_kernel(const float* __restrict__ partial, int splits, int64_t M, int Ng,
                                                              const float* __restrict__ bias, const T* __restrict__ addend,
                                                              const uint8_t* __restrict__ amask, T* __restrict__ out,
                                                              float* __restrict__ stat_partial, int relu,
                                                              const float* __restrict__ affine) {
  __shared__ float red[2][16][64];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int col = blockIdx.y * 64 + tx * 4;
  const int64_t n = M * Ng;
  float bv[4] = {0.f, 0.f, 0.f, 0.f};
  if (bias) {
#pragma unroll
    for (int e = 0; e < 4; ++e) bv[e] = bias[col + e];
  }
  float sv[4] = {1.f, 1.f, 1.f, 1.f};
  if (affine) {  // (no bias then)
#pragma unroll
    for (int e = 0; e < 4; ++e) { sv[e] = affine[col + e]; bv[e] = affine[Ng + col + e]; }
  }
  float ss[4] = {0.f, 0.f, 0.f, 0.f}, qq[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int it = 0; it < ROWS / 16; ++it) {
    const int64_t row = (int64_t)blockIdx.x * ROWS + it * 16 + ty;
    if (row < M) {
      const int64_t i = row * Ng + col;
      v4f acc = {0.f, 0.f, 0.f, 0.f};
      for (int z0 = 0; z0 < splits; z0 += 8) {  // (ranges past the last one read the last one and are not added)
        v4f t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = *reinterpret_cast<const v4f*>(partial + (int64_t)(z0 + u < splits ? z0 + u : splits - 1) * n + i);
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (z0 + u < splits) acc += t[u];
      }
      float r[4];
      // the addend's ReLU bits, if it has any: four consecutive elements lie in one byte (i is a multiple of 4)
      unsigned mb = 0xfu;
      if (addend && amask) mb = sizeof(T) == 2 ? (amask[i >> 3] >> (i & 4)) & 15u : amask[i >> 2] & 15u;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float v = affine ? bn_affine(acc[e], sv[e], bv[e]) : acc[e] + bv[e];
        if (addend && ((mb >> e) & 1u)) v += to_f32(addend[i + e]);
        r[e] = relu ? fmaxf(v, 0.f) : v;
      }
      store_f32<T, 4>(out + i, r);
      if (stat_partial) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float v = to_f32(from_f32<T>(r[e]));  // as stored
          ss[e] += v; qq[e] = __fmaf_rn(v, v, qq[e]);
        }
      }
    }
  }
  if (stat_partial) {  // the 16 row groups of a channel, added in a fixed order
#pragma unroll
    for (int e = 0; e < 4; ++e) { red[0][ty][tx * 4 + e] = ss[e]; red[1][ty][tx * 4 + e] = qq[e]; }
    __syncthreads();
    if (threadIdx.x < 128) {
      const int which = threadIdx.x >> 6, c = threadIdx.x & 63;
      float t = 0.f;
#pragma unroll
      for (int y = 0; y < 16; ++y) t += red[which][y][c];
      stat_partial[((int64_t)blockIdx.x * 2 + which) * Ng + blockIdx.y * 64 + c] = t;
    }
  }
}

template <class T>
static void launch_splitk_epilogue(hipStream_t st, const float* partial, int splits, int64_t M, int Ng, const float* bias,
                                   const void* addend, const uint8_t* amask, void* out, float* stat_partial, int relu,
                                   const float* affine = nullptr) {
  const int rows = split_epi_rows(M, Ng);
  dim3 grid(ceil_div(M, rows), Ng / 64);  // Ng % 64 == 0 for every MFMA convolution
  if (rows == 64)
    OSEQ_LAUNCH((splitk_epilogue_kernel<T, 64>), grid, dim3(256), 0, st, partial, splits, M, Ng, bias, (const T*)addend, amask,
                (T*)out, stat_partial, relu, affine);
  else
    OSEQ_LAUNCH((splitk_epilogue_kernel<T, 16>), grid, dim3(256), 0, st, partial, splits, M, Ng, bias, (const T*)addend, amask,
                (T*)out, stat_partial, relu, affine);
}

// LDS of the patch kernel: two patch buffers of patch_elems elements, three weight stages, the address tables
template <class X> constexpr size_t patch_smem_bytes(int bn, int subt, int64_t patch_elems) {
  return (size_t)(2 * patch_elems + 3 * bn * Frag<X>::PITCH) * sizeof(typename Frag<X>::E) + subt * PATCH_MAX_POS * 8 +
         256 * 8 + 256 * 4;
}
template <class X> constexpr size_t patch_smem_max(int bn, int subt) {
  return patch_smem_bytes<X>(bn, subt, (int64_t)subt * PATCH_MAX_POS * Frag<X>::PITCH);
}

// tile geometry of the patch kernel for a (dstH x dstW) pixel grid gathered with a 3x3 window and sub-tiles of up to
// `cap` pixels; false if it does not fit
static bool patch_geometry_of(int N, int dstH, int dstW, int tc, int cap, PatchArgs& a, int most = PATCH_MAX_POS) {
  int tr = cap / tc; if (tr > dstH) tr = dstH; if (tr < 1) tr = 1;
  int ti = (tr == dstH && tc == dstW) ? cap / (dstH * dstW) : 1;
  if (ti > N) ti = N; if (ti < 1) ti = 1;
  while (ti > 1 && ti * (tr + 2) * (tc + 2) > most) ti /= 2;
  while (tr > 1 && ti * (tr + 2) * (tc + 2) > most) --tr;
  while (tc > 1 && ti * (tr + 2) * (tc + 2) > most) tc /= 2;
  if (ti * (tr + 2) * (tc + 2) > most) return false;
  a.TI = ti; a.TR = tr; a.TC = tc; a.SR = tr + 2; a.SC = tc + 2;
  a.NPOS = ti * a.SR * a.SC; a.TP = ti * tr * tc;
  a.tiles_r = (dstH + tr - 1) / tr; a.tiles_c = (dstW + tc - 1) / tc;
  a.NT = ((N + ti - 1) / ti) * a.tiles_r * a.tiles_c;
  return true;
}
// The widest sub-tile; where three rows of the map leave it less than three quarters of the pixels (64 of 128 on maps of 63 columns or
// more), the narrower one that covers the map with the fewest sub-tiles, then staged positions.  (bf16, us, without -> with: two forward
// passes of 128 channels at 16 x 64 x 64 132 -> 85, a data gradient of them 80 -> 54, at 8 x 112 x 112 200 -> 135 and 122 -> 87; 256
// channels at 2 x 100 x 75 114 -> 70 and 54 -> 33.)
static bool patch_geometry(int N, int dstH, int dstW, int cap, bool narrow, PatchArgs& a, int most = PATCH_MAX_POS) {
  bool ok = patch_geometry_of(N, dstH, dstW, dstW < cap ? dstW : cap, cap, a, most);
  if (!narrow || (ok && a.TP * 4 >= cap * 3)) return ok;
  for (int tc = 64; tc >= 8; tc /= 2) {
    PatchArgs b = a;
    if (tc >= dstW || !patch_geometry_of(N, dstH, dstW, tc, cap, b, most)) continue;
    if (!ok || b.NT < a.NT) { a = b; ok = true; }
    else if (b.NT == a.NT && b.NPOS < a.NPOS) a = b;
  }
  return ok;
}

// Bytes between staged patch rows (patch_rows_apart), kept at SC positions when the padded rows would not fit the patch buffer.
static int patch_row_pitch(const PatchArgs& a, int subt, int pos_bytes, int most = PATCH_MAX_POS) {
  const int rp = patch_rows_apart(a.TC, a.SC, pos_bytes);
  const int64_t rows = (int64_t)subt * a.TI * a.SR;
  return rows * rp <= (int64_t)subt * most * pos_bytes ? rp : a.SC * pos_bytes;
}

// Blocks of the patch kernel whose LDS (given out in units of 1280 bytes) a CU holds.
static int patch_blocks_per_cu(const PatchArgs& a, int row_pitch, int subt, int bn, int pos_bytes) {
  const int64_t patch = ((int64_t)subt * a.TI * a.SR * row_pitch + 15) / 16 * 16;
  const int64_t bytes = 2 * patch + (int64_t)3 * bn * pos_bytes + subt * PATCH_MAX_POS * 8 + 256 * 8 + 256 * 4;
  return (int)(160 * 1024 / ((bytes + 1279) / 1280 * 1280));
}

// Tiles of 64 pixels that read more weights than an XCD's L2 holds for all the blocks it runs, at different depths: rows stay unpadded,
// except in tiles of 8 and 4 columns.  Freed from bank conflicts the blocks drift apart and miss the L2 more often.  One layer forward on
// 15 x 5 maps of 24 675 pixels in bf16, padded to unpadded: 768 -> 768 channels 1.13, 896 -> 896 1.48, 1024 -> 1024 1.21, 1280 -> 896
// 1.59 (at 12 000 pixels), data gradients alike; to either side 704 -> 704 0.92, 1280 -> 640 0.90, 512 -> 1024 0.95, 1280 -> 1280 0.99,
// and 896 -> 896 on 3000 pixels 0.95.  The data gradient in fp32 on 12 000 pixels: 1280 channels 1.12, 1024 0.97.
static bool patch_weights_missed(int dt, int mi, int tiles, int srcC, int Ng) {
  const int64_t bytes = (int64_t)9 * srcC * Ng * (dt == DT_F32 ? 4 : 2);
  return mi == 1 && tiles >= 128 && srcC >= 640 && Ng > 640 && bytes >= (dt == DT_F32 ? 48'000'000 : 10'000'000);
}

// Block shapes of the patch kernel, largest first: {MI, SUBT, widest BN}.  The first one that gives the chip
// `g_patch_fill` blocks is taken, else the one with the most blocks if that reaches `g_patch_min_blocks`
// (shape-only rule, so the choice is the same on every run).
struct PatchShape { int mi, subt, bn, splits; bool wide; };
static constexpr int g_patch_min_blocks = 64;   // compile-time constants
static constexpr int g_patch_fill = 512;
static constexpr int g_patch_shapes = 0x7;      // bit i: candidate i allowed
static constexpr int g_patch_split = 1;         // allow the depth split
static constexpr int g_patch_halo2 = 9;         // largest staged positions : pixels ratio, times two
static constexpr int g_patch_target_small = 512;  // blocks aimed at by the depth split for the smallest block shape in fp32
static constexpr int64_t g_patch_xcd_wbytes = 4 << 20;  // XCD grouping of the blocks: least weight bytes (0: never) ...
static constexpr int g_patch_xcd_rows = 16;              // ... and most row tiles
enum PatchUse { PATCH_FWD, PATCH_EVAL, PATCH_DGRAD };  // forward pass of a step, inference, data gradient
// 16 bits: tiles of 256 pixels x 256 channels, else x 128, by one wavefront per SIMD (k_conv_patch_wide.hip).  A CU holds one such
// block, so the rounds of 256 blocks have to be full: at least 85 % of their products have to be wanted ones, which leaves out
// layers of less than 218 tiles -- one of 128 tiles would leave half of the CUs idle -- and maps that tile badly (14 x 14: 77 %).
// Then, in bf16, time over the narrow tiles' at 16 x 16 pixels a map, one round at 88 % and at 99 %:
//   forward with sums   channels 32 -> 128 0.84 0.85, 64 -> 128 0.85 0.88, 128 -> 128 0.83 0.96, 128 -> 256 0.87 0.90, 512 -> 512 0.77 0.89
//   data gradient       128 -> 128 0.88 1.01, 256 -> 256 0.85 0.96
// Beyond a round nothing covers a block's epilogue and the next one's beginning, where two narrow blocks on a CU are no longer in
// step.  What that costs depends on the products a block has in between:
//   tiles of 128 channels: 32 -> 128 1.11 - 1.30 from two rounds on.  64 and 128 -> 128 in tile rows of up to 32 pixels, of a step
//     with two such layers or blocks on 8 x 8, 16 x 16 or 32 x 32 maps: two rounds 0.96 - 1.01, three 0.98 - 1.01, from the fourth on
//     1.00 - 1.03 (the kernels 0.99 - 1.12 forward, 1.03 - 1.25 in the data gradient); in rows of 64 pixels, with a fifth more
//     positions to stage, 1.02 - 1.04 from the second round on.  256 -> 256, with the BatchNorm sums of a data gradient that 256 pixels
//     a tile make few enough to come with it: a step 0.98 - 0.99, from the fourth round on 0.99 - 1.02 below 93 % and 0.98 above;
//     384 -> 384 0.97 - 1.00, 640 -> 640 0.94 - 0.99
//   of 256 channels: 32 -> 256 0.98 - 1.12, 64 -> 256 0.94 - 1.04, 128 -> 256 0.90 - 0.99, 256 -> 256 and deeper 0.79 - 0.95
// Where the narrow tiles fit a map a tenth worse (4 x 4 and 7 x 7) or not at all the wide ones are ahead at every depth (128 -> 128
// over 131 072 pixels 0.64 and 0.84), and in inference, whose epilogue is short, too: 128 -> 128 in several rounds 0.91, at 64 x 128 1.0.
static bool patch_wide_pays(PatchUse use, int N, int dstH, int dstW, int srcC, int bn, int64_t wanted, const PatchArgs& a, int64_t blocks) {
  const int64_t rounds = (blocks + 255) / 256, offered = rounds * 256 * 256 * bn;
  if (wanted * 20 < offered * 17) return false;
  if (rounds == 1 || use == PATCH_EVAL) return true;
  if (srcC >= (bn == 256 ? 128 : 384)) return true;
  if (srcC >= (bn == 256 ? 64 : 256) && (wanted * 100 >= offered * 93 || (bn == 128 && rounds <= 3))) return true;
  if (bn == 128 && srcC >= 64 && rounds <= 3 && a.TC <= 32) return true;
  PatchArgs n{};
  return !patch_geometry(N, dstH, dstW, 128, true, n) || n.TP * 4 < 128 * 3 || n.NPOS * 2 > n.TP * g_patch_halo2 ||
         (int64_t)n.NT * 10 >= (int64_t)2 * a.NT * 11;
}
static bool patch_pick_wide(PatchUse use, int N, int dstH, int dstW, int srcC, int Ng, PatchShape& shape, PatchArgs& geo) {
  const int64_t wanted = (int64_t)N * dstH * dstW * Ng;
  for (int bn = 256; bn >= 128; bn /= 2) {
    if (Ng % bn != 0 || wanted * 20 < (int64_t)17 * 256 * 256 * bn) continue;  // (fewer than a round's)
    PatchArgs a{};
    if (!patch_geometry(N, dstH, dstW, 256, true, a, PATCH_WIDE_MAX_POS)) continue;
    // as few tiles with a fifth fewer staged positions (wide maps: 16 x 16 pixels for 2 x 128; 128 -> 128 channels at 64 x 128, one full
    // round, forward and data gradient 1.02 and 1.06 of the narrow tiles' time -> 0.98 and 1.01)
    for (int tc = 64; tc >= 8; tc /= 2) {
      PatchArgs b{};
      if (tc < dstW && patch_geometry_of(N, dstH, dstW, tc, 256, b, PATCH_WIDE_MAX_POS) && b.NT <= a.NT && b.NPOS * 5 <= a.NPOS * 4) a = b;
    }
    if ((int64_t)a.TI * (dstH + 2) * (dstW + 2) * srcC >= (int64_t)1 << 30) continue;  // 32-bit offsets within a tile's images
    if (!patch_wide_pays(use, N, dstH, dstW, srcC, bn, wanted, a, (int64_t)a.NT * (Ng / bn))) continue;
    const auto fits = [&] { return conv_patch_wide_lds(bn, (a.TI * a.SR * a.row_pitch + 15) / 16 * 8) <= 160 * 1024; };
    a.row_pitch = patch_row_pitch(a, 1, 80, PATCH_WIDE_MAX_POS);
    if (!fits()) a.row_pitch = a.SC * 80;
    if (!fits()) continue;
    shape = PatchShape{4, 1, bn, 1, true};
    geo = a;
    return true;
  }
  return false;
}
static bool patch_pick(int dt, bool split32, PatchUse use, int N, int dstH, int dstW, int srcC, int Ng, int R, int S, int stride,
                       PatchShape& shape, PatchArgs& geo) {
  if (R != 3 || S != 3 || stride != 1) return false;
  if (srcC % (dt == DT_F32 ? 16 : 32) != 0 || Ng % 64 != 0) return false;
  if (dt != DT_F32 && patch_pick_wide(use, N, dstH, dstW, srcC, Ng, shape, geo)) return true;
  // (Split32: 128 x 128 tiles take the LDS of a CU alone, and a layer of 128 channels at 262 144 pixels 515 us with them, 445 without)
  const int wide = Ng % 128 == 0 && !split32 ? 128 : 64;
  // What is left: fp32, and in 16 bits few pixels or little depth.  Candidates, largest first.  Two co-resident blocks per CU cover
  // each other's prologue, barriers and epilogue, and measured better here than one block of twice the size at every layer of the
  // benchmark networks, so the first candidate that gives g_patch_fill (two per CU) blocks is taken, else the one with the most blocks.
  const PatchShape cand[3] = {{2, 1, wide, 1, false}, {2, 1, 64, 1, false}, {1, 1, 64, 1, false}};
  int best = -1;
  int64_t best_blocks = 0;
  PatchArgs best_geo{};
  for (int i = 0; i < 3; ++i) {
    if (!((g_patch_shapes >> i) & 1)) continue;
    if (i == 1 && wide == 64) continue;  // same as candidate 0
    const int cap = 64 * cand[i].mi / cand[i].subt;
    PatchArgs a{};
    if (!patch_geometry(N, dstH, dstW, cap, dt != DT_F32 || split32, a)) continue;
    if (a.TP * 4 < cap * 3) continue;  // tile rows poorly used
    if (a.NPOS * 2 > a.TP * g_patch_halo2) continue;  // almost only halo: the staged patch costs more than it saves
    const int64_t blocks = (int64_t)((a.NT + cand[i].subt - 1) / cand[i].subt) * (Ng / cand[i].bn);
    if (blocks > best_blocks) { best = i; best_blocks = blocks; best_geo = a; }
    if (blocks >= g_patch_fill) break;
  }
  if (best < 0 || best_blocks < g_patch_min_blocks) return false;
  shape = cand[best];
  geo = best_geo;
  // still short of a block per CU: split the channel chunks over blockIdx.z (at least four chunks per range)
  const int nchunks = srcC / (dt == DT_F32 ? 16 : 32);
  int splits = 1;
  // fp32, smallest shape (one MFMA tile per wavefront, a barrier every 8 MFMAs): two co-resident blocks per CU
  // cover each other's barrier and LDS waits, which is worth the partial sums (measured 96 -> 84 us on 512->512 at 4x4)
  const int target = (shape.mi == 1 && dt == DT_F32) ? g_patch_target_small : 256;
  if (g_patch_split && best_blocks < target) {
    splits = (int)((target + best_blocks - 1) / best_blocks);
    if (splits > nchunks / 4) splits = nchunks / 4;
    if (splits > 4) splits = 4;
    if (splits < 1) splits = 1;
  }
  geo.split32 = split32;
  const int pos_bytes = split32 ? Frag<Split32>::PITCH * 2 : Frag<bf16_t>::PITCH * 2;
  geo.row_pitch = patch_row_pitch(geo, shape.subt, pos_bytes);
  // (not padded where that takes the room of a block that the registers leave and the grid has: 64 -> 64 channels over 70 000 pixels of
  // 50 x 50 maps in fp16, two blocks a CU with padded rows, three without, two layers forward 41 -> 33 us, data gradients 42 -> 33.5;
  // where a CU gets two blocks at most the padding stays: a step of 256 and 512 channels on 8 x 8 and 4 x 4 maps, batch 256, 701 -> 682)
  const int held = (int)std::min<int64_t>(split32 ? shape.mi == 1 ? 3 : 2 : shape.bn == 64 ? 3 : 2, (best_blocks + 255) / 256);
  if (patch_blocks_per_cu(geo, geo.row_pitch, shape.subt, shape.bn, pos_bytes) <
      std::min(held, patch_blocks_per_cu(geo, geo.SC * pos_bytes, shape.subt, shape.bn, pos_bytes)) ||
      (geo.TC != 8 && geo.TC != 4 && patch_weights_missed(dt, shape.mi, geo.NT, srcC, Ng)))
    geo.row_pitch = geo.SC * pos_bytes;
  geo.chunks_per_split = (nchunks + splits - 1) / splits;
  shape.splits = (nchunks + geo.chunks_per_split - 1) / geo.chunks_per_split;  // no empty ranges
  return true;
}

template <class T, class X, int BN, int MI, int SUBT, bool FOLD>
static void launch_patch_v(hipStream_t st, const void* src, const void* wmat, const float* bias, const void* addend, void* out,
                           float* partial, float* stat_partial, int splits, const PatchArgs& a_in) {
  PatchArgs a = a_in;
  dim3 grid((a.NT + SUBT - 1) / SUBT, a.Ng / BN, splits), block(256);
  // The patch buffers are sized for this layer's tile (its staged rows times the row pitch), not for the largest one,
  // so that the 64-channel shapes fit three blocks per CU on most layers.  The epilogue reuses the buffers and the
  // weight stages: they must hold its fp32 tile and the 16 KB of the channel-sum combine.
  constexpr size_t sm_max = patch_smem_max<X>(BN, SUBT);
  constexpr int64_t PITCH_E = Frag<X>::PITCH, ES = sizeof(typename Frag<X>::E);
  const int64_t epi_bytes = std::max<int64_t>((int64_t)32 * MI * (BN + 4) * 4, 16384);
  int64_t pe = ((int64_t)SUBT * a.TI * a.SR * a.row_pitch + 15) / 16 * 16 / ES;
  const int64_t need = (epi_bytes - (int64_t)3 * BN * PITCH_E * ES + 1) / 2;  // bytes per buffer
  if (pe * ES < need) pe = (need + 15) / 16 * 16 / ES;
  if (pe > (int64_t)SUBT * PATCH_MAX_POS * PITCH_E) pe = (int64_t)SUBT * PATCH_MAX_POS * PITCH_E;
  a.patch_elems = (int)pe;
  // from the shape only: weights of at least g_patch_xcd_wbytes that at most g_patch_xcd_rows row tiles share
  a.xcd_group = g_patch_xcd_wbytes > 0 && (int64_t)9 * a.srcC * a.Ng * (int64_t)sizeof(T) >= g_patch_xcd_wbytes &&
                (int)grid.x <= g_patch_xcd_rows && (grid.y * grid.z) % 8 == 0;
  a.row_blocks = (int)grid.x;
  if (!a.xcd_group && grid.y * grid.z >= 2 && grid.x >= 64) {  // (from the shape only)
    a.xcd_group = 2;
    grid.x = (grid.x + 7) / 8 * 8;
  }
  const size_t sm = patch_smem_bytes<X>(BN, SUBT, pe);
  if constexpr (!FOLD) {
    if (a.eval && splits == 1) {
      static bool eval_attr = false;
      if (!eval_attr) {
        (void)hipFuncSetAttribute((const void*)conv3x3_patch_kernel<T, X, BN, MI, SUBT, 0, false, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm_max);
        eval_attr = true;
      }
      OSEQ_LAUNCH((conv3x3_patch_kernel<T, X, BN, MI, SUBT, 0, false, true>), grid, block, sm, st, (const T*)src, (const T*)wmat, bias,
                  (const T*)addend, (T*)out, (float*)nullptr, (float*)nullptr, a);
      return;
    }
    if (a.bn_sums && splits == 1) {
      static bool sums_attr = false;
      if (!sums_attr) {
        (void)hipFuncSetAttribute((const void*)conv3x3_patch_kernel<T, X, BN, MI, SUBT, 2>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm_max);
        sums_attr = true;
      }
      OSEQ_LAUNCH((conv3x3_patch_kernel<T, X, BN, MI, SUBT, 2>), grid, block, sm, st, (const T*)src, (const T*)wmat, bias,
                  (const T*)addend, (T*)out, (float*)nullptr, stat_partial, a);
      return;
    }
  }
  static bool attr_done = false;
  if (!attr_done) {
    (void)hipFuncSetAttribute((const void*)conv3x3_patch_kernel<T, X, BN, MI, SUBT, 0, FOLD>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm_max);
    (void)hipFuncSetAttribute((const void*)conv3x3_patch_kernel<T, X, BN, MI, SUBT, 1, FOLD>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm_max);
    attr_done = true;
  }
  // the variant that also adds up what it stores (BatchNorm statistics) is a separate instantiation, so that the
  // plain one carries none of its registers
  if (splits == 1 && stat_partial)
    OSEQ_LAUNCH((conv3x3_patch_kernel<T, X, BN, MI, SUBT, 1, FOLD>), grid, block, sm, st, (const T*)src, (const T*)wmat, bias,
                       (const T*)addend, (T*)out, (float*)nullptr, stat_partial, a);
  else
    OSEQ_LAUNCH((conv3x3_patch_kernel<T, X, BN, MI, SUBT, 0, FOLD>), grid, block, sm, st, (const T*)src, (const T*)wmat, bias,
                       (const T*)addend, (T*)out, splits > 1 ? partial : (float*)nullptr, (float*)nullptr, a);
}

template <class T, class X>
static void launch_patch_t(hipStream_t st, const void* src, const void* wmat, const float* bias, const void* addend, void* out,
                           float* partial, float* stat_partial, const PatchShape& v, const PatchArgs& a) {
  const int sp = v.splits;
  if constexpr (sizeof(T) == 2) {
    if (a.fold) {  // (16-bit modes only)
      if (v.mi == 2) {
        if (v.bn == 128) launch_patch_v<T, X, 128, 2, 1, true>(st, src, wmat, bias, addend, out, partial, stat_partial, sp, a);
        else launch_patch_v<T, X, 64, 2, 1, true>(st, src, wmat, bias, addend, out, partial, stat_partial, sp, a);
      } else {
        launch_patch_v<T, X, 64, 1, 1, true>(st, src, wmat, bias, addend, out, partial, stat_partial, sp, a);
      }
    }
  }
  if (sizeof(T) != 2 || !a.fold) {
    if (v.mi == 2) {
      if constexpr (!std::is_same_v<X, Split32>) {
        if (v.bn == 128) launch_patch_v<T, X, 128, 2, 1, false>(st, src, wmat, bias, addend, out, partial, stat_partial, sp, a);
      }
      if (v.bn == 64) launch_patch_v<T, X, 64, 2, 1, false>(st, src, wmat, bias, addend, out, partial, stat_partial, sp, a);
    } else {
      launch_patch_v<T, X, 64, 1, 1, false>(st, src, wmat, bias, addend, out, partial, stat_partial, sp, a);
    }
  }
  if (sp > 1)
    launch_splitk_epilogue<T>(st, partial, sp, (int64_t)a.N * a.dstH * a.dstW, a.Ng, a.eval ? nullptr : bias, addend, a.amask, out,
                              stat_partial, a.relu, a.eval ? bias : nullptr);
}

static void launch_patch(hipStream_t st, int dt, const void* src, const void* wmat, const float* bias, const void* addend, void* out,
                         float* partial, float* stat_partial, const PatchShape& v, const PatchArgs& a) {
  if (v.wide) launch_conv_patch_wide(st, dt, src, wmat, bias, addend, out, stat_partial, v.bn, a);
  else if (dt == DT_F32 && a.split32) launch_patch_t<float, Split32>(st, src, wmat, bias, addend, out, partial, stat_partial, v, a);
  else if (dt == DT_F32) launch_patch_t<float, float>(st, src, wmat, bias, addend, out, partial, stat_partial, v, a);
  else if (dt == DT_BF16) launch_patch_t<bf16_t, bf16_t>(st, src, wmat, bias, addend, out, partial, stat_partial, v, a);
  else launch_patch_t<f16_t, f16_t>(st, src, wmat, bias, addend, out, partial, stat_partial, v, a);
}

static constexpr int g_igemm_spread = 1;                         // compile-time switch
constexpr size_t kSpreadLds = 84 * 1024;        // more than half of the 160 KB of LDS per CU

// Rows per block.  A 256-row tile was tried for layers with many pixels: it needs 348-380 registers, so one wavefront
// per SIMD, where two 128-row blocks share a CU; the strided 3x3 layers of the bottleneck network at batch 4096 (bf16)
// take 716 / 646 us with it and 551 / 520 without, the fp32 network on 512 x 512 images 166.4 against 163.2 ms a step.
constexpr int IGEMM_BM = 128;

template <class T, class X, int MODE>
static void launch_igemm_t(hipStream_t st, const void* src, const void* wmat, const float* bias, const void* addend, void* out,
                           float* partial, float* stat_partial, int splits, const IGemmArgs& a0) {
  IGemmArgs a = a0;
  const int bk = Frag<X>::BK;
  a.kt_per_split = ceil_div(a.Kg / bk, splits);
  // 64 channels per block where 128 leave CUs without one, or two in turn (us, 128 -> 64: inference at batch 16, 18 layers, 2 x 4 x 9
  // blocks 10.4 -> 8.0, 32 x 1 x 2 11.8 -> 8.7), or where four classes of different depth share few (32 x 2 x 4 23.6 -> 20.7); a
  // block per CU of equal depth keeps them (64 x 4 of 144 depth tiles 68.8 -> 74).  fp32 forward: 64 x 2 blocks of 8 depth tiles
  // 16.9 -> 12.6, 32 x 1 x 4 20.6 -> 15.9, of nineteen layers none slower.
  const int64_t blocks128 = (int64_t)ceil_div(a.M, IGEMM_BM) * (a.Ng / 128) * (a.cls ? 4 : splits);
  constexpr bool S32 = std::is_same_v<X, Split32>;
  const bool wide = a.Ng % 128 == 0 && !S32 && blocks128 >= (a.cls ? 512 : 256);
  dim3 grid(ceil_div(a.M, IGEMM_BM), a.Ng / (wide ? 128 : 64), a.cls ? 4 : splits), block(256);  // cls: never split
  // A grid of at most one block per CU asks for more than half of a CU's LDS, so that no CU takes two blocks
  // while another idles.
  const bool spread = g_igemm_spread && (int64_t)grid.x * grid.y * grid.z <= 256;
#define IGEMM_LAUNCH(BM_, BN_, SPLIT_)                                                                                   \
  {                                                                                                                      \
    constexpr size_t sm_ = igemm_smem_bytes<X, BM_, BN_>();                                                              \
    constexpr size_t big_ = sm_ > kSpreadLds ? sm_ : kSpreadLds;                                                         \
    static bool attr_ = false;                                                                                           \
    if (!attr_) {                                                                                                        \
      (void)hipFuncSetAttribute((const void*)conv_igemm_kernel<T, X, BM_, BN_, MODE_, SPLIT_>,                               \
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)big_);                                  \
      attr_ = true;                                                                                                      \
    }                                                                                                                    \
    OSEQ_LAUNCH((conv_igemm_kernel<T, X, BM_, BN_, MODE_, SPLIT_>), grid, block, spread ? big_ : sm_, st,             \
                       (const T*)src, (const T*)wmat, bias, (const T*)addend, (T*)out, partial, stat_partial, a);        \
  }
  if (splits > 1) {
    // (the depth ranges are stored as they are: the forward and the inference instantiation would be the same kernel)
    constexpr int MODE_ = MODE == IG_EVAL ? IG_FWD : MODE;
    if constexpr (!S32) { if (wide) IGEMM_LAUNCH(128, 128, true) }
    if (!wide) IGEMM_LAUNCH(128, 64, true)
    launch_splitk_epilogue<T>(st, partial, splits, a.M, a.Ng, MODE == IG_EVAL ? nullptr : bias, addend, a.amask, out, stat_partial,
                              a.relu, MODE == IG_EVAL ? bias : nullptr);
  } else {
    constexpr int MODE_ = MODE;
    if constexpr (!S32) { if (wide) IGEMM_LAUNCH(128, 128, false) }
    if (!wide) IGEMM_LAUNCH(128, 64, false)
  }
#undef IGEMM_LAUNCH
}

template <int MODE>
static void launch_igemm(hipStream_t st, int dt, bool split32, const void* src, const void* wmat, const float* bias, const void* addend,
                         void* out, float* partial, float* stat_partial, int splits, const IGemmArgs& a) {
  if (dt == DT_F32 && split32) launch_igemm_t<float, Split32, MODE>(st, src, wmat, bias, addend, out, partial, stat_partial, splits, a);
  else if (dt == DT_F32) launch_igemm_t<float, float, MODE>(st, src, wmat, bias, addend, out, partial, stat_partial, splits, a);
  else if (dt == DT_BF16) launch_igemm_t<bf16_t, bf16_t, MODE>(st, src, wmat, bias, addend, out, partial, stat_partial, splits, a);
  else launch_igemm_t<f16_t, f16_t, MODE>(st, src, wmat, bias, addend, out, partial, stat_partial, splits, a);
}

// depth splits of a GEMM with M rows, Ng columns and depth Kg: from the shape only
static int igemm_splits(int dt, int64_t M, int Ng, int Kg) {
  const int bk = dt == DT_F32 ? 16 : 32;
  const int64_t blocks = ((M + 127) / 128) * (Ng / (Ng % 128 == 0 ? 128 : 64));
  if (blocks >= 256) return 1;
  int64_t s = (512 + blocks - 1) / blocks;
  const int64_t most = (Kg / bk) / 8;  // at least eight depth tiles per range
  if (s > most) s = most;
  if (s > 32) s = 32;
  return (int)(s < 1 ? 1 : s);
}
// fp32 with the operands split (split32.h): data gradients always; forward passes of 131 072 output pixels or more.  Below,
// the forward sums keep the rounding of the fp32 MFMA although the split is as exact and faster there too (64 -> 128 channels at
// 32 768 pixels 48 -> 33 us): another rounding decides some ReLUs and maxima within 1e-6 of a tie the other way, each of which
// moves the gradients below it by its share of their sums, and over few pixels that is no small one -- a step of the 11-layer
// network at batch 128 moves by 4e-4 to 9e-3, at 512 x 512 by 2e-5 -- where the same decisions reproduce it to 1e-6.
// So the line is a choice between those two and no bound of speed or accuracy; a sample's sums are rounded the one way in a batch
// below it and the other way in one above.
static bool fwd_split32(int dt, const ConvGeom& g) { return dt == DT_F32 && (int64_t)g.N * g.P * g.Q >= 131072; }
static bool fwd_ws3x3(int dt, const ConvGeom& g) { return conv_ws3x3_ok(dt, g.N, g.P, g.Q, g.C, g.K, g.R, g.S, g.stride); }
static bool dgrad_ws3x3(int dt, const ConvGeom& g) { return conv_ws3x3_ok(dt, g.N, g.H, g.W, g.K, g.C, g.R, g.S, g.stride); }
// (a layer that takes the weights-stationary 3x3 kernel never splits its depth, nor would the kernel that takes it when
// something is done to its result: it has at least 1024 tiles of 128 pixels)
int conv_mfma_fwd_splits(int dt, const ConvGeom& g) {
  PatchShape v; PatchArgs pa{};
  if (fwd_ws3x3(dt, g)) return 1;
  if (conv_pointwise_fwd_ok(dt, g)) return 1;
  if (patch_pick(dt, fwd_split32(dt, g), PATCH_FWD, g.N, g.P, g.Q, g.C, g.K, g.R, g.S, g.stride, v, pa)) return v.splits;
  return igemm_splits(dt, (int64_t)g.N * g.P * g.Q, g.K, g.R * g.S * g.C);
}
// stride 2, even image, at most 3x3: the data gradient runs as four parity-class GEMMs in one launch
static constexpr int g_dgrad_classes = 1;  // compile-time switch
static bool dgrad_by_classes(const ConvGeom& g) {
  return g_dgrad_classes && g.stride == 2 && g.H % 2 == 0 && g.W % 2 == 0 && g.R <= 3 && g.S <= 3;
}
int conv_mfma_dgrad_splits(int dt, const ConvGeom& g) {
  PatchShape v; PatchArgs pa{};
  if (dgrad_ws3x3(dt, g)) return 1;
  if (conv_pointwise_dgrad_ok(dt, g)) return 1;
  if (patch_pick(dt, dt == DT_F32, PATCH_DGRAD, g.N, g.H, g.W, g.K, g.C, g.R, g.S, g.stride, v, pa)) return v.splits;
  if (dgrad_by_classes(g)) return 1;
  return igemm_splits(dt, (int64_t)g.N * g.H * g.W, g.C, g.R * g.S * g.K);
}

int conv_patch_blocks_per_cu(int dt, const ConvGeom& g, bool unpadded) {
  PatchShape v; PatchArgs a{};
  const bool split32 = fwd_split32(dt, g);
  if (!patch_pick(dt, split32, PATCH_FWD, g.N, g.P, g.Q, g.C, g.K, g.R, g.S, g.stride, v, a) || v.wide) return 0;
  const int pos_bytes = (split32 ? Frag<Split32>::PITCH : Frag<bf16_t>::PITCH) * 2;
  return patch_blocks_per_cu(a, unpadded ? a.SC * pos_bytes : a.row_pitch, v.subt, v.bn, pos_bytes);
}

bool conv_patch_rows_padded(int dt, const ConvGeom& g) {
  PatchShape v; PatchArgs a{};
  const bool split32 = fwd_split32(dt, g);
  return patch_pick(dt, split32, PATCH_FWD, g.N, g.P, g.Q, g.C, g.K, g.R, g.S, g.stride, v, a) &&
         a.row_pitch > a.SC * (split32 ? Frag<Split32>::PITCH : Frag<bf16_t>::PITCH) * 2;
}

bool conv_mfma_fwd_ok(int dt, const ConvGeom& g) {
  const int bk = dt == DT_F32 ? 16 : 32;
  return g.C % bk == 0 && g.K % 64 == 0;
}
bool conv_mfma_dgrad_ok(int dt, const ConvGeom& g) {
  const int bk = dt == DT_F32 ? 16 : 32;
  return g.K % bk == 0 && g.C % 64 == 0;
}

// Row blocks over which the forward path produces the per-channel sums for BatchNorm: the blocks of the convolution
// kernel, or of the kernel that adds the depth ranges when the depth is split.  From the layer shape only.
int conv_mfma_fwd_stat_blocks(int dt, const ConvGeom& g, bool bias) {
  PatchShape pv; PatchArgs pa{};
  const int64_t M = (int64_t)g.N * g.P * g.Q;
  if (conv_pointwise_fwd_ok(dt, g)) return conv_pointwise_stat_blocks(g);
  if (!bias && fwd_ws3x3(dt, g)) return conv_ws3x3_stat_blocks(g);
  if (patch_pick(dt, fwd_split32(dt, g), PATCH_FWD, g.N, g.P, g.Q, g.C, g.K, g.R, g.S, g.stride, pv, pa))
    return pv.splits > 1 ? ceil_div(M, split_epi_rows(M, g.K)) : (pa.NT + pv.subt - 1) / pv.subt;
  if (igemm_splits(dt, M, g.K, g.R * g.S * g.C) > 1) return ceil_div(M, split_epi_rows(M, g.K));
  return ceil_div(M, IGEMM_BM);
}

// stat_partial: null, or [conv_mfma_fwd_stat_blocks][2][C_out] floats receiving per-block sums and sums of squares
// of the stored outputs
// the 1x1 streaming kernels and, in the 16-bit modes, the 3x3 patch kernel
bool conv_fold_fwd_ok(int dt, const ConvGeom& g) {
  if (conv_pointwise_fwd_ok(dt, g)) return conv_pointwise_fold_ok(dt, g);
  PatchShape pv; PatchArgs pa{};
  return dt != DT_F32 && patch_pick(dt, fwd_split32(dt, g), PATCH_FWD, g.N, g.P, g.Q, g.C, g.K, g.R, g.S, g.stride, pv, pa);
}

void launch_conv_fwd_mfma(hipStream_t st, int dt, const void* x, const void* w, const float* bias, void* out,
                          float* partial, float* stat_partial, int splits, const ConvGeom& g, int relu, const float* fold,
                          const ConvEval& ev) {
  PatchShape pv; PatchArgs pa{};
  if (conv_pointwise_fwd_ok(dt, g)) {
    launch_conv_fwd_pointwise(st, dt, x, w, bias, out, stat_partial, g, relu, fold, ev);
    return;
  }
  if (!ev.affine && !bias && !relu && fwd_ws3x3(dt, g)) {
    launch_conv_fwd_ws3x3(st, dt, x, w, out, stat_partial, g, fold);
    return;
  }
  const bool eval = ev.affine != nullptr;
  if (patch_pick(dt, fwd_split32(dt, g), eval ? PATCH_EVAL : PATCH_FWD, g.N, g.P, g.Q, g.C, g.K, g.R, g.S, g.stride, pv, pa)) {
    pa.N = g.N; pa.srcH = g.H; pa.srcW = g.W; pa.srcC = g.C; pa.dstH = g.P; pa.dstW = g.Q; pa.Ng = g.K;
    pa.pad = g.pad; pa.flip = 0; pa.relu = relu;
    pa.fold = dt == DT_F32 ? nullptr : fold;
    pa.eval = eval;
    launch_patch(st, dt, x, w, eval ? ev.affine : bias, ev.skip, out, partial, stat_partial, pv, pa);
    return;
  }
  IGemmArgs a{g.H, g.W, g.C, g.P, g.Q, g.N * g.P * g.Q, g.K, g.R * g.S * g.C, g.R, g.S, g.stride, g.pad, relu, 0};
  if (eval) launch_igemm<IG_EVAL>(st, dt, fwd_split32(dt, g), x, w, ev.affine, ev.skip, out, partial, nullptr, splits, a);
  else launch_igemm<IG_FWD>(st, dt, fwd_split32(dt, g), x, w, bias, nullptr, out, partial, stat_partial, splits, a);
}

// the 1x1 kernels, whose rows are pixels in order
bool conv_dgrad_image_addend_ok(int dt, const ConvGeom& g) {
  return conv_pointwise_dgrad_ok(dt, g) && g.stride == 1 && (int64_t)g.N * g.H * g.W < (int64_t)1 << 32;
}

// Row blocks over which the data gradient can produce the sums of the BatchNorm backward in front of the layer, 0: it cannot.  (More
// rows than the finishing kernel takes without a fold are not worth it.)
int conv_dgrad_sum_blocks(int dt, const ConvGeom& g) {
  PatchShape pv; PatchArgs pa{};
  if (conv_pointwise_dgrad_ok(dt, g) || dgrad_ws3x3(dt, g)) return 0;
  if (!patch_pick(dt, dt == DT_F32, PATCH_DGRAD, g.N, g.H, g.W, g.K, g.C, g.R, g.S, g.stride, pv, pa) || pv.splits > 1) return 0;
  const int blocks = (pa.NT + pv.subt - 1) / pv.subt;
  return bn_stats_fold_rows(blocks) > 0 ? 0 : blocks;
}

// wt: the (C_in, kh, kw, C_out) transpose of the weights, in the compute type
void launch_conv_dgrad_mfma(hipStream_t st, int dt, const void* dz, const void* wt, const void* addend,
                            const void* addend_mask, bool addend_per_image, void* dx, float* partial, int splits, const ConvGeom& g,
                            const DgradSums& sums) {
  PatchShape pv; PatchArgs pa{};
  const uint8_t* amask = addend ? (const uint8_t*)addend_mask : nullptr;
  if (conv_pointwise_dgrad_ok(dt, g)) {
    launch_conv_dgrad_pointwise(st, dt, dz, wt, addend, amask, addend_per_image, dx, g);
    return;
  }
  if (!addend && dgrad_ws3x3(dt, g)) {
    launch_conv_dgrad_ws3x3(st, dt, dz, wt, dx, g);
    return;
  }
  if (patch_pick(dt, dt == DT_F32, PATCH_DGRAD, g.N, g.H, g.W, g.K, g.C, g.R, g.S, g.stride, pv, pa)) {
    pa.N = g.N; pa.srcH = g.P; pa.srcW = g.Q; pa.srcC = g.K; pa.dstH = g.H; pa.dstW = g.W; pa.Ng = g.C;
    pa.pad = g.R - 1 - g.pad; pa.flip = 1; pa.relu = 0; pa.amask = amask;
    if (sums.partial) {
      pa.bn_sums = 1; pa.relu = sums.relu;
      launch_patch(st, dt, dz, wt, sums.stats, sums.z, dx, partial, sums.partial, pv, pa);
      return;
    }
    launch_patch(st, dt, dz, wt, nullptr, addend, dx, partial, nullptr, pv, pa);
    return;
  }
  IGemmArgs a{g.P, g.Q, g.K, g.H, g.W, g.N * g.H * g.W, g.C, g.R * g.S * g.K, g.R, g.S, g.stride, g.pad, 0, 0};
  a.amask = amask;  // (only stride-1 layers ever get one: the identity shortcut of a block)
  if (dgrad_by_classes(g)) {
    a.cls = 1; a.fullH = g.H; a.fullW = g.W;
    a.dstH = g.H / 2; a.dstW = g.W / 2; a.M = g.N * a.dstH * a.dstW;
    for (int c = 0; c < 4; ++c) {
      const int ph = c >> 1, pw = c & 1;
      a.taps[c] = 0; a.ntaps[c] = 0;
      for (int r = 0; r < g.R; ++r)
        for (int s2 = 0; s2 < g.S; ++s2)
          if (((ph + g.pad - r) & 1) == 0 && ((pw + g.pad - s2) & 1) == 0)
            a.taps[c] |= (r * g.S + s2) << (8 * a.ntaps[c]++);
    }
    launch_igemm<IG_DGRAD>(st, dt, true, dz, wt, nullptr, addend, dx, nullptr, nullptr, 1, a);
    return;
  }
  launch_igemm<IG_DGRAD>(st, dt, true, dz, wt, nullptr, addend, dx, partial, nullptr, splits, a);
}

// (C_out, R*S, C_in) fp32 master weights -> (C_in, R*S, C_out) in the compute type, for all layers of a batch in one
// launch: a block transposes one 32x32 (C_out x C_in) tile of one filter tap through LDS, so that both the reads
// (along C_in) and the writes (along C_out) are contiguous.
template <class T>
__global__ void __launch_bounds__(256) weight_transpose_kernel(const float* __restrict__ wbase, T* __restrict__ wtbase,
                                                               TransposeBatch b) {
  __shared__ float tile[32][33];
  int j = 0;
  while (j + 1 < b.n && (int)blockIdx.x >= b.job[j + 1].first_block) ++j;
  const TransposeJob jb = b.job[j];
  const int tiles_k = (jb.K + 31) / 32, tiles_c = (jb.C + 31) / 32;
  const int local = blockIdx.x - jb.first_block;
  const int tc = local % tiles_c, t2 = local / tiles_c;
  const int tk = t2 % tiles_k, rs = t2 / tiles_k;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const float* w = wbase + jb.w_off;
  T* wt = wtbase + jb.w_off;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int k = tk * 32 + ty + i * 8, c = tc * 32 + tx;
    if (k < jb.K && c < jb.C) tile[ty + i * 8][tx] = w[((int64_t)k * jb.RS + rs) * jb.C + c];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = tc * 32 + ty + i * 8, k = tk * 32 + tx;
    if (c < jb.C && k < jb.K) wt[((int64_t)c * jb.RS + rs) * jb.K + k] = from_f32<T>(tile[tx][ty + i * 8]);
  }
}

// jobs: first_block is filled in here
void launch_weight_transposes(hipStream_t st, int dt, const float* wbase, void* wtbase, const TransposeJob* jobs, int njobs) {
  for (int j0 = 0; j0 < njobs; j0 += TransposeBatch::MAX_JOBS) {
    TransposeBatch b{};
    b.n = njobs - j0 < TransposeBatch::MAX_JOBS ? njobs - j0 : TransposeBatch::MAX_JOBS;
    int blocks = 0;
    for (int j = 0; j < b.n; ++j) {
      b.job[j] = jobs[j0 + j];
      b.job[j].first_block = blocks;
      blocks += b.job[j].RS * ((b.job[j].K + 31) / 32) * ((b.job[j].C + 31) / 32);
    }
    if (blocks == 0) continue;
    if (dt == DT_F32) OSEQ_LAUNCH(weight_transpose_kernel<float>, dim3(blocks), dim3(256), 0, st, wbase, (float*)wtbase, b);
    else if (dt == DT_BF16) OSEQ_LAUNCH(weight_transpose_kernel<bf16_t>, dim3(blocks), dim3(256), 0, st, wbase, (bf16_t*)wtbase, b);
    else OSEQ_LAUNCH(weight_transpose_kernel<f16_t>, dim3(blocks), dim3(256), 0, st, wbase, (f16_t*)wtbase, b);
  }
}

// ------------------------------------------------------------------------------------------------------------
// Weight gradient:  dw[k][tap][c] = sum over pixels m of dz[m][k] * x_tap[m][c]   (fp32 result)
// One block owns a (BM output channels) x (BN input channels) tile of ONE filter tap and a fixed chunk of the
// pixel range (blockIdx.z); chunks are summed afterwards in order, so the result does not depend on scheduling.
// Both operands arrive pixel-major (the reduction index is the slow one), but an MFMA lane wants consecutive
// reduction elements.  The tiles are stored in LDS as loaded (16-byte chunks, [pixel][channel]; fp32 as three such tiles, one
// per bf16 plane: split32.h) and read with the transposing LDS read of gfx950 (ds_read_b64_tr_b16).
// ------------------------------------------------------------------------------------------------------------
struct WGradArgs {
  int H, W, C, K, R, S, stride, pad, P, Q;
  int pixels, chunk;  // chunk: pixels per blockIdx.z, a multiple of the depth tile
  FastDiv divQ, divPQ;
  const float* fold;  // FOLD: x is the z of a BatchNorm + ReLU, this its [4][C] statistics tensor; the pieces of x become
                      // the activation (scale, shift, ReLU, one rounding) on their way to LDS
  int xcd_group;      // 1: the tiles of a pixel range share an XCD (see the kernel); ranges: the number of pixel ranges
  int ranges;
};

// WGM x WGN wavefronts (wave tile BM / WGM x BN / WGN); the 256 x 256 tile of the 1x1 layers with many pixels runs 2 x 4
// wavefronts, two per SIMD, one block per CU: every operand element then crosses from L2 to a CU half as often as with
// 128 x 128 tiles (a 1024 x 256 weight gradient over 262 144 pixels moves 1.07 GB instead of 2.1 GB that way).
template <class T, int BM, int BN, int WGM>
constexpr size_t wgrad_lds_bytes() {
  return (size_t)3 * (sizeof(T) == 4 ? 3 * 16 : 32) * (BM + BN + 2 * 16) * 2;
}

// PW: a 1x1 layer with unit stride and no padding -- pixel m of x is row m, as it is of dz; the loads of a depth tile
// are then one uniform base per tensor plus per-thread offsets that never change (the general path divides every
// pixel index into image, row and column and multiplies it back into an address, a few dozen quarter-rate integer
// multiplies per depth tile that the 256 x 256 tile, with one block per CU, has nobody to hide behind).
// NTL (PW only): 1 / 2: the rows of dz / of x are read by this block's tile alone (one input- / output-channel tile) and
// are loaded non-temporally
template <class T, int BM, int BN, int WGM = 2, int WGN = 2, bool FOLD = false, bool PW = false, int NTL = 0>
__global__ void __launch_bounds__(64 * WGM * WGN) conv_wgrad_kernel(const T* __restrict__ x, const T* __restrict__ dz,
                                                                    float* __restrict__ out, WGradArgs a) {
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int DEPTH = F32 ? 16 : 32;
  constexpr int NT = 64 * WGM * WGN;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int MI = WTM / 32, NI = WTN / 32;
  // one LDS stage, pixel-major as loaded: [PL][DEPTH][BM + pad] then [PL][DEPTH][BN + pad] (pad: 16 elements; PL: planes)
  typedef Frag<std::conditional_t<F32, Split32, T>> FR;
  typedef typename FR::E E;
  constexpr int PADE = 16, PL = F32 ? 3 : 1;
  constexpr int A_PL = DEPTH * (BM + PADE), A_ELEMS = PL * A_PL;
  constexpr int B_PL = DEPTH * (BN + PADE), B_ELEMS = PL * B_PL;
  constexpr int STAGE = A_ELEMS + B_ELEMS;
  extern __shared__ __attribute__((aligned(16))) unsigned char wgrad_smem[];
  E* lds = reinterpret_cast<E*>(wgrad_smem);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN, g = lane >> 5, l32 = lane & 31;
  // Block coordinates: (output-channel tile, tap and input-channel tile, pixel range).  xcd_group: the tiles
  // (and taps) of one pixel range all read the same rows of x and dz; workgroups go to the 8 XCDs round-robin by their linear
  // index and every XCD has an L2 of its own, so the tiles of a range are renumbered onto one XCD, which then fetches
  // those rows once.  The grid's z extent is the number of ranges rounded up to a multiple of 8.
  int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
  if (a.xcd_group) {
    const unsigned tiles = gridDim.x * gridDim.y;
    const unsigned lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const unsigned xcd = lin & 7u, slot = lin >> 3;
    const unsigned tile = slot % tiles;
    bz = (int)((slot / tiles) * 8u + xcd);
    bx = (int)(tile % gridDim.x); by = (int)(tile / gridDim.x);
    if (bz >= a.ranges) return;
  }
  const int k0 = bx * BM;
  const int ctiles = a.C / BN;
  const int tap = by / ctiles, c0 = (by - tap * ctiles) * BN;
  const int r = tap / a.S, s = tap - r * a.S;
  const int mbeg = bz * a.chunk;
  const int mend = mbeg + a.chunk < a.pixels ? mbeg + a.chunk : a.pixels;
  const int n = mend > mbeg ? (mend - mbeg + DEPTH - 1) / DEPTH : 0;
  const int K = a.K, C = a.C, H = a.H, W = a.W, cstride = a.stride, pad = a.pad;
  const FastDiv divQ = a.divQ, divPQ = a.divPQ;

  // staging: 16-byte chunks, rows = pixels (EV elements per chunk)
  constexpr int EV = 16 / (int)sizeof(T);
  constexpr int A_CH32 = DEPTH * (BM / EV) / NT, B_CH32 = DEPTH * (BN / EV) / NT;
  static_assert(A_CH32 >= 1 && B_CH32 >= 1, "tile too small for the block");
  Chunk ra[2][A_CH32], rb[2][B_CH32];
  unsigned va[2] = {0u, 0u}, vb[2] = {0u, 0u};  // validity bits of the pieces in flight, per generation

  // Loads are unconditional (pixels past the range or outside the image read pixel mbeg / the tensor start) and are
  // zeroed when written to LDS, so that later tiles' loads stay in flight during the MFMAs of the current one.
  auto tap_offset = [&](int n_, int p_, int q_, int64_t& off) -> bool {  // x offset of (image, row, col) under this tap
    const int ih = p_ * cstride + r - pad, iw = q_ * cstride + s - pad;
    const bool ok = ih >= 0 && ih < H && iw >= 0 && iw < W;
    off = ok ? (((int64_t)n_ * H + ih) * W + iw) * C : 0;
    return ok;
  };
  // PW: element offsets of a thread's pieces from the first row of a depth tile
  int offa[PW ? A_CH32 : 1], offb[PW ? B_CH32 : 1];
  if constexpr (PW) {
#pragma unroll
    for (int i = 0; i < A_CH32; ++i) {
      const int id = tid + i * NT, px = id / (BM / EV), kv = id % (BM / EV);
      offa[i] = px * K + k0 + kv * EV;
    }
#pragma unroll
    for (int i = 0; i < B_CH32; ++i) {
      const int id = tid + i * NT, px = id / (BN / EV), cv = id % (BN / EV);
      offb[i] = px * C + c0 + cv * EV;
    }
  }
  // CHK = 0: the tile is known to lie inside the range (every tile but a range's last one)
  auto gload = [&](auto G, auto CHKC, int t) {
    constexpr int p = decltype(G)::value;
    constexpr bool CHK = decltype(CHKC)::value != 0;
    const int mt = mbeg + t * DEPTH;
    unsigned ma = 0u, mb = 0u;
    if constexpr (PW) {
      const T* dzt = dz + (int64_t)mt * K;
      const T* xt = x + (int64_t)mt * C;
#pragma unroll
      for (int i = 0; i < A_CH32; ++i) {
        const int px = (tid + i * NT) / (BM / EV);
        const bool ok = !CHK || mt + px < mend;  // a row past the range reads the same piece of the range's first row
        const Chunk* pa = reinterpret_cast<const Chunk*>(ok ? dzt + offa[i] : dz + (int64_t)mbeg * K + (offa[i] - px * K));
        ra[p][i] = NTL == 1 ? __builtin_nontemporal_load(pa) : *pa;
        ma |= ok ? (1u << i) : 0u;
      }
#pragma unroll
      for (int i = 0; i < B_CH32; ++i) {
        const int px = (tid + i * NT) / (BN / EV);
        const bool ok = !CHK || mt + px < mend;
        const Chunk* pb = reinterpret_cast<const Chunk*>(ok ? xt + offb[i] : x + (int64_t)mbeg * C + (offb[i] - px * C));
        rb[p][i] = NTL == 2 ? __builtin_nontemporal_load(pb) : *pb;
        mb |= ok ? (1u << i) : 0u;
      }
      va[p] = ma; vb[p] = mb;
      return;
    }
#pragma unroll
    for (int i = 0; i < A_CH32; ++i) {
      const int id = tid + i * NT, px = id / (BM / EV), kv = id % (BM / EV);
      const int m = mt + px;
      const bool ok = m < mend;
      ra[p][i] = *reinterpret_cast<const Chunk*>(dz + (int64_t)(ok ? m : mbeg) * K + k0 + kv * EV);
      ma |= ok ? (1u << i) : 0u;
    }
#pragma unroll
    for (int i = 0; i < B_CH32; ++i) {
      const int id = tid + i * NT, px = id / (BN / EV), cv = id % (BN / EV);
      const int m = mt + px;
      const int mm = m < mend ? m : mbeg;
      const uint32_t n_ = divPQ.div((uint32_t)mm), rem = (uint32_t)mm - n_ * divPQ.d;
      const uint32_t p_ = divQ.div(rem), q_ = rem - p_ * divQ.d;
      int64_t off;
      const bool ok = tap_offset((int)n_, (int)p_, (int)q_, off) && m < mend;
      rb[p][i] = *reinterpret_cast<const Chunk*>(x + (ok ? off : 0) + c0 + cv * EV);
      mb |= ok ? (1u << i) : 0u;
    }
    va[p] = ma; vb[p] = mb;
  };
  // FOLD: a thread's pieces of x all cover the same EV channels, whose scale and shift it keeps in registers
  static_assert(NT % (BN / EV) == 0, "a thread's pieces of x must share their channels");
  float fsc[EV], fsh[EV];
  if (FOLD) {
    const int cv = tid % (BN / EV);
    load_f32<float, EV>(a.fold + 2 * C + c0 + cv * EV, fsc);
    load_f32<float, EV>(a.fold + 3 * C + c0 + cv * EV, fsh);
  }
  // fp32: half of the sum is made with dz negated (split32.h); within a range where that is long, from an even tile of the steady
  // state on (a test per tile in the pipelined loop: 58 -> 70 us for the 1x1 layers of the 512 x 512 network)
  const bool odd = F32 && (bz & 1) != 0;
  const int flip = F32 && n >= 16 ? wgrad_flip(n) & ~1 : 0;
  // t: the depth tile.  FULL (PW only): every piece of the tile is known to be valid
  auto sstore = [&](auto G, auto FULLC, int stage, int t) {
    constexpr int p = decltype(G)::value;
    constexpr bool FULL = PW && decltype(FULLC)::value != 0;
    E* sa = lds + stage * STAGE;
    E* sb = sa + A_ELEMS;
    // a piece, or zero, to its place in the tile (fp32: in its three planes)
    auto put = [&](E* at, int plane, const Chunk& c, bool ok, uint32_t sign) {
      if constexpr (F32) {
        u32x2_t q[3];
        split32(signed_chunk(c, ok, sign), q);
#pragma unroll
        for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x2_t*>(at + k * plane) = q[k];
      } else {
        *reinterpret_cast<Chunk*>(at) = ok ? c : zero_chunk();
      }
    };
    if (FOLD) {
#pragma unroll
      for (int i = 0; i < B_CH32; ++i) rb[p][i] = bn_fold_chunk<T>(rb[p][i], fsc, fsh);
    }
#pragma unroll
    for (int i = 0; i < A_CH32; ++i) {
      const int id = tid + i * NT, px = id / (BM / EV), kv = id % (BM / EV);
      put(&sa[px * (BM + PADE) + kv * EV], A_PL, ra[p][i], FULL || ((va[p] >> i) & 1u), odd != (t >= flip) ? 0x80000000u : 0u);
    }
#pragma unroll
    for (int i = 0; i < B_CH32; ++i) {
      const int id = tid + i * NT, px = id / (BN / EV), cv = id % (BN / EV);
      put(&sb[px * (BN + PADE) + cv * EV], B_PL, rb[p][i], FULL || ((vb[p] >> i) & 1u), 0u);
    }
  };

  v16f acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // Operand registers, loaded in FR::PHASES parts: 16-bit the two halves (16 pixels each) of the depth tile, fp32 the planes.
  // (lds_tr_read8: 8 pixels for channel tile base + l32.)
  FR fa[MI], fb[NI];
  const int r16 = l32 & 15;
  const int coff = (l32 & 16) + 4 * (r16 & 3);
  auto load_part = [&](int ph, int stage) {
    const int part = F32 ? 2 - ph : ph;
    const int px = (F32 ? g * 8 : g * 16 + ph * 8) + (r16 >> 2);
    const E* sa = lds + stage * STAGE + (F32 ? part * A_PL : 0) + px * (BM + PADE) + wm * WTM + coff;
    const E* sb = lds + stage * STAGE + A_ELEMS + (F32 ? part * B_PL : 0) + px * (BN + PADE) + wn * WTN + coff;
#pragma unroll
    for (int i = 0; i < MI; ++i)
      fa[i].p[part] = lds_tr_read8<std::remove_reference_t<decltype(fa[i].p[part])>>(sa + i * 32, sa + i * 32 + 4 * (BM + PADE));
#pragma unroll
    for (int j = 0; j < NI; ++j)
      fb[j].p[part] = lds_tr_read8<std::remove_reference_t<decltype(fb[j].p[part])>>(sb + j * 32, sb + j * 32 + 4 * (BN + PADE));
  };

  // pipeline as in the forward kernel: three LDS stages, two register generations, operand reload under the MFMAs
  if (n > 0) { gload(IC<0>{}, IC<1>{}, 0); sstore(IC<0>{}, IC<0>{}, 0, 0); }
  if (n > 1) { gload(IC<1>{}, IC<1>{}, 1); sstore(IC<1>{}, IC<0>{}, 1, 1); }
  if (n > 2) gload(IC<0>{}, IC<1>{}, 2);
  __syncthreads();
  if (n > 0) {
#pragma unroll
    for (int ph = 0; ph < FR::PHASES; ++ph) load_part(ph, 0);
  }
  auto negate = [&]() {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int jn = 0; jn < NI; ++jn) acc[i][jn] = -acc[i][jn];
  };
  auto body = [&](auto G, auto TAILC, int j, int stage) {
    constexpr int p = decltype(G)::value;  // = j & 1: this generation holds tile j+2
    constexpr bool TAIL = decltype(TAILC)::value != 0;  // 0: steady state without range checks
    const int nstage = stage == 2 ? 0 : stage + 1;
    const bool has_next = TAIL ? j + 1 < n : true;
    // steady state: tiles j + 2 and j + 3 are not the range's last one, all of their rows are inside it
    if (!TAIL || j + 3 < n) gload(IC<1 - p>{}, IC<TAIL ? 1 : 0>{}, j + 3);
#pragma unroll
    for (int ph = 0; ph < FR::PHASES; ++ph) {
#pragma unroll
      for (int q = 0; q < FR::steps(ph); ++q)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int jn = 0; jn < NI; ++jn) FR::mma(fa[i], fb[jn], acc[i][jn], ph, q);
      __builtin_amdgcn_sched_barrier(0);
      if (has_next) load_part(ph, nstage);
      if (ph + 1 < FR::PHASES) __builtin_amdgcn_sched_barrier(0);
    }
    if (!TAIL || j + 2 < n) sstore(G, IC<TAIL ? 0 : 1>{}, stage == 0 ? 2 : stage - 1, j + 2);
    __syncthreads();
  };
  {
    int stage = 0, j = 0;
#pragma unroll 1
    for (int half = F32 ? 0 : 1; half < 2; ++half) {
      const int end = half ? n - 5 : flip;  // the second body loads tile j + 4 unchecked: the range goes on behind it
      for (; j < end; j += 2) {
        body(IC<0>{}, IC<0>{}, j, stage);
        stage = stage == 2 ? 0 : stage + 1;
        body(IC<1>{}, IC<0>{}, j + 1, stage);
        stage = stage == 2 ? 0 : stage + 1;
      }
      if (half == 0) negate();
    }
    for (; j < n; j += 2) {
      body(IC<0>{}, IC<1>{}, j, stage);
      stage = stage == 2 ? 0 : stage + 1;
      if (j + 1 < n) {
        body(IC<1>{}, IC<1>{}, j + 1, stage);
        stage = stage == 2 ? 0 : stage + 1;
      }
    }
  }

  if (F32 && !odd) negate();  // (from tile `flip` on the sums are those of -dz where the range's first ones are of dz)
  if constexpr (F32) {
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) sum = __fmaf_rn(acc[i][j][e], 0.f, sum);
    if (__syncthreads_or(!(sum == 0.f))) {  // the tile again as chains of fp32 multiply-adds (split32.h)
      float* fa_ = reinterpret_cast<float*>(wgrad_smem);
      float* fb_ = fa_ + DEPTH * BM;
      clear_sums(acc);
#pragma unroll 1
      for (int t = 0; t < n; ++t) {
        gload(IC<0>{}, IC<1>{}, t);
#pragma unroll
        for (int i = 0; i < A_CH32; ++i) *reinterpret_cast<Chunk*>(fa_ + (tid + i * NT) * EV) = ra[0][i];  // [pixel][BM]
#pragma unroll
        for (int i = 0; i < B_CH32; ++i) *reinterpret_cast<Chunk*>(fb_ + (tid + i * NT) * EV) = rb[0][i];
        __syncthreads();
#pragma unroll 1
        for (int px = 0; px < DEPTH; ++px) {  // (pixels that do not count are left out: zero times infinity is none)
          const int m = mbeg + t * DEPTH + px;
          if (m >= mend) break;
          const uint32_t n_ = divPQ.div((uint32_t)m), rem = (uint32_t)m - n_ * divPQ.d;
          const uint32_t p_ = divQ.div(rem);
          int64_t off;
          if (!tap_offset((int)n_, (int)p_, (int)(rem - p_ * divQ.d), off)) continue;
          float xv[NI];
#pragma unroll
          for (int j = 0; j < NI; ++j) xv[j] = fb_[px * BN + wn * WTN + j * 32 + l32];
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              const float d = fa_[px * BM + wm * WTM + i * 32 + 8 * (e >> 2) + 4 * g + (e & 3)];
#pragma unroll
              for (int j = 0; j < NI; ++j) acc[i][j][e] = __fmaf_rn(d, xv[j], acc[i][j][e]);
            }
        }
        __syncthreads();
      }
    }
  }
  const int64_t outputs = (int64_t)K * a.R * a.S * C;
  float* dst = out + (int64_t)bz * outputs;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int c = c0 + wn * WTN + j * 32 + l32;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int k = k0 + wm * WTM + i * 32 + 8 * (e >> 2) + 4 * g + (e & 3);
        dst[((int64_t)k * a.R * a.S + tap) * C + c] = acc[i][j][e];
      }
    }
}

bool conv_mfma_wgrad_ok(int dt, const ConvGeom& g) {
  (void)dt;
  return g.C % 64 == 0 && g.K % 64 == 0 && (int64_t)g.N * g.P * g.Q < (1 << 24) && g.P * g.Q < (1 << 24);
}

// number of pixel chunks, from the layer shape only
// 1x1 layers have only (K / 128) * (C / 128) tiles, often one or two, and hundreds of thousands of pixels: they take
// up to 256 pixel ranges and aim at two blocks per CU (measured on the 1x1 layers of ResNet-50 at batch 128, bf16:
// 64->64 at 56x56 64 -> 23 us, 64->256 91 -> 56 us, 256->128 126 -> 75 us, all fifteen layers 995 -> 743 us)
static constexpr int g_wgrad_blocks = 1024;  // compile-time constants
static constexpr int g_wgrad_max_splits = 64;
static constexpr int g_wgrad_blocks_1x1 = 512;
static constexpr int g_wgrad_max_splits_1x1 = 256;
// 1x1 layers in the 16-bit modes whose channel counts are multiples of 256 and that have at least 64 K pixels take the
// 256 x 256 tile: one block per CU (256 blocks), every pixel range at least 16 depth tiles long
static bool wgrad_large_ok(int dt, const ConvGeom& g) {
  return dt != DT_F32 && g.R * g.S == 1 && g.K % 256 == 0 && g.C % 256 == 0 && (int64_t)g.N * g.P * g.Q >= 65536;
}
static int wgrad_large_splits(const ConvGeom& g) {
  const int64_t tiles = (int64_t)(g.K / 256) * (g.C / 256);
  const int64_t pixels = (int64_t)g.N * g.P * g.Q;
  int64_t want = tiles >= 256 ? 1 : (256 + tiles / 2) / tiles;
  const int64_t most = pixels / (16 * 32);
  if (want > most) want = most;
  if (want > 256) want = 256;
  return (int)(want < 1 ? 1 : want);
}

int conv_mfma_wgrad_splits(int dt, const ConvGeom& g, int64_t room) {
  if (conv_wgrad3x3_ok(dt, g)) return conv_wgrad3x3_splits(dt, g, room);
  if (wgrad_large_ok(dt, g)) return wgrad_large_splits(g);
  const int depth = dt == DT_F32 ? 16 : 32;
  const int bm = g.K % 128 == 0 ? 128 : 64, bn = g.C % 128 == 0 ? 128 : 64;
  const int64_t tiles = (int64_t)(g.K / bm) * (g.C / bn) * g.R * g.S;
  const int64_t pixels = (int64_t)g.N * g.P * g.Q;
  const bool pointwise = g.R * g.S == 1;
  const int target = pointwise ? g_wgrad_blocks_1x1 : g_wgrad_blocks;
  const int cap = pointwise ? g_wgrad_max_splits_1x1 : g_wgrad_max_splits;
  int64_t want = (target + tiles / 2) / tiles;                     // aim at about that many blocks
  const int64_t most = (pixels + 4 * depth - 1) / (4 * depth);     // at least four depth tiles per chunk
  if (want > most) want = most;
  if (want > cap) want = cap;
  return (int)(want < 1 ? 1 : want);
}

template <class T, bool FOLD>
static void launch_wgrad_t(hipStream_t st, const void* x, const void* dz, float* dst, int splits, const ConvGeom& g,
                           const float* fold) {
  constexpr int depth = sizeof(T) == 4 ? 16 : 32;
  WGradArgs a;
  a.H = g.H; a.W = g.W; a.C = g.C; a.K = g.K; a.R = g.R; a.S = g.S; a.stride = g.stride; a.pad = g.pad; a.P = g.P; a.Q = g.Q;
  a.pixels = g.N * g.P * g.Q;
  int chunk = (a.pixels + splits - 1) / splits;
  a.chunk = (chunk + depth - 1) / depth * depth;
  a.divQ = make_fastdiv((uint32_t)g.Q);
  a.divPQ = make_fastdiv((uint32_t)(g.P * g.Q));
  a.fold = fold;
  a.ranges = splits;
  // 3x3: where the ranges spread evenly over the XCDs, in 16 bits (nine taps read every row of dz; 128 -> 128 channels,
  // stride 2, 131 072 pixels in fp16 109 -> 96 us, 64 -> 128 at 65 536 in bf16 36 -> 31; fp32 waits for its matrix
  // instructions instead: 504 -> 537)
  a.xcd_group = g.R * g.S == 1 ? splits >= 8 : sizeof(T) == 2 && splits % 8 == 0;
  const int gz = a.xcd_group ? (splits + 7) / 8 * 8 : splits;
  if constexpr (sizeof(T) == 2) {
    if (wgrad_large_ok(DT_BF16, g)) {
      constexpr size_t sm = wgrad_lds_bytes<T, 256, 256, 2>();
      static bool attr_done = false;
      if (!attr_done) {
        (void)hipFuncSetAttribute((const void*)conv_wgrad_kernel<T, 256, 256, 2, 4, FOLD, false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
        (void)hipFuncSetAttribute((const void*)conv_wgrad_kernel<T, 256, 256, 2, 4, FOLD, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
        (void)hipFuncSetAttribute((const void*)conv_wgrad_kernel<T, 256, 256, 2, 4, FOLD, true, 1>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
        (void)hipFuncSetAttribute((const void*)conv_wgrad_kernel<T, 256, 256, 2, 4, FOLD, true, 2>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
        attr_done = true;
      }
      // rows of x = pixels of dz, and the row offsets fit 32 bits
      const bool pw = g.stride == 1 && g.pad == 0 && (int64_t)32 * std::max(g.K, g.C) < (1 << 30);
      if (pw && g.C == 256 && g.K > 256)
        OSEQ_LAUNCH((conv_wgrad_kernel<T, 256, 256, 2, 4, FOLD, true, 1>), dim3(g.K / 256, g.C / 256, gz), dim3(512), sm, st, (const T*)x,
                    (const T*)dz, dst, a);
      else if (pw && g.K == 256 && g.C > 256)
        OSEQ_LAUNCH((conv_wgrad_kernel<T, 256, 256, 2, 4, FOLD, true, 2>), dim3(g.K / 256, g.C / 256, gz), dim3(512), sm, st, (const T*)x,
                    (const T*)dz, dst, a);
      else if (pw)
        OSEQ_LAUNCH((conv_wgrad_kernel<T, 256, 256, 2, 4, FOLD, true>), dim3(g.K / 256, g.C / 256, gz), dim3(512), sm, st, (const T*)x,
                    (const T*)dz, dst, a);
      else
        OSEQ_LAUNCH((conv_wgrad_kernel<T, 256, 256, 2, 4, FOLD, false>), dim3(g.K / 256, g.C / 256, gz), dim3(512), sm, st, (const T*)x,
                    (const T*)dz, dst, a);
      return;
    }
  }
  const bool m128 = g.K % 128 == 0, n128 = g.C % 128 == 0;
  const int bm = m128 ? 128 : 64, bn = n128 ? 128 : 64;
  dim3 grid(g.K / bm, g.R * g.S * (g.C / bn), gz), block(256);
  // 1x1, unit stride, no padding: rows of x = pixels of dz, and the row offsets fit 32 bits
  const bool pw = g.R * g.S == 1 && g.stride == 1 && g.pad == 0 && (int64_t)32 * std::max(g.K, g.C) < (1 << 30);
#define WGRAD_LAUNCH(BM_, BN_)                                                                                              \
  {                                                                                                                         \
    constexpr size_t sm_ = wgrad_lds_bytes<T, BM_, BN_, 2>();                                                               \
    if constexpr (sm_ > 65536) {                                                                                            \
      static bool attr_ = false;                                                                                            \
      if (!attr_) {                                                                                                         \
        (void)hipFuncSetAttribute((const void*)conv_wgrad_kernel<T, BM_, BN_, 2, 2, FOLD, true>,                            \
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm_);                                    \
        (void)hipFuncSetAttribute((const void*)conv_wgrad_kernel<T, BM_, BN_, 2, 2, FOLD, false>,                           \
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm_);                                    \
        attr_ = true;                                                                                                       \
      }                                                                                                                     \
    }                                                                                                                       \
    if (pw) OSEQ_LAUNCH((conv_wgrad_kernel<T, BM_, BN_, 2, 2, FOLD, true>), grid, block, sm_, st, \
                        (const T*)x, (const T*)dz, dst, a);                                                                 \
    else OSEQ_LAUNCH((conv_wgrad_kernel<T, BM_, BN_, 2, 2, FOLD, false>), grid, block, sm_, st,  \
                     (const T*)x, (const T*)dz, dst, a);                                                                    \
  }
  if (m128 && n128) WGRAD_LAUNCH(128, 128)
  else if (m128) WGRAD_LAUNCH(128, 64)
  else if (n128) WGRAD_LAUNCH(64, 128)
  else WGRAD_LAUNCH(64, 64)
#undef WGRAD_LAUNCH
}

// out[i] = sum over pixel ranges s of partial[s][i], in a fixed order: G groups of threads each add the ranges
// s = g, g + G, ... for the same four outputs, then the G sums are added in group order.  G grows with the number
// of ranges so that small weight tensors with many ranges still fill the chip.
template <int G>
__global__ void __launch_bounds__(256) wgrad_reduce_kernel(const float* __restrict__ partial, float* __restrict__ out, int64_t n,
                                                           int splits) {
  constexpr int QB = 256 / G;  // output quads per block
  __shared__ v4f red[G > 1 ? 256 : 1];
  const int ql = threadIdx.x % QB, sg = threadIdx.x / QB;
  const int64_t i = ((int64_t)blockIdx.x * QB + ql) * 4;
  const bool on = i < n;
  v4f acc = {0.f, 0.f, 0.f, 0.f};
  if (on) {
#pragma unroll 4
    for (int s = sg; s < splits; s += G) acc += *reinterpret_cast<const v4f*>(partial + (int64_t)s * n + i);
  }
  if constexpr (G > 1) {
    red[threadIdx.x] = acc;
    __syncthreads();
    if (sg == 0 && on) {
      v4f t = red[ql];
#pragma unroll
      for (int g = 1; g < G; ++g) t += red[g * QB + ql];
      *reinterpret_cast<v4f*>(out + i) = t;
    }
  } else {
    if (on) *reinterpret_cast<v4f*>(out + i) = acc;
  }
}

void launch_wgrad_reduce(hipStream_t st, const float* partial, float* out, int64_t n, int splits) {
  const int64_t quads = n / 4;  // n is a multiple of 4 (C % 64 == 0)
  if (splits >= 64 || (splits >= 16 && quads < 65536))
    OSEQ_LAUNCH(wgrad_reduce_kernel<16>, dim3(ceil_div(quads, 16)), dim3(256), 0, st, partial, out, n, splits);
  else if (splits >= 8)
    OSEQ_LAUNCH(wgrad_reduce_kernel<4>, dim3(ceil_div(quads, 64)), dim3(256), 0, st, partial, out, n, splits);
  else
    OSEQ_LAUNCH(wgrad_reduce_kernel<1>, dim3(ceil_div(quads, 256)), dim3(256), 0, st, partial, out, n, splits);
}

// the matrix-core kernels in the 16-bit modes
bool conv_fold_wgrad_ok(int dt, const ConvGeom& g) { return dt != DT_F32 && conv_mfma_wgrad_ok(dt, g); }

void launch_conv_wgrad_mfma(hipStream_t st, int dt, const void* x, const void* dz, float* dw, float* partial, int splits,
                            const ConvGeom& g, const float* fold) {
  float* dst = splits > 1 ? partial : dw;
  if (conv_wgrad3x3_ok(dt, g)) launch_conv_wgrad3x3(st, dt, x, dz, dst, splits, g, fold);
  else if (dt == DT_F32) launch_wgrad_t<float, false>(st, x, dz, dst, splits, g, nullptr);
  else if (dt == DT_BF16) {
    if (fold) launch_wgrad_t<bf16_t, true>(st, x, dz, dst, splits, g, fold);
    else launch_wgrad_t<bf16_t, false>(st, x, dz, dst, splits, g, nullptr);
  } else {
    if (fold) launch_wgrad_t<f16_t, true>(st, x, dz, dst, splits, g, fold);
    else launch_wgrad_t<f16_t, false>(st, x, dz, dst, splits, g, nullptr);
  }
  if (splits > 1) {
    launch_wgrad_reduce(st, partial, dw, (int64_t)g.K * g.R * g.S * g.C, splits);
  }
}

}  // namespace oseq
