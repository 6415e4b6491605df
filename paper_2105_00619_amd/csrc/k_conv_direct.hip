// Direct (plain FMA) convolution forward / data gradient / weight gradient for shapes the matrix-core
// kernels do not take: very few channels (the 3-channel stem, the tiny test networks).  NHWC activations,
// (C_out, kh, kw, C_in) weights, fp32 accumulation in a fixed order.
#include <algorithm>

#include "dev_common.h"
#include "epilogue.h"
#include "kernels.h"

namespace oseq {

// I: the index type, int where every tensor has fewer than 2^30 elements (64-bit divisions and address arithmetic are
// most of these kernels' instructions).  V: channels per load, 4 where the channel counts allow it.
template <class T, class I, int V>
__global__ void __launch_bounds__(256) conv_fwd_direct_kernel(const T* __restrict__ x, const T* __restrict__ w,
                                                              const float* __restrict__ bias, T* __restrict__ out,
                                                              ConvGeom g, int relu, const float* __restrict__ affine,
                                                              const T* __restrict__ skip) {
  const I total = (I)g.N * g.P * g.Q * g.K;
  const int64_t i64 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i64 >= (int64_t)total) return;
  const I i = (I)i64;
  const int k = (int)(i % g.K);
  I t = i / g.K;
  const int q = (int)(t % g.Q); t /= g.Q;
  const int p = (int)(t % g.P);
  const int n = (int)(t / g.P);
  float acc = 0.f;
  for (int r = 0; r < g.R; ++r) {
    const int ih = p * g.stride + r - g.pad;
    if (ih < 0 || ih >= g.H) continue;
#pragma unroll 3
    for (int s = 0; s < g.S; ++s) {
      const int iw = q * g.stride + s - g.pad;
      const bool in = iw >= 0 && iw < g.W;  // (a tap outside reads the row's first pixel and adds nothing)
      const T* xp = x + (((I)n * g.H + ih) * g.W + (in ? iw : 0)) * g.C;
      const T* wp = w + (((I)k * g.R + r) * g.S + s) * g.C;
      for (int c = 0; c < g.C; c += V) {
        float xv[V], wv[V];
        load_f32<T, V>(xp + c, xv);
        load_f32<T, V>(wp + c, wv);
#pragma unroll
        for (int u = 0; u < V; ++u) acc = in ? __fmaf_rn(xv[u], wv[u], acc) : acc;
      }
    }
  }
  if (affine) {  // the inference-mode BatchNorm behind the layer (affine: [2][K] scale and shift)
    acc = bn_affine(acc, affine[k], affine[g.K + k]);
    if (skip) acc += to_f32(skip[i]);
  } else if (bias) {
    acc += bias[k];
  }
  if (relu) acc = fmaxf(acc, 0.f);
  out[i] = from_f32<T>(acc);
}

// dx[n,h,w,c] = sum_{r,s,k} dz[n,p,q,k] * w[k,r,s,c] over the (p,q) with p*stride + r - pad == h, q*stride + s - pad == w
template <class T, class I, int V>
__global__ void __launch_bounds__(256) conv_dgrad_direct_kernel(const T* __restrict__ dz, const T* __restrict__ w,
                                                                const T* __restrict__ addend, T* __restrict__ dx,
                                                                ConvGeom g) {
  const I total = (I)g.N * g.H * g.W * g.C;
  const int64_t i64 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i64 >= (int64_t)total) return;
  const I i = (I)i64;
  const int c = (int)(i % g.C);
  I t = i / g.C;
  const int wq = (int)(t % g.W); t /= g.W;
  const int h = (int)(t % g.H);
  const int n = (int)(t / g.H);
  const I wk = (I)g.R * g.S * g.C;
  float acc = 0.f;
  for (int r = 0; r < g.R; ++r) {
    const int ph = h + g.pad - r;
    if (ph < 0 || ph % g.stride) continue;
    const int p = ph / g.stride;
    if (p >= g.P) continue;
#pragma unroll 3
    for (int s = 0; s < g.S; ++s) {
      const int qw = wq + g.pad - s;
      const int q = qw >= 0 ? qw / g.stride : 0;
      const bool in = qw >= 0 && qw % g.stride == 0 && q < g.Q;
      const T* zp = dz + (((I)n * g.P + p) * g.Q + (in ? q : 0)) * g.K;
      const T* wp = w + ((I)r * g.S + s) * g.C + c;
      for (int k = 0; k < g.K; k += V) {
        float zv[V];
        load_f32<T, V>(zp + k, zv);
#pragma unroll
        for (int u = 0; u < V; ++u) {
          const float wv = to_f32(wp[(I)(k + u) * wk]);
          acc = in ? __fmaf_rn(zv[u], wv, acc) : acc;
        }
      }
    }
  }
  if (addend) acc += to_f32(addend[i]);
  dx[i] = from_f32<T>(acc);
}

// dw[k,r,s,c] = sum over pixels (n,p,q) of dz[n,p,q,k] * x[n, p*stride+r-pad, q*stride+s-pad, c];
// blockIdx.y selects a fixed chunk of the pixel range; chunks are summed afterwards in order.  The pixel's coordinates are
// counted up, four pixels are loaded before the first is added (a pixel outside the image reads the tensor's first
// element and adds zero).
template <class T, class I>
__global__ void __launch_bounds__(256) conv_wgrad_direct_kernel(const T* __restrict__ x, const T* __restrict__ dz,
                                                                float* __restrict__ out, ConvGeom g, int64_t chunk) {
  const I outputs = (I)g.K * g.R * g.S * g.C;
  const int64_t o64 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (o64 >= (int64_t)outputs) return;
  const I o = (I)o64;
  const int c = (int)(o % g.C);
  I t = o / g.C;
  const int s = (int)(t % g.S); t /= g.S;
  const int r = (int)(t % g.R);
  const int k = (int)(t / g.R);
  const I pixels = (I)g.N * g.P * g.Q;
  const int64_t first = (int64_t)blockIdx.y * chunk;
  const I m0 = first < (int64_t)pixels ? (I)first : pixels;
  const I m1 = first + chunk < (int64_t)pixels ? (I)(first + chunk) : pixels;
  int q = (int)(m0 % g.Q);
  const I mq = m0 / g.Q;
  int p = (int)(mq % g.P), n = (int)(mq / g.P);
  float acc = 0.f;
  for (I m = m0; m < m1; m += 4) {
    float zv[4], xv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int ih = p * g.stride + r - g.pad, iw = q * g.stride + s - g.pad;
      const bool in = m + u < m1 && ih >= 0 && ih < g.H && iw >= 0 && iw < g.W;
      const float a = to_f32(dz[in ? (m + u) * g.K + k : 0]), b = to_f32(x[in ? (((I)n * g.H + ih) * g.W + iw) * g.C + c : 0]);
      zv[u] = in ? a : 0.f;
      xv[u] = in ? b : 0.f;
      if (++q == g.Q) { q = 0; if (++p == g.P) { p = 0; ++n; } }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) acc = __fmaf_rn(zv[u], xv[u], acc);
  }
  out[(int64_t)blockIdx.y * outputs + o] = acc;
}

// ------------------------------------------------------------------------------------------------------------
// Few input channels (the 3-channel stem): R*S*C <= 36 products per output.  HBM-bound (one activation write per
// 27 multiply-adds per channel), so plain FMAs: a thread keeps its pixel's input patch in registers and produces
// 8 output channels; the 8 x (R*S*C) weights of the block's channel group sit in LDS and are read by broadcast.
// ------------------------------------------------------------------------------------------------------------
constexpr int SMALLC_MAX = 36;

template <class T, int C>
__global__ void __launch_bounds__(256) conv_fwd_smallc_kernel(const T* __restrict__ x, const T* __restrict__ w,
                                                              const float* __restrict__ bias, T* __restrict__ out,
                                                              ConvGeom g, int relu, FastDiv divQ, FastDiv divPQ,
                                                              const float* __restrict__ affine, const T* __restrict__ skip) {
  // block = 128 pixels x 64 output channels (blockIdx.y selects the group of 64); thread = 4 pixels x 8 channels,
  // the 8 threads of a pixel next to each other so that a wavefront writes 8 whole rows of 64 channels, and every
  // weight read from LDS serves four pixels.  The 8 threads of a pixel share the loading of its R*S*C inputs
  // through LDS (vector-memory instructions, not bytes, bound this kernel otherwise).
  constexpr int RSC = 9 * C;  // 3x3 filter
  constexpr int XP = (RSC + 3) / 4 * 4;
  constexpr int PPT = 4;
  __shared__ __attribute__((aligned(16))) float ws[RSC * 64];        // [e][channel]
  __shared__ __attribute__((aligned(16))) float xs[32 * PPT * XP];   // [pixel of the block][e]
  const int kbase = blockIdx.y * 64;
  const int kn = g.K - kbase < 64 ? g.K - kbase : 64;
  for (int i = threadIdx.x; i < RSC * 64; i += 256) {
    const int k = i / RSC, e = i - k * RSC;  // consecutive threads read consecutive weights
    ws[e * 64 + k] = k < kn ? to_f32(w[(kbase + k) * RSC + e]) : 0.f;
  }
  const int grp = threadIdx.x & 7, slot = threadIdx.x >> 3;
  const int pixels = g.N * g.P * g.Q;  // < 2^24 (checked by the launcher), so 32-bit index arithmetic throughout
  const int H = g.H, W = g.W, cstride = g.stride, pad = g.pad;
  int m[PPT];
  // this thread's input elements e = grp + 8u of each of its pixels: filter offsets and channel are pixel-independent
  int er[(RSC + 7) / 8], es[(RSC + 7) / 8], ec[(RSC + 7) / 8];
#pragma unroll
  for (int u = 0; u < (RSC + 7) / 8; ++u) {
    const int e = grp + 8 * u < RSC ? grp + 8 * u : RSC - 1;
    const int tap = e / C;
    ec[u] = e - tap * C; er[u] = tap / 3 - pad; es[u] = tap % 3 - pad;
  }
#pragma unroll
  for (int i = 0; i < PPT; ++i) {
    m[i] = blockIdx.x * (32 * PPT) + slot + 32 * i;
    const uint32_t mm = m[i] < pixels ? (uint32_t)m[i] : 0u;
    const uint32_t n = divPQ.div(mm), rem = mm - n * divPQ.d;
    const uint32_t p = divQ.div(rem), q = rem - p * divQ.d;
    const int ih0 = (int)p * cstride, iw0 = (int)q * cstride, nbase = (int)n * H;
#pragma unroll
    for (int u = 0; u < (RSC + 7) / 8; ++u) {
      const int ih = ih0 + er[u], iw = iw0 + es[u];
      const bool ok = ih >= 0 && ih < H && iw >= 0 && iw < W;
      const float v = to_f32(x[ok ? ((nbase + ih) * W + iw) * C + ec[u] : 0]);
      if (grp + 8 * u < RSC) xs[(slot + 32 * i) * XP + grp + 8 * u] = ok ? v : 0.f;
    }
  }
  __syncthreads();
  float acc[PPT][8];
#pragma unroll
  for (int i = 0; i < PPT; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = 0.f;
  // one filter tap (C inputs) per iteration; not unrolled further: with all R*S*C steps visible the compiler
  // hoists every LDS read to the top and parks the values in accumulation registers
#pragma unroll 1
  for (int tap = 0; tap < 9; ++tap) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int e = tap * C + c;
      const float* wp = &ws[e * 64 + grp * 8];
      float wv[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) wv[j] = wp[j];
#pragma unroll
      for (int i = 0; i < PPT; ++i) {
        const float xv = xs[(slot + 32 * i) * XP + e];
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = __fmaf_rn(xv, wv[j], acc[i][j]);
      }
    }
  }
  if (grp * 8 >= kn) return;
#pragma unroll
  for (int i = 0; i < PPT; ++i) {
    if (m[i] >= pixels) continue;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float a = acc[i][j];
      const int k = kbase + grp * 8 + j;
      if (affine) {  // the inference-mode BatchNorm behind the layer (affine: [2][K] scale and shift)
        a = bn_affine(a, affine[k], affine[g.K + k]);
        if (skip) a += to_f32(skip[(int64_t)m[i] * g.K + k]);
      } else if (bias) {
        a += bias[k];
      }
      acc[i][j] = relu ? fmaxf(a, 0.f) : a;
    }
    store_f32<T, 8>(out + (int64_t)m[i] * g.K + kbase + grp * 8, acc[i]);
  }
}

template <class T> struct StemMma;
template <> struct StemMma<bf16_t> {
  typedef __attribute__((ext_vector_type(8))) __bf16 V;
  typedef __attribute__((ext_vector_type(16))) float A;
  __device__ static __forceinline__ A run(V a, V b, A c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
};
template <> struct StemMma<f16_t> {
  typedef __attribute__((ext_vector_type(8))) _Float16 V;
  typedef __attribute__((ext_vector_type(16))) float A;
  __device__ static __forceinline__ A run(V a, V b, A c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
};

// The same layer in the 16-bit modes, with at most 32 products per output (3x3 on up to 3 channels) and output channels in
// groups of 64, on the matrix cores: HBM-bound on writing the output, so the work per output is kept to a few
// instructions.  Blocks stay and walk tiles of 128 consecutive pixels (a tile's outputs of a 64-channel layer are one
// contiguous 16 KB).  A wavefront multiplies its 32 pixels by 64 channels: the 64 x 32 weights (depth 27..31 zero) live in
// registers, a lane gathers half of the 27 inputs of its own pixel straight into the MFMA operand (one index decomposition
// and one nine-bit mask of taps inside the image per lane and tile), the next tile's inputs are requested before this
// tile's results are stored.  The results are channels x pixels: four consecutive channels of a pixel per lane, rounded in
// pairs, through LDS, stored as 16-byte pieces of whole rows; the storing threads also keep the channel sums of what they
// store for the BatchNorm that follows, one row of block sums per block.
// 262 144 pixels, 3 -> 64 channels, bf16: 15.7 us, 22.4 with the sums.
// (With every thread gathering sixteen elements into an LDS tile, and the fp32 epilogue tile: 21.4 us, and 14 us for the
// sums in a pass of their own.)
// AFF: table of scale and shift per channel: an inference-mode BatchNorm, or a bias (scale 1)
constexpr int STEM_BM = 128;
template <class T, int C, bool AFF, bool STAT>
__global__ void __launch_bounds__(256) conv_stem_fwd_kernel(const T* __restrict__ x, const T* __restrict__ w,
                                                            const float* __restrict__ bias, const float* __restrict__ affine,
                                                            T* __restrict__ out, float* __restrict__ stat_partial, ConvGeom g,
                                                            int relu, FastDiv divQ, FastDiv divPQ) {
  typedef typename StemMma<T>::V FV;
  typedef typename StemMma<T>::A v16f;
  typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
  constexpr int RSC = 9 * C, PITCH = 64 + 8;
  static_assert(RSC <= 32, "one 32-deep step");
  __shared__ __attribute__((aligned(16))) T stg[STEM_BM * PITCH];
  __shared__ float tab[2][64];
  __shared__ float red[STAT ? 2 * 32 * 64 : 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hg = lane >> 5, l32 = lane & 31;
  const int kbase = blockIdx.y * 64;
  const int pixels = g.N * g.P * g.Q;  // < 2^24 (checked by the launcher)
  const int H = g.H, W = g.W, cstride = g.stride, pad = g.pad;
  const int tiles = (pixels + STEM_BM - 1) / STEM_BM;

  // weights: lane group hg owns depth elements [16 hg, + 16), eight per MFMA
  FV wv[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int e = hg * 16 + h * 8 + j;
        const T v = w[(kbase + i * 32 + l32) * RSC + (e < RSC ? e : 0)];
        wv[i][h][j] = e < RSC ? v : from_f32<T>(0.f);
      }
  if (AFF && tid < 64) {
    tab[0][tid] = affine ? affine[kbase + tid] : 1.f;
    tab[1][tid] = affine ? affine[g.K + kbase + tid] : bias[kbase + tid];
  }
  // this lane's sixteen inputs: offset from the pixel's centre element and filter tap
  int off[16], bit[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int e = hg * 16 + j, ec = e < RSC ? e : 0;
    const int tap = ec / C;
    off[j] = ((tap / 3 - pad) * W + (tap % 3 - pad)) * C + (ec - tap * C);
    bit[j] = e < RSC ? 1 << tap : 0;
  }
  T rx[16];
  unsigned taps = 0u;
  auto gather = [&](int tile) {
    const int m = tile * STEM_BM + wave * 32 + l32;
    const uint32_t mm = m < pixels ? (uint32_t)m : 0u;
    const uint32_t n = divPQ.div(mm), rem = mm - n * divPQ.d;
    const uint32_t p = divQ.div(rem), q = rem - p * divQ.d;
    const int ih = (int)p * cstride, iw = (int)q * cstride;
    unsigned cols = 0u;
    taps = 0u;
#pragma unroll
    for (int t = 0; t < 3; ++t) cols |= (iw + t - pad >= 0 && iw + t - pad < W) ? 1u << t : 0u;
#pragma unroll
    for (int t = 0; t < 3; ++t) taps |= (ih + t - pad >= 0 && ih + t - pad < H) ? cols << (3 * t) : 0u;
    if (m >= pixels) taps = 0u;
    const T* px = x + (((int64_t)n * H + ih) * W + iw) * C;
#pragma unroll
    for (int j = 0; j < 16; ++j) rx[j] = *((taps & bit[j]) ? px + off[j] : x);
  };
  float ss[8], qq[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) { ss[k] = 0.f; qq[k] = 0.f; }
  const int c8 = (tid & 7) * 8, erow = tid >> 3;

  int tile = blockIdx.x;
  gather(tile);
  for (; tile < tiles; tile += gridDim.x) {
    FV xv[2];
#pragma unroll
    for (int j = 0; j < 16; ++j) xv[j >> 3][j & 7] = (taps & bit[j]) ? rx[j] : from_f32<T>(0.f);
    v16f acc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
      acc[i] = StemMma<T>::run(wv[i][0], xv[0], acc[i]);
      acc[i] = StemMma<T>::run(wv[i][1], xv[1], acc[i]);
    }
    if (tile + (int)gridDim.x < tiles) gather(tile + gridDim.x);
    __syncthreads();  // the tile before has been stored (and, the first time, the table is there)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = i * 32 + 8 * q + 4 * hg;
        float v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          v[k] = acc[i][4 * q + k];
          if (AFF) v[k] = bn_affine(v[k], tab[0][c + k], tab[1][c + k]);
          if (relu) v[k] = fmaxf(v[k], 0.f);
        }
        u32x2 o;
        o[0] = __builtin_bit_cast(uint32_t, from_f32x2<T>(v[0], v[1]));
        o[1] = __builtin_bit_cast(uint32_t, from_f32x2<T>(v[2], v[3]));
        *reinterpret_cast<u32x2*>(&stg[(wave * 32 + l32) * PITCH + c]) = o;
      }
    __syncthreads();
    Vec<T, 8> tv[4];
    const int m0 = tile * STEM_BM;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int row = erow + 32 * it;
      tv[it] = *reinterpret_cast<const Vec<T, 8>*>(&stg[row * PITCH + c8]);
      if (m0 + row < pixels) *reinterpret_cast<Vec<T, 8>*>(out + (int64_t)(m0 + row) * g.K + kbase + c8) = tv[it];
      else if (STAT) tv[it] = Vec<T, 8>{};  // counts as zero
    }
    if (STAT) {
      typedef typename Dot2<T>::V T2;
      T2 one2;
      one2[0] = from_f32<T>(1.f); one2[1] = from_f32<T>(1.f);
#pragma unroll
      for (int it = 0; it < 4; it += 2)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          T2 p2;
          p2[0] = tv[it].v[k]; p2[1] = tv[it + 1].v[k];
          ss[k] = Dot2<T>::run(p2, one2, ss[k]);
          qq[k] = Dot2<T>::run(p2, p2, qq[k]);
        }
    }
  }
  if (STAT)
    epi_stat_combine_nt<256, 64>(red, tid, ss, qq, stat_partial + ((int64_t)blockIdx.x * 2 + 0) * g.K + kbase,
                                 stat_partial + ((int64_t)blockIdx.x * 2 + 1) * g.K + kbase);
}

// Weight gradient for few input channels (the network stem):  dw[k][e] = sum over pixels of dz[px][k] * col[px][e],
// e = (tap, c) < 36, k in groups of 64 (blockIdx.y; a single group may have fewer).  Bound by reading dz once, and by
// latency: a block has few tiles.  A block reduces a fixed chunk of pixels in tiles of 64: the dz tile [64][64] and the
// im2col tile [64][R*S*C] are staged in LDS as fp32 (two stages; the next tile's global loads are issued before the MFMAs
// of the current one).  Each wavefront multiplies 16 of the 64 pixels with fp32 32x32x2 MFMAs (rows k, columns e); the
// four partial sums are added in wavefront order through LDS.
template <class T>
__global__ void __launch_bounds__(256) conv_wgrad_smallc_kernel(const T* __restrict__ x, const T* __restrict__ dz,
                                                                float* __restrict__ partial, ConvGeom g, int chunk,
                                                                FastDiv divQ, FastDiv divPQ) {
  typedef __attribute__((ext_vector_type(16))) float v16f;
  constexpr int DP = 68, XP = 37;                          // LDS row pitches in floats
  constexpr int NX = (64 * SMALLC_MAX + 255) / 256;        // im2col elements per thread and tile
  constexpr int EV = 16 / (int)sizeof(T), CPP = 64 / EV;   // elements per 16-byte chunk, chunks per dz row
  constexpr int DCH = 64 * CPP / 256;                      // dz chunks per thread and tile
  __shared__ __attribute__((aligned(16))) float dzs[2][64 * DP];
  __shared__ float xs[2][64 * XP];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hg = lane >> 5, l32 = lane & 31;
  const int kbase = blockIdx.y * 64, KN = g.K - kbase < 64 ? g.K - kbase : 64;
  const int K = g.K, C = g.C, H = g.H, W = g.W, rsc = g.R * g.S * g.C, cstride = g.stride;
  const int pixels = g.N * g.P * g.Q;
  const int m0 = blockIdx.x * chunk;
  const int m1 = m0 + chunk < pixels ? m0 + chunk : pixels;
  const int nt = m1 > m0 ? (m1 - m0 + 63) / 64 : 0;

  // This thread's im2col elements: one pixel of the tile (its lane) and the columns e = wave + 4u, so that a tile costs
  // one index decomposition per thread; whether a column's filter tap lies inside the image is one bit of a nine-bit mask
  // per pixel.
  const int xtap0 = wave;  // e = xtap0 + 4u
  int xoff[NX], xbit[NX];
#pragma unroll
  for (int u = 0; u < NX; ++u) {
    const int e = xtap0 + 4 * u < rsc ? xtap0 + 4 * u : 0;
    const int c = e % C, tap = e / C, s = tap % g.S, r = tap / g.S;
    xoff[u] = ((r - g.pad) * W + (s - g.pad)) * C + c;
    xbit[u] = xtap0 + 4 * u < rsc ? tap : -1;
  }
  Chunk rd[DCH];
  float rx[NX];
  unsigned dmask = 0u, xmask = 0u;
  // loads are unconditional (clamped addresses); what lies outside is zeroed when written to LDS
  auto gload = [&](int t) {
    const int mt = m0 + t * 64;
    unsigned dm = 0u, xm = 0u;
#pragma unroll
    for (int i = 0; i < DCH; ++i) {
      const int id = tid + i * 256, px = id / CPP, kv = id - px * CPP;
      const bool ok = mt + px < m1 && kv * EV < KN;
      rd[i] = *reinterpret_cast<const Chunk*>(dz + (int64_t)(ok ? mt + px : m0) * K + kbase + (ok ? kv * EV : 0));
      dm |= ok ? (1u << i) : 0u;
    }
    {
      const int m = mt + lane;
      const bool in = m < m1;
      const uint32_t mm = in ? (uint32_t)m : (uint32_t)m0;
      const uint32_t n_ = divPQ.div(mm), rem = mm - n_ * divPQ.d;
      const uint32_t p_ = divQ.div(rem), q_ = rem - p_ * divQ.d;
      const int ih0 = (int)p_ * cstride - g.pad, iw0 = (int)q_ * cstride - g.pad;
      const int64_t base = (((int64_t)n_ * H + (int)p_ * cstride) * W + (int)q_ * cstride) * C;
      unsigned taps = 0u;  // bit r * S + s: the tap lies inside the image
      for (int r = 0, b = 0; r < g.R; ++r)
        for (int s = 0; s < g.S; ++s, ++b)
          taps |= (in && ih0 + r >= 0 && ih0 + r < H && iw0 + s >= 0 && iw0 + s < W) ? (1u << b) : 0u;
#pragma unroll
      for (int u = 0; u < NX; ++u) {
        const bool ok = xbit[u] >= 0 && ((taps >> (xbit[u] & 31)) & 1u);
        rx[u] = to_f32(x[ok ? base + xoff[u] : 0]);
        xm |= ok ? (1u << u) : 0u;
      }
    }
    dmask = dm; xmask = xm;
  };
  auto sstore = [&](int stage) {
#pragma unroll
    for (int i = 0; i < DCH; ++i) {
      const int id = tid + i * 256, px = id / CPP, kv = id - px * CPP;
      const Chunk c = ((dmask >> i) & 1u) ? rd[i] : zero_chunk();
      float* dst = &dzs[stage][px * DP + kv * EV];
      if constexpr (sizeof(T) == 4) {
        *reinterpret_cast<Chunk*>(dst) = c;
      } else {
        const Vec<T, EV> v = __builtin_bit_cast(Vec<T, EV>, c);
        float f[EV];
#pragma unroll
        for (int k = 0; k < EV; ++k) f[k] = to_f32(v.v[k]);
#pragma unroll
        for (int k = 0; k < EV; k += 4) {
          typedef __attribute__((ext_vector_type(4))) float v4f;
          v4f o = {f[k], f[k + 1], f[k + 2], f[k + 3]};
          *reinterpret_cast<v4f*>(dst + k) = o;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < NX; ++u)
      if (xtap0 + 4 * u < rsc) xs[stage][lane * XP + xtap0 + 4 * u] = ((xmask >> u) & 1u) ? rx[u] : 0.f;
  };

  v16f acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  const bool two_m = KN > 32, two_n = rsc > 32;
  const int e0 = l32 < rsc ? l32 : rsc - 1, e1 = 32 + l32 < rsc ? 32 + l32 : rsc - 1;
  const float z0 = l32 < rsc ? 1.f : 0.f, z1 = 32 + l32 < rsc ? 1.f : 0.f;

  if (nt > 0) { gload(0); sstore(0); }
  __syncthreads();
  for (int t = 0; t < nt; ++t) {
    const int stage = t & 1;
    if (t + 1 < nt) gload(t + 1);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int px = 16 * wave + 8 * hg + u;
      const float a0 = dzs[stage][px * DP + l32];
      const float b0 = xs[stage][px * XP + e0] * z0;
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b0, acc[0][0], 0, 0, 0);
      float a1 = 0.f;
      if (two_m) {
        a1 = dzs[stage][px * DP + 32 + l32];
        acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b0, acc[1][0], 0, 0, 0);
      }
      if (two_n) {
        const float b1 = xs[stage][px * XP + e1] * z1;
        acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b1, acc[0][1], 0, 0, 0);
        if (two_m) acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b1, acc[1][1], 0, 0, 0);
      }
    }
    if (t + 1 < nt) sstore(stage ^ 1);
    __syncthreads();
  }

  // the four wavefronts' sums of one column tile, added in wavefront order: red[wavefront][k][32]
  float* red = &dzs[0][0];
  static_assert(2 * 64 * DP >= 4 * 64 * 32, "the four partial tiles lie over the dz stages");
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (j == 1 && !two_n) break;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) red[wave * 2048 + (i * 32 + 8 * (e >> 2) + 4 * hg + (e & 3)) * 32 + l32] = acc[i][j][e];
    __syncthreads();
    for (int o = tid; o < 2048; o += 256) {
      const int k = o >> 5, e = j * 32 + (o & 31);
      if (k < KN && e < rsc)
        partial[((int64_t)blockIdx.x * K + kbase + k) * rsc + e] = ((red[o] + red[2048 + o]) + red[4096 + o]) + red[6144 + o];
    }
    __syncthreads();
  }
}

// The same in the 16-bit modes with at most 32 columns (3x3 on up to 3 channels) and whole groups of 64 channels, on the
// 16-bit MFMAs: tiles of 128 pixels, dz staged as loaded and read with the transposing LDS read, the im2col columns
// gathered by one pixel per thread and stored column-major, so that a lane's eight consecutive pixels of a column are one
// 16-byte read.  One LDS stage, the next tile's loads in registers, small enough for several blocks per CU to cover each
// other.  262 144 pixels, bf16: 12.5 us (the fp32 kernel above, converting both operands: 47 us).
template <class T, int C>
__global__ void __launch_bounds__(256) conv_stem_wgrad_kernel(const T* __restrict__ x, const T* __restrict__ dz,
                                                              float* __restrict__ partial, ConvGeom g, int chunk, FastDiv divQ,
                                                              FastDiv divPQ) {
  typedef typename StemMma<T>::V FV;
  typedef typename StemMma<T>::A v16f;
  constexpr int RSC = 9 * C, BM = STEM_BM, DP = 64 + 16, XP = BM + 8;
  constexpr int HALF = 16;  // columns gathered by each of a pixel's two threads
  static_assert(RSC <= 32, "one 32-column tile");
  __shared__ __attribute__((aligned(16))) T smem[BM * DP + 32 * XP];  // dz [pixel][channel], im2col [column][pixel]
  static_assert(sizeof(T) * (BM * DP + 32 * XP) >= 4 * 32 * 32 * 4, "the four partial 32 x 32 tiles lie over the operands");
  T* ds = smem;
  T* xs = smem + BM * DP;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hg = lane >> 5, l32 = lane & 31;
  const int kbase = blockIdx.y * 64;
  const int K = g.K, H = g.H, W = g.W, cstride = g.stride, pad = g.pad;
  const int pixels = g.N * g.P * g.Q;
  const int m0 = blockIdx.x * chunk;
  const int m1 = m0 + chunk < pixels ? m0 + chunk : pixels;
  const int nt = m1 > m0 ? (m1 - m0 + BM - 1) / BM : 0;
  const int gpx = tid & (BM - 1), gh = tid >> 7;  // gathering: pixel of the tile, which half of the columns
  Chunk rd[4];
  T rx[HALF];
  unsigned taps = 0u;
  auto gload = [&](int t) {
    const int mt = m0 + t * BM;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int id = tid + i * 256, px = id >> 3, kv = id & 7;
      rd[i] = *reinterpret_cast<const Chunk*>(dz + (int64_t)(mt + px < m1 ? mt + px : m0) * K + kbase + kv * 8);
    }
    const int m = mt + gpx;
    const uint32_t mm = m < m1 ? (uint32_t)m : (uint32_t)m0;
    const uint32_t n = divPQ.div(mm), rem = mm - n * divPQ.d;
    const uint32_t p = divQ.div(rem), q = rem - p * divQ.d;
    const int ih = (int)p * cstride, iw = (int)q * cstride;
    unsigned cols = 0u;
    taps = 0u;
#pragma unroll
    for (int u = 0; u < 3; ++u) cols |= (iw + u - pad >= 0 && iw + u - pad < W) ? 1u << u : 0u;
#pragma unroll
    for (int u = 0; u < 3; ++u) taps |= (ih + u - pad >= 0 && ih + u - pad < H) ? cols << (3 * u) : 0u;
    if (m >= m1) taps = 0u;
    const T* px = x + (((int64_t)n * H + ih) * W + iw) * C;
#pragma unroll
    for (int j = 0; j < HALF; ++j) {
      const int e = gh * HALF + j, ec = e < RSC ? e : 0, tap = ec / C;
      rx[j] = *((taps >> tap) & 1u ? px + ((tap / 3 - pad) * W + (tap % 3 - pad)) * C + (ec - tap * C) : x);
    }
  };
  auto sstore = [&](int t) {
    const int mt = m0 + t * BM;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int id = tid + i * 256, px = id >> 3, kv = id & 7;
      *reinterpret_cast<Chunk*>(&ds[px * DP + kv * 8]) = mt + px < m1 ? rd[i] : zero_chunk();
    }
#pragma unroll
    for (int j = 0; j < HALF; ++j) {
      const int e = gh * HALF + j, tap = (e < RSC ? e : 0) / C;
      xs[e * XP + gpx] = e < RSC && ((taps >> tap) & 1u) ? rx[j] : from_f32<T>(0.f);
    }
  };
  v16f acc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
  // transposing read: within 16 lanes, lane r points at 4 consecutive channels (from 4 * (r % 4)) of pixel r / 4; lane l
  // receives channel l of the 16 at four pixels
  const int r16 = l32 & 15, coff = (l32 & 16) + 4 * (r16 & 3);
  if (nt > 0) gload(0);
  for (int t = 0; t < nt; ++t) {
    sstore(t);
    __syncthreads();
    if (t + 1 < nt) gload(t + 1);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int p0 = wave * 32 + h * 16 + hg * 8;  // the lane group's eight pixels
      const FV b = *reinterpret_cast<const FV*>(&xs[l32 * XP + p0]);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const T* pp = ds + (p0 + (r16 >> 2)) * DP + i * 32 + coff;
        acc[i] = StemMma<T>::run(lds_tr_read8<FV>(pp, pp + 4 * DP), b, acc[i]);
      }
    }
    __syncthreads();
  }
  // the four wavefronts' sums of a 32 x 32 tile, added in wavefront order
  float* red = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
#pragma unroll
    for (int e = 0; e < 16; ++e) red[wave * 1024 + (8 * (e >> 2) + 4 * hg + (e & 3)) * 32 + l32] = acc[i][e];
    __syncthreads();
    for (int o = tid; o < 1024; o += 256) {
      const int k = o >> 5, e = o & 31;
      if (e < RSC)
        partial[((int64_t)blockIdx.x * K + kbase + i * 32 + k) * RSC + e] =
            ((red[o] + red[1024 + o]) + red[2048 + o]) + red[3072 + o];
    }
    __syncthreads();
  }
}

// 16 outputs per block: thread (output, row group) sums the partials of rows group, group + 16, ... (four in flight), the
// 16 group sums of an output are added in order.  (One thread per output walking 256 rows took 57 us for 576 outputs, one
// wavefront per output reads a whole memory line for every four bytes.)
__global__ void __launch_bounds__(256) partial_reduce_kernel(const float* __restrict__ partial, float* __restrict__ out, int64_t n,
                                                             int splits) {
  __shared__ float red[16][17];
  const int ox = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const int64_t o = (int64_t)blockIdx.x * 16 + ox;
  const float* p = partial + (o < n ? o : 0);
  float v = 0.f;
  int s = grp;
  for (; s + 48 < splits; s += 64) {
    const float t0 = p[(int64_t)s * n], t1 = p[(int64_t)(s + 16) * n], t2 = p[(int64_t)(s + 32) * n], t3 = p[(int64_t)(s + 48) * n];
    v += t0; v += t1; v += t2; v += t3;
  }
  for (; s < splits; s += 16) v += p[(int64_t)s * n];
  red[grp][ox] = v;
  __syncthreads();
  if (grp == 0 && o < n) {
#pragma unroll
    for (int g = 1; g < 16; ++g) v += red[g][ox];
    out[o] = v;
  }
}

// 8 to 31 output channels leave most of a group of 64 empty, but only as long as the pixels are few is the direct kernel, whose
// time goes with the outputs and the loads of each, the faster one.  us, direct / tiled, 3 -> K channels: fp32 K = 8 at 8192
// pixels 6.8 / 14.5, 32 768 12.1 / 15.8, 65 536 18.1 / 16.7, 2 M 315 / 129; K = 24 at 8192 12.9 / 17.0, 16 384 20.7 / 16.4, 2 M
// 1386 / 133; bf16 K = 16 at 16 384 11.8 / 15.6, 32 768 20.3 / 14.4.  1 -> 16 at 32 768 12.0 / 11.4, 4 -> 16 12.9 / 15.4 (four
// channels are one load).  The line is drawn at outputs * (loads + 6): 8.7 M at 3 -> 8 and 32 768 pixels, 13 M at 3 -> 24 and 16 384.
bool conv_smallc_fwd_ok(const ConvGeom& g) {
  const int64_t pixels = (int64_t)g.N * g.P * g.Q;
  if (g.K < 32 && pixels * g.K * (9 * (g.C % 4 == 0 ? 1 : g.C) + 6) < 10000000) return false;
  return g.C <= 4 && g.R == 3 && g.S == 3 && g.K % 8 == 0 && pixels < (1 << 24) && (int64_t)g.N * g.H * g.W * g.C < ((int64_t)1 << 31);
}
// the 16-bit kernels of the stem
static bool stem_ok(int dt, const ConvGeom& g) { return dt != DT_F32 && g.C <= 3 && g.R == 3 && g.S == 3 && g.K % 64 == 0; }
static int stem_blocks(const ConvGeom& g) {  // blocks stay: four per CU, or one per tile
  const int64_t tiles = ((int64_t)g.N * g.P * g.Q + STEM_BM - 1) / STEM_BM;
  return (int)(tiles < 1024 ? tiles : 1024);
}
// row blocks over which the forward kernel also sums its outputs for the BatchNorm that follows (0: it does not)
int conv_smallc_stat_blocks(int dt, const ConvGeom& g) { return conv_smallc_fwd_ok(g) && stem_ok(dt, g) ? stem_blocks(g) : 0; }
bool conv_smallc_wgrad_ok(const ConvGeom& g) {
  return g.C <= 4 && g.R * g.S * g.C <= SMALLC_MAX && (g.K <= 64 ? g.K % 8 == 0 : g.K % 64 == 0) &&
         (int64_t)g.N * g.P * g.Q < (1 << 24) && (int64_t)g.N * g.H * g.W * g.C < ((int64_t)1 << 31);
}
int conv_smallc_wgrad_splits(int dt, const ConvGeom& g, int64_t room) {
  const int64_t pixels = (int64_t)g.N * g.P * g.Q;
  // four tiles of 64 pixels per block, fewer where that would leave CUs idle and the partial sums fit the room; the 16-bit
  // kernel of the stem: one tile per block up to two blocks per CU
  const int64_t four = std::min<int64_t>(std::max<int64_t>((pixels + 255) / 256, 1), 1024);
  int64_t b = std::min<int64_t>((pixels + 63) / 64, 512);
  if (stem_ok(dt, g)) b = std::min<int64_t>((pixels + STEM_BM - 1) / STEM_BM, 512);
  else b = std::max(four, b);
  const int64_t fit = room / ((int64_t)g.K * g.R * g.S * g.C * 4);
  return (int)std::max<int64_t>(1, std::min(b, std::max(fit, g.K <= 64 ? four : std::min<int64_t>(four, 64))));
}

template <class T>
static void launch_fwd_smallc_t(hipStream_t st, const void* x, const void* w, const float* bias, void* out, float* stat_partial,
                                const ConvGeom& g, int relu, const ConvEval& ev) {
  dim3 grid(ceil_div((int64_t)g.N * g.P * g.Q, 128), ceil_div(g.K, 64)), block(256);
  const FastDiv dq = make_fastdiv((uint32_t)g.Q), dpq = make_fastdiv((uint32_t)(g.P * g.Q));
  const T* skip = (const T*)ev.skip;
  if constexpr (sizeof(T) == 2) {
    if (stem_ok(DT_BF16, g) && !skip) {  // 16-bit modes: on the matrix cores
      grid.x = stem_blocks(g);
#define STEM_LAUNCH(C_, AFF_, STAT_)                                                                                       \
  OSEQ_LAUNCH((conv_stem_fwd_kernel<T, C_, AFF_, STAT_>), grid, block, 0, st, (const T*)x, (const T*)w, bias, ev.affine,  \
              (T*)out, stat_partial, g, relu, dq, dpq)
#define STEM_C(C_)                                                                                                         \
  {                                                                                                                        \
    if (ev.affine || bias) { if (stat_partial) STEM_LAUNCH(C_, true, true); else STEM_LAUNCH(C_, true, false); }          \
    else if (stat_partial) STEM_LAUNCH(C_, false, true);                                                                   \
    else STEM_LAUNCH(C_, false, false);                                                                                    \
  }
      if (g.C == 1) STEM_C(1) else if (g.C == 2) STEM_C(2) else STEM_C(3)
#undef STEM_C
#undef STEM_LAUNCH
      return;
    }
  }
#define SMALLC_FMA(C_)                                                                                                \
  OSEQ_LAUNCH((conv_fwd_smallc_kernel<T, C_>), grid, block, 0, st, (const T*)x, (const T*)w, bias, (T*)out, g, relu, \
              dq, dpq, ev.affine, skip)
  switch (g.C) {
    case 1: SMALLC_FMA(1); break;
    case 2: SMALLC_FMA(2); break;
    case 3: SMALLC_FMA(3); break;
    default: SMALLC_FMA(4); break;
  }
#undef SMALLC_FMA
}

// stat_partial: null, or [conv_smallc_stat_blocks][2][C_out] floats receiving per-block sums of the stored outputs
void launch_conv_fwd_smallc(hipStream_t st, int dt, const void* x, const void* w, const float* bias, void* out,
                            float* stat_partial, const ConvGeom& g, int relu, const ConvEval& ev) {
  if (dt == DT_F32) launch_fwd_smallc_t<float>(st, x, w, bias, out, stat_partial, g, relu, ev);
  else if (dt == DT_BF16) launch_fwd_smallc_t<bf16_t>(st, x, w, bias, out, stat_partial, g, relu, ev);
  else launch_fwd_smallc_t<f16_t>(st, x, w, bias, out, stat_partial, g, relu, ev);
}

template <class T>
static void launch_wgrad_smallc_t(hipStream_t st, const T* x, const T* dz, float* dst, int splits, const ConvGeom& g) {
  const int64_t pixels = (int64_t)g.N * g.P * g.Q;
  const FastDiv dq = make_fastdiv((uint32_t)g.Q), dpq = make_fastdiv((uint32_t)(g.P * g.Q));
  const dim3 grid(splits, ceil_div(g.K, 64)), block(256);
  const int per = ceil_div(pixels, splits);
  if constexpr (sizeof(T) == 2) {
    if (stem_ok(DT_BF16, g)) {
      const int chunk = ceil_div(per, STEM_BM) * STEM_BM;
      if (g.C == 1) OSEQ_LAUNCH((conv_stem_wgrad_kernel<T, 1>), grid, block, 0, st, x, dz, dst, g, chunk, dq, dpq);
      else if (g.C == 2) OSEQ_LAUNCH((conv_stem_wgrad_kernel<T, 2>), grid, block, 0, st, x, dz, dst, g, chunk, dq, dpq);
      else OSEQ_LAUNCH((conv_stem_wgrad_kernel<T, 3>), grid, block, 0, st, x, dz, dst, g, chunk, dq, dpq);
      return;
    }
  }
  OSEQ_LAUNCH(conv_wgrad_smallc_kernel<T>, grid, block, 0, st, x, dz, dst, g, ceil_div(per, 64) * 64, dq, dpq);
}

// partial: [splits][K][R*S*C] floats; splits: any number, as conv_smallc_wgrad_splits gives it
void launch_conv_wgrad_smallc(hipStream_t st, int dt, const void* x, const void* dz, float* dw, float* partial, int splits,
                              const ConvGeom& g) {
  float* dst = splits > 1 ? partial : dw;
  if (dt == DT_F32) launch_wgrad_smallc_t<float>(st, (const float*)x, (const float*)dz, dst, splits, g);
  else if (dt == DT_BF16) launch_wgrad_smallc_t<bf16_t>(st, (const bf16_t*)x, (const bf16_t*)dz, dst, splits, g);
  else launch_wgrad_smallc_t<f16_t>(st, (const f16_t*)x, (const f16_t*)dz, dst, splits, g);
  if (splits > 1) {
    const int64_t n = (int64_t)g.K * g.R * g.S * g.C;
    OSEQ_LAUNCH(partial_reduce_kernel, dim3(ceil_div(n, 16)), dim3(256), 0, st, partial, dw, n, splits);
  }
}

// 32-bit indices: every tensor of the layer has fewer than 2^30 elements (a step past the end still counts)
static bool direct_small(const ConvGeom& g) {
  const int64_t most = (int64_t)1 << 30;
  return (int64_t)g.N * g.P * g.Q * g.K < most && (int64_t)g.N * g.H * g.W * g.C < most && (int64_t)g.K * g.R * g.S * g.C < most;
}
// the choice of index type and vector width (VEC: four channels per load; the caller has looked at the channel count and at
// the tensors' alignment, weights may start at any element)
#define DIRECT_LAUNCH(KERNEL, T, VEC, ...)                                                       \
  {                                                                                              \
    if (direct_small(g)) {                                                                       \
      if (VEC) OSEQ_LAUNCH((KERNEL<T, int, 4>), grid, block, 0, st, __VA_ARGS__);                \
      else OSEQ_LAUNCH((KERNEL<T, int, 1>), grid, block, 0, st, __VA_ARGS__);                    \
    } else {                                                                                     \
      OSEQ_LAUNCH((KERNEL<T, int64_t, 1>), grid, block, 0, st, __VA_ARGS__);                     \
    }                                                                                            \
  }

void launch_conv_fwd_direct(hipStream_t st, int dt, const void* x, const void* w, const float* bias, void* out,
                            const ConvGeom& g, int relu, const ConvEval& ev) {
  const int64_t total = (int64_t)g.N * g.P * g.Q * g.K;
  dim3 grid(ceil_div(total, 256)), block(256);
  const uintptr_t mask = dt == DT_F32 ? 15 : 7;  // four elements
  const bool vec = g.C % 4 == 0 && (((uintptr_t)x | (uintptr_t)w) & mask) == 0;
#define CALL(T)                                                                                                              \
  DIRECT_LAUNCH(conv_fwd_direct_kernel, T, vec, (const T*)x, (const T*)w, bias, (T*)out, g, relu, ev.affine, (const T*)ev.skip)
  if (dt == DT_F32) CALL(float) else if (dt == DT_BF16) CALL(bf16_t) else CALL(f16_t)
#undef CALL
}

void launch_conv_dgrad_direct(hipStream_t st, int dt, const void* dz, const void* w, const void* addend, void* dx,
                              const ConvGeom& g) {
  const int64_t total = (int64_t)g.N * g.H * g.W * g.C;
  dim3 grid(ceil_div(total, 256)), block(256);
  const bool vec = g.K % 4 == 0 && ((uintptr_t)dz & (dt == DT_F32 ? 15 : 7)) == 0;
#define CALL(T) DIRECT_LAUNCH(conv_dgrad_direct_kernel, T, vec, (const T*)dz, (const T*)w, (const T*)addend, (T*)dx, g)
  if (dt == DT_F32) CALL(float) else if (dt == DT_BF16) CALL(bf16_t) else CALL(f16_t)
#undef CALL
}

void launch_conv_wgrad_direct(hipStream_t st, int dt, const void* x, const void* dz, float* dw, float* partial, int splits,
                              const ConvGeom& g) {
  const int64_t outputs = (int64_t)g.K * g.R * g.S * g.C;
  const int64_t pixels = (int64_t)g.N * g.P * g.Q;
  const int64_t chunk = (pixels + splits - 1) / splits;
  float* dst = splits > 1 ? partial : dw;
  dim3 grid(ceil_div(outputs, 256), splits), block(256);
#define CALL(T)                                                                                                              \
  {                                                                                                                          \
    if (direct_small(g)) OSEQ_LAUNCH((conv_wgrad_direct_kernel<T, int>), grid, block, 0, st, (const T*)x, (const T*)dz, dst, g, chunk); \
    else OSEQ_LAUNCH((conv_wgrad_direct_kernel<T, int64_t>), grid, block, 0, st, (const T*)x, (const T*)dz, dst, g, chunk);  \
  }
  if (dt == DT_F32) CALL(float) else if (dt == DT_BF16) CALL(bf16_t) else CALL(f16_t)
#undef CALL
  if (splits > 1)
    OSEQ_LAUNCH(partial_reduce_kernel, dim3(ceil_div(outputs, 16)), dim3(256), 0, st, partial, dw, outputs, splits);
}

}  // namespace oseq
