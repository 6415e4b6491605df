// Backward pass of a 1x1 layer of 64 input and 256 output channels and of the BatchNorm behind it, in one pass over its tensors
// (16-bit storage; the last layer of a bottleneck block and the projection shortcut in the first stage of the networks).
//
//   dz[m][k]  = scale * (dy - mean(dy) - xhat * mean(dy * xhat)),  dy = ReLU decisions of dA   (the BatchNorm's apply pass)
//   dx[m][c]  = sum over k of dz[m][k] * w[k][c]
//   dw[k][c]  = sum over pixels m of dz[m][k] * x[m][c]
//
// Apart, these are three kernels: the first reads dA and z and writes dz, the others read dz again, one of them x -- at 4.2 M
// pixels in bf16 1176 + 516 + 520 us for 6.6 + 2.7 + 2.7 GB.  Here a pixel's dz exists in LDS only: 5.4 GB.  Bound by HBM.
//
// A block of 512 threads (8 wavefronts, one block per CU: 256 blocks) walks a range of tiles of 64 pixels.  Per tile: the pieces
// of dA, z, mask and x, requested a tile ahead, become dz and x in LDS (pixel-major); then every wavefront makes 16 pixels x 32
// channels of dx (16x16x32 MFMAs, the transposed weights stay in LDS) and adds the tile to its 32 x 64 part of dw, whose
// accumulators (32 registers) live as long as the block; dx goes through LDS to whole-row stores.  Two barriers a tile.
// The operands of the weight gradient come from the transposing LDS read (ds_read_b64_tr_b16), as in the other weight gradients.
#include "bn_fold.h"
#include "dev_common.h"
#include "epilogue.h"
#include "kernels.h"

namespace oseq {

namespace {

typedef __attribute__((ext_vector_type(16))) float v16f;
typedef __attribute__((ext_vector_type(4))) float v4f;
typedef __attribute__((ext_vector_type(8))) __bf16 v8bf;
typedef __attribute__((ext_vector_type(8))) _Float16 v8h;

template <class T> struct Op;
template <> struct Op<bf16_t> {
  typedef v8bf V;
  __device__ static __forceinline__ v4f mma16(V a, V b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
  __device__ static __forceinline__ v16f mma32(V a, V b, v16f c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
};
template <> struct Op<f16_t> {
  typedef v8h V;
  __device__ static __forceinline__ v4f mma16(V a, V b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
  __device__ static __forceinline__ v16f mma32(V a, V b, v16f c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
};

constexpr int BC = 64, BK = 256, PM = 64, NT = 512;
constexpr int DP = BK + 16, XP = BC + 16, WP = BK + 8, OP = BC + 4;  // LDS row pitches: dz, x, weights; dx (floats)
constexpr size_t BWD1_LDS = (size_t)(PM * DP + PM * XP + BC * WP) * 2 + (size_t)PM * OP * 4;

struct Bwd1Args {
  int64_t M;           // pixels
  int tiles_per_block, relu;
  FastDiv div_hw;      // GV: pixels per image
};

// MS: ReLU decisions redone from z (0; none if relu is not set) or from the bits of mask (2); GV: dA is the gradient per image
// (both as in bn_bwd_apply_kernel, whose dz this is, bit for bit).  FOLD: x is the z of a BatchNorm + ReLU, fold its statistics.
// sums (with FOLD, or null): the block's row of the sums that the folded BatchNorm's backward pass begins with, dx being the gradient
// behind it and its z at hand (at 4.2 M pixels the pass over both took 183 us)
template <class T, int MS, bool GV, bool FOLD>
__global__ void __launch_bounds__(NT) conv1x1_bwd_kernel(const T* __restrict__ da, const T* __restrict__ z,
                                                         const uint8_t* __restrict__ mask, const float* __restrict__ stats,
                                                         const float* __restrict__ coef, const T* __restrict__ x,
                                                         const float* __restrict__ fold, const T* __restrict__ wt,
                                                         T* __restrict__ dx, float* __restrict__ dw, float* __restrict__ sums,
                                                         Bwd1Args a) {
  typedef typename Op<T>::V V;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  T* Ds = reinterpret_cast<T*>(smem_raw);
  T* Xs = Ds + PM * DP;
  T* Ws = Xs + PM * XP;
  float* Os = reinterpret_cast<float*>(Ws + BC * WP);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // weights: [64][256]
#pragma unroll
  for (int i = 0; i < BC * BK / 8 / NT; ++i) {
    const int id = tid + i * NT, c = id / (BK / 8), k8 = id % (BK / 8);
    *reinterpret_cast<Chunk*>(&Ws[c * WP + k8 * 8]) = *reinterpret_cast<const Chunk*>(wt + (int64_t)c * BK + k8 * 8);
  }
  // this thread's pieces: channels [8 * (tid % 32), + 8) of dz for pixels tid / 32 + 16 i, channels [8 * (tid % 8), + 8) of x and dx
  // for pixel tid / 8
  const int k0 = (tid & 31) * 8, pd = tid >> 5;
  const int c0 = (tid & 7) * 8, px = tid >> 3;
  float mean[8], rstd[8], scale[8], shift[8], cb[8], cg[8];
  load_f32<float, 8>(stats + k0, mean);
  load_f32<float, 8>(stats + BK + k0, rstd);
  load_f32<float, 8>(stats + 2 * BK + k0, scale);
  if (MS == 0) load_f32<float, 8>(stats + 3 * BK + k0, shift);
#pragma unroll
  for (int k = 0; k < 8; ++k) { cb[k] = coef[k0 + k]; cg[k] = coef[BK + k0 + k]; }
  float fsc[8], fsh[8], xmean[8], xrstd[8], ss[8], qq[8];
  if (FOLD) {
    load_f32<float, 8>(fold + c0, xmean);
    load_f32<float, 8>(fold + BC + c0, xrstd);
#pragma unroll
    for (int k = 0; k < 8; ++k) ss[k] = qq[k] = 0.f;
    load_f32<float, 8>(fold + 2 * BC + c0, fsc);
    load_f32<float, 8>(fold + 3 * BC + c0, fsh);
  }

  const int64_t ntiles = (a.M + PM - 1) / PM;
  const int64_t t0 = (int64_t)blockIdx.x * a.tiles_per_block;
  const int64_t t1 = t0 + a.tiles_per_block < ntiles ? t0 + a.tiles_per_block : ntiles;

  constexpr int ND = PM * (BK / 8) / NT;  // pieces of dz per thread
  Chunk ra[ND], rz[ND], rx;
  unsigned rm[ND];
  auto gload = [&](int64_t t) {  // pixels past the last one read that one
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      int64_t m = t * PM + pd + i * (PM / ND);
      m = m < a.M ? m : a.M - 1;
      // (read once; non-temporal 1166 -> 1139 us at 4.2 M pixels, with the gradient per image 879 -> 904)
      const Chunk* zp = reinterpret_cast<const Chunk*>(z + m * BK + k0);
      rz[i] = GV ? *zp : __builtin_nontemporal_load(zp);
      if (!GV) ra[i] = __builtin_nontemporal_load(reinterpret_cast<const Chunk*>(da + m * BK + k0));
      rm[i] = MS == 2 ? mask[m * (BK / 8) + (tid & 31)] : 0u;
    }
    int64_t m = t * PM + px;
    m = m < a.M ? m : a.M - 1;
    rx = *reinterpret_cast<const Chunk*>(x + m * BC + c0);
    if (GV) {  // (the divisions stay behind the loads from memory)
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        int64_t md = t * PM + pd + i * (PM / ND);
        md = md < a.M ? md : a.M - 1;
        ra[i] = *reinterpret_cast<const Chunk*>(da + (int64_t)a.div_hw.div((uint32_t)md) * BK + k0);
      }
    }
  };
  auto sstore = [&](int64_t t) {
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const int p = pd + i * (PM / ND);
      const Vec<T, 8> va = __builtin_bit_cast(Vec<T, 8>, ra[i]), vz = __builtin_bit_cast(Vec<T, 8>, rz[i]);
      float r[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float zf = to_f32(vz.v[k]);
        bool on = true;
        if (MS == 2) on = (rm[i] >> k) & 1u;
        else if (a.relu) on = bn_affine(zf, scale[k], shift[k]) > 0.f;
        const float dy = on ? to_f32(va.v[k]) : 0.f;
        const float xh = (zf - mean[k]) * rstd[k];
        r[k] = scale[k] * (dy - cb[k] - xh * cg[k]);
      }
      const Chunk c = __builtin_bit_cast(Chunk, round_vec<T, 8>(r));
      *reinterpret_cast<Chunk*>(&Ds[p * DP + k0]) = t * PM + p < a.M ? c : zero_chunk();
    }
    const Chunk c = FOLD ? bn_fold_chunk<T>(rx, fsc, fsh) : rx;
    *reinterpret_cast<Chunk*>(&Xs[px * XP + c0]) = t * PM + px < a.M ? c : zero_chunk();
  };

  v16f acc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;

  const int l16 = lane & 15, kg = lane >> 4;
  const int drow = (wave & 3) * 16, dcol = (wave >> 2) * 32;
  const int hg = lane >> 5, r16 = lane & 15;
  const int coff = (lane & 16) + 4 * (r16 & 3), prow = hg * 8 + (r16 >> 2);

  if (t0 < t1) gload(t0);
  for (int64_t t = t0; t < t1; ++t) {
    sstore(t);
    const Vec<T, 8> xz = __builtin_bit_cast(Vec<T, 8>, rx);  // (FOLD: this thread's z for its piece of dx)
    __syncthreads();
    if (t + 1 < t1) gload(t + 1);
    // dx: 16 pixels x 32 channels
    v4f o[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[j][e] = 0.f;
#pragma unroll
    for (int s = 0; s < BK / 32; ++s) {
      const V fa = *reinterpret_cast<const V*>(&Ds[(drow + l16) * DP + s * 32 + kg * 8]);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const V fb = *reinterpret_cast<const V*>(&Ws[(dcol + j * 16 + l16) * WP + s * 32 + kg * 8]);
        o[j] = Op<T>::mma16(fa, fb, o[j]);
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) Os[(drow + 4 * kg + e) * OP + dcol + j * 16 + l16] = o[j][e];
    // dw: output channels [32 * wave, + 32), all input channels
#pragma unroll
    for (int s = 0; s < PM / 16; ++s) {
      const T* pa = Ds + (s * 16 + prow) * DP + wave * 32 + coff;
      const V fa = lds_tr_read8<V>(pa, pa + 4 * DP);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const T* pb = Xs + (s * 16 + prow) * XP + j * 32 + coff;
        acc[j] = Op<T>::mma32(fa, lds_tr_read8<V>(pb, pb + 4 * XP), acc[j]);
      }
    }
    __syncthreads();
    const int64_t m = t * PM + px;
    const v4f o0 = *reinterpret_cast<const v4f*>(&Os[px * OP + c0]), o1 = *reinterpret_cast<const v4f*>(&Os[px * OP + c0 + 4]);
    const float v[8] = {o0[0], o0[1], o0[2], o0[3], o1[0], o1[1], o1[2], o1[3]};
    const Vec<T, 8> r = round_vec<T, 8>(v);
    if (m < a.M) *reinterpret_cast<Vec<T, 8>*>(dx + m * BC + c0) = r;
    if (FOLD) {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float zf = to_f32(xz.v[k]);
        const float dy = m < a.M && bn_affine(zf, fsc[k], fsh[k]) > 0.f ? to_f32(r.v[k]) : 0.f;
        ss[k] += dy;
        qq[k] = __fmaf_rn(dy, (zf - xmean[k]) * xrstd[k], qq[k]);
      }
    }
  }

  if (FOLD && sums)
    epi_stat_combine_nt<NT, BC>(reinterpret_cast<float*>(smem_raw), tid, ss, qq, sums + (int64_t)blockIdx.x * 2 * BC,
                                sums + ((int64_t)blockIdx.x * 2 + 1) * BC);
  float* dst = dw + (int64_t)blockIdx.x * BK * BC;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) dst[(wave * 32 + 8 * (e >> 2) + 4 * hg + (e & 3)) * BC + j * 32 + (lane & 31)] = acc[j][e];
}

template <class T, int MS, bool GV, bool FOLD>
void launch_t(hipStream_t st, const void* da, const void* z, const uint8_t* mask, const float* stats, const float* coef, const void* x,
              const float* fold, const void* wt, void* dx, float* dw, float* sums, int blocks, const Bwd1Args& a) {
  static bool attr_done = false;
  if (!attr_done) {
    (void)hipFuncSetAttribute((const void*)conv1x1_bwd_kernel<T, MS, GV, FOLD>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)BWD1_LDS);
    attr_done = true;
  }
  OSEQ_LAUNCH((conv1x1_bwd_kernel<T, MS, GV, FOLD>), dim3(blocks), dim3(NT), BWD1_LDS, st, (const T*)da, (const T*)z, mask, stats, coef,
              (const T*)x, fold, (const T*)wt, (T*)dx, dw, sums, a);
}

template <class T, int MS, bool GV>
void launch_f(hipStream_t st, const void* da, const void* z, const uint8_t* mask, const float* stats, const float* coef, const void* x,
              const float* fold, const void* wt, void* dx, float* dw, float* sums, int blocks, const Bwd1Args& a) {
  if (fold) launch_t<T, MS, GV, true>(st, da, z, mask, stats, coef, x, fold, wt, dx, dw, sums, blocks, a);
  else launch_t<T, MS, GV, false>(st, da, z, mask, stats, coef, x, fold, wt, dx, dw, sums, blocks, a);
}

template <class T>
void launch_dt(hipStream_t st, const void* da, const void* z, const uint8_t* mask, const float* stats, const float* coef, const void* x,
               const float* fold, const void* wt, void* dx, float* dw, float* sums, int blocks, const Bwd1Args& a, bool gv) {
  if (mask && gv) launch_f<T, 2, true>(st, da, z, mask, stats, coef, x, fold, wt, dx, dw, sums, blocks, a);
  else if (mask) launch_f<T, 2, false>(st, da, z, mask, stats, coef, x, fold, wt, dx, dw, sums, blocks, a);
  else if (gv) launch_f<T, 0, true>(st, da, z, mask, stats, coef, x, fold, wt, dx, dw, sums, blocks, a);
  else launch_f<T, 0, false>(st, da, z, mask, stats, coef, x, fold, wt, dx, dw, sums, blocks, a);
}

// Four tiles a block.  A step of a 64 -> 256 and a 256 -> 256 block in bf16, us with separate kernels -> with this one: 65 536 pixels 636 -> 566,
// 131 072 932 -> 811; below the line it would gain too (16 384: 442 -> 413), down to one tile a block at 4096 (369 -> 344).
constexpr int64_t g_bwd1_min_pixels = 65536;

}  // namespace

bool conv_bwd1x1_ok(int dt, const ConvGeom& g) {
  return dt != DT_F32 && g.R == 1 && g.S == 1 && g.stride == 1 && g.pad == 0 && g.C == BC && g.K == BK &&
         (int64_t)g.N * g.P * g.Q >= g_bwd1_min_pixels && (int64_t)g.N * g.P * g.Q < (int64_t)1 << 32;
}

int conv_bwd1x1_splits(const ConvGeom& g) {
  const int64_t tiles = ((int64_t)g.N * g.P * g.Q + PM - 1) / PM, per = (tiles + 255) / 256;
  return (int)((tiles + per - 1) / per);  // no empty ranges
}

void launch_conv_bwd1x1(hipStream_t st, int dt, const void* da, const void* z, const void* mask, const float* stats, const float* coef,
                        int relu, int per_image, const void* x, const float* fold, const void* wt, void* dx, float* dw, float* partial,
                        int splits, const ConvGeom& g, float* sums) {
  Bwd1Args a;
  a.M = (int64_t)g.N * g.P * g.Q;
  a.tiles_per_block = (int)(((a.M + PM - 1) / PM + splits - 1) / splits);
  a.relu = relu;
  a.div_hw = make_fastdiv((uint32_t)(per_image > 0 ? per_image : 1));
  float* dst = splits > 1 ? partial : dw;
  if (dt == DT_BF16) launch_dt<bf16_t>(st, da, z, (const uint8_t*)mask, stats, coef, x, fold, wt, dx, dst, sums, splits, a, per_image > 0);
  else launch_dt<f16_t>(st, da, z, (const uint8_t*)mask, stats, coef, x, fold, wt, dx, dst, sums, splits, a, per_image > 0);
  if (splits > 1) launch_wgrad_reduce(st, partial, dw, (int64_t)BK * BC, splits);
}

}  // namespace oseq
