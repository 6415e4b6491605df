// Backward pass of a 1x1 layer of 64 input and 256 output channels and of the BatchNorm behind it, in one pass over its tensors
// (16-bit storage; the last layer of a bottleneck block and the projection shortcut in the first stage of the networks).
//
//   dz[m][k]  = scale * (dy - mean(dy) - xhat * mean(dy * xhat)),  dy = ReLU decisions of dA   (the BatchNorm's apply pass; as
//               scale * dy + (the two other factors of xhat's term at once) * (z - mean) + ..., two multiply-adds, two roundings less)
//   dx[m][c]  = sum over k of dz[m][k] * w[k][c]
//   dw[k][c]  = sum over pixels m of dz[m][k] * x[m][c]
//
// Apart, these are three kernels: the first reads dA and z and writes dz, the others read dz again, one of them x -- at 4.2 M
// pixels in bf16 1176 + 516 + 520 us for 6.6 + 2.7 + 2.7 GB.  Here a pixel's dz exists in LDS only, and its z too: that is the
// layer's own output, made again from the x that is here for the weight gradient (a third of the products, in the forward kernel's
// order, hence its bits).  Reading z (5.4 GB) was bound by HBM; without it (3.4 GB counted) the LDS (100 KB a tile; busy half of
// the cycles, a third of those conflicts) and the vector instructions around it take as long as memory.  us, z read -> made again,
// also where it is in memory anyway, without and with a BatchNorm in front: 4.2 M pixels 1134 -> 820, 1087 -> 905; 131 072
// 43 -> 35, 42 -> 38.5; 65 536 26 -> 23.5, 26.8 -> 25.9.  With dA per image z is the one large tensor to read, and always there:
// read, at the same three sizes, 811, 35.3 and 24.4 (made again 950, 38.4 and 26.7).
//
// A block of 512 threads (8 wavefronts, one block per CU: 256 blocks) walks a range of tiles of 64 pixels.  Per tile, two barriers:
// dz of the tile from z (LDS) and the pieces of dA and mask, requested a tile ahead, and the next tile's x into LDS; then every
// wavefront makes 32 pixels x 32 channels of half of dx (32x32x16 MFMAs, the transposed weights of its half of the depth in
// registers: from LDS they were most of its traffic), adds the tile to its 32 x 64 part of dw, whose accumulators (32 registers)
// live as long as the block, and makes its 32 channels of the next tile's z; dx goes through LDS to whole-row stores.
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
  __device__ static __forceinline__ v16f mma32(V a, V b, v16f c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
};
template <> struct Op<f16_t> {
  typedef v8h V;
  __device__ static __forceinline__ v16f mma32(V a, V b, v16f c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
};

constexpr int BC = 64, BK = 256, PM = 64, NT = 512;
constexpr int DP = BK + 16, ZP = BK + 8, XP = BC + 16, WP = BC + 8, OP = BC + 4;  // LDS row pitches: dz, z, x, weights; dx (floats)
constexpr size_t BWD1_LDS = (size_t)(PM * DP + PM * ZP + 2 * PM * XP + BK * WP) * 2 + (size_t)2 * PM * OP * 4;

struct Bwd1Args {
  int64_t M;           // pixels
  int tiles_per_block, relu;
  FastDiv div_hw;      // GV: pixels per image
};

// MS: ReLU decisions redone from z (0; none if relu is not set) or from the bits of mask (2); GV: dA is the gradient per image
// (both as in bn_bwd_apply_kernel), and z is read.  FOLD: x is the z of a BatchNorm + ReLU, fold its statistics.
// sums (with FOLD, or null): the block's row of the sums that the folded BatchNorm's backward pass begins with, dx being the gradient
// behind it and its z at hand (at 4.2 M pixels the pass over both took 183 us)
template <class T, int MS, bool GV, bool FOLD>
__global__ void __launch_bounds__(NT) conv1x1_bwd_kernel(const T* __restrict__ da, const T* __restrict__ z,
                                                         const uint8_t* __restrict__ mask, const float* __restrict__ stats,
                                                         const float* __restrict__ coef, const T* __restrict__ x,
                                                         const float* __restrict__ fold, const T* __restrict__ w,
                                                         const T* __restrict__ wt, T* __restrict__ dx, float* __restrict__ dw,
                                                         float* __restrict__ sums, Bwd1Args a) {
  typedef typename Op<T>::V V;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  T* Ds = reinterpret_cast<T*>(smem_raw);
  T* Zs = Ds + PM * DP;
  T* Xs = Zs + PM * ZP;  // two tiles
  T* Ws = Xs + 2 * PM * XP;
  float* Os = reinterpret_cast<float*>(Ws + BK * WP);  // two halves of the sum

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int hg = lane >> 5, l32 = lane & 31;
  // weights: [256][64]
#pragma unroll
  for (int i = 0; i < (GV ? 0 : BC * BK / 8 / NT); ++i) {
    const int id = tid + i * NT, k = id / (BC / 8), c8 = id % (BC / 8);
    *reinterpret_cast<Chunk*>(&Ws[k * WP + c8 * 8]) = *reinterpret_cast<const Chunk*>(w + (int64_t)k * BC + c8 * 8);
  }
  // dx: a wavefront makes 32 pixels x 32 channels, half of the depth; its weights (their transpose) stay in registers
  const int drow = (wave & 1) * 32, dcol = ((wave >> 1) & 1) * 32, dk = (wave >> 2) * (BK / 2);
  V fd[BK / 2 / 16];
#pragma unroll
  for (int s = 0; s < BK / 2 / 16; ++s) fd[s] = *reinterpret_cast<const V*>(wt + (int64_t)(dcol + l32) * BK + dk + s * 16 + hg * 8);
  // this thread's pieces: channels [8 * (tid % 32), + 8) of dz for pixels tid / 32 + 16 i, channels [8 * (tid % 8), + 8) of x and dx
  // for pixel tid / 8
  const int k0 = (tid & 31) * 8, pd = tid >> 5;
  const int c0 = (tid & 7) * 8, px = tid >> 3;
  float mean[8], scale[8], shift[8], cb[8], cg[8];  // cb, cg: the terms behind dy, times the scale
  load_f32<float, 8>(stats + k0, mean);
  load_f32<float, 8>(stats + BK + k0, cg);
  load_f32<float, 8>(stats + 2 * BK + k0, scale);
  if (MS == 0) load_f32<float, 8>(stats + 3 * BK + k0, shift);
#pragma unroll
  for (int k = 0; k < 8; ++k) { cb[k] = -scale[k] * coef[k0 + k]; cg[k] = -scale[k] * (cg[k] * coef[BK + k0 + k]); }
  float fsc[8], fsh[8], xmean[8], ss[8], qq[8];
  if (FOLD) {
    load_f32<float, 8>(fold + c0, xmean);
#pragma unroll
    for (int k = 0; k < 8; ++k) ss[k] = qq[k] = 0.f;
    load_f32<float, 8>(fold + 2 * BC + c0, fsc);
    load_f32<float, 8>(fold + 3 * BC + c0, fsh);
  }

  const int64_t ntiles = (a.M + PM - 1) / PM;
  const int64_t t0 = (int64_t)blockIdx.x * a.tiles_per_block;
  const int64_t t1 = t0 + a.tiles_per_block < ntiles ? t0 + a.tiles_per_block : ntiles;

  constexpr int ND = PM * (BK / 8) / NT;  // pieces of dz per thread
  Chunk ra[ND], rz[GV ? ND : 1], rx;
  unsigned rm[ND];
  auto gload_x = [&](int64_t t) {  // pixels past the last one read that one
    int64_t m = t * PM + px;
    m = m < a.M ? m : a.M - 1;
    rx = *reinterpret_cast<const Chunk*>(x + m * BC + c0);
  };
  auto gload = [&](int64_t t) {
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      int64_t m = t * PM + pd + i * (PM / ND);
      m = m < a.M ? m : a.M - 1;
      // (read once; non-temporal 1166 -> 1139 us at 4.2 M pixels, z under a pool 879 -> 904)
      if (GV) rz[i] = *reinterpret_cast<const Chunk*>(z + m * BK + k0);
      else ra[i] = __builtin_nontemporal_load(reinterpret_cast<const Chunk*>(da + m * BK + k0));
      rm[i] = MS == 2 ? mask[m * (BK / 8) + (tid & 31)] : 0u;
    }
    if (GV) {  // (the divisions stay behind the loads from memory)
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        int64_t md = t * PM + pd + i * (PM / ND);
        md = md < a.M ? md : a.M - 1;
        ra[i] = *reinterpret_cast<const Chunk*>(da + (int64_t)a.div_hw.div((uint32_t)md) * BK + k0);
      }
    }
  };
  auto xstore = [&](int64_t t) {  // tile t of x, as activations
    const Chunk c = FOLD ? bn_fold_chunk<T>(rx, fsc, fsh) : rx;
    *reinterpret_cast<Chunk*>(&Xs[(t & 1) * (PM * XP) + px * XP + c0]) = t * PM + px < a.M ? c : zero_chunk();
  };
  auto dzstore = [&](int64_t t) {
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const int p = pd + i * (PM / ND);
      const Vec<T, 8> va = __builtin_bit_cast(Vec<T, 8>, ra[i]);
      const Vec<T, 8> vz = GV ? __builtin_bit_cast(Vec<T, 8>, rz[GV ? i : 0]) : *reinterpret_cast<const Vec<T, 8>*>(&Zs[p * ZP + k0]);
      float r[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float zf = to_f32(vz.v[k]);
        bool on = true;
        if (MS == 2) on = (rm[i] >> k) & 1u;
        else if (a.relu) on = bn_affine(zf, scale[k], shift[k]) > 0.f;
        const float dy = on ? to_f32(va.v[k]) : 0.f;
        r[k] = __fmaf_rn(scale[k], dy, __fmaf_rn(cg[k], zf - mean[k], cb[k]));
      }
      const Chunk c = __builtin_bit_cast(Chunk, round_vec<T, 8>(r));
      *reinterpret_cast<Chunk*>(&Ds[p * DP + k0]) = t * PM + p < a.M ? c : zero_chunk();
    }
  };
  // z of tile t: the forward kernels' products (k_conv_pointwise.hip) in their order and their rounding, hence the values stored.  The
  // weights are the first operand: a lane has four neighbouring channels of a pixel, one store of 8 bytes.
  auto zstore = [&](int64_t t) {
    const T* xt = Xs + (t & 1) * (PM * XP) + l32 * XP + hg * 16;
    const T* wr = Ws + (wave * 32 + l32) * WP + hg * 16;
    v16f za[PM / 32];
#pragma unroll
    for (int i = 0; i < PM / 32; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) za[i][e] = 0.f;
#pragma unroll
    for (int q = 0; q < BC / 16; ++q) {
      const V fw = *reinterpret_cast<const V*>(wr + (q >> 1) * 32 + (q & 1) * 8);
#pragma unroll
      for (int i = 0; i < PM / 32; ++i)
        za[i] = Op<T>::mma32(fw, *reinterpret_cast<const V*>(xt + i * 32 * XP + (q >> 1) * 32 + (q & 1) * 8), za[i]);
    }
#pragma unroll
    for (int i = 0; i < PM / 32; ++i)
#pragma unroll
      for (int e = 0; e < 16; e += 4) {
        const float v[4] = {za[i][e], za[i][e + 1], za[i][e + 2], za[i][e + 3]};
        *reinterpret_cast<Vec<T, 4>*>(&Zs[(i * 32 + l32) * ZP + wave * 32 + 2 * e + 4 * hg]) = round_vec<T, 4>(v);
      }
  };

  v16f acc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;

  const int r16 = lane & 15;
  const int coff = (lane & 16) + 4 * (r16 & 3), prow = hg * 8 + (r16 >> 2);

  Chunk xz = zero_chunk(), xnext;  // this thread's piece of x as it was read: of tile t, of tile t + 1
  if (t0 < t1) {
    gload_x(t0);
    gload(t0);
    xstore(t0);
    xz = rx;
    gload_x(t0 + 1);
    if (!GV) {
      __syncthreads();
      zstore(t0);
      __syncthreads();
    }
  }
  for (int64_t t = t0; t < t1; ++t) {
    dzstore(t);
    xstore(t + 1);  // (a tile past the block's last one is never read)
    xnext = rx;
    if (t + 1 < t1) { gload(t + 1); gload_x(t + 2); }
    __syncthreads();
    // dx (the channels as rows: four neighbouring ones of a pixel to a lane)
    v16f o;
#pragma unroll
    for (int e = 0; e < 16; ++e) o[e] = 0.f;
#pragma unroll
    for (int s = 0; s < BK / 2 / 16; ++s)
      o = Op<T>::mma32(fd[s], *reinterpret_cast<const V*>(&Ds[(drow + l32) * DP + dk + s * 16 + hg * 8]), o);
#pragma unroll
    for (int e = 0; e < 16; e += 4) {
      const v4f q = {o[e], o[e + 1], o[e + 2], o[e + 3]};
      *reinterpret_cast<v4f*>(&Os[((wave >> 2) * PM + drow + l32) * OP + dcol + 2 * e + 4 * hg]) = q;
    }
    // dw: output channels [32 * wave, + 32), all input channels
    const T* xt = Xs + (t & 1) * (PM * XP);
#pragma unroll
    for (int s = 0; s < PM / 16; ++s) {
      const T* pa = Ds + (s * 16 + prow) * DP + wave * 32 + coff;
      const V fa = lds_tr_read8<V>(pa, pa + 4 * DP);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const T* pb = xt + (s * 16 + prow) * XP + j * 32 + coff;
        acc[j] = Op<T>::mma32(fa, lds_tr_read8<V>(pb, pb + 4 * XP), acc[j]);
      }
    }
    if (!GV && t + 1 < t1) zstore(t + 1);
    __syncthreads();
    const int64_t m = t * PM + px;
    const v4f* oa = reinterpret_cast<const v4f*>(&Os[px * OP + c0]);
    const v4f* ob = reinterpret_cast<const v4f*>(&Os[(PM + px) * OP + c0]);
    const v4f o0 = oa[0] + ob[0], o1 = oa[1] + ob[1];
    const float v[8] = {o0[0], o0[1], o0[2], o0[3], o1[0], o1[1], o1[2], o1[3]};
    const Vec<T, 8> r = round_vec<T, 8>(v);
    if (m < a.M) *reinterpret_cast<Vec<T, 8>*>(dx + m * BC + c0) = r;
    if (FOLD) {
      const Vec<T, 8> xv = __builtin_bit_cast(Vec<T, 8>, xz);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float zf = to_f32(xv.v[k]);
        const float dy = m < a.M && bn_affine(zf, fsc[k], fsh[k]) > 0.f ? to_f32(r.v[k]) : 0.f;
        ss[k] += dy;
        qq[k] = __fmaf_rn(dy, zf - xmean[k], qq[k]);
      }
    }
    xz = xnext;
  }

  if (FOLD && sums) {
    float xrstd[8];
    load_f32<float, 8>(fold + BC + c0, xrstd);
#pragma unroll
    for (int k = 0; k < 8; ++k) qq[k] *= xrstd[k];
    epi_stat_combine_nt<NT, BC>(reinterpret_cast<float*>(smem_raw), tid, ss, qq, sums + (int64_t)blockIdx.x * 2 * BC,
                                sums + ((int64_t)blockIdx.x * 2 + 1) * BC);
  }
  float* dst = dw + (int64_t)blockIdx.x * BK * BC;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) dst[(wave * 32 + 8 * (e >> 2) + 4 * hg + (e & 3)) * BC + j * 32 + (lane & 31)] = acc[j][e];
}

template <class T, int MS, bool GV, bool FOLD>
void launch_t(hipStream_t st, const void* da, const void* z, const uint8_t* mask, const float* stats, const float* coef, const void* x, const float* fold,
              const void* w, const void* wt, void* dx, float* dw, float* sums, int blocks, const Bwd1Args& a) {
  static bool attr_done = false;
  if (!attr_done) {
    (void)hipFuncSetAttribute((const void*)conv1x1_bwd_kernel<T, MS, GV, FOLD>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)BWD1_LDS);
    attr_done = true;
  }
  OSEQ_LAUNCH((conv1x1_bwd_kernel<T, MS, GV, FOLD>), dim3(blocks), dim3(NT), BWD1_LDS, st, (const T*)da, (const T*)z, mask, stats, coef, (const T*)x,
              fold, (const T*)w, (const T*)wt, (T*)dx, dw, sums, a);
}

template <class T, int MS, bool GV>
void launch_f(hipStream_t st, const void* da, const void* z, const uint8_t* mask, const float* stats, const float* coef, const void* x, const float* fold,
              const void* w, const void* wt, void* dx, float* dw, float* sums, int blocks, const Bwd1Args& a) {
  if (fold) launch_t<T, MS, GV, true>(st, da, z, mask, stats, coef, x, fold, w, wt, dx, dw, sums, blocks, a);
  else launch_t<T, MS, GV, false>(st, da, z, mask, stats, coef, x, fold, w, wt, dx, dw, sums, blocks, a);
}

template <class T>
void launch_dt(hipStream_t st, const void* da, const void* z, const uint8_t* mask, const float* stats, const float* coef, const void* x, const float* fold,
               const void* w, const void* wt, void* dx, float* dw, float* sums, int blocks, const Bwd1Args& a, bool gv) {
  if (mask && gv) launch_f<T, 2, true>(st, da, z, mask, stats, coef, x, fold, w, wt, dx, dw, sums, blocks, a);
  else if (mask) launch_f<T, 2, false>(st, da, z, mask, stats, coef, x, fold, w, wt, dx, dw, sums, blocks, a);
  else if (gv) launch_f<T, 0, true>(st, da, z, mask, stats, coef, x, fold, w, wt, dx, dw, sums, blocks, a);
  else launch_f<T, 0, false>(st, da, z, mask, stats, coef, x, fold, w, wt, dx, dw, sums, blocks, a);
}

// Four tiles a block.  A step of a 64 -> 256 and a 256 -> 256 block in bf16, us with separate kernels -> with this one in its form that
// reads z (which is slower than this one throughout, see above): 65 536 pixels 636 -> 566, 131 072 932 -> 811; below the line that
// gained too (16 384: 442 -> 413), down to one tile a block at 4096 (369 -> 344).
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

void launch_conv_bwd1x1(hipStream_t st, int dt, const void* da, const void* z, const void* mask, const float* stats, const float* coef, int relu,
                        int per_image, const void* x, const float* fold, const void* w, const void* wt, void* dx, float* dw, float* partial,
                        int splits, const ConvGeom& g, float* sums) {
  Bwd1Args a;
  a.M = (int64_t)g.N * g.P * g.Q;
  a.tiles_per_block = (int)(((a.M + PM - 1) / PM + splits - 1) / splits);
  a.relu = relu;
  a.div_hw = make_fastdiv((uint32_t)(per_image > 0 ? per_image : 1));
  float* dst = splits > 1 ? partial : dw;
  if (dt == DT_BF16) launch_dt<bf16_t>(st, da, z, (const uint8_t*)mask, stats, coef, x, fold, w, wt, dx, dst, sums, splits, a, per_image > 0);
  else launch_dt<f16_t>(st, da, z, (const uint8_t*)mask, stats, coef, x, fold, w, wt, dx, dst, sums, splits, a, per_image > 0);
  if (splits > 1) launch_wgrad_reduce(st, partial, dw, (int64_t)BK * BC, splits);
}

}  // namespace oseq
