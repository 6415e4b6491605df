// 3x3, stride 1, 64 input channels, 16-bit storage, many pixels: forward and data gradient with the weights stationary.
//
// With 64 input channels the depth is only 576, and the patch kernel (k_conv_mfma.hip) spends its blocks on 18 steps of a
// few MFMAs, each with a barrier, a weight tile through LDS and three operand reads per two MFMAs, between a start-up that
// waits for HBM and an epilogue.  Here a block stays: a wavefront keeps the weights of its 32 output channels, all 576 of
// their depth, in registers as MFMA operands (144 of them), and the block walks tiles of up to 128 pixels.  The patch of a
// tile (its pixels and their halo, all 64 channels) goes through LDS once and serves all nine taps without a barrier in
// between: one 16-byte LDS read per MFMA, which is what bounds the loop (four SIMDs read 4 KB per 32 cycles, the LDS
// delivers 128 bytes per cycle).
//   block = 256 threads = 4 wavefronts: 2 groups of 32 channels x 2 groups of 64 pixels; two blocks per CU cover each
//   other's barriers and epilogues.  The next tile's patch is requested before the MFMAs of the current one and waits in
//   registers.  Results are channels x pixels: a lane holds four consecutive channels of a pixel, rounded in pairs,
//   through LDS, stored as 16-byte pieces of whole rows; the storing threads keep the channel sums for the BatchNorm that
//   follows, a tile at a time, and every WS3_FLUSH tiles add them up, in double, to one row of block sums (no fp32 chain is
//   longer than those of the patch kernel's rows of 128 pixels, however many tiles a block has).
// The data gradient is the same computation on dz with the taps in reverse and the transposed weights.
// Taken where the result is stored as it is (no bias, ReLU, skip connection or addend: those would need registers that are
// not there, 128 to 264 bytes of them spilled, 117 against 68 us for an inference layer) and from 131 072 pixels on, two
// tiles a block; see ws3_args for maps that the patch kernel's tiles fill.  64 -> 64 channels, bf16, patch kernel -> this
// one, us at 4.2 M pixels (4096 x 32 x 32): data gradient 478 -> 362, forward on a folded BatchNorm 513 -> 383, with the
// channel sums 562 -> 463; with rows that keep LDS reads apart (patch_rows_apart) 344 -> 324, 360 -> 350 and 453 -> 443 on another
// card.  Forward, sums finished, plus data gradient at the line, us a layer (a third is the weights' way
// into the registers): 137 984 pixels of 112 x 112 maps 82 -> 59, 125 440 of 56 x 56 67 -> 56, 132 300 of 21 x 21 58 -> 57.
#include "bn_fold.h"
#include "dev_common.h"
#include "epilogue.h"
#include "kernels.h"
#include "patch.h"

namespace oseq {
namespace {

template <class T> struct Mma3;
template <> struct Mma3<bf16_t> {
  typedef __attribute__((ext_vector_type(8))) __bf16 V;
  typedef __attribute__((ext_vector_type(16))) float A;
  __device__ static __forceinline__ A run(V a, V b, A c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
};
template <> struct Mma3<f16_t> {
  typedef __attribute__((ext_vector_type(8))) _Float16 V;
  typedef __attribute__((ext_vector_type(16))) float A;
  __device__ static __forceinline__ A run(V a, V b, A c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
};

constexpr int64_t WS3_MIN_PIXELS = 131072, WS3_MIN_WHOLE = 163840;
constexpr int WS3_C = 64, WS3_PX = 128, WS3_BLOCKS = 512;
constexpr int WS3_PITCH = WS3_C + 8;      // elements per staged position and per staged output row (144 bytes: 16
                                          // neighbouring positions read 16 bytes each from all 64 banks)
constexpr int WS3_SLOTS = 7;              // 16-byte pieces of a patch per thread
constexpr int WS3_MAX_POS = WS3_SLOTS * 256 / 8;
constexpr int WS3_PATCH = 20480;          // elements of a patch, its padded rows
constexpr int WS3_FLUSH = 16;             // tiles per row of sums: one addition per thread and tile

struct Ws3Args {
  int N, srcH, srcW, dstH, dstW, Ng, pad, flip;
  int TI, TR, TC;                 // tile: images x rows x columns of output pixels
  int tiles_r, tiles_c, NT;
  int row_pitch;                  // elements between the rows of a patch
  int flushes;                    // rows of sums per block
};

// FOLD: src is the z of a BatchNorm + ReLU, `fold` its [4][64] statistics tensor
template <class T, bool STAT, bool FOLD>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
conv_ws3x3_kernel(const T* __restrict__ src, const T* __restrict__ wmat, const float* __restrict__ fold, T* __restrict__ out,
                  float* __restrict__ stat_partial, Ws3Args a) {
  typedef typename Mma3<T>::V FV;
  typedef typename Mma3<T>::A v16f;
  typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
  constexpr int PITCH = WS3_PITCH;
  __shared__ __attribute__((aligned(16))) T patch[WS3_PATCH];
  __shared__ __attribute__((aligned(16))) T stg[WS3_PX * PITCH];
  // kept out of registers, of which the weights leave few: the folded BatchNorm's scale and shift, the threads' channel sums
  __shared__ __attribute__((aligned(16))) float ftab[FOLD ? 2 : 1][FOLD ? 64 : 4];
  __shared__ __attribute__((aligned(16))) float sums[STAT ? 4 : 1][STAT ? 256 * 4 : 4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 5, l32 = lane & 31;
  const int cgrp = wave & 1, pgrp = wave >> 1;
  const int n0 = blockIdx.y * 64;
  const int SR = a.TR + 2, SC = a.TC + 2, NPOS = a.TI * SR * SC, TP = a.TI * a.TR * a.TC;

  // the lane's weights: channel n0 + 32 cgrp + l32, tap t, depth elements [16 q + 8 g, + 8)
  FV wv[36];
  {
    const T* wrow = wmat + (int64_t)(n0 + cgrp * 32 + l32) * (9 * WS3_C) + g * 8;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) wv[t * 4 + q] = *reinterpret_cast<const FV*>(wrow + (a.flip ? 8 - t : t) * WS3_C + q * 16);
  }
  // this thread's pieces of a patch: channels [8 (tid % 8), + 8) of positions tid / 8 + 32 i.  Packed coordinates within the
  // tile: image, row, column; -1: no such position
  const int pc8 = (tid & 7) * 8;
  int pco[WS3_SLOTS];
#pragma unroll
  for (int i = 0; i < WS3_SLOTS; ++i) {
    const int e = (tid >> 3) + 32 * i;
    const int ti = e / (SR * SC), rr = e - ti * (SR * SC), sy = rr / SC, sx = rr - sy * SC;
    pco[i] = e < NPOS ? (ti << 16) | (sy << 8) | sx : -1;
  }
  if (FOLD && tid < 64) { ftab[0][tid] = fold[2 * WS3_C + tid]; ftab[1][tid] = fold[3 * WS3_C + tid]; }
  Chunk pr[WS3_SLOTS];
  unsigned pvalid = 0u;
  auto tile_origin = [&](int tile, int& ii, int& y0, int& x0) {
    const int ci = tile % a.tiles_c, t2 = tile / a.tiles_c;
    const int ri = t2 % a.tiles_r;
    ii = (t2 / a.tiles_r) * a.TI; y0 = ri * a.TR; x0 = ci * a.TC;
  };
  // Loads are unconditional (a position outside the image reads the tensor's first pixel) and zeroed when stored to LDS.
  auto pload = [&](int tile) {
    int ii, y0, x0;
    tile_origin(tile, ii, y0, x0);
    const T* base = src + (int64_t)ii * a.srcH * a.srcW * WS3_C + pc8;
    pvalid = 0u;
#pragma unroll
    for (int i = 0; i < WS3_SLOTS; ++i) {
      const int ti = pco[i] >> 16, y = y0 - a.pad + ((pco[i] >> 8) & 255), x = x0 - a.pad + (pco[i] & 255);
      const bool ok = pco[i] >= 0 && ii + ti < a.N && y >= 0 && y < a.srcH && x >= 0 && x < a.srcW;
      pr[i] = *reinterpret_cast<const Chunk*>(ok ? base + ((ti * a.srcH + y) * a.srcW + x) * WS3_C : src + pc8);
      pvalid |= ok ? 1u << i : 0u;
    }
  };
  auto pstore = [&]() {
    float fsc[8], fsh[8];
    if (FOLD) {
      load_f32<float, 8>(&ftab[0][pc8], fsc);
      load_f32<float, 8>(&ftab[1][pc8], fsh);
    }
#pragma unroll
    for (int i = 0; i < WS3_SLOTS; ++i) {
      Chunk v = pr[i];
      if (FOLD) v = bn_fold_chunk<T>(v, fsc, fsh);
      if (pco[i] >= 0)
        *reinterpret_cast<Chunk*>(&patch[__mul24(__mul24(pco[i] >> 16, SR) + ((pco[i] >> 8) & 255), a.row_pitch) + __mul24(pco[i] & 255, PITCH) + pc8]) = ((pvalid >> i) & 1u) ? v : zero_chunk();
    }
  };
  // LDS position of this lane's two pixels (tap (0, 0)); pixels past the tile's last one read its first
  int prow[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    int m = pgrp * 64 + p * 32 + l32;
    if (m >= TP) m = 0;
    const int ti = m / (a.TR * a.TC), rr = m - ti * (a.TR * a.TC), tr = rr / a.TC, tc = rr - tr * a.TC;
    prow[p] = (ti * SR + tr) * a.row_pitch + tc * PITCH + g * 8;
  }
  // this thread's rows of the staged results: packed coordinates as above
  const int c8 = (tid & 7) * 8, erow = tid >> 3;
  int oco[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = erow + 32 * i;
    const int ti = m / (a.TR * a.TC), rr = m - ti * (a.TR * a.TC), tr = rr / a.TC, tc = rr - tr * a.TC;
    oco[i] = m < TP ? (ti << 16) | (tr << 8) | tc : -1;
  }
  // STAT: the threads' sums as one row; a channel's 32 threads are every eighth
  auto flush = [&](int row) {
    int id = tid;
    asm volatile("" : "+v"(id));  // (addresses made here and not kept in registers over the loop: those would be spilled)
    if (id < 128) {
      const int which = id >> 6, c = id & 63;
      const float* p = &sums[which * 2 + ((c & 7) >> 2)][(c >> 3) * 4 + (c & 3)];
      double t = 0.0;
#pragma unroll 4
      for (int r = 0; r < 32; ++r) t += (double)p[r * 32];
      stat_partial[(((int64_t)row * gridDim.x + blockIdx.x) * 2 + which) * a.Ng + n0 + c] = (float)t;
    }
  };
  int summed = 0, row = 0;  // tiles in the sums, rows written

  int tile = blockIdx.x;  // < NT
  pload(tile);
  if (FOLD) __syncthreads();  // the table
  pstore();
  __syncthreads();
  const int row1 = a.row_pitch, row2 = 2 * a.row_pitch;
  for (;;) {
    const int next = tile + gridDim.x;
    if (next < a.NT) pload(next);
    v16f acc[2];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[p][e] = 0.f;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const T* b = patch + prow[p] + (t >= 6 ? row2 : t >= 3 ? row1 : 0) + (t % 3) * PITCH + q * 16;
          acc[p] = Mma3<T>::run(wv[t * 4 + q], *reinterpret_cast<const FV*>(b), acc[p]);
        }
    __syncthreads();  // the patch has been read, the results of the tile before have been stored
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = cgrp * 32 + 8 * q + 4 * g;
        u32x2 o;
        o[0] = __builtin_bit_cast(uint32_t, from_f32x2<T>(acc[p][4 * q], acc[p][4 * q + 1]));
        o[1] = __builtin_bit_cast(uint32_t, from_f32x2<T>(acc[p][4 * q + 2], acc[p][4 * q + 3]));
        *reinterpret_cast<u32x2*>(&stg[(pgrp * 64 + p * 32 + l32) * PITCH + c]) = o;
      }
    if (next < a.NT) pstore();
    if (STAT && summed == WS3_FLUSH) { flush(row++); summed = 0; }
    __syncthreads();
    {
      int ii, y0, x0;
      tile_origin(tile, ii, y0, x0);
      T* base = out + (int64_t)ii * a.dstH * a.dstW * a.Ng + n0 + c8;
      Vec<T, 8> tv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        tv[i] = *reinterpret_cast<const Vec<T, 8>*>(&stg[(erow + 32 * i) * PITCH + c8]);
        const int ti = oco[i] >> 16, y = y0 + ((oco[i] >> 8) & 255), x = x0 + (oco[i] & 255);
        if (oco[i] >= 0 && ii + ti < a.N && y < a.dstH && x < a.dstW)
          *reinterpret_cast<Vec<T, 8>*>(base + (int64_t)((ti * a.dstH + y) * a.dstW + x) * a.Ng) = tv[i];
        else if (STAT) tv[i] = Vec<T, 8>{};  // not stored: counts as zero
      }
      if (STAT) {
        typedef typename Dot2<T>::V T2;
        T2 one2;
        one2[0] = from_f32<T>(1.f); one2[1] = from_f32<T>(1.f);
#pragma unroll
        for (int j = 0; j < 2; ++j) {  // channels 4j .. 4j + 3 of the thread's eight
          float s4[4] = {0.f, 0.f, 0.f, 0.f}, q4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int i = 0; i < 4; i += 2)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              T2 p2;
              p2[0] = tv[i].v[4 * j + k]; p2[1] = tv[i + 1].v[4 * j + k];
              s4[k] = Dot2<T>::run(p2, one2, s4[k]);
              q4[k] = Dot2<T>::run(p2, p2, q4[k]);
            }
          // (the tile from zero, then the total: squares of 16-bit values added to a long sum one pair at a time are rounded
          // down more often than up -- 1.3e-4 of the variance in fp16 where the mean is 40 deviations off)
          if (summed) {
            float s0[4], q0[4];
            load_f32<float, 4>(&sums[j][tid * 4], s0);
            load_f32<float, 4>(&sums[2 + j][tid * 4], q0);
#pragma unroll
            for (int k = 0; k < 4; ++k) { s4[k] += s0[k]; q4[k] += q0[k]; }
          }
          store_f32<float, 4>(&sums[j][tid * 4], s4);
          store_f32<float, 4>(&sums[2 + j][tid * 4], q4);
        }
        ++summed;
      }
    }
    if (next >= a.NT) break;
    tile = next;
  }
  if (STAT) {
    __syncthreads();
    flush(row++);
    if (row < a.flushes && tid < 128)  // a block with one tile less than others may have a row less
      stat_partial[(((int64_t)row * gridDim.x + blockIdx.x) * 2 + (tid >> 6)) * a.Ng + n0 + (tid & 63)] = 0.f;
  }
}

// tile of at most 128 pixels and WS3_MAX_POS staged positions with the fewest tiles (then the smallest halo)
bool ws3_geometry(int N, int dstH, int dstW, Ws3Args& a) {
  int64_t best = -1;
  int best_pos = 0;
  for (int tc = 1; tc <= dstW && tc <= 64; ++tc) {
    int tr = WS3_PX / tc;
    if (tr > dstH) tr = dstH;
    if (tr > 64) tr = 64;
    if (tr < 1) continue;
    int ti = (tr == dstH && tc == dstW) ? WS3_PX / (dstH * dstW) : 1;
    if (ti > N) ti = N;
    while (ti > 1 && ti * (tr + 2) * (tc + 2) > WS3_MAX_POS) --ti;
    while (tr > 1 && ti * (tr + 2) * (tc + 2) > WS3_MAX_POS) --tr;
    if (ti * (tr + 2) * (tc + 2) > WS3_MAX_POS || (ti > 1 && tr != dstH)) continue;
    const int pos = ti * (tr + 2) * (tc + 2);
    const int64_t nt = (int64_t)((N + ti - 1) / ti) * ((dstH + tr - 1) / tr) * ((dstW + tc - 1) / tc);
    if (best < 0 || nt < best || (nt == best && pos < best_pos)) {
      best = nt; best_pos = pos;
      a.TI = ti; a.TR = tr; a.TC = tc;
      a.tiles_r = (dstH + tr - 1) / tr; a.tiles_c = (dstW + tc - 1) / tc;
    }
  }
  if (best < 0 || best >= ((int64_t)1 << 30)) return false;
  a.NT = (int)best;
  a.row_pitch = patch_rows_apart(a.TC, a.TC + 2, WS3_PITCH * 2) / 2;
  if (a.TI * (a.TR + 2) * a.row_pitch > WS3_PATCH) a.row_pitch = (a.TC + 2) * WS3_PITCH;
  return true;
}

int ws3_blocks(const Ws3Args& a) {  // two blocks per CU over all channel groups
  const int groups = a.Ng / 64;
  const int b = WS3_BLOCKS / groups > 0 ? WS3_BLOCKS / groups : 1;
  return a.NT < b ? a.NT : b;
}
int ws3_flushes(const Ws3Args& a) { return ceil_div(ceil_div(a.NT, ws3_blocks(a)), WS3_FLUSH); }

template <class T>
void launch_ws3(hipStream_t st, const void* src, const void* wmat, const float* fold, void* out, float* stat_partial, const Ws3Args& a) {
  const dim3 grid(ws3_blocks(a), a.Ng / 64), block(256);
#define WS3_LAUNCH(ST, FO)                                                                                                   \
  OSEQ_LAUNCH((conv_ws3x3_kernel<T, ST, FO>), grid, block, 0, st, (const T*)src, (const T*)wmat, fold, (T*)out, stat_partial, a)
  if (fold) { if (stat_partial) WS3_LAUNCH(true, true); else WS3_LAUNCH(false, true); }
  else if (stat_partial) WS3_LAUNCH(true, false);
  else WS3_LAUNCH(false, false);
#undef WS3_LAUNCH
}

}  // namespace

// From the layer shape only: 64 channels in, two tiles per block, the offsets within a tile's images in 32 bits.
static bool ws3_args(int dt, int N, int dstH, int dstW, int srcC, int Ng, int R, int S, int stride, Ws3Args& a) {
  if (dt == DT_F32 || R != 3 || S != 3 || stride != 1 || srcC != WS3_C || Ng % 64 != 0 || Ng > 64 * WS3_BLOCKS) return false;
  if ((int64_t)N * dstH * dstW < WS3_MIN_PIXELS) return false;
  if ((int64_t)(dstH + 2) * (dstW + 2) * 64 * (int64_t)(srcC > Ng ? srcC : Ng) >= ((int64_t)1 << 31)) return false;
  // Maps that tiles of 128 pixels fill (32 x 32, 8 x 8): the patch kernel wastes nothing there, and with less than two and a
  // half tiles a block it is ahead.  Four 64 -> 64 layers of a step, forward, sums and data gradients, us in bf16 and fp16,
  // patch kernel and this one: 131 072 pixels 192, 197 and 200, 200; 163 840: 214, 221 and 216, 217; 196 608: 242, 254 and
  // 237, 236; 131 072 of 8 x 8 maps: 193, 200 and 201, 199.
  const bool whole = dstH * dstW <= WS3_PX ? WS3_PX % (dstH * dstW) == 0 : WS3_PX % dstW == 0 && dstH % (WS3_PX / dstW) == 0;
  if (whole && (int64_t)N * dstH * dstW * (Ng / 64) < WS3_MIN_WHOLE) return false;
  a = Ws3Args{};
  a.N = N; a.dstH = dstH; a.dstW = dstW; a.Ng = Ng;
  if (!ws3_geometry(N, dstH, dstW, a)) return false;
  a.flushes = ws3_flushes(a);
  return true;
}
bool conv_ws3x3_ok(int dt, int N, int dstH, int dstW, int srcC, int Ng, int R, int S, int stride) {
  Ws3Args a;
  return ws3_args(dt, N, dstH, dstW, srcC, Ng, R, S, stride, a);
}
int conv_ws3x3_stat_blocks(const ConvGeom& g) {
  Ws3Args a;
  return ws3_args(DT_BF16, g.N, g.P, g.Q, g.C, g.K, g.R, g.S, g.stride, a) ? ws3_blocks(a) * a.flushes : 0;
}

void launch_conv_fwd_ws3x3(hipStream_t st, int dt, const void* x, const void* w, void* out, float* stat_partial, const ConvGeom& g,
                           const float* fold) {
  Ws3Args a;
  if (!ws3_args(dt, g.N, g.P, g.Q, g.C, g.K, g.R, g.S, g.stride, a)) return;
  a.srcH = g.H; a.srcW = g.W; a.pad = g.pad; a.flip = 0;
  if (dt == DT_BF16) launch_ws3<bf16_t>(st, x, w, fold, out, stat_partial, a);
  else launch_ws3<f16_t>(st, x, w, fold, out, stat_partial, a);
}

// wt: the (C_in, kh, kw, C_out) transpose of the weights; C_out is 64
void launch_conv_dgrad_ws3x3(hipStream_t st, int dt, const void* dz, const void* wt, void* dx, const ConvGeom& g) {
  Ws3Args a;
  if (!ws3_args(dt, g.N, g.H, g.W, g.K, g.C, g.R, g.S, g.stride, a)) return;
  a.srcH = g.P; a.srcW = g.Q; a.pad = g.R - 1 - g.pad; a.flip = 1;
  if (dt == DT_BF16) launch_ws3<bf16_t>(st, dz, wt, nullptr, dx, nullptr, a);
  else launch_ws3<f16_t>(st, dz, wt, nullptr, dx, nullptr, a);
}

}  // namespace oseq
