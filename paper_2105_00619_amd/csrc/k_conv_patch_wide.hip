// 3x3 convolutions of stride 1 in 16 bits, forward and data gradient, with block tiles of 256 pixels x 256 or 128 channels: the
// patch kernel (k_conv_mfma.hip) for layers that give every CU such a tile.
//
// A wavefront of the patch kernel has a tile of 64 x 64: four operand reads from LDS per four MFMAs, 128 bytes a cycle, all that LDS
// delivers, before the weights are written there.  Here one wavefront per SIMD has 128 x 128 (or 128 x 64): half (three quarters) of
// the reads per MFMA, in 512 registers, 256 of them accumulators.  Nobody else runs while it waits, so nothing may wait: operands of
// a depth step (16 values) are read during the step before, weights travel from L2 two taps ahead of their store to LDS, the next
// channel chunk's patch five steps and more, and every access has its place between two MFMAs (the slots of the loop), as have the
// instructions of a folded BatchNorm, a few to a slot (a piece's thirty in one slot: 8 % of the loop's cycles).
// 256 -> 256 channels over 262 144 pixels, bf16, in a step (us, patch kernel -> this): forward with sums on a folded BatchNorm
// 338 -> 280, without sums 329 -> 269, data gradient with the sums of the BatchNorm in front 343 -> 308; 128 and 256 channels over
// 131 072 and 32 768 pixels in inference, on 256 x 128, 48.6 -> 40.8.  A tile's loop takes 96 000 cycles for 73 700 of MFMAs, and the
// clock falls from 2.2 to 1.7 GHz under it: it is the power that bounds these layers (fewer idle cycles run at a lower clock; the
// library's product of the same sizes takes 341), which is why the bytes read from LDS count.
//   LDS: 2 patch buffers, 3 weight stages [BN][80 B], address tables; the epilogue's rows in their place.
#include <algorithm>

#include "bn_fold.h"
#include "dev_common.h"
#include "epilogue.h"
#include "kernels.h"
#include "patch.h"

namespace oseq {

namespace {

typedef __attribute__((ext_vector_type(16))) float v16f;
template <class T> struct Op;
template <> struct Op<bf16_t> {
  typedef __attribute__((ext_vector_type(8))) __bf16 V;
  __device__ static __forceinline__ void mma(const V& a, const V& b, v16f& c) { c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
};
template <> struct Op<f16_t> {
  typedef __attribute__((ext_vector_type(8))) _Float16 V;
  __device__ static __forceinline__ void mma(const V& a, const V& b, v16f& c) { c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
};

constexpr int ROWS = 256;                 // pixels of a tile
constexpr int CCE = 32, PITCH = CCE + 8;  // channels of a chunk, elements of a position in LDS
constexpr int NSLOT = PATCH_WIDE_MAX_POS * 4 / 256;  // 16-byte pieces of a patch per thread
constexpr int HR = 32;                    // rows of an epilogue pass in fp32
// bytes in front of the buffers: out_off[ROWS] (int64), apos[ROWS] (int), 1 KB that pieces beyond the patch are written to
constexpr int HEAD = ROWS * 8 + ROWS * 4 + 1024;

constexpr int epi_bytes(int bn) { return std::max(ROWS * (bn + 8) * 2, 2 * HR * (bn + 4) * 4); }

// EVAL, STAT and what bias, addend and a.relu are then: as conv3x3_patch_kernel; ADD: an addend (STAT 0)
template <class T, int NI, int STAT, bool FOLD, bool EVAL, bool ADD>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
conv3x3_wide_kernel(const T* __restrict__ src, const T* __restrict__ wmat, const float* __restrict__ bias,
                    const T* __restrict__ addend, T* __restrict__ out, float* __restrict__ stat_partial, PatchWideArgs a) {
  typedef typename Op<T>::V V;
  constexpr int MI = ROWS / 64, BN = 64 * NI;
  constexpr int NW = BN / 64;  // weight pieces per thread and tap
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  int64_t* out_off = reinterpret_cast<int64_t*>(smem_raw);
  int* apos = reinterpret_cast<int*>(out_off + ROWS);
  T* patch = reinterpret_cast<T*>(smem_raw + HEAD);
  const int PBUF = a.patch_elems;
  T* Bs = patch + 2 * PBUF;
  int* src_off = reinterpret_cast<int*>(Bs + 2 * BN * PITCH);  // (in the third weight stage, which the loop is the first to fill)

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, g = lane >> 5, l32 = lane & 31;
  int bx = blockIdx.x, by = blockIdx.y;
  if (a.xcd_group == 2) {  // the channel blocks of a row tile on one XCD, as in the patch kernel
    const unsigned lin = blockIdx.x + gridDim.x * blockIdx.y;
    const unsigned xcd = lin & 7u, slot = lin >> 3;
    bx = (int)((slot / gridDim.y) * 8u + xcd); by = (int)(slot % gridDim.y);
    if (bx >= a.row_blocks) return;
  }
  const int n0c = by * BN;
  const int srcC = a.srcC, SC = a.SC, RPE = a.row_pitch / (int)sizeof(T);

  // ---- address tables: offsets from the tile's first image ----------------------------------------------------------
  const int t2 = a.div_tiles_c.div(bx), ci = bx - t2 * a.tiles_c, i2 = a.div_tiles_r.div(t2), ri = t2 - i2 * a.tiles_r;
  const int n_first = i2 * a.TI;
  for (int e = tid; e < a.NPOS; e += 256) {
    const int ti = a.div_image.div(e), rr = e - ti * (a.SR * SC);
    const int sy = a.div_row.div(rr), sx = rr - sy * SC;
    const int y = ri * a.TR - a.pad + sy, x = ci * a.TC - a.pad + sx;
    const bool in = n_first + ti < a.N && y >= 0 && y < a.srcH && x >= 0 && x < a.srcW;
    src_off[e] = in ? ((ti * a.srcH + y) * a.srcW + x) * srcC : -1;
  }
  {
    int64_t off = -1;
    int ap = 0;
    if (tid < a.TP) {
      const int ti = a.div_tile.div(tid), rr = tid - ti * (a.TR * a.TC);
      const int tr = a.div_tcol.div(rr), tc = rr - tr * a.TC;
      const int n = n_first + ti, p = ri * a.TR + tr, q = ci * a.TC + tc;
      ap = (ti * a.SR + tr) * RPE + tc * PITCH;
      if (n < a.N && p < a.dstH && q < a.dstW) off = (((int64_t)n * a.dstH + p) * a.dstW + q) * a.Ng;
    }
    out_off[tid] = off;
    apos[tid] = ap;
  }
  __syncthreads();

  // ---- loaders: a uniform address and a thread's own 32-bit offset -----------------------------------------------------
  const char* sbase = reinterpret_cast<const char*>(src + (int64_t)n_first * a.srcH * a.srcW * srcC);
  uint32_t poff[NSLOT];
  int pdst[NSLOT];  // LDS byte offset from the patch buffer (pieces beyond the patch: negative, in front of both buffers)
  unsigned pvalid = 0u;
#pragma unroll
  for (int sl = 0; sl < NSLOT; ++sl) {
    const int pos = sl * 64 + (tid >> 2), v = tid & 3;
    poff[sl] = (uint32_t)v * 16u;
    pdst[sl] = 0;
    if (pos < a.NPOS) {
      const int o = src_off[pos];
      if (o >= 0) { poff[sl] += (uint32_t)o * (uint32_t)sizeof(T); pvalid |= 1u << sl; }
      const int prow = a.div_row.div(pos);
      pdst[sl] = (prow * RPE + (pos - prow * SC) * PITCH) * (int)sizeof(T) + v * 16;
    } else {
      pdst[sl] = -1;
    }
  }
  unsigned char* const pbytes = reinterpret_cast<unsigned char*>(patch);
  unsigned char* const spare = smem_raw + HEAD - 1024 + lane * 16;
  Chunk PR[NSLOT];
  auto patch_load = [&](int sl, int chunk) { PR[sl] = *reinterpret_cast<const Chunk*>(sbase + (size_t)chunk * (CCE * sizeof(T)) + poff[sl]); };
  float fsc[8], fsh[8];  // FOLD: scale and shift of the chunk's channels [(tid & 3) * 8, + 8)
  auto fold_load = [&](int chunk) {
    if (FOLD) {
      load_f32<float, 8>(a.fold + 2 * srcC + chunk * CCE + (tid & 3) * 8, fsc);
      load_f32<float, 8>(a.fold + 3 * srcC + chunk * CCE + (tid & 3) * 8, fsh);
    }
  };
  auto patch_fold = [&](int sl, int k) {  // two of a piece's eight values
    if (FOLD) PR[sl][k] = bn_fold_pair<T>(PR[sl][k], fsc[2 * k], fsh[2 * k], fsc[2 * k + 1], fsh[2 * k + 1]);
  };
  auto patch_store = [&](int sl, int buf) {
    Chunk v = PR[sl];
    if (!((pvalid >> sl) & 1u)) v = zero_chunk();
    unsigned char* d = pbytes + buf * PBUF * (int)sizeof(T) + pdst[sl];
    if (pdst[sl] < 0) d = spare;
    *reinterpret_cast<Chunk*>(d) = v;
  };
  const int Kg = 9 * srcC;
  const char* wbase = reinterpret_cast<const char*>(wmat + (int64_t)n0c * Kg);
  const uint32_t woff = (uint32_t)((tid >> 2) * Kg + (tid & 3) * 8) * (uint32_t)sizeof(T);
  Chunk WR[3][NW];  // weight tiles on their way: that of step tile i in number i % 3
  const int last_chunk = srcC / CCE - 1;
  auto w_load = [&](int gen, int tap, int chunk) {  // (chunks behind the last: the last once more)
    const int c = chunk > last_chunk ? last_chunk : chunk;
    const int tp = a.flip ? 8 - tap : tap;
    const char* p = wbase + (int64_t)(tp * srcC + c * CCE) * (int)sizeof(T);
#pragma unroll
    for (int i = 0; i < NW; ++i) WR[gen][i] = *reinterpret_cast<const Chunk*>(p + (int64_t)(64 * i) * Kg * (int)sizeof(T) + woff);
  };
  const int wdst = (tid >> 2) * PITCH + (tid & 3) * 8;
  auto w_store = [&](int gen, int i) { *reinterpret_cast<Chunk*>(&Bs[(gen * BN + 64 * i) * PITCH + wdst]) = WR[gen][i]; };

  // ---- prologue -----------------------------------------------------------------------------------------------------
#pragma unroll
  for (int sl = 0; sl < NSLOT; ++sl) patch_load(sl, 0);
  fold_load(0);
  w_load(0, 0, 0);
  w_load(1, 1, 0);
  w_load(2, 2, 0);
#pragma unroll
  for (int sl = 0; sl < NSLOT; ++sl) {
#pragma unroll
    for (int k = 0; k < 4; ++k) patch_fold(sl, k);
    patch_store(sl, 0);
  }
#pragma unroll
  for (int i = 0; i < NW; ++i) { w_store(0, i); w_store(1, i); }
  w_load(0, 3, 0);
  w_load(1, 4, 0);
  __syncthreads();

  int arow[MI];
#pragma unroll
  for (int i = 0; i < MI; ++i) arow[i] = apos[wm * (32 * MI) + i * 32 + l32] + g * 16;
  const int brow = (wn * (BN / 2) + l32) * PITCH + g * 16;

  v16f acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  V fa[2][MI], fb[2][NI];  // operands of this step and of the next
#pragma unroll
  for (int i = 0; i < MI; ++i) fa[0][i] = *reinterpret_cast<const V*>(patch + arow[i]);
#pragma unroll
  for (int j = 0; j < NI; ++j) fb[0][j] = *reinterpret_cast<const V*>(Bs + brow + j * 32 * PITCH);

  // ---- a channel chunk: nine taps of two depth steps ------------------------------------------------------------------
  // Step s = 2 * tap + half works on the operands read in step s - 1.  Weight tile t + 2 goes to LDS in the first step of tap t
  // (the barrier behind tap t shows it, its first reads are in the second step of tap t + 1), tile t + 5 is requested in the second.
  // The next chunk's pieces are requested in the first three steps and stored in steps 7 to 15: before the barrier of tap 7, as
  // the first operands of the next chunk are read in step 17.
  for (int chunk = 0; chunk <= last_chunk; ++chunk) {
    const T* pcur = patch + (chunk & 1) * PBUF;
    const T* pnxt = patch + ((chunk & 1) ^ 1) * PBUF;
    const int cnext = chunk < last_chunk ? chunk + 1 : last_chunk;
#pragma unroll
    for (int s = 0; s < 18; ++s) {
      const int t = s >> 1, h = s & 1, cur = s & 1, nxt = cur ^ 1;
      const int sn = (s + 1) % 18, tn = sn >> 1, hn = sn & 1;
      const T* an = (s + 1 < 18 ? pcur : pnxt) + (tn / 3) * RPE + (tn % 3) * PITCH + hn * 8;
      const T* bn_ = Bs + ((t + (s & 1)) % 3) * BN * PITCH + brow + hn * 8;
      constexpr int Q = MI * NI;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        // the first operands that the next step needs first: a0, b0, b1, ...
        Op<T>::mma(fb[cur][q % NI], fa[cur][q / NI], acc[q / NI][q % NI]);
        __builtin_amdgcn_sched_barrier(0);
        // slot q: what is issued while the MFMA runs
        if (q == 0) fa[nxt][0] = *reinterpret_cast<const V*>(an + arow[0]);
        else if (q <= NI) fb[nxt][q - 1] = *reinterpret_cast<const V*>(bn_ + (q - 1) * 32 * PITCH);
        else if (q < MI + NI) fa[nxt][q - NI] = *reinterpret_cast<const V*>(an + arow[q - NI]);
        if (h == 0) {  // weight tile t + 2: from its registers to LDS
          if (q >= Q - 1 - NW && q < Q - 1) w_store((t + 2) % 3, q - (Q - 1 - NW));
        } else if (q == Q - 1) {
          w_load((t + 5) % 3, (t + 5) % 9, t + 5 < 9 ? chunk : chunk + 1);
        }
        if (s < 3 && q >= Q - 4 && q < Q - 1) patch_load(3 * s + q - (Q - 4), cnext);
        if (s == 0 && q == Q - 1) fold_load(cnext);
        if (s >= 7 && s < 16) {
          constexpr int F0 = Q == 16 ? 8 : 3;
          if (q >= F0 && q < F0 + 4) patch_fold(s - 7, q - F0);
          if (q == F0 + 4) patch_store(s - 7, (chunk & 1) ^ 1);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (h == 1) __syncthreads();
    }
  }

  // ---- epilogue -----------------------------------------------------------------------------------------------------
  // The weights are the MFMA's first operand, so a lane has four neighbouring channels of one pixel.
  constexpr int GROUPS = BN / 8, RG = 256 / GROUPS;
  const int c8 = (tid % GROUPS) * 8, erow = tid / GROUPS;
  if constexpr (ADD) {
    // something is added before the rounding: HR rows at a time through LDS as fp32, in two buffers
    float* ep = reinterpret_cast<float*>(patch);
    constexpr int EP_PITCH = BN + 4;
    float ss[8], qq[8];  // (no sums)
#pragma unroll
    for (int u = 0; u < 2 * MI; ++u) {
      float* e0 = ep + (u & 1) * HR * EP_PITCH;
      if (wm == u / MI) {
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
          for (int e = 0; e < 16; e += 4) {
            const v16f& c = acc[u % MI][j];
            const epi_v4f v = {c[e], c[e + 1], c[e + 2], c[e + 3]};
            *reinterpret_cast<epi_v4f*>(&e0[l32 * EP_PITCH + wn * (BN / 2) + j * 32 + 2 * e + 4 * g]) = v;
          }
      }
      __syncthreads();
      auto rowoff = [&](int row) -> int64_t { return out_off[u * HR + row]; };
      if constexpr (EVAL)
        epi_store_rows_nt<256, T, BN, HR, EPI_AFFINE, true, false>(e0, tid, n0c, bias, addend, nullptr, out, a.relu, rowoff, ss, qq, a.Ng);
      else
        epi_store_rows_nt<256, T, BN, HR, 0, true, false>(e0, tid, n0c, bias, addend, a.amask, out, a.relu, rowoff, ss, qq);
    }
    return;
  }
  // nothing to add: all rows at once, rounded, then stored row by row with the sums of what is stored
  T* const ep = patch;
  constexpr int EP = BN + 8, RT = 4, ITERS = ROWS / (RG * RT);  // rows of a thread and turn, turns
  int64_t ro[RT];
  Vec<T, 8> zv[RT];  // STAT 2: z of the next turn is requested before this turn's rows are stored
  auto z_load = [&](int it) {
#pragma unroll
    for (int k = 0; k < RT; ++k) {  // (rows that are not stored: the tensor's first)
      const int64_t o = out_off[(it * RT + k) * RG + erow];
      zv[k] = *reinterpret_cast<const Vec<T, 8>*>(addend + (o >= 0 ? o : 0) + n0c + c8);
    }
  };
  if constexpr (STAT == 2) z_load(0);
#pragma unroll
  for (int j = 0; j < NI; ++j)
#pragma unroll
    for (int e = 0; e < 16; e += 4) {
      const int c = wn * (BN / 2) + j * 32 + 2 * e + 4 * g;
      epi_v4f b4 = {0.f, 0.f, 0.f, 0.f}, s4 = b4;
      if (EVAL) {
        s4 = *reinterpret_cast<const epi_v4f*>(bias + n0c + c);
        b4 = *reinterpret_cast<const epi_v4f*>(bias + a.Ng + n0c + c);
      } else if (STAT != 2 && bias) {
        b4 = *reinterpret_cast<const epi_v4f*>(bias + n0c + c);
      }
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        float v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          v[k] = acc[i][j][e + k];
          if (EVAL) v[k] = bn_affine(v[k], s4[k], b4[k]);
          else if (STAT != 2 && bias) v[k] += b4[k];
          if (STAT != 2 && a.relu) v[k] = fmaxf(v[k], 0.f);
        }
        *reinterpret_cast<Vec<T, 4>*>(&ep[(wm * (32 * MI) + i * 32 + l32) * EP + c]) = round_vec<T, 4>(v);
      }
    }
  __syncthreads();
  float ss[8], qq[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) { ss[k] = 0.f; qq[k] = 0.f; }
  float mean[8], rstd[8], scale[8], shift[8];
  if constexpr (STAT == 2) {
    load_f32<float, 8>(bias + n0c + c8, mean);
    load_f32<float, 8>(bias + a.Ng + n0c + c8, rstd);
    load_f32<float, 8>(bias + 2 * a.Ng + n0c + c8, scale);
    load_f32<float, 8>(bias + 3 * a.Ng + n0c + c8, shift);
  }
#pragma unroll 1
  for (int it = 0; it < ITERS; ++it) {
    Vec<T, 8> t[RT], z[RT];
#pragma unroll
    for (int k = 0; k < RT; ++k) {
      const int row = (it * RT + k) * RG + erow;
      ro[k] = out_off[row];
      t[k] = *reinterpret_cast<const Vec<T, 8>*>(&ep[row * EP + c8]);
      if (STAT == 2) z[k] = zv[k];
    }
    if constexpr (STAT == 2) {
      if (it + 1 < ITERS) z_load(it + 1);
    }
#pragma unroll
    for (int k = 0; k < RT; ++k)
      if (ro[k] >= 0) *reinterpret_cast<Vec<T, 8>*>(out + ro[k] + n0c + c8) = t[k];
    if constexpr (STAT != 0) {
#pragma unroll
      for (int k = 0; k < RT; ++k)
        if (ro[k] < 0) t[k] = Vec<T, 8>{};  // a row that is not stored counts as zero
    }
    if constexpr (STAT == 1) {
      typename Dot2<T>::V one2, p2;
      one2[0] = from_f32<T>(1.f); one2[1] = from_f32<T>(1.f);
#pragma unroll
      for (int r = 0; r < RT; r += 2)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          p2[0] = t[r].v[k]; p2[1] = t[r + 1].v[k];
          ss[k] = Dot2<T>::run(p2, one2, ss[k]);
          qq[k] = Dot2<T>::run(p2, p2, qq[k]);
        }
    }
    if constexpr (STAT == 2) {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float zf = to_f32(z[r].v[k]);
          const float dy = !a.relu || bn_affine(zf, scale[k], shift[k]) > 0.f ? to_f32(t[r].v[k]) : 0.f;
          ss[k] += dy;
          qq[k] = __fmaf_rn(dy, (zf - mean[k]) * rstd[k], qq[k]);
        }
    }
  }
  if (STAT)
    epi_stat_combine<BN>(reinterpret_cast<float*>(patch), tid, ss, qq, stat_partial + ((int64_t)bx * 2 + 0) * a.Ng + n0c,
                         stat_partial + ((int64_t)bx * 2 + 1) * a.Ng + n0c);
}

template <class T, int NI, int STAT, bool FOLD, bool EVAL, bool ADD>
void launch_one(hipStream_t st, const void* src, const void* wmat, const float* bias, const void* addend, void* out, float* stat_partial,
                dim3 grid, size_t sm, const PatchWideArgs& a) {
  static bool done = false;
  if (!done) {
    (void)hipFuncSetAttribute((const void*)conv3x3_wide_kernel<T, NI, STAT, FOLD, EVAL, ADD>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    done = true;
  }
  OSEQ_LAUNCH((conv3x3_wide_kernel<T, NI, STAT, FOLD, EVAL, ADD>), grid, dim3(256), sm, st, (const T*)src, (const T*)wmat, bias,
              (const T*)addend, (T*)out, stat_partial, a);
}

template <class T, int NI>
void launch_shape(hipStream_t st, const void* src, const void* wmat, const float* bias, const void* addend, void* out, float* stat_partial,
                  const PatchArgs& shape) {
  PatchWideArgs a;
  static_cast<PatchArgs&>(a) = shape;
  dim3 grid(a.NT, a.Ng / (64 * NI));
  a.patch_elems = (a.TI * a.SR * a.row_pitch + 15) / 16 * 16 / (int)sizeof(T);
  a.row_blocks = (int)grid.x;
  a.div_image = make_fastdiv(a.SR * a.SC); a.div_row = make_fastdiv(a.SC);
  a.div_tile = make_fastdiv(a.TR * a.TC); a.div_tcol = make_fastdiv(a.TC);
  a.div_tiles_r = make_fastdiv(a.tiles_r); a.div_tiles_c = make_fastdiv(a.tiles_c);
  const int per_xcd = conv_patch_wide_rows_per_xcd(a.NT, (int)grid.y);
  a.xcd_group = per_xcd > 0 ? 2 : 0;
  if (per_xcd > 0) grid.x = per_xcd * 8;
  const size_t sm = conv_patch_wide_lds(64 * NI, a.patch_elems);
#define LAUNCH(STAT, FOLD, EVAL, ADD) launch_one<T, NI, STAT, FOLD, EVAL, ADD>(st, src, wmat, bias, addend, out, stat_partial, grid, sm, a)
  if (a.eval && addend) LAUNCH(0, false, true, true);
  else if (a.eval) LAUNCH(0, false, true, false);
  else if (a.bn_sums) LAUNCH(2, false, false, false);
  else if (addend) LAUNCH(0, false, false, true);  // (data gradient)
  else if (a.fold && stat_partial) LAUNCH(1, true, false, false);
  else if (a.fold) LAUNCH(0, true, false, false);
  else if (stat_partial) LAUNCH(1, false, false, false);
  else LAUNCH(0, false, false, false);
#undef LAUNCH
}

template <class T>
void launch_type(hipStream_t st, const void* src, const void* wmat, const float* bias, const void* addend, void* out, float* stat_partial,
                 int bn, const PatchArgs& a) {
  if (bn == 128) launch_shape<T, 2>(st, src, wmat, bias, addend, out, stat_partial, a);
  else launch_shape<T, 4>(st, src, wmat, bias, addend, out, stat_partial, a);
}

}  // namespace

// From the shape only.  Not where the 32 CUs of an XCD would have more rounds to do than the 256 have together: three channel blocks of
// 84 row tiles are 252 blocks, but 33 of them on an XCD (256 -> 384 channels over 21 504 pixels in bf16, us forward: narrow tiles 48, with
// the blocks grouped 66, without 38; 640 -> 640 over 25 600 361, 444 and 314).
int conv_patch_wide_rows_per_xcd(int row_tiles, int channel_blocks) {
  const int64_t rows = (row_tiles + (int64_t)7) / 8, rounds = ((int64_t)row_tiles * channel_blocks + 255) / 256;
  return channel_blocks >= 2 && row_tiles >= 64 && (rows * channel_blocks + 31) / 32 <= rounds ? (int)rows : 0;
}

size_t conv_patch_wide_lds(int bn, int patch_elems) {
  return (size_t)HEAD + std::max<size_t>((size_t)(2 * patch_elems + 3 * bn * PITCH) * 2, (size_t)epi_bytes(bn));
}

void launch_conv_patch_wide(hipStream_t st, int dt, const void* src, const void* wmat, const float* bias, const void* addend, void* out,
                            float* stat_partial, int bn, const PatchArgs& a) {
  if (dt == DT_BF16) launch_type<bf16_t>(st, src, wmat, bias, addend, out, stat_partial, bn, a);
  else launch_type<f16_t>(st, src, wmat, bias, addend, out, stat_partial, bn, a);
}

}  // namespace oseq
