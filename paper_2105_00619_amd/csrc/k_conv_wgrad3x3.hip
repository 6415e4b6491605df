// Weight gradient of 3x3, stride-1 convolutions on the matrix cores, all nine filter taps in one block.
//
//   dw[k][r][s][c] = sum over output pixels (n, p, q) of dz[n, p, q, k] * x[n, p + r - pad, q + s - pad, c]
//
// One block owns 64*MI output channels k, 64 input channels c, all nine taps, and a fixed range of pixel sub-tiles
// (blockIdx.z); the ranges are summed afterwards in order, so the result does not depend on scheduling.  A sub-tile is
// TI images x TR rows x TC columns of output pixels (at most CAP); its dz rows and the x positions it touches (the
// sub-tile plus a one-pixel halo, zero outside the image) are staged once in LDS, pixel-major as loaded, and serve
// all nine taps: a tap only shifts the x position that is paired with a dz pixel.  Compared with one tap per block
// this reads dz once instead of nine times and x about twice instead of nine times, which is what bounds the
// 16-bit kernel (the path from L2 to LDS), and it leaves nine MFMAs per operand fetch.
//
//   block = 8 wavefronts, two per SIMD (144 accumulator registers each), so that one's LDS reads and address arithmetic run
//   under the other's MFMAs: wavefront (wm, wn) owns k rows [wm*32*MI, +32*MI) and c columns [wn*32, +32) of every tap: MI x 9
//   accumulator tiles of 32x32.  128 output channels (the plan says where): 4 x 2 of them (256 -> 256 channels at 8 x 8, batch
//   4096, bf16: 481 us with 2 x 2 wavefronts of MI = 2, 304 us with 4 x 2, now 287; the one-tap-per-block kernel: 479 us).  64: 2 x 2 in
//   two groups that share a sub-tile's pixels, their sums added at the end (64 -> 64 channels over 4.2 M pixels, bf16, BatchNorm
//   folded in: 556 us with four wavefronts, 431 with eight, 411 with the next sub-tile staged at different times).  fp32: 2 x 2, one per SIMD and block, two blocks per CU.
//   MFMA 32x32x16, operands come from the transposing LDS read (ds_read_b64_tr_b16), whose per-lane row addresses make the
//   tap shift a plain change of address.  fp32: three bf16 planes per operand, six MFMAs (split32.h).
//   16-bit: two LDS stages; the next sub-tile's pieces are under way in registers during the MFMAs of the current one and go to the
//   other stage before or behind them (see the loop): one barrier per sub-tile.  fp32: one stage, sized for the layer's
//   sub-tile (79 KB on 8 x 8 pixels), so that two blocks share a CU and one loads and converts while the other computes; nothing
//   is parked, whose registers the accumulators need (spilled, 64 -> 64 channels at 1 048 576 pixels took 635 us).
#include <algorithm>
#include <type_traits>

#include "bn_fold.h"
#include "dev_common.h"
#include "kernels.h"
#include "split32.h"

namespace oseq {

static constexpr int g_w9_wide_min = 4;  // compile-time constant: fewest sub-tiles per block for 128-channel blocks

namespace {

typedef __attribute__((ext_vector_type(16))) float v16f;
typedef __attribute__((ext_vector_type(8))) __bf16 v8bf;
typedef __attribute__((ext_vector_type(8))) _Float16 v8h;

struct W9Args {
  int N, H, W, C, K, P, Q, pad;
  int TI, TR, TC, SR, SC, NPOS, TP;  // sub-tile: images, rows, columns; staged rows / columns; positions; pixels
  int tiles_r, tiles_c, NT;          // sub-tiles per image rows / columns; in total
  int tiles_per_split;
  int swap;                          // 1: the SWAP instantiation; TC is a multiple of 8
  int xcd_group, splits;  // xcd_group: the tiles of a pixel range share an XCD (see the kernel); splits: pixel ranges
  const float* fold;  // FOLD: x is the z of a BatchNorm + ReLU, this its [4][C] statistics tensor; the staged pieces of x
                      // become the activation (scale, shift, ReLU, one rounding); positions outside the image stay zero
};

template <class T> struct W9Cfg;
template <> struct W9Cfg<float> { static constexpr int CAP = 64, MAXPOS = 144; };
template <> struct W9Cfg<bf16_t> { static constexpr int CAP = 128, MAXPOS = 256; };
template <> struct W9Cfg<f16_t> { static constexpr int CAP = 128, MAXPOS = 256; };

// WGM wavefront rows of 32 * MI output channels each (2 wavefront columns of 32 input channels): 64 * WGM threads
// PG: groups of wavefronts that share a block's pixels (see the kernel)
constexpr int w9_groups(int bytes, int wgm) { return bytes == 2 && wgm == 2 ? 2 : 1; }
template <class T, int MI, int WGM, bool SWAP = false> struct W9Lds {
  static constexpr bool F32 = sizeof(T) == 4;
  static constexpr int CAP = W9Cfg<T>::CAP, MAXPOS = W9Cfg<T>::MAXPOS;
  static constexpr int BMK = 32 * MI * WGM;
  // elements per staged x position and dz pixel: 32 bytes of padding; SWAP: none, the 64-byte parts are exchanged instead (swz)
  static constexpr int PX = SWAP ? 64 : 80;
  static constexpr int PK = SWAP ? BMK : BMK + 16;
  static constexpr int PL = F32 ? 3 : 1;            // planes
  // elements of a plane of x (fp32: of the layer's positions, not of the most there can be), of dz; of a stage
  static constexpr int xs(int npos) { return (F32 ? npos : MAXPOS) * PX; }
  static constexpr int DS = CAP * PK;
  static constexpr int stage(int npos) { return PL * (xs(npos) + DS); }
  static constexpr size_t bytes(int npos) {
    const size_t loop = (size_t)(F32 ? 1 : 2) * stage(npos) * 2 + CAP * sizeof(int);
    const size_t sums = w9_groups(sizeof(T), WGM) == 2 ? (size_t)2 * WGM * MI * 9 * 16 * 64 * 4 : 0;  // a group's accumulators
    return loop > sums ? loop : sums;
  }
};

__device__ __forceinline__ v16f mfma16(v8bf a, v8bf b, v16f c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ v16f mfma16(v8h a, v8h b, v16f c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
template <class T> struct V8;
template <> struct V8<bf16_t> { typedef v8bf type; };
template <> struct V8<f16_t> { typedef v8h type; };
template <> struct V8<float> { typedef v8bf type; };

// WHOLE: every sub-tile is TI whole images (small images: 8 x 8, 4 x 4).  The (row, column) part of a chunk's address and
// of its bounds check is then the same for every sub-tile: a chunk keeps its pixel index within the sub-tile, the
// sub-tile adds its first image's, and one full-rate 24-bit multiply by the channel count gives the address (pixel
// indices and channel counts are below 2^24 where this kernel is chosen) -- the general path decodes image, row and
// column, checks each against the image and multiplies them back together with quarter-rate 32- and 64-bit multiplies,
// per chunk and sub-tile, in a kernel whose instruction stream is what bounds it.
//
// SWAP (blocks of 128 channels, TC a multiple of eight): the four pixels of a transposing read are neighbours in a row.  They fall on the
// same banks unless padded; here the 64-byte parts of a pixel are exchanged by its number instead (swz), which any four neighbours keep
// apart, and a staged row has a multiple of four positions, so that this order is that of the rows above and below.  Without conflicts and
// with one address per two reads 304 -> 287 us for 256 -> 256 channels over 262 144 pixels in bf16, 40.4 -> 37.3 for 128 -> 128 over
// 65 536.  (Going down a sub-tile's rows, a row of x at its three shifts for three rows of dz, 8 reads per nine MFMAs for 20: 350 us, spilled.
// In blocks of 64 channels nothing spills, but a tap at a time is as fast or faster on every map -- over 330 000 pixels, 64 -> 64, 92 us for 92 at
// 32 x 32, 95 for 106 at 24 x 24, 93 for 133 at 41 x 41 -- since what bounds them is the instructions around the staging.)
template <class T, int MI, int WGM, bool FOLD = false, bool WHOLE = false, bool SWAP = false>
__global__ void __launch_bounds__(128 * WGM * w9_groups(sizeof(T), WGM)) __attribute__((amdgpu_waves_per_eu(2, 2)))
conv_wgrad3x3_kernel(const T* __restrict__ x, const T* __restrict__ dz, float* __restrict__ out, W9Args a) {
  typedef W9Lds<T, MI, WGM, SWAP> L;
  constexpr bool F32 = L::F32;
  constexpr int PG = w9_groups(sizeof(T), WGM);
  constexpr int NTH = 128 * WGM * PG;                     // threads
  constexpr int CAP = L::CAP, MAXPOS = L::MAXPOS, BMK = L::BMK, PX = L::PX, PK = L::PK;
  constexpr int EV = 16 / (int)sizeof(T);
  constexpr int XCP = 64 / EV, DCP = BMK / EV;            // 16-byte chunks per x position / dz pixel
  constexpr int XSLOTS = (MAXPOS * XCP + NTH - 1) / NTH;  // chunks per thread and sub-tile
  constexpr int DSLOTS = CAP * DCP / NTH;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  typedef std::conditional_t<F32, bf16_t, T> E;  // staged element
  const int XS = L::xs(a.NPOS), STAGE = L::stage(a.NPOS);
  E* lds = reinterpret_cast<E*>(smem_raw);
  int* apos = reinterpret_cast<int*>(lds + (F32 ? 1 : 2) * STAGE);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int grp = PG == 2 ? __builtin_amdgcn_readfirstlane(wave / (2 * WGM)) : 0, wq = PG == 2 ? wave % (2 * WGM) : wave;
  const int wm = wq >> 1, wn = wq & 1, hg = lane >> 5, l32 = lane & 31;
  // Block coordinates: (output-channel tile, input-channel tile, pixel range).  The tiles of one pixel range all read
  // the same pixels of x and dz; workgroups go to the 8 XCDs round-robin by their linear index and every XCD has an L2
  // of its own, so with xcd_group the tiles of a range are renumbered onto one XCD, which then fetches those pixels
  // from HBM once (256 -> 256 channels at 262 144 pixels, bf16: 788 MB per launch without it for 268 MB of operands).
  // The grid's z extent is then the number of ranges rounded up to a multiple of 8.
  int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
  if (a.xcd_group) {
    const unsigned tiles = gridDim.x * gridDim.y;
    const unsigned lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const unsigned xcd = lin & 7u, slot = lin >> 3;
    const unsigned tile = slot % tiles;
    bz = (int)((slot / tiles) * 8u + xcd);
    bx = (int)(tile % gridDim.x); by = (int)(tile / gridDim.x);
    if (bz >= a.splits) return;
  }
  const int k0 = bx * BMK, c0 = by * 64;
  const int N = a.N, H = a.H, W = a.W, C = a.C, K = a.K, P = a.P, Q = a.Q, pad = a.pad;
  const int TI = a.TI, TR = a.TR, TC = a.TC, SC = a.SC, NPOS = a.NPOS, TP = a.TP;
  const int t0 = bz * a.tiles_per_split;
  const int t1 = t0 + a.tiles_per_split < a.NT ? t0 + a.tiles_per_split : a.NT;
  const int nst = t1 > t0 ? t1 - t0 : 0;

  // position of tap (0,0) in the staged x tile for every pixel of a sub-tile (the same for all sub-tiles)
  for (int m = tid; m < CAP; m += NTH) {
    int ap = 0;
    if (m < TP) {
      const int ti = m / (TR * TC), rr = m - ti * (TR * TC);
      const int tr = rr / TC, tc = rr - tr * TC;
      ap = (ti * a.SR + tr) * SC + tc;
    }
    apos[m] = ap;
  }

  // sub-tile-independent part of this thread's chunks: (image, row, column) within the sub-tile, packed
  int xinfo[XSLOTS], dinfo[DSLOTS];
#pragma unroll
  for (int sl = 0; sl < XSLOTS; ++sl) {
    const int idx = sl * NTH + tid, pos = idx / XCP;
    int info = -1;
    if (pos < NPOS) {
      const int ti = pos / (a.SR * SC), rr = pos - ti * (a.SR * SC);
      const int sy = rr / SC, sx = rr - sy * SC;
      info = (ti << 20) | (sy << 10) | sx;
      if (WHOLE) {  // image in the high bits, (ti * H + y) * W + x in the low ones; a halo position outside the image: none
        const int y = sy - pad, xx = sx - pad;
        info = y >= 0 && y < H && xx >= 0 && xx < W ? (ti << 20) | ((ti * H + y) * W + xx) : -1;
      }
    }
    xinfo[sl] = info;
  }
#pragma unroll
  for (int sl = 0; sl < DSLOTS; ++sl) {
    const int idx = sl * NTH + tid, m = idx / DCP;
    int info = -1;
    if (m < TP) {
      const int ti = m / (TR * TC), rr = m - ti * (TR * TC);
      const int tr = rr / TC, tc = rr - tr * TC;
      info = (ti << 20) | (tr << 10) | tc;
      if (WHOLE) info = (ti << 20) | ((ti * P + tr) * Q + tc);
    }
    dinfo[sl] = info;
  }

  // Loads are unconditional (clamped to the tensor start when outside) and zeroed when written to LDS.
  Chunk xr[XSLOTS], dr[DSLOTS];
  unsigned xok = 0u, dok = 0u;
  auto gload = [&](int tile) {
    if constexpr (WHOLE) {
      const int nb = tile * TI;
      const uint32_t xbase = (uint32_t)nb * (uint32_t)(H * W), dbase = (uint32_t)nb * (uint32_t)(P * Q);
      unsigned xm = 0u, dm = 0u;
#pragma unroll
      for (int sl = 0; sl < XSLOTS; ++sl) {
        const int info = xinfo[sl];
        const bool ok = info >= 0 && nb + (info >> 20) < N;
        const uint64_t off = ok ? (uint64_t)((xbase + (uint32_t)(info & 0xfffff)) & 0xffffffu) * (uint64_t)((uint32_t)C & 0xffffffu) : 0;
        const int v = (sl * NTH + tid) % XCP;
        xr[sl] = *reinterpret_cast<const Chunk*>(x + off + c0 + v * EV);
        xm |= ok ? (1u << sl) : 0u;
      }
#pragma unroll
      for (int sl = 0; sl < DSLOTS; ++sl) {
        const int info = dinfo[sl];
        const bool ok = info >= 0 && nb + (info >> 20) < N;
        const uint64_t off = ok ? (uint64_t)((dbase + (uint32_t)(info & 0xfffff)) & 0xffffffu) * (uint64_t)((uint32_t)K & 0xffffffu) : 0;
        const int v = (sl * NTH + tid) % DCP;
        dr[sl] = *reinterpret_cast<const Chunk*>(dz + off + k0 + v * EV);
        dm |= ok ? (1u << sl) : 0u;
      }
      xok = xm; dok = dm;
      return;
    }
    const int ci = tile % a.tiles_c, t2 = tile / a.tiles_c;
    const int ri = t2 % a.tiles_r, ii = t2 / a.tiles_r;
    const int nb = ii * TI, yb = ri * TR, xb = ci * TC;
    unsigned xm = 0u, dm = 0u;
    if constexpr (!FOLD) {
      // Pixels are counted from the sub-tile's first image (one uniform base per tensor): fewer than 2^24, so that every product
      // is a full-rate 24-bit one.  A position outside reads that image's first pixel.
      // us, 64-bit products -> this: 64 -> 64 channels at 65 536 pixels in bf16 47 -> 37, at 1 048 576 in fp32 833 -> 794;
      // with the BatchNorm folded in, whose registers leave the loads less room, 78 -> 86 at 262 144: that keeps the former.
      const T* xt = x + (int64_t)nb * H * W * C + c0;
      const T* dt = dz + (int64_t)nb * P * Q * K + k0;
      const uint32_t c24 = (uint32_t)C & 0xffffffu, k24 = (uint32_t)K & 0xffffffu;
#pragma unroll
      for (int sl = 0; sl < XSLOTS; ++sl) {
        const int info = xinfo[sl], ti = info >> 20;
        const int y = yb - pad + ((info >> 10) & 1023), xx = xb - pad + (info & 1023);
        const bool ok = info >= 0 && nb + ti < N && (unsigned)y < (unsigned)H && (unsigned)xx < (unsigned)W;
        const uint32_t pix = ok ? (uint32_t)(__mul24(__mul24(ti, H) + y, W) + xx) : 0u;
        const int v = (sl * NTH + tid) % XCP;
        xr[sl] = *reinterpret_cast<const Chunk*>(xt + (uint64_t)(pix & 0xffffffu) * (uint64_t)c24 + v * EV);
        xm |= ok ? (1u << sl) : 0u;
      }
#pragma unroll
      for (int sl = 0; sl < DSLOTS; ++sl) {
        const int info = dinfo[sl], ti = info >> 20;
        const int p = yb + ((info >> 10) & 1023), q = xb + (info & 1023);
        const bool ok = info >= 0 && nb + ti < N && p < P && q < Q;
        const uint32_t pix = ok ? (uint32_t)(__mul24(__mul24(ti, P) + p, Q) + q) : 0u;
        const int v = (sl * NTH + tid) % DCP;
        dr[sl] = *reinterpret_cast<const Chunk*>(dt + (uint64_t)(pix & 0xffffffu) * (uint64_t)k24 + v * EV);
        dm |= ok ? (1u << sl) : 0u;
      }
    } else {
#pragma unroll
      for (int sl = 0; sl < XSLOTS; ++sl) {
        const int info = xinfo[sl];
        const int n = nb + (info >> 20), y = yb - pad + ((info >> 10) & 1023), xx = xb - pad + (info & 1023);
        const bool ok = info >= 0 && n < N && y >= 0 && y < H && xx >= 0 && xx < W;
        const int v = (sl * NTH + tid) % XCP;
        const int64_t off = ok ? (((int64_t)n * H + y) * W + xx) * C : 0;
        xr[sl] = *reinterpret_cast<const Chunk*>(x + off + c0 + v * EV);
        xm |= ok ? (1u << sl) : 0u;
      }
#pragma unroll
      for (int sl = 0; sl < DSLOTS; ++sl) {
        const int info = dinfo[sl];
        const int n = nb + (info >> 20), p = yb + ((info >> 10) & 1023), q = xb + (info & 1023);
        const bool ok = info >= 0 && n < N && p < P && q < Q;
        const int v = (sl * NTH + tid) % DCP;
        const int64_t off = ok ? (((int64_t)n * P + p) * Q + q) * K : 0;
        dr[sl] = *reinterpret_cast<const Chunk*>(dz + off + k0 + v * EV);
        dm |= ok ? (1u << sl) : 0u;
      }
    }
    xok = xm; dok = dm;
  };
  // FOLD: a thread's pieces of x all cover the same EV channels, whose scale and shift it keeps in registers
  static_assert(NTH % XCP == 0, "a thread's pieces of x must share their channels");
  float fsc[EV], fsh[EV];
  if (FOLD) {
    load_f32<float, EV>(a.fold + 2 * C + c0 + (tid % XCP) * EV, fsc);
    load_f32<float, EV>(a.fold + 3 * C + c0 + (tid % XCP) * EV, fsh);
  }
  // SWAP: where channel c of a position (of x, of dz) lies within it
  auto swz = [](int pos, int c) { return c ^ (((pos >> 1) & 1) << 5); };
  auto swz_d = [](int m, int c) { return c ^ ((m & 3) << 5); };
  const int xput = SWAP ? tid / XCP * PX + swz(tid / XCP, tid % XCP * EV) : 0, dput = SWAP ? tid / DCP * PK + swz_d(tid / DCP, tid % DCP * EV) : 0;
  auto sstore = [&](int stage) {
    E* xs = lds + stage * STAGE;
    E* ds = xs + L::PL * XS;
    if constexpr (SWAP) {  // (positions 4 n apart keep their parts in the same order)
      static_assert(BMK == 128, "the order of dz is that of four parts");
      static_assert(NTH / XCP % 4 == 0 && NTH / DCP % 4 == 0 && MAXPOS * XCP % NTH == 0, "a slot's pieces are whole positions");
#pragma unroll
      for (int sl = 0; sl < XSLOTS; ++sl) {
        if (FOLD) xr[sl] = bn_fold_chunk<T>(xr[sl], fsc, fsh);
        *reinterpret_cast<Chunk*>(&xs[xput + sl * (NTH / XCP) * PX]) = ((xok >> sl) & 1u) ? xr[sl] : zero_chunk();
      }
#pragma unroll
      for (int sl = 0; sl < DSLOTS; ++sl)
        *reinterpret_cast<Chunk*>(&ds[dput + sl * (NTH / DCP) * PK]) = ((dok >> sl) & 1u) ? dr[sl] : zero_chunk();
      return;
    }
    if (FOLD) {
#pragma unroll
      for (int sl = 0; sl < XSLOTS; ++sl) xr[sl] = bn_fold_chunk<T>(xr[sl], fsc, fsh);
    }
#pragma unroll
    for (int sl = 0; sl < XSLOTS; ++sl) {
      const int idx = sl * NTH + tid, pos = idx / XCP, v = idx - pos * XCP;
      if (pos < MAXPOS) *reinterpret_cast<Chunk*>(&xs[pos * PX + v * EV]) = ((xok >> sl) & 1u) ? xr[sl] : zero_chunk();
    }
#pragma unroll
    for (int sl = 0; sl < DSLOTS; ++sl) {
      const int idx = sl * NTH + tid, m = idx / DCP, v = idx - m * DCP;
      *reinterpret_cast<Chunk*>(&ds[m * PK + v * EV]) = ((dok >> sl) & 1u) ? dr[sl] : zero_chunk();
    }
  };

  // fp32: a sub-tile from memory to its planes in LDS, half of the pieces of x at a time; addresses as in gload; neg: dz negated
  auto stage32 = [&](int tile, bool neg) {
    E* xs = lds;
    E* ds = lds + L::PL * XS;
    const int ci = tile % a.tiles_c, t2 = tile / a.tiles_c;
    const int ri = t2 % a.tiles_r, nb = t2 / a.tiles_r * TI;
    const int yb = ri * TR - pad, xb = ci * TC - pad;
    const T* xt = x + (int64_t)nb * H * W * C + c0;
    const T* dt = dz + (int64_t)nb * P * Q * K + k0;
    const uint32_t sign = neg ? 0x80000000u : 0u;
    auto put = [&](E* at, int plane, const Chunk& c) {
      u32x2_t q[3];
      split32(c, q);
#pragma unroll
      for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x2_t*>(at + k * plane) = q[k];
    };
    constexpr int HALF = (XSLOTS + 1) / 2;
    auto load_x = [&](auto FIRST) {
#pragma unroll
      for (int i = 0; i < HALF; ++i) {
        const int sl = decltype(FIRST)::value + i;
        if (sl >= XSLOTS || sl * NTH >= NPOS * XCP) break;
        const int info = xinfo[sl], ti = info >> 20;
        const int y = yb + ((info >> 10) & 1023), xx = xb + (info & 1023);
        const bool ok = info >= 0 && nb + ti < N && (unsigned)y < (unsigned)H && (unsigned)xx < (unsigned)W;
        const uint32_t pix = ok ? (uint32_t)(__mul24(__mul24(ti, H) + y, W) + xx) : 0u;
        xr[i] = *reinterpret_cast<const Chunk*>(xt + (uint64_t)(pix & 0xffffffu) * (uint64_t)((uint32_t)C & 0xffffffu) + (sl * NTH + tid) % XCP * EV);
        xok = i == 0 ? (ok ? 1u : 0u) : xok | (ok ? 1u << i : 0u);
      }
    };
    auto put_x = [&](auto FIRST) {
#pragma unroll
      for (int i = 0; i < HALF; ++i) {
        const int sl = decltype(FIRST)::value + i;
        if (sl >= XSLOTS || sl * NTH >= NPOS * XCP) break;
        const int idx = sl * NTH + tid, pos = idx / XCP;
        if (pos < NPOS) put(&xs[pos * PX + idx % XCP * EV], XS, (xok >> i) & 1u ? xr[i] : zero_chunk());
      }
    };
    load_x(std::integral_constant<int, 0>{});
#pragma unroll
    for (int sl = 0; sl < DSLOTS; ++sl) {
      const int info = dinfo[sl], ti = info >> 20;
      const int p = ri * TR + ((info >> 10) & 1023), q = ci * TC + (info & 1023);
      const bool ok = info >= 0 && nb + ti < N && p < P && q < Q;
      const uint32_t pix = ok ? (uint32_t)(__mul24(__mul24(ti, P) + p, Q) + q) : 0u;
      dr[sl] = *reinterpret_cast<const Chunk*>(dt + (uint64_t)(pix & 0xffffffu) * (uint64_t)((uint32_t)K & 0xffffffu) + (sl * NTH + tid) % DCP * EV);
      dok = sl == 0 ? (ok ? 1u : 0u) : dok | (ok ? 1u << sl : 0u);
    }
    put_x(std::integral_constant<int, 0>{});
    load_x(std::integral_constant<int, HALF>{});
#pragma unroll
    for (int sl = 0; sl < DSLOTS; ++sl) {
      const int idx = sl * NTH + tid;
      put(&ds[idx / DCP * PK + idx % DCP * EV], L::DS, signed_chunk(dr[sl], (dok >> sl) & 1u, sign));
    }
    put_x(std::integral_constant<int, HALF>{});
  };

  v16f acc[MI][9];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][t][e] = 0.f;

  int toff[9];  // element offset of tap t relative to tap (0,0) in the staged x tile
#pragma unroll
  for (int t = 0; t < 9; ++t) toff[t] = ((t / 3) * SC + (t % 3)) * PX;

  auto compute = [&](int stage) {
    const E* xs = lds + stage * STAGE;
    const E* ds = xs + L::PL * XS;
    const int r16 = l32 & 15;
    const int colsel = (l32 & 16) + 4 * (r16 & 3);
    const E* tx = xs + wn * 32 + colsel;
    const E* td = ds + wm * 32 * MI + colsel;
    const int nss = (TP + 15) >> 4;
    if constexpr (F32) {
#pragma unroll 1
      for (int ss = 0; ss < nss; ++ss) {
        const int ma = ss * 16 + hg * 8 + (r16 >> 2), mb = ma + 4;
        const E* xa = tx + apos[ma] * PX;
        const E* xb = tx + apos[mb] * PX;
        v8bf fa[MI][3];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int q = 0; q < 3; ++q) fa[i][q] = lds_tr_read8<typename V8<T>::type>(td + q * L::DS + ma * PK + i * 32, td + q * L::DS + mb * PK + i * 32);
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
          v8bf fb[3];
#pragma unroll
          for (int q = 0; q < 3; ++q) fb[q] = lds_tr_read8<typename V8<T>::type>(xa + q * XS + toff[tap], xb + q * XS + toff[tap]);
          constexpr int QA[6] = {2, 0, 1, 1, 0, 0}, QB[6] = {0, 2, 1, 0, 1, 0};  // the smallest first
#pragma unroll
          for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int i = 0; i < MI; ++i) acc[i][tap] = mfma16(fa[i][QA[q]], fb[QB[q]], acc[i][tap]);
        }
      }
    } else if constexpr (SWAP) {
#pragma unroll 2
      for (int ss = 0; ss < nss; ++ss) {
        const int m = ss * 16 + hg * 8 + (r16 >> 2), pos = apos[m];
        const typename V8<T>::type f = lds_tr_read8<typename V8<T>::type>(ds + m * PK + swz_d(m, wm * 32 + colsel), ds + m * PK + swz_d(m, wm * 32 + colsel) + 4 * PK);
        const T* xq[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) xq[s] = xs + (pos + s) * PX + swz(pos + s, wn * 32 + colsel);
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
          const T* q = xq[tap % 3] + tap / 3 * SC * PX;
          acc[0][tap] = mfma16(f, lds_tr_read8<typename V8<T>::type>(q, q + 4 * PX), acc[0][tap]);
        }
      }
    } else {
#pragma unroll 2
      for (int ss = grp; ss < nss; ss += PG) {
        const int ma = ss * 16 + hg * 8 + (r16 >> 2), mb = ma + 4;
        const T* xa = tx + apos[ma] * PX;
        const T* xb = tx + apos[mb] * PX;
        typename V8<T>::type fa[MI];
#pragma unroll
        for (int i = 0; i < MI; ++i) fa[i] = lds_tr_read8<typename V8<T>::type>(td + ma * PK + i * 32, td + mb * PK + i * 32);
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
          const typename V8<T>::type fb = lds_tr_read8<typename V8<T>::type>(xa + toff[tap], xb + toff[tap]);
#pragma unroll
          for (int i = 0; i < MI; ++i) acc[i][tap] = mfma16(fa[i], fb, acc[i][tap]);
        }
      }
    }
  };

  if constexpr (F32) {
    // (split32.h: half of the sum with dz negated)
    bool neg = (bz & 1) != 0;
    auto negate = [&]() {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[i][t] = -acc[i][t];
    };
    const int flip = wgrad_flip(nst);
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
      const int g1 = half ? nst : flip;
#pragma unroll 1
      for (int g = half ? flip : 0; g < g1; ++g) {
        if (g > 0) __syncthreads();
        stage32(t0 + g, neg);
        __syncthreads();
        compute(0);
      }
      if (half == 0 || neg) { neg = !neg; negate(); }
    }
  } else {
    if (nst > 0) { gload(t0); sstore(0); }
    if constexpr (PG == 2) {
      // While sub-tile g is multiplied, g + 1 goes from registers to the other stage and g + 2 is requested: by one group of
      // wavefronts before its MFMAs, by the other behind them, so that on every SIMD the conversions and addresses of one run
      // under the MFMAs of the other (64 -> 64 channels over 4.2 M pixels: 431 us with both behind, 411 so).
      auto stage_next = [&](int g) {
        sstore((g + 1) & 1);
        if (g + 2 < nst) gload(t0 + g + 2);
      };
      if (nst > 1) gload(t0 + 1);
      __syncthreads();
      for (int g = 0; g + 1 < nst; ++g) {
        if (grp == 0) stage_next(g);
        compute(g & 1);
        if (grp != 0) stage_next(g);
        __syncthreads();
      }
    } else {  // (128 channels: no gain from that)
      __syncthreads();
      for (int g = 0; g + 1 < nst; ++g) {
        gload(t0 + g + 1);
        compute(g & 1);
        sstore((g + 1) & 1);
        __syncthreads();
      }
    }
    if (nst > 0) compute((nst - 1) & 1);
  }

  if constexpr (F32) {
    static_assert(!F32 || MI == 1, "one output-channel tile per wavefront");
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) sum = __fmaf_rn(acc[0][t][e], 0.f, sum);
    if (__syncthreads_or(!(sum == 0.f))) {  // the tile again as chains of fp32 multiply-adds (split32.h)
      float* fx = reinterpret_cast<float*>(smem_raw);  // [NPOS][64]
      float* fd = fx + NPOS * 64;                      // [TP][BMK]
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[0][t][e] = 0.f;
#pragma unroll 1
      for (int tile = t0; tile < t1; ++tile) {
        const int ci = tile % a.tiles_c, t2 = tile / a.tiles_c;
        const int ri = t2 % a.tiles_r, nb = t2 / a.tiles_r * TI;
        for (int idx = tid; idx < NPOS * XCP; idx += NTH) {
          const int pos = idx / XCP, ti = pos / (a.SR * SC), rr = pos - ti * (a.SR * SC);
          const int n = nb + ti, y = ri * TR - pad + rr / SC, xx = ci * TC - pad + rr % SC;
          const bool ok = n < N && y >= 0 && y < H && xx >= 0 && xx < W;
          const int64_t off = ok ? (((int64_t)n * H + y) * W + xx) * C : 0;
          *reinterpret_cast<Chunk*>(fx + idx * EV) = *reinterpret_cast<const Chunk*>(x + off + c0 + idx % XCP * EV);
        }
        for (int idx = tid; idx < TP * DCP; idx += NTH) {
          const int m = idx / DCP, ti = m / (TR * TC), rr = m - ti * (TR * TC);
          const int n = nb + ti, p = ri * TR + rr / TC, q = ci * TC + rr % TC;
          const bool ok = n < N && p < P && q < Q;
          const int64_t off = ok ? (((int64_t)n * P + p) * Q + q) * K : 0;
          *reinterpret_cast<Chunk*>(fd + idx * EV) = *reinterpret_cast<const Chunk*>(dz + off + k0 + idx % DCP * EV);
        }
        __syncthreads();
#pragma unroll 1
        for (int m = 0; m < TP; ++m) {  // (pixels and taps that do not count are left out: zero times infinity is none)
          const int ti = m / (TR * TC), rr = m - ti * (TR * TC), tr = rr / TC, tc = rr - tr * TC;
          const int p = ri * TR + tr, q = ci * TC + tc;
          if (nb + ti >= N || p >= P || q >= Q) continue;
          const float* xv = fx + ((ti * a.SR + tr) * SC + tc) * 64 + wn * 32 + l32;
          float d[16];
#pragma unroll
          for (int e = 0; e < 16; ++e) d[e] = fd[m * BMK + wm * 32 + 8 * (e >> 2) + 4 * hg + (e & 3)];
#pragma unroll
          for (int tap = 0; tap < 9; ++tap) {
            const int y = p + tap / 3 - pad, xx = q + tap % 3 - pad;
            if (y < 0 || y >= H || xx < 0 || xx >= W) continue;
            const float v = xv[(tap / 3 * SC + tap % 3) * 64];
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[0][tap][e] = __fmaf_rn(d[e], v, acc[0][tap][e]);
          }
        }
        __syncthreads();
      }
    }
  }

  const int64_t outputs = (int64_t)K * 9 * C;
  float* dst = out + (int64_t)bz * outputs + (int64_t)(k0 + wm * 32 * MI + 4 * hg) * 9 * C + c0 + wn * 32 + l32;
  float* red = reinterpret_cast<float*>(smem_raw) + (wq * MI * 9 * 16) * 64 + lane;
  auto each = [&](auto FIRST, auto LAST, auto body) {  // taps [FIRST, LAST)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int tap = decltype(FIRST)::value; tap < decltype(LAST)::value; ++tap) {
#pragma unroll
        for (int e = 0; e < 16; ++e) body(i, tap, e);
        __builtin_amdgcn_sched_barrier(0);  // (no more than a tap's values at once beside the accumulators)
      }
  };
  auto put = [&](int i, int tap, int e) { red[((i * 9 + tap) * 16 + e) * 64] = acc[i][tap][e]; };
  auto store = [&](int i, int tap, int e) {
    const float v = PG == 2 ? acc[i][tap][e] + red[((i * 9 + tap) * 16 + e) * 64] : acc[i][tap][e];
    dst[((int64_t)(i * 32 + 8 * (e >> 2) + (e & 3)) * 9 + tap) * C] = v;
  };
  using std::integral_constant;
  typedef integral_constant<int, 0> I0; typedef integral_constant<int, 5> I5; typedef integral_constant<int, 9> I9;
  if constexpr (PG == 2) {  // the groups' sums added: the first group stores taps 0 to 4, the second the others
    __syncthreads();
    if (grp == 0) each(I5{}, I9{}, put); else each(I0{}, I5{}, put);
    __syncthreads();
    if (grp == 0) each(I0{}, I5{}, store); else each(I5{}, I9{}, store);
  } else {
    each(I0{}, I9{}, store);
  }
}

// sub-tile geometry for a (P x Q) output grid: up to `cap` pixels and `maxpos` staged positions
bool w9_geometry_of(int N, int P, int Q, int tc, int cap, int maxpos, int halo, W9Args& a) {
  int tr = cap / tc; if (tr > P) tr = P; if (tr < 1) tr = 1;
  int ti = (tr == P && tc == Q) ? cap / (P * Q) : 1;
  if (ti > N) ti = N; if (ti < 1) ti = 1;
  while (ti > 1 && ti * (tr + 2) * (tc + halo) > maxpos) ti /= 2;
  while (tr > 1 && ti * (tr + 2) * (tc + halo) > maxpos) --tr;
  while (tc > 1 && ti * (tr + 2) * (tc + halo) > maxpos) tc /= 2;
  if (ti * (tr + 2) * (tc + halo) > maxpos) return false;
  a.TI = ti; a.TR = tr; a.TC = tc; a.SR = tr + 2; a.SC = tc + halo;
  a.NPOS = ti * a.SR * a.SC; a.TP = ti * tr * tc;
  a.tiles_r = (P + tr - 1) / tr; a.tiles_c = (Q + tc - 1) / tc;
  a.NT = ((N + ti - 1) / ti) * a.tiles_r * a.tiles_c;
  return true;
}
// The widest sub-tile; where three rows of the map leave it less than three quarters of the pixels (512 columns: 32 of 64 with 102
// staged positions), the narrower one that covers the map with the fewest sub-tiles, then staged positions.  (bf16, three layers of
// 128 channels at 8 x 112 x 112 232 -> 158 us without -> with, at 16 x 64 x 64 151 -> 137.)
// halo: staged columns beyond those of the pixels: 2, SWAP 4
bool w9_geometry(int N, int P, int Q, int cap, int maxpos, W9Args& a, int halo = 2) {
  bool ok = w9_geometry_of(N, P, Q, Q < cap ? Q : cap, cap, maxpos, halo, a);
  if (ok && a.TP * 4 >= cap * 3) return ok;
  for (int tc = 64; tc >= 8; tc /= 2) {
    W9Args b = a;
    if (tc >= Q || !w9_geometry_of(N, P, Q, tc, cap, maxpos, halo, b)) continue;
    if (!ok || b.NT < a.NT || (b.NT == a.NT && b.NPOS < a.NPOS)) { a = b; ok = true; }
  }
  return ok;
}

// everything decided from the layer shape: block shape, sub-tile geometry, number of pixel ranges
struct W9Plan { W9Args a; int mi, splits; };
// room: bytes of partial sums that do not enlarge the activation arena; ranges (when the kernel is launched): the number of
// ranges that the layer was given, 0: not yet
bool w9_plan(int dt, const ConvGeom& g, int64_t room, int ranges, W9Plan& pl) {
  if (g.R != 3 || g.S != 3 || g.stride != 1 || g.C % 64 != 0 || g.K % 64 != 0) return false;
  if (g.C >= 1 << 24 || g.K >= 1 << 24) return false;  // 24-bit products
  if (g.H >= 1024 || g.W >= 1024) return false;  // packed (image within the sub-tile, row, column) fields
  const int cap = dt == DT_F32 ? W9Cfg<float>::CAP : W9Cfg<bf16_t>::CAP;
  const int maxpos = dt == DT_F32 ? W9Cfg<float>::MAXPOS : W9Cfg<bf16_t>::MAXPOS;
  W9Args a{};
  if (!w9_geometry(g.N, g.P, g.Q, cap, maxpos, a)) return false;
  if (a.TP * 2 < cap) return false;  // short sub-tiles: too little work between barriers
  a.N = g.N; a.H = g.H; a.W = g.W; a.C = g.C; a.K = g.K; a.P = g.P; a.Q = g.Q; a.pad = g.pad;
  // 128 output channels per block when possible (fewer operand fetches per MFMA, two wavefronts per SIMD), unless the blocks
  // would then get fewer than g_w9_wide_min sub-tiles each: a block's accumulators (9 taps x 64*MI x 64 floats) are
  // written out once per pixel range and read again by the reduction, and with few sub-tiles per range that traffic
  // outweighs the operand reuse (128->128 at 16x16, batch 256, bf16: 49.6 us with 64-channel blocks, 48.1 with
  // 128-channel blocks of four sub-tiles each).  At that size the 75 MB of partial sums written and read back are most
  // of the time: 19 GFLOP would take 8 us at the matrix cores' peak.
  // fp32: 64 output channels per block, two blocks per CU where there is room for their partial sums (64 -> 64 channels at 1 048 576
  // pixels 367 us, 472 with one; on the fp32 MFMA 800), a quarter of it left for what the placement of the tensors loses.
  const bool f32 = dt == DT_F32;
  for (int mi = f32 ? 2 : g.K % 128 == 0 ? 2 : 1; mi >= 1; --mi) {
    const int target = f32 && mi == 2 ? 512 : 256;  // blocks
    const int bk = f32 ? 64 : 64 * mi;
    const int64_t tiles = (int64_t)(g.K / bk) * (g.C / 64);
    int64_t s = tiles >= target ? 1 : (target + tiles / 2) / tiles;
    if (s > a.NT) s = a.NT;
    if (s > target) s = target;
    if (s < 1) s = 1;
    a.tiles_per_split = (int)((a.NT + s - 1) / s);
    s = (a.NT + a.tiles_per_split - 1) / a.tiles_per_split;  // no empty ranges
    if (mi == 2 && a.tiles_per_split < g_w9_wide_min) continue;
    if (mi == 2 && f32 && (ranges ? s != ranges : s * g.K * 9 * g.C * 4 > room / 4 * 3)) continue;
    if (tiles * s < 128) return false;  // too few blocks for the chip: one tap per block does better
    // 16 bits, blocks of 128 channels: SWAP where the columns need no padding (and sub-tiles hold no fewer pixels for their staged rows).
    // Its own sub-tiles, in no more ranges (whose sums take room in the activation arena).
    W9Args r = a;
    if (!f32 && mi == 2 && g.Q % 8 == 0 && w9_geometry(g.N, g.P, g.Q, cap, maxpos, r, 4) && r.TC % 8 == 0 &&
        (int64_t)r.NT * ((r.TI * (r.TC / 8) + 1) / 2) * r.TR * 4 <= (int64_t)a.NT * ((a.TP + 15) / 16) * 5) {
      a = r;
      a.swap = 1;
      a.tiles_per_split = (int)((a.NT + s - 1) / s);
      s = (a.NT + a.tiles_per_split - 1) / a.tiles_per_split;
    }
    pl.a = a; pl.mi = f32 ? 1 : mi; pl.splits = (int)s;
    return true;
  }
  return false;
}

template <class T, int MI, int WGM, bool FOLD, bool WHOLE, bool SWAP>
void launch_w9_one(hipStream_t st, const void* x, const void* dz, float* dst, dim3 grid, const W9Args& a) {
  typedef W9Lds<T, MI, WGM, SWAP> L;
  static bool attr_done = false;
  if (!attr_done) {
    (void)hipFuncSetAttribute((const void*)conv_wgrad3x3_kernel<T, MI, WGM, FOLD, WHOLE, SWAP>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)L::bytes(W9Cfg<T>::MAXPOS));
    attr_done = true;
  }
  OSEQ_LAUNCH((conv_wgrad3x3_kernel<T, MI, WGM, FOLD, WHOLE, SWAP>), grid, dim3(128 * WGM * w9_groups(sizeof(T), WGM)), L::bytes(a.NPOS), st,
              (const T*)x, (const T*)dz, dst, a);
}
template <class T, int MI, int WGM, bool FOLD>
void launch_w9(hipStream_t st, const void* x, const void* dz, float* dst, const W9Plan& pl) {
  W9Args a = pl.a;
  const int tiles = (a.K / (32 * MI * WGM)) * (a.C / 64);
  a.splits = pl.splits;
  a.xcd_group = tiles > 1 && pl.splits >= 8;  // (from the shape only)
  dim3 grid(a.K / (32 * MI * WGM), a.C / 64, a.xcd_group ? (pl.splits + 7) / 8 * 8 : pl.splits);
  // sub-tiles of whole images, every index that is multiplied below 2^24, the pixel index within a sub-tile below 2^20
  const bool whole = a.tiles_r == 1 && a.tiles_c == 1 && a.TR == a.P && a.TC == a.Q && a.H == a.P && a.W == a.Q &&
                     (int64_t)a.N * a.H * a.W + (int64_t)a.TI * a.H * a.W < (1 << 24) && a.C < (1 << 24) && a.K < (1 << 24) &&
                     a.TI < 256 && (int64_t)a.TI * a.H * a.W < (1 << 20);
  if constexpr (sizeof(T) == 2 && WGM == 4) {
    if (a.swap) {
      if (whole) launch_w9_one<T, MI, WGM, FOLD, true, true>(st, x, dz, dst, grid, a);
      else launch_w9_one<T, MI, WGM, FOLD, false, true>(st, x, dz, dst, grid, a);
      return;
    }
  }
  if constexpr (sizeof(T) == 2) {
    if (whole) {
      launch_w9_one<T, MI, WGM, FOLD, true, false>(st, x, dz, dst, grid, a);
      return;
    }
  }
  launch_w9_one<T, MI, WGM, FOLD, false, false>(st, x, dz, dst, grid, a);
}

template <class T>
void launch_w9_16(hipStream_t st, const void* x, const void* dz, float* dst, const W9Plan& pl) {
  // 128 output channels per block: four wavefront rows of 32 channels (eight wavefronts, two per SIMD)
  if (pl.a.fold) {
    if (pl.mi == 2) launch_w9<T, 1, 4, true>(st, x, dz, dst, pl); else launch_w9<T, 1, 2, true>(st, x, dz, dst, pl);
  } else {
    if (pl.mi == 2) launch_w9<T, 1, 4, false>(st, x, dz, dst, pl); else launch_w9<T, 1, 2, false>(st, x, dz, dst, pl);
  }
}

}  // namespace

static constexpr int g_wgrad3x3 = 1;  // compile-time switch

bool conv_wgrad3x3_ok(int dt, const ConvGeom& g) {
  W9Plan pl;
  return g_wgrad3x3 && w9_plan(dt, g, 0, 0, pl);
}

bool conv_wgrad3x3_swaps(int dt, const ConvGeom& g) {
  W9Plan pl;
  return w9_plan(dt, g, 0, 0, pl) && pl.a.swap;
}

int conv_wgrad3x3_splits(int dt, const ConvGeom& g, int64_t room) {
  W9Plan pl;
  return w9_plan(dt, g, room, 0, pl) ? pl.splits : 1;
}

// dst: [splits][K][9][C] floats (dw itself when splits == 1); fold: see W9Args (16-bit modes only)
void launch_conv_wgrad3x3(hipStream_t st, int dt, const void* x, const void* dz, float* dst, int splits, const ConvGeom& g,
                          const float* fold) {
  W9Plan pl;
  if (!w9_plan(dt, g, 0, splits, pl)) return;
  pl.a.fold = dt == DT_F32 ? nullptr : fold;
  if (dt == DT_F32) launch_w9<float, 1, 2, false>(st, x, dz, dst, pl);
  else if (dt == DT_BF16) launch_w9_16<bf16_t>(st, x, dz, dst, pl);
  else launch_w9_16<f16_t>(st, x, dz, dst, pl);
}

}  // namespace oseq
