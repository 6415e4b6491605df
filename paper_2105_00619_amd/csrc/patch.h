// What the two kernels for 3x3 layers of stride 1 that stage a patch of the input share (k_conv_mfma.hip, k_conv_patch_wide.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fastdiv.h"

namespace oseq {

struct PatchArgs {
  int N, srcH, srcW, srcC;   // gathered tensor
  int dstH, dstW, Ng;        // pixel grid and channels of the result
  int pad, flip;             // border of the gather; flip: weight tap index 8 - t (data gradient)
  int TI, TR, TC, SR, SC, NPOS, TP;
  int tiles_r, tiles_c, NT;
  int relu;
  int chunks_per_split;      // channel chunks per blockIdx.z (all of them when the depth is not split)
  int row_pitch;             // bytes between staged patch rows in LDS (at least SC positions, padded against bank conflicts)
  int patch_elems;           // elements of one staged patch buffer (its rows times row_pitch, rounded up to 16 bytes)
  int xcd_group;             // 1: blocks are renumbered so that the row tiles of one weight slice run on one XCD;
                             // 2: so that the channel blocks and depth ranges of one row tile do (row_blocks: row tiles)
  int row_blocks;
  const uint8_t* amask;      // data gradient with an addend: ReLU bit mask the addend is multiplied by, or null
  int eval;                  // 1: the EVAL instantiation
  int bn_sums;               // 1: STAT 2
  int split32;               // fp32: 1: the Split32 instantiation
  const float* fold;         // FOLD (forward): src is the z of a BatchNorm + ReLU, this its [4][srcC] statistics tensor; the
                             // pieces of the patch become the activation (scale, shift, ReLU, one rounding) on their way
                             // to LDS; positions outside the image stay zero
};

struct PatchWideArgs : PatchArgs {  // k_conv_patch_wide.hip
  // positions of a patch's image and of its row, pixels of a tile's image and of its row, tiles
  FastDiv div_image, div_row, div_tile, div_tcol, div_tiles_r, div_tiles_c;
};

// Bytes between the staged rows of a patch, sc positions or more.  A wavefront reads 16 bytes at 32 consecutive pixels, and LDS
// takes lanes 0-3, 12-15 and 20-27 of them at once, then the others: sixteen whose numbers are all different modulo 16.
// With an odd number of 16-byte units per position, units of unit * pixel therefore fall on all 64 banks -- if going to the next row of the
// tile moves by as much, modulo 256 bytes, as tc pixels do, which is what the padding sees to.  (Tiles of 8 x 16 pixels of 144
// bytes without it: 62 % of the reads' cycles were conflicts; 16 x 8 of 112 bytes 43 %.)
inline int patch_rows_apart(int tc, int sc, int pos_bytes) {
  const int base = sc * pos_bytes;
  if (tc % 32 == 0) return base;  // (no wavefront's 32 pixels cross a row: padding would only cost a third block per CU its room)
  return base + ((tc * pos_bytes - base) % 256 + 256) % 256;
}

// block tiles of 256 pixels x bn (256 or 128) channels by one wavefront per SIMD (k_conv_patch_wide.hip)
constexpr int PATCH_WIDE_MAX_POS = 576;  // positions of its patch
size_t conv_patch_wide_lds(int bn, int patch_elems);
// row tiles whose channel blocks run on one XCD, 0: blocks in their own order
int conv_patch_wide_rows_per_xcd(int row_tiles, int channel_blocks);
void launch_conv_patch_wide(hipStream_t st, int dt, const void* src, const void* wmat, const float* bias, const void* addend, void* out,
                            float* stat_partial, int bn, const PatchArgs& a);

}  // namespace oseq
