// 1x1 layers of 64 input and 256 output channels whose output z is never in memory (16-bit storage; the last layer of a bottleneck
// block and the projection shortcut in the first stage of the networks, whose block outputs are the largest tensors there are).
// z has four times the bytes of the layer's input x, and the products that make it take less time than reading it: 64 multiply-adds
// a value against two bytes.  So whoever needs z multiplies x by the weights again (as the backward kernel of these layers does,
// k_conv_bwd1x1.hip) -- the forward kernels' products (k_conv_pointwise.hip) in their order and their rounding, hence the same bits:
//
//   again_stats_kernel   the forward pass of the layer as far as its BatchNorm: the channel sums of z, nothing else is written
//   again_apply_kernel   the BatchNorm's apply pass with the skip connection: a tensor, or that of a projection shortcut, from its x
//   again_sums_kernel    the sums that the BatchNorm's backward pass begins with, and those of the shortcut's in the same pass
//
// At 4.2 M pixels in bf16, us, with z in memory -> like this: a layer's forward pass 513 -> 187 (without a BatchNorm in front 490 ->
// 165), in a replay none; the apply pass with a projection shortcut 1220 -> 719; the sums of both 990 -> 718.  The training step of
// c64 n256 n256 at batch 4096 18.8 -> 15.6 ms, of which 0.6 is the backward kernel's not reading z.
//
// A block's 8 wavefronts own 32 channels each, the weights in registers; a tile of x goes through LDS (turned into activations on
// the way if a BatchNorm is folded in), its z is rounded into LDS, and from there on a thread has eight neighbouring channels of a
// pixel, as in the elementwise kernels, whose arithmetic this is.  With the weights as the first operand of the MFMA a lane holds
// four neighbouring channels of a pixel: z goes to LDS in stores of 8 bytes (16 of 2 bytes otherwise).
#include "bn_fold.h"
#include "dev_common.h"
#include "epilogue.h"
#include "kernels.h"

namespace oseq {

namespace {

typedef __attribute__((ext_vector_type(16))) float v16f;
typedef __attribute__((ext_vector_type(8))) __bf16 v8bf;
typedef __attribute__((ext_vector_type(8))) _Float16 v8h;

template <class T> struct Op;
template <> struct Op<bf16_t> {
  typedef v8bf V;
  __device__ static __forceinline__ v16f mma(V a, V b, v16f c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
};
template <> struct Op<f16_t> {
  typedef v8h V;
  __device__ static __forceinline__ v16f mma(V a, V b, v16f c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
};

constexpr int BC = 64, BK = 256, NT = 512;
constexpr int XP = BC + 8, ZP = BK + 8;  // LDS row pitches of x and z
constexpr int QK = BC / 16;              // MFMA steps

struct AgainArgs {
  int64_t M;  // pixels
  int MT;     // tiles
};

// the lane's weights, as the forward kernels': lane group hg owns the depths [32 s + 16 hg, + 16) of every 32
template <class T>
__device__ __forceinline__ void load_weights(const T* w, int channel, int hg, typename Op<T>::V (&f)[QK]) {
#pragma unroll
  for (int q = 0; q < QK; ++q)
    f[q] = *reinterpret_cast<const typename Op<T>::V*>(w + channel * BC + hg * 16 + (q >> 1) * 32 + (q & 1) * 8);
}

// z of a tile of BM pixels: the wavefront's 32 channels, rounded into zs
template <class T, int BM>
__device__ __forceinline__ void z_tile(const T* xs, const typename Op<T>::V (&f)[QK], T* zs, int wave, int hg, int l32) {
  typedef typename Op<T>::V V;
  constexpr int MI = BM / 32;
  v16f acc[MI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
#pragma unroll
  for (int q = 0; q < QK; ++q)
#pragma unroll
    for (int i = 0; i < MI; ++i)
      acc[i] = Op<T>::mma(f[q], *reinterpret_cast<const V*>(xs + (i * 32 + l32) * XP + hg * 16 + (q >> 1) * 32 + (q & 1) * 8), acc[i]);
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int e = 0; e < 16; e += 4) {
      const float v[4] = {acc[i][e], acc[i][e + 1], acc[i][e + 2], acc[i][e + 3]};
      *reinterpret_cast<Vec<T, 4>*>(&zs[(i * 32 + l32) * ZP + wave * 32 + 2 * e + 4 * hg]) = round_vec<T, 4>(v);
    }
}

// Channel sums of z, as conv1x1_ws_kernel makes them beside z: the same tiles of 128 pixels in the same order, so that the
// statistics do not depend on whether z is kept.  Bound by the products, the rounding and the dot-product instructions of the sums
// (0.54 GB counted in 165 us; matrix cores busy in 42 % of the cycles, vector units in 43).  Four tiles of x in flight per block: a tile's products are over in less than a
// load takes.  One barrier a tile.
constexpr int ST_BM = 128, ST_BLOCKS = 256, ST_AHEAD = 4;
template <class T, bool FOLD>
__global__ void __launch_bounds__(NT) again_stats_kernel(const T* __restrict__ x, const float* __restrict__ fold,
                                                         const T* __restrict__ w, float* __restrict__ stat_partial, AgainArgs a) {
  typedef typename Op<T>::V V;
  typedef typename Dot2<T>::V T2;
  constexpr int MI = ST_BM / 32;
  __shared__ __attribute__((aligned(16))) T xs[2][ST_BM * XP];
  __shared__ float red[4][BK];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hg = lane >> 5, l32 = lane & 31;
  const int cc = (tid & 7) * 8, r0 = tid >> 3, cj = wave * 32 + l32;
  V f[QK];
  load_weights<T>(w, cj, hg, f);
  float sc[8], sh[8];
  if (FOLD) {
    load_f32<float, 8>(fold + 2 * BC + cc, sc);
    load_f32<float, 8>(fold + 3 * BC + cc, sh);
  }
  Chunk ra[ST_AHEAD][2];
  auto gload = [&](auto P, int t) {  // rows past the last pixel (tiles past the last one) read row 0: nothing of them is added
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int64_t m = (int64_t)t * ST_BM + r0 + i * 64;
      ra[decltype(P)::value][i] = *reinterpret_cast<const Chunk*>(x + (m < a.M ? m : 0) * BC + cc);
    }
  };
  auto stage = [&](auto P, int buf) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const Chunk c = ra[decltype(P)::value][i];
      *reinterpret_cast<Chunk*>(&xs[buf][(r0 + i * 64) * XP + cc]) = FOLD ? bn_fold_chunk<T>(c, sc, sh) : c;
    }
  };
  float S1 = 0.f, S2 = 0.f;
  T2 one2;
  one2[0] = from_f32<T>(1.f); one2[1] = from_f32<T>(1.f);
  // the tile in buffer P & 1; the one after it is staged, the one ST_AHEAD on requested
  auto tile = [&](auto P, int t) {
    constexpr int p = decltype(P)::value;
    __syncthreads();
    stage(std::integral_constant<int, (p + 1) % ST_AHEAD>{}, (p + 1) & 1);
    gload(std::integral_constant<int, (p + 1) % ST_AHEAD>{}, t + (1 + ST_AHEAD) * ST_BLOCKS);
    v16f acc[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
#pragma unroll
    for (int q = 0; q < QK; ++q)
#pragma unroll
      for (int i = 0; i < MI; ++i)
        acc[i] = Op<T>::mma(*reinterpret_cast<const V*>(&xs[p & 1][(i * 32 + l32) * XP + hg * 16 + (q >> 1) * 32 + (q & 1) * 8]),
                            f[q], acc[i]);
    const int64_t m0 = (int64_t)t * ST_BM;
    auto add = [&](auto RAGGED) {
      float s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
          const int r = i * 32 + 8 * (e >> 2) + 4 * hg + (e & 3);  // and r + 1
          float v0 = acc[i][e], v1 = acc[i][e + 1];
          if (decltype(RAGGED)::value) {  // rows past the last pixel count as zero
            if (m0 + r >= a.M) v0 = 0.f;
            if (m0 + r + 1 >= a.M) v1 = 0.f;
          }
          const T2 p2 = from_f32x2<T>(v0, v1);
          s1 = Dot2<T>::run(p2, one2, s1);
          s2 = Dot2<T>::run(p2, p2, s2);
        }
      S1 += s1; S2 += s2;
    };
    if (m0 + ST_BM > a.M) add(std::true_type{});
    else add(std::false_type{});
  };
  int t = blockIdx.x;
  gload(std::integral_constant<int, 0>{}, t);
  gload(std::integral_constant<int, 1>{}, t + ST_BLOCKS);
  gload(std::integral_constant<int, 2>{}, t + 2 * ST_BLOCKS);
  gload(std::integral_constant<int, 3>{}, t + 3 * ST_BLOCKS);
  stage(std::integral_constant<int, 0>{}, 0);
  gload(std::integral_constant<int, 0>{}, t + 4 * ST_BLOCKS);
  while (t < a.MT) {  // (the same for the whole block)
    tile(std::integral_constant<int, 0>{}, t);
    if ((t += ST_BLOCKS) >= a.MT) break;
    tile(std::integral_constant<int, 1>{}, t);
    if ((t += ST_BLOCKS) >= a.MT) break;
    tile(std::integral_constant<int, 2>{}, t);
    if ((t += ST_BLOCKS) >= a.MT) break;
    tile(std::integral_constant<int, 3>{}, t);
    t += ST_BLOCKS;
  }
  red[hg][cj] = S1;  // the two lane groups of a channel in a fixed order
  red[2 + hg][cj] = S2;
  __syncthreads();
  if (tid < BK) {
    stat_partial[((int64_t)blockIdx.x * 2 + 0) * BK + tid] = red[0][tid] + red[1][tid];
    stat_partial[((int64_t)blockIdx.x * 2 + 1) * BK + tid] = red[2][tid] + red[3][tid];
  }
}

// What the two row kernels share: two blocks a CU, each walks tiles b, b + 512, ...; two barriers a tile.  PAIR: the layer and its
// block's projection shortcut, 32 pixels of both (the first half of the threads stages x, the other x2), else 64 pixels.
constexpr int ROW_BLOCKS = 512;
template <bool PAIR> constexpr int row_bm() { return PAIR ? 32 : 64; }
template <class T, bool PAIR> constexpr size_t row_lds() {
  return (size_t)(64 * XP + (PAIR ? 2 : 1) * row_bm<PAIR>() * ZP) * sizeof(T) + (4 * BC + 2 * BK) * sizeof(float);
}

template <class T, bool PAIR>
struct RowTiles {
  static constexpr int BM = row_bm<PAIR>(), PIECES = BM * (BK / 8) / NT, STEP = BM / PIECES;  // a thread's rows: row0 + STEP i
  const T* src;  // the thread's rows of x (or x2)
  T *xs, *zs;
  float *ftab, *means;  // scale and shift of the BatchNorm in front (PAIR: of both); means of the two behind (sums kernel, PAIR)
  int64_t M;
  int tid, wave, hg, l32, cc, xr, c8, row0;
  bool folds;
  typename Op<T>::V f[QK], f2[PAIR ? QK : 1];
  Chunk rx;

  __device__ __forceinline__ RowTiles(unsigned char* smem, const T* x, const T* x2, const float* fold, const float* fold2, const T* w,
                                      const T* w2, int64_t M_)
      : M(M_), tid(threadIdx.x) {
    xs = reinterpret_cast<T*>(smem);
    zs = xs + 64 * XP;
    ftab = reinterpret_cast<float*>(zs + (PAIR ? 2 : 1) * BM * ZP);
    means = ftab + 4 * BC;
    const int lane = tid & 63;
    wave = tid >> 6; hg = lane >> 5; l32 = lane & 31;
    cc = (tid & 7) * 8;
    xr = PAIR ? (tid >> 3) & 31 : tid >> 3;
    src = PAIR && tid >= NT / 2 ? x2 : x;
    folds = (PAIR && tid >= NT / 2 ? fold2 : fold) != nullptr;
    c8 = (tid & 31) * 8; row0 = tid >> 5;
    load_weights<T>(w, wave * 32 + l32, hg, f);
    if constexpr (PAIR) load_weights<T>(w2, wave * 32 + l32, hg, f2);
    const float* fp = PAIR && tid >= 2 * BC ? fold2 : fold;
    if (tid < (PAIR ? 4 : 2) * BC && fp) ftab[tid] = fp[2 * BC + (tid & (2 * BC - 1))];
  }
  // Offset of a row of tile t from the tile's first (the same for every thread, as a tile's base address is: a row's offset takes one
  // register); rows past the last pixel read the last one, tiles past the last one the first.
  __device__ __forceinline__ int64_t base(int t) const { return (int64_t)t * BM < M ? (int64_t)t * BM : 0; }
  __device__ __forceinline__ int rows(int t) const { return M - base(t) < BM ? (int)(M - base(t)) : BM; }
  __device__ __forceinline__ static int within(int row, int rows) { return row < rows ? row : rows - 1; }
  __device__ __forceinline__ void request(int t) {
    rx = *reinterpret_cast<const Chunk*>(src + base(t) * BC + (within(xr, rows(t)) * BC + cc));
  }
  __device__ __forceinline__ void stage() {
    Chunk c = rx;
    if (folds) {  // (the same for a whole wavefront)
      float sc[8], sh[8];
      const float* tab = ftab + (PAIR && tid >= NT / 2 ? 2 * BC : 0) + cc;
      load_f32<float, 8>(tab, sc);
      load_f32<float, 8>(tab + BC, sh);
      c = bn_fold_chunk<T>(c, sc, sh);
    }
    *reinterpret_cast<Chunk*>(&xs[(tid >> 3) * XP + cc]) = c;
  }
  __device__ __forceinline__ void products() {
    z_tile<T, BM>(xs, f, zs, wave, hg, l32);
    if constexpr (PAIR) z_tile<T, BM>(xs + 32 * XP, f2, zs + BM * ZP, wave, hg, l32);
  }
  __device__ __forceinline__ Vec<T, 8> z(int i) const { return *reinterpret_cast<const Vec<T, 8>*>(&zs[(row0 + i * STEP) * ZP + c8]); }
  __device__ __forceinline__ Vec<T, 8> z2(int i) const { return *reinterpret_cast<const Vec<T, 8>*>(&zs[(BM + row0 + i * STEP) * ZP + c8]); }
};

// out = ReLU(scale * z + shift + skip), the decisions as bits (bn_apply_kernel's values).  PROJ: skip is the BatchNorm of the
// projection shortcut, from its input x2, weights and statistics; else the tensor.  Counted at 4.2 M pixels with a projection
// shortcut: 1.07 GB read and 2.28 written, what it has to, in 719 us: 4.7 TB/s where the plain apply pass has 5.6.  LDS is busy in
// a third of the cycles (a quarter of them conflicts), the vector units in 60 %, the matrix cores in 17: with two barriers a tile
// they do not all run under the loads.
template <class T, bool PROJ>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 4)))
again_apply_kernel(const T* __restrict__ x, const float* __restrict__ fold, const T* __restrict__ w, const float* __restrict__ stats,
                   const T* __restrict__ skip, const T* __restrict__ x2, const float* __restrict__ fold2, const T* __restrict__ w2,
                   const float* __restrict__ stats2, T* __restrict__ out, uint8_t* __restrict__ mask, AgainArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  typedef RowTiles<T, PROJ> R;
  R r(smem_raw, x, x2, fold, fold2, w, w2, a.M);
  float scale[8], shift[8], sc2[8], sh2[8];
  load_f32<float, 8>(stats + 2 * BK + r.c8, scale);
  load_f32<float, 8>(stats + 3 * BK + r.c8, shift);
  if (PROJ) {
    load_f32<float, 8>(stats2 + 2 * BK + r.c8, sc2);
    load_f32<float, 8>(stats2 + 3 * BK + r.c8, sh2);
  }
  Chunk rs[PROJ ? 1 : R::PIECES];
  auto srequest = [&](int t, int i) {
    rs[i] = *reinterpret_cast<const Chunk*>(skip + r.base(t) * BK + (r.within(r.row0 + i * R::STEP, r.rows(t)) * BK + r.c8));
  };
  int t = blockIdx.x;
  r.request(t);
  if constexpr (!PROJ) {
#pragma unroll
    for (int i = 0; i < R::PIECES; ++i) srequest(t, i);
  }
  __syncthreads();  // the tables
  for (; t < a.MT; t += ROW_BLOCKS) {
    r.stage();
    r.request(t + ROW_BLOCKS);
    __syncthreads();
    r.products();
    __syncthreads();
#pragma unroll
    for (int i = 0; i < R::PIECES; ++i) {
      const int row = r.row0 + i * R::STEP;
      const Vec<T, 8> z = r.z(i);
      float vs[8], vo[8];
      if constexpr (PROJ) {
        const Vec<T, 8> z2 = r.z2(i);
#pragma unroll
        for (int k = 0; k < 8; ++k) vs[k] = bn_affine(to_f32(z2.v[k]), sc2[k], sh2[k]);
        const Vec<T, 8> sv = round_vec<T, 8>(vs);
#pragma unroll
        for (int k = 0; k < 8; ++k) vs[k] = to_f32(sv.v[k]);
      } else {
        const Vec<T, 8> sv = __builtin_bit_cast(Vec<T, 8>, rs[i]);
#pragma unroll
        for (int k = 0; k < 8; ++k) vs[k] = to_f32(sv.v[k]);
        srequest(t + ROW_BLOCKS, i);  // (ahead of the stores: loads and stores share one in-order counter)
      }
      unsigned bits = 0u;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        vo[k] = fmaxf(__fadd_rn(bn_affine(to_f32(z.v[k]), scale[k], shift[k]), vs[k]), 0.f);
        bits |= (vo[k] > 0.f ? 1u : 0u) << k;
      }
      if (row < r.rows(t)) {
        store_f32<T, 8>(out + r.base(t) * BK + (row * BK + r.c8), vo);
        if (mask) mask[r.base(t) * (BK / 8) + (row * (BK / 8) + (r.tid & 31))] = (uint8_t)bits;
      }
    }
  }
}

// The block's row of sums over its pixels of dy and dy * (z - mean) * rstd, dy = dA where the ReLU's bit is set; PAIR: also those of
// the projection shortcut's BatchNorm, which has the same dy.  (The factor rstd is a channel's: applied to the sum.)  Counted like the apply kernel, of both BatchNorms:
// 3.36 GB read in 718 us (4.7 TB/s), LDS busy in 46 % of the cycles, vector units in 70, matrix cores in 18.
template <class T, bool PAIR>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 4)))
again_sums_kernel(const T* __restrict__ da, const uint8_t* __restrict__ mask, const T* __restrict__ x, const float* __restrict__ fold,
                  const T* __restrict__ w, const float* __restrict__ stats, const T* __restrict__ x2, const float* __restrict__ fold2,
                  const T* __restrict__ w2, const float* __restrict__ stats2, float* __restrict__ partial, float* __restrict__ partial2, AgainArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  typedef RowTiles<T, PAIR> R;
  R r(smem_raw, x, x2, fold, fold2, w, w2, a.M);
  float mean[8], mean2[8], s0[8], s1[8], s2[8];
  if (PAIR) r.means[r.tid] = r.tid < BK ? stats[r.tid] : stats2[r.tid - BK];  // (in registers they would not fit)
  else load_f32<float, 8>(stats + r.c8, mean);
#pragma unroll
  for (int k = 0; k < 8; ++k) s0[k] = s1[k] = s2[k] = 0.f;
  Chunk ra[R::PIECES];
  unsigned rm[R::PIECES];
  auto drequest = [&](int t, int i) {
    const int row = r.within(r.row0 + i * R::STEP, r.rows(t));
    ra[i] = __builtin_nontemporal_load(reinterpret_cast<const Chunk*>(da + r.base(t) * BK + (row * BK + r.c8)));
    rm[i] = mask[r.base(t) * (BK / 8) + (row * (BK / 8) + (r.tid & 31))];
  };
  int t = blockIdx.x;
  r.request(t);
#pragma unroll
  for (int i = 0; i < R::PIECES; ++i) drequest(t, i);
  __syncthreads();  // the tables
  for (; t < a.MT; t += ROW_BLOCKS) {
    r.stage();
    r.request(t + ROW_BLOCKS);
    __syncthreads();
    r.products();
    __syncthreads();
    if (PAIR) {
      load_f32<float, 8>(r.means + r.c8, mean);
      load_f32<float, 8>(r.means + BK + r.c8, mean2);
    }
#pragma unroll
    for (int i = 0; i < R::PIECES; ++i) {
      const Vec<T, 8> z = r.z(i), va = __builtin_bit_cast(Vec<T, 8>, ra[i]);
      Vec<T, 8> z2{};
      if constexpr (PAIR) z2 = r.z2(i);
      const unsigned bits = r.row0 + i * R::STEP < r.rows(t) ? rm[i] : 0u;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float dy = (bits >> k) & 1u ? to_f32(va.v[k]) : 0.f;
        s0[k] += dy;
        s1[k] = __fmaf_rn(dy, to_f32(z.v[k]) - mean[k], s1[k]);
        if (PAIR) s2[k] = __fmaf_rn(dy, to_f32(z2.v[k]) - mean2[k], s2[k]);
      }
      drequest(t + ROW_BLOCKS, i);
    }
  }
  auto finish = [&](float (&s)[8], const float* st, float* p) {
    float rstd[8];
    load_f32<float, 8>(st + BK + r.c8, rstd);
#pragma unroll
    for (int k = 0; k < 8; ++k) s[k] *= rstd[k];
    epi_stat_combine_nt<NT, BK>(reinterpret_cast<float*>(smem_raw), r.tid, s0, s, p + (int64_t)blockIdx.x * 2 * BK,
                                p + ((int64_t)blockIdx.x * 2 + 1) * BK);
  };
  finish(s1, stats, partial);
  if constexpr (PAIR) finish(s2, stats2, partial2);
}

AgainArgs make_args(const ConvGeom& g, int bm) {
  AgainArgs a;
  a.M = (int64_t)g.N * g.P * g.Q;
  a.MT = ceil_div(a.M, bm);
  return a;
}

int row_blocks(const AgainArgs& a) { return a.MT < ROW_BLOCKS ? a.MT : ROW_BLOCKS; }

template <class T, bool PAIR>
void apply_t(hipStream_t st, const AgainSource& z, const void* skip, const AgainSource* proj, void* out, void* mask, const ConvGeom& g) {
  const AgainArgs a = make_args(g, row_bm<PAIR>());
  OSEQ_LAUNCH((again_apply_kernel<T, PAIR>), dim3(row_blocks(a)), dim3(NT), (row_lds<T, PAIR>()), st, (const T*)z.x, z.fold,
              (const T*)z.w, z.stats, (const T*)skip, PAIR ? (const T*)proj->x : nullptr, PAIR ? proj->fold : nullptr,
              PAIR ? (const T*)proj->w : nullptr, PAIR ? proj->stats : nullptr, (T*)out, (uint8_t*)mask, a);
}

template <class T, bool PAIR>
void sums_t(hipStream_t st, const void* da, const void* mask, const AgainSource& z, const AgainSource* proj, float* ws, float* ws2,
            const ConvGeom& g) {
  const AgainArgs a = make_args(g, row_bm<PAIR>());
  OSEQ_LAUNCH((again_sums_kernel<T, PAIR>), dim3(ROW_BLOCKS), dim3(NT), (row_lds<T, PAIR>()), st, (const T*)da,
              (const uint8_t*)mask, (const T*)z.x, z.fold, (const T*)z.w, z.stats, PAIR ? (const T*)proj->x : nullptr,
              PAIR ? proj->fold : nullptr, PAIR ? (const T*)proj->w : nullptr, PAIR ? proj->stats : nullptr, ws, ws2, a);
}

template <class T>
void stats_f(hipStream_t st, const void* x, const float* fold, const void* w, float* stat_partial, const AgainArgs& a) {
  if (fold) OSEQ_LAUNCH((again_stats_kernel<T, true>), dim3(ST_BLOCKS), dim3(NT), 0, st, (const T*)x, fold, (const T*)w, stat_partial, a);
  else OSEQ_LAUNCH((again_stats_kernel<T, false>), dim3(ST_BLOCKS), dim3(NT), 0, st, (const T*)x, fold, (const T*)w, stat_partial, a);
}

}  // namespace

// Where the weights-stationary forward kernel is taken and the backward kernel that reads no z: four tiles of 128 pixels a block, 130 945
// pixels.  Below it the forward kernel's sums are another partition's, and the bits of a step would depend on whether z is kept.  The step of
// c64 n256 n256 n256 in bf16 at 131 072 pixels 1333 us with z in memory, 1239 so.
bool conv_again_ok(int dt, const ConvGeom& g) {
  const int64_t M = (int64_t)g.N * g.P * g.Q;
  return conv_bwd1x1_ok(dt, g) && g.C == BC && g.K == BK && conv_pointwise_fwd_ok(dt, g) && conv_pointwise_stat_blocks(g) == ST_BLOCKS &&
         ceil_div(M, ST_BM) >= 4 * ST_BLOCKS;
}

int conv_again_sum_blocks() { return ROW_BLOCKS; }

void launch_conv_again_stats(hipStream_t st, int dt, const void* x, const float* fold, const void* w, float* stat_partial, const ConvGeom& g) {
  const AgainArgs a = make_args(g, ST_BM);
  if (dt == DT_BF16) stats_f<bf16_t>(st, x, fold, w, stat_partial, a);
  else stats_f<f16_t>(st, x, fold, w, stat_partial, a);
}

void launch_bn_apply_again(hipStream_t st, int dt, const AgainSource& z, const void* skip, const AgainSource* proj, void* out, void* mask,
                           const ConvGeom& g) {
  if (dt == DT_BF16 && proj) apply_t<bf16_t, true>(st, z, skip, proj, out, mask, g);
  else if (dt == DT_BF16) apply_t<bf16_t, false>(st, z, skip, proj, out, mask, g);
  else if (proj) apply_t<f16_t, true>(st, z, skip, proj, out, mask, g);
  else apply_t<f16_t, false>(st, z, skip, proj, out, mask, g);
}

void launch_bn_bwd_sums_again(hipStream_t st, int dt, const void* da, const void* mask, const AgainSource& z, const AgainSource* proj,
                              float* ws, float* ws2, const ConvGeom& g) {
  if (dt == DT_BF16 && proj) sums_t<bf16_t, true>(st, da, mask, z, proj, ws, ws2, g);
  else if (dt == DT_BF16) sums_t<bf16_t, false>(st, da, mask, z, proj, ws, ws2, g);
  else if (proj) sums_t<f16_t, true>(st, da, mask, z, proj, ws, ws2, g);
  else sums_t<f16_t, false>(st, da, mask, z, proj, ws, ws2, g);
}

}  // namespace oseq
