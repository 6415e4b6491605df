// HBM-bound kernels over NHWC tensors viewed as [rows = N*H*W][C]:
//   input cast, per-channel reductions (BatchNorm statistics, BatchNorm backward sums, bias gradient),
//   BatchNorm apply (+skip, +ReLU), BatchNorm backward apply, ReLU backward, 2x2 max-pool forward/backward.
// Every lane moves 16 bytes per access along the channel axis; per-channel sums are reduced in a fixed
// order (lane-private partials -> LDS -> one partial row per block -> one finishing thread per channel,
// in double), so results do not depend on scheduling.
#include <type_traits>

#include "dev_common.h"
#include "kernels.h"

namespace oseq {

// ------------------------------------------------------------------ cast ----
// V elements per thread and trip: 8 where the caller's pointer lies on 16 bytes (one element: 268 M elements to bf16 at 4.4 TB/s, 8 at
// 5.1), the last n % V by the first threads; BEGIN: the first block also starts the training step
template <class T, int V, bool BEGIN>
__global__ void __launch_bounds__(256) cast_in_kernel(const float* __restrict__ x, T* __restrict__ out, int64_t n, StepBegin begin) {
  if (BEGIN && blockIdx.x == 0) step_begin(begin);
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * 256, groups = n / V;
  for (int64_t i = t; i < groups; i += stride) {
    float v[V];
    if constexpr (V == 8) {
      load_f32<float, 4>(x + i * 8, reinterpret_cast<float (&)[4]>(v[0]));
      load_f32<float, 4>(x + i * 8 + 4, reinterpret_cast<float (&)[4]>(v[4]));
    } else {
      load_f32<float, V>(x + i * V, v);
    }
    if constexpr (V == 8 && sizeof(T) == 4) {
      store_f32<T, 4>(out + i * 8, reinterpret_cast<float (&)[4]>(v[0]));
      store_f32<T, 4>(out + i * 8 + 4, reinterpret_cast<float (&)[4]>(v[4]));
    } else {
      store_f32<T, V>(out + i * V, v);
    }
  }
  if (V > 1 && t < n - groups * V) out[groups * V + t] = from_f32<T>(x[groups * V + t]);
}

template <class T>
__global__ void cast_out_kernel(const T* __restrict__ x, float* __restrict__ out, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) out[i] = to_f32(x[i]);
}

// ----------------------------------------------------- column reductions ----
// RED_BN_BWD: ReLU decisions redone from z (or none); _AOUT: from the sign of the block output; _MASK: from the bits
// RED_BIAS_RELU: the gradient behind a ReLU with output aout: where that is positive, stored to dz (the same memory) and summed
enum { RED_STATS = 0, RED_BN_BWD = 1, RED_BIAS = 2, RED_BN_BWD_AOUT = 3, RED_BN_BWD_MASK = 4, RED_BIAS_RELU = 5 };

struct RedArgs {
  const void* a;       // STATS: z ; BN_BWD: dA ; BIAS: dz
  const void* z;       // BN_BWD: z
  const void* aout;    // BN_BWD with skip: block output (ReLU mask source); else null
  const uint8_t* mask; // BN_BWD: ReLU decisions as bits, byte (row * C + c) / V holds those of V = 16 / sizeof(T) channels;
                       // takes the place of aout (and of the ReLU flag: the bits are applied as they are)
  const float* stats;  // BN_BWD: [4][C] mean, rstd, scale, shift
  float* partial;      // [nblk][2][C]
  void* dz;            // BIAS_RELU
  const void* z2;      // DUAL: z and statistics of a second BatchNorm with the same dA and decisions, and its partial sums
  const float* stats2;
  float* partial2;
  int64_t rows;
  int C, relu, nblk, rows_per_block;
  FastDiv div_hw;      // GV: rows per image
};

// The block's row of partial sums from its threads' sums (TY rows of TX threads, V channels each): every one of the
// block's 2 * TX * V sums is added up by a thread of its own, the TY rows in order.  (With the TX threads of row 0 doing
// it, a 64-channel reduction in 16 bits added 2 x 8 sums of 32 values per thread one after the other.)
template <int V>
__device__ __forceinline__ void col_combine(float* smem, const float (&s0)[V], const float (&s1)[V], bool active, int tx,
                                            int ty, int TX, int TY, int CG, int C, float* __restrict__ partial) {
  const int W = TX * V;
  if (active) {
#pragma unroll
    for (int i = 0; i < V; ++i) { smem[ty * W + tx * V + i] = s0[i]; smem[(TY + ty) * W + tx * V + i] = s1[i]; }
  }
  __syncthreads();
  for (int o = threadIdx.x; o < 2 * W; o += 256) {
    const int which = o >= W ? 1 : 0, col = o - which * W;
    const int c = blockIdx.y * W + col;
    if (c >= CG * V) continue;
    const float* p = smem + which * TY * W + col;
    float t = 0.f;
#pragma unroll 8
    for (int y = 0; y < TY; ++y) t += p[y * W];
    partial[((int64_t)blockIdx.x * 2 + which) * C + c] = t;
  }
}

// GV (the BatchNorm-backward modes): a is the gradient per image, [images][C], of a block output that only a global average
// pool reads -- the same value at every pixel, so the tensor it would fill is neither written nor read
// DUAL (from the bits): a block output's BatchNorm and that of its projection shortcut, which share dA and the decisions, in one pass
// over them (at 4.2 M x 256 in bf16 two passes took 666 us each)
template <class T, int V, int MODE, bool GV = false, bool DUAL = false>
__global__ void __launch_bounds__(256) colreduce_kernel(RedArgs g) {
  extern __shared__ float smem[];  // [2][TY][TX*V]
  const int CG = g.C / V;
  const int TX = CG < 256 ? CG : 256;
  const int TY = 256 / TX;
  const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
  const int cg = blockIdx.y * TX + tx;
  const bool active = cg < CG && ty < TY;
  const int c0 = cg * V;
  float s0[V], s1[V], s2[V], mean2[V], rstd2[V];
#pragma unroll
  for (int i = 0; i < V; ++i) s0[i] = s1[i] = s2[i] = 0.f;
  constexpr bool BWD = MODE == RED_BN_BWD || MODE == RED_BN_BWD_AOUT || MODE == RED_BN_BWD_MASK;
  float mean[V], rstd[V], scale[V], shift[V];
  if (BWD && active) {
#pragma unroll
    for (int i = 0; i < V; ++i) {
      mean[i] = g.stats[c0 + i]; rstd[i] = g.stats[g.C + c0 + i];
      if (MODE == RED_BN_BWD) { scale[i] = g.stats[2 * g.C + c0 + i]; shift[i] = g.stats[3 * g.C + c0 + i]; }
      if (DUAL) { mean2[i] = g.stats2[c0 + i]; rstd2[i] = g.stats2[g.C + c0 + i]; }
    }
  }
  const int64_t r0 = (int64_t)blockIdx.x * g.rows_per_block;
  const int64_t r1 = r0 + g.rows_per_block < g.rows ? r0 + g.rows_per_block : g.rows;
  if (active) {
    const T* a = static_cast<const T*>(g.a);
    const T* z = static_cast<const T*>(g.z);
    const T* ao = MODE == RED_BN_BWD_AOUT || MODE == RED_BIAS_RELU ? static_cast<const T*>(g.aout) : nullptr;
    const uint8_t* mk = MODE == RED_BN_BWD_MASK ? g.mask : nullptr;
    // (the row loads below are non-temporal: nothing a reduction reads is read again from the cache it would fill --
    // -2 % on the BatchNorm backward of the bottleneck networks; in the apply kernels, whose output the next kernel
    // reads, the same hint slowed that reader down by as much as it gained)
    // one row's contribution, from values already in registers
    // (vo: DUAL the second z)
    auto accumulate = [&](const float (&va)[V], const float (&vz)[V], const float (&vo)[V], unsigned bits) {
      if (MODE == RED_STATS) {
#pragma unroll
        for (int i = 0; i < V; ++i) { s0[i] += va[i]; s1[i] = __fmaf_rn(va[i], va[i], s1[i]); }
      } else if (MODE == RED_BIAS_RELU) {
#pragma unroll
        for (int i = 0; i < V; ++i) s0[i] += vo[i] > 0.f ? va[i] : 0.f;
      } else if (MODE == RED_BIAS) {
#pragma unroll
        for (int i = 0; i < V; ++i) s0[i] += va[i];
      } else {
#pragma unroll
        for (int i = 0; i < V; ++i) {
          bool on = true;
          if (MODE == RED_BN_BWD_MASK) on = (bits >> i) & 1u;
          else if (MODE == RED_BN_BWD_AOUT) { if (g.relu) on = vo[i] > 0.f; }
          else if (g.relu) on = bn_affine(vz[i], scale[i], shift[i]) > 0.f;
          const float dy = on ? va[i] : 0.f;
          const float xh = (vz[i] - mean[i]) * rstd[i];
          s0[i] += dy; s1[i] = __fmaf_rn(dy, xh, s1[i]);
          if (DUAL) s2[i] = __fmaf_rn(dy, (vo[i] - mean2[i]) * rstd2[i], s2[i]);
        }
      }
    };
    // RT rows per trip while RT remain: their loads are all issued before the first value is used; the rows are still
    // added in the same order.  (Two tensors per row in the BatchNorm-backward modes: two rows per trip measured as
    // well as four or a little better, with fewer registers; with the gradient per image it is one tensor again.)
    constexpr int RT = BWD && !GV ? 2 : 4;
    int64_t r = r0 + ty;
    for (; r + (RT - 1) * (int64_t)TY < r1; r += RT * (int64_t)TY) {
      float va[RT][V], vz[RT][V], vo[RT][V];
      unsigned mb[RT];
#pragma unroll
      for (int u = 0; u < RT; ++u) {
        const int64_t off = (r + (int64_t)u * TY) * g.C + c0;
        if (GV) load_f32<T, V>(a + (int64_t)g.div_hw.div((uint32_t)(r + (int64_t)u * TY)) * g.C + c0, va[u]);
        else load_f32_nt<T, V>(a + off, va[u]);
        mb[u] = 0u;
        if (BWD) {
          load_f32_nt<T, V>(z + off, vz[u]);
          if (MODE == RED_BN_BWD_MASK) mb[u] = mk[(r + (int64_t)u * TY) * CG + cg];
          if (DUAL) load_f32_nt<T, V>(static_cast<const T*>(g.z2) + off, vo[u]);
          else if (MODE == RED_BN_BWD_AOUT) load_f32<T, V>(ao + off, vo[u]);
        }
        if (MODE == RED_BIAS_RELU) load_f32<T, V>(ao + off, vo[u]);
      }
      if (MODE == RED_BIAS_RELU) {
#pragma unroll
        for (int u = 0; u < RT; ++u) {
          float d[V];
#pragma unroll
          for (int i = 0; i < V; ++i) d[i] = vo[u][i] > 0.f ? va[u][i] : 0.f;
          store_f32<T, V>(static_cast<T*>(g.dz) + (r + (int64_t)u * TY) * g.C + c0, d);
        }
      }
#pragma unroll
      for (int u = 0; u < RT; ++u) accumulate(va[u], vz[u], vo[u], mb[u]);
    }
    for (; r < r1; r += TY) {
      const int64_t off = r * g.C + c0;
      float va[V], vz[V], vo[V];
      unsigned mb = 0u;
      if (GV) load_f32<T, V>(a + (int64_t)g.div_hw.div((uint32_t)r) * g.C + c0, va);
      else load_f32_nt<T, V>(a + off, va);
      if (BWD) {
        load_f32_nt<T, V>(z + off, vz);
        if (MODE == RED_BN_BWD_MASK) mb = mk[r * CG + cg];
        else if (MODE == RED_BN_BWD_AOUT) load_f32<T, V>(ao + off, vo);
        if (DUAL) load_f32_nt<T, V>(static_cast<const T*>(g.z2) + off, vo);
      }
      if (MODE == RED_BIAS_RELU) {
        float d[V];
        load_f32<T, V>(ao + off, vo);
#pragma unroll
        for (int i = 0; i < V; ++i) d[i] = vo[i] > 0.f ? va[i] : 0.f;
        store_f32<T, V>(static_cast<T*>(g.dz) + off, d);
      }
      accumulate(va, vz, vo, mb);
    }
  }
  col_combine<V>(smem, s0, s1, active, tx, ty, TX, TY, CG, g.C, g.partial);
  if (DUAL) {
    __syncthreads();
    col_combine<V>(smem, s0, s2, active, tx, ty, TX, TY, CG, g.C, g.partial2);
  }
}

template <class T, int MODE, bool GV>
static void launch_colreduce_t(hipStream_t st, const RedArgs& g0) {
  RedArgs g = g0;
  const int vmax = 16 / (int)sizeof(T);
  const int V = (g.C % vmax == 0) ? vmax : 1;
  const int CG = g.C / V;
  const int TX = CG < 256 ? CG : 256;
  const int TY = 256 / TX;
  g.rows_per_block = ceil_div(g.rows, g.nblk);
  dim3 grid(g.nblk, ceil_div(CG, TX));
  const size_t sm = (size_t)2 * TY * TX * V * sizeof(float);
  if constexpr (MODE == RED_BN_BWD_MASK) {
    if (g.z2) {  // (the bits exist for whole groups only)
      OSEQ_LAUNCH((colreduce_kernel<T, 16 / sizeof(T), MODE, GV, true>), grid, dim3(256), sm, st, g);
      return;
    }
  }
  if (V == vmax) OSEQ_LAUNCH((colreduce_kernel<T, 16 / sizeof(T), MODE, GV>), grid, dim3(256), sm, st, g);
  else if constexpr (!GV) OSEQ_LAUNCH((colreduce_kernel<T, 1, MODE>), grid, dim3(256), sm, st, g);  // (GV: whole groups only)
}

template <int MODE, bool GV = false>
static void launch_colreduce(hipStream_t st, int dt, const RedArgs& g) {
  if (dt == DT_F32) launch_colreduce_t<float, MODE, GV>(st, g);
  else if (dt == DT_BF16) launch_colreduce_t<bf16_t, MODE, GV>(st, g);
  else launch_colreduce_t<f16_t, MODE, GV>(st, g);
}

// Finishing kernels: the block partials [nblk][2][C] of V neighbouring channels per block of 256 threads (V = 4 where C
// allows it).  Thread t sums the rows t, t + 256, ... in double, the loads of four rows (V floats each) issued before the
// first value is used; the lanes of a wavefront are combined by a fixed exchange that halves the number of values a lane
// carries while it halves the distance, the four wavefronts through LDS in order.  Bound by latency: the rows were written
// by blocks on other XCDs, so they come from beyond the L2, and a wavefront per channel that waits for one row's two floats
// at a time takes 4.7-5.5 us for 512 rows; with 16 channels in one block too few CUs share the work (13 us for 2048 rows).
template <int V>
__device__ __forceinline__ void partial_sums(const float* __restrict__ partial, int nblk, int C, double (&red)[4][2 * V],
                                             double& s, double& q) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double v[2 * V];
#pragma unroll
  for (int k = 0; k < 2 * V; ++k) v[k] = 0.0;
  const float* p = partial + blockIdx.x * V;
  auto rows = [&](auto UC, int b) {  // UC rows of this thread, which exist (UC = 1) or are checked
    constexpr int U = decltype(UC)::value;
    float t[U][2][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = b + u * 256 < nblk ? b + u * 256 : b;
      load_f32<float, V>(p + (int64_t)(2 * r) * C, t[u][0]);
      load_f32<float, V>(p + (int64_t)(2 * r + 1) * C, t[u][1]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (b + u * 256 < nblk) {
#pragma unroll
        for (int k = 0; k < V; ++k) { v[k] += (double)t[u][0][k]; v[V + k] += (double)t[u][1][k]; }
      }
  };
  int b = threadIdx.x;
  if (nblk > 512)
    for (; b + 512 < nblk; b += 1024) rows(std::integral_constant<int, 4>{}, b);
  if (b < nblk) rows(std::integral_constant<int, 2>{}, b);
  // (each exchange with its own constants: an array indexed by a variable would live in LDS)
  int which = 0;  // the value a lane ends up with: one bit per halving exchange, the first one highest
  auto halve = [&](auto NC, int off) {
    constexpr int n = decltype(NC)::value;
    const bool up = lane & off;
    which = which * 2 + (up ? 1 : 0);
#pragma unroll
    for (int k = 0; k < n; ++k) {
      const double keep = up ? v[n + k] : v[k], give = up ? v[k] : v[n + k];
      v[k] = keep + __shfl_xor(give, off, 64);
    }
  };
  if constexpr (V == 4) {
    halve(std::integral_constant<int, 4>{}, 32);
    halve(std::integral_constant<int, 2>{}, 16);
    halve(std::integral_constant<int, 1>{}, 8);
  } else {
    static_assert(V == 1, "four channels or one");
    halve(std::integral_constant<int, 1>{}, 32);
  }
#pragma unroll
  for (int off = 32 / (2 * V); off > 0; off >>= 1) v[0] += __shfl_xor(v[0], off, 64);
  if ((lane & (64 / (2 * V) - 1)) == 0) red[wave][which] = v[0];
  __syncthreads();
  if (threadIdx.x < V) {
    s = ((red[0][threadIdx.x] + red[1][threadIdx.x]) + red[2][threadIdx.x]) + red[3][threadIdx.x];
    q = ((red[0][V + threadIdx.x] + red[1][V + threadIdx.x]) + red[2][V + threadIdx.x]) + red[3][V + threadIdx.x];
  }
}

// Many row blocks (a convolution over a large batch writes one row of sums per 128 pixels): the rows are first added
// in STAT_FOLD_ROWS fixed ranges, with coalesced reads (thread = channel, four rows in flight per block), so that the
// finishing kernel, in which a block of 256 threads walks the columns of four channels (of one, where their number is not a
// multiple of four), has only that many rows left.  The line is where the launch more pays at every width (at 2048 rows it
// does in such a step, but not in the bottleneck network at 8 x 8).  A step of four 1x1 layers, bf16, us without and with the
// fold, 64, 256 and 1024 channels: 1024 rows 322, 950 and 320, 954; 2048: 488, 1693, 9467 and 476, 1677, 9440; 3072: 650,
// 2456, 14314 and 623, 2445, 14295; 4095: 822, 3171 and 785, 3135.
constexpr int STAT_FOLD_ROWS = 64;
constexpr int STAT_FOLD_MIN = 3072;
__global__ void __launch_bounds__(256) stat_fold_kernel(const float* __restrict__ partial, int nblk, int C, int rows_per_range,
                                                        float* __restrict__ folded) {
  __shared__ double red[2][4][64];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + tx;
  const int b0 = blockIdx.y * rows_per_range;
  const int b1 = b0 + rows_per_range < nblk ? b0 + rows_per_range : nblk;
  double s = 0.0, q = 0.0;
  if (c < C) {
    int b = b0 + ty;
    for (; b + 12 < b1; b += 16) {  // four rows of this thread per trip, loads first
      float vs[4], vq[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        vs[u] = partial[((int64_t)(b + 4 * u) * 2) * C + c];
        vq[u] = partial[((int64_t)(b + 4 * u) * 2 + 1) * C + c];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) { s += (double)vs[u]; q += (double)vq[u]; }
    }
    for (; b < b1; b += 4) {
      s += (double)partial[((int64_t)b * 2) * C + c];
      q += (double)partial[((int64_t)b * 2 + 1) * C + c];
    }
  }
  red[0][ty][tx] = s; red[1][ty][tx] = q;
  __syncthreads();
  if (ty == 0 && c < C) {
    const double ts = ((red[0][0][tx] + red[0][1][tx]) + red[0][2][tx]) + red[0][3][tx];
    const double tq = ((red[1][0][tx] + red[1][1][tx]) + red[1][2][tx]) + red[1][3][tx];
    folded[((int64_t)blockIdx.y * 2) * C + c] = (float)ts;
    folded[((int64_t)blockIdx.y * 2 + 1) * C + c] = (float)tq;
  }
}

template <int V>
__global__ void __launch_bounds__(256) bn_stats_finalize_kernel(const float* __restrict__ partial, int nblk, int C, double m,
                                                                float eps, float mom, const float* __restrict__ gamma,
                                                                const float* __restrict__ beta, float* __restrict__ stats,
                                                                float* __restrict__ running,
                                                                const int* __restrict__ flags) {
  __shared__ double red[4][2 * V];
  // (requested ahead of the sums, so that their latency does not follow the reduction's)
  const int cc = blockIdx.x * V + (threadIdx.x < V ? threadIdx.x : 0);
  const double ga = (double)gamma[cc], be = (double)beta[cc];
  const float r0 = running ? running[cc] : 0.f, r1 = running ? running[C + cc] : 0.f;
  const int bad = flags ? flags[1] : 0;
  double s, q;
  partial_sums<V>(partial, nblk, C, red, s, q);
  const int c = blockIdx.x * V + threadIdx.x;
  if (threadIdx.x >= V) return;
  const double mean = s / m;
  double var = q / m - mean * mean;
  if (var < 0.0) var = 0.0;
  const double rstd = 1.0 / sqrt(var + (double)eps);
  stats[c] = (float)mean;
  stats[C + c] = (float)rstd;
  stats[2 * C + c] = (float)(ga * rstd);
  stats[3 * C + c] = (float)(be - mean * ga * rstd);
  if (running && !bad) {  // a step with an invalid label leaves the running statistics alone
    const double unbiased = m > 1.0 ? var * m / (m - 1.0) : var;
    running[c] = (float)((1.0 - mom) * (double)r0 + mom * mean);
    running[C + c] = (float)((1.0 - mom) * (double)r1 + mom * unbiased);
  }
}

// inference mode, all BatchNorms of the network in one launch (a launch per BatchNorm was 6 % of a 50-layer network's
// inference at batch 512, an eighth at batch 16): scale and shift, the bias of the convolution in front folded in.  (Block
// column = BatchNorm; searching the job list for a running block index took 14 us for 53 of them.)
__global__ void __launch_bounds__(256) bn_eval_affine_kernel(const float* __restrict__ w, const float* __restrict__ running,
                                                             float eps, float* __restrict__ affine, EvalBatch jobs) {
  const EvalJob& e = jobs.job[blockIdx.y];
  const int c = (int)blockIdx.x * 256 + (int)threadIdx.x;
  if (c >= e.C) return;
  const float* run = running + e.rs_off;
  const double gamma = (double)w[e.gamma_off + c], beta = (double)w[e.beta_off + c];
  const double mean = (double)run[c], rstd = 1.0 / sqrt((double)run[e.C + c] + (double)eps);
  const float scale = (float)(gamma * rstd);
  double shift = beta - mean * gamma * rstd;
  if (e.bias_off >= 0) shift += gamma * rstd * (double)w[e.bias_off + c];
  affine[e.rs_off + c] = scale;
  affine[e.rs_off + e.C + c] = (float)shift;
}

template <int V>
__global__ void __launch_bounds__(256) bn_bwd_finalize_kernel(const float* __restrict__ partial, int nblk, int C, double m,
                                                              float* __restrict__ dgamma, float* __restrict__ dbeta,
                                                              float* __restrict__ coef) {
  __shared__ double red[4][2 * V];
  double s, q;
  partial_sums<V>(partial, nblk, C, red, s, q);
  const int c = blockIdx.x * V + threadIdx.x;
  if (threadIdx.x >= V) return;
  dbeta[c] = (float)s;
  dgamma[c] = (float)q;
  coef[c] = (float)(s / m);
  coef[C + c] = (float)(q / m);
}

template <int V>
__global__ void __launch_bounds__(256) bias_finalize_kernel(const float* __restrict__ partial, int nblk, int C,
                                                            float* __restrict__ dbias) {
  __shared__ double red[4][2 * V];
  double s, q;
  partial_sums<V>(partial, nblk, C, red, s, q);
  const int c = blockIdx.x * V + threadIdx.x;
  if (threadIdx.x < V) dbias[c] = (float)s;
}

// ------------------------------------------------------------- BN apply -----
// The backward apply kernel is tiled like the column reductions: a thread owns V consecutive channels, keeps their
// per-channel constants in registers and walks the rows of its block (blockIdx.x) with stride TY, two rows per trip
// with all loads of the trip issued before its first store (loads and stores share one in-order counter).  The
// optional tensors are template parameters, so that each variant is straight-line code (also in the forward kernel).
struct RowArgs {
  int64_t rows;
  int C, relu, rows_per_block;
  FastDiv div_hw;  // GV: rows per image
};

// (the forward apply kernel, with one load and one store stream, measured faster as one group of V channels per
// thread; its per-channel constants are fetched as whole vectors)
// mask (with a skip connection, V = 16 / sizeof(T)): byte i receives the ReLU decisions of group i, bit k = output k > 0
// SKIP: 0 no skip connection, 1 the tensor `skip`, 2 the BatchNorm (without ReLU) of a projection shortcut, taken from its z
// (`skip`) and statistics here instead of from a pass of its own (round(scale * z + shift), the bits that pass stored): at
// 4.2 M x 256 in bf16 that pass took 707 us for its 4.3 GB
template <class T, int V, int SKIP>
__global__ void __launch_bounds__(256) bn_apply_kernel(const T* __restrict__ z, const float* __restrict__ stats,
                                                       const T* __restrict__ skip, const float* __restrict__ skip_stats,
                                                       T* __restrict__ out, uint8_t* __restrict__ mask, int64_t groups, int C,
                                                       int relu) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= groups) return;
  const int CG = C / V;
  const int c0 = (int)(i % CG) * V;
  const int64_t off = i * V;
  float vz[V], vs[V], vo[V], scale[V], shift[V];
  load_f32<T, V>(z + off, vz);
  if (SKIP) load_f32<T, V>(skip + off, vs);
  load_f32<float, V>(stats + 2 * C + c0, scale);
  load_f32<float, V>(stats + 3 * C + c0, shift);
  if (SKIP == 2) {
    float sc2[V], sh2[V];
    load_f32<float, V>(skip_stats + 2 * C + c0, sc2);
    load_f32<float, V>(skip_stats + 3 * C + c0, sh2);
#pragma unroll
    for (int k = 0; k < V; ++k) vs[k] = bn_affine(vs[k], sc2[k], sh2[k]);
    // (rounded as a store would: in pairs, or with the value kept apart from the multiply-add in front of it -- a scalar conversion
    // to fp16 is merged with that into one instruction, which rounds once)
    if constexpr (V == 1) asm("" : "+v"(vs[0]));
    const Vec<T, V> sv = round_vec<T, V>(vs);
#pragma unroll
    for (int k = 0; k < V; ++k) vs[k] = to_f32(sv.v[k]);
  }
#pragma unroll
  for (int k = 0; k < V; ++k) {
    float y = bn_affine(vz[k], scale[k], shift[k]);
    if (SKIP) y = __fadd_rn(y, vs[k]);
    vo[k] = relu ? fmaxf(y, 0.f) : y;
  }
  store_f32<T, V>(out + off, vo);
  if (SKIP && V > 1 && mask) {
    unsigned bits = 0u;
#pragma unroll
    for (int k = 0; k < V; ++k) bits |= (vo[k] > 0.f ? 1u : 0u) << k;
    mask[i] = (uint8_t)bits;
  }
}

// BatchNorm apply (+ReLU) and the 2x2 max-pool that follows it in one pass over z: a thread owns one pooled position
// of V channels, i.e. the four activations of its window.  The activations are rounded to the storage type before the
// maximum is taken, as the separate pooling kernel finds them in memory, so the result is the same bits.  WRITE_A:
// the activations themselves are also kept (they are when backward needs them).
template <class T, int V, bool WRITE_A>
__global__ void __launch_bounds__(256) bn_apply_pool_kernel(const T* __restrict__ z, const float* __restrict__ stats,
                                                            T* __restrict__ a, T* __restrict__ y, int N, int H, int W, int C,
                                                            int relu) {
  const int CG = C / V, P = H / 2, Q = W / 2;
  const int64_t total = (int64_t)N * P * Q * CG;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int cg = (int)(i % CG);
  int64_t t = i / CG;
  const int q = (int)(t % Q); t /= Q;
  const int pp = (int)(t % P);
  const int n = (int)(t / P);
  const int c0 = cg * V;
  const int64_t base = (((int64_t)n * H + 2 * pp) * W + 2 * q) * C + c0;
  const int64_t offs[4] = {0, (int64_t)C, (int64_t)W * C, (int64_t)W * C + C};
  float vz[4][V], scale[V], shift[V];
#pragma unroll
  for (int u = 0; u < 4; ++u) load_f32<T, V>(z + base + offs[u], vz[u]);
  load_f32<float, V>(stats + 2 * C + c0, scale);
  load_f32<float, V>(stats + 3 * C + c0, shift);
  float m[V];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    float va[V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
      const float yv = bn_affine(vz[u][k], scale[k], shift[k]);
      va[k] = to_f32(from_f32<T>(relu ? fmaxf(yv, 0.f) : yv));
      m[k] = (u == 0 || va[k] > m[k]) ? va[k] : m[k];
    }
    if (WRITE_A) store_f32<T, V>(a + base + offs[u], va);
  }
  store_f32<T, V>(y + i * V, m);
}

// AOUT: the ReLU mask comes from the block output (a residual sum) instead of being rebuilt from z; DSKIP: the masked
// gradient is also written out for the skip branch
// MS: where the ReLU decisions come from: 0 redone from z, 1 the sign of the block output aout, 2 the bits of mask
// GV: da is the gradient per image, [images][C] (as in colreduce_kernel)
template <class T, int V, int MS, bool DSKIP, bool GV = false>
__global__ void __launch_bounds__(256) bn_bwd_apply_kernel(const T* __restrict__ da, const T* __restrict__ z,
                                                           const T* __restrict__ aout, const uint8_t* __restrict__ mask,
                                                           const float* __restrict__ stats,
                                                           const float* __restrict__ coef, T* __restrict__ dz,
                                                           T* __restrict__ dskip, RowArgs g) {
  const int CG = g.C / V;
  const int TX = CG < 256 ? CG : 256;
  const int TY = 256 / TX;
  const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
  const int cg = blockIdx.y * TX + tx;
  if (cg >= CG || ty >= TY) return;
  const int c0 = cg * V;
  constexpr bool AOUT = MS == 1;
  float mean[V], rstd[V], scale[V], shift[V], cb[V], cg2[V];
#pragma unroll
  for (int k = 0; k < V; ++k) {
    const int c = c0 + k;
    mean[k] = stats[c]; rstd[k] = stats[g.C + c]; scale[k] = stats[2 * g.C + c]; shift[k] = stats[3 * g.C + c];
    cb[k] = coef[c]; cg2[k] = coef[g.C + c];
  }
  const int64_t r0 = (int64_t)blockIdx.x * g.rows_per_block;
  const int64_t r1 = r0 + g.rows_per_block < g.rows ? r0 + g.rows_per_block : g.rows;
  auto one = [&](const float (&va)[V], const float (&vz)[V], const float (&vo)[V], unsigned bits, float (&rz)[V],
                 float (&rs)[V]) {
#pragma unroll
    for (int k = 0; k < V; ++k) {
      bool on = true;
      if (MS == 2) on = (bits >> k) & 1u;
      else if (g.relu) on = AOUT ? (vo[k] > 0.f) : (bn_affine(vz[k], scale[k], shift[k]) > 0.f);
      const float dy = on ? va[k] : 0.f;
      const float xh = (vz[k] - mean[k]) * rstd[k];
      rz[k] = scale[k] * (dy - cb[k] - xh * cg2[k]);
      rs[k] = dy;
    }
  };
  // two rows per trip, all loads before the stores (four rows: 575 against 544 us for the whole backward of a block
  // output at 262 144 x 1024, bf16; one row: 550)
  constexpr int RT = 2;
  int64_t r = r0 + ty;
  for (; r + (RT - 1) * (int64_t)TY < r1; r += RT * (int64_t)TY) {
    float va[RT][V], vz[RT][V], vo[RT][V], rz[RT][V], rs[RT][V];
    unsigned mb[RT];
#pragma unroll
    for (int u = 0; u < RT; ++u) {
      const int64_t off = (r + (int64_t)u * TY) * g.C + c0;
      if (!GV) load_f32<T, V>(da + off, va[u]);
      load_f32<T, V>(z + off, vz[u]);
      if (AOUT) load_f32<T, V>(aout + off, vo[u]);
      mb[u] = MS == 2 ? mask[(r + (int64_t)u * TY) * CG + cg] : 0u;
    }
    if (GV) {  // (the division in its address stays behind the loads from memory)
#pragma unroll
      for (int u = 0; u < RT; ++u) load_f32<T, V>(da + (int64_t)g.div_hw.div((uint32_t)(r + (int64_t)u * TY)) * g.C + c0, va[u]);
    }
#pragma unroll
    for (int u = 0; u < RT; ++u) one(va[u], vz[u], vo[u], mb[u], rz[u], rs[u]);
#pragma unroll
    for (int u = 0; u < RT; ++u) {
      const int64_t off = (r + (int64_t)u * TY) * g.C + c0;
      store_f32<T, V>(dz + off, rz[u]);
      if (DSKIP) store_f32<T, V>(dskip + off, rs[u]);
    }
  }
  for (; r < r1; r += TY) {
    const int64_t off = r * g.C + c0;
    float va[V], vz[V], vo[V], rz[V], rs[V];
    unsigned mb = 0u;
    load_f32<T, V>(GV ? da + (int64_t)g.div_hw.div((uint32_t)r) * g.C + c0 : da + off, va);
    load_f32<T, V>(z + off, vz);
    if (AOUT) load_f32<T, V>(aout + off, vo);
    if (MS == 2) mb = mask[r * CG + cg];
    one(va, vz, vo, mb, rz, rs);
    store_f32<T, V>(dz + off, rz);
    if (DSKIP) store_f32<T, V>(dskip + off, rs);
  }
}

// ---- BatchNorm(+ReLU) backward through the 2x2 max-pool behind it ---------------------------------------------
// The pool's backward, the gradient it would write (dA, full resolution) and the activation it would read are all
// skipped: a thread owns one pooled position of V channels, reads the four z of its window and the pooled gradient,
// rebuilds the four activations as the forward kernel computed them (rounded to the storage type), finds the first
// maximum in scan order, and so knows dA at its four positions.  Two kernels with the same tiling: the per-channel
// sums (as colreduce: row blocks of pooled positions, partial [nblk][2][C]) and, after the finishing kernel, dz.
struct PoolBwdArgs {
  int64_t rows;  // pooled positions N * P * Q
  int C, relu, rows_per_block, W, Q, PQ, HW;  // full-resolution width, pooled width, pooled / full positions per image
};

template <class T, int V>
__device__ __forceinline__ void pool_window_grad(const T* __restrict__ z, const T* __restrict__ dy, int64_t r, int c0,
                                                 const PoolBwdArgs& g, const float (&scale)[V], const float (&shift)[V],
                                                 float (&vz)[4][V], float (&dyv)[4][V], int64_t (&off)[4]) {
  const int64_t n = r / g.PQ;
  const int rem = (int)(r - n * g.PQ);
  const int p = rem / g.Q, q = rem - p * g.Q;
  off[0] = ((n * g.HW + (int64_t)(2 * p) * g.W + 2 * q)) * g.C + c0;
  off[1] = off[0] + g.C; off[2] = off[0] + (int64_t)g.W * g.C; off[3] = off[2] + g.C;
  float gy[V];
#pragma unroll
  for (int u = 0; u < 4; ++u) load_f32<T, V>(z + off[u], vz[u]);
  load_f32<T, V>(dy + r * g.C + c0, gy);
#pragma unroll
  for (int k = 0; k < V; ++k) {
    float y[4], m = 0.f;
    int arg = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      y[u] = bn_affine(vz[u][k], scale[k], shift[k]);
      const float a = to_f32(from_f32<T>(g.relu ? fmaxf(y[u], 0.f) : y[u]));
      if (u == 0 || a > m) { m = a; arg = u; }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool on = !g.relu || y[u] > 0.f;
      dyv[u][k] = (arg == u && on) ? gy[k] : 0.f;
    }
  }
}

template <class T, int V>
__global__ void __launch_bounds__(256) bn_bwd_pool_reduce_kernel(const T* __restrict__ dy, const T* __restrict__ z,
                                                                 const float* __restrict__ stats, float* __restrict__ partial,
                                                                 PoolBwdArgs g) {
  extern __shared__ float smem[];  // [2][TY][TX*V]
  const int CG = g.C / V;
  const int TX = CG < 256 ? CG : 256;
  const int TY = 256 / TX;
  const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
  const int cg = blockIdx.y * TX + tx;
  const bool active = cg < CG && ty < TY;
  const int c0 = cg * V;
  float s0[V], s1[V];
#pragma unroll
  for (int i = 0; i < V; ++i) s0[i] = s1[i] = 0.f;
  if (active) {
    float mean[V], rstd[V], scale[V], shift[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
      mean[i] = stats[c0 + i]; rstd[i] = stats[g.C + c0 + i];
      scale[i] = stats[2 * g.C + c0 + i]; shift[i] = stats[3 * g.C + c0 + i];
    }
    const int64_t r0 = (int64_t)blockIdx.x * g.rows_per_block;
    const int64_t r1 = r0 + g.rows_per_block < g.rows ? r0 + g.rows_per_block : g.rows;
    for (int64_t r = r0 + ty; r < r1; r += TY) {
      float vz[4][V], dyv[4][V];
      int64_t off[4];
      pool_window_grad<T, V>(z, dy, r, c0, g, scale, shift, vz, dyv, off);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < V; ++i) {
          const float xh = (vz[u][i] - mean[i]) * rstd[i];
          s0[i] += dyv[u][i]; s1[i] = __fmaf_rn(dyv[u][i], xh, s1[i]);
        }
    }
  }
  col_combine<V>(smem, s0, s1, active, tx, ty, TX, TY, CG, g.C, partial);
}

template <class T, int V>
__global__ void __launch_bounds__(256) bn_bwd_pool_apply_kernel(const T* __restrict__ dy, const T* __restrict__ z,
                                                                const float* __restrict__ stats, const float* __restrict__ coef,
                                                                T* __restrict__ dz, PoolBwdArgs g) {
  const int CG = g.C / V;
  const int TX = CG < 256 ? CG : 256;
  const int TY = 256 / TX;
  const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
  const int cg = blockIdx.y * TX + tx;
  if (cg >= CG || ty >= TY) return;
  const int c0 = cg * V;
  float mean[V], rstd[V], scale[V], shift[V], cb[V], cg2[V];
#pragma unroll
  for (int k = 0; k < V; ++k) {
    const int c = c0 + k;
    mean[k] = stats[c]; rstd[k] = stats[g.C + c]; scale[k] = stats[2 * g.C + c]; shift[k] = stats[3 * g.C + c];
    cb[k] = coef[c]; cg2[k] = coef[g.C + c];
  }
  const int64_t r0 = (int64_t)blockIdx.x * g.rows_per_block;
  const int64_t r1 = r0 + g.rows_per_block < g.rows ? r0 + g.rows_per_block : g.rows;
  for (int64_t r = r0 + ty; r < r1; r += TY) {
    float vz[4][V], dyv[4][V];
    int64_t off[4];
    pool_window_grad<T, V>(z, dy, r, c0, g, scale, shift, vz, dyv, off);
    float rz[4][V];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int k = 0; k < V; ++k) {
        const float xh = (vz[u][k] - mean[k]) * rstd[k];
        rz[u][k] = scale[k] * (dyv[u][k] - cb[k] - xh * cg2[k]);
      }
#pragma unroll
    for (int u = 0; u < 4; ++u) store_f32<T, V>(dz + off[u], rz[u]);
  }
}

template <class T, int V>
__global__ void __launch_bounds__(256) relu_bwd_kernel(const T* __restrict__ da, const T* __restrict__ a,
                                                       T* __restrict__ dz, int64_t groups) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= groups) return;
  float va[V], vo[V], r[V];
  load_f32<T, V>(da + i * V, va);
  load_f32<T, V>(a + i * V, vo);
#pragma unroll
  for (int k = 0; k < V; ++k) r[k] = vo[k] > 0.f ? va[k] : 0.f;
  store_f32<T, V>(dz + i * V, r);
}

// -------------------------------------------------------------- max-pool ----
template <class T, int V>
__global__ void __launch_bounds__(256) maxpool_fwd_kernel(const T* __restrict__ x, T* __restrict__ y, int N, int H, int W,
                                                          int C, int P, int Q) {
  const int CG = C / V;
  const int64_t total = (int64_t)N * P * Q * CG;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int cg = (int)(i % CG);
  int64_t t = i / CG;
  const int q = (int)(t % Q); t /= Q;
  const int p = (int)(t % P);
  const int n = (int)(t / P);
  const T* base = x + (((int64_t)n * H + 2 * p) * W + 2 * q) * C + cg * V;
  float m[V], v[V];
  load_f32<T, V>(base, m);
  load_f32<T, V>(base + C, v);
#pragma unroll
  for (int k = 0; k < V; ++k) m[k] = v[k] > m[k] ? v[k] : m[k];
  load_f32<T, V>(base + (int64_t)W * C, v);
#pragma unroll
  for (int k = 0; k < V; ++k) m[k] = v[k] > m[k] ? v[k] : m[k];
  load_f32<T, V>(base + (int64_t)W * C + C, v);
#pragma unroll
  for (int k = 0; k < V; ++k) m[k] = v[k] > m[k] ? v[k] : m[k];
  store_f32<T, V>(y + i * V, m);
}

// One thread per input position: the gradient of its window goes to the first maximum in scan order.
template <class T, int V>
__global__ void __launch_bounds__(256) maxpool_bwd_kernel(const T* __restrict__ x, const T* __restrict__ dy,
                                                          T* __restrict__ dx, int N, int H, int W, int C, int P, int Q) {
  const int CG = C / V;
  const int64_t total = (int64_t)N * H * W * CG;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int cg = (int)(i % CG);
  int64_t t = i / CG;
  const int w = (int)(t % W); t /= W;
  const int h = (int)(t % H);
  const int n = (int)(t / H);
  float r[V];
#pragma unroll
  for (int k = 0; k < V; ++k) r[k] = 0.f;
  const int p = h >> 1, q = w >> 1;
  if (p < P && q < Q) {
    const T* base = x + (((int64_t)n * H + 2 * p) * W + 2 * q) * C + cg * V;
    float m[V], v[V], g[V];
    int arg[V];
    load_f32<T, V>(base, m);
#pragma unroll
    for (int k = 0; k < V; ++k) arg[k] = 0;
    load_f32<T, V>(base + C, v);
#pragma unroll
    for (int k = 0; k < V; ++k) if (v[k] > m[k]) { m[k] = v[k]; arg[k] = 1; }
    load_f32<T, V>(base + (int64_t)W * C, v);
#pragma unroll
    for (int k = 0; k < V; ++k) if (v[k] > m[k]) { m[k] = v[k]; arg[k] = 2; }
    load_f32<T, V>(base + (int64_t)W * C + C, v);
#pragma unroll
    for (int k = 0; k < V; ++k) if (v[k] > m[k]) { m[k] = v[k]; arg[k] = 3; }
    load_f32<T, V>(dy + (((int64_t)n * P + p) * Q + q) * C + cg * V, g);
    const int me = (h & 1) * 2 + (w & 1);
#pragma unroll
    for (int k = 0; k < V; ++k) r[k] = arg[k] == me ? g[k] : 0.f;
  }
  store_f32<T, V>(dx + i * V, r);
}

// ---------------------------------------------------------------- launch ----
#define DISPATCH_TV(dt, C, CALL)                                               \
  do {                                                                         \
    if (dt == DT_F32) { if ((C) % 4 == 0) { CALL(float, 4); } else { CALL(float, 1); } } \
    else if (dt == DT_BF16) { if ((C) % 8 == 0) { CALL(bf16_t, 8); } else { CALL(bf16_t, 1); } } \
    else { if ((C) % 8 == 0) { CALL(f16_t, 8); } else { CALL(f16_t, 1); } }     \
  } while (0)

// a finishing kernel over C channels: four per block, or one where C is not a multiple of four
#define FIN_LAUNCH(KERNEL, ...)                                                             \
  do {                                                                                      \
    if (C % 4 == 0) OSEQ_LAUNCH(KERNEL<4>, dim3(C / 4), dim3(256), __VA_ARGS__);            \
    else OSEQ_LAUNCH(KERNEL<1>, dim3(C), dim3(256), __VA_ARGS__);                           \
  } while (0)

template <class T, int V>
static void launch_cast_v(hipStream_t st, const float* x, void* out, int64_t n, const StepBegin* begin) {
  const int64_t want = (n / V + 255) / 256;
  const dim3 grid((unsigned)(want < 1 ? 1 : want < 8192 ? want : 8192));
  const StepBegin none{};
  if (begin) OSEQ_LAUNCH((cast_in_kernel<T, V, true>), grid, dim3(256), 0, st, x, (T*)out, n, *begin);
  else OSEQ_LAUNCH((cast_in_kernel<T, V, false>), grid, dim3(256), 0, st, x, (T*)out, n, none);
}
template <class T>
static void launch_cast_t(hipStream_t st, const float* x, void* out, int64_t n, const StepBegin* begin) {
  // (few elements: one per thread spreads them over more CUs)
  if ((reinterpret_cast<uintptr_t>(x) & 15) == 0 && n >= 1 << 20) launch_cast_v<T, 8>(st, x, out, n, begin);
  else launch_cast_v<T, 1>(st, x, out, n, begin);
}
void launch_cast_in(hipStream_t st, int dt, const float* x, void* out, int64_t n, const StepBegin* begin) {
  if (dt == DT_F32) launch_cast_t<float>(st, x, out, n, begin);
  else if (dt == DT_BF16) launch_cast_t<bf16_t>(st, x, out, n, begin);
  else launch_cast_t<f16_t>(st, x, out, n, begin);
}

void launch_cast_out(hipStream_t st, int dt, const void* x, float* out, int64_t n) {
  const int blocks = (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
  if (dt == DT_F32) OSEQ_LAUNCH(cast_out_kernel<float>, dim3(blocks), dim3(256), 0, st, (const float*)x, out, n);
  else if (dt == DT_BF16) OSEQ_LAUNCH(cast_out_kernel<bf16_t>, dim3(blocks), dim3(256), 0, st, (const bf16_t*)x, out, n);
  else OSEQ_LAUNCH(cast_out_kernel<f16_t>, dim3(blocks), dim3(256), 0, st, (const f16_t*)x, out, n);
}

void launch_bn_stats(hipStream_t st, int dt, const void* z, int64_t rows, int C, int nblk, float* partial, float eps,
                     float mom, const float* gamma, const float* beta, float* stats, float* running,
                     const int* flags) {
  RedArgs g{}; g.a = z; g.partial = partial; g.rows = rows; g.C = C; g.nblk = nblk;
  launch_colreduce<RED_STATS>(st, dt, g);
  FIN_LAUNCH(bn_stats_finalize_kernel, 0, st, partial, nblk, C, (double)rows,
                     eps, mom, gamma, beta, stats, running, flags);
}

int bn_stats_fold_rows(int nblk) { return nblk >= STAT_FOLD_MIN ? STAT_FOLD_ROWS : 0; }

// partial: [nblk][2][C] block sums, followed by room for [bn_stats_fold_rows(nblk)][2][C] floats
void launch_bn_stats_finalize(hipStream_t st, float* partial, int64_t rows, int C, int nblk, float eps, float mom,
                              const float* gamma, const float* beta, float* stats, float* running,
                              const int* flags) {
  if (bn_stats_fold_rows(nblk) > 0) {
    float* folded = partial + (int64_t)nblk * 2 * C;
    const int per = ceil_div(nblk, STAT_FOLD_ROWS);
    const int ranges = ceil_div(nblk, per);  // no empty range
    OSEQ_LAUNCH(stat_fold_kernel, dim3(ceil_div(C, 64), ranges), dim3(256), 0, st, partial, nblk, C, per, folded);
    partial = folded;
    nblk = ranges;
  }
  FIN_LAUNCH(bn_stats_finalize_kernel, 0, st, partial, nblk, C, (double)rows,
                     eps, mom, gamma, beta, stats, running, flags);
}

// Row blocks of the apply kernels: eight rows per thread (the per-channel constants are fetched once per block; with
// two-row trips the whole backward of a block output at 262 144 x 1024, bf16, takes 556 / 543 / 532 / 545 / 575 us at
// 32 / 16 / 8 / 4 / 2 rows) when that still leaves about four blocks per CU, else fewer (small tensors), from the
// shape only.
static void row_tiling(int64_t rows, int C, int V, RowArgs& g, dim3& grid) {
  const int CG = C / V;
  const int TX = CG < 256 ? CG : 256;
  const int TY = 256 / TX;
  const int ytiles = ceil_div(CG, TX);
  int per_thread = 8;
  while (per_thread > 1 && (int64_t)ceil_div(rows, (int64_t)TY * per_thread) * ytiles < 1024) per_thread /= 2;
  g.rows = rows; g.C = C; g.rows_per_block = TY * per_thread;
  grid = dim3(ceil_div(rows, g.rows_per_block), ytiles);
}

void launch_bn_eval_affine(hipStream_t st, const float* w, const float* running, float eps, float* affine, const EvalJob* jobs,
                           int njobs) {
  for (int j0 = 0; j0 < njobs; j0 += EvalBatch::MAX_JOBS) {
    EvalBatch b{};
    b.n = njobs - j0 < EvalBatch::MAX_JOBS ? njobs - j0 : EvalBatch::MAX_JOBS;
    int most = 1;  // channels
    for (int j = 0; j < b.n; ++j) {
      b.job[j] = jobs[j0 + j];
      if (b.job[j].C > most) most = b.job[j].C;
    }
    OSEQ_LAUNCH(bn_eval_affine_kernel, dim3(ceil_div(most, 256), b.n), dim3(256), 0, st, w, running, eps, affine, b);
  }
}

void launch_bn_apply(hipStream_t st, int dt, const void* z, const float* stats, const void* skip, const float* skip_stats,
                     void* out, void* mask, int64_t rows, int C, int relu) {
#define APPLY(T, V, SK)                                                                                                \
  OSEQ_LAUNCH((bn_apply_kernel<T, V, SK>), dim3(ceil_div(groups, 256)), dim3(256), 0, st, (const T*)z, stats,         \
              (const T*)skip, skip_stats, (T*)out, mk, groups, C, relu)
#define CALL(T, V)                                                                                                     \
  { const int64_t groups = rows * (C / V);                                                                              \
    uint8_t* mk = V > 1 ? (uint8_t*)mask : nullptr;                                                                     \
    if (skip_stats) APPLY(T, V, 2); else if (skip) APPLY(T, V, 1); else APPLY(T, V, 0); }
  DISPATCH_TV(dt, C, CALL);
#undef CALL
#undef APPLY
}

void launch_bn_apply_pool(hipStream_t st, int dt, const void* z, const float* stats, void* a, void* y, int N, int H, int W,
                          int C, int relu) {
#define CALL(T, V)                                                                                                     \
  { const int64_t total = (int64_t)N * (H / 2) * (W / 2) * (C / V);                                                     \
    if (a) OSEQ_LAUNCH((bn_apply_pool_kernel<T, V, true>), dim3(ceil_div(total, 256)), dim3(256), 0, st, (const T*)z,   \
                       stats, (T*)a, (T*)y, N, H, W, C, relu);                                                          \
    else OSEQ_LAUNCH((bn_apply_pool_kernel<T, V, false>), dim3(ceil_div(total, 256)), dim3(256), 0, st, (const T*)z,    \
                     stats, (T*)a, (T*)y, N, H, W, C, relu); }
  DISPATCH_TV(dt, C, CALL);
#undef CALL
}

void launch_bn_bwd(hipStream_t st, int dt, const void* da, const void* z, const void* aout, const void* mask,
                   const float* stats, int64_t rows, int C, int relu, int nblk, float* ws, float* dgamma, float* dbeta,
                   void* dz, void* dskip, int per_image, bool summed, const BnBwdDual& dual) {
  RedArgs g{}; g.div_hw = make_fastdiv(per_image ? (uint32_t)per_image : 1u); g.a = da; g.z = z; g.aout = aout; g.mask = (const uint8_t*)mask; g.stats = stats; g.partial = ws; g.rows = rows;
  g.C = C; g.relu = relu; g.nblk = nblk;
  g.z2 = dual.z; g.stats2 = dual.stats; g.partial2 = dual.ws;
  // the same choice of the ReLU decisions' source as the apply kernel below makes
  const int vmax = dt == DT_F32 ? 4 : 8;
  if (summed) {
  } else if (per_image) {
    if (mask) launch_colreduce<RED_BN_BWD_MASK, true>(st, dt, g);
    else launch_colreduce<RED_BN_BWD, true>(st, dt, g);
  } else if (mask && C % vmax == 0) launch_colreduce<RED_BN_BWD_MASK>(st, dt, g);
  else if (aout) launch_colreduce<RED_BN_BWD_AOUT>(st, dt, g);
  else launch_colreduce<RED_BN_BWD>(st, dt, g);
  float* coef = ws + (int64_t)nblk * 2 * C;
  FIN_LAUNCH(bn_bwd_finalize_kernel, 0, st, ws, nblk, C, (double)rows, dgamma,
                     dbeta, coef);
  if (!dz) return;
#define APPLY(T, V, MS, ...)                                                                                            \
  OSEQ_LAUNCH((bn_bwd_apply_kernel<T, V, MS, __VA_ARGS__>), grid, dim3(256), 0, st, (const T*)da, (const T*)z,             \
                     (const T*)aout, (const uint8_t*)mask, stats, coef, (T*)dz, (T*)dskip, ra)
#define CALL(T, V)                                                                                                      \
  { RowArgs ra{}; dim3 grid; row_tiling(rows, C, V, ra, grid); ra.relu = relu; ra.div_hw = g.div_hw;                     \
    if (per_image && V > 1) { if (mask) APPLY(T, V, 2, false, true); else APPLY(T, V, 0, false, true); }                 \
    else if (mask && V > 1) { if (dskip) APPLY(T, V, 2, true); else APPLY(T, V, 2, false); }                                  \
    else if (aout) { if (dskip) APPLY(T, V, 1, true); else APPLY(T, V, 1, false); }                                      \
    else { if (dskip) APPLY(T, V, 0, true); else APPLY(T, V, 0, false); } }
  DISPATCH_TV(dt, C, CALL);
#undef CALL
#undef APPLY
}

// BatchNorm(+ReLU) backward where dy is the gradient of the 2x2 max-pool behind the activation: z [N][H][W][C] (H, W
// even), dy [N][H/2][W/2][C]; ws as for launch_bn_bwd
void launch_bn_bwd_pool(hipStream_t st, int dt, const void* dy, const void* z, const float* stats, int N, int H, int W, int C,
                        int relu, int nblk, float* ws, float* dgamma, float* dbeta, void* dz) {
  PoolBwdArgs g{};
  g.rows = (int64_t)N * (H / 2) * (W / 2); g.C = C; g.relu = relu; g.W = W; g.Q = W / 2; g.PQ = (H / 2) * (W / 2); g.HW = H * W;
  float* coef = ws + (int64_t)nblk * 2 * C;
#define CALL(T, V)                                                                                                       \
  { const int CG = C / V, TX = CG < 256 ? CG : 256, TY = 256 / TX, ytiles = ceil_div(CG, TX);                              \
    PoolBwdArgs gr = g; gr.rows_per_block = ceil_div(g.rows, nblk);                                                        \
    OSEQ_LAUNCH((bn_bwd_pool_reduce_kernel<T, V>), dim3(nblk, ytiles), dim3(256), (size_t)2 * TY * TX * V * sizeof(float), \
                st, (const T*)dy, (const T*)z, stats, ws, gr);                                                             \
    FIN_LAUNCH(bn_bwd_finalize_kernel, 0, st, ws, nblk, C, (double)N * H * W, dgamma,    \
                dbeta, coef);                                                                                              \
    PoolBwdArgs ga = g; int per = 2;                                                                                       \
    while (per > 1 && (int64_t)ceil_div(g.rows, (int64_t)TY * per) * ytiles < 1024) per /= 2;                              \
    ga.rows_per_block = TY * per;                                                                                          \
    OSEQ_LAUNCH((bn_bwd_pool_apply_kernel<T, V>), dim3(ceil_div(g.rows, ga.rows_per_block), ytiles), dim3(256), 0, st,     \
                (const T*)dy, (const T*)z, stats, coef, (T*)dz, ga); }
  DISPATCH_TV(dt, C, CALL);
#undef CALL
}

void launch_relu_bwd(hipStream_t st, int dt, const void* da, const void* a, void* dz, int64_t rows, int C) {
#define CALL(T, V)                                                                                                  \
  { const int64_t groups = rows * (C / V);                                                                           \
    OSEQ_LAUNCH((relu_bwd_kernel<T, V>), dim3(ceil_div(groups, 256)), dim3(256), 0, st, (const T*)da,         \
                       (const T*)a, (T*)dz, groups); }
  DISPATCH_TV(dt, C, CALL);
#undef CALL
}

void launch_bias_grad(hipStream_t st, int dt, void* dz, const void* a, int64_t rows, int C, int nblk, float* partial,
                      float* dbias) {
  RedArgs g{}; g.a = dz; g.aout = a; g.dz = dz; g.partial = partial; g.rows = rows; g.C = C; g.nblk = nblk;
  if (a) launch_colreduce<RED_BIAS_RELU>(st, dt, g);
  else launch_colreduce<RED_BIAS>(st, dt, g);
  FIN_LAUNCH(bias_finalize_kernel, 0, st, partial, nblk, C, dbias);
}

void launch_maxpool_fwd(hipStream_t st, int dt, const void* x, void* y, int N, int H, int W, int C) {
  const int P = H / 2, Q = W / 2;
#define CALL(T, V)                                                                                                  \
  { const int64_t total = (int64_t)N * P * Q * (C / V);                                                              \
    OSEQ_LAUNCH((maxpool_fwd_kernel<T, V>), dim3(ceil_div(total, 256)), dim3(256), 0, st, (const T*)x, (T*)y, \
                       N, H, W, C, P, Q); }
  DISPATCH_TV(dt, C, CALL);
#undef CALL
}

void launch_maxpool_bwd(hipStream_t st, int dt, const void* x, const void* dy, void* dx, int N, int H, int W, int C) {
  const int P = H / 2, Q = W / 2;
#define CALL(T, V)                                                                                                  \
  { const int64_t total = (int64_t)N * H * W * (C / V);                                                              \
    OSEQ_LAUNCH((maxpool_bwd_kernel<T, V>), dim3(ceil_div(total, 256)), dim3(256), 0, st, (const T*)x,        \
                       (const T*)dy, (T*)dx, N, H, W, C, P, Q); }
  DISPATCH_TV(dt, C, CALL);
#undef CALL
}

}  // namespace oseq
