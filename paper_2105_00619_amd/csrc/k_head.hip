// Loss head: global average pool / flatten, linear layer, mean softmax cross-entropy, and their backward.
// All arithmetic in fp32 on fp32 master weights (the head is a few MFLOP; it is kept out of the 16-bit path
// for stability, in line with keeping loss computation in single precision).  Every sum runs in a fixed order.
#include <type_traits>

#include "dev_common.h"
#include "kernels.h"

namespace oseq {

typedef __attribute__((ext_vector_type(16))) float head_v16f;

constexpr int HEAD_ONE_BLOCK = 64;
// Samples behind the first sixteen follow one another in that block, and it is one CU's: a step's time, two launches -> one, us, with 16
// samples and 1000 / 4096 / 32 768 classes -3, -3, +24; 32 and 400 / 1000: -1, +10; 48 and 200 / 400: -2, +1; 64 and 200 / 400 /
// 1000: -2, +9, +34.
bool head_loss_in_one(int N, int J) { return N <= HEAD_ONE_BLOCK && J <= 4096 && (int64_t)(N - 16) * J <= 8192; }

// flatten: feat[n][f] = x[n][f] in fp32, V features per thread
template <class T, int V>
__global__ void __launch_bounds__(256) flatten_kernel(const T* __restrict__ x, float* __restrict__ feat, int64_t groups) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= groups) return;
  float v[V];
  load_f32<T, V>(x + i * V, v);
  store_f32<float, V>(feat + i * V, v);
}

// Global average pool: block (image, group of channels, range of pixels) of TX threads of V channels and TY rows of them;
// a thread adds every TY-th pixel (eight 16-byte loads in flight, added in pairs), the TY sums of a channel are added in a fixed order.  Bound by
// reading the map once.  With one range the mean is stored; with several (few images of many pixels, which would leave most
// CUs idle: 4 images of 256 x 256 x 128 in fp32 took 1153 us in one block per image and 64 channels, 27 us like this) the
// sums go to `partial` [ranges][N][C] and gap_finish_kernel adds the ranges in order.
// APPLY: -1 x is the map; else x is the z of the BatchNorm apply in front, whose output -- the values bn_apply_kernel stores, SKIP
// as there -- is added without being written, its ReLU decisions going to mask.  (262 144 x 1024 in bf16: apply 287 us and pooling
// 119 apart.)
template <class T, int V, int APPLY = -1>
__global__ void __launch_bounds__(256) gap_sum_kernel(const T* __restrict__ x, float* __restrict__ feat,
                                                      float* __restrict__ partial, int N, int HW, int C, int TX, int per_range,
                                                      HeadApply ap) {
  __shared__ float red[256 * V];
  const int TY = 256 / TX, tx = threadIdx.x % TX, ty = threadIdx.x / TX;
  const int n = blockIdx.x;
  const int cg = blockIdx.y * TX + tx;
  const bool active = cg < C / V && ty < TY;
  const int p0 = blockIdx.z * per_range, p1 = p0 + per_range < HW ? p0 + per_range : HW;
  float s[V];
#pragma unroll
  for (int k = 0; k < V; ++k) s[k] = 0.f;
  if (active) {
    const int64_t first = (int64_t)n * HW * C + cg * V;
    const T* col = x + first;
    const T* sk = APPLY > 0 ? static_cast<const T*>(ap.skip) + first : nullptr;
    uint8_t* mk = APPLY >= 0 && ap.mask ? static_cast<uint8_t*>(ap.mask) + first / V : nullptr;
    float scale[V], shift[V], scale2[V], shift2[V];
    if (APPLY >= 0) {
      load_f32<float, V>(ap.stats + 2 * C + cg * V, scale);
      load_f32<float, V>(ap.stats + 3 * C + cg * V, shift);
    }
    if (APPLY == 2) {
      load_f32<float, V>(ap.skip_stats + 2 * C + cg * V, scale2);
      load_f32<float, V>(ap.skip_stats + 3 * C + cg * V, shift2);
    }
    auto value = [&](const Vec<T, V>& z, const Vec<T, V>& q, int p, float (&v)[V]) {  // pixel p's values
      if constexpr (APPLY < 0) {
#pragma unroll
        for (int k = 0; k < V; ++k) v[k] = to_f32(z.v[k]);
      } else {
        float vs[V], vo[V];
        if (APPLY > 0) {
#pragma unroll
          for (int k = 0; k < V; ++k) vs[k] = to_f32(q.v[k]);
        }
        if (APPLY == 2) {
#pragma unroll
          for (int k = 0; k < V; ++k) vs[k] = bn_affine(vs[k], scale2[k], shift2[k]);
          const Vec<T, V> sv = round_vec<T, V>(vs);
#pragma unroll
          for (int k = 0; k < V; ++k) vs[k] = to_f32(sv.v[k]);
        }
        unsigned bits = 0u;
#pragma unroll
        for (int k = 0; k < V; ++k) {
          float y = bn_affine(to_f32(z.v[k]), scale[k], shift[k]);
          if (APPLY > 0) y = __fadd_rn(y, vs[k]);
          vo[k] = ap.relu ? fmaxf(y, 0.f) : y;
          bits |= (vo[k] > 0.f ? 1u : 0u) << k;
        }
        if (APPLY > 0 && mk) mk[(int64_t)p * (C / V)] = (uint8_t)bits;
        const Vec<T, V> t = round_vec<T, V>(vo);
#pragma unroll
        for (int k = 0; k < V; ++k) v[k] = to_f32(t.v[k]);
      }
    };
    constexpr int U = 8;
    int p = p0 + ty;
    for (; p + (U - 1) * TY < p1; p += U * TY) {
      Vec<T, V> z[U], q[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        z[u] = *reinterpret_cast<const Vec<T, V>*>(col + (int64_t)(p + u * TY) * C);
        if (APPLY > 0) q[u] = *reinterpret_cast<const Vec<T, V>*>(sk + (int64_t)(p + u * TY) * C);
      }
      float v[U][V];
#pragma unroll
      for (int u = 0; u < U; ++u) value(z[u], q[u], p + u * TY, v[u]);
#pragma unroll
      for (int k = 0; k < V; ++k)
        s[k] += ((v[0][k] + v[1][k]) + (v[2][k] + v[3][k])) + ((v[4][k] + v[5][k]) + (v[6][k] + v[7][k]));
    }
    for (; p < p1; p += TY) {
      Vec<T, V> q{};
      float v[V];
      if (APPLY > 0) q = *reinterpret_cast<const Vec<T, V>*>(sk + (int64_t)p * C);
      value(*reinterpret_cast<const Vec<T, V>*>(col + (int64_t)p * C), q, p, v);
#pragma unroll
      for (int k = 0; k < V; ++k) s[k] += v[k];
    }
#pragma unroll
    for (int k = 0; k < V; ++k) red[ty * TX * V + tx * V + k] = s[k];
  }
  __syncthreads();
  const int W = TX * V;
  for (int o = threadIdx.x; o < W; o += 256) {
    const int c = blockIdx.y * W + o;
    if (c >= C) continue;
    float t = 0.f;
    int y = 0;
    for (; y + 4 <= TY; y += 4)
      t += (red[y * W + o] + red[(y + 1) * W + o]) + (red[(y + 2) * W + o] + red[(y + 3) * W + o]);
    for (; y < TY; ++y) t += red[y * W + o];
    if (partial) partial[((int64_t)blockIdx.z * N + n) * C + c] = t;
    else feat[(int64_t)n * C + c] = t / (float)HW;
  }
}

__global__ void __launch_bounds__(256) gap_finish_kernel(const float* __restrict__ partial, float* __restrict__ feat, int64_t n,
                                                         int ranges, int HW) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  float t = 0.f;
#pragma unroll 16
  for (int r = 0; r < ranges; ++r) t += partial[(int64_t)r * n + i];
  feat[i] = t / (float)HW;
}

// The three products of the linear layer on the fp32 matrix cores: out[row][col] = sum over k of A(row, k) * B(k, col),
//   HG_FWD  logits[n][j] = b[j] + sum_f feat[n][f] * w[j][f]        rows n, columns j, depth F
//   HG_DW   dw[j][f]     =        sum_n dlogits[n][j] * feat[n][f]  rows j, columns f (column F: the bias gradient), depth N
//   HG_DX   dfeat[n][f]  =        sum_j dlogits[n][j] * w[j][f]     rows n, columns f, depth J
// A block of KW wavefronts owns a 32 x 32 tile; wavefront w takes the 16-deep pieces w, w + KW, ... of the depth (of the
// range blockIdx.z, when the depth is split), UP of them requested at a time (four, or one where there are fewer), and the KW
// partial tiles are added in pairs through LDS.  SHORT: short chains of fp32 sums -- every piece (half of one, where registers
// are free) is summed from zero, those of a request are added in pairs, and that joins the wavefront's total.  One running sum over the
// depth has up to eight times the error of lanes striding over it (logits relative to 64 bits, 4096 samples, 2048
// features, 1000 classes: 8.1e-7 against 1.25e-7, SHORT 1.1e-7); SHORT costs the forward product 2 % of its time.
// The weight gradient needs it where one wavefront has a tile to itself (four share the depth otherwise, as they did when a
// thread owned an output), the feature gradient nowhere: a thread added all classes in a row.
// Bound by latency and by the fp32 MFMA rate (64 cycles per 32 x 32 x 2); a wavefront per
// (sample, class), or a thread per feature, re-read one operand per output: with 4096 samples, 1024 features and 100 classes
// the three took 62, 172 and 54 us (now 24, 36 and 22), with 512 samples and 2048 features the first 74 us (now 22).
// Lane l of an MFMA holds row (column) l % 32 at depth l / 32; the 16-deep piece gives lane group g the depths [8g, 8g + 8),
// so that a lane reads eight neighbours where the depth is the fast index.
enum { HG_FWD = 0, HG_DW = 1, HG_DX = 2 };
template <int KIND, int KW, int UP, bool SHORT>
__global__ void __launch_bounds__(64 * KW) head_gemm_kernel(const float* __restrict__ a, const float* __restrict__ b,
                                                            const float* __restrict__ bias, float* __restrict__ out,
                                                            float* __restrict__ out_bias, int rows, int cols, int depth, int lda,
                                                            int ldb, int depth_per_range) {
  constexpr bool A_FAST = KIND != HG_DW, B_FAST = KIND == HG_FWD;  // is the depth the fast index of the operand?
  __shared__ float red[KW > 1 ? KW * 32 * 32 : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 5, l32 = lane & 31;
  const int row0 = blockIdx.y * 32, col0 = blockIdx.x * 32;
  const int ar = row0 + l32 < rows ? row0 + l32 : 0;  // (rows and columns outside are read at 0 and not stored)
  const int bc = col0 + l32 < cols ? col0 + l32 : 0;
  const bool ones = KIND == HG_DW && col0 + l32 == cols;
  const int d0 = blockIdx.z * depth_per_range, d1 = d0 + depth_per_range < depth ? d0 + depth_per_range : depth;
  const float* ap = A_FAST ? a + (int64_t)ar * lda : a + ar;
  const float* bp = B_FAST ? b + (int64_t)bc * ldb : b + bc;
  head_v16f acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  auto piece = [&](const float* p, bool fast, int ld, int k, bool full, float (&v)[8]) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const bool in = full || k + t < d1;
      const float x = p[in ? (fast ? (int64_t)(k + t) : (int64_t)(k + t) * ld) : 0];
      v[t] = in ? x : 0.f;
    }
  };
  auto pieces = [&](auto NC, int k, bool full) {
    constexpr int n = decltype(NC)::value;
    float va[n][8], vb[n][8];
#pragma unroll
    for (int u = 0; u < n; ++u) {
      piece(ap, A_FAST, lda, k + u * 16 * KW + 8 * g, full, va[u]);
      piece(bp, B_FAST, ldb, k + u * 16 * KW + 8 * g, full, vb[u]);
    }
    auto bv = [&](int u, int t) {  // (the column of the bias gradient: ones)
      if (KIND == HG_DW) {
        const int kk = k + u * 16 * KW + 8 * g + t;
        return ones ? (full || kk < d1 ? 1.f : 0.f) : vb[u][t];
      }
      return vb[u][t];
    };
    if constexpr (!SHORT) {
#pragma unroll
      for (int u = 0; u < n; ++u)
#pragma unroll
        for (int t = 0; t < 8; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(va[u][t], bv(u, t), acc, 0, 0, 0);
    } else {
      constexpr int HALVES = KW == 8 || n == 1 ? 2 : 1, P = n * HALVES;  // pieces, or halves of them where registers are free
      head_v16f part[P];
#pragma unroll
      for (int q = 0; q < P; ++q)
#pragma unroll
        for (int e = 0; e < 16; ++e) part[q][e] = 0.f;
#pragma unroll
      for (int t = 0; t < 8 / HALVES; ++t)
#pragma unroll
        for (int q = 0; q < P; ++q) {
          const int u = q / HALVES, tt = q % HALVES * 4 + t;
          part[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[u][tt], bv(u, tt), part[q], 0, 0, 0);
        }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        float t = part[0][e] + part[1][e];
        if constexpr (P >= 4) t += part[2][e] + part[3][e];
        if constexpr (P == 8) t += (part[4][e] + part[5][e]) + (part[6][e] + part[7][e]);
        acc[e] += t;
      }
    }
  };
  int k = d0 + wave * 16;
  if constexpr (UP > 1)
    for (; k + (UP - 1) * 16 * KW + 16 <= d1; k += UP * 16 * KW) pieces(std::integral_constant<int, UP>{}, k, true);
#pragma unroll 1
  for (; k < d1; k += 16 * KW) pieces(std::integral_constant<int, 1>{}, k, false);
  auto store = [&](int r, int c, float v) {
    if (r >= rows) return;
    if (KIND == HG_FWD) {
      if (c < cols) out[((int64_t)blockIdx.z * rows + r) * cols + c] = bias ? v + bias[c] : v;
    } else {
      if (c < cols) out[(int64_t)r * cols + c] = v;
      else if (KIND == HG_DW && c == cols) out_bias[r] = v;
    }
  };
  if constexpr (KW == 1) {
#pragma unroll
    for (int e = 0; e < 16; ++e) store(row0 + 8 * (e >> 2) + 4 * g + (e & 3), col0 + l32, acc[e]);
  } else {
#pragma unroll
    for (int e = 0; e < 16; ++e) red[wave * 1024 + (8 * (e >> 2) + 4 * g + (e & 3)) * 32 + l32] = acc[e];
    __syncthreads();
    for (int o = threadIdx.x; o < 1024; o += 64 * KW) {
      float t = (red[o] + red[1024 + o]) + (red[2048 + o] + red[3072 + o]);
      if constexpr (KW == 8) t += (red[4096 + o] + red[5120 + o]) + (red[6144 + o] + red[7168 + o]);
      store(row0 + (o >> 5), col0 + (o & 31), t);
    }
  }
}

// the ranges of a split depth, added in order, and the bias
__global__ void __launch_bounds__(256) head_reduce_kernel(const float* __restrict__ partial, const float* __restrict__ bias,
                                                          float* __restrict__ out, int64_t n, int cols, int ranges) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  float t = 0.f;
#pragma unroll 8
  for (int r = 0; r < ranges; ++r) t += partial[(int64_t)r * n + i];
  out[i] = t + bias[i % cols];
}

template <int KIND>
static void launch_head_gemm(hipStream_t st, const float* a, const float* b, const float* bias, float* out, float* out_bias,
                             int rows, int cols, int depth, int lda, int ldb, int ranges) {
  const dim3 grid(ceil_div(cols + (KIND == HG_DW ? 1 : 0), 32), ceil_div(rows, 32), ranges);
  const int64_t tiles = (int64_t)grid.x * grid.y * grid.z;
  const int per = ceil_div(ceil_div(depth, ranges), 16) * 16;
  // wavefronts per tile: about eight per CU in all, at least four for a depth from 1024 on (short chains of sums), no more than
  // there are pieces
  int kw = tiles >= 2048 && (per < 1024 || KIND == HG_DX) ? 1 : tiles >= 512 ? 4 : 8;
  while (kw > 1 && kw * 16 > per) kw = kw == 8 ? 4 : 1;
#define HG_LAUNCH(KW_, UP_, SHORT_)                                                                                             \
  OSEQ_LAUNCH((head_gemm_kernel<KIND, KW_, UP_, SHORT_>), grid, dim3(64 * KW_), 0, st, a, b, bias, out, out_bias, rows, cols, \
              depth, lda, ldb, per)
  if constexpr (KIND == HG_FWD) {
    const bool four = per >= 64 * kw;
    if (kw == 8) { if (four) HG_LAUNCH(8, 4, true); else HG_LAUNCH(8, 1, true); }
    else if (kw == 4) { if (four) HG_LAUNCH(4, 4, true); else HG_LAUNCH(4, 1, true); }
    else if (four) HG_LAUNCH(1, 4, true);
    else HG_LAUNCH(1, 1, true);
  } else {
    if constexpr (KIND == HG_DW) {
      if (tiles >= 2048 && per > 128) {
        if (kw == 4) HG_LAUNCH(4, 4, true); else HG_LAUNCH(1, 4, true);
        return;
      }
    }
    if (kw == 8) HG_LAUNCH(8, 4, false);
    else if (kw == 4) HG_LAUNCH(4, 4, false);
    else HG_LAUNCH(1, 4, false);
  }
#undef HG_LAUNCH
}

// per sample: loss_n = logsumexp(logits_n) - logits_n[y_n]; dlogits = (softmax - onehot) * gscale
// one wavefront per sample; lanes stride over the classes, maxima and sums by a fixed butterfly
// MEAN: few samples (head_loss_in_one): one block of 16 wavefronts takes them all and their mean loss too
template <bool MEAN>
__global__ void __launch_bounds__(MEAN ? 1024 : 256) softmax_ce_kernel(const float* __restrict__ logits, const int32_t* __restrict__ y,
                                                         float* __restrict__ loss_n, float* __restrict__ dlogits, int N, int J,
                                                         float gscale, int* __restrict__ flags, float* __restrict__ loss_out) {
  __shared__ float losses[MEAN ? HEAD_ONE_BLOCK : 1];
  const int lane = threadIdx.x & 63;
  for (int n = MEAN ? (int)(threadIdx.x >> 6) : (int)(blockIdx.x * 4 + (threadIdx.x >> 6)); n < N; n += MEAN ? 16 : N) {
    const float* lp = logits + (int64_t)n * J;
    float mx = -INFINITY;
    for (int j = lane; j < J; j += 64) mx = fmaxf(mx, lp[j]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    float se = 0.f;
    for (int j = lane; j < J; j += 64) se += expf(lp[j] - mx);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) se += __shfl_xor(se, off, 64);
    const float lse = mx + logf(se);
    int lab = y[n];
    if (lab < 0 || lab >= J) { if (lane == 0) atomicOr(flags + 1, 1); lab = 0; }
    if (lane == 0) {
      loss_n[n] = lse - lp[lab];
      if (MEAN) losses[n] = lse - lp[lab];
    }
    const float inv = 1.f / se;
    for (int j = lane; j < J; j += 64) {
      const float pj = expf(lp[j] - mx) * inv;
      dlogits[(int64_t)n * J + j] = (pj - (j == lab ? 1.f : 0.f)) * gscale;
    }
  }
  if constexpr (MEAN) {  // added as loss_mean_kernel does
    __syncthreads();
    if (threadIdx.x < 64) {
      double t = (int)threadIdx.x < N ? (double)losses[threadIdx.x] : 0.0;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) t += __shfl_down(t, off, 64);
      if (threadIdx.x == 0) loss_out[0] = (float)(t / (double)N);
    }
  }
}

__global__ void __launch_bounds__(256) loss_mean_kernel(const float* __restrict__ loss_n, int N, float* __restrict__ out) {
  __shared__ double sm[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < N; i += 256) s += (double)loss_n[i];
  sm[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) sm[threadIdx.x] += sm[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = (float)(sm[0] / (double)N);
}

template <class T>
__global__ void head_feat_bwd_kernel(const float* __restrict__ dfeat, T* __restrict__ dx, int64_t total, int HW, int C, int gap) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  if (!gap) { dx[i] = from_f32<T>(dfeat[i]); return; }
  const int c = (int)(i % C);
  const int64_t n = i / ((int64_t)HW * C);
  dx[i] = from_f32<T>(dfeat[n * C + c] / (float)HW);
}

// the gradient per image of a map that is only averaged: the value every one of its pixels has
template <class T>
__global__ void __launch_bounds__(256) gap_bwd_image_kernel(const float* __restrict__ dfeat, T* __restrict__ dx, int64_t n, int HW) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) dx[i] = from_f32<T>(dfeat[i] / (float)HW);
}

// GAP backward for channel counts that are a multiple of V: block (chunk of rows, image n); a thread owns V channels,
// reads their gradient once and writes it to every TY-th pixel of the block's rows (16-byte stores, no divisions
// per element)
template <class T, int V>
__global__ void __launch_bounds__(256) gap_bwd_rows_kernel(const float* __restrict__ dfeat, T* __restrict__ dx, int HW, int C,
                                                           int rows_per_block) {
  const int CG = C / V;
  const int TX = CG < 256 ? CG : 256;
  const int TY = 256 / TX;
  const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
  const int n = blockIdx.y;
  const int p0 = blockIdx.x * rows_per_block;
  const int p1 = p0 + rows_per_block < HW ? p0 + rows_per_block : HW;
  if (ty >= TY) return;
  for (int cg = tx; cg < CG; cg += TX) {
    float v[V];
#pragma unroll
    for (int k = 0; k < V; ++k) v[k] = dfeat[(int64_t)n * C + cg * V + k] / (float)HW;
    Vec<T, V> t;
#pragma unroll
    for (int k = 0; k < V; ++k) t.v[k] = from_f32<T>(v[k]);
    T* base = dx + ((int64_t)n * HW) * C + cg * V;
    for (int p = p0 + ty; p < p1; p += TY) *reinterpret_cast<Vec<T, V>*>(base + (int64_t)p * C) = t;
  }
}

template <class T>
static void launch_feat_bwd(hipStream_t st, const float* dfeat, void* dx, int N, int HW, int C, int gap) {
  constexpr int V = 16 / (int)sizeof(T);
  const int64_t total = (int64_t)N * HW * C;
  if (gap && C % V == 0 && HW >= 64) {
    const int rows_per_block = 64;
    OSEQ_LAUNCH((gap_bwd_rows_kernel<T, V>), dim3(ceil_div(HW, rows_per_block), N), dim3(256), 0, st, dfeat, (T*)dx, HW, C,
                rows_per_block);
  } else {
    OSEQ_LAUNCH(head_feat_bwd_kernel<T>, dim3(ceil_div(total, 256)), dim3(256), 0, st, dfeat, (T*)dx, total, HW, C, gap);
  }
}

// Ranges of pixels (GAP) or of the depth of the linear layer (flatten) over which the head's forward pass is split, from
// the shape only: about four blocks per CU, ranges of at least 32 rows of threads (GAP) or four pieces per wavefront; and no
// more bytes of partial sums than the head's input has, so that a step's activation arena is not larger for them: the backward
// pass has the input's gradient in their place, and where there is none (the input is the network's own) they lie in the input
// itself, which the conversion has read by then.  (GAP reads it while it adds, but has 32 times as many pixels as ranges.)
static int gap_tx(int C, int V) { const int CG = C / V; return CG < 256 ? CG : 256; }
int head_ranges(int dt, int N, int HW, int C, int gap, int F, int J) {
  int64_t blocks, most;
  if (gap) {
    const int vmax = dt == DT_F32 ? 4 : 8, V = C % vmax == 0 ? vmax : 1, TX = gap_tx(C, V), TY = 256 / TX;
    blocks = (int64_t)N * ceil_div(C / V, TX);
    most = HW / (TY * 32);
  } else {
    blocks = (int64_t)ceil_div(N, 32) * ceil_div(J, 32) * 2;
    most = F / (16 * 8 * 4);
    if (most > (int64_t)F * (dt == DT_F32 ? 4 : 2) / (4 * (int64_t)J)) most = (int64_t)F * (dt == DT_F32 ? 4 : 2) / (4 * (int64_t)J);
  }
  int64_t want = (1024 + blocks - 1) / blocks;
  if (want > most) want = most;
  if (want > 128) want = 128;
  return (int)(want < 1 ? 1 : want);
}
// floats of workspace the forward pass needs for them; in_x: it has to lie in the head's input (GAP: then there is none)
int64_t head_ws_floats(int dt, int N, int HW, int C, int gap, int F, int J, bool in_x) {
  if (gap && in_x) return 0;
  const int r = head_ranges(dt, N, HW, C, gap, F, J);
  return r > 1 ? (int64_t)r * N * (gap ? C : J) : 0;
}

template <class T>
static void launch_feat_t(hipStream_t st, const T* x, int N, int HW, int C, int gap, int ranges, float* feat, float* ws,
                          const HeadApply* ap) {
  constexpr int VM = 16 / (int)sizeof(T);
  if (!gap) {
    const int64_t n = (int64_t)N * HW * C;
    if (C % VM == 0) OSEQ_LAUNCH((flatten_kernel<T, VM>), dim3(ceil_div(n / VM, 256)), dim3(256), 0, st, x, feat, n / VM);
    else OSEQ_LAUNCH((flatten_kernel<T, 1>), dim3(ceil_div(n, 256)), dim3(256), 0, st, x, feat, n);
    return;
  }
  const int V = C % VM == 0 ? VM : 1, TX = gap_tx(C, V), per = ceil_div(HW, ranges);
  const dim3 grid(N, ceil_div(C / V, TX), ranges);
  float* partial = ranges > 1 ? ws : nullptr;
  const HeadApply none{};
  if (ap && ap->skip_stats) OSEQ_LAUNCH((gap_sum_kernel<T, VM, 2>), grid, dim3(256), 0, st, x, feat, partial, N, HW, C, TX, per, *ap);
  else if (ap && ap->skip) OSEQ_LAUNCH((gap_sum_kernel<T, VM, 1>), grid, dim3(256), 0, st, x, feat, partial, N, HW, C, TX, per, *ap);
  else if (ap) OSEQ_LAUNCH((gap_sum_kernel<T, VM, 0>), grid, dim3(256), 0, st, x, feat, partial, N, HW, C, TX, per, *ap);
  else if (V == VM) OSEQ_LAUNCH((gap_sum_kernel<T, VM>), grid, dim3(256), 0, st, x, feat, partial, N, HW, C, TX, per, none);
  else OSEQ_LAUNCH((gap_sum_kernel<T, 1>), grid, dim3(256), 0, st, x, feat, partial, N, HW, C, TX, per, none);
  if (partial)
    OSEQ_LAUNCH(gap_finish_kernel, dim3(ceil_div((int64_t)N * C, 256)), dim3(256), 0, st, partial, feat, (int64_t)N * C, ranges, HW);
}

// ws: head_ws_floats(...) floats (null if that is 0: one range)
void launch_head_logits(hipStream_t st, int dt, const void* x, int N, int HW, int C, int gap, int F, int J, const float* w,
                        const float* b, float* feat, float* logits, float* ws, const HeadApply* apply) {
  const int ranges = ws ? head_ranges(dt, N, HW, C, gap, F, J) : 1;
  if (dt == DT_F32) launch_feat_t<float>(st, (const float*)x, N, HW, C, gap, ranges, feat, ws, apply);
  else if (dt == DT_BF16) launch_feat_t<bf16_t>(st, (const bf16_t*)x, N, HW, C, gap, ranges, feat, ws, apply);
  else launch_feat_t<f16_t>(st, (const f16_t*)x, N, HW, C, gap, ranges, feat, ws, apply);
  if (gap || ranges == 1) {
    launch_head_gemm<HG_FWD>(st, feat, w, b, logits, nullptr, N, J, F, F, F, 1);
  } else {
    launch_head_gemm<HG_FWD>(st, feat, w, nullptr, ws, nullptr, N, J, F, F, F, ranges);
    OSEQ_LAUNCH(head_reduce_kernel, dim3(ceil_div((int64_t)N * J, 256)), dim3(256), 0, st, ws, b, logits, (int64_t)N * J, J, ranges);
  }
}

void launch_head_fwd(hipStream_t st, int dt, const void* x, int N, int HW, int C, int gap, int F, int J, const float* w,
                     const float* b, const int32_t* y, float gscale, float* feat, float* logits, float* dlogits,
                     float* loss_n, float* loss_out, int* flags, float* ws, const HeadApply* apply) {
  launch_head_logits(st, dt, x, N, HW, C, gap, F, J, w, b, feat, logits, ws, apply);
  if (head_loss_in_one(N, J)) {
    OSEQ_LAUNCH(softmax_ce_kernel<true>, dim3(1), dim3(1024), 0, st, logits, y, loss_n, dlogits, N, J, gscale, flags, loss_out);
    return;
  }
  OSEQ_LAUNCH(softmax_ce_kernel<false>, dim3(ceil_div(N, 4)), dim3(256), 0, st, logits, y, loss_n, dlogits, N, J, gscale, flags, loss_out);
  OSEQ_LAUNCH(loss_mean_kernel, dim3(1), dim3(256), 0, st, loss_n, N, loss_out);
}

void launch_head_bwd(hipStream_t st, int dt, const float* feat, const float* dlogits, const float* w, int N, int HW, int C,
                     int gap, int F, int J, float* dw, float* db, float* dfeat, void* dx, void* dx_image) {
  launch_head_gemm<HG_DW>(st, dlogits, feat, nullptr, dw, db, J, F, N, J, F, 1);
  if (!dx && !dx_image) return;
  launch_head_gemm<HG_DX>(st, dlogits, w, nullptr, dfeat, nullptr, N, F, J, J, F, 1);
  if (dx_image) {
    const int64_t n = (int64_t)N * C;
    const dim3 grid(ceil_div(n, 256)), block(256);
    if (dt == DT_F32) OSEQ_LAUNCH(gap_bwd_image_kernel<float>, grid, block, 0, st, dfeat, (float*)dx_image, n, HW);
    else if (dt == DT_BF16) OSEQ_LAUNCH(gap_bwd_image_kernel<bf16_t>, grid, block, 0, st, dfeat, (bf16_t*)dx_image, n, HW);
    else OSEQ_LAUNCH(gap_bwd_image_kernel<f16_t>, grid, block, 0, st, dfeat, (f16_t*)dx_image, n, HW);
  }
  if (!dx) return;
  if (dt == DT_F32) launch_feat_bwd<float>(st, dfeat, dx, N, HW, C, gap);
  else if (dt == DT_BF16) launch_feat_bwd<bf16_t>(st, dfeat, dx, N, HW, C, gap);
  else launch_feat_bwd<f16_t>(st, dfeat, dx, N, HW, C, gap);
}

}  // namespace oseq
