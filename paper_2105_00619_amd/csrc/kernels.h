// Host-callable launchers of the HIP kernels.  Plain device pointers and sizes; `dt` is the storage type of
// activations and 16-bit weight copies (0 fp32, 1 bf16, 2 fp16).  All launches are asynchronous on `st`.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace oseq {

enum { DT_F32 = 0, DT_BF16 = 1, DT_F16 = 2 };

struct ConvGeom { int N, H, W, C, K, R, S, stride, pad, P, Q; };

// The inference-mode BatchNorm behind a convolution, done in the convolution's epilogue: out = [ReLU](scale * sum + shift
// [+ skip]), one rounding.  affine: [2][C_out] scale and shift, null for a convolution on its own; skip: null or the
// activation of the skip connection, shaped as the output.
struct ConvEval { const float* affine = nullptr; const void* skip = nullptr; };

// scale and shift of every BatchNorm of the network from the running statistics, all in one launch per 96 of them
struct EvalJob { int64_t gamma_off, beta_off, bias_off, rs_off; int C; };  // bias_off: the convolution's, or -1
struct EvalBatch { static constexpr int MAX_JOBS = 96; EvalJob job[MAX_JOBS]; int n; };
// w: master weights; running: [..](mean[C], var[C]) at rs_off; affine: [..](scale[C], shift[C]) at rs_off
void launch_bn_eval_affine(hipStream_t st, const float* w, const float* running, float eps, float* affine, const EvalJob* jobs,
                           int njobs);

// flags (four ints) cleared, flags[1] = a label lies outside [0, classes)
struct StepBegin { int* flags; const int32_t* y; int n, classes; };
// begin: null, or the start of a training step, done by the same launch
void launch_cast_in(hipStream_t st, int dt, const float* x, void* out, int64_t n, const StepBegin* begin = nullptr);
// storage type -> fp32 (read-back of an activation for inspection)
void launch_cast_out(hipStream_t st, int dt, const void* x, float* out, int64_t n);
void launch_bn_stats(hipStream_t st, int dt, const void* z, int64_t rows, int C, int nblk, float* partial, float eps,
                     float mom, const float* gamma, const float* beta, float* stats, float* running, const int* flags);
// flags[1] != 0 (an invalid label in this step's batch) keeps `running` as it is.
// the same from per-block sums a convolution already produced: partial [nblk][2][C]
// (with many blocks the rows are first folded into bn_stats_fold_rows(nblk) rows, written behind the block sums:
// partial has room for [nblk + bn_stats_fold_rows(nblk)][2][C] floats)
int bn_stats_fold_rows(int nblk);
void launch_bn_stats_finalize(hipStream_t st, float* partial, int64_t rows, int C, int nblk, float eps, float mom,
                              const float* gamma, const float* beta, float* stats, float* running, const int* flags);
// mask (null, or with a skip connection and C a multiple of 16 / element size): receives the ReLU decisions as bits,
// byte (row * C + c) / V for the V = 16 / element size channels from c
// skip_stats (null: none): skip is not the skip connection but the z of its BatchNorm (a projection shortcut's, without
// ReLU) and this that BatchNorm's statistics tensor
void launch_bn_apply(hipStream_t st, int dt, const void* z, const float* stats, const void* skip, const float* skip_stats,
                     void* out, void* mask, int64_t rows, int C, int relu);
// BatchNorm apply and the 2x2 max-pool behind it in one pass (H, W even): z [N][H][W][C] -> a (may be null: not kept)
// and y [N][H/2][W/2][C]
void launch_bn_apply_pool(hipStream_t st, int dt, const void* z, const float* stats, void* a, void* y, int N, int H, int W,
                          int C, int relu);
// per_image (0: no): da is the gradient per image, [rows / per_image][C], of a tensor that only a global average pool reads;
// then C is a multiple of 16 / element size, aout and dskip are null, rows < 2^32
// dz null: the sums, dgamma, dbeta and, behind the partial sums in ws, their means [2][C] only
// ReLU decisions: from mask (bits as launch_bn_apply writes them, applied whatever relu says) if given, else from the
// sign of aout if given, else redone from z when relu is set
// dual (with a mask; C a multiple of 16 / element size): also the nblk rows of partial sums of a second BatchNorm with the same da and mask
struct BnBwdDual { const void* z = nullptr; const float* stats = nullptr; float* ws = nullptr; };
void launch_bn_bwd(hipStream_t st, int dt, const void* da, const void* z, const void* aout, const void* mask,
                   const float* stats, int64_t rows, int C, int relu, int nblk, float* ws, float* dgamma, float* dbeta,
                   void* dz, void* dskip, int per_image, bool summed = false, const BnBwdDual& dual = BnBwdDual());
// summed: ws holds the nblk rows of partial sums already
// the same where dy is the gradient of the 2x2 max-pool that follows the activation ([N][H/2][W/2][C]; H, W even): the
// pool's own backward pass is not run
void launch_bn_bwd_pool(hipStream_t st, int dt, const void* dy, const void* z, const float* stats, int N, int H, int W, int C,
                        int relu, int nblk, float* ws, float* dgamma, float* dbeta, void* dz);
void launch_relu_bwd(hipStream_t st, int dt, const void* da, const void* a, void* dz, int64_t rows, int C);
// a (or null): dz is the gradient behind a ReLU whose output is a; it gets the ReLU applied, in place, and is then summed
void launch_bias_grad(hipStream_t st, int dt, void* dz, const void* a, int64_t rows, int C, int nblk, float* partial,
                      float* dbias);
void launch_maxpool_fwd(hipStream_t st, int dt, const void* x, void* y, int N, int H, int W, int C);
void launch_maxpool_bwd(hipStream_t st, int dt, const void* x, const void* dy, void* dx, int N, int H, int W, int C);

// The BatchNorm apply whose output only the head's global average pool reads, done by the pooling kernel (x is then its z): the
// output itself is never written.  As launch_bn_apply; C a multiple of 16 / element size
struct HeadApply { const float* stats; const void* skip; const float* skip_stats; void* mask; int relu; };
// few samples and classes: the losses and their mean in one launch
bool head_loss_in_one(int N, int J);
void launch_head_fwd(hipStream_t st, int dt, const void* x, int N, int HW, int C, int gap, int F, int J, const float* w,
                     const float* b, const int32_t* y, float gscale, float* feat, float* logits, float* dlogits,
                     float* loss_n, float* loss_out, int* flags, float* ws, const HeadApply* apply = nullptr);
// forward of the head up to the logits (no loss): inference
void launch_head_logits(hipStream_t st, int dt, const void* x, int N, int HW, int C, int gap, int F, int J, const float* w,
                        const float* b, float* feat, float* logits, float* ws, const HeadApply* apply = nullptr);
// ws: workspace of the forward pass, where its sums are split over ranges (null: they are not)
// in_x: it is to lie in the head's input, of which only the first kernel (pooling, conversion) reads
int64_t head_ws_floats(int dt, int N, int HW, int C, int gap, int F, int J, bool in_x);
// dx: gradient of the head's input, or null; dx_image (GAP): the same per image, [N][C] in the storage type, or null
void launch_head_bwd(hipStream_t st, int dt, const float* feat, const float* dlogits, const float* w, int N, int HW, int C,
                     int gap, int F, int J, float* dw, float* db, float* dfeat, void* dx, void* dx_image);

void launch_conv_fwd_direct(hipStream_t st, int dt, const void* x, const void* w, const float* bias, void* out,
                            const ConvGeom& g, int relu, const ConvEval& ev = ConvEval());
void launch_conv_dgrad_direct(hipStream_t st, int dt, const void* dz, const void* w, const void* addend, void* dx,
                              const ConvGeom& g);
void launch_conv_wgrad_direct(hipStream_t st, int dt, const void* x, const void* dz, float* dw, float* partial, int splits,
                              const ConvGeom& g);

// few input channels (the stem): plain-FMA kernels with the weights in LDS
bool conv_smallc_fwd_ok(const ConvGeom& g);
bool conv_smallc_wgrad_ok(const ConvGeom& g);
int conv_smallc_wgrad_splits(int dt, const ConvGeom& g, int64_t room);  // room: as for conv_mfma_wgrad_splits
int conv_smallc_stat_blocks(int dt, const ConvGeom& g);
void launch_conv_fwd_smallc(hipStream_t st, int dt, const void* x, const void* w, const float* bias, void* out,
                            float* stat_partial, const ConvGeom& g, int relu, const ConvEval& ev = ConvEval());
void launch_conv_wgrad_smallc(hipStream_t st, int dt, const void* x, const void* dz, float* dw, float* partial, int splits,
                              const ConvGeom& g);

// matrix-core implicit GEMM (k_conv_mfma.hip); the *_ok predicates depend on the layer shape only
bool conv_mfma_fwd_ok(int dt, const ConvGeom& g);
bool conv_mfma_dgrad_ok(int dt, const ConvGeom& g);
int conv_mfma_fwd_splits(int dt, const ConvGeom& g);
int conv_mfma_dgrad_splits(int dt, const ConvGeom& g);
// partial: fp32 workspace of splits * (output elements) floats when splits > 1, else unused
int conv_mfma_fwd_stat_blocks(int dt, const ConvGeom& g, bool bias);  // bias: the layer adds one in front of its BatchNorm
// blocks of the forward pass's 3x3 patch kernel whose LDS a CU holds (unpadded: would hold without padding between the rows of a
// patch), 0: the layer does not take it; for the tests
int conv_patch_blocks_per_cu(int dt, const ConvGeom& g, bool unpadded);
// whether it keeps the rows of a patch apart in LDS; for the tests
bool conv_patch_rows_padded(int dt, const ConvGeom& g);
// fold (null: none): x is not the input activation but the z of the BatchNorm + ReLU in front of the layer, and fold
// that BatchNorm's [4][C_in] statistics tensor (mean, rstd, scale, shift): the kernel turns z into the activation --
// the very values the apply kernel would have stored -- while it stages its operand.  Only where conv_fold_fwd_ok /
// conv_fold_wgrad_ok say so (from the layer shape only), and only for a BatchNorm that is followed by a ReLU.
bool conv_fold_fwd_ok(int dt, const ConvGeom& g);
bool conv_fold_wgrad_ok(int dt, const ConvGeom& g);
void launch_conv_fwd_mfma(hipStream_t st, int dt, const void* x, const void* w, const float* bias, void* out,
                          float* partial, float* stat_partial, int splits, const ConvGeom& g, int relu,
                          const float* fold = nullptr, const ConvEval& ev = ConvEval());
// addend_mask (null, or with an addend): ReLU decisions as bits (as launch_bn_apply writes them); the addend counts
// as zero where its bit is clear.  addend_per_image (only where conv_dgrad_image_addend_ok): the addend is [N][C_in]
bool conv_dgrad_image_addend_ok(int dt, const ConvGeom& g);
// The gradient that a data gradient writes is the one behind a BatchNorm (+ReLU): its kernel also produces the sums that the
// BatchNorm's backward pass begins with, partial [conv_dgrad_sum_blocks][2][C_in] (null: not; never with an addend)
int conv_dgrad_sum_blocks(int dt, const ConvGeom& g);
struct DgradSums { float* partial = nullptr; const void* z = nullptr; const float* stats = nullptr; int relu = 0; };
void launch_conv_dgrad_mfma(hipStream_t st, int dt, const void* dz, const void* wt, const void* addend,
                            const void* addend_mask, bool addend_per_image, void* dx, float* partial, int splits, const ConvGeom& g,
                            const DgradSums& sums = DgradSums());
// 1x1 convolutions in 16-bit storage as a streaming GEMM (k_conv_pointwise.hip); used by the MFMA launchers above
bool conv_pointwise_fwd_ok(int dt, const ConvGeom& g);
bool conv_pointwise_dgrad_ok(int dt, const ConvGeom& g);
int conv_pointwise_stat_blocks(const ConvGeom& g);
bool conv_pointwise_fold_ok(int dt, const ConvGeom& g);
void launch_conv_fwd_pointwise(hipStream_t st, int dt, const void* x, const void* w, const float* bias, void* out,
                               float* stat_partial, const ConvGeom& g, int relu, const float* fold, const ConvEval& ev);
void launch_conv_dgrad_pointwise(hipStream_t st, int dt, const void* dz, const void* wt, const void* addend,
                                 const uint8_t* addend_mask, bool addend_per_image, void* dx, const ConvGeom& g);
// 3x3 stride-1 layers of 64 input channels and many pixels with the weights stationary (k_conv_ws3x3.hip); used by the MFMA
// launchers above where nothing is added to the result
bool conv_ws3x3_ok(int dt, int N, int dstH, int dstW, int srcC, int Ng, int R, int S, int stride);
int conv_ws3x3_stat_blocks(const ConvGeom& g);
void launch_conv_fwd_ws3x3(hipStream_t st, int dt, const void* x, const void* w, void* out, float* stat_partial, const ConvGeom& g,
                           const float* fold);
void launch_conv_dgrad_ws3x3(hipStream_t st, int dt, const void* dz, const void* wt, void* dx, const ConvGeom& g);
// 3x3 stride-1 weight gradient with all nine taps per block (k_conv_wgrad3x3.hip); used by the MFMA launcher below
bool conv_wgrad3x3_ok(int dt, const ConvGeom& g);
int conv_wgrad3x3_splits(int dt, const ConvGeom& g, int64_t room);
bool conv_wgrad3x3_swaps(int dt, const ConvGeom& g);  // whether its pixels' parts are exchanged in LDS (for the tests)
void launch_conv_wgrad3x3(hipStream_t st, int dt, const void* x, const void* dz, float* dst, int splits, const ConvGeom& g,
                          const float* fold);
bool conv_mfma_wgrad_ok(int dt, const ConvGeom& g);
// room: bytes of partial sums that do not enlarge the activation arena
int conv_mfma_wgrad_splits(int dt, const ConvGeom& g, int64_t room);
void launch_conv_wgrad_mfma(hipStream_t st, int dt, const void* x, const void* dz, float* dw, float* partial, int splits,
                            const ConvGeom& g, const float* fold = nullptr);
// The backward pass of a 1x1 layer and of the BatchNorm behind it as one kernel (k_conv_bwd1x1.hip).  da .. relu, per_image as for
// launch_bn_bwd (decisions from mask or redone from z; z: only read with per_image, made again otherwise); coef: what its finishing kernel left behind the partial sums, [2][C_out];
// x, fold, partial, splits as for the weight gradient, wt, dx as for the data gradient
bool conv_bwd1x1_ok(int dt, const ConvGeom& g);
int conv_bwd1x1_splits(const ConvGeom& g);
void launch_conv_bwd1x1(hipStream_t st, int dt, const void* da, const void* z, const void* mask, const float* stats, const float* coef, int relu,
                        int per_image, const void* x, const float* fold, const void* w, const void* wt, void* dx, float* dw, float* partial,
                        int splits, const ConvGeom& g, float* sums);
// sums (null, or with fold): as DgradSums::partial for the folded BatchNorm, [splits][2][C_in]
// 1x1 layers whose output z (in front of a BatchNorm) is never in memory: made again from the layer's input by whoever reads it
// (k_conv_again.hip).  x, fold, w: the layer's input, the statistics of a BatchNorm to fold into it (or null), the weights; stats:
// those of the BatchNorm behind the layer
struct AgainSource { const void* x; const float* fold; const void* w; const float* stats; };
bool conv_again_ok(int dt, const ConvGeom& g);
// the layer's forward pass: its channel sums only (stat_partial as launch_conv_fwd_mfma leaves it)
void launch_conv_again_stats(hipStream_t st, int dt, const void* x, const float* fold, const void* w, float* stat_partial, const ConvGeom& g);
// the apply pass with ReLU and a skip connection: the tensor skip, or the BatchNorm of a projection shortcut (proj)
void launch_bn_apply_again(hipStream_t st, int dt, const AgainSource& z, const void* skip, const AgainSource* proj, void* out, void* mask,
                           const ConvGeom& g);
// rows of sums, [conv_again_sum_blocks()][2][C_out], for launch_bn_bwd (summed) from dA and its ReLU decisions as bits; with proj
// also the shortcut's, into ws2
int conv_again_sum_blocks();
void launch_bn_bwd_sums_again(hipStream_t st, int dt, const void* da, const void* mask, const AgainSource& z, const AgainSource* proj,
                              float* ws, float* ws2, const ConvGeom& g);
// adds the pixel ranges' partial sums [splits][n] in order
void launch_wgrad_reduce(hipStream_t st, const float* partial, float* out, int64_t n, int splits);
// Transposed weight copies for the data-gradient GEMMs, all layers in one launch (per 48 layers).  w_off: element
// offset of the layer's weights in the flat parameter vector (the same offset is used in the transposed copy).
struct TransposeJob { int64_t w_off; int K, RS, C, first_block; };
struct TransposeBatch { static constexpr int MAX_JOBS = 48; TransposeJob job[MAX_JOBS]; int n; };
void launch_weight_transposes(hipStream_t st, int dt, const float* wbase, void* wtbase, const TransposeJob* jobs, int njobs);

// device address and size of the per-GPU static activation arena (optorch_seq_step_static), current device
hipError_t static_arena(void** ptr, uint64_t* bytes);
void launch_step_init(hipStream_t st, const StepBegin& begin);
void launch_optim(hipStream_t st, int dt, float* w, float* v, const float* g, void* w16, float* gout, int64_t n, float lr,
                  float mom, float inv_scale, int* flags, const float* report, float* report_host);
// report, report_host: 32 floats (loss and flags) copied to page-locked host memory when the step's flags are final
void launch_cast_params(hipStream_t st, int dt, const float* w, void* w16, int64_t n);
void launch_fill(hipStream_t st, float* p, int64_t n, float v);

// Image data-flow (x uint8 [B][P]; a uint64 [ceil(B / z)][P][words]; o uint32 [ceil(B / z)][P]); z and the pointers
// are validated by the callers.  scale / shift: host arrays of `channels` (<= 16) floats.
void launch_encode(hipStream_t st, const uint8_t* x, int64_t B, int64_t P, int z, uint64_t* a);
void launch_decode(hipStream_t st, const uint64_t* a, int64_t B, int64_t P, int z, uint8_t* x);
void launch_decode_cast(hipStream_t st, int dt, const uint64_t* a, int64_t B, int64_t P, int z, int channels,
                        const float* scale, const float* shift, void* out);
void launch_encode_lossless(hipStream_t st, const uint8_t* x, int64_t B, int64_t P, int z, uint64_t* a, uint32_t* o);
void launch_decode_lossless(hipStream_t st, const uint64_t* a, const uint32_t* o, int64_t B, int64_t P, int z, uint8_t* x);

}  // namespace oseq
