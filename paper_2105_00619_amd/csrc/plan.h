// Host-side planning of the checkpointed training step: expansion of units into
// kernel-level operations, choice of segment boundaries, the static schedule
// (forward without keeping intermediates, forward of the last segment, then per
// segment in reverse: replay + backward), tensor lifetimes and offsets in the
// activation arena.  Pure host code; nothing here touches a device.
//
// Paper: Introduction (segments; inputs of segments are kept; all segments but the
// last discard intermediates) and Section "Sequential-checkpoint training" (the
// forward pass is run again from the previous checkpoint during back-propagation).
#pragma once
#include <cstdint>
#include <string>
#include <vector>

#include "optorch_seq.h"

namespace oseq {

constexpr uint64_t kAlign = 256;
inline uint64_t align_up(uint64_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// A tensor of the forward graph (one per value of the network, independent of how many
// times the schedule materialises it).
struct LTensor {
  int64_t n = 0, h = 0, w = 0, c = 0;
  int esize = 4;          // bytes per element
  uint64_t bytes = 0;     // exact, unpadded
  bool needs_grad = true; // false for the network input
  int unit = -1;          // unit that produces it (-1: network input)
};

enum FKind { F_CAST_IN, F_CONV, F_BN_STATS, F_BN_APPLY, F_POOL, F_HEAD };

enum ConvAlgo { ALGO_DIRECT = 0, ALGO_MFMA = 1, ALGO_SMALLC = 2 };

// One forward operation of the network.
struct FOp {
  FKind kind = F_CONV;
  int unit = -1;
  int x = -1, skip = -1, stats = -1, out = -1;  // LTensor ids
  int mask = -1;  // F_BN_APPLY with a skip connection: LTensor of the ReLU decisions, one bit per element (one byte per
                  // 16 bytes of the output), which the backward pass reads instead of the output itself; -1: none
  int fold = 0;       // F_BN_APPLY: 1 = never run; the one convolution that reads its output applies scale, shift and
                      // ReLU to z while it stages its operand (forward and weight gradient), so the output is never stored
  int fold_src = -1;  // F_CONV: the folded F_BN_APPLY operation its input comes from, or -1
  int fold_skip = -1; // F_BN_APPLY with a skip connection: the F_BN_APPLY of the projection shortcut that it does as well
                      // (that one's fold is 1: it reads the shortcut's z and statistics instead of its output), or -1
  int aux[3] = {-1, -1, -1};                     // head: feat, logits, dlogits
  int N = 0, H = 0, W = 0, C = 0, K = 0, R = 1, S = 1, stride = 1, pad = 0, P = 0, Q = 0;
  int relu = 0, has_bias = 0, has_bn = 0;
  int64_t w_off = -1, b_off = -1, gamma_off = -1, beta_off = -1;  // element offsets, flat parameter vector
  int64_t rs_off = -1;       // element offset of (running mean, running var) in the running-stat block
  int gap = 0, feat_dim = 0, classes = 0;
  int64_t head_ws = 0;       // floats of workspace of the head's forward pass; launches_of counts its extra launch
  bool head_one = false;     // its losses and their mean are one launch (few samples and classes)
  bool head_ws_in_x = false; // it lies in the head's input, which is the network's own and read for the last time by the first
                             // of the head's kernels
  int dgrad_sums = 0;        // F_CONV: row blocks over which the data gradient can sum for the BatchNorm backward in front of it, or 0
  int image_addend = 0;      // F_CONV: 1 = the data gradient can add one row per image (the gradient of a global average pool)
  int bwd_splits = 0;        // F_CONV: pixel ranges of the kernel that does the BatchNorm backward behind it (whose sums are known) and
                             // both gradients where the schedule allows it (S_CONV_BWD), 0: there is none for its shape
  int again_rows = 0;        // F_CONV: there are kernels for its shape that make its output z again from its input, those of the sums of
                             // the BatchNorm backward over so many row blocks; 0: there are not
  int again = 0;             // F_CONV, and the F_BN_APPLY behind it: they are used (choose_again) and z is never written.  Its place in
                             // the arena stays: the plan's figures count it, and inference at the schedule's offsets writes there
  int again_skip = -1;       // F_BN_APPLY with a skip connection, again: the F_BN_APPLY of its projection shortcut, again too, or -1
  int fwd_algo = ALGO_DIRECT, dgrad_algo = ALGO_DIRECT, wgrad_algo = ALGO_DIRECT;
  int wgrad_splits = 1;      // fixed by shape only: deterministic split of the pixel reduction
  int fwd_splits = 1, dgrad_splits = 1;  // fixed by shape only: deterministic split of the GEMM depth
  int red_blocks = 1;        // row blocks of the per-channel reductions (BN statistics, BN backward)
  int stat_blocks = 0;       // > 0: the convolution's forward kernel also writes per-block channel sums for the
                             // BatchNorm that follows (that many row blocks); set on the conv and on its F_BN_STATS
  int stat_fold = 0;         // rows into which the finishing step first folds those block sums (0: none); extra workspace
};

enum SKind {
  S_CAST_IN, S_CONV_FWD, S_BN_STATS, S_BN_APPLY, S_POOL_FWD, S_HEAD_FWD,
  S_HEAD_BWD, S_BN_BWD, S_RELU_BWD, S_BIAS_GRAD, S_WGRAD, S_DGRAD, S_POOL_BWD,
  S_CONV_BWD  // FOp::bwd_splits: apply pass of the BatchNorm backward, weight and data gradient of the convolution `fop`
};
enum Phase { PH_FWD_NOSAVE = 0, PH_FWD_LAST = 1, PH_REPLAY = 2, PH_BWD = 3 };

// One materialisation of a tensor in the activation arena.
struct Inst {
  int logical = -1;       // LTensor id, or -1 for workspaces
  uint64_t bytes = 0;
  int def_op = -1, last_use = -1;
  uint64_t offset = 0;
  bool fwd_value = false; // produced by a forward-kind operation
  bool held = false;      // checkpoint or kept for backward (counts as "saved")
  bool allocated = false;
};

// One entry of the static schedule.
struct SOp {
  SKind kind = S_CONV_FWD;
  int fop = -1;
  int phase = 0, seg = 0;
  int in[7] = {-1, -1, -1, -1, -1, -1, -1};
  int out[6] = {-1, -1, -1, -1, -1, -1};
  int variant = 0;  // S_BN_BWD: 1 = in[0] is the gradient of the 2x2 max-pool behind the activation (pooled size);
                    // 2 = in[3] is a bit mask of ReLU decisions (FOp::mask) to apply to in[0], not an activation.
                    // S_DGRAD: in[2] >= 0 is such a mask for the addend in[1]
                    // S_CONV_FWD with in[1] >= 0, S_WGRAD with in[2] >= 0: in[0] is the z of a folded BatchNorm apply
                    // and that slot its statistics tensor (FOp::fold_src)
                    // S_BN_APPLY with in[3] >= 0: in[2] is the z of the projection shortcut's BatchNorm, in[3] its
                    // statistics tensor (FOp::fold_skip)
                    // S_BN_BWD with out[0] < 0: the sums only, for the S_CONV_BWD that follows.  That one has in[0..3] as the
                    // S_BN_BWD, in[4] its workspace (for the means behind the sums), in[5] the convolution's input (the z of a
                    // folded BatchNorm with in[6] its statistics tensor), out[0] the data gradient, out[1] the weight gradient's
                    // partial sums
                    // S_DGRAD with out[2] >= 0: it makes the sums of the BatchNorm backward in front, whose z is in[3] and
                    // statistics in[4]; variant: whether a ReLU follows that BatchNorm.  S_CONV_BWD likewise (in[5], in[6]).
                    // S_BN_BWD with out[3] >= 0: it also makes those of the projection shortcut's BatchNorm (z in[5],
                    // statistics in[6]); with in[4] >= 0: its sums, made that way, which are its workspace
                    // S_BIAS_GRAD with in[1] >= 0: in[0] is the gradient behind the ReLU, in[1] the output of that; in[0]
                    // becomes the gradient in front of it, in place
                    // S_HEAD_FWD: 1 = also the BatchNorm apply operation in front of it, whose in[0..3] it has; out[5] its mask
  bool again = false;             // FOp::again.  S_CONV_FWD makes the channel sums only, which a replay does without; S_BN_APPLY and
                                  // S_BN_BWD (the sums) read src in place of their z's:
  int src[4] = {-1, -1, -1, -1};  // the convolution's input and the statistics tensor of a BatchNorm to fold into it (or -1); those of
                                  // the projection shortcut's
  int rows = 0;  // S_BN_BWD, S_CONV_BWD: rows of partial sums in the BatchNorm backward's workspace
  bool per_image = false;  // S_DGRAD: in[1] is an addend per image, [N][C]. S_BN_BWD: in[0] is the gradient per image, [N][C] (the output is only read by a global average
                           // pool).  S_HEAD_BWD: out[2] >= 0 receives it, out[0] the whole tensor where a reader needs it
  bool live = true;
};

// One entry of the inference schedule: a forward operation with the BatchNorm behind a convolution done in that
// convolution's epilogue.  Offsets into the activation arena, -1: none.  S_BN_APPLY: a copy from `in` to `out`
// (inference_in_schedule).
struct IOp {
  SKind kind = S_CONV_FWD;
  int fop = -1, apply = -1;  // apply: the F_BN_APPLY operation of the BatchNorm behind the convolution, or -1
  int64_t in = -1, skip = -1, out = -1, ws = -1;  // head: out = features, skip unused
};

constexpr char SUMS_INSIDE = 1, SUMS_SHORTCUT = 2;

struct Plan {
  // inputs
  std::vector<optorch_unit_t> units;
  optorch_seq_config_t cfg{};
  int esize = 4;  // bytes per activation element
  // forward graph
  std::vector<LTensor> tensors;
  std::vector<FOp> fops;
  std::vector<int> unit_first_fop, unit_last_fop;  // [unit] range of fops (inclusive first, exclusive last)
  std::vector<int> unit_in, unit_out;              // [unit] LTensor ids
  uint64_t n_params = 0;
  uint64_t n_running = 0;  // floats of BN running statistics
  std::vector<char> unit_sums;  // [unit] SUMS_INSIDE: kernels that write a gradient inside the unit also make the sums of the BatchNorm
                                // backward in front; SUMS_SHORTCUT: the sums of a projection shortcut's BatchNorm come with its
                                // block output's (choose_sums); empty: none
  bool z_written = false;       // FOp::again: passes that keep nothing write z nevertheless (build_schedule compares)
  bool separate = false;        // schedule every pass of the backward as an operation of its own (what choose_sums measures by)
  uint64_t separate_arena = 0;  // while build_schedule runs: the arena of such a schedule of this partition, 0 unknown
  // partition
  std::vector<int> seg_begin;  // k+1 entries, unit indices
  // schedule
  std::vector<Inst> insts;
  std::vector<SOp> sched;
  uint64_t arena_bytes = 0;       // high-water mark of the activation arena (aligned offsets)
  uint64_t peak_saved_bytes = 0;  // exact tensor sizes, no alignment
  uint64_t peak_live_bytes = 0;   // all live tensors incl. transients, exact sizes
  int n_launches = 0, n_replay_launches = 0;
  // inference: its own schedule and offsets in the same arena
  std::vector<IOp> infer;
  uint64_t infer_bytes = 0;
  std::string error;
};

// Builds the forward graph from the unit list.  Returns false and sets plan.error on failure.
bool build_graph(Plan& p);
// Chooses segment boundaries (explicit, equal count, or min peak) into plan.seg_begin.
bool choose_segments(Plan& p);
// Builds schedule, lifetimes, offsets and peak figures for plan.seg_begin.  enough: an arena of that many bytes need not be
// made smaller.
bool build_schedule(Plan& p, uint64_t enough = 0);
// [F_CONV operation] bytes of partial sums its weight gradient can write without becoming the fullest moment of its unit's
// backward pass: whatever else is alive stays alive throughout that pass, so this holds for every partition; the smaller value
// of the storage modes that keep and that rebuild activations.  From the network and the kernel choices so far only.
std::vector<int64_t> wgrad_room(const Plan& p);
// Sets unit_sums: for the units whose backward pass is then no fuller than with every pass an operation of its own, in any storage
// mode (folded: the plan with its BatchNorms folded, as modes 0 and 1 run it; p without).  Likewise from the network and the kernel
// choices so far only.
void choose_sums(Plan& p, const Plan& folded);
// Sets FOp::again in p and in folded (the plan with its BatchNorms folded), the same layers in both: from the network and the kernel
// choices only.
void choose_again(Plan& p, Plan& folded);
// Builds the inference schedule with offsets of its own; needs the kernel choices of the convolutions (workspaces of split
// depths).
void build_inference(Plan& p);
// The same operations at the offsets of the training schedule's forward entries, for a plan whose arena is too small for
// those offsets (holes between tensors of different sizes).
void inference_in_schedule(Plan& p);
// Peak saved bytes of the partition given by seg_begin, from the closed form
//   max_j ( sum_{i<=j} checkpoint_i + saved_j ),
// with per-unit saved bytes taken from the all-stored schedule.  Used by the min-peak planner.
uint64_t model_peak_saved(const Plan& p, const std::vector<int>& seg_begin);

int launches_of(const SOp& op, const FOp& f);

}  // namespace oseq
