// Host-side planner; see plan.h.
#include "plan.h"

#include <algorithm>
#include <cstdio>
#include <map>

namespace oseq {

namespace {

struct ConvParams { int64_t w = -1, b = -1, gamma = -1, beta = -1, rs = -1; };

struct Builder {
  Plan& p;
  int N;
  explicit Builder(Plan& pl) : p(pl), N(pl.cfg.batch) {}

  bool fail(const std::string& m) { p.error = m; return false; }

  int new_tensor(int64_t n, int64_t h, int64_t w, int64_t c, int esize, int unit) {
    LTensor t;
    t.n = n; t.h = h; t.w = w; t.c = c; t.esize = esize; t.unit = unit;
    t.bytes = (uint64_t)n * h * w * c * esize;
    p.tensors.push_back(t);
    return (int)p.tensors.size() - 1;
  }

  ConvParams alloc_conv_params(int cin, int cout, int k, int bn, int bias) {
    ConvParams q;
    q.w = (int64_t)p.n_params; p.n_params += (uint64_t)cout * k * k * cin;
    if (bias) { q.b = (int64_t)p.n_params; p.n_params += cout; }
    if (bn) {
      q.gamma = (int64_t)p.n_params; p.n_params += cout;
      q.beta = (int64_t)p.n_params; p.n_params += cout;
      q.rs = (int64_t)p.n_running; p.n_running += 2 * (uint64_t)cout;
    }
    return q;
  }

  // conv [+bias] [+BN [+skip]] [+ReLU]; appends the forward operations, returns the output tensor
  int add_cbr(int unit, int x, const ConvParams& q, int cout, int k, int stride, int pad, int bn,
              int relu, int bias, int skip) {
    const LTensor tx = p.tensors[x];
    FOp f;
    f.kind = F_CONV; f.unit = unit; f.x = x;
    f.N = (int)tx.n; f.H = (int)tx.h; f.W = (int)tx.w; f.C = (int)tx.c; f.K = cout; f.R = k; f.S = k;
    f.stride = stride; f.pad = pad;
    f.P = (f.H + 2 * pad - k) / stride + 1;
    f.Q = (f.W + 2 * pad - k) / stride + 1;
    f.has_bias = bias; f.has_bn = bn; f.relu = bn ? 0 : relu;
    f.w_off = q.w; f.b_off = q.b;
    const int64_t pixels = (int64_t)f.N * f.P * f.Q;
    const int64_t outputs = (int64_t)f.K * f.R * f.S * f.C;
    int64_t splits = (262144 + outputs - 1) / outputs;
    splits = std::min<int64_t>(splits, std::max<int64_t>(1, pixels / 32));
    f.wgrad_splits = (int)std::max<int64_t>(1, std::min<int64_t>(splits, 256));
    f.red_blocks = (int)std::max<int64_t>(1, std::min<int64_t>(pixels / 32, 512));
    int z = new_tensor(f.N, f.P, f.Q, cout, p.esize, unit);
    f.out = z;
    p.fops.push_back(f);
    if (!bn) return z;

    FOp s;
    s.kind = F_BN_STATS; s.unit = unit; s.x = z;
    s.N = f.N; s.H = f.P; s.W = f.Q; s.C = cout; s.K = cout; s.P = f.P; s.Q = f.Q;
    s.gamma_off = q.gamma; s.beta_off = q.beta; s.rs_off = q.rs;
    s.red_blocks = (int)std::max<int64_t>(1, std::min<int64_t>(pixels / 32, 512));
    s.stats = new_tensor(1, 1, 4, cout, 4, unit);  // mean, rstd, scale, shift
    s.out = s.stats;
    p.fops.push_back(s);

    FOp a = s;
    a.kind = F_BN_APPLY; a.skip = skip; a.relu = relu;
    a.out = new_tensor(f.N, f.P, f.Q, cout, p.esize, unit);
    // The ReLU behind a skip connection cannot be redone from z alone; backward needs its decisions.  They are kept as
    // one bit per element (one byte per group of 16 / esize channels), a sixteenth of the bytes of the output that
    // backward would otherwise read twice.
    const int vgroup = 16 / p.esize;
    if (skip >= 0 && relu && cout % vgroup == 0) {
      a.mask = new_tensor(f.N, f.P, f.Q, cout / vgroup, 1, unit);
      p.tensors[a.mask].needs_grad = false;
    }
    p.fops.push_back(a);
    return a.out;
  }

  bool run() {
    const optorch_seq_config_t& c = p.cfg;
    p.esize = c.precision == OPTORCH_FP32 ? 4 : 2;
    if (p.units.empty()) return fail("empty unit list");
    int cur = new_tensor(N, c.height, c.width, c.channels, p.esize, -1);
    p.tensors[cur].needs_grad = false;
    {
      FOp f; f.kind = F_CAST_IN; f.unit = -1; f.out = cur;
      f.N = N; f.H = c.height; f.W = c.width; f.C = c.channels;
      p.fops.push_back(f);
    }
    const int nu = (int)p.units.size();
    p.unit_first_fop.assign(nu, 0); p.unit_last_fop.assign(nu, 0);
    p.unit_in.assign(nu, -1); p.unit_out.assign(nu, -1);
    for (int ui = 0; ui < nu; ++ui) {
      const optorch_unit_t& u = p.units[ui];
      const LTensor tx = p.tensors[cur];
      p.unit_first_fop[ui] = (int)p.fops.size();
      p.unit_in[ui] = cur;
      char where[64]; snprintf(where, sizeof where, "unit %d: ", ui);
      const bool is_head = u.kind == OPTORCH_GAP_LINEAR_CE || u.kind == OPTORCH_FLATTEN_LINEAR_CE;
      if (is_head != (ui == nu - 1)) return fail(std::string(where) + "exactly the last unit must be a loss head");
      switch (u.kind) {
        case OPTORCH_CONV: {
          if (u.cin != tx.c) return fail(std::string(where) + "cin does not match the incoming channel count");
          if (!(u.ksize == 1 || u.ksize == 3) || !(u.stride == 1 || u.stride == 2) || u.cout < 1 || u.pad < 0 ||
              u.pad > u.ksize / 2)
            return fail(std::string(where) + "unsupported convolution geometry (ksize 1|3, stride 1|2, pad <= ksize/2)");
          if (tx.h + 2 * u.pad < u.ksize || tx.w + 2 * u.pad < u.ksize) return fail(std::string(where) + "input smaller than the filter");
          ConvParams q = alloc_conv_params(u.cin, u.cout, u.ksize, u.has_bn, u.has_bias);
          cur = add_cbr(ui, cur, q, u.cout, u.ksize, u.stride, u.pad, u.has_bn != 0, u.has_relu != 0, u.has_bias != 0, -1);
          break;
        }
        case OPTORCH_MAXPOOL2: {
          if (tx.h < 2 || tx.w < 2) return fail(std::string(where) + "max-pool input smaller than 2x2");
          FOp f; f.kind = F_POOL; f.unit = ui; f.x = cur;
          f.N = N; f.H = (int)tx.h; f.W = (int)tx.w; f.C = (int)tx.c; f.K = f.C; f.P = f.H / 2; f.Q = f.W / 2;
          f.out = new_tensor(N, f.P, f.Q, f.C, p.esize, ui);
          p.tensors[f.out].needs_grad = p.tensors[f.x].needs_grad;
          p.fops.push_back(f);
          cur = f.out;
          break;
        }
        case OPTORCH_BASIC_BLOCK:
        case OPTORCH_BOTTLENECK: {
          if (u.cin != tx.c) return fail(std::string(where) + "cin does not match the incoming channel count");
          if (!(u.stride == 1 || u.stride == 2) || u.cout < 1) return fail(std::string(where) + "unsupported block geometry");
          const bool bott = u.kind == OPTORCH_BOTTLENECK;
          if (bott && (u.cout % 4 != 0)) return fail(std::string(where) + "bottleneck cout must be a multiple of 4");
          const bool proj = (u.cin != u.cout) || (u.stride != 1);
          const int mid = bott ? u.cout / 4 : u.cout;
          ConvParams q1, q2, q3, qs;
          if (bott) {
            q1 = alloc_conv_params(u.cin, mid, 1, 1, 0);
            q2 = alloc_conv_params(mid, mid, 3, 1, 0);
            q3 = alloc_conv_params(mid, u.cout, 1, 1, 0);
          } else {
            q1 = alloc_conv_params(u.cin, u.cout, 3, 1, 0);
            q2 = alloc_conv_params(u.cout, u.cout, 3, 1, 0);
          }
          if (proj) qs = alloc_conv_params(u.cin, u.cout, 1, 1, 0);
          const int x = cur;
          int a;
          if (bott) {
            a = add_cbr(ui, x, q1, mid, 1, 1, 0, 1, 1, 0, -1);
            a = add_cbr(ui, a, q2, mid, 3, u.stride, 1, 1, 1, 0, -1);
          } else {
            a = add_cbr(ui, x, q1, u.cout, 3, u.stride, 1, 1, 1, 0, -1);
          }
          int skip = x;
          if (proj) skip = add_cbr(ui, x, qs, u.cout, 1, u.stride, 0, 1, 0, 0, -1);
          if (bott) cur = add_cbr(ui, a, q3, u.cout, 1, 1, 0, 1, 1, 0, skip);
          else      cur = add_cbr(ui, a, q2, u.cout, 3, 1, 1, 1, 1, 0, skip);
          break;
        }
        case OPTORCH_GAP_LINEAR_CE:
        case OPTORCH_FLATTEN_LINEAR_CE: {
          if (u.cin != tx.c) return fail(std::string(where) + "cin does not match the incoming channel count");
          if (u.cout != c.num_classes) return fail(std::string(where) + "cout must equal num_classes");
          FOp f; f.kind = F_HEAD; f.unit = ui; f.x = cur;
          f.N = N; f.H = (int)tx.h; f.W = (int)tx.w; f.C = (int)tx.c;
          f.gap = u.kind == OPTORCH_GAP_LINEAR_CE;
          f.feat_dim = f.gap ? f.C : f.H * f.W * f.C;
          f.classes = u.cout; f.has_bias = 1;
          f.w_off = (int64_t)p.n_params; p.n_params += (uint64_t)f.classes * f.feat_dim;
          f.b_off = (int64_t)p.n_params; p.n_params += f.classes;
          f.aux[0] = new_tensor(N, 1, 1, f.feat_dim, 4, ui);
          f.aux[1] = new_tensor(N, 1, 1, f.classes, 4, ui);
          f.aux[2] = new_tensor(N, 1, 1, f.classes, 4, ui);
          f.out = new_tensor(N, 1, 1, 1, 4, ui);
          p.fops.push_back(f);
          cur = f.out;
          break;
        }
        default:
          return fail(std::string(where) + "unknown unit kind");
      }
      p.unit_last_fop[ui] = (int)p.fops.size();
      p.unit_out[ui] = cur;
    }
    return true;
  }
};

// ---------------------------------------------------------------- arena -----
struct FreeList {
  std::map<uint64_t, uint64_t> free_;  // offset -> size
  uint64_t end_ = 0;                    // current top of the arena
  uint64_t high_ = 0;

  uint64_t alloc(uint64_t bytes) {
    bytes = align_up(std::max<uint64_t>(bytes, 1));
    auto best = free_.end();
    for (auto it = free_.begin(); it != free_.end(); ++it)
      if (it->second >= bytes && (best == free_.end() || it->second < best->second)) best = it;
    if (best != free_.end()) {
      uint64_t off = best->first, sz = best->second;
      free_.erase(best);
      if (sz > bytes) free_[off + bytes] = sz - bytes;
      return off;
    }
    // grow: extend a free block that touches the top, if any
    uint64_t off = end_;
    if (!free_.empty()) {
      auto last = std::prev(free_.end());
      if (last->first + last->second == end_) { off = last->first; free_.erase(last); }
    }
    end_ = off + bytes;
    high_ = std::max(high_, end_);
    return off;
  }
  void release(uint64_t off, uint64_t bytes) {
    bytes = align_up(std::max<uint64_t>(bytes, 1));
    auto it = free_.emplace(off, bytes).first;
    auto nx = std::next(it);
    if (nx != free_.end() && it->first + it->second == nx->first) { it->second += nx->second; free_.erase(nx); }
    if (it != free_.begin()) {
      auto pv = std::prev(it);
      if (pv->first + pv->second == it->first) { pv->second += it->second; free_.erase(it); it = pv; }
    }
    if (it->first + it->second == end_) { end_ = it->first; free_.erase(it); }
  }
};

// A tensor to be placed: bytes (aligned), the first and last step it is alive at, and where it goes.
struct Span { uint64_t bytes; int first, last; uint64_t offset; };

// Places tensors, given in the order of their first step, so that no two that are alive at the same step overlap; returns the
// arena's size.  First in the order of the steps, each at the tightest hole.  Where that leaves holes that a later tensor does
// not fit (a workspace between kept tensors), also one tensor after the other, each at the lowest offset that is free while it is
// alive, in these orders: the largest first; those alive at the fullest step ahead of the others; those ahead with most bytes
// times steps; the order of the steps; the longest alive first; each also with the tensor that ended up on top ahead of all others,
// seven times.  The smallest result is kept; the search ends at one of `enough` bytes.  longer: also the largest first with every
// size weighted by a fixed number between a half and one and a half, 395 times over.  most_alive (or null): what no placement can
// go below.
uint64_t place(std::vector<Span>& spans, int n_steps, uint64_t enough, bool longer = false, uint64_t* most_alive = nullptr) {
  const int n = (int)spans.size();
  std::vector<std::vector<int>> dies(n_steps);
  for (int i = 0; i < n; ++i) dies[spans[i].last].push_back(i);
  FreeList fl;
  uint64_t alive = 0, least = 0;  // least: what is alive at the fullest step
  int fullest = 0;
  for (int t = 0, next = 0; t < n_steps; ++t) {
    for (; next < n && spans[next].first == t; ++next) {
      spans[next].offset = fl.alloc(spans[next].bytes);
      alive += spans[next].bytes;
    }
    if (alive > least) { least = alive; fullest = t; }
    for (int i : dies[t]) { fl.release(spans[i].offset, spans[i].bytes); alive -= spans[i].bytes; }
  }
  if (most_alive) *most_alive = least;
  uint64_t best = fl.high_;
  enough = std::max(enough, least);
  std::vector<int> order(n), placed;  // placed: by offset
  std::vector<uint64_t> at(n);
  for (int way = 0; way < (longer ? 400 : 5) && best > enough; ++way) {
    auto ahead = [&](int i) { return way == 1 && spans[i].first <= fullest && spans[i].last >= fullest; };
    auto weight = [&](int i) -> uint64_t {
      const uint64_t steps = (uint64_t)(spans[i].last - spans[i].first + 1);
      if (way < 5) return way == 2 ? spans[i].bytes * steps : way == 4 ? steps : spans[i].bytes;
      const uint32_t h = ((uint32_t)i * 2654435761u + (uint32_t)way * 40503u) * 2246822519u;
      return spans[i].bytes / 256 * (128 + (h >> 24));
    };
    for (int i = 0; i < n; ++i) order[i] = i;
    if (way != 3)
      std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return ahead(a) != ahead(b) ? ahead(a) : weight(a) > weight(b); });
    for (int tries = 0; tries < 8 && best > enough; ++tries) {
      uint64_t high = 0;
      int top = 0;  // its place in the order
      placed.clear();
      for (int o = 0; o < n; ++o) {
        const int i = order[o];
        const Span& s = spans[i];
        uint64_t off = 0;
        for (int j : placed) {
          const Span& q = spans[j];
          if (q.last < s.first || s.last < q.first) continue;
          if (at[j] >= off + s.bytes) break;
          off = std::max(off, at[j] + q.bytes);
        }
        at[i] = off;
        if (off + s.bytes > high) { high = off + s.bytes; top = o; }
        if (high >= best) break;
        placed.insert(std::upper_bound(placed.begin(), placed.end(), off, [&](uint64_t v, int j) { return v < at[j]; }), i);
      }
      if (high < best) {
        best = high;
        for (int i = 0; i < n; ++i) spans[i].offset = at[i];
      }
      std::rotate(order.begin(), order.begin() + top, order.begin() + top + 1);
    }
  }
  return best;
}

uint64_t aligned(uint64_t bytes) { return align_up(std::max<uint64_t>(bytes, 1)); }

bool is_fwd_kind(SKind k) { return k <= S_HEAD_FWD; }

bool has_side_effect(SKind k) {
  // writes parameter gradients, the loss, or BN running statistics
  return k == S_HEAD_FWD || k == S_HEAD_BWD || k == S_BN_BWD || k == S_BIAS_GRAD || k == S_WGRAD || k == S_BN_STATS ||
         k == S_CONV_BWD;
}

struct Scheduler {
  Plan& p;
  std::vector<int> cur, grad;  // [LTensor] -> Inst id
  std::vector<int> stat_ws;    // [LTensor of a conv output] -> Inst id of the channel sums its forward kernel wrote
  std::vector<int> bn_apply_of;  // [LTensor] -> the F_BN_APPLY operation that produces it, or -1
  std::vector<char> rebuilt;     // [LTensor] backward has already rebuilt it (storage mode 1)
  std::vector<int> readers;      // [LTensor] -> number of forward operations that read it
  std::vector<int> via_pool;     // [LTensor] -> Inst id of the gradient of the max-pool output behind it, when the
                                 //              pool's backward is left to the BatchNorm backward in front of it
  std::vector<int> gmask;        // [LTensor] -> Inst id of a ReLU bit mask that grad[t] still has to be multiplied by
                                 //              (the gradient through a skip connection is not written out: its
                                 //              reader applies the mask to the block output's gradient itself), or -1
  std::vector<char> per_image;   // [LTensor] -> grad[t] (or image_grad[t]) holds one value per image and channel
  std::vector<int> fused_bwd;    // [FOp of a convolution] -> entry of the BatchNorm-backward sums that its S_CONV_BWD goes on from, or -1
  std::vector<int> bn_sums, bn_sum_rows;  // [LTensor] -> Inst id of the BatchNorm-backward sums that came with grad[t], or -1, and their rows
  std::vector<int> image_grad;   // [LTensor] -> Inst id of the gradient per image of the global average pool's input, or -1
  explicit Scheduler(Plan& pl)
      : p(pl), cur(pl.tensors.size(), -1), grad(pl.tensors.size(), -1), stat_ws(pl.tensors.size(), -1),
        bn_apply_of(pl.tensors.size(), -1), rebuilt(pl.tensors.size(), 0), readers(pl.tensors.size(), 0),
        via_pool(pl.tensors.size(), -1), gmask(pl.tensors.size(), -1), per_image(pl.tensors.size(), 0),
        fused_bwd(pl.fops.size(), -1), bn_sums(pl.tensors.size(), -1), bn_sum_rows(pl.tensors.size(), 0), image_grad(pl.tensors.size(), -1) {
    for (size_t fi = 0; fi < pl.fops.size(); ++fi) {
      const FOp& f = pl.fops[fi];
      if (f.kind == F_BN_APPLY) bn_apply_of[f.out] = (int)fi;
      if (f.x >= 0) ++readers[f.x];
      if (f.skip >= 0) ++readers[f.skip];
    }
  }

  // Is forward operation fi a 2x2 max-pool whose backward the BatchNorm backward in front of it does as well?  The
  // activation between them must be read by nothing else; the rule looks at the network only (never at the segments),
  // so the sums of that BatchNorm backward are added in the same order for every k.
  bool pool_bwd_fused(int fi) const {
    if (fi < 1) return false;
    const FOp& pool = p.fops[fi];
    const FOp& ap = p.fops[fi - 1];
    if (pool.kind != F_POOL || ap.kind != F_BN_APPLY || pool.x != ap.out || ap.skip >= 0) return false;
    return ap.P % 2 == 0 && ap.Q % 2 == 0 && readers[ap.out] == 1 && p.tensors[ap.out].needs_grad;
  }

  int new_inst(int logical, uint64_t bytes, bool fwd_value) {
    Inst i; i.logical = logical; i.bytes = bytes; i.fwd_value = fwd_value;
    p.insts.push_back(i);
    return (int)p.insts.size() - 1;
  }
  // the sums of a BatchNorm backward over `rows` row blocks, and their means behind them
  int sums_inst(int rows, int C) { return new_inst(-1, ((uint64_t)rows * 2 + 2) * C * 4, false); }
  bool sums_ok(int unit, int which) const { return !p.separate && unit >= 0 && unit < (int)p.unit_sums.size() && (p.unit_sums[unit] & which); }
  int value_inst(int t) { return cur[t] = new_inst(t, p.tensors[t].bytes, true); }
  int grad_inst(int t) { return new_inst(t, p.tensors[t].bytes, false); }

  SOp& push(SKind k, int fop, int phase, int seg) {
    SOp s; s.kind = k; s.fop = fop; s.phase = phase; s.seg = seg;
    p.sched.push_back(s);
    return p.sched.back();
  }

  // Is forward operation fi a 2x2 max-pool that the BatchNorm apply right in front of it computes as well?  Both must
  // lie in segment `seg` (a pool that opens a segment is replayed from the segment's kept input), the apply must add
  // no skip connection, and the map must have even sides.
  bool pool_fused(int fi, int seg) const {
    if (fi < 1 || fi >= (int)p.fops.size()) return false;
    const FOp& pool = p.fops[fi];
    const FOp& ap = p.fops[fi - 1];
    if (pool.kind != F_POOL || ap.kind != F_BN_APPLY || pool.x != ap.out || ap.skip >= 0) return false;
    if (ap.P % 2 != 0 || ap.Q % 2 != 0) return false;
    return ap.unit >= p.seg_begin[seg] && pool.unit < p.seg_begin[seg + 1];
  }

  // Is forward operation fi a global average pool that does the BatchNorm apply in front of it as well?  Nothing else reads that
  // one's output, both lie in segment `seg`, whole groups of channels, and backward has the ReLU decisions of an output with
  // a skip connection as bits.  (storage mode 2 keeps every activation)
  bool gap_fused(int fi, int seg) const {
    if (fi < 1 || fi >= (int)p.fops.size() || p.cfg.storage_mode == 2 || p.separate) return false;
    const FOp& head = p.fops[fi];
    const FOp& ap = p.fops[fi - 1];
    if (head.kind != F_HEAD || !head.gap || ap.kind != F_BN_APPLY || head.x != ap.out || ap.fold || readers[ap.out] != 1) return false;
    if (ap.C % (16 / p.esize) != 0 || (ap.skip >= 0 && ap.mask < 0)) return false;
    return ap.unit >= p.seg_begin[seg] && head.unit < p.seg_begin[seg + 1];
  }

  // Is z, the output of convolution f or the input of the BatchNorm apply f, not written in this phase?  (In storage mode 2 a
  // projection shortcut's BatchNorm has an apply pass of its own, which reads it.)
  bool unwritten(const FOp& f, int phase) const {
    return f.again && !p.separate && p.cfg.storage_mode != 2 && !(p.z_written && phase == PH_FWD_NOSAVE);
  }
  // What the z of a FOp::again convolution is made again from: its input tensor t or, with its statistics, the z of the BatchNorm
  // that t is the output of -- whichever is alive anyway where the pass keeps something for backward.
  void again_source(int t, int unit, int phase, int seg, int* src) const {
    const int fa = bn_apply_of[t];
    if (fa >= 0 && (p.fops[fa].unit == unit ||
                    (p.cfg.storage_mode == 1 && phase != PH_FWD_NOSAVE && p.fops[fa].skip < 0 && p.fops[fa].unit >= p.seg_begin[seg]))) {
      src[0] = cur[p.fops[fa].x]; src[1] = cur[p.fops[fa].stats];
    } else {
      src[0] = cur[t];
    }
  }

  void emit_fop_forward(int fi, int phase, int seg) {
    const FOp& f = p.fops[fi];
    switch (f.kind) {
      case F_CAST_IN: { SOp& s = push(S_CAST_IN, fi, phase, seg); s.out[0] = value_inst(f.out); break; }
      case F_CONV: {
        SOp& s = push(S_CONV_FWD, fi, phase, seg);
        s.in[0] = cur[f.x];
        if (f.fold_src >= 0) { s.in[0] = cur[p.fops[f.fold_src].x]; s.in[1] = cur[p.fops[f.fold_src].stats]; }
        s.again = unwritten(f, phase);
        s.out[0] = value_inst(f.out);
        if (f.fwd_splits > 1) s.out[1] = new_inst(-1, (uint64_t)f.fwd_splits * f.N * f.P * f.Q * f.K * 4, false);
        if (f.stat_blocks > 0 && phase != PH_REPLAY) {  // per-block channel sums for the BatchNorm that follows
          s.out[2] = new_inst(-1, (uint64_t)(f.stat_blocks + f.stat_fold) * 2 * f.K * 4, false);
          stat_ws[f.out] = s.out[2];
        }
        break;
      }
      case F_BN_STATS: {
        if (phase == PH_REPLAY) break;  // the statistics of the first forward pass are kept and reused
        SOp& s = push(S_BN_STATS, fi, phase, seg);
        s.in[0] = cur[f.x]; s.out[0] = value_inst(f.stats);
        if (f.stat_blocks > 0) s.in[1] = stat_ws[f.x];  // sums come from the convolution: only the finishing kernel runs
        else s.out[1] = new_inst(-1, (uint64_t)f.red_blocks * 2 * f.C * 4, false);
        break;
      }
      case F_BN_APPLY: {
        if (f.fold) break;  // done by the operation that reads it
        if (gap_fused(fi + 1, seg)) break;  // likewise
        SOp& s = push(S_BN_APPLY, fi, phase, seg);
        s.in[0] = cur[f.x]; s.in[1] = cur[f.stats]; s.in[2] = f.skip >= 0 ? cur[f.skip] : -1;
        if (f.fold_skip >= 0) { s.in[2] = cur[p.fops[f.fold_skip].x]; s.in[3] = cur[p.fops[f.fold_skip].stats]; }
        if (unwritten(f, phase)) {
          s.again = true;
          again_source(p.fops[fi - 2].x, f.unit, phase, seg, s.src);
          if (f.again_skip >= 0) again_source(p.fops[f.again_skip - 2].x, f.unit, phase, seg, s.src + 2);
        }
        s.out[0] = value_inst(f.out);
        if (pool_fused(fi + 1, seg)) s.out[1] = value_inst(p.fops[fi + 1].out);  // the same kernel also pools
        if (f.mask >= 0) s.out[2] = value_inst(f.mask);
        break;
      }
      case F_POOL: {
        if (pool_fused(fi, seg)) break;  // done by the BatchNorm apply in front of it
        SOp& s = push(S_POOL_FWD, fi, phase, seg); s.in[0] = cur[f.x]; s.out[0] = value_inst(f.out);
        break;
      }
      case F_HEAD: {
        SOp& s = push(S_HEAD_FWD, fi, phase, seg);
        s.in[0] = cur[f.x];
        if (gap_fused(fi, seg)) {
          const FOp& ap = p.fops[fi - 1];
          s.variant = 1;
          s.in[0] = cur[ap.x]; s.in[1] = cur[ap.stats]; s.in[2] = ap.skip >= 0 ? cur[ap.skip] : -1;
          if (ap.fold_skip >= 0) { s.in[2] = cur[p.fops[ap.fold_skip].x]; s.in[3] = cur[p.fops[ap.fold_skip].stats]; }
          if (ap.mask >= 0) s.out[5] = value_inst(ap.mask);
        }
        s.out[0] = value_inst(f.aux[0]); s.out[1] = value_inst(f.aux[1]);
        s.out[2] = value_inst(f.aux[2]); s.out[3] = value_inst(f.out);
        if (f.head_ws > 0 && !f.head_ws_in_x) s.out[4] = new_inst(-1, (uint64_t)f.head_ws * 4, false);
        break;
      }
    }
  }

  // The instance of forward tensor t that a backward operation of segment `seg` reads.  Storage mode 1: an
  // activation A = ReLU(BN(Z)) without a skip connection, produced inside this segment, is not kept from the forward
  // pass; the first backward operation that needs it has it rebuilt from Z and the kept statistics by the same
  // elementwise kernel (hence the same bits), as a transient of the backward pass.
  int backward_input(int t, int seg) {
    const int fa = bn_apply_of[t];
    if (p.cfg.storage_mode != 1 || fa < 0 || rebuilt[t]) return cur[t];
    const FOp& f = p.fops[fa];
    if (f.skip >= 0 || f.unit < p.seg_begin[seg] || f.unit >= p.seg_begin[seg + 1]) return cur[t];
    SOp& s = push(S_BN_APPLY, fa, PH_BWD, seg);
    s.in[0] = cur[f.x]; s.in[1] = cur[f.stats];
    s.out[0] = cur[t] = new_inst(t, p.tensors[t].bytes, false);
    rebuilt[t] = 1;
    return cur[t];
  }

  // May the reader of the gradient through operation fi's skip connection take it as (gradient of the block output,
  // ReLU bit mask) instead of a tensor of its own?  A BatchNorm backward (projection shortcut) always can; a
  // convolution's data gradient can where it runs on the matrix cores (their shared epilogue applies the mask).
  bool masked_skip_grad_ok(int fi) const {
    const FOp& f = p.fops[fi];
    if (f.mask < 0 || f.skip < 0) return false;
    if (bn_apply_of[f.skip] >= 0 && p.fops[bn_apply_of[f.skip]].unit == f.unit) return true;
    for (int j = p.unit_first_fop[f.unit]; j < p.unit_last_fop[f.unit]; ++j)
      if (p.fops[j].kind == F_CONV && p.fops[j].x == f.skip) return p.fops[j].dgrad_algo == ALGO_MFMA;
    return false;
  }

  // Does the first convolution of operation fi's block, which reads its identity skip connection, add a gradient per image?
  bool image_addend_ok(int fi) const {
    const FOp& f = p.fops[fi];
    for (int j = p.unit_first_fop[f.unit]; j < p.unit_last_fop[f.unit]; ++j)
      if (p.fops[j].kind == F_CONV && p.fops[j].x == f.skip) return p.fops[j].image_addend != 0 && !p.separate;
    return false;
  }

  // May the kernel that writes the gradient of convolution fi's input produce the sums of the BatchNorm backward in front of it?
  // Inside a unit only, whatever the segments are: a BatchNorm without a skip connection, which nothing else reads.
  int summed_apply(int fi) const {
    const FOp& f = p.fops[fi];
    const int ap = bn_apply_of[f.x];
    if (ap < 0 || grad[f.x] >= 0 || readers[f.x] != 1 || !sums_ok(f.unit, SUMS_INSIDE)) return -1;
    const FOp& b = p.fops[ap];
    return b.unit == f.unit && b.skip < 0 && b.mask < 0 ? ap : -1;
  }

  // The projection shortcut's BatchNorm apply whose output operation fi adds, or -1.
  int projection_of(int fi) const {
    const FOp& f = p.fops[fi];
    if (f.skip < 0) return -1;
    const int b = bn_apply_of[f.skip];
    return b >= 0 && p.fops[b].unit == f.unit ? b : -1;
  }

  // May the BatchNorm backward of operation fi, whose output only a global average pool reads, take the gradient
  // per image?  Its kernels do in whole groups of 16 / esize channels and count rows in 32 bits; a skip connection's gradient
  // must not need a tensor written from it.
  bool per_image_ok(int fi) const {
    const FOp& f = p.fops[fi];
    if (f.C % (16 / p.esize) != 0 || (int64_t)f.N * f.P * f.Q >= (int64_t)1 << 32) return false;
    return f.skip < 0 || masked_skip_grad_ok(fi);
  }

  // The convolution that the BatchNorm apply operation fi belongs to, if its S_CONV_BWD does that one's backward pass as well:
  // a gradient of the skip connection must not need a tensor written from it, the ReLU decisions must not come from the
  // output, and nothing may have been added to the gradient of the convolution's input yet.
  int fused_conv_of(int fi) const {
    const FOp& f = p.fops[fi];
    if (fi < 2 || p.separate || p.fops[fi - 2].kind != F_CONV || p.fops[fi - 2].bwd_splits == 0 || p.fops[fi - 2].out != f.x) return -1;
    if (f.skip >= 0 && (f.mask < 0 || !masked_skip_grad_ok(fi))) return -1;
    if (!p.tensors[p.fops[fi - 2].x].needs_grad || grad[p.fops[fi - 2].x] >= 0) return -1;
    return fi - 2;
  }

  bool emit_fop_backward(int fi, int seg) {
    const FOp& f = p.fops[fi];
    switch (f.kind) {
      case F_CAST_IN: case F_BN_STATS: return true;
      case F_HEAD: {
        SOp& s = push(S_HEAD_BWD, fi, PH_BWD, seg);
        s.in[0] = cur[f.aux[0]]; s.in[1] = cur[f.aux[2]];
        if (p.tensors[f.x].needs_grad) {
          const int ap = bn_apply_of[f.x];
          bool whole = true;  // the gradient as a whole tensor
          if (f.gap && ap >= 0 && readers[f.x] == 1 && per_image_ok(ap)) {
            s.out[2] = image_grad[f.x] = new_inst(-1, (uint64_t)f.N * f.C * p.esize, false);
            // the data gradient of an identity shortcut's first convolution may have to add it as a tensor
            const int skip = p.fops[ap].skip;
            whole = skip >= 0 && projection_of(ap) < 0 && p.tensors[skip].needs_grad && !image_addend_ok(ap);
          }
          if (whole) { s.out[0] = grad_inst(f.x); grad[f.x] = s.out[0]; }
        }
        s.out[1] = new_inst(-1, (uint64_t)f.N * f.feat_dim * 4, false);
        return true;
      }
      case F_BN_APPLY: {
        int gin = grad[f.out], variant = 0;
        bool image = per_image[f.out] != 0;
        const int whole = gin;  // (the skip connection's reader of an identity shortcut)
        if (image_grad[f.out] >= 0) { gin = image_grad[f.out]; image = true; }
        if (gin < 0 && via_pool[f.out] >= 0) { gin = via_pool[f.out]; variant = 1; }  // through the pool behind it
        if (gin < 0) { p.error = "internal: BN output has no gradient"; return false; }
        if (f.skip >= 0 && !f.relu) { p.error = "skip connection without ReLU is not supported"; return false; }
        const int gin_mask = gmask[f.out];  // the incoming gradient still wants a mask (projection shortcut's BatchNorm)
        const bool again = f.again && !p.separate;
        SOp& s = push(S_BN_BWD, fi, PH_BWD, seg);
        const size_t at = p.sched.size() - 1;
        s.variant = variant;
        s.per_image = image;
        s.again = again;
        s.in[0] = gin; s.in[1] = cur[f.x]; s.in[2] = cur[f.stats];
        s.in[3] = (f.skip >= 0) ? cur[f.out] : -1;
        if (gin_mask >= 0) {
          if (f.skip >= 0 || variant != 0) { p.error = "internal: masked gradient into a BatchNorm with a skip connection"; return false; }
          s.in[3] = gin_mask; s.variant = 2;
        } else if (f.mask >= 0) {
          s.in[3] = cur[f.mask]; s.variant = 2;
        }
        const int conv = variant == 0 ? fused_conv_of(fi) : -1;
        if (conv >= 0) fused_bwd[conv] = (int)p.sched.size() - 1;
        else { s.out[0] = grad_inst(f.x); grad[f.x] = s.out[0]; gmask[f.x] = -1; }
        if (f.skip >= 0 && p.tensors[f.skip].needs_grad) {
          if (grad[f.skip] >= 0) { p.error = "internal: skip gradient must be the first contribution"; return false; }
          if (masked_skip_grad_ok(fi)) {  // nothing written
            const bool vec = image && (projection_of(fi) >= 0 || image_addend_ok(fi));
            grad[f.skip] = vec ? gin : whole; per_image[f.skip] = vec; gmask[f.skip] = cur[f.mask];
          }
          else { s.out[1] = grad_inst(f.skip); grad[f.skip] = s.out[1]; gmask[f.skip] = -1; }
        }
        SOp& b = p.sched[at];
        if (again && (conv < 0 || b.variant != 2 || image)) { p.error = "internal: z is made again for a backward pass that reads it"; return false; }
        b.rows = again ? p.fops[fi - 2].again_rows : f.red_blocks;
        // the BatchNorm of a projection shortcut has the same gradient and decisions (masked_skip_grad_ok): its sums in the same pass
        const int shortcut = f.skip >= 0 && b.variant == 2 ? projection_of(fi) : -1;
        if (shortcut >= 0 && gmask[f.skip] >= 0 && grad[f.skip] == b.in[0] && f.C % (16 / p.esize) == 0 && sums_ok(f.unit, SUMS_SHORTCUT)) {
          const FOp& q = p.fops[shortcut];
          b.in[5] = cur[q.x]; b.in[6] = cur[q.stats];
          b.out[3] = bn_sums[f.skip] = sums_inst(b.rows, f.C);
          bn_sum_rows[f.skip] = b.rows;
          if (again) again_source(p.fops[shortcut - 2].x, f.unit, PH_BWD, seg, b.src + 2);
        }
        if (bn_sums[f.out] >= 0 && variant == 0) { b.in[4] = bn_sums[f.out]; b.rows = bn_sum_rows[f.out]; }
        else b.out[2] = sums_inst(b.rows, f.C);
        if (again && b.in[4] < 0) again_source(p.fops[fi - 2].x, f.unit, PH_BWD, seg, b.src);
        return true;
      }
      case F_CONV: {
        if (fused_bwd[fi] >= 0) {
          // (with the sums of the BatchNorm in front it reads that one's z in every storage mode)
          const int sums_for = summed_apply(fi) >= 0 && p.fops[summed_apply(fi)].relu ? summed_apply(fi) : -1;
          const int from_z = f.fold_src >= 0 ? f.fold_src : sums_for;
          const int xin = from_z >= 0 ? cur[p.fops[from_z].x] : backward_input(f.x, seg);
          const SOp sums = p.sched[fused_bwd[fi]];
          SOp& s = push(S_CONV_BWD, fi, PH_BWD, seg);
          for (int i = 0; i < 4; ++i) s.in[i] = sums.in[i];
          s.variant = sums.variant; s.per_image = sums.per_image;
          s.in[4] = sums.in[4] >= 0 ? sums.in[4] : sums.out[2];
          s.in[5] = xin;
          if (from_z >= 0) s.in[6] = cur[p.fops[from_z].stats];
          s.out[0] = grad_inst(f.x); grad[f.x] = s.out[0]; gmask[f.x] = -1;
          s.rows = sums.rows;
          if (f.bwd_splits > 1) s.out[1] = new_inst(-1, (uint64_t)f.bwd_splits * f.K * f.R * f.S * f.C * 4, false);
          if (sums_for >= 0) {
            s.out[2] = bn_sums[f.x] = sums_inst(f.bwd_splits, f.C);
            bn_sum_rows[f.x] = f.bwd_splits;
          }
          return true;
        }
        int g = grad[f.out];
        if (g < 0) { p.error = "internal: conv output has no gradient"; return false; }
        const bool in_place = !f.has_bn && f.relu && f.has_bias && !p.separate;
        if (!f.has_bn && f.relu && !in_place) {
          SOp& s = push(S_RELU_BWD, fi, PH_BWD, seg);
          s.in[0] = g; s.in[1] = cur[f.out];
          s.out[0] = grad_inst(f.out); g = s.out[0];
        }
        if (f.has_bias) {
          SOp& s = push(S_BIAS_GRAD, fi, PH_BWD, seg);
          s.in[0] = g;
          if (in_place) s.in[1] = cur[f.out];  // (and the ReLU, in place: nothing else reads this gradient)
          s.out[0] = new_inst(-1, (uint64_t)f.red_blocks * 2 * f.K * 4, false);
        }
        {
          const int xin = f.fold_src >= 0 ? cur[p.fops[f.fold_src].x] : backward_input(f.x, seg);
          SOp& s = push(S_WGRAD, fi, PH_BWD, seg);
          s.in[0] = xin; s.in[1] = g;
          if (f.fold_src >= 0) s.in[2] = cur[p.fops[f.fold_src].stats];
          if (f.wgrad_splits > 1)
            s.out[0] = new_inst(-1, (uint64_t)f.wgrad_splits * f.K * f.R * f.S * f.C * 4, false);
        }
        if (p.tensors[f.x].needs_grad) {
          SOp& s = push(S_DGRAD, fi, PH_BWD, seg);
          s.in[0] = g; s.in[1] = grad[f.x]; s.in[2] = grad[f.x] >= 0 ? gmask[f.x] : -1;
          s.per_image = grad[f.x] >= 0 && per_image[f.x];
          const int ap = f.dgrad_sums > 0 ? summed_apply(fi) : -1;
          if (ap >= 0) {
            s.in[3] = cur[p.fops[ap].x]; s.in[4] = cur[p.fops[ap].stats]; s.variant = p.fops[ap].relu;
            s.out[2] = bn_sums[f.x] = sums_inst(f.dgrad_sums, f.C);
            bn_sum_rows[f.x] = f.dgrad_sums;
          }
          s.out[0] = grad_inst(f.x); grad[f.x] = s.out[0]; gmask[f.x] = -1; per_image[f.x] = 0;
          if (f.dgrad_splits > 1) s.out[1] = new_inst(-1, (uint64_t)f.dgrad_splits * f.N * f.H * f.W * f.C * 4, false);
        }
        return true;
      }
      case F_POOL: {
        if (!p.tensors[f.x].needs_grad) return true;
        if (grad[f.out] < 0) { p.error = "internal: pool output has no gradient"; return false; }
        if (grad[f.x] >= 0) { p.error = "internal: pool input already has a gradient"; return false; }
        if (pool_bwd_fused(fi)) { via_pool[f.x] = grad[f.out]; return true; }
        const int xin = backward_input(f.x, seg);
        SOp& s = push(S_POOL_BWD, fi, PH_BWD, seg);
        s.in[0] = xin; s.in[1] = grad[f.out];
        s.out[0] = grad_inst(f.x); grad[f.x] = s.out[0];
        return true;
      }
    }
    return true;
  }

  bool run() {
    const int k = (int)p.seg_begin.size() - 1;
    p.insts.clear(); p.sched.clear();
    emit_fop_forward(0, k == 1 ? PH_FWD_LAST : PH_FWD_NOSAVE, 0);
    auto forward_seg = [&](int j, int phase) {
      for (int u = p.seg_begin[j]; u < p.seg_begin[j + 1]; ++u)
        for (int fi = p.unit_first_fop[u]; fi < p.unit_last_fop[u]; ++fi) emit_fop_forward(fi, phase, j);
    };
    for (int j = 0; j < k - 1; ++j) forward_seg(j, PH_FWD_NOSAVE);
    forward_seg(k - 1, PH_FWD_LAST);
    for (int j = k - 1; j >= 0; --j) {
      if (j < k - 1) forward_seg(j, PH_REPLAY);
      for (int u = p.seg_begin[j + 1] - 1; u >= p.seg_begin[j]; --u)
        for (int fi = p.unit_last_fop[u] - 1; fi >= p.unit_first_fop[u]; --fi)
          if (!emit_fop_backward(fi, j)) return false;
    }
    return true;
  }
};

}  // namespace

int launches_of(const SOp& op, const FOp& f) {
  switch (op.kind) {
    case S_BN_STATS: return f.stat_blocks > 0 ? (f.stat_fold > 0 ? 2 : 1) : 2;
    case S_HEAD_FWD: return (f.head_ws > 0 ? 5 : 4) - (f.head_one ? 1 : 0);
    case S_HEAD_BWD:  // the weight gradient; the feature gradient and where it goes: the whole map, one value per image
      return 1 + (op.out[0] >= 0 || op.out[2] >= 0) + (op.out[0] >= 0) + (op.out[2] >= 0);
    case S_BN_BWD: return (op.out[0] >= 0 ? 3 : 2) - (op.in[4] >= 0 ? 1 : 0);
    case S_BIAS_GRAD: return 2;
    case S_WGRAD: return f.wgrad_splits > 1 ? 2 : 1;
    case S_CONV_BWD: return f.bwd_splits > 1 ? 2 : 1;
    case S_CONV_FWD: return op.again && op.phase == PH_REPLAY ? 0 : f.fwd_splits > 1 ? 2 : 1;
    case S_DGRAD: return f.dgrad_splits > 1 ? 2 : 1;
    default: return 1;
  }
}

bool build_graph(Plan& p) {
  p.tensors.clear(); p.fops.clear(); p.n_params = 0; p.n_running = 0;
  const optorch_seq_config_t& c = p.cfg;
  if (c.batch < 1 || c.height < 1 || c.width < 1 || c.channels < 1 || c.num_classes < 2) {
    p.error = "batch, height, width, channels must be >= 1 and num_classes >= 2";
    return false;
  }
  if (c.precision < 0 || c.precision > 2) { p.error = "precision must be 0 (fp32), 1 (bf16) or 2 (fp16)"; return false; }
  if (c.storage_mode < 0 || c.storage_mode > 2) { p.error = "storage_mode must be 0, 1 or 2"; return false; }
  if ((int64_t)c.batch * c.height * c.width * 2048 > (int64_t)1 << 40) { p.error = "batch too large"; return false; }
  Builder b(p);
  return b.run();
}

// the schedule and the lifetimes of its tensors
static bool schedule_operations(Plan& p) {
  Scheduler s(p);
  if (!s.run()) return false;
  const int n = (int)p.sched.size();
  // dead-operation elimination (a replayed operation whose result nobody reads is not run)
  std::vector<int> uses(p.insts.size(), 0);
  for (int i = n - 1; i >= 0; --i) {
    SOp& op = p.sched[i];
    bool live = has_side_effect(op.kind);
    for (int o : op.out) if (o >= 0 && uses[o] > 0) live = true;
    op.live = live;
    if (live && op.kind == S_BN_APPLY && op.out[1] >= 0) {  // apply + pool: an output nobody reads is not written
      if (uses[op.out[0]] == 0) op.out[0] = -1;
      else if (uses[op.out[1]] == 0) op.out[1] = -1;
    }
    if (live && op.kind == S_BN_APPLY && op.out[2] >= 0 && uses[op.out[2]] == 0) op.out[2] = -1;  // the mask likewise
    if (live) {
      for (int x : op.in) if (x >= 0) ++uses[x];
      for (int x : op.src) if (x >= 0) ++uses[x];
    }
  }
  // lifetimes
  for (Inst& t : p.insts) { t.def_op = -1; t.last_use = -1; t.held = false; t.allocated = false; }
  for (int i = 0; i < n; ++i) {
    const SOp& op = p.sched[i];
    if (!op.live) continue;
    for (int o : op.out) if (o >= 0) { p.insts[o].def_op = i; p.insts[o].last_use = std::max(p.insts[o].last_use, i); }
    for (int i0 = 0; i0 < 11; ++i0) {
      const int x = i0 < 7 ? op.in[i0] : op.src[i0 - 7];
      if (x < 0) continue;
      Inst& t = p.insts[x];
      if (t.def_op < 0) { p.error = "internal: operation reads a tensor that was never produced"; return false; }
      t.last_use = std::max(t.last_use, i);
      const SOp& d = p.sched[t.def_op];
      if (t.fwd_value && (op.phase == PH_BWD || op.phase != d.phase || op.seg != d.seg)) t.held = true;
    }
  }
  return true;
}

// The most bytes alive at a step if passes that keep nothing wrote every z (an arena of such a plan is no smaller); ~0 if they do.
static uint64_t alive_with_z_written(const Plan& p) {
  std::vector<int> last(p.insts.size(), -1);
  bool differs = false;
  for (int i = 0; i < (int)p.sched.size(); ++i) {
    const SOp& op = p.sched[i];
    if (!op.live) continue;
    for (int o : op.out) if (o >= 0) last[o] = i;
    for (int x : op.in) if (x >= 0) last[x] = i;
    if (op.phase == PH_FWD_NOSAVE && op.kind == S_BN_APPLY) differs = differs || op.again;
    else for (int x : op.src) if (x >= 0) last[x] = i;
  }
  if (!differs) return ~0ull;
  std::vector<int64_t> born(p.sched.size() + 1, 0);
  for (size_t t = 0; t < p.insts.size(); ++t)
    if (last[t] >= 0) {
      born[p.insts[t].def_op] += (int64_t)aligned(p.insts[t].bytes);
      born[last[t] + 1] -= (int64_t)aligned(p.insts[t].bytes);
    }
  int64_t alive = 0, most = 0;
  for (int64_t b : born) most = std::max(most, alive += b);
  return (uint64_t)most;
}

bool build_schedule(Plan& p, uint64_t enough) {
  if (!schedule_operations(p)) return false;
  const int n = (int)p.sched.size();
  // peak figures, by walking the schedule, and arena offsets
  std::vector<std::vector<int>> dies(n);
  for (size_t t = 0; t < p.insts.size(); ++t)
    if (p.insts[t].def_op >= 0) dies[p.insts[t].last_use].push_back((int)t);
  std::vector<Span> spans;
  std::vector<int> span_inst;
  uint64_t live_b = 0, held_b = 0;
  p.peak_saved_bytes = p.peak_live_bytes = 0;
  p.n_launches = p.n_replay_launches = 0;
  for (int i = 0; i < n; ++i) {
    const SOp& op = p.sched[i];
    if (!op.live) continue;
    int nl = launches_of(op, p.fops[op.fop]);
    p.n_launches += nl;
    if (op.phase == PH_REPLAY) p.n_replay_launches += nl;
    for (int o : op.out) if (o >= 0) {
      Inst& t = p.insts[o];
      t.allocated = true;
      spans.push_back(Span{aligned(t.bytes), i, t.last_use, 0});
      span_inst.push_back(o);
      live_b += t.bytes;
      if (t.held) held_b += t.bytes;
    }
    p.peak_live_bytes = std::max(p.peak_live_bytes, live_b);
    p.peak_saved_bytes = std::max(p.peak_saved_bytes, held_b);
    for (int t : dies[i]) {
      live_b -= p.insts[t].bytes;
      if (p.insts[t].held) held_b -= p.insts[t].bytes;
    }
  }
  uint64_t most_alive = 0;
  p.arena_bytes = place(spans, n, enough, false, &most_alive);
  if (!p.separate && p.arena_bytes > std::max(enough, most_alive)) {
    // merged passes hold no more at any step, but may be placed worse: then a longer search, so that what a budget allowed without
    // them it allows with them (of 40 000 random networks 33 are still larger, by up to 2 % or some KB)
    if (p.separate_arena == 0) {
      Plan q = p;
      q.separate = true;
      p.separate_arena = build_schedule(q) ? q.arena_bytes : ~0ull;
    }
    if (p.separate_arena < p.arena_bytes) p.arena_bytes = place(spans, n, std::max(enough, p.separate_arena), true);
  }
  for (size_t i = 0; i < spans.size(); ++i) p.insts[span_inst[i]].offset = spans[i].offset;
  if (p.arena_bytes > std::max(enough, alive_with_z_written(p))) {
    // ... and the same for a z that is not written: what it is made from stays until the apply pass, which may be the fullest moment of a
    // pass that keeps nothing, or placed worse.  Then z is written in those passes, so that what a budget allows does not depend on it.
    // (The values are the same.  Passes that keep something keep the source too.  Of 420 000 random networks 15 are smaller with it
    // written; comparing the bytes alive first leaves 1.6 % of those with such layers to be built twice.)
    Plan q = p;
    q.z_written = true;
    if (!build_schedule(q, enough)) { p.error = q.error; return false; }
    if (q.arena_bytes < p.arena_bytes) {
      p = q;
      p.z_written = false;
    }
  }
  p.separate_arena = 0;
  return true;
}

// Schedules q as one segment in storage mode `mode`: bytes alive at every operation, and the most at any of a unit's backward pass.
static bool fullest_moments(Plan& q, int mode, std::vector<int64_t>& alive, std::vector<int64_t>& most) {
  q.cfg.storage_mode = mode;
  q.seg_begin = {0, (int)q.units.size()};
  if (!schedule_operations(q)) return false;
  std::vector<int64_t> born(q.sched.size() + 1, 0);
  alive.assign(q.sched.size(), 0);
  most.assign(q.units.size(), 0);
  for (const Inst& t : q.insts)
    if (t.def_op >= 0) { born[t.def_op] += (int64_t)t.bytes; born[t.last_use + 1] -= (int64_t)t.bytes; }
  int64_t sum = 0;
  for (size_t i = 0; i < q.sched.size(); ++i) {
    alive[i] = sum += born[i];
    const int unit = q.fops[q.sched[i].fop].unit;
    if (q.sched[i].live && q.sched[i].phase == PH_BWD) most[unit] = std::max(most[unit], sum);
  }
  return true;
}

void choose_sums(Plan& p, const Plan& folded) {
  const size_t nu = p.units.size();
  bool inside = false, shortcut = false;
  for (const FOp& f : p.fops) {
    inside = inside || f.dgrad_sums > 0 || f.bwd_splits > 0;
    shortcut = shortcut || (f.skip >= 0 && f.skip != p.unit_in[f.unit]);
  }
  p.unit_sums.assign(nu, 0);
  std::vector<int64_t> alive, with, before[3];
  for (char which : {SUMS_INSIDE, SUMS_SHORTCUT}) {  // (the sums of a shortcut's BatchNorm are alive for longer)
    if (!(which == SUMS_INSIDE ? inside : shortcut)) continue;
    std::vector<char> ok(nu, 1);
    for (int mode = 0; mode < 3; ++mode) {
      Plan q = mode == 2 ? p : folded;
      q.separate = true;
      if (before[mode].empty() && !fullest_moments(q, mode, alive, before[mode])) return;
      q.separate = false;
      q.unit_sums = p.unit_sums;
      for (char& u : q.unit_sums) u = (char)(u | which);
      if (!fullest_moments(q, mode, alive, with)) return;
      for (size_t u = 0; u < nu; ++u) ok[u] = ok[u] && with[u] <= before[mode][u];
    }
    for (size_t u = 0; u < nu; ++u) if (ok[u]) p.unit_sums[u] = (char)(p.unit_sums[u] | which);
  }
}

void choose_again(Plan& p, Plan& folded) {
  auto relu_in_front = [&](const FOp& cv) {  // (a BatchNorm in front of the unit: the kernels fold it with its ReLU)
    for (const FOp& f : folded.fops) if (f.kind == F_BN_APPLY && f.out == cv.x) return cv.fold_src < 0 && f.relu != 0;
    return cv.fold_src < 0;
  };
  auto layer = [&](int apply, bool fold) {  // the convolution two operations ahead
    if (apply < 2) return false;
    const FOp& cv = folded.fops[apply - 2];
    return cv.kind == F_CONV && cv.out == folded.fops[apply].x && cv.again_rows > 0 && cv.bwd_splits > 0 && cv.stat_blocks > 0 &&
           cv.stat_fold == 0 && !cv.has_bias && folded.tensors[cv.x].needs_grad && (fold ? cv.fold_src >= 0 : relu_in_front(cv));
  };
  for (int i = 0; i < (int)folded.fops.size(); ++i) {
    const FOp& a = folded.fops[i];
    if (a.kind != F_BN_APPLY || a.skip < 0 || a.mask < 0 || !a.relu || a.fold || !layer(i, true)) continue;
    if (i + 1 < (int)folded.fops.size() && folded.fops[i + 1].kind == F_HEAD) continue;  // (pooled, the gradient per image: from z)
    int proj = -1, reader = -1;
    for (int j = folded.unit_first_fop[a.unit]; j < folded.unit_last_fop[a.unit]; ++j) {
      if (folded.fops[j].kind == F_BN_APPLY && folded.fops[j].out == a.skip) proj = j;
      if (folded.fops[j].kind == F_CONV && folded.fops[j].x == a.skip) reader = j;
    }
    if (proj >= 0 ? a.fold_skip != proj || !layer(proj, false)
                  : reader < 0 || folded.fops[reader].dgrad_algo != ALGO_MFMA) continue;
    for (Plan* q : {&p, &folded}) {
      q->fops[i].again = q->fops[i - 2].again = 1;
      q->fops[i].again_skip = proj;
      if (proj >= 0) q->fops[proj].again = q->fops[proj - 2].again = 1;
    }
  }
}

std::vector<int64_t> wgrad_room(const Plan& p) {
  std::vector<int64_t> room(p.fops.size(), 0);
  for (int mode = 0; mode < 2; ++mode) {
    Plan q = p;
    std::vector<int64_t> alive, most;
    if (!fullest_moments(q, mode, alive, most)) return room;  // (a network that cannot be scheduled is refused later)
    for (size_t i = 0; i < q.sched.size(); ++i) {
      const SOp& s = q.sched[i];
      if (!s.live || s.kind != S_WGRAD) continue;
      const int64_t ws = s.out[0] >= 0 ? (int64_t)q.insts[s.out[0]].bytes : 0;
      const int64_t r = most[q.fops[s.fop].unit] - (alive[i] - ws);
      room[s.fop] = mode ? std::min(room[s.fop], r) : r;
    }
  }
  return room;
}

void build_inference(Plan& p) {
  p.infer.clear();
  std::vector<Span> spans;
  std::vector<int> span(p.tensors.size(), -1);  // [LTensor] -> its span
  // (until the tensors are placed, the offsets of an entry are spans)
  auto make = [&](uint64_t bytes) {
    const int t = (int)p.infer.size();
    spans.push_back(Span{aligned(bytes), t, t, 0});
    return (int64_t)spans.size() - 1;
  };
  auto read = [&](int t) -> int64_t {
    spans[span[t]].last = (int)p.infer.size();
    return span[t];
  };
  for (int i = 0; i < (int)p.fops.size(); ++i) {
    const FOp& f = p.fops[i];
    if (f.kind == F_BN_STATS || f.kind == F_BN_APPLY) continue;  // in the convolution's epilogue
    IOp o;
    o.fop = i;
    o.kind = f.kind == F_CAST_IN ? S_CAST_IN : f.kind == F_CONV ? S_CONV_FWD : f.kind == F_POOL ? S_POOL_FWD : S_HEAD_FWD;
    int out = f.kind == F_HEAD ? f.aux[0] : f.out;
    if (f.x >= 0) o.in = read(f.x);
    if (f.kind == F_CONV && f.has_bn) {  // followed by its statistics and apply operations
      o.apply = i + 2;
      const FOp& ap = p.fops[o.apply];
      out = ap.out;
      if (ap.skip >= 0) o.skip = read(ap.skip);
    }
    o.out = span[out] = (int)make(p.tensors[out].bytes);
    if (f.kind == F_CONV && f.fwd_splits > 1) o.ws = make((uint64_t)f.fwd_splits * f.N * f.P * f.Q * f.K * 4);
    if (f.kind == F_HEAD && f.head_ws > 0) o.ws = f.head_ws_in_x ? o.in : make((uint64_t)f.head_ws * 4);
    p.infer.push_back(o);
  }
  p.infer_bytes = place(spans, (int)p.infer.size(), 0);
  for (IOp& o : p.infer)
    for (int64_t* off : {&o.in, &o.skip, &o.out, &o.ws})
      if (*off >= 0) *off = (int64_t)spans[*off].offset;
}

// Training keeps a convolution's output z until its BatchNorm apply has read it, and the skip connection with it; nothing else
// lies there meanwhile.  So the convolution writes the activation itself to the place of z, and the apply operation becomes a
// copy to the activation's place (or the pooling behind it); where the apply is folded into its reader, that reads the place of
// z.  The kernels and their operands are those of build_inference, hence the same bits for every partition and every budget.
void inference_in_schedule(Plan& p) {
  p.infer.clear();
  p.infer_bytes = p.arena_bytes;
  std::vector<int64_t> at(p.tensors.size(), -1);  // place of an activation
  auto place = [&](int inst) { return inst < 0 ? (int64_t)-1 : (int64_t)p.insts[inst].offset; };
  for (const SOp& s : p.sched) {
    if (!s.live || (s.phase != PH_FWD_NOSAVE && s.phase != PH_FWD_LAST)) continue;
    const FOp& f = p.fops[s.fop];
    IOp o;
    o.kind = s.kind;
    o.fop = s.fop;
    o.in = place(s.in[0]);
    o.out = place(s.out[0]);
    switch (s.kind) {
      case S_CONV_FWD: {
        int out = f.out;
        if (f.has_bn) {
          o.apply = s.fop + 2;
          const FOp& ap = p.fops[o.apply];
          out = ap.out;
          if (ap.skip >= 0) o.skip = at[ap.skip];
        }
        at[out] = o.out;
        o.ws = place(s.out[1]);
        break;
      }
      case S_BN_STATS: continue;
      case S_BN_APPLY:
        if (s.out[1] >= 0) {
          IOp pool = o;
          pool.kind = S_POOL_FWD;
          pool.fop = s.fop + 1;
          pool.out = at[p.fops[pool.fop].out] = place(s.out[1]);
          p.infer.push_back(pool);
          if (s.out[0] < 0) continue;
        }
        at[f.out] = o.out;
        break;
      case S_HEAD_FWD: o.ws = f.head_ws_in_x ? o.in : place(s.out[4]); break;
      default: at[f.out] = o.out;  // the input's cast, a pool of its own
    }
    p.infer.push_back(o);
  }
}

// Per-unit byte model of what a segment holds for its backward pass, read off a k = 1 schedule.  A tensor kept for
// backward counts for the unit that made it, except a unit's output: that is kept as the input of the next unit (whose
// backward reads it), so inside a segment it counts for every unit but the last, and for the last one only where the
// unit's own backward reads it.  The first unit's input is the segment's checkpoint and is counted separately.
struct SegModel {
  std::vector<uint64_t> own_pre, out_pre, out_self, ck;
  explicit SegModel(const Plan& all) {
    const int nu = (int)all.units.size();
    std::vector<uint64_t> own(nu, 0), outb(nu, 0);
    std::vector<char> self(nu, 0);
    for (const Inst& t : all.insts) {
      if (!t.held || t.logical < 0) continue;
      const int u = all.tensors[t.logical].unit;
      if (u < 0) continue;
      if (t.logical == all.unit_out[u]) outb[u] += t.bytes; else own[u] += t.bytes;
    }
    for (const SOp& s : all.sched) {
      if (!s.live || s.phase != PH_BWD || s.fop < 0) continue;
      const int u = all.fops[s.fop].unit;
      if (u < 0) continue;
      for (int i : s.in)
        if (i >= 0 && all.insts[i].fwd_value && all.insts[i].logical == all.unit_out[u]) self[u] = 1;
    }
    own_pre.assign(nu + 1, 0); out_pre.assign(nu + 1, 0); out_self.assign(nu, 0); ck.assign(nu, 0);
    for (int u = 0; u < nu; ++u) {
      own_pre[u + 1] = own_pre[u] + own[u];
      out_pre[u + 1] = out_pre[u] + outb[u];
      out_self[u] = self[u] ? outb[u] : 0;
      ck[u] = all.tensors[all.unit_in[u]].bytes;
    }
  }
  // bytes units [s, e) hold at the end of their forward pass or replay
  uint64_t saved(int s, int e) const { return (own_pre[e] - own_pre[s]) + (out_pre[e - 1] - out_pre[s]) + out_self[e - 1]; }
  uint64_t total() const { return own_pre.back() + out_pre.back(); }
};

uint64_t model_peak_saved(const Plan& all_stored, const std::vector<int>& seg_begin) {
  const SegModel m(all_stored);
  uint64_t ck = 0, peak = 0;
  for (size_t j = 0; j + 1 < seg_begin.size(); ++j) {
    ck += m.ck[seg_begin[j]];
    peak = std::max(peak, ck + m.saved(seg_begin[j], seg_begin[j + 1]));
  }
  return peak;
}

bool choose_segments(Plan& p) {
  const int nu = (int)p.units.size();
  const int k = p.cfg.k_segments;
  if (k < 1 || k > nu) { p.error = "k_segments must be between 1 and the number of units"; return false; }
  p.seg_begin.assign(1, 0);
  if (p.cfg.boundaries) {
    int prev = 0;
    for (int j = 0; j < k - 1; ++j) {
      int b = p.cfg.boundaries[j];
      if (b <= prev || b >= nu) { p.error = "boundaries must be ascending unit indices in (0, n_units)"; return false; }
      p.seg_begin.push_back(b); prev = b;
    }
    p.seg_begin.push_back(nu);
    return true;
  }
  if (p.cfg.plan_mode == 0 || k == 1) {
    int per = nu / k;
    for (int j = 1; j < k; ++j) p.seg_begin.push_back(j * per);
    p.seg_begin.push_back(nu);
    return true;
  }
  if (p.cfg.plan_mode != 1 && p.cfg.plan_mode != 2) { p.error = "plan_mode must be 0, 1 or 2"; return false; }
  // min-peak: per-unit byte model from the all-stored schedule, then the smallest threshold T for which a
  // partition into k segments exists with  sum_{i<=j} checkpoint_i + saved_j <= T  for every j.
  Plan all = p;
  all.cfg.boundaries = nullptr;
  all.seg_begin = {0, nu};
  if (!schedule_operations(all)) { p.error = all.error; return false; }
  const SegModel model(all);
  const std::vector<uint64_t>& ck = model.ck;
  const uint64_t INF = ~0ull;
  std::vector<int> best;
  auto feasible = [&](uint64_t T, std::vector<int>* cuts) {
    // g[j][e]: least checkpoint total with j segments covering units [0, e)
    std::vector<std::vector<uint64_t>> g(k + 1, std::vector<uint64_t>(nu + 1, INF));
    std::vector<std::vector<int>> from(k + 1, std::vector<int>(nu + 1, -1));
    g[0][0] = 0;
    for (int j = 1; j <= k; ++j)
      for (int e = j; e <= nu; ++e)
        for (int s = j - 1; s < e; ++s) {
          if (g[j - 1][s] == INF) continue;
          uint64_t c = g[j - 1][s] + ck[s];
          if (c + model.saved(s, e) > T) continue;
          if (c < g[j][e]) { g[j][e] = c; from[j][e] = s; }
        }
    if (g[k][nu] == INF) return false;
    if (cuts) {
      cuts->assign(k + 1, 0);
      int e = nu;
      for (int j = k; j >= 1; --j) { (*cuts)[j] = e; e = from[j][e]; }
      (*cuts)[0] = 0;
    }
    return true;
  };
  uint64_t lo = 0, hi = model.total();
  for (int u = 0; u < nu; ++u) hi += ck[u];
  while (lo < hi) {
    uint64_t mid = lo + (hi - lo) / 2;
    if (feasible(mid, nullptr)) hi = mid; else lo = mid + 1;
  }
  if (!feasible(lo, &best)) { p.error = "internal: min-peak planner found no partition"; return false; }
  p.seg_begin = best;
  if (p.cfg.plan_mode == 1) return true;

  // plan_mode 2: least recomputation.  The last segment is never replayed, so among the partitions whose modelled
  // peak stays within a threshold the one with the cheapest replay (the forward pass of all segments but the last,
  // from a rough per-unit time estimate) is taken.  The threshold is the minimum peak found above; with a budget it
  // starts at the budget instead and is lowered until the schedule built for the partition fits the budget.
  std::vector<double> cost(nu, 0.0), cpre(nu + 1, 0.0);
  {
    const double rate = p.cfg.precision == OPTORCH_FP32 ? 9e13 : 4.5e14, bw = 4e12, launch = 4e-6, e = (double)p.esize;
    for (const FOp& f : p.fops) {
      if (f.unit < 0) continue;
      const double in_px = (double)f.N * f.H * f.W, out_px = (double)f.N * f.P * f.Q;
      double t = launch;
      if (f.kind == F_CONV) {
        const double w = (double)f.K * f.R * f.S * f.C;
        t += 2.0 * out_px * w / rate + e * (in_px * f.C + out_px * f.K + w) / bw;
      } else if (f.kind == F_BN_APPLY) {
        t += e * out_px * f.C * (f.skip >= 0 ? 3 : 2) / bw;
      } else if (f.kind == F_POOL) {
        t += e * in_px * f.C * 1.25 / bw;
      }
      cost[f.unit] += t;
    }
    for (int u = 0; u < nu; ++u) cpre[u + 1] = cpre[u] + cost[u];
  }
  struct St { uint64_t ck; double cost; int from_s, from_i; };
  auto cheapest = [&](uint64_t T, std::vector<int>* cuts) {
    // per (segments used, units covered): the states no other state beats in both checkpoint bytes and replay cost
    std::vector<std::vector<std::vector<St>>> S(k + 1, std::vector<std::vector<St>>(nu + 1));
    S[0][0].push_back(St{0, 0.0, -1, -1});
    for (int j = 1; j <= k; ++j)
      for (int e = j; e <= nu - (k - j); ++e) {
        if (j == k && e != nu) continue;
        std::vector<St> cand;
        for (int s0 = j - 1; s0 < e; ++s0)
          for (size_t i = 0; i < S[j - 1][s0].size(); ++i) {
            const St& st = S[j - 1][s0][i];
            const uint64_t c = st.ck + ck[s0];
            if (c + model.saved(s0, e) > T) continue;
            cand.push_back(St{c, st.cost + (e == nu ? 0.0 : cpre[e] - cpre[s0]), s0, (int)i});
          }
        std::sort(cand.begin(), cand.end(), [](const St& a, const St& b) { return a.ck != b.ck ? a.ck < b.ck : a.cost < b.cost; });
        double least = 1e300;
        for (const St& c : cand)
          if (c.cost < least) { S[j][e].push_back(c); least = c.cost; }
      }
    if (S[k][nu].empty()) return false;
    size_t bi = 0;
    for (size_t i = 1; i < S[k][nu].size(); ++i)
      if (S[k][nu][i].cost < S[k][nu][bi].cost) bi = i;
    cuts->assign(k + 1, 0);
    int e = nu; size_t idx = bi;
    for (int j = k; j >= 1; --j) {
      (*cuts)[j] = e;
      const St& st = S[j][e][idx];
      e = st.from_s; idx = (size_t)st.from_i;
    }
    return true;
  };
  const uint64_t budget = p.cfg.activation_budget_bytes;
  if (!budget) {
    std::vector<int> cuts;
    if (cheapest(lo, &cuts)) { p.seg_begin = cuts; return true; }
    p.seg_begin = best;
    return true;
  }
  // With a budget: the modelled peak (saved tensors only) of a partition is below its arena (transients, alignment,
  // fragmentation), so the threshold that just fits the budget is searched: lowered in sixteenths from the budget until
  // the scheduled arena fits, then bisected between that threshold and the last one that did not.
  auto fits = [&](uint64_t T, std::vector<int>* cuts, bool* error) {
    *error = false;
    if (!cheapest(T, cuts)) return false;
    Plan trial = p;
    trial.cfg.boundaries = nullptr;
    trial.seg_begin = *cuts;
    if (!build_schedule(trial, budget)) { p.error = trial.error; *error = true; return false; }
    return trial.arena_bytes <= budget;
  };
  uint64_t T = budget > lo ? budget : lo, too_big = 0;
  std::vector<int> good;
  uint64_t good_T = 0;
  for (int attempt = 0; attempt < 24; ++attempt) {
    std::vector<int> cuts;
    bool error;
    if (fits(T, &cuts, &error)) { good = cuts; good_T = T; break; }
    if (error) return false;
    too_big = T;
    if (T == lo) break;
    T = std::max<uint64_t>(lo, T - T / 16);
  }
  if (!good.empty()) {
    for (int it = 0; it < 8 && too_big > good_T + (budget >> 10); ++it) {
      const uint64_t mid = good_T + (too_big - good_T) / 2;
      std::vector<int> cuts;
      bool error;
      if (fits(mid, &cuts, &error)) { good = cuts; good_T = mid; }
      else { if (error) return false; too_big = mid; }
    }
    p.seg_begin = good;
    return true;
  }
  p.seg_begin = best;  // nothing cheaper fits: the minimum-peak partition
  return true;
}

}  // namespace oseq
