// Host-only validity check of the static plan, built with AddressSanitizer and UBSan by tests/test_plan_validity.py.
// For a network description read from stdin it builds the graph, chooses the segments and builds the schedule with
// the planner's own sources, then walks the schedule and checks what the kernels rely on:
//   * every operation reads only tensors that an earlier live operation produced and that are not yet released;
//   * no two tensors that are alive at the same time overlap in the activation arena, and all lie inside it;
//   * the reported peaks are what the walk finds;
//   * inference, at offsets of its own and at those of the schedule: every operation finds the activations it reads whole
//     where it looks for them, writes neither over them nor over its own workspace, and stays inside its arena.
// All of it twice: with the planner's defaults, and as the library's kernel choices would have it: workspaces for split depths,
// BatchNorms folded into their readers, their backward sums made with the gradient, 1x1 layers whose backward is one kernel or
// whose outputs are made again where they are read; and those once more with such outputs written in passes that keep nothing, which
// the planner does where it makes the arena smaller.
// Input: "k plan_mode precision batch height width channels classes storage_mode n_units" then n_units lines of
// "kind cin cout ksize stride pad has_bn has_relu has_bias".  Output: "ok <arena> <peak_saved> <launches>" or an error; with an
// argument instead, for the library's choices, "again <outputs made again> <outputs written in passes that keep nothing> <memory
// allocations of the schedule> <those of one whose comparison with written outputs is left out>".
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "plan.h"

using namespace oseq;

static long g_allocations = 0;
void* operator new(std::size_t n, const std::nothrow_t&) noexcept {
  ++g_allocations;
  return std::malloc(n ? n : 1);
}
void* operator new(std::size_t n) {
  if (void* q = operator new(n, std::nothrow)) return q;
  throw std::bad_alloc();
}
void operator delete(void* q, const std::nothrow_t&) noexcept { std::free(q); }
void operator delete(void* q) noexcept { std::free(q); }
void operator delete(void* q, std::size_t) noexcept { std::free(q); }

static int fail(const char* what, int op, int inst) {
  std::printf("error: %s (operation %d, tensor %d)\n", what, op, inst);
  return 1;
}

static int check_schedule(const Plan& p) {
  const int n = (int)p.sched.size();
  std::vector<char> alive(p.insts.size(), 0);
  std::vector<int> live_list;
  uint64_t live_saved = 0, peak_saved = 0;
  int launches = 0;
  for (int i = 0; i < n; ++i) {
    const SOp& op = p.sched[i];
    if (!op.live) continue;
    launches += launches_of(op, p.fops[op.fop]);
    for (int x : op.in)
      if (x >= 0) {
        if (x >= (int)p.insts.size()) return fail("input index out of range", i, x);
        if (!alive[x]) return fail("reads a tensor that is not alive", i, x);
      }
    if (op.again && op.kind == S_BN_APPLY && (p.fops[op.fop].skip < 0 || op.src[0] < 0 || (p.fops[op.fop].again_skip >= 0 && op.src[2] < 0)))
      return fail("an apply pass that makes z again has no skip connection or no source", i, -1);
    if (op.again && op.kind == S_BN_BWD && ((op.in[4] < 0 && op.src[0] < 0) || (op.out[3] >= 0 && op.src[2] < 0) || op.in[3] < 0))
      return fail("sums that make z again have no source or no mask", i, -1);
    for (int x : op.src)
      if (x >= 0 && (x >= (int)p.insts.size() || !alive[x])) return fail("makes a tensor again from one that is not alive", i, x);
    for (int o : op.out)
      if (o >= 0) {
        const Inst& t = p.insts[o];
        if (alive[o]) return fail("produced twice", i, o);
        if (!t.allocated || t.def_op != i) return fail("output not allocated by this operation", i, o);
        if (t.offset % kAlign != 0 || t.offset + t.bytes > p.arena_bytes) return fail("outside the arena", i, o);
        for (int other : live_list)
          if (alive[other]) {
            const Inst& q = p.insts[other];
            const uint64_t a0 = t.offset, a1 = t.offset + (t.bytes ? t.bytes : 1);
            const uint64_t b0 = q.offset, b1 = q.offset + (q.bytes ? q.bytes : 1);
            if (a0 < b1 && b0 < a1) return fail("overlaps a live tensor", i, other);
          }
        alive[o] = 1;
        live_list.push_back(o);
        if (t.held) live_saved += t.bytes;
      }
    if (live_saved > peak_saved) peak_saved = live_saved;
    for (size_t t = 0; t < p.insts.size(); ++t)
      if (alive[t] && p.insts[t].last_use == i) {
        alive[t] = 0;
        if (p.insts[t].held) live_saved -= p.insts[t].bytes;
      }
  }
  for (size_t t = 0; t < p.insts.size(); ++t)
    if (alive[t]) return fail("never released", n, (int)t);
  if (peak_saved != p.peak_saved_bytes) return fail("peak of saved bytes differs from the plan's", -1, -1);
  if (launches != p.n_launches) return fail("launch count differs from the plan's", -1, -1);
  return 0;
}

static int check_inference(const Plan& p) {
  struct Region { uint64_t a, b; int tensor; };  // what the last writer left there; -1: workspace
  std::vector<Region> mem;
  std::vector<int> ran(p.fops.size(), 0);
  for (size_t i = 0; i < p.infer.size(); ++i) {
    const IOp& o = p.infer[i];
    const FOp& f = p.fops[o.fop];
    const int op = (int)i;
    const bool conv = o.kind == S_CONV_FWD, head = o.kind == S_HEAD_FWD, copy = o.kind == S_BN_APPLY;
    ++ran[o.fop];
    const int in = o.kind == S_CAST_IN ? -1 : copy ? f.out : f.x;
    const int skip = conv && o.apply >= 0 ? p.fops[o.apply].skip : -1;
    const int out = head ? f.aux[0] : conv && o.apply >= 0 ? p.fops[o.apply].out : f.out;
    if (conv && f.has_bn && (o.apply < 0 || p.fops[o.apply].kind != F_BN_APPLY || p.fops[o.apply].x != f.out))
      return fail("inference: not the BatchNorm behind the convolution", op, out);
    const uint64_t ws = conv && f.fwd_splits > 1 ? (uint64_t)f.fwd_splits * f.N * f.P * f.Q * f.K * 4 : head ? (uint64_t)f.head_ws * 4 : 0;
    std::vector<Region> mine;  // read by this operation
    for (int r = 0; r < 2; ++r) {
      const int t = r ? skip : in;
      const int64_t at = r ? o.skip : o.in;
      if (t < 0) continue;
      bool found = false;
      for (const Region& m : mem) found = found || (m.tensor == t && (int64_t)m.a == at && m.b - m.a == p.tensors[t].bytes);
      if (!found) return fail("inference: an activation is not where it is read", op, t);
      mine.push_back(Region{(uint64_t)at, at + p.tensors[t].bytes, t});
    }
    for (int w = 0; w < 2; ++w) {
      const int64_t at = w ? o.ws : o.out;
      const uint64_t bytes = w ? ws : p.tensors[out].bytes;  // (a head on the network's own input may lay its workspace over that)
      if (bytes == 0) continue;
      if (at < 0 || at % kAlign != 0 || at + bytes > p.infer_bytes) return fail("inference: outside the arena", op, w ? -1 : out);
      for (const Region& m : mine)
        if ((uint64_t)at < m.b && m.a < at + bytes && !(w && f.head_ws_in_x && m.tensor == f.x && bytes <= m.b - m.a)) return fail("inference: writes over what it uses", op, m.tensor);
      const Region made{(uint64_t)at, at + bytes, w ? -1 : out};
      std::vector<Region> kept;
      for (const Region& m : mem)
        if (!(made.a < m.b && m.a < made.b)) kept.push_back(m);
      kept.push_back(made);
      mem.swap(kept);
      mine.push_back(made);
    }
  }
  for (size_t i = 0; i < p.fops.size(); ++i) {
    const FKind kind = p.fops[i].kind;
    if (kind != F_BN_STATS && kind != F_BN_APPLY && ran[i] != 1) return fail("inference: an operation does not run once", (int)i, -1);
  }
  return 0;
}

// what the library's kernel choices change in the plan: depth splits, the head's ranges, folded BatchNorms
static void choose_as_the_library(Plan& p) {
  p.unit_sums.assign(p.units.size(), SUMS_INSIDE | SUMS_SHORTCUT);
  std::vector<int> readers(p.tensors.size(), 0), reader(p.tensors.size(), -1);
  for (size_t i = 0; i < p.fops.size(); ++i) {
    FOp& f = p.fops[i];
    if (f.x >= 0) { ++readers[f.x]; reader[f.x] = (int)i; }
    if (f.skip >= 0) { ++readers[f.skip]; reader[f.skip] = (int)i; }
    if (f.kind == F_CONV && i % 3 == 1) f.fwd_splits = 2 + (int)i % 4;
    if (f.kind == F_CONV) {
      f.dgrad_algo = ALGO_MFMA;
      if (f.R == 1 && f.stride == 1) {
        f.image_addend = 1;
        if (f.has_bn && !f.has_bias && f.K > f.C) f.bwd_splits = 1 + (int)i % 3;
        if (f.has_bn && !f.has_bias && f.K > f.C) f.again_rows = 1 + (int)i % 7, f.stat_blocks = p.fops[i + 1].stat_blocks = 1 + (int)i % 2;
      } else {
        f.dgrad_sums = 1 + (int)i % 5;
      }
    }
    if (f.kind == F_HEAD) {
      f.head_ws_in_x = !p.tensors[f.x].needs_grad;
      f.head_ws = f.head_ws_in_x ? (int64_t)(p.tensors[f.x].bytes / 4) : (int64_t)4 * f.N * (f.gap ? f.C : f.classes);
    }
  }
  Plan given = p;
  for (size_t i = 0; i < p.fops.size(); ++i) {
    FOp& b = p.fops[i];
    if (b.kind != F_BN_APPLY) continue;
    if (b.relu && b.skip < 0 && b.mask < 0 && readers[b.out] == 1) {
      FOp& cv = p.fops[reader[b.out]];
      if (cv.kind == F_CONV && cv.x == b.out && cv.unit == b.unit && cv.stride == 1) { b.fold = 1; cv.fold_src = (int)i; }
    }
    if (b.skip >= 0 && readers[b.skip] == 1)
      for (size_t j = 0; j < i; ++j) {
        FOp& s = p.fops[j];
        if (s.kind == F_BN_APPLY && s.out == b.skip && s.unit == b.unit && !s.relu && s.skip < 0) { s.fold = 1; b.fold_skip = (int)j; }
      }
  }
  choose_again(given, p);
  if (p.cfg.storage_mode == 2) p = given;
}

// The chosen plan with z written in passes that keep nothing: valid, and no smaller; how often z is made again, what building took.
static int check_written(const Plan& p, Plan built, bool print) {
  Plan q = p;
  long at = g_allocations;
  if (!build_schedule(q)) return fail("a second build fails", -1, -1);
  const long whole = g_allocations - at;
  if (q.arena_bytes != built.arena_bytes) return fail("a second build gives another arena", -1, -1);
  Plan w = p;
  w.z_written = true;
  at = g_allocations;
  if (!build_schedule(w)) return fail("no plan with z written", -1, -1);
  const long once = g_allocations - at;
  if (check_schedule(w)) return 1;
  if (built.arena_bytes > w.arena_bytes) return fail("the arena is larger than with z written", -1, -1);
  int again = 0, written = 0;
  for (const SOp& s : built.sched)
    if (s.live && s.kind == S_CONV_FWD && built.fops[s.fop].again) {
      again += s.again;
      written += !s.again;
      if (!s.again && s.phase != PH_FWD_NOSAVE) return fail("z is written in a pass that keeps something", -1, -1);
    }
  if (print) std::printf("again %d %d %ld %ld\n", again, written, whole, once);
  return 0;
}

int main(int argc, char**) {
  Plan given;
  int n_units = 0;
  optorch_seq_config_t& c = given.cfg;
  if (std::scanf("%d %d %d %d %d %d %d %d %d %d", &c.k_segments, &c.plan_mode, &c.precision, &c.batch, &c.height, &c.width,
                 &c.channels, &c.num_classes, &c.storage_mode, &n_units) != 10) return fail("bad header", -1, -1);
  for (int i = 0; i < n_units; ++i) {
    optorch_unit_t u{};
    if (std::scanf("%d %d %d %d %d %d %d %d %d", &u.kind, &u.cin, &u.cout, &u.ksize, &u.stride, &u.pad, &u.has_bn, &u.has_relu,
                   &u.has_bias) != 9) return fail("bad unit", i, -1);
    given.units.push_back(u);
  }
  Plan first;
  for (int chosen = 0; chosen < 2; ++chosen) {
    Plan p = given;
    if (!build_graph(p)) { std::printf("error: %s\n", p.error.c_str()); return 1; }
    if (chosen) choose_as_the_library(p);
    if (!choose_segments(p)) { std::printf("error: %s\n", p.error.c_str()); return 1; }
    const Plan unbuilt = p;
    if (!build_schedule(p)) { std::printf("error: %s\n", p.error.c_str()); return 1; }
    if (check_schedule(p)) return 1;
    if (chosen && p.cfg.storage_mode != 2 && check_written(unbuilt, p, argc > 1)) return 1;
    build_inference(p);
    if (check_inference(p)) return 1;
    inference_in_schedule(p);
    if (p.infer_bytes != p.arena_bytes) return fail("inference: not the schedule's arena", -1, -1);
    if (check_inference(p)) return 1;
    if (!chosen) first = p;
  }
  if (argc == 1) std::printf("ok %llu %llu %d\n", (unsigned long long)first.arena_bytes, (unsigned long long)first.peak_saved_bytes, first.n_launches);
  return 0;
}
