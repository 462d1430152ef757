// sweeps.cpp -- the sweeps that hs_simulate runs for a whole plan.
//
// A plan's parts are bounded by the k its caller chose, and every qubit of a
// gate counts.  What a sweep of the state can hold is bounded by the kernels'
// tile, and by less: an amplitude's index tells the value of every qubit, so
// that CZ and CP, which multiply by a factor the index selects, need no qubit
// in the tile, and a CX only its target.  hs_simulate applies the whole
// circuit, so it cuts the plan's gates once more, by the closure partitioner
// over what each gate needs (active_gates) and the order that binds them
// (commuting_dag), with the tile as the limit (the multi-level partition of
// Sec. IV.B, first level), and runs one sweep of HBM per piece.  Sweeps, in
// place of parts: random circuit on 30 qubits, k = 7, complex64 16 of 59;
// layered circuit on 28 qubits, k = 6, 31 of 94; QFT on 32 qubits 5 of 45.
// hs_simulate_part keeps to the plan's parts.
//
// Every sweep gathers runs of 128 bytes, one cache line: the tile holds qubits
// 0..3 (complex64) or 0..2 (complex128) besides the gates' own.  The parts'
// 512 B to 1 KiB runs are read 6% faster but leave two or three qubits fewer
// for gates (complex64, random circuit on 30 qubits, tiles of 13, all qubits
// counted: 42 sweeps of 3.29 ms with six padding qubits, 33 of 3.46 ms with
// four).
#include <algorithm>

#include "hisv_internal.h"

namespace hisv {

namespace {

// Tile width.  Wide states: 13 qubits (complex64) or 12 (complex128) leave two
// to five workgroups on a CU, so that the loads of one tile overlap the
// arithmetic of another; with one qubit more they hardly do (30 qubits, random
// circuit complex64, 12 / 13 / 14 qubits: 18, 16, 15 sweeps, 65.7 / 61.8 / 72.8
// ms; complex128, 11 / 12 / 13: 145 / 119 / 134 ms).  Small states: a narrower
// tile, so that there are tiles for the 256 CUs (layered circuit on 17 qubits
// complex128, 13 / 12 / 11: 99 / 75 / 68 us).  The interpreter is bound by its
// instructions, not by the sweeps, and loses with 1,024-thread workgroups (25
// qubits complex128, 13 / 12 / 11: 8.9 / 7.4 / 7.5 ms).
int tile_width(int n, hs_dtype dtype, bool spec, const CompileOptions& opt) {
  const bool f32 = dtype == HS_C64;
  const int widest = max_tile_qubits(opt), lo = std::min(widest, f32 ? 11 : 10);
  const int top = std::min(widest, (f32 ? 12 : 11) + (spec ? 1 : 0));
  return std::min(n, std::max(lo, std::min(top, n - (f32 && spec ? 7 : 8))));
}

// A complex64 sweep of more instructions an amplitude than this holds 16
// amplitudes a lane instead of 32: a stage then takes four bits, for one
// re-layout more a sweep, but twice the wavefronts overlap loads and
// arithmetic.  Tiles of 13 qubits, 32 / 16 amplitudes: layered circuit (160
// instructions and three re-layouts a sweep) 1.33 / 1.22 ms a sweep, random (55,
// three) 3.87 / 3.72, QFT (30, one) 7.24 / 8.36.
constexpr double kManyInstructions = 32;

// The plan's reduced gates (p->mu held).
void reduce_plan(Plan* p) {
  if (!p->reduced.empty()) return;
  p->reduced = reduce_gates(p->n, p->gates);
  p->reduced_active = active_gates(p->reduced);
  p->reduced_dag = commuting_dag(p->n, p->reduced);
}

// A plan keeps its parts unless regrouping takes at least a tenth of the
// sweeps away: the wider tiles have one or two LDS re-layouts more (3% of a
// sweep each).
constexpr double kWorthwhile = 0.9;

}  // namespace

std::vector<Gate> active_gates(const std::vector<Gate>& gates) {
  std::vector<Gate> out;
  out.reserve(gates.size());
  for (const Gate& g : gates) {
    Gate a{};
    a.kind = kMatrixGate;
    a.q0 = a.q1 = -1;
    switch (g.kind) {
      case HS_CZ: case HS_CP: break;
      case HS_CX: a.q0 = g.q1; break;
      case HS_SWAP: a.q0 = g.q0; a.q1 = g.q1; break;
      default:
        if (!(g.u[1] == cd(0, 0) && g.u[2] == cd(0, 0))) a.q0 = g.q0;
    }
    out.push_back(a);
  }
  return out;
}

Dag commuting_dag(int n, const std::vector<Gate>& gates) {
  // How a gate acts on one of its qubits; gates of one class (but kOther)
  // commute on it.
  enum Class { kValue, kXLike, kOther };
  struct Wire {
    Class cls = kOther;
    std::vector<int> group, before;  // the latest run of one class, and the one it follows
  };
  Dag d;
  d.G = (int)gates.size();
  d.succ.resize(d.G);
  d.pred.resize(d.G);
  std::vector<Wire> wire(n);
  for (int i = 0; i < d.G; ++i) {
    const Gate& g = gates[i];
    auto visit = [&](int q, Class c) {
      Wire& w = wire[q];
      if (c == kOther || c != w.cls) {
        w.before.swap(w.group);
        w.group.clear();
        w.cls = c;
      }
      w.group.push_back(i);
      for (int b : w.before) d.pred[i].push_back(b);
    };
    const bool diag1 = g.arity() == 1 && g.u[1] == cd(0, 0) && g.u[2] == cd(0, 0);
    visit(g.q0, g.kind == HS_CX || g.kind == HS_CZ || g.kind == HS_CP || diag1 ? kValue : kOther);
    if (g.q1 >= 0) visit(g.q1, g.kind == HS_CX ? kXLike : g.kind == HS_SWAP ? kOther : kValue);
    std::sort(d.pred[i].begin(), d.pred[i].end());
    d.pred[i].erase(std::unique(d.pred[i].begin(), d.pred[i].end()), d.pred[i].end());
    for (int b : d.pred[i]) d.succ[b].push_back(i);
  }
  return d;
}

hs_status plan_sweeps(Plan* p, hs_dtype dtype, bool spec, const SweepSet** out) {
  std::lock_guard<std::mutex> lk(p->mu);
  SweepSet& set = p->sweeps[spec][dtype];
  *out = &set;
  if (set.ready) return HS_OK;
  CompileOptions opt = default_options(dtype, spec);
  // a part that no tile holds, or a gate that no stage does, stays an error,
  // which the parts' path reports
  bool parts_fit = p->parts.size() > 1 && !p->plain(dtype, spec);
  for (uint64_t mask : p->masks) parts_fit &= part_fits(p->n, mask, opt);
  for (const Gate& g : p->gates) parts_fit &= g.arity() <= opt.rb;
  opt.contig = dtype == HS_C64 ? 4 : 3;
  const uint64_t pad = (uint64_t(1) << std::min(opt.contig, p->n)) - 1;
  if (parts_fit) reduce_plan(p);
  const std::vector<Gate>& gates = p->reduced;
  // controls and phases are read off an amplitude's index: only what a gate
  // needs in registers binds its sweep
  opt.conditions = true;
  opt.fuse2 = false;  // merged ops would need both qubits in registers
  // Below 20 qubits a sweep takes some 20 us whatever it holds, and 32 orders
  // cost a plan's first pass 0.1 ms (200 gates on 12 qubits: 549 / 440 us with
  // 32 / 8).  8 orders give 3% more re-layouts on circuits of 10 to 19 qubits;
  // later passes take the same (72 us).
  if (!spec && p->n < 20) opt.stage_trials = 8;
  std::vector<int32_t> best;
  int count = 0;
  // The interpreter's plans, often run once, are cut by the plain closure rule
  // (2 ms per 1,000 gates); kernels that are built for many runs get the beam
  // search: 5-12% fewer sweeps at width 4 and up to 5% fewer again at 16, which
  // sweeps of 16 GiB and more repay in a few runs.
  const int beam = !spec ? 1 : p->n >= 31 ? 16 : 4;
  const int m = tile_width(p->n, dtype, spec, opt);
  for (const Gate& g : p->reduced_active) parts_fit &= __builtin_popcountll(g.mask() | pad) <= m;
  if (parts_fit) count = partition_closure(p->reduced_active, p->reduced_dag, m, beam, &best, pad, true);
  if (count > kWorthwhile * (double)p->parts.size()) count = 0;
  std::vector<std::vector<Gate>> piece(count);
  for (size_t i = 0; count && i < gates.size(); ++i) piece[best[i]].push_back(gates[i]);
  std::vector<CompiledPart> comp(count);
  for (int i = 0; i < count; ++i) {
    if (hs_status rc = compile_part(p->n, piece[i], opt, &comp[i])) return rc;
    if (spec && dtype == HS_C64 && opt.rb == 5 && comp[i].lds_round_trips > 1 && comp[i].work > kManyInstructions) {
      CompileOptions narrow = opt;
      narrow.rb = 4;
      CompiledPart alt;
      if (compile_part(p->n, piece[i], narrow, &alt) == HS_OK) comp[i] = std::move(alt);
      else clear_error();
    }
    comp[i].launch = opt.launch;
  }
  set.comp.swap(comp);
  set.ready = true;
  return HS_OK;
}

// The fused kernels cost hardly more for five qubits than for four (they wait
// on HBM), 1.4 times as much for six and 2.6 times for seven, so a plan for
// five-qubit parts runs faster cut for six: 19 pieces instead of 38 for the
// 28-qubit dressed-pair circuit.  Parts that have no fused form stay an error,
// which the parts' path reports.
hs_status plan_fused_set(Plan* p, hs_dtype dtype, bool build, const FusedSet** out) {
  std::lock_guard<std::mutex> lk(p->mu);
  FusedSet& set = p->fused_set[dtype];
  *out = &set;
  if (!set.ready) {
    double cost = 0;
    for (uint64_t mask : p->masks) cost += fused_part_cost(p->n, mask, dtype);
    cost *= kWorthwhile;
    constexpr int w = 6;
    std::vector<int32_t> part;
    if (p->n >= w + 4 && cost < 1e29) {
      reduce_plan(p);
      const std::vector<Gate>& gates = p->reduced;
      const int c = partition_closure(gates, p->reduced_dag, w, 1, &part);
      std::vector<uint64_t> masks(c, 0);
      for (size_t i = 0; i < gates.size(); ++i) masks[part[i]] |= gates[i].mask();
      for (uint64_t mask : masks) set.cost += fused_part_cost(p->n, mask, dtype);
      if (set.cost < cost) {
        set.gates.assign(c, {});
        for (size_t i = 0; i < gates.size(); ++i) set.gates[part[i]].push_back(gates[i]);
      }
    }
    set.ready = true;
  }
  if (!build || set.built) return HS_OK;
  std::vector<FusedPart> parts(set.gates.size());
  for (size_t i = 0; i < parts.size(); ++i)
    if (hs_status rc = compile_fused(p->n, set.gates[i], &parts[i])) return rc;
  set.parts.swap(parts);
  set.built = true;
  return HS_OK;
}

}  // namespace hisv
