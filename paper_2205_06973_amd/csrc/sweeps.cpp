// sweeps.cpp -- the sweeps that hs_simulate runs for a whole plan.
//
// A plan's parts are bounded by the k its caller chose; what a sweep of the
// state can hold is bounded by the kernels' tile.  hs_simulate applies the
// whole circuit, so it cuts the plan's gates once more, by the closure
// partitioner with the tile as the limit (the multi-level partition of Sec.
// IV.B, first level), and runs one sweep of HBM per piece: 33 sweeps instead
// of 59 parts for the 30-qubit random circuit at k = 7 in complex64, 42 instead
// of 94 for the 28-qubit layered one at k = 6.  hs_simulate_part keeps to the
// plan's parts.
//
// Every sweep gathers runs of 128 bytes, one cache line: the tile holds qubits
// 0..3 (complex64) or 0..2 (complex128) besides the gates' own.  The parts'
// 512 B to 1 KiB runs are read 6% faster but leave two or three qubits fewer
// for gates (complex64, random circuit on 30 qubits, tiles of 13: 42 sweeps of
// 3.29 ms with six padding qubits, 33 of 3.46 ms with four).
#include <algorithm>

#include "hisv_internal.h"

namespace hisv {

namespace {

// Tile widths to try.  Wide states: 13 qubits (complex64) or 12 (complex128)
// leave two to five workgroups on a CU, so that the loads of one tile overlap
// the arithmetic of another; one qubit more takes the whole CU and pays only
// where it saves enough sweeps (random circuit on 30 qubits complex64, 13 / 14:
// 33 sweeps of 3.46 ms, 29 of 4.02; 32-qubit QFT: 21 and 16 sweeps).  Small
// states: a narrower tile, so that there are tiles for the 256 CUs (layered
// circuit on 17 qubits complex128, tiles of 13 / 12 / 11: 99 / 75 / 68 us).
// The interpreter is bound by its instructions, not by the sweeps, and loses
// with 1,024-thread workgroups (25 qubits complex128, 13 / 12 / 11: 8.9 / 7.4 /
// 7.5 ms).
std::vector<int> tile_widths(int n, hs_dtype dtype, bool spec, const CompileOptions& opt) {
  const bool f32 = dtype == HS_C64;
  const int widest = max_tile_qubits(opt), lo = std::min(widest, f32 ? 11 : 10);
  const int top = std::min(widest, (f32 ? 12 : 11) + (spec ? 1 : 0));
  const int m = std::min(n, std::max(lo, std::min(top, n - (f32 && spec ? 7 : 8))));
  std::vector<int> out{m};
  if (spec && m == top && m + 1 <= widest) out.push_back(m + 1);
  return out;
}

// Relative cost of a sweep over m-qubit tiles (see tile_widths).
double tile_cost(int m, hs_dtype dtype) { return m >= (dtype == HS_C64 ? 14 : 13) ? 1.16 : 1.0; }

// A plan keeps its parts unless regrouping takes at least a tenth of the
// sweeps away: the wider tiles have one or two LDS re-layouts more (3% of a
// sweep each).
constexpr double kWorthwhile = 0.9;

}  // namespace

hs_status plan_sweeps(Plan* p, hs_dtype dtype, bool spec, const SweepSet** out) {
  std::lock_guard<std::mutex> lk(p->mu);
  SweepSet& set = p->sweeps[spec][dtype];
  *out = &set;
  if (set.ready) return HS_OK;
  CompileOptions opt = default_options(dtype, spec);
  // a part that no tile holds stays an error, which the parts' path reports
  bool parts_fit = p->parts.size() > 1 && !p->plain(dtype, spec);
  for (uint64_t mask : p->masks) parts_fit &= part_fits(p->n, mask, opt);
  opt.contig = dtype == HS_C64 ? 4 : 3;
  const uint64_t pad = (uint64_t(1) << std::min(opt.contig, p->n)) - 1;
  std::vector<int32_t> best, part;
  int count = 0;
  double cost = kWorthwhile * (double)p->parts.size();
  // The plain closure rule chooses the width; kernels that are built for many
  // runs get the beam search on top: 5-10% fewer sweeps at width 4 (10-14 ms
  // per 1,000 gates) and up to 3% fewer again at 16 (20-30 ms), which a sweep
  // of 16 GiB and more repays in one run.
  int width = 0;
  if (parts_fit)
    for (int m : tile_widths(p->n, dtype, spec, opt)) {
      bool fits = true;
      for (const Gate& g : p->gates) fits &= __builtin_popcountll(g.mask() | pad) <= m;
      if (!fits) continue;
      const int c = partition_closure(p->gates, p->dag, m, 1, &part, pad);
      if (c * tile_cost(m, dtype) < cost) {
        cost = c * tile_cost(m, dtype);
        count = c;
        width = m;
        best.swap(part);
      }
    }
  if (count && spec) count = partition_closure(p->gates, p->dag, width, p->n >= 31 ? 16 : 4, &best, pad);
  std::vector<std::vector<Gate>> gates(count);
  for (size_t i = 0; count && i < p->gates.size(); ++i) gates[best[i]].push_back(p->gates[i]);
  std::vector<CompiledPart> comp(count);
  for (int i = 0; i < count; ++i) {
    if (hs_status rc = compile_part(p->n, gates[i], opt, &comp[i])) return rc;
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
    std::vector<int32_t> best, part;
    for (int w = 5; w <= kMaxFusedQubits && p->n >= w + 4 && cost < 1e29; ++w) {
      const int c = partition_closure(p->gates, p->dag, w, 1, &part);
      std::vector<uint64_t> masks(c, 0);
      for (size_t i = 0; i < p->gates.size(); ++i) masks[part[i]] |= p->gates[i].mask();
      double sum = 0;
      for (uint64_t mask : masks) sum += fused_part_cost(p->n, mask, dtype);
      if (sum >= cost) continue;
      cost = set.cost = sum;
      best.swap(part);
      set.gates.assign(c, {});
    }
    for (size_t i = 0; i < best.size(); ++i) set.gates[best[i]].push_back(p->gates[i]);
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
