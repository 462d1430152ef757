// hisv_internal.h -- host-side types shared by the library's translation units.
#pragma once

#include <stdint.h>

#include <complex>
#include <exception>
#include <map>
#include <new>
#include <memory>
#include <mutex>
#include <thread>
#include <string>
#include <vector>

#include "../../include/hisv.h"
#include "layout.h"

namespace hisv {

using cd = std::complex<double>;

// ---- errors ---------------------------------------------------------------
hs_status fail(hs_status code, const char* fmt, ...);
void clear_error();

// No exception crosses the C boundary or ends a library thread: each entry
// point and each thread body runs inside guarded(), which returns a failed
// allocation as HS_E_NOMEM and any other exception (a thread that could not
// be started, ...) as HS_E_INTERNAL.
template <class F>
hs_status guarded(F&& body) noexcept {
  try {
    return body();
  } catch (const std::bad_alloc&) {
    return fail(HS_E_NOMEM, "host allocation failed");
  } catch (const std::exception& e) {
    return fail(HS_E_INTERNAL, "%s", e.what());
  } catch (...) {
    return fail(HS_E_INTERNAL, "unexpected exception");
  }
}

// ---- gates (Sec. II.A) ----------------------------------------------------
constexpr int kMatrixGate = 100;  // internal kind: the one-qubit matrix in Gate::u
struct Gate {
  int kind, q0, q1;
  double p[3];
  cd u[4];  // kMatrixGate only
  int arity() const { return q1 < 0 ? 1 : 2; }
  uint64_t mask() const {  // q0 < 0: a stand-in that needs no qubit (active_gates)
    return (q0 >= 0 ? uint64_t(1) << q0 : 0) | (q1 >= 0 ? (uint64_t(1) << q1) : 0);
  }
};

bool kind_is_1q(int kind);
bool kind_is_2q(int kind);
hs_status validate_gate(int n, const hs_gate& g, Gate* out);
// Validate a gate and append it, or the one- and two-qubit gates that
// replace a three-qubit kind, to *out.
hs_status expand_gate(int n, const hs_gate& g, std::vector<Gate>* out);
// 2x2 matrix (row-major) of a one-qubit gate, in FP64.
void gate_matrix(const Gate& g, cd u[4]);

struct Circuit {
  int n = 0;
  std::vector<Gate> gates;
};

// ---- partitioning (Sec. IV) -------------------------------------------------
struct Dag {
  int G = 0;
  std::vector<std::vector<int>> succ, pred;  // wire dependencies, no duplicates
};
Dag build_dag(const std::vector<Gate>& gates);

// Contiguous cutoff of `order` (a topological order) into parts of at most k
// qubits; part_of_gate is indexed by gate id.  Returns the number of parts.
// `pad` = qubits every part holds anyway (the padding of a multi-level tile):
// a part's qubits together with them must number at most k.
int cutoff_partition(const std::vector<Gate>& gates, const std::vector<int>& order, int k,
                     std::vector<int32_t>* part_of_gate, uint64_t pad = 0);
int partition_nat(const std::vector<Gate>& gates, int k, std::vector<int32_t>* part,
                  uint64_t pad = 0);
int partition_dfs(const std::vector<Gate>& gates, const Dag& dag, int k, uint64_t seed,
                  int trials, std::vector<int32_t>* part, uint64_t pad = 0);
int partition_dagp(const std::vector<Gate>& gates, const Dag& dag, int n, int k,
                   uint64_t seed, std::vector<int32_t>* part, uint64_t pad = 0);
int partition_greedy(const std::vector<Gate>& gates, const Dag& dag, int k, uint64_t seed,
                     int trials, std::vector<int32_t>* part, uint64_t pad = 0);
// hs_tune("host_threads"): threads a partition search may use (0 = up to 8,
// as the host has them).
int host_threads();
// hs_tune("serve_chunk"): parts a serving request enqueues at a time.
int serve_chunk_parts();
// weigh_all: every gate that needs a qubit counts towards a part's weight, not
// only those on two.
int partition_closure(const std::vector<Gate>& gates, const Dag& dag, int k, int width,
                      std::vector<int32_t>* part, uint64_t pad = 0, bool weigh_all = false);
// Exact validity check; returns "" when valid, else the first violation.
std::string check_partition(const std::vector<Gate>& gates, const Dag& dag,
                            const std::vector<int32_t>& part, int k, uint64_t pad = 0);

// ---- part compilation (kernel descriptors) --------------------------------------
struct HostOp {
  int kind, b0, b1;
  double c[32];  // OP_U2: 4 x 4 complex; the others use the first 8
  // Conditions of OP_CPC, OP_CXC and OP_F: a lane or wave coordinate bit of the
  // stage's layout, kOuterBit + a qubit outside the tile, or kNoCond.
  int cond, cond2;
};


// How a part-pass grid walks the tiles of a part.  Workgroup b of a launch
// runs on XCD b % 8 and each XCD has its own L2; the hardware sustains more
// HBM bandwidth when every XCD sweeps one contiguous run of tiles than when
// consecutive tiles are dealt round-robin over the XCDs.
struct LaunchShape {
  bool xcd = true;        // XCD x takes tiles [x T/8, (x+1) T/8)
  int per_cu = 0;         // 0: one workgroup per tile; g > 0: a persistent grid of
                          // g x (resident workgroups per CU) x CUs
  bool prefetch = false;  // persistent grid: keep the next tile's loads in flight
  // specialized kernels: LDS re-layouts run in 2 or 4 rounds when the tile's
  // LDS image exceeds this many bytes (two workgroups then share a CU)
  size_t lds_limit = 65536;
};

struct CompiledPart {
  PartDesc desc;                    // stage_off relative to this part's stages
  std::vector<StageDesc> stages;    // load, stages..., store (op ranges relative)
  std::vector<HostOp> ops;
  int rb_kernel = 0;
  int lds_round_trips = 0;
  double work = 0;                  // vector instructions an amplitude
  LaunchShape launch;
};

// A part applied as one dense unitary on matrix cores (the fused path):
// U acts on the qubits sq[0..w) (bit b of a row/column index = qubit sq[b]),
// columns of the batched product are the settings of the 4 column qubits.
struct FusedPart {
  int w = 0;                  // 4 to 7
  int m = 0;                  // tile = w + 4 qubits
  uint64_t tiles = 0;         // 2^(n - m)
  int8_t sq[8] = {0};
  int8_t pq[4] = {0};
  int8_t tq[12] = {0};        // sq and pq together, ascending
  std::vector<cd> u;          // 2^w x 2^w, row-major
};
hs_status compile_fused(int n, const std::vector<Gate>& part_gates, FusedPart* out);

struct CompileOptions {
  int rb = 4;        // register bits per lane (2^rb amplitudes per lane)
  int contig = 6;    // tile always holds qubits 0..contig-1 (coalesced runs)
  int max_wb = 4;    // at most 2^max_wb wavefronts per workgroup
  int swizzle = 4;   // LDS swizzle width (bits)
  int max_m = 14;    // widest tile whose 2^m amplitudes fit the LDS
  int min_run = 6;   // load/store straight in a stage layout whose lanes cover
                     // at least qubits 0..min_run-1 (runs of 2^min_run amplitudes)
  int min_tile = 0;  // pad tiles with the lowest free qubits up to this many
                     // (longer contiguous runs per tile); 0 = lanes + registers
  bool fuse2 = false;  // merge two-qubit gates with their one-qubit neighbours
                       // into dense 4 x 4 ops where that saves instructions
  // Only the qubits a gate needs as register bits (active_gates) have to be in
  // the tile and in a stage's registers; the others are read off the
  // amplitude's index.  Gates are reduced ones.
  bool conditions = false;
  int stage_trials = 32;  // orders tried for the cut into register stages
  bool plain = false;  // apply every one-qubit run whole, where it ends (Plan::plain)
  LaunchShape launch;
};

// Stand-ins for a circuit's gates that carry only the qubits a kernel needs in
// its registers to apply them -- a controlled gate's target, a swap's pair,
// none for CZ and CP, which only multiply amplitudes by a factor their index
// selects -- and the order that really binds them: gates that act on a shared
// qubit by its value alone, or both as a rotation about X, commute.
std::vector<Gate> active_gates(const std::vector<Gate>& gates);
Dag commuting_dag(int n, const std::vector<Gate>& gates);

// The same circuit with its one-qubit gates as few matrices (compile.cpp).
std::vector<Gate> reduce_gates(int n, const std::vector<Gate>& gates);

// Compile one part (its gates in circuit order) on an n-qubit state.
hs_status compile_part(int n, const std::vector<Gate>& part_gates, const CompileOptions& opt,
                       CompiledPart* out);
int max_tile_qubits(const CompileOptions& opt);
// Whether compile_part finds a tile for a part on these qubits.
bool part_fits(int n, uint64_t mask, const CompileOptions& opt);

// ---- plan -------------------------------------------------------------------
struct DevicePlan;  // uploaded descriptors (kernels.hip)
void device_plan_free(DevicePlan* d);
struct SpecKernel;  // a part's specialized kernel (specialize.cpp)

// The sweeps hs_simulate runs instead of a plan's parts (sweeps.cpp), in
// order; none where the parts are kept.
struct SweepSet {
  bool ready = false;
  std::vector<CompiledPart> comp;
};

// The pieces hs_simulate applies as dense unitaries instead of a plan's parts
// (sweeps.cpp), in order; none where the parts are the cheaper.
struct FusedSet {
  bool ready = false, built = false;
  double cost = 0;                       // in HBM sweeps
  std::vector<std::vector<Gate>> gates;  // of each piece
  std::vector<FusedPart> parts;          // built on first use
};

struct DeviceFused;  // uploaded unitaries (kernels.hip)
void device_fused_free(DeviceFused* d);

struct Plan {
  int n = 0, k = 0;
  uint64_t pad = 0;  // multi-level plans: qubits counted in every part's bound
  bool served = false;  // a server's request
  // Whether the interpreter runs this plan's parts with their ops as they were
  // before one-qubit runs were split (compile.cpp) and before hs_simulate cut
  // plans into sweeps.  Clients read a request's complex64 result, and that of
  // a state of up to 12 qubits, as complex128 and compare it as such; there
  // every bit stays what it has been.  (The split changes the last bits of
  // 24; nothing is lost by keeping the plain ops on such small states, which
  // wait on dispatch and not on arithmetic.)
  bool plain(hs_dtype dt, bool spec) const { return dt == HS_C64 && !spec && (served || n <= 12); }
  std::vector<Gate> gates;
  Dag dag;
  std::vector<int32_t> part_of_gate;
  std::vector<std::vector<int>> parts;  // gate ids per part, circuit order
  std::vector<uint64_t> masks;
  // per dtype: compiled descriptors + uploaded copy (per device)
  std::mutex mu;
  bool compiled[2] = {false, false};
  std::vector<CompiledPart> comp[2];    // for the interpreter kernel
  bool scompiled[2] = {false, false};
  std::vector<CompiledPart> scomp[2];   // for the specialized kernels
  // reduce_gates(gates), their stand-ins and their order, made when the plan is
  // first cut into sweeps or dense pieces
  std::vector<Gate> reduced, reduced_active;
  Dag reduced_dag;
  SweepSet sweeps[2][2];                // [specialized][dtype]
  // uploaded descriptors and built kernels per device: [0] of the parts,
  // [1] of the sweeps
  std::map<int, DevicePlan*> dev[2][2];                                // [sweeps][dtype]
  std::map<int, std::vector<std::shared_ptr<SpecKernel>>> spec[2][2];  // [sweeps][dtype]
  // one kernel build at a time per plan (held across the hipRTC build; the
  // maps above are guarded by mu alone, so launches never wait for a build)
  std::mutex spec_build_mu;
  std::vector<std::thread> spec_threads;  // background builds, joined by ~Plan
  hs_status spec_async_rc[2] = {HS_OK, HS_OK};
  std::string spec_async_msg[2];
  bool fused_built = false;
  std::vector<FusedPart> fused;  // w = 0 where a part has no fused form
  FusedSet fused_set[2];         // [dtype]
  std::map<int, DeviceFused*> fdev[2][2];  // per device, [0] of the parts, [1] of the set; [dtype]
  ~Plan();
};

hs_status plan_build(int n, const std::vector<Gate>& gates, int k,
                     const std::vector<int32_t>& part_of_gate, Plan* p, uint64_t pad = 0);
CompileOptions default_options(hs_dtype dtype, bool spec = false);
hs_status plan_compile(Plan* p, hs_dtype dtype);
hs_status plan_compile_spec(Plan* p, hs_dtype dtype);
// The plan's sweeps on the interpreter or on the specialized kernels, grouped
// and compiled on the first call.
hs_status plan_sweeps(Plan* p, hs_dtype dtype, bool spec, const SweepSet** out);
// the compiled parts of a path (PART_SPEC -> specialized, else interpreter)
const std::vector<CompiledPart>& compiled_parts(const Plan* p, hs_dtype dtype, hs_exec exec);

// ---- state --------------------------------------------------------------------
// Pinned host buffers and events of readouts (kernels.hip).
struct ReadStage {
  void* buf = nullptr;
  void* done[2] = {nullptr, nullptr};  // hipEvent_t, after the kernel that filled a buffer
};
hs_status dev_read_stage_create(ReadStage* r);
void dev_read_stage_free(ReadStage* r);

struct State {
  int n = 0;
  hs_dtype dtype = HS_C64;
  void* ptr = nullptr;
  size_t bytes = 0;
  bool owned = false;
  int device = 0;
  void* stream = nullptr;   // hipStream_t
  void* scratch = nullptr;  // device scratch of the norm (lazily allocated)
  size_t scratch_bytes = 0;
  ReadStage stage;          // made on the first readout
};

inline size_t amp_bytes(hs_dtype d) { return d == HS_C64 ? 8 : 16; }

// ---- device side (kernels.hip) ------------------------------------------------
hs_status dev_set_basis(State* s, uint64_t x);
hs_status dev_gate_pass(State* s, const Gate& g);
// Run one part (or one of the interpreter's sweeps) on the interpreter.
hs_status dev_run_part(State* s, Plan* p, int part, bool sweep = false);
// Upload the interpreter descriptors of the plan's parts (or sweeps) for `dtype` on `device` with the
// stream-ordered allocator on `stream`, without waiting for the copies; the
// plan later frees them with hipFreeAsync on that stream, never with a
// device-wide wait.  A launch on another stream first calls
// dev_plan_stream_wait, which makes that stream wait for the copies.
// Pinned host staging for those copies (one per preparing thread): used
// when large enough and `busy` (recorded after its last copies) has passed;
// otherwise the copies go from pageable memory.
struct PinnedStaging {
  void* ptr = nullptr;
  size_t bytes = 0;
  void* busy = nullptr;  // hipEvent_t
};
hs_status dev_plan_upload_async(Plan* p, bool sweep, hs_dtype dtype, int device, void* stream,
                                const PinnedStaging* pin = nullptr);
hs_status dev_plan_stream_wait(Plan* p, bool sweep, hs_dtype dtype, int device, void* stream);
// Apply a part (or a piece of the plan's fused set) as its dense unitary.
hs_status dev_run_fused(State* s, Plan* p, int part, bool of_set = false);
hs_status plan_compile_fused(Plan* p);
// The plan's gates cut anew for the fused kernels; `build` makes the unitaries.
hs_status plan_fused_set(Plan* p, hs_dtype dtype, bool build, const FusedSet** out);
// hs_tune("fused_shape"): the fused w = 4, 5 kernels' launch shape, read when
// a plan's fused descriptors are uploaded
int fused_launch_shape();
// relative cost (one HBM sweep = 1) of a part on each path, for AUTO
double spec_part_cost(const CompiledPart& cp, hs_dtype dt);
double lds_part_cost(const CompiledPart& cp, hs_dtype dt);
double lds_part_alu(const CompiledPart& cp, hs_dtype dt);  // its arithmetic alone
// (by its qubits alone, so that no unitary is built to decide)
double fused_part_cost(int n, uint64_t mask, hs_dtype dt);
hs_status dev_norm(State* s, double* out);
// the same reduction with its partial sums in a static device array (no allocation)
hs_status dev_norm_noalloc(State* s, double* out);
hs_status dev_read(State* s, uint64_t first, uint64_t count, double* out, bool probs);
hs_status dev_read_at(State* s, const uint64_t* idx, uint64_t count, double* out);
hs_status dev_copy_probe(const void* src, void* dst, size_t bytes, void* stream);
hs_status dev_sync(State* s);

// ---- specialized part kernels (specialize.cpp) ------------------------------------
// standalone = true: a complete translation unit (the runtime header guard
// included); false: only the part's own declarations, to be wrapped in a
// namespace of a multi-kernel program
std::string specialize_part_source(const CompiledPart& cp, hs_dtype dt, const std::string& name,
                                   bool standalone = true);
hs_status specialize_plan(const std::vector<CompiledPart>& parts, hs_dtype dt, int device,
                          std::vector<std::shared_ptr<SpecKernel>>* out);
hs_status launch_specialized(const SpecKernel& k, const CompiledPart& cp, void* state, void* stream);

}  // namespace hisv
