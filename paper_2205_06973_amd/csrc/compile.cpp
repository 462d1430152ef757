// compile.cpp -- compile a part into the descriptors of the part-pass kernel.
//
// Alg. 1 (Sec. III.C) for one part p with qubit set S_p: for every setting
// of the qubits outside the part, gather the amplitudes addressed by S_p,
// run the part's gates, scatter back.  The kernel gathers a *tile*:
//   T_p = S_p plus the lowest qubits not in S_p, m qubits in all.
// Padding with low qubits is the rule of the multi-level scheme (Sec. IV:
// a part with fewer qubits than the level's limit takes extra qubits for
// spatial locality); here it makes each tile a set of contiguous runs of
// at least 2^contig amplitudes, so global loads and stores coalesce.
//
// Inside the tile the part's gates (circuit order, Sec. IV.A) are cut by the
// natural cutoff (Sec. IV.B.1) with limit rb into stages, each of which
// runs entirely on register bits; this is the second level of the
// multi-level partitioning of Sec. IV, mapped to LDS (level 1: the tile) and
// registers (level 2: the stage).  Each stage's register bits are its
// qubits, padded with high tile bits; its lane bits are the lowest
// remaining tile bits (so that lanes touch neighbouring LDS slots and, in
// the load and store layouts, neighbouring global addresses).
//
// Runs of one-qubit gates on the same bit with no other gate on that bit in
// between are multiplied into one 2x2 in extended precision (gates on different
// bits commute, so the product can be applied where the run ends), and the 2x2
// is split so that as little of it as possible runs (split_gate below).
#include <algorithm>
#include <array>
#include <cmath>
#include <cstring>

#include "hisv_internal.h"

namespace hisv {

int max_tile_qubits(const CompileOptions& opt) {
  return std::min(std::min(kMaxTile, opt.max_m), kLaneBits + opt.max_wb + opt.rb);
}

namespace {

struct Layout {
  int8_t pos[kMaxTile];
};

// Layout with the given register bits (ascending); lanes take the lowest
// other tile bits, waves the rest.
Layout make_layout(int m, int lb, int wb, uint32_t regs) {
  Layout L;
  std::memset(L.pos, 0, sizeof L.pos);
  int c = 0;
  int lane_left = lb;
  std::vector<int> waves;
  for (int t = 0; t < m; ++t) {
    if (regs >> t & 1) continue;
    if (lane_left) {
      L.pos[c++] = (int8_t)t;
      --lane_left;
    } else {
      waves.push_back(t);
    }
  }
  for (int t : waves) L.pos[c++] = (int8_t)t;
  for (int t = 0; t < m; ++t)
    if (regs >> t & 1) L.pos[c++] = (int8_t)t;
  (void)wb;
  return L;
}

// Pad `regs` to exactly rb tile bits: first with bits of `keep` (the
// previous layout's register bits, highest first), then with the highest
// free tile bits.  Keeping register bits across stages lets consecutive
// layouts coincide (no re-layout) or share a register bit (a re-layout can
// then run in two halves through half the LDS).
uint32_t pad_regs(uint32_t regs, int m, int rb, uint32_t keep = 0) {
  for (int t = m - 1; t >= 0 && __builtin_popcount(regs) < rb; --t)
    if (keep >> t & 1) regs |= 1u << t;
  for (int t = m - 1; t >= 0 && __builtin_popcount(regs) < rb; --t) regs |= 1u << t;
  return regs;
}

bool lanes_are_low(const Layout& L, int lb) {
  for (int c = 0; c < lb; ++c)
    if (L.pos[c] != c) return false;
  return true;
}

// Number of leading lane bits that are tile bits 0, 1, 2, ... (the length,
// in bits, of the contiguous global run each group of lanes touches).
int low_run(const Layout& L, int lb) {
  int c = 0;
  while (c < lb && L.pos[c] == c) ++c;
  return c;
}

bool same_layout(const Layout& a, const Layout& b, int m) {
  return std::memcmp(a.pos, b.pos, (size_t)m) == 0;
}

bool is_exact(const cd& z, double re, double im) { return z.real() == re && z.imag() == im; }

// Pending runs and their splits are kept in extended precision, so that a
// coefficient is rounded to FP64 once, when its op is made, however many gates
// and splits it comes from (layered circuit on 25 qubits complex128, error
// against FP64 arithmetic: 5.9e-15 with FP64 runs, 2.5e-15 with plain gates).
using cl = std::complex<long double>;

cd to_cd(const cl& z) { return cd((double)z.real(), (double)z.imag()); }

// products and reciprocals written out: the operators of std::complex also
// order out NaNs and overflow, at ten times the cost
cl mul(const cl& a, const cl& b) {
  return cl(a.real() * b.real() - a.imag() * b.imag(), a.real() * b.imag() + a.imag() * b.real());
}
cl inv(const cl& a) {
  const long double s = 1 / (a.real() * a.real() + a.imag() * a.imag());
  return cl(a.real() * s, -a.imag() * s);
}

void matmul2(const cl a[4], const cl b[4], cl out[4]) {  // out = a * b
  const cl r[4] = {mul(a[0], b[0]) + mul(a[1], b[2]), mul(a[0], b[1]) + mul(a[1], b[3]),
                   mul(a[2], b[0]) + mul(a[3], b[2]), mul(a[2], b[1]) + mul(a[3], b[3])};
  for (int i = 0; i < 4; ++i) out[i] = r[i];
}

void matmul2(const cd a[4], const cd b[4], cd out[4]) {  // out = a * b
  cd r[4];
  r[0] = a[0] * b[0] + a[1] * b[2];
  r[1] = a[0] * b[1] + a[1] * b[3];
  r[2] = a[2] * b[0] + a[3] * b[2];
  r[3] = a[2] * b[1] + a[3] * b[3];
  for (int i = 0; i < 4; ++i) out[i] = r[i];
}

void emit_1q(int b, const cd u[4], std::vector<HostOp>* ops) {
  HostOp op{};
  op.b0 = b;
  op.b1 = -1;
  const bool diag = is_exact(u[1], 0, 0) && is_exact(u[2], 0, 0);
  if (diag) {
    if (is_exact(u[0], 1, 0) && is_exact(u[3], 1, 0)) return;  // identity
    if (is_exact(u[0], 1, 0)) {
      op.kind = OP_D1;
      op.c[0] = u[3].real();
      op.c[1] = u[3].imag();
    } else {
      op.kind = OP_D;
      op.c[0] = u[0].real(); op.c[1] = u[0].imag();
      op.c[2] = u[3].real(); op.c[3] = u[3].imag();
    }
  } else if (is_exact(u[0], 0, 0) && is_exact(u[3], 0, 0) && is_exact(u[1], 1, 0) &&
             is_exact(u[2], 1, 0)) {
    op.kind = OP_X;
  } else if (u[0].imag() == 0 && u[1].imag() == 0 && u[2].imag() == 0 && u[3].imag() == 0) {
    op.kind = OP_R;
    for (int i = 0; i < 4; ++i) op.c[i] = u[i].real();
  } else {
    op.kind = OP_U;
    for (int i = 0; i < 4; ++i) {
      op.c[2 * i] = u[i].real();
      op.c[2 * i + 1] = u[i].imag();
    }
  }
  ops->push_back(op);
}

// ---- one-qubit gates as factors of the part's unitary ---------------------------
//
// A gate run pending on a bit is a 2x2 unitary M.  What the kernels spend on
// it is vector instructions, and those depend on its entries: a term with
// coefficient 1 costs nothing, -1 an add, a real or imaginary one one FMA a
// component, a complex one two.  So M is written as S L K:
//   S  a complex number.  It commutes with everything, is multiplied up over
//      the part and goes into one op at the end.
//   L  the factor that commutes with the two-qubit gate the bit meets next
//      (diagonal for CZ, CP and a control; a rotation about X for a target).
//      It stays pending and merges into the bit's next gate on the host.
//   K  what has to run now, scaled so that its entries are 1 where possible:
//      [[1, b], [-conj(b), 1]] for a generic M, 8 FMAs a pair of amplitudes
//      instead of 16 multiplies and FMAs for M itself (a Hadamard: 4 adds; a
//      rotation about one axis: 4 FMAs).
// Instructions an amplitude of the specialized kernels, before and after: the
// random circuit (30 qubits, k = 7) 2,192 and 1,062, layered 28 qubits, k = 6
// 8,960 and 5,870, dressed pairs 9,992 and 4,476.  Layered 28 qubits complex64
// specialized 83.0 -> 77.2 ms, 20 qubits 660 -> 541 us; the interpreter on 25
// qubits complex128 11.64 -> 10.53 ms.
// The amplitudes grow by 1/|S| on the way (at most a factor sqrt(2) an op);
// past kMaxGrowth S goes into the op at hand, so that an unnormalised state
// keeps all but 10 of its 127 (1023) binary orders of headroom.
constexpr double kMaxGrowth = 1024.0;

enum Role { kRoleZ, kRoleX, kRoleLast };  // kRoleLast: nothing may stay pending

// The parts of a coefficient that are rounding noise of its computation in
// extended precision (a tenth of FP64's) are set to zero, so that products such
// as RZ H keep the real form of H.
cl clean(const cl& z) {
  constexpr long double eps = 1e-17L;
  long double re = z.real(), im = z.imag();
  const long double mag = std::max(std::fabs(re), std::fabs(im));
  if (std::fabs(re) <= eps * mag) re = 0;
  if (std::fabs(im) <= eps * mag) im = 0;
  if (im == 0 && std::fabs(std::fabs(re) - 1) <= eps) re = std::copysign(1.0L, re);
  if (re == 0 && std::fabs(std::fabs(im) - 1) <= eps) im = std::copysign(1.0L, im);
  return cl(re, im);
}

// Vector instructions a pair of amplitudes (real and imaginary parts) for
// y = K x when every term is written out.
template <typename C>
int pair_cost(const C k[4]) {
  int c = 0;
  for (int r = 0; r < 2; ++r) {
    int terms = 0;
    bool unit = false;
    for (int i = 0; i < 2; ++i) {
      const C& z = k[2 * r + i];
      if (z == C(0, 0)) continue;
      terms += (z.real() != 0 && z.imag() != 0) ? 4 : 2;
      unit |= std::fabs(z.real()) + std::fabs(z.imag()) == 1;
    }
    c += terms - (unit ? 2 : 0);
  }
  return c;
}

bool is_identity(const cl k[4]) {
  return k[0] == cl(1, 0) && k[3] == cl(1, 0) && k[1] == cl(0, 0) && k[2] == cl(0, 0);
}

struct Split {
  cl S = 1, K[4] = {1, 0, 0, 1}, L[4] = {1, 0, 0, 1};
  int cost = 0;        // pair_cost(K)
  double rank = 1e30;  // what the candidates are compared by
};

// M = S L K with L allowed by `role`; the cheapest of a few candidates.
Split split_gate(const cl M[4], Role role) {
  // scale: M may be a unitary times a number
  const long double unit = std::max(std::abs(M[0]), std::abs(M[1]));
  if (!(unit > 0)) {
    Split whole;
    std::copy(M, M + 4, whole.K);
    whole.cost = pair_cost(M);
    return whole;
  }
  const long double iu = 1 / unit;
  const cl a = M[0] * iu, b = M[1] * iu, c = M[2] * iu, d = M[3] * iu, zero(0, 0);
  Split best;
  auto offer = [&](cl S, cl l0, cl l1, cl l2, cl l3, cl k0, cl k1, cl k2, cl k3) {
    Split s;
    s.S = S;
    const cl l[4] = {l0, l1, l2, l3}, k[4] = {k0, k1, k2, k3};
    for (int i = 0; i < 4; ++i) {
      s.L[i] = clean(l[i]);
      s.K[i] = clean(k[i]);
    }
    s.cost = is_identity(s.K) ? 0 : pair_cost(s.K);
    // a factor left pending may have to run later (up to 4); growth 1/|S|
    s.rank = s.cost + (is_identity(s.L) ? 0.0 : 1.0) - 0.5 * std::log2(std::min(1.0, (double)std::abs(S)));
    if (s.rank < best.rank) best = s;
  };
  const bool diag = b == zero && c == zero, anti = a == zero && d == zero;
  const long double na = std::abs(a), nb = std::abs(b);
  constexpr long double kSmall = 0.125;
  // nothing pending: M over one of its entries
  const cl ia = na >= kSmall ? inv(a) : zero, ib = nb >= kSmall ? inv(b) : zero;
  if (na >= kSmall) offer(a, 1, 0, 0, 1, 1, mul(b, ia), mul(c, ia), mul(d, ia));
  if (nb >= kSmall) offer(b, 1, 0, 0, 1, mul(a, ib), 1, mul(c, ib), mul(d, ib));
  if (role == kRoleZ) {
    if (diag) offer(a, 1, 0, 0, mul(d, ia), 1, 0, 0, 1);
    else if (anti) offer(b, 1, 0, 0, mul(c, ib), 0, 1, 1, 0);
    else {
      if (na >= kSmall) offer(a, 1, 0, 0, mul(d, ia), 1, mul(b, ia), mul(c, inv(d)), 1);
      if (nb >= kSmall) offer(b, 1, 0, 0, mul(c, ib), mul(a, ib), 1, 1, mul(d, inv(c)));
    }
  } else if (role == kRoleX) {
    // M = e^{ig} (w - i (x X + y Y + z Z)); L = cos t - i sin t X with
    // tan t = z / y leaves K without a Z component: [[w', -y'-ix'], [y'-ix', w']]
    const cl ph = std::sqrt(mul(a, d) - mul(b, c));
    const cl ip = inv(ph), u0 = mul(a, ip), u1 = mul(b, ip);
    const long double w = u0.real(), z = -u0.imag(), y = -u1.real(), x = -u1.imag();
    const long double r = std::hypot(y, z);
    if (r <= 1e-18L) {
      offer(ph, cl(w, 0), cl(0, -x), cl(0, -x), cl(w, 0), 1, 0, 0, 1);
    } else {
      const long double ct = y / r, sn = z / r;
      const long double w1 = w * ct + sn * x, x1 = x * ct - sn * w, y1 = r;
      if (std::fabs(w1) >= kSmall)
        offer(ph * w1, cl(ct, 0), cl(0, -sn), cl(0, -sn), cl(ct, 0), 1, cl(-y1, -x1) / w1, cl(y1, -x1) / w1, 1);
    }
  }
  best.S *= unit;
  return best;
}

}  // namespace

// What hs_simulate's sweeps are cut from: the circuit with every run of
// one-qubit gates split as above, L carried on to the qubit's next gate --
// also where that lies in another sweep -- and K (scaled to a unitary) left as
// one matrix gate.  A part on its own has to finish every run it holds; over
// the circuit only the last run of each qubit is left (instructions an
// amplitude of the specialized kernels, 28-qubit layered circuit of 40 layers:
// 5,650 with every sweep finishing its runs, 4,900 this way).
std::vector<Gate> reduce_gates(int n, const std::vector<Gate>& gates) {
  std::vector<Gate> out;
  out.reserve(gates.size());
  std::vector<std::array<cl, 4>> pend(n);
  std::vector<char> has(n, 0);
  cl phase = 1;
  int last = -1;  // a matrix gate to carry the phase
  auto put = [&](int q, const cl u[4]) {
    Gate g{};
    g.kind = kMatrixGate;
    g.q0 = q;
    g.q1 = -1;
    for (int i = 0; i < 4; ++i) g.u[i] = to_cd(u[i]);
    last = (int)out.size();
    out.push_back(g);
  };
  auto flush = [&](int q, Role role) {
    if (!has[q]) return;
    Split f = split_gate(pend[q].data(), role);
    const long double mag = std::abs(f.S);
    phase = mul(phase, f.S / mag);
    std::copy(f.L, f.L + 4, pend[q].begin());
    has[q] = !is_identity(f.L);
    if (is_identity(f.K)) return;
    for (cl& z : f.K) z *= mag;
    put(q, f.K);
  };
  for (const Gate& g : gates) {
    if (g.arity() == 1) {
      cd m[4];
      gate_matrix(g, m);
      const cl u[4] = {m[0], m[1], m[2], m[3]};
      if (has[g.q0]) matmul2(u, pend[g.q0].data(), pend[g.q0].data());
      else std::copy(u, u + 4, pend[g.q0].begin());
      has[g.q0] = 1;
      continue;
    }
    if (g.kind == HS_SWAP) {
      std::swap(pend[g.q0], pend[g.q1]);
      std::swap(has[g.q0], has[g.q1]);
    } else {
      flush(g.q0, kRoleZ);
      flush(g.q1, g.kind == HS_CX ? kRoleX : kRoleZ);
    }
    out.push_back(g);
  }
  for (int q = 0; q < n; ++q) flush(q, kRoleLast);
  if (clean(phase) != cl(1, 0)) {
    const cl d[4] = {phase, 0, 0, phase};
    if (last < 0) put(0, d);
    else
      for (cd& z : out[last].u) z = to_cd(cl(z) * phase);
  }
  return out;
}

namespace {

// Vector instructions an amplitude for one op on the kernels.
double op_work(const HostOp& op) {
  switch (op.kind) {
    case OP_U: {
      cd k[4];
      for (int i = 0; i < 4; ++i) k[i] = cd(op.c[2 * i], op.c[2 * i + 1]);
      return 0.5 * pair_cost(k);
    }
    case OP_R: {
      cd k[4];
      for (int i = 0; i < 4; ++i) k[i] = op.c[i];
      return 0.5 * pair_cost(k);
    }
    case OP_D: return 4;
    case OP_D1: return 2;
    case OP_CP: return 1;
    case OP_U2: return 16;
    case OP_CPC: case OP_CXC: return 2;
    case OP_FA: return op.b0 ? 2 : 4;
    case OP_GA: return op.b1 ? 1 : 2;
    default: return 0;  // permutations and sign changes
  }
}

// The interpreter's cost of an op on A = 2^rb amplitudes a lane: its
// arithmetic (register moves for a permutation) and the dispatch.  Plain ops
// (CompileOptions::plain) are chosen by the estimate they have always been
// chosen by.
int op_cost(int kind, int A, bool plain) {
  if (plain) switch (kind) {
    case -1: return 0;
    case OP_R: case OP_D: return 5 * A + 10;
    case OP_D1: case OP_X: return 3 * A + 10;
    case OP_CX: case OP_CP: case OP_SWAP: return 2 * A + 10;
    case OP_CZ: return A / 2 + A + 10;
    case OP_U2: return 17 * A + 10;
    default: return 9 * A + 10;
  }
  int c = 0;
  switch (kind) {
    case OP_CX: case OP_CP: case OP_SWAP: c = 2 * A; break;
    case OP_CZ: c = A; break;
    case OP_U2: c = 16 * A; break;
    default: c = 8 * A;
  }
  return c + 10;
}

// Kind emit_1q gives u (-1: identity, no op).
int kind_1q(const cd u[4]) {
  std::vector<HostOp> op;
  emit_1q(0, u, &op);
  return op.empty() ? -1 : op[0].kind;
}

// The 2x2 of a one-qubit op.
bool op_matrix(const HostOp& op, cd k[4]) {
  k[0] = k[3] = 1;
  k[1] = k[2] = 0;
  switch (op.kind) {
    case OP_U: for (int i = 0; i < 4; ++i) k[i] = cd(op.c[2 * i], op.c[2 * i + 1]); return true;
    case OP_R: for (int i = 0; i < 4; ++i) k[i] = op.c[i]; return true;
    case OP_D: k[0] = cd(op.c[0], op.c[1]); k[3] = cd(op.c[2], op.c[3]); return true;
    case OP_D1: k[3] = cd(op.c[0], op.c[1]); return true;
    case OP_X: k[0] = k[3] = 0; k[1] = k[2] = 1; return true;
    default: return false;
  }
}

// 4 x 4 matrices, basis index i = bit(b0) + 2 bit(b1), row-major.
void matmul4(const cd a[16], const cd b[16], cd out[16]) {  // out = a * b
  cd r[16];
  for (int i = 0; i < 4; ++i)
    for (int k = 0; k < 4; ++k) {
      cd z = 0;
      for (int j = 0; j < 4; ++j) z += a[4 * i + j] * b[4 * j + k];
      r[4 * i + k] = z;
    }
  for (int i = 0; i < 16; ++i) out[i] = r[i];
}

// The same operator with the roles of the two bits exchanged.
void swap_bits4(const cd a[16], cd out[16]) {
  auto sg = [](int i) { return (i >> 1) | ((i & 1) << 1); };
  cd r[16];
  for (int i = 0; i < 4; ++i)
    for (int k = 0; k < 4; ++k) r[4 * sg(i) + sg(k)] = a[4 * i + k];
  for (int i = 0; i < 16; ++i) out[i] = r[i];
}

// u0 on bit 0 and u1 on bit 1 of the 4 x 4 index (u1 (x) u0).
void kron2(const cd u0[4], const cd u1[4], cd out[16]) {
  for (int i = 0; i < 4; ++i)
    for (int k = 0; k < 4; ++k) out[4 * i + k] = u0[2 * (i & 1) + (k & 1)] * u1[2 * (i >> 1) + (k >> 1)];
}

// A two-qubit gate on (q0 -> bit 0, q1 -> bit 1); CX: q0 controls.
hs_status gate4(const Gate& g, cd out[16]) {
  for (int i = 0; i < 16; ++i) out[i] = 0;
  switch (g.kind) {
    case HS_CX: out[0] = out[4 * 2 + 2] = out[4 * 1 + 3] = out[4 * 3 + 1] = 1; break;
    case HS_CZ: out[0] = out[5] = out[10] = 1; out[15] = -1; break;
    case HS_CP: out[0] = out[5] = out[10] = 1; out[15] = cd(cos(g.p[0]), sin(g.p[0])); break;
    case HS_SWAP: out[0] = out[4 * 1 + 2] = out[4 * 2 + 1] = out[15] = 1; break;
    default: return fail(HS_E_ARG, "unknown two-qubit kind %d", g.kind);
  }
  return HS_OK;
}

void set_u2(HostOp* op, const cd m[16]) {
  for (int i = 0; i < 16; ++i) {
    op->c[2 * i] = m[i].real();
    op->c[2 * i + 1] = m[i].imag();
  }
}

void get_u2(const HostOp& op, cd m[16]) {
  for (int i = 0; i < 16; ++i) m[i] = cd(op.c[2 * i], op.c[2 * i + 1]);
}

// Left-multiply the U2 op by `m`, given on (r0 -> bit 0, r1 -> bit 1).
void u2_apply_after(HostOp* op, int r0, const cd m[16]) {
  cd mm[16], cur[16];
  if (r0 == op->b0) {
    for (int i = 0; i < 16; ++i) mm[i] = m[i];
  } else {
    swap_bits4(m, mm);
  }
  get_u2(*op, cur);
  matmul4(mm, cur, cur);
  set_u2(op, cur);
}

// Multiply the part's scalar S into the op where that adds the fewest
// instructions (a dense 4 x 4 takes it for nothing, diag(1, d) costs the
// other half of the amplitudes), or append it as a diagonal.
void fold_scalar(const cl& S, std::vector<HostOp>* ops) {
  if (clean(S) == cl(1, 0)) return;
  int at = -1, cost = 8;  // a diagonal of its own: 8 instructions a pair
  cd k[4], best[4] = {to_cd(S), 0, 0, to_cd(S)};
  for (int i = 0; i < (int)ops->size(); ++i) {
    HostOp& op = (*ops)[i];
    if (op.kind == OP_U2) {
      cd m[16];
      get_u2(op, m);
      for (cd& z : m) z = to_cd(cl(z) * S);
      set_u2(&op, m);
      return;
    }
    if (!op_matrix(op, k)) continue;
    const int before = op.kind == OP_X ? 0 : pair_cost(k);
    for (cd& z : k) z = to_cd(clean(cl(z) * S));
    if (pair_cost(k) - before < cost) {
      cost = pair_cost(k) - before;
      at = i;
      for (int j = 0; j < 4; ++j) best[j] = k[j];
    }
  }
  std::vector<HostOp> made;
  emit_1q(at < 0 ? 0 : (*ops)[at].b0, best, &made);
  if (at < 0) ops->insert(ops->end(), made.begin(), made.end());
  else if (!made.empty()) (*ops)[at] = made[0];
  else (*ops)[at].kind = OP_D, (*ops)[at].c[0] = (*ops)[at].c[2] = 1, (*ops)[at].c[1] = (*ops)[at].c[3] = 0;
}

// Register-stage cut: the seed of the orders tried per part.
constexpr uint64_t kStageSeed = 0x5eed;

}  // namespace

bool part_fits(int n, uint64_t mask, const CompileOptions& opt) {
  const int C = std::min(opt.contig, n);
  return __builtin_popcountll(mask | ((uint64_t(1) << C) - 1)) <= max_tile_qubits(opt);
}

hs_status compile_part(int n, const std::vector<Gate>& pg, const CompileOptions& opt,
                       CompiledPart* out) {
  if (pg.empty()) return fail(HS_E_ARG, "empty part");
  // what the gates need in the tile, and in the registers of their stage
  const std::vector<Gate> stand_ins = opt.conditions ? active_gates(pg) : std::vector<Gate>();
  const std::vector<Gate>& act = opt.conditions ? stand_ins : pg;
  uint64_t S = 0;
  for (const Gate& g : act) S |= g.mask();
  const int C = std::min(opt.contig, n);
  const uint64_t need = S | ((C >= 64) ? ~0ull : ((1ull << C) - 1));
  int m = std::max(__builtin_popcountll(need),
                   std::min(n, std::max(kLaneBits + opt.rb,
                                        std::min(opt.min_tile, max_tile_qubits(opt)))));
  if (m > max_tile_qubits(opt))
    return fail(HS_E_UNSUPPORTED, "part needs a %d-qubit tile; the kernel holds at most %d",
                m, max_tile_qubits(opt));
  const int rb = std::min(opt.rb, m);
  const int lb = std::min(kLaneBits, m - rb);
  const int wb = m - rb - lb;
  if (wb > opt.max_wb) return fail(HS_E_UNSUPPORTED, "tile needs %d wave bits", wb);

  // tile qubits: S plus the lowest qubits outside S
  uint64_t T = S;
  for (int q = 0; q < n && __builtin_popcountll(T) < m; ++q) T |= 1ull << q;
  int8_t tq[kMaxTile] = {0};
  int bit_of[64];
  for (int q = 0, t = 0; q < n; ++q) {
    bit_of[q] = -1;
    if (T >> q & 1) {
      tq[t] = (int8_t)q;
      bit_of[q] = t++;
    }
  }

  // Second level of the multi-level partition (Sec. IV): the part's gates
  // are cut into register stages of at most rb qubits by the DFS
  // partitioner (Sec. IV.B.2; its first trial is the circuit order) and by
  // the greedy one; the cut with fewer stages, hence fewer LDS re-layouts,
  // is kept (DFS on ties).  Stages run in creation order, a topological
  // order of the stage graph; a stage's gates keep circuit order.
  struct Stage {
    uint32_t bits = 0;
    std::vector<int> gates;
  };
  for (const Gate& g : act)
    if (g.arity() > rb) return fail(HS_E_UNSUPPORTED, "gate wider than the register stage");
  std::vector<int32_t> stage_of, greedy_of;
  const Dag pdag = opt.conditions ? commuting_dag(n, pg) : build_dag(pg);
  int nst = partition_dfs(act, pdag, rb, kStageSeed, opt.stage_trials, &stage_of);
  const int ngr = partition_greedy(act, pdag, rb, kStageSeed, opt.stage_trials, &greedy_of);
  if (ngr < nst) {
    nst = ngr;
    stage_of.swap(greedy_of);
  }
  std::vector<Stage> st(nst);
  for (int i = 0; i < (int)pg.size(); ++i)
    for (uint64_t qs = act[i].mask(); qs; qs &= qs - 1) st[stage_of[i]].bits |= 1u << bit_of[__builtin_ctzll(qs)];

  out->desc = PartDesc{};
  out->desc.m = m;
  out->desc.lb = lb;
  out->desc.wb = wb;
  out->desc.rb = rb;
  out->desc.tiles = uint64_t(1) << (n - m);
  std::memcpy(out->desc.tq, tq, sizeof tq);
  out->rb_kernel = rb;
  out->stages.clear();
  out->ops.clear();

  std::vector<Layout> lay;
  uint32_t prev_regs = pad_regs(0u, m, rb);  // the registers of a fresh load layout
  for (const Stage& s : st) {
    const uint32_t regs = pad_regs(s.bits, m, rb, prev_regs);
    lay.push_back(make_layout(m, lb, wb, regs));
    prev_regs = regs;
  }
  auto is_reg = [&](int q, int s) {
    for (int r = 0; r < rb; ++r)
      if (q >= 0 && lay[s].pos[lb + wb + r] == bit_of[q]) return true;
    return false;
  };
  // A gate that needs no register bit goes to the first stage, up to those of
  // the gates that follow it, where one of its qubits is one: it then
  // multiplies half of the registers instead of the lane's factor.
  for (int i = (int)pg.size() - 1; i >= 0 && opt.conditions; --i) {
    if (act[i].mask()) continue;
    int limit = nst - 1;
    for (int j : pdag.succ[i]) limit = std::min(limit, (int)stage_of[j]);
    for (int s = stage_of[i]; s <= limit; ++s)
      if (is_reg(pg[i].q0, s) || is_reg(pg[i].q1, s)) {
        stage_of[i] = s;
        break;
      }
  }
  for (int i = 0; i < (int)pg.size(); ++i) st[stage_of[i]].gates.push_back(i);
  // load and store layouts: lanes on tile bits 0..lb-1 (contiguous global runs)
  auto io_layout = [&](const Layout& near) {
    if (lanes_are_low(near, lb) || low_run(near, lb) >= std::min(opt.min_run, lb)) return near;
    return make_layout(m, lb, wb, pad_regs(0u, m, rb));
  };
  const Layout load = io_layout(lay.front());
  const Layout store = io_layout(lay.back());

  auto push_entry = [&](const Layout& L, const Layout* prev) {
    StageDesc e{};
    std::memcpy(e.pos, L.pos, sizeof e.pos);
    e.transition = (prev && !same_layout(L, *prev, m)) ? 1 : 0;
    e.op_begin = e.op_end = (int)out->ops.size();
    out->stages.push_back(e);
    return &out->stages.back();
  };
  int trips = 0;
  push_entry(load, nullptr);
  const Layout* prev = &load;
  // One-qubit runs pending per tile bit.  A run stays pending over a change
  // of stage when a later stage has gates on its bit.
  cl pend[kMaxTile][4];
  bool has[kMaxTile] = {false};
  int last_stage[kMaxTile];
  for (int t = 0; t < kMaxTile; ++t) last_stage[t] = -1;
  for (size_t s = 0; s < st.size(); ++s)
    for (int t = 0; t < m; ++t)
      if (st[s].bits >> t & 1) last_stage[t] = (int)s;
  cl scale = 1;  // the part's scalar S
  const int A = 1 << rb;
  const cd I2[4] = {1, 0, 0, 1};
  for (size_t s = 0; s < st.size(); ++s) {
    StageDesc* e = push_entry(lay[s], prev);
    trips += e->transition;
    // register index of each tile bit in this layout
    int reg_of[kMaxTile];
    for (int t = 0; t < kMaxTile; ++t) reg_of[t] = -1;
    for (int r = 0; r < rb; ++r) reg_of[lay[s].pos[lb + wb + r]] = r;
    // latest op on each tile bit in this stage (-1: none): a dense 4 x 4 op
    // that is still the latest on a bit absorbs later gates there
    int last[kMaxTile];
    for (int t = 0; t < kMaxTile; ++t) last[t] = -1;
    auto open_u2 = [&](int t) { return opt.fuse2 && last[t] >= 0 && out->ops[last[t]].kind == OP_U2; };
    auto pending = [&](int t, cd u[4]) {
      for (int j = 0; j < 4; ++j) u[j] = to_cd(pend[t][j]);
    };
    // Phases on a register bit under conditions commute until something mixes
    // the bit's pairs.  They are collected until then: one is applied as it is,
    // several are multiplied into the lane's factor (six instructions each
    // instead of two an amplitude) and applied together.
    std::vector<HostOp> phases[kMaxTile];
    auto apply_phases = [&](int t) {
      std::vector<HostOp>& ph = phases[t];
      if (ph.empty()) return;
      if (ph.size() == 1) {
        out->ops.push_back(ph[0]);
      } else {
        HostOp all{};
        all.kind = OP_GA;
        all.b0 = ph[0].b0;
        all.b1 = 1;
        for (HostOp& op : ph) {
          op.kind = OP_F;
          if (op.c[1] != 0) all.b1 = 0;
          out->ops.push_back(op);
        }
        out->ops.push_back(all);
      }
      ph.clear();
    };
    // run what is pending on bit t, as far as `role` does not let it wait
    auto flush = [&](int t, Role role) {
      if (!has[t]) return;
      if (open_u2(t)) {
        has[t] = false;
        HostOp& o = out->ops[last[t]];
        cd m4[16];
        cd run[4];
        pending(t, run);
        kron2(reg_of[t] == o.b0 ? run : I2, reg_of[t] == o.b0 ? I2 : run, m4);
        u2_apply_after(&o, o.b0, m4);
        return;
      }
      Split f;
      if (opt.plain) std::copy(pend[t], pend[t] + 4, f.K);
      else f = split_gate(pend[t], role);
      scale = mul(scale, f.S);
      for (int j = 0; j < 4; ++j) pend[t][j] = f.L[j];
      has[t] = !is_identity(f.L);
      if (is_identity(f.K)) return;
      if (std::abs(scale) < 1.0 / kMaxGrowth) {
        for (cl& z : f.K) z = mul(z, scale);
        scale = 1;
      }
      const size_t before = out->ops.size();
      if (!(f.K[1] == cl(0, 0) && f.K[2] == cl(0, 0))) apply_phases(t);
      const cd k[4] = {to_cd(f.K[0]), to_cd(f.K[1]), to_cd(f.K[2]), to_cd(f.K[3])};
      emit_1q(reg_of[t], k, &out->ops);
      if (out->ops.size() > before) last[t] = (int)before;
    };
    // interpreter cost of what a two-qubit gate with this role makes run
    auto pend_cost = [&](int t, Role role) {
      if (!has[t] || open_u2(t)) return 0;
      if (opt.plain) {
        cd run[4];
        pending(t, run);
        return op_cost(kind_1q(run), A, true);
      }
      const int c = split_gate(pend[t], role).cost;
      return c ? c * A / 2 + 10 : 0;
    };
    // the stage's next two-qubit gate on each of a gate's bits (-1: none)
    std::vector<std::array<int, 2>> next(opt.fuse2 ? st[s].gates.size() : 0);
    int upcoming[kMaxTile];
    for (int t = 0; t < kMaxTile; ++t) upcoming[t] = -1;
    for (int o = (int)next.size() - 1; o >= 0; --o) {
      const Gate& g = pg[st[s].gates[o]];
      if (g.arity() == 1) continue;
      const int t0 = bit_of[g.q0], t1 = bit_of[g.q1];
      next[o] = {upcoming[t0], upcoming[t1]};
      upcoming[t0] = upcoming[t1] = o;
    }
    // where the value of a qubit that is no register bit is found
    auto cond_of = [&](int q) {
      if (bit_of[q] < 0) return kOuterBit + q;
      int c = 0;
      while (lay[s].pos[c] != bit_of[q]) ++c;
      return c;
    };
    auto in_reg = [&](int q) { return bit_of[q] >= 0 && reg_of[bit_of[q]] >= 0; };
    // factors of all amplitudes of a lane; they commute with everything in the
    // stage and are applied together at its end
    std::vector<HostOp> factors;
    auto put_factor = [&](int cond, int cond2, const cl& d) {
      HostOp op{};
      op.kind = OP_F;
      op.cond = cond;
      op.cond2 = cond2;
      const cd z = to_cd(clean(d));
      op.c[0] = z.real();
      op.c[1] = z.imag();
      factors.push_back(op);
    };
    for (size_t o = 0; o < st[s].gates.size(); ++o) {
      const Gate& g = pg[st[s].gates[o]];
      const int t0 = bit_of[g.q0];
      if (opt.conditions && g.arity() == 1 && t0 < 0) {  // a diagonal on a qubit outside the tile
        scale = mul(scale, g.u[0]);
        put_factor(cond_of(g.q0), kNoCond, mul(g.u[3], inv(g.u[0])));
        continue;
      }
      // CZ, CP or CX with a qubit that is no register bit; what is pending on
      // that qubit is diagonal and commutes
      if (opt.conditions && g.arity() == 2 && !(in_reg(g.q0) && in_reg(g.q1))) {
        const cl d = g.kind == HS_CZ ? cl(-1, 0) : cl(cos(g.p[0]), sin(g.p[0]));
        if (!in_reg(g.q0) && !in_reg(g.q1)) {
          put_factor(cond_of(g.q0), cond_of(g.q1), d);
          continue;
        }
        const int q = in_reg(g.q1) ? g.q1 : g.q0, other = q == g.q0 ? g.q1 : g.q0;
        flush(bit_of[q], g.kind == HS_CX ? kRoleX : kRoleZ);
        HostOp op{};
        op.kind = g.kind == HS_CX ? OP_CXC : OP_CPC;
        op.b0 = reg_of[bit_of[q]];
        op.b1 = -1;
        op.cond = cond_of(other);
        op.cond2 = kNoCond;
        op.c[0] = to_cd(d).real();
        op.c[1] = to_cd(d).imag();
        if (op.kind == OP_CPC) {
          phases[bit_of[q]].push_back(op);
        } else {
          apply_phases(bit_of[q]);
          out->ops.push_back(op);
        }
        continue;
      }
      if (g.arity() == 1) {
        cd u[4];
        gate_matrix(g, u);
        if (has[t0] && opt.plain) {
          cd run[4];
          pending(t0, run);
          matmul2(u, run, run);
          for (int j = 0; j < 4; ++j) pend[t0][j] = run[j];
        } else if (has[t0]) {
          const cl v[4] = {u[0], u[1], u[2], u[3]};
          matmul2(v, pend[t0], pend[t0]);
        } else {
          for (int j = 0; j < 4; ++j) pend[t0][j] = u[j];
          has[t0] = true;
        }
        continue;
      }
      const int t1 = bit_of[g.q1];
      const Role role1 = g.kind == HS_CX ? kRoleX : kRoleZ;
      if (opt.fuse2) {
        cd m4[16], pm[16];
        if (hs_status rc = gate4(g, m4)) return rc;
        cd run0[4], run1[4];
        pending(t0, run0);
        pending(t1, run1);
        kron2(has[t0] ? run0 : I2, has[t1] ? run1 : I2, pm);
        matmul4(m4, pm, m4);  // the pending one-qubit gates come first
        const int r0 = reg_of[t0], r1 = reg_of[t1];
        const int gk = g.kind == HS_CX ? OP_CX : g.kind == HS_CZ ? OP_CZ : g.kind == HS_CP ? OP_CP : OP_SWAP;
        if (open_u2(t0) && last[t0] == last[t1]) {  // same pair: absorb
          u2_apply_after(&out->ops[last[t0]], r0, m4);
          has[t0] = has[t1] = false;
          continue;
        }
        // what a 4 x 4 op also saves: the bits' next gate, if it is on the
        // same pair, or the run that a bit's last gate leaves pending
        int saved = 0;
        if (opt.plain) saved = 0;
        else if (next[o][0] >= 0 && next[o][0] == next[o][1]) saved = 2 * (4 * A + 10) + op_cost(gk, A, false);
        else
          for (int j = 0; j < 2; ++j)
            if (next[o][j] < 0 && last_stage[j ? t1 : t0] <= (int)s) saved += 6 * A + 10;
        if (op_cost(OP_U2, A, opt.plain) <
            pend_cost(t0, kRoleZ) + pend_cost(t1, role1) + op_cost(gk, A, opt.plain) + saved) {
          HostOp op{};
          op.kind = OP_U2;
          op.b0 = std::min(r0, r1);
          op.b1 = std::max(r0, r1);
          cd mm[16];
          if (r0 < r1) {
            for (int j = 0; j < 16; ++j) mm[j] = m4[j];
          } else {
            swap_bits4(m4, mm);
          }
          set_u2(&op, mm);
          has[t0] = has[t1] = false;
          last[t0] = last[t1] = (int)out->ops.size();
          out->ops.push_back(op);
          continue;
        }
      }
      if (g.kind == HS_SWAP && !opt.plain) {  // what is pending moves with the qubits
        std::swap(has[t0], has[t1]);
        for (int j = 0; j < 4; ++j) std::swap(pend[t0][j], pend[t1][j]);
      } else {
        flush(t0, kRoleZ);
        flush(t1, role1);
      }
      if (g.kind == HS_SWAP) apply_phases(t0);
      if (g.kind == HS_SWAP || g.kind == HS_CX) apply_phases(t1);
      last[t0] = last[t1] = (int)out->ops.size();
      HostOp op{};
      op.b0 = reg_of[t0];
      op.b1 = reg_of[t1];
      switch (g.kind) {
        case HS_CX: op.kind = OP_CX; break;
        case HS_CZ: op.kind = OP_CZ; break;
        case HS_CP:
          op.kind = OP_CP;
          op.c[0] = cos(g.p[0]);
          op.c[1] = sin(g.p[0]);
          break;
        case HS_SWAP: op.kind = OP_SWAP; break;
        default: return fail(HS_E_ARG, "unknown two-qubit kind %d", g.kind);
      }
      out->ops.push_back(op);
    }
    for (int r = 0; r < rb; ++r) {
      const int t = lay[s].pos[lb + wb + r];
      const bool end = s + 1 == st.size();
      if (opt.conditions) flush(t, end ? kRoleLast : kRoleZ);  // only diagonals wait for another stage
      else if (open_u2(t) || last_stage[t] <= (int)s || opt.plain) flush(t, kRoleLast);
    }
    for (int t = 0; t < m; ++t) apply_phases(t);
    if (s + 1 == st.size() && opt.conditions) {
      for (int t = 0; t < m; ++t)
        if (has[t]) {  // a diagonal on a lane or wave bit
          scale = mul(scale, pend[t][0]);
          put_factor(cond_of(tq[t]), kNoCond, mul(pend[t][3], inv(pend[t][0])));
        }
      if (!factors.empty() && clean(scale) != cl(1, 0)) {
        put_factor(kNoCond, kNoCond, scale);
        scale = 1;
      }
    }
    if (!factors.empty()) {
      HostOp all{};
      all.kind = OP_FA;
      all.b0 = 1;
      for (const HostOp& op : factors) {
        if (op.c[1] != 0) all.b0 = 0;
        out->ops.push_back(op);
      }
      out->ops.push_back(all);
    }
    if (s + 1 == st.size()) fold_scalar(scale, &out->ops);
    out->stages.back().op_end = (int)out->ops.size();
    prev = &lay[s];
  }
  StageDesc* e = push_entry(store, prev);
  trips += e->transition;
  out->desc.n_stages = (int)out->stages.size();
  out->desc.lds_bytes = 0;  // set per dtype at upload
  out->lds_round_trips = trips;
  out->work = 0;
  for (const HostOp& op : out->ops) out->work += op_work(op);
  return HS_OK;
}

}  // namespace hisv

namespace hisv {

// ---- fused path: one dense unitary per part -----------------------------------
//
// U_p = product of the part's gates (circuit order), built in FP64 by
// applying each gate to every column of the identity as a state of the
// part's qubits (inner slot b = the b-th smallest part qubit, the slot order
// of Alg. 1's worked example).  Parts narrower than 4 qubits take the lowest
// other qubits as extra slots (U acts as the identity on them).
hs_status compile_fused(int n, const std::vector<Gate>& pg, FusedPart* out) {
  uint64_t S = 0;
  for (const Gate& g : pg) S |= g.mask();
  for (int q = 0; q < n && __builtin_popcountll(S) < 4; ++q) S |= 1ull << q;
  const int w = __builtin_popcountll(S);
  if (w > kMaxFusedQubits)
    return fail(HS_E_UNSUPPORTED, "fused path takes parts of at most %d qubits (got %d)", kMaxFusedQubits, w);
  if (n < w + 4) return fail(HS_E_UNSUPPORTED, "fused path needs n >= %d", w + 4);
  FusedPart f;
  f.w = w;
  f.m = w + 4;
  f.tiles = uint64_t(1) << (n - f.m);
  int slot[64];
  for (int q = 0, b = 0; q < n; ++q) {
    slot[q] = -1;
    if (S >> q & 1) {
      f.sq[b] = (int8_t)q;
      slot[q] = b++;
    }
  }
  uint64_t T = S;
  for (int q = 0, c = 0; q < n && c < 4; ++q)
    if (!(S >> q & 1)) {
      f.pq[c++] = (int8_t)q;
      T |= 1ull << q;
    }
  for (int q = 0, t = 0; q < n; ++q)
    if (T >> q & 1) f.tq[t++] = (int8_t)q;
  const int R = 1 << w;
  f.u.assign((size_t)R * R, cd(0.0, 0.0));
  for (int i = 0; i < R; ++i) f.u[(size_t)i * R + i] = 1.0;
  // apply a gate to every column: column c is a 2^w state vector
  for (const Gate& g : pg) {
    const int a = slot[g.q0];
    if (g.arity() == 1) {
      cd m[4];
      gate_matrix(g, m);
      // row by row, in real arithmetic (a complex product of std::complex
      // checks for NaN: 128 x 128 with 100 gates 25 ms against 3 ms)
      for (int r0 = 0; r0 < R; ++r0) {
        if (r0 >> a & 1) continue;
        double* x = reinterpret_cast<double*>(&f.u[(size_t)r0 * R]);
        double* y = reinterpret_cast<double*>(&f.u[(size_t)(r0 | (1 << a)) * R]);
        const double ar = m[0].real(), ai = m[0].imag(), br = m[1].real(), bi = m[1].imag();
        const double cr = m[2].real(), ci = m[2].imag(), dr = m[3].real(), di = m[3].imag();
        for (int c = 0; c < 2 * R; c += 2) {
          const double xr = x[c], xi = x[c + 1], yr = y[c], yi = y[c + 1];
          x[c] = (ar * xr - ai * xi) + (br * yr - bi * yi);
          x[c + 1] = (ar * xi + ai * xr) + (br * yi + bi * yr);
          y[c] = (cr * xr - ci * xi) + (dr * yr - di * yi);
          y[c + 1] = (cr * xi + ci * xr) + (dr * yi + di * yr);
        }
      }
      continue;
    }
    const int b = slot[g.q1];
    const cd ph = g.kind == HS_CP ? std::polar(1.0, g.p[0]) : cd(-1.0, 0.0);
    for (int r = 0; r < R; ++r) {
      const bool ba = r >> a & 1, bb = r >> b & 1;
      cd* v = &f.u[(size_t)r * R];
      switch (g.kind) {
        case HS_CX:  // control a, target b: swap the pair with a = 1
          if (ba && !bb) std::swap_ranges(v, v + R, &f.u[(size_t)(r | (1 << b)) * R]);
          break;
        case HS_CZ:
        case HS_CP:
          if (ba && bb)
            for (int c = 0; c < R; ++c)
              v[c] = cd(v[c].real() * ph.real() - v[c].imag() * ph.imag(),
                        v[c].real() * ph.imag() + v[c].imag() * ph.real());
          break;
        case HS_SWAP:
          if (ba && !bb) std::swap_ranges(v, v + R, &f.u[(size_t)(r ^ (1 << a) ^ (1 << b)) * R]);
          break;
        default: return fail(HS_E_ARG, "unknown two-qubit kind %d", g.kind);
      }
    }
  }
  *out = std::move(f);
  return HS_OK;
}

}  // namespace hisv

namespace hisv {

// Relative cost of a part or sweep on the interpreter kernel (one HBM sweep of
// the state = 1), fitted to the timings of 1,058 of them on 28-qubit complex64
// and 27-qubit complex128 states (random, layered, dressed-pair and QFT
// circuits, tiles of 9 to 14 qubits; mean |log error| 0.08): a smooth maximum
// of the sweep (+0.04 per LDS re-layout) and the arithmetic, 0.007 / 0.006
// sweep (complex64 / complex128) per vector instruction an amplitude (op_work)
// and 0.02 per register op.  A tile that fills the CU overlaps neither with
// another tile.  Used by AUTO only.
double lds_part_alu(const CompiledPart& cp, hs_dtype dt) {
  return (dt == HS_C64 ? 0.007 : 0.006) * cp.work + 0.02 * (double)cp.ops.size();
}

double lds_part_cost(const CompiledPart& cp, hs_dtype dt) {
  const bool f32 = dt == HS_C64;
  const double mem = 0.9 + 0.04 * cp.lds_round_trips, alu = lds_part_alu(cp, dt);
  return (cp.desc.m >= (f32 ? 14 : 13) ? 1.5 : 1.0) * std::sqrt(mem * mem + alu * alu);
}

// The same for the specialized kernels: the sweep (+0.04 per LDS re-layout) or
// 0.007 sweep per vector instruction an amplitude, a tile that fills the CU 15%
// (complex64) or 30% more.  Register permutations (X, CX, SWAP) are free
// (compile-time renames).  870 timings as above, mean |log error| 0.09 / 0.07.
double spec_part_cost(const CompiledPart& cp, hs_dtype dt) {
  const bool f32 = dt == HS_C64;
  const double mem = 0.9 + 0.04 * cp.lds_round_trips;
  const double alu = 0.007 * cp.work;
  return (cp.desc.m < (f32 ? 14 : 13) ? 1.0 : f32 ? 1.15 : 1.3) * std::cbrt(mem * mem * mem + alu * alu * alu);
}

// The fused kernels do 8 * 2^w flops per amplitude on matrix cores against
// 2 * s bytes of HBM traffic (s = 8 or 16 bytes per amplitude).  Per-part
// timings of dressed-pair circuits on 28 qubits, in sweeps: w = 6 and 7 are
// matrix-core bound.  A complex64 part pays for each of qubits 0..3 that it
// holds (the 16 columns of a wave are then not one contiguous run; complex128
// rows are a cache line each either way, until all four are held).
double fused_part_cost(int n, uint64_t mask, hs_dtype dt) {
  static const double c64[8] = {0, 0, 0, 0, 1.0, 1.02, 1.42, 2.6};
  static const double c128[8] = {0, 0, 0, 0, 0.93, 0.97, 1.21, 2.66};
  for (int q = 0; q < n && __builtin_popcountll(mask) < 4; ++q) mask |= uint64_t(1) << q;  // as compile_fused widens
  const int w = __builtin_popcountll(mask);
  if (w < 4 || w > kMaxFusedQubits || n < w + 4) return 1e30;
  const int low = __builtin_popcountll(mask & 15);
  if (dt == HS_C64) return c64[w] + 0.1 * low;
  return c128[w] + (low == 4 ? 0.15 : 0.0);
}

}  // namespace hisv
