// kernels.hip -- gfx950 kernels of the partitioned state-vector path.
//
//   part_pass_kernel   Alg. 1 (Sec. III.C) for one part, in place: each
//                      workgroup gathers tiles (one outer setting each) from
//                      HBM into registers with coalesced loads, runs the
//                      part's register stages (LDS re-layouts in between) and
//                      scatters the tile back -- one HBM read and one write
//                      per amplitude per part.
//   fused_pass_kernel, fused_lds_kernel  a part's dense unitary on the matrix
//                      cores.
//   gate_pass_1q/diag/2q  the non-hierarchical case (Sec. III.A-B): one sweep
//                      per gate, over the amplitudes it changes.
//   set_basis, norm, probabilities/amplitude readout, copy probe.
//
// Amplitudes are interleaved complex (float2 / double2), index bit q =
// qubit q.  complex64 states compute in FP32, complex128 in FP64; the norm
// and probabilities are accumulated in FP64 for both.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstring>
#include <map>
#include <type_traits>

#include "hisv_internal.h"

namespace hisv {

template <typename T>
struct alignas(2 * sizeof(T)) cplx {
  T x, y;
};

// ---------------------------------------------------------------------------
// register operations (one lane's 2^RB amplitudes; bit positions compile-time)
// ---------------------------------------------------------------------------
template <int N>
using IC = std::integral_constant<int, N>;

template <int RB, typename F>
__device__ __forceinline__ void for_bit(int b, F&& f) {
  switch (b) {
    case 0: if constexpr (RB > 0) { f(IC<0>{}); break; } else __builtin_unreachable();
    case 1: if constexpr (RB > 1) { f(IC<1>{}); break; } else __builtin_unreachable();
    case 2: if constexpr (RB > 2) { f(IC<2>{}); break; } else __builtin_unreachable();
    case 3: if constexpr (RB > 3) { f(IC<3>{}); break; } else __builtin_unreachable();
    case 4: if constexpr (RB > 4) { f(IC<4>{}); break; } else __builtin_unreachable();
    case 5: if constexpr (RB > 5) { f(IC<5>{}); break; } else __builtin_unreachable();
    default: __builtin_unreachable();
  }
}

template <int RB, typename F>
__device__ __forceinline__ void for_pair(int b0, int b1, F&& f) {
  for_bit<RB>(b0, [&](auto B0) __attribute__((always_inline)) {
    for_bit<RB>(b1, [&](auto B1) __attribute__((always_inline)) {
      if constexpr (decltype(B0)::value != decltype(B1)::value) f(B0, B1);
      else __builtin_unreachable();
    });
  });
}

// A lane's 2^RB amplitudes (re at 2j, im at 2j+1).  Every access below has
// a compile-time index, so the array is split into independent scalars that
// stay in VGPRs.  (A vector value did the same but must occupy one
// contiguous register range, which cost extra register copies per op:
// 1,643 against 1,109 moves in the complex64 kernel, 2.4% on a 28-qubit
// layered circuit.)
template <typename T, int RB>
struct RegV {
  T v[2 << RB];
  __device__ __forceinline__ T& operator[](int i) { return v[i]; }
  __device__ __forceinline__ const T& operator[](int i) const { return v[i]; }
};

// Every register operation reads one register set (a) and writes every
// register of another (b).  The interpreter alternates the two sets from op
// to op, so the switch over op kinds leaves its results where the next op
// reads them.  (Updating one set in place made the compiler assign each
// case's results to fresh registers and copy the whole set back after
// every op: 32 moves per op for complex64 with 16 amplitudes a lane.)
template <typename T>
__device__ __forceinline__ void cmul(cplx<T>& v, T cr, T ci) {
  const cplx<T> p = v;
  v.x = p.x * cr - p.y * ci;
  v.y = p.x * ci + p.y * cr;
}

// A register copy.  The empty asm keeps the compiler from merging the
// copies of different cases (different register indices) into copies
// through a selected address, which would move the register set to memory.
template <typename T, int RB>
__device__ __forceinline__ void cp_at(const RegV<T, RB>& a, RegV<T, RB>& b, int j, int k) {
  T x = a[2 * k], y = a[2 * k + 1];
  asm volatile("" : "+v"(x), "+v"(y));
  b[2 * j] = x;
  b[2 * j + 1] = y;
}

template <typename T, int RB>
__device__ __forceinline__ void cmul_at(const RegV<T, RB>& a, RegV<T, RB>& b, int j, T cr, T ci) {
  const T px = a[2 * j], py = a[2 * j + 1];
  b[2 * j] = px * cr - py * ci;
  b[2 * j + 1] = px * ci + py * cr;
}

template <typename T, int RB, int B>
__device__ __forceinline__ void r_u(const RegV<T, RB>& a, RegV<T, RB>& b, const T* __restrict__ c) {
  const T u00r = c[0], u00i = c[1], u01r = c[2], u01i = c[3];
  const T u10r = c[4], u10i = c[5], u11r = c[6], u11i = c[7];
#pragma unroll
  for (int j = 0; j < (1 << RB); ++j) {
    if (j & (1 << B)) continue;
    const int k = j | (1 << B);
    const T px = a[2 * j], py = a[2 * j + 1], qx = a[2 * k], qy = a[2 * k + 1];
    b[2 * j] = u00r * px - u00i * py + u01r * qx - u01i * qy;
    b[2 * j + 1] = u00r * py + u00i * px + u01r * qy + u01i * qx;
    b[2 * k] = u10r * px - u10i * py + u11r * qx - u11i * qy;
    b[2 * k + 1] = u10r * py + u10i * px + u11r * qy + u11i * qx;
  }
}

template <typename T, int RB, int B>
__device__ __forceinline__ void r_r(const RegV<T, RB>& a, RegV<T, RB>& b, const T* __restrict__ c) {
  const T u00 = c[0], u01 = c[1], u10 = c[2], u11 = c[3];
#pragma unroll
  for (int j = 0; j < (1 << RB); ++j) {
    if (j & (1 << B)) continue;
    const int k = j | (1 << B);
    const T px = a[2 * j], py = a[2 * j + 1], qx = a[2 * k], qy = a[2 * k + 1];
    b[2 * j] = u00 * px + u01 * qx;
    b[2 * j + 1] = u00 * py + u01 * qy;
    b[2 * k] = u10 * px + u11 * qx;
    b[2 * k + 1] = u10 * py + u11 * qy;
  }
}

// The scaled forms of a 2x2 (unit entries need no multiplication): 8 FMAs a
// pair for K and P, 4 for KR and KI, 4 adds for H, 12 for W, against 16 for U
// and 8 for R.
template <typename T, int RB, int B, int KIND>
__device__ __forceinline__ void r_k(const RegV<T, RB>& a, RegV<T, RB>& b, const T* __restrict__ c) {
  const T c0 = c[0], c1 = c[1], c2 = c[2], c3 = c[3], c4 = c[4], c5 = c[5];
#pragma unroll
  for (int j = 0; j < (1 << RB); ++j) {
    if (j & (1 << B)) continue;
    const int k = j | (1 << B);
    const T px = a[2 * j], py = a[2 * j + 1], qx = a[2 * k], qy = a[2 * k + 1];
    T rx, ry, sx, sy;
    if constexpr (KIND == OP_KR) {
      rx = px + c0 * qx; ry = py + c0 * qy;
      sx = qx + c1 * px; sy = qy + c1 * py;
    } else if constexpr (KIND == OP_KI) {
      rx = px - c0 * qy; ry = py + c0 * qx;
      sx = qx - c1 * py; sy = qy + c1 * px;
    } else if constexpr (KIND == OP_H) {
      rx = px + qx; ry = py + qy;
      sx = px - qx; sy = py - qy;
    } else if constexpr (KIND == OP_P) {
      rx = qx + c0 * px - c1 * py; ry = qy + c0 * py + c1 * px;
      sx = px + c2 * qx - c3 * qy; sy = py + c2 * qy + c3 * qx;
    } else {
      rx = px + c0 * qx - c1 * qy; ry = py + c0 * qy + c1 * qx;
      if constexpr (KIND == OP_K) {
        sx = qx + c2 * px - c3 * py; sy = qy + c2 * py + c3 * px;
      } else {  // OP_W
        sx = c2 * px - c3 * py + c4 * qx - c5 * qy;
        sy = c2 * py + c3 * px + c4 * qy + c5 * qx;
      }
    }
    b[2 * j] = rx;
    b[2 * j + 1] = ry;
    b[2 * k] = sx;
    b[2 * k + 1] = sy;
  }
}

template <typename T, int RB, int B>
__device__ __forceinline__ void r_d(const RegV<T, RB>& a, RegV<T, RB>& b, const T* __restrict__ c) {
  const T d0r = c[0], d0i = c[1], d1r = c[2], d1i = c[3];
#pragma unroll
  for (int j = 0; j < (1 << RB); ++j) {
    if (j & (1 << B)) cmul_at<T, RB>(a, b, j, d1r, d1i);
    else cmul_at<T, RB>(a, b, j, d0r, d0i);
  }
}

template <typename T, int RB, int B>
__device__ __forceinline__ void r_d1(const RegV<T, RB>& a, RegV<T, RB>& b, const T* __restrict__ c) {
  const T d1r = c[0], d1i = c[1];
#pragma unroll
  for (int j = 0; j < (1 << RB); ++j) {
    if (j & (1 << B)) cmul_at<T, RB>(a, b, j, d1r, d1i);
    else cp_at<T, RB>(a, b, j, j);
  }
}

template <typename T, int RB, int B>
__device__ __forceinline__ void r_x(const RegV<T, RB>& a, RegV<T, RB>& b) {
#pragma unroll
  for (int j = 0; j < (1 << RB); ++j) cp_at<T, RB>(a, b, j, j ^ (1 << B));
}

template <typename T, int RB, int C, int G>
__device__ __forceinline__ void r_cx(const RegV<T, RB>& a, RegV<T, RB>& b) {
#pragma unroll
  for (int j = 0; j < (1 << RB); ++j) cp_at<T, RB>(a, b, j, (j & (1 << C)) ? j ^ (1 << G) : j);
}

template <typename T, int RB, int B0, int B1>
__device__ __forceinline__ void r_swap(const RegV<T, RB>& a, RegV<T, RB>& b) {
#pragma unroll
  for (int j = 0; j < (1 << RB); ++j) {
    const int k = ((j >> B0 & 1) != (j >> B1 & 1)) ? j ^ (1 << B0) ^ (1 << B1) : j;
    cp_at<T, RB>(a, b, j, k);
  }
}

template <typename T, int RB, int B0, int B1>
__device__ __forceinline__ void r_cz(const RegV<T, RB>& a, RegV<T, RB>& b) {
#pragma unroll
  for (int j = 0; j < (1 << RB); ++j) {
    if ((j & (1 << B0)) && (j & (1 << B1))) {
      b[2 * j] = -a[2 * j];
      b[2 * j + 1] = -a[2 * j + 1];
    } else {
      cp_at<T, RB>(a, b, j, j);
    }
  }
}

template <typename T, int RB, int B0, int B1>
__device__ __forceinline__ void r_cp(const RegV<T, RB>& a, RegV<T, RB>& b, const T* __restrict__ c) {
  const T cr = c[0], ci = c[1];
#pragma unroll
  for (int j = 0; j < (1 << RB); ++j) {
    if ((j & (1 << B0)) && (j & (1 << B1))) cmul_at<T, RB>(a, b, j, cr, ci);
    else cp_at<T, RB>(a, b, j, j);
  }
}

// Dense 4 x 4 on bits B0 < B1: y = M x over every quad of amplitudes that
// differ only in those bits (index within the quad = bit B0 + 2 bit B1).
template <typename T, int RB, int B0, int B1>
__device__ __forceinline__ void r_u2(const RegV<T, RB>& a, RegV<T, RB>& b, const T* __restrict__ c) {
#pragma unroll
  for (int j = 0; j < (1 << RB); ++j) {
    if ((j >> B0 & 1) || (j >> B1 & 1)) continue;
    const int ix[4] = {j, j | (1 << B0), j | (1 << B1), j | (1 << B0) | (1 << B1)};
    T xr[4], xi[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      xr[q] = a[2 * ix[q]];
      xi[q] = a[2 * ix[q] + 1];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const T* m = c + 8 * i;
      T yr = m[0] * xr[0] - m[1] * xi[0];
      T yi = m[0] * xi[0] + m[1] * xr[0];
#pragma unroll
      for (int k = 1; k < 4; ++k) {
        yr += m[2 * k] * xr[k] - m[2 * k + 1] * xi[k];
        yi += m[2 * k] * xi[k] + m[2 * k + 1] * xr[k];
      }
      b[2 * ix[i]] = yr;
      b[2 * ix[i] + 1] = yi;
    }
  }
}

// Ops under a condition on a qubit that is no register bit (OP_CPC, OP_CXC, OP_F):
// `pos` says where its value is found (HostOp::cond); `thr` holds the lane's lane
// and wave coordinates, `base` the tile's outer index.
__device__ __forceinline__ bool condition(int pos, uint32_t thr, uint64_t base) {
  return pos >= kOuterBit ? (base >> (pos - kOuterBit) & 1) != 0 : (thr >> pos & 1u) != 0;
}

template <typename T, int RB, int B>
__device__ __forceinline__ void r_cxc(const RegV<T, RB>& a, RegV<T, RB>& b, bool on) {
#pragma unroll
  for (int j = 0; j < (1 << RB); ++j) {
    const int k = j ^ (1 << B);
    b[2 * j] = on ? a[2 * k] : a[2 * j];
    b[2 * j + 1] = on ? a[2 * k + 1] : a[2 * j + 1];
  }
}

// Multiply by fr + i fi where bit B is set (B = RB: everywhere).
template <typename T, int RB, int B>
__device__ __forceinline__ void r_phase(const RegV<T, RB>& a, RegV<T, RB>& b, T fr, T fi) {
#pragma unroll
  for (int j = 0; j < (1 << RB); ++j) {
    if (B == RB || (j & (1 << B))) cmul_at<T, RB>(a, b, j, fr, fi);
    else cp_at<T, RB>(a, b, j, j);
  }
}

// b = op(a).  Returns the descriptors used: a factor's op is followed by the
// `b1` factors that are multiplied into it first.
template <typename T, int RB>
__device__ __forceinline__ int apply_op(const RegV<T, RB>& a, RegV<T, RB>& b,
                                        const OpDesc<T>* __restrict__ op, uint32_t thr, uint64_t base) {
  const int kind = __builtin_amdgcn_readfirstlane(op->kind);
  const int b0 = __builtin_amdgcn_readfirstlane(op->b0);
  const int b1 = __builtin_amdgcn_readfirstlane(op->b1);
  const T* c = op->c;
  switch (kind) {
    case OP_U: for_bit<RB>(b0, [&](auto B) __attribute__((always_inline)) { r_u<T, RB, decltype(B)::value>(a, b, c); }); break;
    case OP_R: for_bit<RB>(b0, [&](auto B) __attribute__((always_inline)) { r_r<T, RB, decltype(B)::value>(a, b, c); }); break;
    case OP_K: for_bit<RB>(b0, [&](auto B) __attribute__((always_inline)) { r_k<T, RB, decltype(B)::value, OP_K>(a, b, c); }); break;
    case OP_KR: for_bit<RB>(b0, [&](auto B) __attribute__((always_inline)) { r_k<T, RB, decltype(B)::value, OP_KR>(a, b, c); }); break;
    case OP_KI: for_bit<RB>(b0, [&](auto B) __attribute__((always_inline)) { r_k<T, RB, decltype(B)::value, OP_KI>(a, b, c); }); break;
    case OP_H: for_bit<RB>(b0, [&](auto B) __attribute__((always_inline)) { r_k<T, RB, decltype(B)::value, OP_H>(a, b, c); }); break;
    case OP_P: for_bit<RB>(b0, [&](auto B) __attribute__((always_inline)) { r_k<T, RB, decltype(B)::value, OP_P>(a, b, c); }); break;
    case OP_W: for_bit<RB>(b0, [&](auto B) __attribute__((always_inline)) { r_k<T, RB, decltype(B)::value, OP_W>(a, b, c); }); break;
    case OP_D: for_bit<RB>(b0, [&](auto B) __attribute__((always_inline)) { r_d<T, RB, decltype(B)::value>(a, b, c); }); break;
    case OP_D1: for_bit<RB>(b0, [&](auto B) __attribute__((always_inline)) { r_d1<T, RB, decltype(B)::value>(a, b, c); }); break;
    case OP_X: for_bit<RB>(b0, [&](auto B) __attribute__((always_inline)) { r_x<T, RB, decltype(B)::value>(a, b); }); break;
    case OP_CX:
      for_pair<RB>(b0, b1, [&](auto B0, auto B1) __attribute__((always_inline)) {
        r_cx<T, RB, decltype(B0)::value, decltype(B1)::value>(a, b);
      });
      break;
    case OP_CZ:
      for_pair<RB>(b0, b1, [&](auto B0, auto B1) __attribute__((always_inline)) {
        r_cz<T, RB, decltype(B0)::value, decltype(B1)::value>(a, b);
      });
      break;
    case OP_CP:
      for_pair<RB>(b0, b1, [&](auto B0, auto B1) __attribute__((always_inline)) {
        r_cp<T, RB, decltype(B0)::value, decltype(B1)::value>(a, b, c);
      });
      break;
    case OP_SWAP:
      for_pair<RB>(b0, b1, [&](auto B0, auto B1) __attribute__((always_inline)) {
        r_swap<T, RB, decltype(B0)::value, decltype(B1)::value>(a, b);
      });
      break;
    case OP_U2:
      if constexpr (RB >= 2) {
        for_pair<RB>(b0, b1, [&](auto B0, auto B1) __attribute__((always_inline)) {
          if constexpr (decltype(B0)::value < decltype(B1)::value)
            r_u2<T, RB, decltype(B0)::value, decltype(B1)::value>(a, b, c);
          else
            __builtin_unreachable();
        });
        break;
      } else {
        __builtin_unreachable();
      }
    case OP_CXC: {
      const bool on = condition(b1, thr, base);
      for_bit<RB>(b0, [&](auto B) __attribute__((always_inline)) { r_cxc<T, RB, decltype(B)::value>(a, b, on); });
      break;
    }
    case OP_CPC: {
      const bool on = condition(b1, thr, base);
      const T fr = on ? c[0] : T(1), fi = on ? c[1] : T(0);
      for_bit<RB>(b0, [&](auto B) __attribute__((always_inline)) { r_phase<T, RB, decltype(B)::value>(a, b, fr, fi); });
      break;
    }
    case OP_FA:
    case OP_GA: {
      T fr = T(1), fi = T(0);
      for (int i = 1; i <= b1; ++i) {
        const int p0 = __builtin_amdgcn_readfirstlane(op[i].b0), p1 = __builtin_amdgcn_readfirstlane(op[i].b1);
        const bool on = (p0 == kNoCond || condition(p0, thr, base)) && (p1 == kNoCond || condition(p1, thr, base));
        const T dr = on ? op[i].c[0] : T(1), di = on ? op[i].c[1] : T(0), t = fr;
        fr = t * dr - fi * di;
        fi = t * di + fi * dr;
      }
      if (kind == OP_FA) r_phase<T, RB, RB>(a, b, fr, fi);
      else for_bit<RB>(b0, [&](auto B) __attribute__((always_inline)) { r_phase<T, RB, decltype(B)::value>(a, b, fr, fi); });
      return 1 + b1;
    }
    default: __builtin_unreachable();
  }
  return 1;
}

// LDS swizzle width: the bank window holds 2^sw amplitudes (128 B).
template <typename T>
constexpr int lds_sw() { return sizeof(T) == 4 ? 4 : 3; }

// Sum of the per-bit offsets selected by the bits of v (global offsets);
// masks rather than branches, since v is per lane.
template <int N>
__device__ __forceinline__ uint64_t bit_sum(const uint64_t* w, uint32_t v) {
  uint64_t s = 0;
#pragma unroll
  for (int c = 0; c < N; ++c) s += w[c] & (uint64_t(0) - uint64_t(v >> c & 1u));
  return s;
}

// XOR of the per-bit LDS offsets selected by the bits of v.
template <int N>
__device__ __forceinline__ uint32_t bit_xor(const uint32_t* w, uint32_t v) {
  uint32_t s = 0;
#pragma unroll
  for (int c = 0; c < N; ++c) s ^= w[c] & (0u - (v >> c & 1u));
  return s;
}

// Base index of a tile: the outer setting `tile` with a zero bit inserted at
// every tile qubit (Alg. 1: the amplitudes of one outer setting).
__device__ __forceinline__ uint64_t tile_base32(uint64_t tile, const int32_t* tq, int m) {
  uint64_t b = tile;
  for (int i = 0; i < m; ++i) {
    const int q = tq[i];
    const uint64_t low = b & ((uint64_t(1) << q) - 1);
    b = ((b >> q) << (q + 1)) | low;
  }
  return b;
}

// Move the tile between HBM and registers.  `p` is the lane's address of
// register 0; register j adds the (uniform) offsets of its register bits.
template <typename T, int RB, bool STORE>
__device__ __forceinline__ void tile_io(cplx<T>* p, RegV<T, RB>& a, const uint64_t* reg) {
#pragma unroll
  for (int j = 0; j < (1 << RB); ++j) {
    cplx<T>* q = p + bit_sum<RB>(reg, (uint32_t)j);
    if constexpr (STORE) {
      cplx<T> v;
      v.x = a[2 * j];
      v.y = a[2 * j + 1];
      *q = v;
    } else {
      const cplx<T> v = *q;
      a[2 * j] = v.x;
      a[2 * j + 1] = v.y;
    }
  }
}

// ---------------------------------------------------------------------------
// part-pass kernel (Alg. 1 for one part), interpreting the part's ops
// ---------------------------------------------------------------------------
template <typename T, int RB>
__global__ void __launch_bounds__(1024)
part_pass_kernel(cplx<T>* __restrict__ st, const IPart* __restrict__ pd,
                 const IStage* __restrict__ sd, const OpDesc<T>* __restrict__ ops, uint32_t xcd) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int NR = 1 << RB;
  const int m = pd->m;
  const int ne = pd->n_stages;
  const uint64_t tiles = pd->tiles;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool active = lane < (1u << pd->lb);
  const uint32_t thr = lane | wave << pd->lb;

  // Tile-independent parts of the addresses.  Bits a layout lacks have zero
  // offsets, so lanes beyond the tile's lane bits stay in bounds.
  uint64_t ld_lane = bit_sum<kLaneBits>(pd->load.lane, lane) +
                           bit_sum<kMaxWaveBits>(pd->load.wave, wave);
  uint64_t sv_lane = bit_sum<kLaneBits>(pd->store.lane, lane) +
                           bit_sum<kMaxWaveBits>(pd->store.wave, wave);
  const uint32_t slot0 = bit_xor<kLaneBits>(sd[0].lane, lane) ^ bit_xor<kMaxWaveBits>(sd[0].wave, wave);
  // opaque: each stays one register value (otherwise the compiler keeps the
  // per-bit terms live across the tile loop and re-adds them per tile)
  asm volatile("" : "+v"(ld_lane), "+v"(sv_lane));

  // Tiles of this workgroup: with xcd set (grid and tile count multiples of
  // 8), XCD x = blockIdx % 8 sweeps the contiguous run [x T/8, (x+1) T/8).
  uint64_t tile = blockIdx.x, step = gridDim.x, end = tiles;
  if (xcd) {
    const uint64_t per = tiles >> 3;
    const uint32_t x = blockIdx.x & 7u;
    tile = x * per + (blockIdx.x >> 3);
    step = gridDim.x >> 3;
    end = (x + 1) * per;
  }
  // (no software prefetch of the next tile: with up to 1024 threads a lane
  // has 128 VGPRs, and a second tile's registers would spill)
  RegV<T, RB> a, b;
  for (; tile < end; tile += step) {
    const uint64_t outer = tile_base32(tile, pd->tq, m);
    cplx<T>* const base = st + outer;
    if (active) tile_io<T, RB, false>(base + ld_lane, a, pd->load.reg);
    // ---- execute: stages, re-laid out through LDS where the layout changes
    uint32_t slot = slot0;  // this lane's LDS offset in the current layout
    // an opaque copy of the lane index: keeps the per-bit lane masks of the
    // re-layouts from being hoisted out of the tile loop into live registers
    uint32_t ln = lane;
    asm volatile("" : "+v"(ln));
    for (int s = 1; s < ne; ++s) {
      const IStage& e = sd[s];
      if (e.transition) {
        const IStage& f = sd[s - 1];
        __syncthreads();
        if (active) {
#pragma unroll
          for (int j = 0; j < NR; ++j) {
            cplx<T> v;
            v.x = a[2 * j];
            v.y = a[2 * j + 1];
            *reinterpret_cast<cplx<T>*>(smem_raw + (slot ^ bit_xor<RB>(f.reg, (uint32_t)j))) = v;
          }
        }
        __syncthreads();
        slot = bit_xor<kLaneBits>(e.lane, ln) ^ bit_xor<kMaxWaveBits>(e.wave, wave);
#pragma unroll
        for (int j = 0; j < NR; ++j) {
          const cplx<T> v =
              *reinterpret_cast<const cplx<T>*>(smem_raw + (slot ^ bit_xor<RB>(e.reg, (uint32_t)j)));
          a[2 * j] = v.x;
          a[2 * j + 1] = v.y;
        }
      }
      // two ops an iteration: a -> b, then b -> a
      const int o1 = e.op_end;
      int o = e.op_begin;
      while (o < o1) {
        o += apply_op<T, RB>(a, b, ops + o, thr, outer);
        if (o >= o1) {
          a = b;
          break;
        }
        o += apply_op<T, RB>(b, a, ops + o, thr, outer);
      }
    }
    // ---- scatter (last entry is the store layout)
    if (active) tile_io<T, RB, true>(base + sv_lane, a, pd->store.reg);
  }
}

// ---------------------------------------------------------------------------
// fused part-pass kernel: one dense unitary per part on matrix cores
// ---------------------------------------------------------------------------
// For a part on w qubits (w = 4 to 7) every outer setting is a column of X
// (2^w rows, one per setting of the part's qubits); Y = U X for all columns.
// A wavefront takes 16 columns at a time -- the settings of the 4 lowest
// other qubits, so column runs are contiguous -- and computes the complex
// product as four real products on 16x16x4 MFMA tiles:
//   Yr = Ur Xr - Ui Xi,  Yi = Ur Xi + Ui Xr.
// (Gauss's three-product form, T3 = (Ur + Ui)(Xr + Xi), measured no faster
// for w = 4, 5 on 30-qubit states: those widths wait on memory, not on the
// matrix cores.)
// Operand layouts of the 16x16x4 MFMA (64 lanes, l = lane):
//   A[i][k]: i = l % 16, k = l / 16;   B[k][j]: j = l % 16, k = l / 16;
//   D[i][j] (4 registers v): j = l % 16 and
//     i = 4 * (l / 16) + v  for the FP32 instruction,
//     i = l / 16 + 4 * v    for the FP64 instruction
// (checked on gfx950 with a probe that feeds lane numbers through A and B).
template <typename T>
struct Mfma;
template <>
struct Mfma<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mma(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mfma<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mma(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};

// deposit the low bits of v onto the listed qubits
__device__ __forceinline__ uint64_t deposit(uint32_t v, const int8_t* q, int count) {
  uint64_t g = 0;
  for (int b = 0; b < count; ++b) g |= uint64_t((v >> b) & 1u) << q[b];
  return g;
}

// U arrives in fragment order: fragment f = rb * (2^w / 4) + ks holds, in lane
// l, U[16 rb + l % 16][4 ks + l / 16]; the real parts of all fragments come
// first, then the imaginary parts.  For w <= 5 a wave keeps all of U in
// registers (complex128 at w = 5 excepted); wider U (complex128 w = 7) is read
// fragment by fragment from the L2-resident copy -- one contiguous wave load
// per fragment.

template <typename T, int W, bool PIPE>
__global__ void __launch_bounds__(256)
fused_pass_kernel(cplx<T>* __restrict__ st, const FusedDesc* __restrict__ fd, const T* __restrict__ umat,
                  uint32_t xcd) {
  using v4 = typename Mfma<T>::v4;
  constexpr int R = 1 << W;   // rows of U
  constexpr int RBK = R / 16; // 16-row blocks
  constexpr int KS = R / 4;   // K steps of 4
  constexpr int NF = RBK * KS;
  // U in registers for w <= 5, except complex128 at w = 5 (96 more VGPRs:
  // one wave per SIMD), which reads U from the L1/L2-resident copy instead
  constexpr bool kRegU = W <= 4 || (W == 5 && sizeof(T) == 4);
  constexpr bool kPipe = PIPE && W <= 5;  // software-pipelined (see below)
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t i16 = lane & 15, g4 = lane >> 4;
  const int m = fd->m;
  const uint64_t tiles = fd->tiles;
  const T* Ur = umat + fd->u_off;
  const T* Ui = Ur + NF * 64;
  T ur[kRegU ? RBK : 1][kRegU ? KS : 1], ui[kRegU ? RBK : 1][kRegU ? KS : 1],
      nui[kRegU ? RBK : 1][kRegU ? KS : 1];
  if (kRegU) {
#pragma unroll
    for (int rb = 0; rb < (kRegU ? RBK : 1); ++rb)
#pragma unroll
      for (int ks = 0; ks < (kRegU ? KS : 1); ++ks) {
        const int f = rb * KS + ks;
        ur[rb][ks] = Ur[f * 64 + lane];
        ui[rb][ks] = Ui[f * 64 + lane];
        nui[rb][ks] = -ui[rb][ks];
      }
  }
  // The qubit lists (sq[8], pq[4], tq[12]: 24 contiguous bytes of the
  // descriptor) as six uniform dwords, read once: byte loads inside the tile
  // loop would be vector loads followed by a full wait on every memory
  // operation in flight, prefetched tiles and stores included.
  static_assert(offsetof(FusedDesc, sq) % 4 == 0 && offsetof(FusedDesc, pq) == offsetof(FusedDesc, sq) + 8 &&
                    offsetof(FusedDesc, tq) == offsetof(FusedDesc, sq) + 12 && sizeof(FusedDesc::tq) == 12,
                "the qubit lists must be 24 contiguous bytes on a dword boundary");
  uint32_t qw[6];
  {
    const uint32_t* q32 = reinterpret_cast<const uint32_t*>(fd->sq);
#pragma unroll
    for (int i = 0; i < 6; ++i) qw[i] = __builtin_amdgcn_readfirstlane(q32[i]);
  }
  // qubit of list byte b (sq: 0-7, pq: 8-11, tq: 12-23); b is a constant
  auto qb = [&](int b) -> int { return (int)(int8_t)(qw[b >> 2] >> (8 * (b & 3))); };
  // deposit the low `count` bits of v onto the qubits of bytes first..
  auto dep = [&](uint32_t v, int first, int count) -> uint64_t {
    uint64_t g = 0;
#pragma unroll
    for (int b = 0; b < count; ++b) g |= uint64_t((v >> b) & 1u) << qb(first + b);
    return g;
  };
  // base index of a tile: a zero bit inserted at every tile qubit (ascending)
  auto base_of = [&](uint64_t t) -> uint64_t {
#pragma unroll
    for (int i = 0; i < 12; ++i)
      if (i < m) {
        const int q = qb(12 + i);
        t = ((t >> q) << (q + 1)) | (t & ((uint64_t(1) << q) - 1));
      }
    return t;
  };
  // lane parts of the addresses: B rows k = 4*ks + g4 (slots 0-1 from the
  // lane); D rows i = 16*rb + 4*g4 + v (FP32: slots 2-3 from the lane) or
  // 16*rb + 4*v + g4 (FP64: slots 0-1 from the lane); columns j = i16 on
  // the column qubits
  constexpr bool f64 = sizeof(T) == 8;
  const uint64_t col = dep(i16, 8, 4);
  const uint64_t lane_ld = col + dep(g4, 0, 2);
  const uint64_t lane_st = f64 ? lane_ld : col + dep(g4 << 2, 0, W);
  uint64_t row_ld[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) row_ld[ks] = dep(4 * ks, 0, W);
  // a workgroup's 4 waves take 4 consecutive tiles; with xcd set (grid
  // and group count multiples of 8) XCD x = blockIdx % 8 sweeps a contiguous
  // run
  const uint64_t groups = (tiles + 3) / 4;
  uint64_t g = blockIdx.x, step = gridDim.x, end = groups;
  if (xcd) {
    const uint64_t per = groups >> 3;
    const uint32_t x = blockIdx.x & 7u;
    g = x * per + (blockIdx.x >> 3);
    step = gridDim.x >> 3;
    end = (x + 1) * per;
  }
  // wave-uniform: tile indices, bases and the valid flags stay in scalar
  // registers (address arithmetic on the SALU, stores under a scalar branch)
  const uint64_t wave_tile = (uint64_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // X of this wave's tile in group gg
  // (branch-free: a wave past the last tile reads tile 0 and discards its
  // products, so no load sits in a conditional block or feeds a select --
  // either would make the wave wait for the load right away)
  // tiles is a power of two (2^(n-m)): a tile index is in range when no bit
  // at or above log2(tiles) is set -- a 64-bit test the scalar unit has (it
  // has no 64-bit ordered compare)
  const uint64_t past = ~(tiles - 1);
  auto load = [&](uint64_t gg, T (&xr)[KS], T (&xi)[KS], uint64_t& base, bool& valid) {
    const uint64_t tile = gg * 4 + wave_tile;
    valid = (tile & past) == 0;
    base = base_of(valid ? tile : 0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const cplx<T> v = st[base + row_ld[ks] + lane_ld];
      xr[ks] = v.x;
      xi[ks] = v.y;
    }
  };
  // Y = U X on the matrix cores, stored in place
  auto product = [&](const T (&xr)[KS], const T (&xi)[KS], uint64_t base, bool valid) {
    constexpr int kRbUnroll = kRegU ? RBK : 1;
#pragma unroll kRbUnroll
    for (int rb = 0; rb < RBK; ++rb) {
      v4 yr = v4{0, 0, 0, 0}, yi = v4{0, 0, 0, 0};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        T ar, ai, nai;
        if (kRegU) {
          ar = ur[kRegU ? rb : 0][kRegU ? ks : 0];
          ai = ui[kRegU ? rb : 0][kRegU ? ks : 0];
          nai = nui[kRegU ? rb : 0][kRegU ? ks : 0];
        } else {
          const int f = rb * KS + ks;
          ar = Ur[f * 64 + lane];
          ai = Ui[f * 64 + lane];
          nai = -ai;
        }
        yr = Mfma<T>::mma(ar, xr[ks], yr);
        yr = Mfma<T>::mma(nai, xi[ks], yr);
        yi = Mfma<T>::mma(ar, xi[ks], yi);
        yi = Mfma<T>::mma(ai, xr[ks], yi);
      }
      if (valid) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          cplx<T> o;
          o.x = yr[v];
          o.y = yi[v];
          st[base + dep(16 * rb + (f64 ? 4 * v : v), 0, W) + lane_st] = o;
        }
      }
    }
  };
  T xr[KS], xi[KS];
  uint64_t base;
  bool valid;
  if (kPipe) {
    // w <= 5: a persistent grid, software-pipelined per wave -- the next
    // group's loads are issued before this group's products, so each wave
    // overlaps its own HBM traffic with its matrix-core work (loads, products
    // and stores of one tile would otherwise run as three serial phases).
    // Two register sets alternate (no copies between iterations, which
    // would wait for the loads), and the loads are unconditional: past the
    // end a wave re-reads its current group, whose products it discards.
    T yr2[KS], yi2[KS];
    uint64_t base2;
    bool valid2;
    if (g < end) load(g, xr, xi, base, valid);
    while (g < end) {
      const uint64_t g1 = g + step;
      load(g1 < end ? g1 : g, yr2, yi2, base2, valid2);
      product(xr, xi, base, valid);
      if (g1 >= end) break;
      const uint64_t g2 = g1 + step;
      load(g2 < end ? g2 : g1, xr, xi, base, valid);
      product(yr2, yi2, base2, valid2);
      g = g2;
    }
  } else {
    for (; g < end; g += step) {
      load(g, xr, xi, base, valid);
      product(xr, xi, base, valid);
    }
  }
}

// The same product with U in LDS, for widths whose U fits there beside enough
// waves (complex64 w = 5, 6, 7: 8, 32, 128 KiB; complex128 w = 5, 6: 16, 64 KiB).
// A persistent grid reads U once a workgroup.  The K loop is outermost: all
// row blocks accumulate at once, so X[ks] is dead after its products and the
// next tile's X[ks] is loaded into its registers right there.  A wave so has
// the next tile's loads in flight under a whole tile's products, without a
// second register set.
template <typename T, int W>
constexpr int fused_lds_threads() { return W == 7 ? 512 : 256; }

template <typename T, int W>
__global__ void __launch_bounds__((fused_lds_threads<T, W>()))
fused_lds_kernel(cplx<T>* __restrict__ st, const FusedDesc* __restrict__ fd, const T* __restrict__ umat,
                 uint32_t xcd, uint32_t chunk) {
  using v4 = typename Mfma<T>::v4;
  constexpr int R = 1 << W, RBK = R / 16, KS = R / 4, NF = RBK * KS;
  constexpr int NT = fused_lds_threads<T, W>(), WAVES = NT / 64;
  // fragment f = ks * RBK + rb: lane l's (re, im) of U[16 rb + l % 16][4 ks + l / 16]
  __shared__ cplx<T> us[NF * 64];
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t i16 = lane & 15, g4 = lane >> 4;
  const uint64_t tiles = fd->tiles;
  const T* Ur = umat + fd->u_off;
  for (int i = threadIdx.x; i < NF * 64; i += NT) {
    const int f = i >> 6, o = ((f % RBK) * KS + f / RBK) * 64 + (i & 63);
    us[i].x = Ur[o];
    us[i].y = Ur[NF * 64 + o];
  }
  __syncthreads();
  uint32_t qw[6];
  {
    const uint32_t* q32 = reinterpret_cast<const uint32_t*>(fd->sq);
#pragma unroll
    for (int i = 0; i < 6; ++i) qw[i] = __builtin_amdgcn_readfirstlane(q32[i]);
  }
  auto qb = [&](int b) -> int { return (int)(int8_t)(qw[b >> 2] >> (8 * (b & 3))); };
  auto dep = [&](uint32_t v, int first, int count) -> uint64_t {
    uint64_t g = 0;
#pragma unroll
    for (int b = 0; b < count; ++b) g |= uint64_t((v >> b) & 1u) << qb(first + b);
    return g;
  };
  auto base_of = [&](uint64_t t) -> uint64_t {
#pragma unroll
    for (int i = 0; i < W + 4; ++i) {
      const int q = qb(12 + i);
      t = ((t >> q) << (q + 1)) | (t & ((uint64_t(1) << q) - 1));
    }
    return t;
  };
  constexpr bool f64 = sizeof(T) == 8;
  const uint64_t col = dep(i16, 8, 4);
  const uint64_t lane_ld = col + dep(g4, 0, 2);
  const uint64_t lane_st = f64 ? lane_ld : col + dep(g4 << 2, 0, W);
  const uint64_t groups = (tiles + WAVES - 1) / WAVES;
  uint64_t g = (uint64_t)blockIdx.x * chunk, end = groups;
  if (xcd) {
    const uint64_t per = groups >> 3;
    const uint32_t x = blockIdx.x & 7u;
    g = x * per + (uint64_t)(blockIdx.x >> 3) * chunk;
    end = (x + 1) * per;
  }
  if (g + chunk < end) end = g + chunk;
  const uint64_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t past = ~(tiles - 1);  // tiles is a power of two
  cplx<T>* const p_ld = st + lane_ld;
  cplx<T>* const p_st = st + lane_st;
  // Offsets of the row bits.  Opaque in each iteration: the sums below are
  // then formed where they are used, on the scalar unit, instead of being
  // kept in registers (one 64-bit value a lane for each row) over the loop.
  uint64_t bit[W];
#pragma unroll
  for (int b = 0; b < W; ++b) bit[b] = uint64_t(1) << qb(b);
  auto row = [&](int r) -> uint64_t {
    uint64_t o = 0;
#pragma unroll
    for (int b = 0; b < W; ++b)
      if (r >> b & 1) o += bit[b];
    return o;
  };
  T xr[KS], xi[KS];
  uint64_t tile = g * WAVES + wave;
  bool valid = g < end && (tile & past) == 0;
  uint64_t base = base_of(valid ? tile : 0);
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const cplx<T> v = p_ld[base + row(4 * ks)];
    xr[ks] = v.x;
    xi[ks] = v.y;
  }
  cplx<T> a[RBK];
#pragma unroll
  for (int rb = 0; rb < RBK; ++rb) a[rb] = us[rb * 64 + lane];
  for (; g < end; ++g) {
#pragma unroll
    for (int b = 0; b < W; ++b) asm volatile("" : "+s"(bit[b]));
    // the next group's tile; past the end the wave re-reads tile 0 for nothing
    const uint64_t gn = g + 1;
    tile = gn * WAVES + wave;
    const bool next_valid = gn < end && (tile & past) == 0;
    const uint64_t next = base_of(next_valid ? tile : 0);
    v4 yr[RBK], yi[RBK];
#pragma unroll
    for (int rb = 0; rb < RBK; ++rb) yr[rb] = yi[rb] = v4{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      // U's next column of fragments, this step's products, X's refill; the
      // barrier keeps the compiler from sinking the refills below the products
      const T br = xr[ks], bi = xi[ks], nbi = -bi;
      cplx<T> an[RBK];
#pragma unroll
      for (int rb = 0; rb < RBK; ++rb) an[rb] = us[((ks + 1) % KS * RBK + rb) * 64 + lane];
#pragma unroll
      for (int rb = 0; rb < RBK; ++rb) {
        yr[rb] = Mfma<T>::mma(a[rb].x, br, yr[rb]);
        yi[rb] = Mfma<T>::mma(a[rb].x, bi, yi[rb]);
        yr[rb] = Mfma<T>::mma(a[rb].y, nbi, yr[rb]);
        yi[rb] = Mfma<T>::mma(a[rb].y, br, yi[rb]);
      }
      const cplx<T> v = p_ld[next + row(4 * ks)];
      xr[ks] = v.x;
      xi[ks] = v.y;
#pragma unroll
      for (int rb = 0; rb < RBK; ++rb) a[rb] = an[rb];
      __builtin_amdgcn_sched_barrier(0);
    }
    if (valid) {
#pragma unroll
      for (int rb = 0; rb < RBK; ++rb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          cplx<T> o;
          o.x = yr[rb][v];
          o.y = yi[rb][v];
          p_st[base + row(16 * rb + (f64 ? 4 * v : v))] = o;
        }
    }
    base = next;
    valid = next_valid;
  }
}

// ---------------------------------------------------------------------------
// gate-per-pass baseline: one sweep of the whole state per gate
// ---------------------------------------------------------------------------
template <typename T>
struct M2 {
  T c[8];
};

// Work items [first, end) with stride `step` of a thread in a streaming
// kernel.  With xcd set (grid a multiple of 8, count a multiple of 8), XCD
// x = blockIdx % 8 sweeps the contiguous eighth [x count/8, (x+1) count/8).
struct Walk {
  uint64_t first, step, end;
};
__device__ __forceinline__ Walk stream_walk(uint64_t count, uint32_t xcd) {
  if (!xcd)
    return {(uint64_t)blockIdx.x * blockDim.x + threadIdx.x, (uint64_t)gridDim.x * blockDim.x, count};
  const uint64_t per = count >> 3;
  const uint32_t x = blockIdx.x & 7u;
  return {x * per + (uint64_t)(blockIdx.x >> 3) * blockDim.x + threadIdx.x,
          (uint64_t)(gridDim.x >> 3) * blockDim.x, (x + 1) * per};
}

// VEC consecutive amplitudes, moved as one 16 B access: two of a complex64
// state (where its address allows it), one of a complex128 state.
template <typename T, int VEC>
struct alignas(VEC * 2 * sizeof(T)) Amps {
  cplx<T> a[VEC];
};

template <typename T>
__device__ __forceinline__ void pair_1q(const M2<T>& u, cplx<T>& x, cplx<T>& y) {
  cplx<T> r0, r1;
  r0.x = u.c[0] * x.x - u.c[1] * x.y + u.c[2] * y.x - u.c[3] * y.y;
  r0.y = u.c[0] * x.y + u.c[1] * x.x + u.c[2] * y.y + u.c[3] * y.x;
  r1.x = u.c[4] * x.x - u.c[5] * x.y + u.c[6] * y.x - u.c[7] * y.y;
  r1.y = u.c[4] * x.y + u.c[5] * x.x + u.c[6] * y.y + u.c[7] * y.x;
  x = r0;
  y = r1;
}

// index with a zero bit inserted at position q
__device__ __forceinline__ uint64_t insert_zero(uint64_t p, int q) {
  return ((p >> q) << (q + 1)) | (p & ((uint64_t(1) << q) - 1));
}

// One-qubit sweep over pairs of vectors; q counts vectors (the qubit less
// log2(VEC)).  q = -1: the pair is inside the vector (qubit 0, VEC = 2).
template <typename T, int VEC>
__global__ void __launch_bounds__(256)
gate_pass_1q(Amps<T, VEC>* __restrict__ st, int q, uint64_t count, M2<T> u, uint32_t xcd) {
  const Walk w = stream_walk(count, xcd);
  for (uint64_t p = w.first; p < w.end; p += w.step) {
    if (VEC == 2 && q < 0) {
      Amps<T, VEC> s = st[p];
      pair_1q(u, s.a[0], s.a[VEC - 1]);
      st[p] = s;
      continue;
    }
    const uint64_t i0 = insert_zero(p, q), i1 = i0 | (uint64_t(1) << q);
    Amps<T, VEC> x = st[i0], y = st[i1];
#pragma unroll
    for (int v = 0; v < VEC; ++v) pair_1q(u, x.a[v], y.a[v]);
    st[i0] = x;
    st[i1] = y;
  }
}

// Diagonal one-qubit sweep: amplitudes times d0 or d1 by their bit.  HALF
// (d0 = 1): only the vectors with the bit set are touched.
template <typename T, int VEC, bool HALF>
__global__ void __launch_bounds__(256)
gate_pass_diag(Amps<T, VEC>* __restrict__ st, int q, uint64_t count, cplx<T> d0, cplx<T> d1, uint32_t xcd) {
  const Walk w = stream_walk(count, xcd);
  for (uint64_t p = w.first; p < w.end; p += w.step) {
    const uint64_t i = HALF ? insert_zero(p, q) | (uint64_t(1) << q) : p;
    Amps<T, VEC> s = st[i];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      const bool one = HALF || (q < 0 ? v != 0 : (i >> q & 1) != 0);
      cmul(s.a[v], one ? d1.x : d0.x, one ? d1.y : d0.y);
    }
    st[i] = s;
  }
}

// Two-qubit sweep: only the amplitudes the gate changes are read and written --
// half of the state for CX (control set) and SWAP (bits different), a quarter
// for CZ and CP (both set), where reading the whole quad moved three quarters.
// Bits count vectors.  KIND: 0 CX(q0 control, q1 target), 1 CZ, 2 CP(c), 3 SWAP
template <typename T, int VEC, int KIND>
__global__ void __launch_bounds__(256)
gate_pass_2q(Amps<T, VEC>* __restrict__ st, int q0, int q1, uint64_t count, cplx<T> c, uint32_t xcd) {
  const int lo = min(q0, q1), hi = max(q0, q1);
  const Walk w = stream_walk(count, xcd);
  const uint64_t m0 = uint64_t(1) << q0, m1 = uint64_t(1) << q1;
  for (uint64_t p = w.first; p < w.end; p += w.step) {
    const uint64_t i = insert_zero(insert_zero(p, lo), hi);
    if constexpr (KIND == 0 || KIND == 3) {
      const uint64_t j = i | m0, k = KIND == 0 ? i | m0 | m1 : i | m1;
      const Amps<T, VEC> x = st[j], y = st[k];
      st[j] = y;
      st[k] = x;
    } else {
      Amps<T, VEC> s = st[i | m0 | m1];
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        if constexpr (KIND == 1) {
          s.a[v].x = -s.a[v].x;
          s.a[v].y = -s.a[v].y;
        } else {
          cmul(s.a[v], c.x, c.y);
        }
      }
      st[i | m0 | m1] = s;
    }
  }
}

// ---------------------------------------------------------------------------
// init, readout, probe
// ---------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256) set_basis_kernel(cplx<T>* __restrict__ st, uint64_t N, uint64_t x) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride) {
    cplx<T> v;
    v.x = (i == x) ? T(1) : T(0);
    v.y = T(0);
    st[i] = v;
  }
}

constexpr int kNormBlocks = 1024;
constexpr int kNormThreads = 256;

// Fixed-shape two-level FP64 reduction: thread t of block b sums |a_i|^2 for
// i = b*256 + t + k*(1024*256), k = 0, 1, ...; each block reduces its 256
// partial sums by a fixed binary tree; one block then reduces the 1024
// block sums by the same tree.  The order never depends on the device.
template <typename T>
__global__ void __launch_bounds__(kNormThreads)
norm_partial(const cplx<T>* __restrict__ st, uint64_t N, double* __restrict__ part) {
  __shared__ double sh[kNormThreads];
  double acc = 0.0;
  const uint64_t stride = (uint64_t)kNormBlocks * kNormThreads;
  uint64_t i = (uint64_t)blockIdx.x * kNormThreads + threadIdx.x;
  // eight loads in flight a thread, added up in the same order (one at a time
  // leaves HBM waiting: 27 qubits complex64 3.6 TB/s)
  for (; i + 7 * stride < N; i += 8 * stride) {
    cplx<T> v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = st[i + k * stride];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc += (double)v[k].x * (double)v[k].x + (double)v[k].y * (double)v[k].y;
  }
  for (; i < N; i += stride) {
    const cplx<T> v = st[i];
    acc += (double)v.x * (double)v.x + (double)v.y * (double)v.y;
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kNormThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ void __launch_bounds__(kNormThreads) norm_final(const double* __restrict__ part, double* __restrict__ out) {
  __shared__ double sh[kNormThreads];
  double acc = 0.0;
  for (int i = threadIdx.x; i < kNormBlocks; i += kNormThreads) acc += part[i];
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kNormThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = sh[0];
}

// probs = 0: widen amplitudes to complex128; probs = 1: |a|^2 in FP64.
template <typename T>
__global__ void __launch_bounds__(256)
readout_kernel(const cplx<T>* __restrict__ st, uint64_t first, uint64_t count, int probs,
               double* __restrict__ out) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) {
    const cplx<T> v = st[first + i];
    const double re = (double)v.x, im = (double)v.y;
    if (probs) {
      out[i] = re * re + im * im;
    } else {
      out[2 * i] = re;
      out[2 * i + 1] = im;
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(256)
gather_kernel(const cplx<T>* __restrict__ st, const uint64_t* __restrict__ idx, uint64_t count,
              double* __restrict__ out) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) {
    const cplx<T> v = st[idx[i]];
    out[2 * i] = (double)v.x;
    out[2 * i + 1] = (double)v.y;
  }
}

__global__ void __launch_bounds__(256)
copy_probe_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, uint64_t n16) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
    dst[i] = src[i];
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
#define HIP_TRY(expr)                                                              \
  do {                                                                             \
    hipError_t e_ = (expr);                                                        \
    if (e_ != hipSuccess) return fail(HS_E_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

struct DevInfo {
  int cus = 0;
};

static std::mutex g_dev_mu;
static std::map<int, DevInfo> g_dev;

static hs_status device_info(int dev, DevInfo* out) {
  std::lock_guard<std::mutex> lk(g_dev_mu);
  auto it = g_dev.find(dev);
  if (it != g_dev.end()) {
    *out = it->second;
    return HS_OK;
  }
  DevInfo d;
  HIP_TRY(hipDeviceGetAttribute(&d.cus, hipDeviceAttributeMultiprocessorCount, dev));
  g_dev[dev] = d;
  *out = d;
  return HS_OK;
}

static inline hipStream_t stream_of(State* s) { return (hipStream_t)s->stream; }

// streaming grid: enough blocks of 256 to fill the device a few times over
static hs_status stream_grid(int dev, uint64_t work, unsigned* grid) {
  DevInfo d;
  hs_status rc = device_info(dev, &d);
  if (rc) return rc;
  const uint64_t want = (work + 255) / 256;
  *grid = (unsigned)std::max<uint64_t>(1, std::min<uint64_t>(want, (uint64_t)d.cus * 16));
  return HS_OK;
}

hs_status dev_set_basis(State* s, uint64_t x) {
  HIP_TRY(hipSetDevice(s->device));
  const uint64_t N = uint64_t(1) << s->n;
  unsigned grid;
  if (hs_status rc = stream_grid(s->device, N, &grid)) return rc;
  if (s->dtype == HS_C64)
    hipLaunchKernelGGL(set_basis_kernel<float>, dim3(grid), dim3(256), 0, stream_of(s),
                       (cplx<float>*)s->ptr, N, x);
  else
    hipLaunchKernelGGL(set_basis_kernel<double>, dim3(grid), dim3(256), 0, stream_of(s),
                       (cplx<double>*)s->ptr, N, x);
  HIP_TRY(hipGetLastError());
  return HS_OK;
}

// Grid of a gate sweep over `work` items: one item per thread up to 2^31
// threads, XCD-contiguous runs when the grid and the item count allow.
static void sweep_grid(uint64_t work, unsigned* grid, uint32_t* xcd) {
  uint64_t g = std::max<uint64_t>(1, std::min<uint64_t>((work + 255) / 256, (uint64_t(1) << 31) / 256));
  *xcd = 0;
  if (work % 8 == 0 && g >= 8) {
    g &= ~uint64_t(7);
    *xcd = 1;
  }
  *grid = (unsigned)g;
}

// One gate as a sweep, on vectors of VEC amplitudes where its qubits allow it.
template <typename T, int VEC>
static hs_status gate_pass_v(State* s, const Gate& g) {
  constexpr int L = VEC == 2 ? 1 : 0;
  const uint64_t N = uint64_t(1) << (s->n - L);  // vectors
  auto* st = (Amps<T, VEC>*)s->ptr;
  const int q = g.q0 - L;
  unsigned grid;
  uint32_t xcd;
  if (g.arity() == 1) {
    cd u[4];
    gate_matrix(g, u);
    if (u[1] == cd(0, 0) && u[2] == cd(0, 0)) {
      const cplx<T> d0{(T)u[0].real(), (T)u[0].imag()}, d1{(T)u[3].real(), (T)u[3].imag()};
      const bool half = u[0] == cd(1, 0) && q >= 0;
      sweep_grid(half ? N / 2 : N, &grid, &xcd);
      if (half)
        hipLaunchKernelGGL((gate_pass_diag<T, VEC, true>), dim3(grid), dim3(256), 0, stream_of(s), st, q, N / 2, d0,
                           d1, xcd);
      else
        hipLaunchKernelGGL((gate_pass_diag<T, VEC, false>), dim3(grid), dim3(256), 0, stream_of(s), st, q, N, d0, d1,
                           xcd);
    } else {
      M2<T> m;
      for (int i = 0; i < 4; ++i) {
        m.c[2 * i] = (T)u[i].real();
        m.c[2 * i + 1] = (T)u[i].imag();
      }
      const uint64_t items = q < 0 ? N : N / 2;
      sweep_grid(items, &grid, &xcd);
      hipLaunchKernelGGL((gate_pass_1q<T, VEC>), dim3(grid), dim3(256), 0, stream_of(s), st, q, items, m, xcd);
    }
  } else {
    const int p = g.q1 - L;
    cplx<T> c{0, 0};
    sweep_grid(N / 4, &grid, &xcd);
#define HS_GATE_2Q(KIND_)                                                                                         \
  hipLaunchKernelGGL((gate_pass_2q<T, VEC, KIND_>), dim3(grid), dim3(256), 0, stream_of(s), st, q, p, N / 4, c, xcd)
    switch (g.kind) {
      case HS_CX: HS_GATE_2Q(0); break;
      case HS_CZ: HS_GATE_2Q(1); break;
      case HS_CP:
        c = {(T)cos(g.p[0]), (T)sin(g.p[0])};
        HS_GATE_2Q(2);
        break;
      case HS_SWAP: HS_GATE_2Q(3); break;
      default: return fail(HS_E_ARG, "unknown two-qubit kind %d", g.kind);
    }
#undef HS_GATE_2Q
  }
  HIP_TRY(hipGetLastError());
  return HS_OK;
}

hs_status dev_gate_pass(State* s, const Gate& g) {
  HIP_TRY(hipSetDevice(s->device));
  if (g.arity() == 2 && s->n < 2) return fail(HS_E_ARG, "two-qubit gate on a 1-qubit state");
  if (s->dtype == HS_C128) return gate_pass_v<double, 1>(s, g);
  // pairs of complex64 amplitudes as 16 B accesses, unless the state starts
  // inside one (hs_state_wrap asks for the alignment of an amplitude) or a
  // two-qubit gate acts on qubit 0
  const bool pairs = (uintptr_t)s->ptr % 16 == 0 && (g.arity() == 1 || (g.q0 > 0 && g.q1 > 0));
  return pairs ? gate_pass_v<float, 2>(s, g) : gate_pass_v<float, 1>(s, g);
}

// ---- uploaded plan ----------------------------------------------------------
struct DevicePlan {
  int device = 0;
  // descriptors from the stream-ordered allocator (serving): freed with
  // hipFreeAsync on free_stream, so a teardown never waits for the device
  bool async_alloc = false;
  void* free_stream = nullptr;
  // recorded after the asynchronous descriptor copies on free_stream; a
  // launch on another stream waits for it on the device
  hipEvent_t upload_done = nullptr;
  IPart* parts = nullptr;
  IStage* stages = nullptr;
  void* ops = nullptr;
  std::vector<PartDesc> h_parts;     // host copy (absolute offsets)
  std::vector<int> rb;               // register bits of the kernel per part
  std::vector<unsigned> grid;        // grid per part
  std::vector<uint8_t> xcd;          // XCD-contiguous tile runs
};

// ---- uploaded unitaries -------------------------------------------------------
// The kernel and launch of a fused part.
struct FusedLaunch {
  int w = 0;
  const void* fn = nullptr;
  int block = 256;
  unsigned grid = 1;
  uint32_t xcd = 0;    // XCD-contiguous tile runs
  uint32_t chunk = 0;  // consecutive tile groups of a workgroup (fused_lds_kernel)
};

struct DeviceFused {
  int device = 0;
  FusedDesc* parts = nullptr;
  void* mat = nullptr;
  std::vector<FusedLaunch> launch;
};

void device_fused_free(DeviceFused* d) {
  if (!d) return;
  (void)hipSetDevice(d->device);
  if (d->parts) (void)hipFree(d->parts);
  if (d->mat) (void)hipFree(d->mat);
  delete d;
}

// Best effort: called from destructors, where an error cannot be returned.
void device_plan_free(DevicePlan* d) {
  if (!d) return;
  (void)hipSetDevice(d->device);
  for (void* ptr : {(void*)d->parts, (void*)d->stages, d->ops}) {
    if (!ptr) continue;
    if (d->async_alloc) (void)hipFreeAsync(ptr, (hipStream_t)d->free_stream);
    else (void)hipFree(ptr);
  }
  if (d->upload_done) (void)hipEventDestroy(d->upload_done);
  delete d;
}

// Host copies of a plan's descriptors, kept until the asynchronous copies
// from them have run (a host function on the copy stream deletes them).
template <typename T>
struct HostDescriptors {
  std::vector<IPart> parts;
  std::vector<IStage> stages;
  std::vector<OpDesc<T>> ops;
  static void release(void* p) { delete static_cast<HostDescriptors*>(p); }
};

template <typename T, int RB>
static hs_status resident_per_cu(int block, size_t lds, int* per_cu) {
  if (lds > 65536)
    HIP_TRY(hipFuncSetAttribute((const void*)part_pass_kernel<T, RB>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, part_pass_kernel<T, RB>, block, lds));
  if (*per_cu < 1) return fail(HS_E_UNSUPPORTED, "part kernel cannot be resident (block %d, lds %zu)",
                               block, lds);
  return HS_OK;
}

template <typename T>
static hs_status resident_rb(int rb, int block, size_t lds, int* per_cu) {
  switch (rb) {
    case 1: return resident_per_cu<T, 1>(block, lds, per_cu);
    case 2: return resident_per_cu<T, 2>(block, lds, per_cu);
    case 3: return resident_per_cu<T, 3>(block, lds, per_cu);
    case 4: return resident_per_cu<T, 4>(block, lds, per_cu);
    default: return fail(HS_E_UNSUPPORTED, "no kernel with %d register bits", rb);
  }
}

// Grid of one part-pass launch for launch shape `ls`: one workgroup per tile,
// or a persistent grid sized by occupancy; XCD-contiguous tile runs need the
// grid and the tile count to be multiples of 8.
static void part_grid(const LaunchShape& ls, uint64_t tiles, int block, int per_cu, int cus,
                      unsigned* grid, uint8_t* xcd) {
  uint64_t g = tiles;
  if (ls.per_cu > 0) g = std::min<uint64_t>(tiles, (uint64_t)ls.per_cu * per_cu * cus);
  g = std::max<uint64_t>(1, std::min<uint64_t>(g, (uint64_t(1) << 31) / (uint64_t)block));
  *xcd = 0;
  if (ls.xcd && tiles % 8 == 0 && g >= 8) {
    g &= ~uint64_t(7);
    *xcd = 1;
  }
  *grid = (unsigned)g;
}

// Interpreter tables of one layout (host side of IStage / IoOffsets).
template <typename T>
static IStage interp_stage(const StageDesc& e, const PartDesc& d) {
  IStage o{};
  const int sw = lds_sw<T>();
  auto slot = [&](int c) { return lds_slot(1u << e.pos[c], sw) * (uint32_t)sizeof(cplx<T>); };
  for (int c = 0; c < d.lb; ++c) o.lane[c] = slot(c);
  for (int c = 0; c < d.wb; ++c) o.wave[c] = slot(d.lb + c);
  for (int r = 0; r < d.rb; ++r) o.reg[r] = slot(d.lb + d.wb + r);
  o.op_begin = e.op_begin;
  o.op_end = e.op_end;
  o.transition = e.transition;
  return o;
}

static IoOffsets interp_io(const StageDesc& e, const PartDesc& d) {
  IoOffsets o{};
  auto off = [&](int c) { return uint64_t(1) << d.tq[e.pos[c]]; };
  for (int c = 0; c < d.lb; ++c) o.lane[c] = off(c);
  for (int c = 0; c < d.wb; ++c) o.wave[c] = off(d.lb + c);
  for (int r = 0; r < d.rb; ++r) o.reg[r] = off(d.lb + d.wb + r);
  return o;
}

// The interpreter's descriptor of an op: a dense or real 2x2 with unit entries
// takes the form that leaves their multiplications out.
template <typename T>
static OpDesc<T> device_op(const HostOp& h) {
  OpDesc<T> o{};
  o.kind = h.kind;
  o.b0 = h.b0;
  o.b1 = h.b1;
  for (int i = 0; i < 32; ++i) o.c[i] = (T)h.c[i];
  if (h.kind == OP_CPC || h.kind == OP_CXC) o.b1 = h.cond;
  if (h.kind == OP_F) {
    o.b0 = h.cond;
    o.b1 = h.cond2;
  }
  if (h.kind != OP_U && h.kind != OP_R) return o;
  cd u[4];
  for (int i = 0; i < 4; ++i) u[i] = h.kind == OP_U ? cd(h.c[2 * i], h.c[2 * i + 1]) : cd(h.c[i], 0);
  const cd one(1, 0);
  auto set = [&](int kind, std::initializer_list<double> c) {
    o.kind = kind;
    std::fill(o.c, o.c + 32, T(0));
    int i = 0;
    for (double v : c) o.c[i++] = (T)v;
  };
  if (u[0] == one && u[3] == one) {
    if (u[1].imag() == 0 && u[2].imag() == 0) set(OP_KR, {u[1].real(), u[2].real()});
    else if (u[1].real() == 0 && u[2].real() == 0) set(OP_KI, {u[1].imag(), u[2].imag()});
    else set(OP_K, {u[1].real(), u[1].imag(), u[2].real(), u[2].imag()});
  } else if (u[0] == one && u[1] == one && u[2] == one && u[3] == -one) {
    set(OP_H, {});
  } else if (u[1] == one && u[2] == one) {
    set(OP_P, {u[0].real(), u[0].imag(), u[3].real(), u[3].imag()});
  } else if (u[0] == one && h.kind == OP_U) {
    set(OP_W, {u[1].real(), u[1].imag(), u[2].real(), u[2].imag(), u[3].real(), u[3].imag()});
  }
  return o;
}

// Upload a plan's interpreter descriptors.  stream = NULL: hipMalloc and
// blocking copies; otherwise the stream-ordered allocator and asynchronous
// copies on `stream`, waited for before returning.
template <typename T>
static hs_status upload_plan(const std::vector<CompiledPart>& comp, int dev, DevicePlan** out, hipStream_t stream,
                             const PinnedStaging* pin = nullptr) {
  std::vector<PartDesc> hparts;
  std::vector<IPart> parts;
  std::vector<IStage> stages;
  std::vector<OpDesc<T>> ops;
  auto dp = std::make_unique<DevicePlan>();
  dp->device = dev;
  DevInfo dinfo;
  if (hs_status rc = device_info(dev, &dinfo)) return rc;
  for (const CompiledPart& cp : comp) {
    PartDesc d = cp.desc;
    if (d.rb > kMaxRegBits || d.wb > kMaxWaveBits || d.lb > kLaneBits || cp.stages.size() < 2)
      return fail(HS_E_UNSUPPORTED, "part layout outside the interpreter's limits");
    d.stage_off = (int)stages.size();
    d.lds_bytes = cp.lds_round_trips ? (int)((size_t(1) << d.m) * sizeof(cplx<T>)) : 0;
    const int op0 = (int)ops.size();
    for (const StageDesc& e : cp.stages) {
      IStage is = interp_stage<T>(e, d);
      is.op_begin += op0;
      is.op_end += op0;
      stages.push_back(is);
    }
    IPart ip{};
    ip.load = interp_io(cp.stages.front(), d);
    ip.store = interp_io(cp.stages.back(), d);
    ip.tiles = d.tiles;
    ip.m = d.m;
    ip.lb = d.lb;
    ip.n_stages = d.n_stages;
    for (int i = 0; i < kMaxTile; ++i) ip.tq[i] = d.tq[i];
    for (size_t i = 0; i < cp.ops.size(); ++i) {
      const HostOp& h = cp.ops[i];
      // a factor's op goes before its factors (see apply_op), with their number
      if (h.kind == OP_F && (i == 0 || cp.ops[i - 1].kind != OP_F)) {
        size_t last = i;
        while (cp.ops[last].kind == OP_F) ++last;
        OpDesc<T> all = device_op<T>(cp.ops[last]);
        all.b1 = (int32_t)(last - i);
        ops.push_back(all);
      }
      if (h.kind == OP_FA || h.kind == OP_GA) continue;
      ops.push_back(device_op<T>(h));
    }
    hparts.push_back(d);
    parts.push_back(ip);
    dp->rb.push_back(cp.rb_kernel);
    const int block = 64 << d.wb;
    int per_cu = 0;
    if (hs_status rc = resident_rb<T>(cp.rb_kernel, block, (size_t)d.lds_bytes, &per_cu)) return rc;
    unsigned g = 1;
    uint8_t x = 0;
    part_grid(cp.launch, d.tiles, block, per_cu, dinfo.cus, &g, &x);
    dp->grid.push_back(g);
    dp->xcd.push_back(x);
  }
  if (ops.empty()) ops.push_back(OpDesc<T>{});
  if (parts.empty()) parts.push_back(IPart{});
  if (stages.empty()) stages.push_back(IStage{});
  if (stream) {
    // Nothing here waits for the device: the stream may share a hardware
    // queue with long-running part kernels, and a host wait would hold the
    // caller (a serving thread) until they drain.  The host copies live
    // until a host function after the copies deletes them, and launches
    // elsewhere wait for upload_done on the device.
    dp->async_alloc = true;
    dp->free_stream = stream;
    const size_t b_parts = parts.size() * sizeof(IPart), b_stages = stages.size() * sizeof(IStage),
                 b_ops = ops.size() * sizeof(OpDesc<T>);
    // pinned staging, when it is free and large enough: the copies are then
    // plain DMA with nothing to stage on the host
    const size_t o_stages = (b_parts + 255) & ~size_t(255), o_ops = (o_stages + b_stages + 255) & ~size_t(255);
    if (pin && pin->ptr && o_ops + b_ops <= pin->bytes && hipEventQuery((hipEvent_t)pin->busy) == hipSuccess) {
      char* h = static_cast<char*>(pin->ptr);
      std::memcpy(h, parts.data(), b_parts);
      std::memcpy(h + o_stages, stages.data(), b_stages);
      std::memcpy(h + o_ops, ops.data(), b_ops);
      HIP_TRY(hipMallocAsync((void**)&dp->parts, b_parts, stream));
      HIP_TRY(hipMallocAsync((void**)&dp->stages, b_stages, stream));
      HIP_TRY(hipMallocAsync(&dp->ops, b_ops, stream));
      HIP_TRY(hipMemcpyAsync(dp->parts, h, b_parts, hipMemcpyHostToDevice, stream));
      HIP_TRY(hipMemcpyAsync(dp->stages, h + o_stages, b_stages, hipMemcpyHostToDevice, stream));
      HIP_TRY(hipMemcpyAsync(dp->ops, h + o_ops, b_ops, hipMemcpyHostToDevice, stream));
      HIP_TRY(hipEventRecord((hipEvent_t)pin->busy, stream));  // the staging is free again once this passes
      HIP_TRY(hipEventCreateWithFlags(&dp->upload_done, hipEventDisableTiming));
      HIP_TRY(hipEventRecord(dp->upload_done, stream));
      dp->h_parts = hparts;
      *out = dp.release();
      return HS_OK;
    }
    auto host = std::make_unique<HostDescriptors<T>>();
    host->parts = std::move(parts);
    host->stages = std::move(stages);
    host->ops = std::move(ops);
    HIP_TRY(hipMallocAsync((void**)&dp->parts, host->parts.size() * sizeof(IPart), stream));
    HIP_TRY(hipMallocAsync((void**)&dp->stages, host->stages.size() * sizeof(IStage), stream));
    HIP_TRY(hipMallocAsync(&dp->ops, host->ops.size() * sizeof(OpDesc<T>), stream));
    HIP_TRY(hipMemcpyAsync(dp->parts, host->parts.data(), host->parts.size() * sizeof(IPart),
                           hipMemcpyHostToDevice, stream));
    HIP_TRY(hipMemcpyAsync(dp->stages, host->stages.data(), host->stages.size() * sizeof(IStage),
                           hipMemcpyHostToDevice, stream));
    HIP_TRY(hipMemcpyAsync(dp->ops, host->ops.data(), host->ops.size() * sizeof(OpDesc<T>),
                           hipMemcpyHostToDevice, stream));
    HIP_TRY(hipEventCreateWithFlags(&dp->upload_done, hipEventDisableTiming));
    HIP_TRY(hipEventRecord(dp->upload_done, stream));
    if (hipLaunchHostFunc(stream, HostDescriptors<T>::release, host.get()) == hipSuccess) {
      host.release();  // deleted by the host function
    } else {
      (void)hipGetLastError();
      HIP_TRY(hipStreamSynchronize(stream));  // fallback: wait, then free here
    }
  } else {
    HIP_TRY(hipMalloc(&dp->parts, parts.size() * sizeof(IPart)));
    HIP_TRY(hipMalloc(&dp->stages, stages.size() * sizeof(IStage)));
    HIP_TRY(hipMalloc(&dp->ops, ops.size() * sizeof(OpDesc<T>)));
    HIP_TRY(hipMemcpy(dp->parts, parts.data(), parts.size() * sizeof(IPart), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(dp->stages, stages.data(), stages.size() * sizeof(IStage), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(dp->ops, ops.data(), ops.size() * sizeof(OpDesc<T>), hipMemcpyHostToDevice));
  }
  dp->h_parts = hparts;
  *out = dp.release();
  return HS_OK;
}

template <typename T>
static hs_status launch_part(State* s, DevicePlan* dp, int part) {
  const PartDesc& d = dp->h_parts[part];
  const int block = 64 << d.wb;
  const unsigned grid = dp->grid[part];
  const size_t lds = (size_t)d.lds_bytes;
  cplx<T>* st = (cplx<T>*)s->ptr;
  const IPart* pd = dp->parts + part;
  const IStage* sd = dp->stages + d.stage_off;
  const OpDesc<T>* ops = (const OpDesc<T>*)dp->ops;
  hipStream_t str = stream_of(s);
  const uint32_t xcd = dp->xcd[part];
#define HS_LAUNCH_PART(RB_)                                                                     \
  hipLaunchKernelGGL((part_pass_kernel<T, RB_>), dim3(grid), dim3(block), lds, str, st, pd, sd, ops, \
                     xcd);                                                                      \
  break;
  switch (dp->rb[part]) {
    case 1: HS_LAUNCH_PART(1)
    case 2: HS_LAUNCH_PART(2)
    case 3: HS_LAUNCH_PART(3)
    case 4: HS_LAUNCH_PART(4)
    default: return fail(HS_E_UNSUPPORTED, "no kernel with %d register bits", dp->rb[part]);
  }
#undef HS_LAUNCH_PART
  HIP_TRY(hipGetLastError());
  return HS_OK;
}

// what the interpreter runs for a plan: its parts or its sweeps
static const std::vector<CompiledPart>& interpreted(const Plan* p, bool sweep, int dt) {
  return sweep ? p->sweeps[0][dt].comp : p->comp[dt];
}

static hs_status device_plan(State* s, Plan* p, bool sweep, DevicePlan** out) {
  const int dt = (int)s->dtype;
  auto it = p->dev[sweep][dt].find(s->device);
  if (it != p->dev[sweep][dt].end()) {
    *out = it->second;
    return HS_OK;
  }
  DevicePlan* dp = nullptr;
  const std::vector<CompiledPart>& comp = interpreted(p, sweep, dt);
  hs_status rc = dt == HS_C64 ? upload_plan<float>(comp, s->device, &dp, nullptr)
                              : upload_plan<double>(comp, s->device, &dp, nullptr);
  if (rc) return rc;
  p->dev[sweep][dt][s->device] = dp;
  *out = dp;
  return HS_OK;
}

hs_status dev_plan_upload_async(Plan* p, bool sweep, hs_dtype dtype, int device, void* stream,
                                const PinnedStaging* pin) {
  HIP_TRY(hipSetDevice(device));
  std::lock_guard<std::mutex> lk(p->mu);
  const int dt = (int)dtype;
  if (p->dev[sweep][dt].count(device)) return HS_OK;
  DevicePlan* dp = nullptr;
  const std::vector<CompiledPart>& comp = interpreted(p, sweep, dt);
  hs_status rc = dt == HS_C64 ? upload_plan<float>(comp, device, &dp, (hipStream_t)stream, pin)
                              : upload_plan<double>(comp, device, &dp, (hipStream_t)stream, pin);
  if (rc) {
    device_plan_free(dp);
    return rc;
  }
  p->dev[sweep][dt][device] = dp;
  return HS_OK;
}

hs_status dev_plan_stream_wait(Plan* p, bool sweep, hs_dtype dtype, int device, void* stream) {
  HIP_TRY(hipSetDevice(device));
  hipEvent_t ev = nullptr;
  {
    std::lock_guard<std::mutex> lk(p->mu);
    auto it = p->dev[sweep][(int)dtype].find(device);
    if (it == p->dev[sweep][(int)dtype].end()) return fail(HS_E_STATE, "plan not uploaded for this device");
    ev = it->second->upload_done;
  }
  if (ev) HIP_TRY(hipStreamWaitEvent((hipStream_t)stream, ev, 0));
  return HS_OK;
}

hs_status dev_run_part(State* s, Plan* p, int part, bool sweep) {
  HIP_TRY(hipSetDevice(s->device));
  DevicePlan* dp = nullptr;
  {
    std::lock_guard<std::mutex> lk(p->mu);
    if (hs_status rc = device_plan(s, p, sweep, &dp)) return rc;
  }
  return s->dtype == HS_C64 ? launch_part<float>(s, dp, part) : launch_part<double>(s, dp, part);
}

// Kernel and launch shape of a fused part on `tiles` tiles.
//
// w = 4 and complex128 w = 7 (U is 256 KiB) run the plain kernel, one group of
// tiles a workgroup; w = 5 and up run fused_lds_kernel.  Its workgroups take
// `chunk` consecutive groups.  w = 5 waits on HBM, which goes fastest when the
// workgroups in flight cover one narrow run of memory: as few groups as pay
// for reading U (28 qubits, sweeps of the state; complex64 chunks of 2 / 4 /
// 16 and a persistent grid: 1.02 / 1.00 / 1.08 / 1.09; complex128 0.94 / 1.00 /
// 1.21 / 1.06).  w = 6 and 7 wait on the matrix cores and on reading U: one
// round of two workgroups a CU (w = 7: one, by its LDS; complex64 w = 6 chunks
// of 4 / 16 / that: 1.47 / 1.48 / 1.38).
//
// hs_tune("fused_shape") asks for the kernel that keeps U in registers or reads
// it from L2 for w = 4, 5: 0 = one group a workgroup, 1 = its software-pipelined
// form and 2 = its plain form on a persistent grid.
template <typename T>
static hs_status fused_launch(int w, uint64_t tiles, int device, FusedLaunch* l) {
  l->w = w;
  if (!w) return HS_OK;
  const int shape = w <= 5 ? fused_launch_shape() : -1;
  const bool lds = w > 4 && shape < 0 && !(w == 7 && sizeof(T) == 8);
  switch (w) {
    case 4:
      l->fn = shape == 1 ? (const void*)fused_pass_kernel<T, 4, true> : (const void*)fused_pass_kernel<T, 4, false>;
      break;
    case 5:
      l->fn = lds          ? (const void*)fused_lds_kernel<T, 5>
              : shape == 1 ? (const void*)fused_pass_kernel<T, 5, true>
                           : (const void*)fused_pass_kernel<T, 5, false>;
      break;
    case 6: l->fn = (const void*)fused_lds_kernel<T, 6>; break;
    case 7:
      if constexpr (sizeof(T) == 4) l->fn = (const void*)fused_lds_kernel<T, 7>;
      else l->fn = (const void*)fused_pass_kernel<T, 7, false>;
      break;
    default: return fail(HS_E_UNSUPPORTED, "no fused kernel for %d qubits", w);
  }
  DevInfo di;
  if (hs_status rc = device_info(device, &di)) return rc;
  if (lds) l->block = w == 7 ? fused_lds_threads<T, 7>() : fused_lds_threads<T, 6>();
  const uint64_t per_wg = l->block / 64, groups = (tiles + per_wg - 1) / per_wg;
  uint64_t chunk = 1, g = groups;
  if (lds) {
    if (w == 5) chunk = sizeof(T) == 4 ? 4 : 2;
    else chunk = std::max<uint64_t>(1, groups / ((uint64_t)di.cus * (w == 6 ? 2 : 1)));
    g = (groups + chunk - 1) / chunk;
  } else if (shape > 0) {
    int per_cu = 0;
    HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, l->fn, l->block, 0));
    g = std::min<uint64_t>(groups, (uint64_t)std::max(1, per_cu) * di.cus);
  }
  const uint64_t most = (uint64_t(1) << 31) / l->block;
  if (g > most && lds) {
    chunk = (groups + most - 1) / most;
    g = (groups + chunk - 1) / chunk;
  }
  g = std::max<uint64_t>(1, std::min(g, most));
  // each XCD sweeps a contiguous eighth of the groups; with chunks, the eighth
  // has to be whole chunks
  if (groups % (8 * chunk) == 0 && g >= 8) {
    g &= ~uint64_t(7);
    l->xcd = 1;
  }
  l->chunk = (uint32_t)chunk;
  l->grid = (unsigned)g;
  return HS_OK;
}

template <typename T>
static hs_status upload_fused(const std::vector<FusedPart>& parts, int device, DeviceFused** out) {
  std::vector<FusedDesc> fds;
  std::vector<T> mats;
  auto dp = std::unique_ptr<DeviceFused, void (*)(DeviceFused*)>(new DeviceFused, device_fused_free);
  dp->device = device;
  for (const FusedPart& f : parts) {
    FusedDesc d{};
    d.w = f.w;
    d.m = f.m;
    d.tiles = f.tiles;
    d.u_off = (int32_t)mats.size();
    std::memcpy(d.sq, f.sq, sizeof d.sq);
    std::memcpy(d.pq, f.pq, sizeof d.pq);
    std::memcpy(d.tq, f.tq, sizeof d.tq);
    // fragment order (see fused_pass_kernel): real parts, then imaginary
    const int R = 1 << f.w;
    for (int part_im = 0; part_im < 2 && f.w > 0; ++part_im)
      for (int rb = 0; rb < R / 16; ++rb)
        for (int ks = 0; ks < R / 4; ++ks)
          for (int l = 0; l < 64; ++l) {
            const cd z = f.u[(size_t)(16 * rb + l % 16) * R + 4 * ks + l / 16];
            mats.push_back((T)(part_im ? z.imag() : z.real()));
          }
    fds.push_back(d);
    FusedLaunch l;
    if (hs_status rc = fused_launch<T>(f.w, f.tiles, device, &l)) return rc;
    dp->launch.push_back(l);
  }
  if (mats.empty()) mats.push_back(T(0));
  if (fds.empty()) fds.push_back(FusedDesc{});
  HIP_TRY(hipMalloc(&dp->parts, fds.size() * sizeof(FusedDesc)));
  HIP_TRY(hipMalloc(&dp->mat, mats.size() * sizeof(T)));
  HIP_TRY(hipMemcpy(dp->parts, fds.data(), fds.size() * sizeof(FusedDesc), hipMemcpyHostToDevice));
  HIP_TRY(hipMemcpy(dp->mat, mats.data(), mats.size() * sizeof(T), hipMemcpyHostToDevice));
  *out = dp.release();
  return HS_OK;
}

hs_status dev_run_fused(State* s, Plan* p, int part, bool of_set) {
  HIP_TRY(hipSetDevice(s->device));
  const int dt = (int)s->dtype;
  DeviceFused* dp = nullptr;
  {
    std::lock_guard<std::mutex> lk(p->mu);
    auto it = p->fdev[of_set][dt].find(s->device);
    if (it != p->fdev[of_set][dt].end()) {
      dp = it->second;
    } else {
      const std::vector<FusedPart>& parts = of_set ? p->fused_set[dt].parts : p->fused;
      hs_status rc = s->dtype == HS_C64 ? upload_fused<float>(parts, s->device, &dp)
                                        : upload_fused<double>(parts, s->device, &dp);
      if (rc) return rc;
      p->fdev[of_set][dt][s->device] = dp;
    }
  }
  FusedLaunch& l = dp->launch[part];
  if (!l.w) return fail(HS_E_UNSUPPORTED, "part %d has no fused form", part);
  void* st = s->ptr;
  const FusedDesc* fd = dp->parts + part;
  void* args[] = {&st, &fd, &dp->mat, &l.xcd, &l.chunk};  // the plain kernels have no fifth argument
  HIP_TRY(hipLaunchKernel(l.fn, dim3(l.grid), dim3(l.block), args, 0, stream_of(s)));
  return HS_OK;
}

// ---- readout ----------------------------------------------------------------
static hs_status ensure_scratch(State* s, size_t bytes) {
  if (s->scratch_bytes >= bytes) return HS_OK;
  if (s->scratch) HIP_TRY(hipFree(s->scratch));
  s->scratch = nullptr;
  s->scratch_bytes = 0;
  HIP_TRY(hipMalloc(&s->scratch, bytes));
  s->scratch_bytes = bytes;
  return HS_OK;
}

// Pinned staging of readouts, made on a state's first one: two buffers that
// the readout kernels write over PCIe, one being copied out by the host while
// the kernel of the next chunk fills the other.  (Device scratch, a copy into
// the caller's pageable memory and a wait for every chunk took 615 us for 2^20
// probabilities of a 27-qubit state and 28 us for 4,096 amplitudes.)
constexpr size_t kStageBytes = size_t(1) << 20;

hs_status dev_read_stage_create(ReadStage* r) {
  if (r->buf) return HS_OK;
  void* buf = nullptr;
  if (hipHostMalloc(&buf, 2 * kStageBytes, hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    return fail(HS_E_NOMEM, "pinned readout staging of %zu bytes", 2 * kStageBytes);
  }
  r->buf = buf;
  for (void*& ev : r->done) {
    hipEvent_t e = nullptr;
    HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    ev = e;
  }
  return HS_OK;
}

void dev_read_stage_free(ReadStage* r) {
  for (void*& ev : r->done) {
    if (ev) (void)hipEventDestroy((hipEvent_t)ev);
    ev = nullptr;
  }
  if (r->buf) (void)hipHostFree(r->buf);
  r->buf = nullptr;
}

// `count` items in chunks of `chunk` through the two buffers: launch(b, done, c)
// queues the kernel of items [done, done + c) on buffer b, take(b, done, c)
// copies them out.
template <typename Launch, typename Take>
static hs_status staged(State* s, uint64_t count, uint64_t chunk, Launch&& launch, Take&& take) {
  uint64_t queued = 0;
  for (uint64_t done = 0, i = 0; done < count; ++i) {
    while (queued < count && queued < (i + 2) * chunk) {
      const uint64_t c = std::min(chunk, count - queued);
      const int b = (int)(queued / chunk & 1);
      if (hs_status rc = launch(b, queued, c)) {
        (void)hipStreamSynchronize(stream_of(s));  // the other buffer's kernel may be running
        return rc;
      }
      HIP_TRY(hipEventRecord((hipEvent_t)s->stage.done[b], stream_of(s)));
      queued += c;
    }
    const uint64_t c = std::min(chunk, count - done);
    HIP_TRY(hipEventSynchronize((hipEvent_t)s->stage.done[i & 1]));
    take((int)(i & 1), done, c);
    done += c;
  }
  return HS_OK;
}

hs_status dev_norm(State* s, double* out) {
  HIP_TRY(hipSetDevice(s->device));
  if (hs_status rc = ensure_scratch(s, kNormBlocks * sizeof(double))) return rc;
  if (hs_status rc = dev_read_stage_create(&s->stage)) return rc;
  double* part = (double*)s->scratch;
  double* res = (double*)s->stage.buf;
  const uint64_t N = uint64_t(1) << s->n;
  if (s->dtype == HS_C64)
    hipLaunchKernelGGL(norm_partial<float>, dim3(kNormBlocks), dim3(kNormThreads), 0, stream_of(s),
                       (const cplx<float>*)s->ptr, N, part);
  else
    hipLaunchKernelGGL(norm_partial<double>, dim3(kNormBlocks), dim3(kNormThreads), 0, stream_of(s),
                       (const cplx<double>*)s->ptr, N, part);
  hipLaunchKernelGGL(norm_final, dim3(1), dim3(kNormThreads), 0, stream_of(s), part, res);
  HIP_TRY(hipGetLastError());
  HIP_TRY(hipStreamSynchronize(stream_of(s)));
  *out = *res;
  return HS_OK;
}

// ---- the norm without allocation -------------------------------------------
// The norm's partial sums live in a file-scope device array instead of the
// state's lazily allocated scratch, so this path never calls the allocator.
// Each device holds its own copy; host code uses only the address that
// hipGetSymbolAddress reports for the current device (the array's name is a
// host-side stand-in, not a device address).  Every call on a device shares
// that device's copy: calls that overlap on one device race.  Nothing in it
// must start at zero: norm_partial writes every one of its kNormBlocks
// partial sums (zero for a block with no amplitudes) before norm_final
// reads them, and norm_final writes the result slot.
constexpr int kNoAllocDoubles = kNormBlocks + 8;  // 8,256 bytes per device
static __device__ __align__(256) double scratch[kNoAllocDoubles];

constexpr int kMaxDevices = 64;
static std::mutex g_noalloc_mu;
static double* g_noalloc_ptr[kMaxDevices] = {};

// Address of this device's copy of `scratch`, looked up once per device with
// that device current.
static hs_status noalloc_scratch(int device, double** out) {
  if (device < 0 || device >= kMaxDevices) return fail(HS_E_ARG, "device %d out of range", device);
  std::lock_guard<std::mutex> lk(g_noalloc_mu);
  if (!g_noalloc_ptr[device]) {
    HIP_TRY(hipSetDevice(device));
    void* ptr = nullptr;
    HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    g_noalloc_ptr[device] = (double*)ptr;
  }
  *out = g_noalloc_ptr[device];
  return HS_OK;
}

hs_status dev_norm_noalloc(State* s, double* out) {
  HIP_TRY(hipSetDevice(s->device));
  static_assert(kNormBlocks + 1 <= kNoAllocDoubles, "partials and result must fit the array");
  double* part = nullptr;
  if (hs_status rc = noalloc_scratch(s->device, &part)) return rc;
  double* res = part + kNormBlocks;
  const uint64_t N = uint64_t(1) << s->n;
  if (s->dtype == HS_C64)
    hipLaunchKernelGGL(norm_partial<float>, dim3(kNormBlocks), dim3(kNormThreads), 0, stream_of(s),
                       (const cplx<float>*)s->ptr, N, part);
  else
    hipLaunchKernelGGL(norm_partial<double>, dim3(kNormBlocks), dim3(kNormThreads), 0, stream_of(s),
                       (const cplx<double>*)s->ptr, N, part);
  hipLaunchKernelGGL(norm_final, dim3(1), dim3(kNormThreads), 0, stream_of(s), part, res);
  HIP_TRY(hipGetLastError());
  HIP_TRY(hipMemcpyAsync(out, res, sizeof(double), hipMemcpyDeviceToHost, stream_of(s)));
  HIP_TRY(hipStreamSynchronize(stream_of(s)));
  return HS_OK;
}

hs_status dev_read(State* s, uint64_t first, uint64_t count, double* out, bool probs) {
  HIP_TRY(hipSetDevice(s->device));
  if (hs_status rc = dev_read_stage_create(&s->stage)) return rc;
  const uint64_t per = probs ? 1 : 2, chunk = kStageBytes / (per * sizeof(double));
  auto buffer = [&](int b) { return (double*)((char*)s->stage.buf + b * kStageBytes); };
  return staged(
      s, count, chunk,
      [&](int b, uint64_t at, uint64_t c) -> hs_status {
        unsigned grid;
        if (hs_status rc = stream_grid(s->device, c, &grid)) return rc;
        if (s->dtype == HS_C64)
          hipLaunchKernelGGL(readout_kernel<float>, dim3(grid), dim3(256), 0, stream_of(s),
                             (const cplx<float>*)s->ptr, first + at, c, probs ? 1 : 0, buffer(b));
        else
          hipLaunchKernelGGL(readout_kernel<double>, dim3(grid), dim3(256), 0, stream_of(s),
                             (const cplx<double>*)s->ptr, first + at, c, probs ? 1 : 0, buffer(b));
        HIP_TRY(hipGetLastError());
        return HS_OK;
      },
      [&](int b, uint64_t at, uint64_t c) { std::memcpy(out + at * per, buffer(b), c * per * sizeof(double)); });
}

// Amplitudes at host-given indices (validated < 2^n by the caller), widened
// to complex128; the kernel reads the indices from the staging buffer too.
hs_status dev_read_at(State* s, const uint64_t* idx, uint64_t count, double* out) {
  HIP_TRY(hipSetDevice(s->device));
  if (hs_status rc = dev_read_stage_create(&s->stage)) return rc;
  const uint64_t chunk = kStageBytes / 32;  // 256 KiB of indices, 512 KiB of output
  auto indices = [&](int b) { return (uint64_t*)((char*)s->stage.buf + b * kStageBytes); };
  auto values = [&](int b) { return (double*)(indices(b) + chunk); };
  return staged(
      s, count, chunk,
      [&](int b, uint64_t at, uint64_t c) -> hs_status {
        unsigned grid;
        if (hs_status rc = stream_grid(s->device, c, &grid)) return rc;
        std::memcpy(indices(b), idx + at, c * sizeof(uint64_t));
        if (s->dtype == HS_C64)
          hipLaunchKernelGGL(gather_kernel<float>, dim3(grid), dim3(256), 0, stream_of(s),
                             (const cplx<float>*)s->ptr, indices(b), c, values(b));
        else
          hipLaunchKernelGGL(gather_kernel<double>, dim3(grid), dim3(256), 0, stream_of(s),
                             (const cplx<double>*)s->ptr, indices(b), c, values(b));
        HIP_TRY(hipGetLastError());
        return HS_OK;
      },
      [&](int b, uint64_t at, uint64_t c) { std::memcpy(out + 2 * at, values(b), c * 2 * sizeof(double)); });
}

hs_status dev_copy_probe(const void* src, void* dst, size_t bytes, void* stream) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  unsigned grid;
  const uint64_t n16 = bytes / 16;
  if (hs_status rc = stream_grid(dev, n16, &grid)) return rc;
  hipLaunchKernelGGL(copy_probe_kernel, dim3(grid), dim3(256), 0, (hipStream_t)stream,
                     (const uint4*)src, (uint4*)dst, n16);
  HIP_TRY(hipGetLastError());
  return HS_OK;
}

hs_status dev_sync(State* s) {
  HIP_TRY(hipSetDevice(s->device));
  HIP_TRY(hipStreamSynchronize(stream_of(s)));
  return HS_OK;
}

}  // namespace hisv
