// gfx950 kernels of the median-dual Nabla operators.
//
// Every operator is a gather over a node's incident edges (the edge sums of
// the finite-volume operators listed in Section 2.3 of the report, evaluated
// node by node): the output element (node i, level k) is written by exactly
// one lane, neighbour values are read in a fixed slot order, and nothing is
// accumulated across lanes, so there are no atomics and reruns are bitwise
// identical.  The path is a sparse stencil whose dense dimension is the level
// column, so it is bound by memory traffic and uses no matrix cores.
//
// Mapping.  Fields are [node][level] with levels innermost.  A 64-lane wave
// owns G = 64 / P nodes at a time, P lanes per node; lane t of a node handles
// levels t, t + P, t + 2P, ... of its column.  P is chosen per level count so
// that the column fills the lanes well (P = nlev for columns of at most 32
// levels, else 64, 32 or 16, e.g. 16 lanes x 9 slices for 137 levels).  The
// lane -> node assignment is fixed, so each lane reads its node's table row
// (neighbour offsets and coefficient pairs) once and keeps it in registers for
// the whole column.  U level slices are processed per iteration with all
// neighbour loads issued before any arithmetic, which keeps many independent
// loads in flight per wave; loads of slices past the column end are clamped
// to the last level (cache hits) and their results are not stored.
//
// Cache reuse.  Each node value is read by the node and its ~6 neighbours,
// two of them in the row above and two in the row below; at 137 FP32 levels
// three rows of the O1280 grid already exceed an XCD's 4 MB L2.  Work
// therefore follows a node order built on the host: bands of rows, nodes of a
// band sorted by longitude, so the rows above and below are touched at the
// same longitude at about the same time.  Workgroups are dispatched
// round-robin over the eight XCDs; with remapping on, workgroup b works on
// logical block (b mod 8) * ceil(nblocks / 8) + b / 8, so each XCD walks a
// contiguous part of the order (whole bands) in its own L2.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <mutex>
#include <type_traits>

#include "launch.hpp"

namespace atlasnabla {

namespace {

using bf16_t = uint16_t;

constexpr int kLapStride = 24;   // two-ring record: up to 23 entries + the count

template <class S> struct Traits;
template <> struct Traits<double> { using C = double; using C2 = double2; };
template <> struct Traits<float> { using C = float; using C2 = float2; };
template <> struct Traits<bf16_t> { using C = float; using C2 = float2; };

__device__ __forceinline__ float bf16_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

// FP32 to BF16, round to nearest even, a NaN kept as a quiet NaN with its
// payload's top bits: gfx950's v_cvt_pk_bf16_f32, one instruction for two
// values (checked equal, on all 2^32 inputs, to the rounding written out on
// the bits: add 0x7fff plus the lowest kept bit, keep the top half).
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t f32_to_bf16(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ uint32_t f32x2_to_bf16x2(float x, float y) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2_t));
}

__device__ __forceinline__ double ld1(const double* p) { return *p; }
__device__ __forceinline__ float ld1(const float* p) { return *p; }
__device__ __forceinline__ float ld1(const bf16_t* p) { return bf16_to_f32(*p); }

__device__ __forceinline__ double2 ld2(const double* p) { return *reinterpret_cast<const double2*>(p); }
__device__ __forceinline__ float2 ld2(const float* p) { return *reinterpret_cast<const float2*>(p); }
__device__ __forceinline__ float2 ld2(const bf16_t* p) {
  const uint32_t w = *reinterpret_cast<const uint32_t*>(p);
  return make_float2(bf16_to_f32(w & 0xffffu), bf16_to_f32(w >> 16));
}

// Output stores: plain, or non-temporal (streamed past L2) when the launch
// asks for it.  Plain stores let L2 merge the partial cache lines shared by
// the columns of neighbouring nodes.
typedef double f64x2 __attribute__((ext_vector_type(2)));

template <bool NT, class T>
__device__ __forceinline__ void st_raw(T* p, T v) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

template <bool NT>
__device__ __forceinline__ void st1(double* p, double v) { st_raw<NT>(p, v); }
template <bool NT>
__device__ __forceinline__ void st1(float* p, float v) { st_raw<NT>(p, v); }
template <bool NT>
__device__ __forceinline__ void st1(bf16_t* p, float v) { st_raw<NT>(p, (bf16_t)f32_to_bf16(v)); }

template <bool NT>
__device__ __forceinline__ void st2(double* p, double x, double y) {
  st_raw<NT>(reinterpret_cast<f64x2*>(p), f64x2{x, y});
}
template <bool NT>
__device__ __forceinline__ void st2(float* p, float x, float y) {
  st_raw<NT>(reinterpret_cast<f32x2*>(p), f32x2{x, y});
}
template <bool NT>
__device__ __forceinline__ void st2(bf16_t* p, float x, float y) {
  st_raw<NT>(reinterpret_cast<uint32_t*>(p), f32x2_to_bf16x2(x, y));
}

// Read-only table data read through the constant address space: with a
// wave-uniform address the compiler fetches it with scalar loads into scalar
// registers.  Valid because no kernel writes the tables.
template <class T>
__device__ __forceinline__ T ld_const(const T* p) {
  return *(const __attribute__((address_space(4))) T*)(p);
}
__device__ __forceinline__ int32_t ld_uniform(const int32_t* p) { return ld_const(p); }
__device__ __forceinline__ float2 ld_uniform(const float2* p) {
  const float* q = reinterpret_cast<const float*>(p);
  return make_float2(ld_const(q), ld_const(q + 1));
}
__device__ __forceinline__ double2 ld_uniform(const double2* p) {
  const double* q = reinterpret_cast<const double*>(p);
  return make_double2(ld_const(q), ld_const(q + 1));
}

}  // namespace

struct Args {
  const int32_t* order; // [V] node processing order (a permutation)
  const int32_t* runs;  // [nruns][2] (first node, count): the same order as row runs
  int64_t nruns;
  const int32_t* nbr;   // [V][8] neighbour table or [V][24] two-ring table
  const void* coef;     // coefficient pairs or two-ring weights (same row layout)
  const void* in;
  void* out;
  int64_t V;
  int32_t L;            // levels
  int32_t P;            // lanes per node (64 / P nodes per wave)
  int32_t npw;          // node groups (or runs) per wave per workgroup
  int32_t nt;           // non-temporal output stores
};

namespace {

// ---- one node group per wave --------------------------------------------------
//
// NS: table entries read per node (7 = every slot, padded with the node itself
// and zero coefficients; 6 when every node of the wave has degree 6; 23 or 18
// for the two-ring table).  Padding entries add exact zeros.  Entries are
// consumed in slot order, which fixes the summation order of every element.

template <class S, int OP, int NS, int U>
__device__ __forceinline__ void run_1ring(const Args& a, int64_t nd, bool ok, int t) {
  using C = typename Traits<S>::C;
  using C2 = typename Traits<S>::C2;
  const int32_t* nbp = a.nbr + nd * 8;
  const C2* cfp = static_cast<const C2*>(a.coef) + nd * 8;
  const uint32_t L = (uint32_t)a.L;
  uint32_t off[NS];
  C2 cf[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    off[s] = (uint32_t)nbp[s] * L;
    cf[s] = cfp[s];
  }
  const C2 dg = cfp[7];
  const uint32_t self = (uint32_t)nd * L;
  const S* __restrict__ in = static_cast<const S*>(a.in);
  S* __restrict__ out = static_cast<S*>(a.out);
  const int P = a.P;
  const int nsl = (a.L + P - 1) / P;
  for (int r0 = 0; r0 < nsl; r0 += U) {
    uint32_t kc[U];
    bool st[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t k = (uint32_t)(t + P * (r0 + u));
      st[u] = ok && k < L;
      kc[u] = k < L ? k : L - 1;
    }
    if constexpr (OP == OP_GRAD || OP == OP_DIVT) {
      C v[U][NS], x0[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int s = 0; s < NS; ++s) v[u][s] = ld1(in + (size_t)(off[s] + kc[u]));
        x0[u] = ld1(in + (size_t)(self + kc[u]));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        C ax, ay;
        if constexpr (OP == OP_GRAD) {
          // difference form: sum_s (a, b)_s (f_n - f_i)
          ax = 0;
          ay = 0;
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            const C d = v[u][s] - x0[u];
            ax = fma(cf[s].x, d, ax);
            ay = fma(cf[s].y, d, ay);
          }
        } else {
          // divergence adjoint: (A, B)_i d_i + sum_s (c, d)_{n,rev} d_n
          ax = dg.x * x0[u];
          ay = dg.y * x0[u];
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            ax = fma(cf[s].x, v[u][s], ax);
            ay = fma(cf[s].y, v[u][s], ay);
          }
        }
        if (st[u]) {
          if (a.nt) st2<true>(out + 2 * (size_t)(self + kc[u]), ax, ay);
          else st2<false>(out + 2 * (size_t)(self + kc[u]), ax, ay);
        }
      }
    } else {
      // divergence and gradient adjoint: diag . in_i + sum_s (x, y)_s . in_n
      C2 v[U][NS], x0[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int s = 0; s < NS; ++s) v[u][s] = ld2(in + 2 * (size_t)(off[s] + kc[u]));
        x0[u] = ld2(in + 2 * (size_t)(self + kc[u]));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        C acc = dg.x * x0[u].x;
        acc = fma(dg.y, x0[u].y, acc);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          acc = fma(cf[s].x, v[u][s].x, acc);
          acc = fma(cf[s].y, v[u][s].y, acc);
        }
        if (st[u]) {
          if (a.nt) st1<true>(out + (size_t)(self + kc[u]), acc);
          else st1<false>(out + (size_t)(self + kc[u]), acc);
        }
      }
    }
  }
}

// fused Laplacian over the two-ring: sum_m W_im (f_m - f_i)
template <class S, int NS, int U>
__device__ __forceinline__ void run_lap(const Args& a, int64_t nd, bool ok, int t) {
  using C = typename Traits<S>::C;
  const int32_t* nbp = a.nbr + nd * kLapStride;
  const C* wp = static_cast<const C*>(a.coef) + nd * kLapStride;
  const uint32_t L = (uint32_t)a.L;
  uint32_t off[NS];
  C w[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    off[s] = (uint32_t)nbp[s] * L;
    w[s] = wp[s];
  }
  const uint32_t self = (uint32_t)nd * L;
  const S* __restrict__ in = static_cast<const S*>(a.in);
  S* __restrict__ out = static_cast<S*>(a.out);
  const int P = a.P;
  const int nsl = (a.L + P - 1) / P;
  for (int r0 = 0; r0 < nsl; r0 += U) {
    uint32_t kc[U];
    bool st[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t k = (uint32_t)(t + P * (r0 + u));
      st[u] = ok && k < L;
      kc[u] = k < L ? k : L - 1;
    }
    C v[U][NS], x0[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int s = 0; s < NS; ++s) v[u][s] = ld1(in + (size_t)(off[s] + kc[u]));
      x0[u] = ld1(in + (size_t)(self + kc[u]));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      C acc = 0;
#pragma unroll
      for (int s = 0; s < NS; ++s) acc = fma(w[s], v[u][s] - x0[u], acc);
      if (st[u]) {
        if (a.nt) st1<true>(out + (size_t)(self + kc[u]), acc);
        else st1<false>(out + (size_t)(self + kc[u]), acc);
      }
    }
  }
}

// gbase: first position (in the node order) of the wave's group of G nodes.
template <class S, int OP, int U>
__device__ __forceinline__ void run_group(const Args& a, int64_t gbase, int lane) {
  const int P = a.P;
  const int G = 64 / P;
  const int j = lane / P;
  const int t = lane - j * P;
  const int64_t q = gbase + j;
  const bool ok = j < G && q < a.V;
  const int64_t nd = a.order[ok ? q : gbase];   // gbase < V: a valid node for idle lanes
  // The padded wide variants serve the few waves that touch a node of
  // degree 5 or 7 (16 + 4 per mesh) or a wide two-ring; they run one slice
  // per iteration so that they do not set the register budget of the kernel.
  if constexpr (OP == OP_LAP) {
    const int cnt = a.nbr[nd * kLapStride + kLapStride - 1];
    if (__all(cnt <= 18)) run_lap<S, 18, U>(a, nd, ok, t);
    else run_lap<S, kLapStride - 1, 1>(a, nd, ok, t);
  } else {
    const int deg = a.nbr[nd * 8 + 7] & 0xff;
    if (__all(deg == 6)) run_1ring<S, OP, 6, U>(a, nd, ok, t);
    else run_1ring<S, OP, 7, 1>(a, nd, ok, t);
  }
}

// ---- row-window walk (1-ring operators, columns of more than 32 levels) ----
//
// A wave walks a run of consecutive nodes of one latitude row, 64 lanes =
// 64 levels, U slices of the column at once.  For a window-eligible node the
// slots in neighbour order are [row above (cu), left, right, row below (cl)],
// the previous node's self and right neighbour are this node's left and self,
// and the previous node's last neighbour above (below) is this node's first
// one above (below).  So a node needs only 1 + (cu - 1) + (cl - 1) new column
// loads (3 for the usual cu = cl = 2) instead of deg + 1.  Other nodes (run
// starts, polar rows, neighbours wrapping past the zero meridian) load every
// slot.  Either way the values are combined in slot order with the same fused
// multiply-adds as the per-lane path, so all paths give identical bits.

// The operators of two output components.
template <int OP>
constexpr bool kTwoOut = OP == OP_GRAD || OP == OP_DIVT || OP == OP_DIVTA;

template <class S, int OP>
struct WinT {
  using C = typename Traits<S>::C;
  using C2 = typename Traits<S>::C2;
  static constexpr bool kVecIn = (OP == OP_DIV || OP == OP_GRADT || OP == OP_DIVCURL);
  using X = typename std::conditional<kVecIn, C2, C>::type;
  static __device__ __forceinline__ X ld(const S* __restrict__ in, uint32_t idx) {
    if constexpr (kVecIn) return ld2(in + 2 * (size_t)idx);
    else return ld1(in + (size_t)idx);
  }
};

// Combine deg slot values (slot order) with the node's coefficients: r0 (and
// r1 for the two-component outputs of OP_GRAD and OP_DIVT).
template <class S, int OP, int DEG>
__device__ __forceinline__ void win_combine(const typename WinT<S, OP>::X x0, const typename WinT<S, OP>::X* v,
                                            const typename Traits<S>::C2* cf, typename Traits<S>::C2 dg,
                                            typename Traits<S>::C& r0, typename Traits<S>::C& r1) {
  using C = typename Traits<S>::C;
  if constexpr (kTwoOut<OP>) {
    C ax, ay;
    if constexpr (OP == OP_GRAD) {
      ax = 0;
      ay = 0;
#pragma unroll
      for (int s = 0; s < DEG; ++s) {
        const C d = v[s] - x0;
        ax = fma(cf[s].x, d, ax);
        ay = fma(cf[s].y, d, ay);
      }
    } else {
      ax = dg.x * x0;
      ay = dg.y * x0;
#pragma unroll
      for (int s = 0; s < DEG; ++s) {
        ax = fma(cf[s].x, v[s], ax);
        ay = fma(cf[s].y, v[s], ay);
      }
    }
    r0 = ax;
    r1 = ay;
  } else {
    C acc = dg.x * x0.x;
    acc = fma(dg.y, x0.y, acc);
#pragma unroll
    for (int s = 0; s < DEG; ++s) {
      acc = fma(cf[s].x, v[s].x, acc);
      acc = fma(cf[s].y, v[s].y, acc);
    }
    r0 = acc;
    r1 = 0;
  }
}

// Store of a combined value at node-level index o (two components for
// OP_GRAD and OP_DIVT).
template <class S, int OP>
__device__ __forceinline__ void win_store(S* __restrict__ out, uint32_t o, int nt, typename Traits<S>::C r0,
                                          typename Traits<S>::C r1) {
  if constexpr (kTwoOut<OP>) {
    if (nt) st2<true>(out + 2 * (size_t)o, r0, r1);
    else st2<false>(out + 2 * (size_t)o, r0, r1);
  } else {
    if (nt) st1<true>(out + (size_t)o, r0);
    else st1<false>(out + (size_t)o, r0);
  }
}

// Combine and store (lanes with st set).
template <class S, int OP, int DEG>
__device__ __forceinline__ void win_emit(S* __restrict__ out, uint32_t o, bool st, int nt,
                                         const typename WinT<S, OP>::X x0, const typename WinT<S, OP>::X* v,
                                         const typename Traits<S>::C2* cf, typename Traits<S>::C2 dg) {
  typename Traits<S>::C r0, r1;
  win_combine<S, OP, DEG>(x0, v, cf, dg, r0, r1);
  if (st) win_store<S, OP>(out, o, nt, r0, r1);
}

// Run-time choice among register values, written as element-wise selects so
// that no private array is indexed at run time.
__device__ __forceinline__ float pick3(int k, float a, float b, float c) { return k == 0 ? a : (k == 1 ? b : c); }
__device__ __forceinline__ double pick3(int k, double a, double b, double c) { return k == 0 ? a : (k == 1 ? b : c); }
__device__ __forceinline__ float2 pick3(int k, float2 a, float2 b, float2 c) {
  return make_float2(pick3(k, a.x, b.x, c.x), pick3(k, a.y, b.y, c.y));
}
__device__ __forceinline__ double2 pick3(int k, double2 a, double2 b, double2 c) {
  return make_double2(pick3(k, a.x, b.x, c.x), pick3(k, a.y, b.y, c.y));
}
template <class T>
__device__ __forceinline__ T pick4(int k, T a, T b, T c, T d) { return k == 3 ? d : pick3(k, a, b, c); }

template <class S, int OP, int U>
struct WinState {
  typename WinT<S, OP>::X self[U], right[U], up[U], lo[U];
};

// Full step: every slot loaded (slot order), one slice at a time.
template <class S, int OP, int U>
__device__ __forceinline__ void win_full(const Args& a, int32_t i, const int32_t* nbp, int deg, int cu, bool eligible,
                                         const typename Traits<S>::C2* cf, typename Traits<S>::C2 dg,
                                         const uint32_t* kc, const bool* st, WinState<S, OP, U>& w) {
  using X = typename WinT<S, OP>::X;
  const S* __restrict__ in = static_cast<const S*>(a.in);
  const uint32_t L = (uint32_t)a.L;
  uint32_t off[7];
#pragma unroll
  for (int s = 0; s < 7; ++s) off[s] = (uint32_t)ld_uniform(nbp + s) * L;   // padded with the node itself
  const uint32_t self = (uint32_t)i * L;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    X v[7];
#pragma unroll
    for (int s = 0; s < 7; ++s) v[s] = WinT<S, OP>::ld(in, off[s] + kc[u]);
    const X x0 = WinT<S, OP>::ld(in, self + kc[u]);
    S* out = static_cast<S*>(a.out);
    switch (deg) {
      case 6: win_emit<S, OP, 6>(out, self + kc[u], st[u], a.nt, x0, v, cf, dg); break;
      case 5: win_emit<S, OP, 5>(out, self + kc[u], st[u], a.nt, x0, v, cf, dg); break;
      case 7: win_emit<S, OP, 7>(out, self + kc[u], st[u], a.nt, x0, v, cf, dg); break;
      case 4: win_emit<S, OP, 4>(out, self + kc[u], st[u], a.nt, x0, v, cf, dg); break;
      default: win_emit<S, OP, 3>(out, self + kc[u], st[u], a.nt, x0, v, cf, dg); break;
    }
    if (eligible) {
      // eligible nodes have cu in 1..3 and deg = cu + cl + 2 with cl in 1..3
      w.self[u] = x0;
      w.right[u] = pick3(cu - 1, v[2], v[3], v[4]);
      w.up[u] = pick3(cu - 1, v[0], v[1], v[2]);
      w.lo[u] = pick4(deg - 4, v[3], v[4], v[5], v[6]);
    }
  }
}

// Window step of a window-eligible node with CU neighbours above and CL
// below: loads only the columns that are new to the window (the right
// neighbour, above 2..CU, below 2..CL) and slides the window by one node.
template <class S, int OP, int U, int CU, int CL>
__device__ __forceinline__ void win_step(const Args& a, int32_t i, const int32_t* nbp,
                                         const typename Traits<S>::C2* cf, typename Traits<S>::C2 dg,
                                         const uint32_t* kc, const bool* st, WinState<S, OP, U>& w) {
  using X = typename WinT<S, OP>::X;
  constexpr int DEG = CU + CL + 2;
  const S* __restrict__ in = static_cast<const S*>(a.in);
  const uint32_t L = (uint32_t)a.L;
  uint32_t offu[CU > 1 ? CU - 1 : 1], offl[CL > 1 ? CL - 1 : 1];
#pragma unroll
  for (int t = 1; t < CU; ++t) offu[t - 1] = (uint32_t)ld_uniform(nbp + t) * L;
#pragma unroll
  for (int t = 1; t < CL; ++t) offl[t - 1] = (uint32_t)ld_uniform(nbp + CU + 2 + t) * L;
  const uint32_t offr = (uint32_t)(i + 1) * L;
  X nu[U][CU > 1 ? CU - 1 : 1], nl[U][CL > 1 ? CL - 1 : 1], nr[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    nr[u] = WinT<S, OP>::ld(in, offr + kc[u]);
#pragma unroll
    for (int t = 0; t < CU - 1; ++t) nu[u][t] = WinT<S, OP>::ld(in, offu[t] + kc[u]);
#pragma unroll
    for (int t = 0; t < CL - 1; ++t) nl[u][t] = WinT<S, OP>::ld(in, offl[t] + kc[u]);
  }
  const uint32_t self = (uint32_t)i * L;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    X v[DEG];
    v[0] = w.up[u];
#pragma unroll
    for (int t = 1; t < CU; ++t) v[t] = nu[u][t - 1];
    v[CU] = w.self[u];           // left neighbour = previous node
    v[CU + 1] = nr[u];           // right neighbour
    v[CU + 2] = w.lo[u];
#pragma unroll
    for (int t = 1; t < CL; ++t) v[CU + 2 + t] = nl[u][t - 1];
    const X x0 = w.right[u];     // this node = previous right neighbour
    win_emit<S, OP, DEG>(static_cast<S*>(a.out), self + kc[u], st[u], a.nt, x0, v, cf, dg);
    w.self[u] = x0;
    w.right[u] = nr[u];
    w.up[u] = v[CU - 1];
    w.lo[u] = v[DEG - 1];
  }
}

// One wave walks one run of consecutive nodes of a row, U level slices of 64
// at a time; the first node of a run, and any node outside the window pattern,
// takes a full step that reloads every slot.
template <class S, int OP, int U>
__device__ __forceinline__ void win_run(const Args& a, int32_t i0, int cnt, int lane) {
  using C2 = typename Traits<S>::C2;
  const uint32_t L = (uint32_t)a.L;
  for (uint32_t k0 = 0; k0 < L; k0 += 64u * U) {
    uint32_t kc[U];
    bool st[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t k = k0 + 64u * u + (uint32_t)lane;
      st[u] = k < L;
      kc[u] = k < L ? k : L - 1;
    }
    WinState<S, OP, U> w;
    bool have = false;
    for (int n = 0; n < cnt; ++n) {
      const int32_t i = i0 + n;
      const int32_t* nbp = a.nbr + (int64_t)i * 8;
      const int meta = ld_uniform(nbp + 7);
      const int deg = meta & 0xff;
      const int cu = (meta >> 8) & 0xff;
      const bool eligible = (meta >> 16) & 1;
      const C2* cfp = static_cast<const C2*>(a.coef) + (int64_t)i * 8;
      C2 cf[7];
#pragma unroll
      for (int s = 0; s < 7; ++s) cf[s] = ld_uniform(cfp + s);
      const C2 dg = ld_uniform(cfp + 7);
      const int cl = deg - cu - 2;
      if (have && eligible && cu == 2 && cl == 2) win_step<S, OP, U, 2, 2>(a, i, nbp, cf, dg, kc, st, w);
      else if (have && eligible && cu == 1 && cl == 3) win_step<S, OP, U, 1, 3>(a, i, nbp, cf, dg, kc, st, w);
      else if (have && eligible && cu == 3 && cl == 1) win_step<S, OP, U, 3, 1>(a, i, nbp, cf, dg, kc, st, w);
      else if (have && eligible && cu == 1 && cl == 2) win_step<S, OP, U, 1, 2>(a, i, nbp, cf, dg, kc, st, w);
      else if (have && eligible && cu == 2 && cl == 1) win_step<S, OP, U, 2, 1>(a, i, nbp, cf, dg, kc, st, w);
      else win_full<S, OP, U>(a, i, nbp, deg, cu, eligible, cf, dg, kc, st, w);
      have = eligible;
    }
  }
}

// Work of logical block `lb` on the run list: waves_per_block * npw runs.
template <class S, int OP, int U>
__device__ __forceinline__ void process_runs(const Args& a, int64_t lb) {
  const int wpb = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  for (int r = 0; r < a.npw; ++r) {
    const int64_t run = (lb * a.npw + r) * wpb + wave;
    if (run >= a.nruns) break;
    const int32_t i0 = ld_uniform(a.runs + 2 * run);
    const int32_t cnt = ld_uniform(a.runs + 2 * run + 1);
    win_run<S, OP, U>(a, i0, cnt, lane);
  }
}

// Work of logical block `lb`: waves_per_block * npw node groups.
template <class S, int OP, int U>
__device__ __forceinline__ void process_block(const Args& a, int64_t lb) {
  const int wpb = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int G = 64 / a.P;
  for (int r = 0; r < a.npw; ++r) {
    const int64_t gbase = ((lb * a.npw + r) * wpb + wave) * G;
    if (gbase >= a.V) break;
    run_group<S, OP, U>(a, gbase, lane);
  }
}

__device__ __forceinline__ int64_t logical_block(int64_t b, int64_t nblocks, int remap) {
  if (!remap) return b;
  const int64_t per = (nblocks + 7) / 8;
  return (b & 7) * per + (b >> 3);
}

template <class S, int OP, int U>
__global__ __launch_bounds__(256) void k_op(Args a, int64_t nblocks, int remap) {
  const int64_t lb = logical_block(blockIdx.x, nblocks, remap);
  if (lb >= nblocks) return;
  process_block<S, OP, U>(a, lb);
}

template <class S, int OP, int U>
__global__ __launch_bounds__(256) void k_win(Args a, int64_t nblocks, int remap) {
  const int64_t lb = logical_block(blockIdx.x, nblocks, remap);
  if (lb >= nblocks) return;
  process_runs<S, OP, U>(a, lb);
}

// ---- LDS tiles -------------------------------------------------------------------
//
// A workgroup takes one tile: a set of nodes (a few latitude rows by one
// longitude sector) and the sorted set of every column their stencils read,
// stored as segments of consecutive nodes.  Columns of consecutive nodes are
// contiguous in memory, so each segment is one contiguous block, which a wave
// copies with direct global->LDS loads (16 bytes per lane, no registers
// involved); the tile's node records (coefficients, LDS positions of the
// stencil entries, node index), packed in tile order when the tiling is set
// up, arrive in one more contiguous copy.  One wait and one barrier end the
// copy.  Each wave then takes nodes of the tile in turn, 64 lanes = 64
// levels, and reads its stencil and record from LDS; only the output goes
// back to memory.  No global load sits on a node's critical path, every wave
// keeps many independent loads in flight during the copy, and the
// workgroups sharing a CU overlap each other's copy and compute phases.
// Tiles stacked in latitude follow each other, so the halo columns they share
// are L2 hits.

}  // namespace

struct TileArgs {
  const int32_t* info;   // [ntiles][4]: first segment, first record, columns | blocks << 16, nodes | segments << 16
  const int32_t* segs;   // [nseg (+ 8 padding)][2]: first node, count
  const char* rec;       // [V] node records in tile order (see tile_record_bytes)
  const void* in;
  void* out;
  void* out2;            // OP_GRADLAP: the gradient ([V][L][2]); out gets the Laplacian; OP_DIVTA: the addend (read)
  int64_t ntiles;
  int32_t L;             // levels
  int32_t KL;            // levels per chunk (L: whole columns)
  int32_t nchunks;
  int32_t nt;
};

namespace {

// win_store of a tile's value; OP_DIVTA: plus the addend at the same place,
// after the rounding to the field's type that storing it would make.
// Bound by memory like the divergence adjoint itself: the addend is read once
// where the sum as a pass of its own reads two fields and writes one (backward
// of the one-pass gradient and Laplacian with its forward, O320 x 60 FP32: 379
// -> 312 us).
template <class S, int OP>
__device__ __forceinline__ void tile_store(const TileArgs& a, S* __restrict__ out, uint32_t o, typename Traits<S>::C r0,
                                           typename Traits<S>::C r1) {
  if constexpr (OP == OP_DIVTA) {
    const S* add = static_cast<const S*>(a.out2) + ((out + 2 * (size_t)o) - static_cast<S*>(a.out));
    const typename Traits<S>::C2 b = ld2(add);
    if constexpr (sizeof(S) == 2) {
      r0 = bf16_to_f32(f32_to_bf16(r0));
      r1 = bf16_to_f32(f32_to_bf16(r1));
    }
    r0 += b.x;
    r1 += b.y;
  }
  win_store<S, OP>(out, o, a.nt, r0, r1);
}

// Node record of the tile path: coefficient row (8 pairs, ring 1, followed
// for OP_DIVCURL by the 8 pairs of the second operator, the curl's or, for
// OP_DIVGRADT, the gradient adjoint's; 24 weights, ring 2, followed for
// OP_GRADLAP by the gradient's 8 pairs), LDS
// position row (8 or 24 uint16), node index (int32), zero padding to 16
// bytes.
template <class S, int OP>
struct TileRec {
  using C = typename Traits<S>::C;
  using C2 = typename Traits<S>::C2;
  static constexpr bool kRing2 = OP == OP_LAP || OP == OP_GRADLAP;
  static constexpr bool kGrad = OP == OP_GRADLAP;   // gradient pairs after the weights
  static constexpr bool kDual = OP == OP_DIVCURL;    // second pairs after the divergence pairs
  static constexpr int kEntries = kRing2 ? kLapStride : 8;
  static constexpr uint32_t kLapB = kEntries * sizeof(C);   // ring 2: the 24 weights
  static constexpr uint32_t kCoefB = kRing2 ? kLapB + (kGrad ? 8 * sizeof(C2) : 0)
                                            : 8 * sizeof(C2) * (kDual ? 2 : 1);
  static constexpr uint32_t kLocB = 2 * kEntries;
  static constexpr uint32_t kIdOff = kCoefB + kLocB;
  static constexpr uint32_t kBytes = (kIdOff + 4 + 15) & ~15u;
  static constexpr int kCin = (OP == OP_DIV || OP == OP_GRADT || OP == OP_DIVCURL) ? 2 : 1;
};

constexpr int kLocCountShift = 11;

typedef __attribute__((address_space(3))) void* lds_vptr;

// s_waitcnt immediate with lgkmcnt = 0 and vmcnt, expcnt left at their
// maxima (vmcnt bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8).  Issued
// through the builtin rather than inline assembly so that the compiler's own
// wait insertion accounts for it.
constexpr int kWaitLgkm0 = 0xC07F;

constexpr uint64_t kLdsPerCu = 160 * 1024;   // gfx950 LDS per CU
constexpr int64_t kBf16ColExtra = 12;        // BF16 tiles: LDS bytes per column beyond the data

// Direct loads of nbytes (a multiple of 4) from global src to LDS byte offset
// dst: 16 bytes per lane (lane l of instruction q moves bytes 16 (64 q + l)
// onwards; gfx950 accepts any 4-byte alignment on both sides), then the last
// 0..3 dwords one per lane.  Instruction q goes to wave (ctr + q) mod W (W a
// power of two), ctr counting the instructions of the workgroup's earlier
// copies, so that small copies spread over the waves.
__device__ __forceinline__ void dma_copy(const char* src, char* lds, uint32_t dst, uint32_t nbytes, int wave, int W,
                                         int lane, uint32_t& ctr) {
  const uint32_t n16 = nbytes >> 4;
  const uint32_t ninst = (n16 + 63) >> 6;
  const uint32_t wm = (uint32_t)W - 1;   // W is a power of two
  for (uint32_t q = ((uint32_t)wave - ctr) & wm; q < ninst; q += (uint32_t)W) {
    const uint32_t d = q * 64 + (uint32_t)lane;
    if (d < n16)
      __builtin_amdgcn_global_load_lds(src + 16 * (size_t)d, (lds_vptr)(lds + dst + 1024 * q), 16, 0, 0);
  }
  ctr += ninst;
  const uint32_t rem = (nbytes & 15u) >> 2;
  if (rem) {
    if ((uint32_t)wave == (ctr & wm) && (uint32_t)lane < rem)
      __builtin_amdgcn_global_load_lds(src + 16 * (size_t)n16 + 4 * lane, (lds_vptr)(lds + dst + 16 * n16), 4, 0, 0);
    ++ctr;
  }
}

// Direct loads of cnt column chunks of nb bytes each (nb a multiple of 4),
// chunk c at global src + c * gstride, packed back to back at LDS byte offset
// dst.  The LDS image is contiguous, so each instruction still fills 64
// consecutive units (16 bytes when nb allows, else 4); a lane finds its
// chunk by dividing its unit index by the units per chunk.
__device__ __forceinline__ void dma_copy_strided(const char* src, size_t gstride, uint32_t cnt, uint32_t nb,
                                                 char* lds, uint32_t dst, int wave, int W, int lane,
                                                 uint32_t& ctr) {
  const bool wide = (nb & 15u) == 0;
  const uint32_t ub = wide ? 16u : 4u;
  const uint32_t upc = nb / ub;                       // units per chunk
  const uint32_t total = cnt * upc;
  const uint32_t ninst = (total + 63) >> 6;
  const uint32_t wm = (uint32_t)W - 1;   // W is a power of two
  for (uint32_t q = ((uint32_t)wave - ctr) & wm; q < ninst; q += (uint32_t)W) {
    const uint32_t u = q * 64 + (uint32_t)lane;
    if (u < total) {
      const uint32_t c = u / upc, o = u - c * upc;
      const char* g = src + (size_t)c * gstride + (size_t)o * ub;
      if (wide) __builtin_amdgcn_global_load_lds(g, (lds_vptr)(lds + dst + 1024 * q), 16, 0, 0);
      else __builtin_amdgcn_global_load_lds(g, (lds_vptr)(lds + dst + 256 * q), 4, 0, 0);
    }
  }
  ctr += ninst;
}

// Calls f(first, count) for pairs [b, e) of a (first, count) table, in order.
// Pairs come eight at a time from independent scalar loads (one wait per
// eight); the tables carry eight pairs of padding so the loads stay in
// bounds.  Scalar loads leave the vector memory counter alone, so fetching
// the next pairs never waits for direct loads already in flight.
template <class F>
__device__ __forceinline__ void for_pairs(const int32_t* tab, int32_t b, int32_t e, F&& f) {
  for (int32_t base = b; base < e; base += 8) {
    int32_t v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = ld_uniform(tab + 2 * (size_t)base + j);
    const int32_t n = e - base;
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (q < n) f(v[2 * q], v[2 * q + 1]);
  }
}

template <class T>
__device__ __forceinline__ T lds_ld(const char* lds, uint32_t off) {
  return *reinterpret_cast<const T*>(lds + off);
}

__device__ __forceinline__ uint32_t uni(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

// One stencil value from an LDS tile, in the arithmetic type X (BF16 columns
// widen to FP32).
template <class S, class X>
__device__ __forceinline__ X lds_elem(const char* lds, uint32_t off) {
  if constexpr (sizeof(S) != 2) {
    return lds_ld<X>(lds, off);
  } else if constexpr (sizeof(X) == 4) {
    return bf16_to_f32(lds_ld<uint16_t>(lds, off));
  } else {
    const uint32_t w = lds_ld<uint32_t>(lds, off);
    return make_float2(bf16_to_f32(w & 0xffffu), bf16_to_f32(w >> 16));
  }
}

// LDS positions of a node's entries (wave-uniform): pos[s] for the stencil
// slots, own position and entry count from the last record entry.
template <int NREC>
__device__ __forceinline__ void tile_positions(const char* lds, uint32_t off, uint32_t* pos, uint32_t& self,
                                               int& cnt) {
  uint32_t w[NREC / 2];
#pragma unroll
  for (int q = 0; q < NREC / 8; ++q) {
    const uint4 r = lds_ld<uint4>(lds, off + 16 * q);
    w[4 * q] = uni(r.x);
    w[4 * q + 1] = uni(r.y);
    w[4 * q + 2] = uni(r.z);
    w[4 * q + 3] = uni(r.w);
  }
#pragma unroll
  for (int s = 0; s < NREC - 1; ++s) pos[s] = (s & 1) ? (w[s >> 1] >> 16) : (w[s >> 1] & 0xffffu);
  const uint32_t last = w[NREC / 2 - 1] >> 16;
  self = last & ((1u << kLocCountShift) - 1);
  cnt = (int)(last >> kLocCountShift);
}

// Marks a value as computed here: the compiler may not sink its computation
// (and the LDS reads feeding it) into the predicated store that follows, so
// the reads of all slices of a step issue together.
template <class T>
__device__ __forceinline__ void keep(T& v) {
  asm volatile("" : "+v"(v));
}

// One node of a 1-ring operator: DEG slots, U slices of 64 levels per step.
// Each lane's LDS address of a slot is formed once per node; the level slices
// of a step then sit at constant offsets from it.  Lanes past the chunk's
// last level read (and drop) values beyond their column, which stay inside
// the tail behind the tile buffer (tile_tail_bytes).
template <class S, int OP, int U, int DEG>
__device__ __forceinline__ void tile_node1(const TileArgs& a, const char* lds, const uint32_t* so, uint32_t xo,
                                           const typename Traits<S>::C2* cf, typename Traits<S>::C2 dg,
                                           uint32_t obase, int klc, int lane) {
  using X = typename WinT<S, OP>::X;
  using C = typename Traits<S>::C;
  using R = TileRec<S, OP>;
  constexpr uint32_t kEl = (uint32_t)sizeof(S) * R::kCin;   // bytes per level in LDS
  constexpr uint32_t kOut = kTwoOut<OP> ? 2 : 1;
  // BF16: values are left to the compiler's placement, which keeps the
  // vector-input kernels within 64 VGPRs (four workgroups per CU)
  constexpr bool kKeep = sizeof(S) != 2;
  const uint32_t lo = (uint32_t)lane * kEl;
  uint32_t vb[DEG];
#pragma unroll
  for (int s = 0; s < DEG; ++s) vb[s] = so[s] + lo;
  const uint32_t vx = xo + lo;
  S* __restrict__ out = static_cast<S*>(a.out) + (size_t)kOut * (obase + (uint32_t)lane);
  auto step = [&](int kb) {
    const uint32_t ko = (uint32_t)kb * kEl;
    X v[U][DEG], x0[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int s = 0; s < DEG; ++s) v[u][s] = lds_elem<S, X>(lds, vb[s] + ko + 64u * kEl * u);
      x0[u] = lds_elem<S, X>(lds, vx + ko + 64u * kEl * u);
    }
    C r0[U], r1[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      win_combine<S, OP, DEG>(x0[u], v[u], cf, dg, r0[u], r1[u]);
      if constexpr (kKeep) {
        keep(r0[u]);
        if constexpr (kOut == 2) keep(r1[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (kb + 64 * u + lane < klc) tile_store<S, OP>(a, out + (size_t)kOut * kb, 64u * u, r0[u], r1[u]);
  };
  step(0);
  for (int kb = 64 * U; kb < klc; kb += 64 * U) step(kb);
}

// One node of the two-ring Laplacian: NS entries (padded with the node itself
// and zero weights, which add exact zeros), sum_m W_im (f_m - f_i).  Addresses
// as in tile_node1.
template <class S, int U, int NS>
__device__ __forceinline__ void tile_node2(const TileArgs& a, const char* lds, const uint32_t* so, uint32_t xo,
                                           const typename Traits<S>::C* w, uint32_t obase, int klc, int lane) {
  using C = typename Traits<S>::C;
  constexpr uint32_t kEl = (uint32_t)sizeof(S);
  const uint32_t lo = (uint32_t)lane * kEl;
  uint32_t vb[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) vb[s] = so[s] + lo;
  const uint32_t vx = xo + lo;
  S* __restrict__ out = static_cast<S*>(a.out) + (size_t)(obase + (uint32_t)lane);
  auto step = [&](int kb) {
    const uint32_t ko = (uint32_t)kb * kEl;
    C v[U][NS], x0[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int s = 0; s < NS; ++s) v[u][s] = lds_elem<S, C>(lds, vb[s] + ko + 64u * kEl * u);
      x0[u] = lds_elem<S, C>(lds, vx + ko + 64u * kEl * u);
    }
    C acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc[u] = 0;
#pragma unroll
      for (int s = 0; s < NS; ++s) acc[u] = fma(w[s], v[u][s] - x0[u], acc[u]);
      keep(acc[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (kb + 64 * u + lane < klc) {
        S* o = out + (size_t)(kb + 64 * u);
        if (a.nt) st1<true>(o, acc[u]);
        else st1<false>(o, acc[u]);
      }
    }
  };
  step(0);
  for (int kb = 64 * U; kb < klc; kb += 64 * U) step(kb);
}

// Difference of entry s as the gradient takes it (every node has three
// neighbours; pairs of zeros past its degree).
template <class C, class C2>
__device__ __forceinline__ C grad_diff(int s, C2 pair, C d) {
  return s >= 3 && pair.x == 0 && pair.y == 0 ? C(0) : d;
}

// One node of the fused gradient and two-ring Laplacian (OP_GRADLAP): the
// differences f_m - f_i of the NS entries feed both sums; the first 7 entries
// are the node's 1-ring neighbours in slot order (the two-ring tables are
// ordered so), weighted by the gradient pairs (zero past the node's degree,
// where the entry is of the second ring and its difference is taken as zero:
// it need not be finite).  Same slot-order arithmetic as tile_node2 and the
// gradient's tile_node1.
template <class S, int U, int NS>
__device__ __forceinline__ void tile_node2g(const TileArgs& a, const char* lds, const uint32_t* so, uint32_t xo,
                                            const typename Traits<S>::C* w, const typename Traits<S>::C2* cf,
                                            uint32_t obase, int klc, int lane) {
  using C = typename Traits<S>::C;
  constexpr uint32_t kEl = (uint32_t)sizeof(S);
  const uint32_t lo = (uint32_t)lane * kEl;
  uint32_t vb[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) vb[s] = so[s] + lo;
  const uint32_t vx = xo + lo;
  S* __restrict__ out = static_cast<S*>(a.out) + (size_t)(obase + (uint32_t)lane);
  S* __restrict__ og = static_cast<S*>(a.out2) + 2 * (size_t)(obase + (uint32_t)lane);
  auto step = [&](int kb) {
    const uint32_t ko = (uint32_t)kb * kEl;
    C v[U][NS], x0[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int s = 0; s < NS; ++s) v[u][s] = lds_elem<S, C>(lds, vb[s] + ko + 64u * kEl * u);
      x0[u] = lds_elem<S, C>(lds, vx + ko + 64u * kEl * u);
    }
    C acc[U], ax[U], ay[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc[u] = 0;
      ax[u] = 0;
      ay[u] = 0;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const C d = v[u][s] - x0[u];
        acc[u] = fma(w[s], d, acc[u]);
        if (s < 7) {
          const C e = grad_diff<C>(s, cf[s], d);
          ax[u] = fma(cf[s].x, e, ax[u]);
          ay[u] = fma(cf[s].y, e, ay[u]);
        }
      }
      keep(acc[u]);
      keep(ax[u]);
      keep(ay[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (kb + 64 * u + lane < klc) {
        const size_t k = (size_t)(kb + 64 * u);
        if (a.nt) {
          st1<true>(out + k, acc[u]);
          st2<true>(og + 2 * k, ax[u], ay[u]);
        } else {
          st1<false>(out + k, acc[u]);
          st2<false>(og + 2 * k, ax[u], ay[u]);
        }
      }
    }
  };
  step(0);
  for (int kb = 64 * U; kb < klc; kb += 64 * U) step(kb);
}

// One node of the divergence and a second operator of one vector field
// (OP_DIVCURL: the curl, or the gradient adjoint on OP_DIVGRADT's records):
// the same loads feed the divergence-form sums with the divergence pairs
// (out) and with the second pairs (out2), each exactly as tile_node1
// computes it for that operator.
template <class S, int U, int DEG>
__device__ __forceinline__ void tile_node1d(const TileArgs& a, const char* lds, const uint32_t* so, uint32_t xo,
                                            const typename Traits<S>::C2* cf, typename Traits<S>::C2 dg,
                                            const typename Traits<S>::C2* cf2, typename Traits<S>::C2 dg2,
                                            uint32_t obase, int klc, int lane) {
  using X = typename WinT<S, OP_DIVCURL>::X;
  using C = typename Traits<S>::C;
  constexpr uint32_t kEl = (uint32_t)sizeof(S) * 2;
  const uint32_t lo = (uint32_t)lane * kEl;
  uint32_t vb[DEG];
#pragma unroll
  for (int s = 0; s < DEG; ++s) vb[s] = so[s] + lo;
  const uint32_t vx = xo + lo;
  S* __restrict__ out = static_cast<S*>(a.out) + (size_t)(obase + (uint32_t)lane);
  S* __restrict__ oz = static_cast<S*>(a.out2) + (size_t)(obase + (uint32_t)lane);
  auto step = [&](int kb) {
    const uint32_t ko = (uint32_t)kb * kEl;
    X v[U][DEG], x0[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int s = 0; s < DEG; ++s) v[u][s] = lds_elem<S, X>(lds, vb[s] + ko + 64u * kEl * u);
      x0[u] = lds_elem<S, X>(lds, vx + ko + 64u * kEl * u);
    }
    C r0[U], z0[U], unused;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      win_combine<S, OP_DIVCURL, DEG>(x0[u], v[u], cf, dg, r0[u], unused);
      win_combine<S, OP_DIVCURL, DEG>(x0[u], v[u], cf2, dg2, z0[u], unused);
      keep(r0[u]);
      keep(z0[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (kb + 64 * u + lane < klc) {
        win_store<S, OP_DIVCURL>(out + kb, 64u * u, a.nt, r0[u], 0);
        win_store<S, OP_DIVCURL>(oz + kb, 64u * u, a.nt, z0[u], 0);
      }
  };
  step(0);
  for (int kb = 64 * U; kb < klc; kb += 64 * U) step(kb);
}

// Copy of one tile (chunk) into an LDS buffer by W waves: the records as one
// copy spread over the waves, then each column segment by one wave (segment
// i by wave i mod W), so each wave sets up only its own copies.
template <class S, int OP>
__device__ __forceinline__ void tile_copy(const TileArgs& a, int64_t tile, int k0, int klc, char* buf, int wave,
                                          int W, int lane) {
  using R = TileRec<S, OP>;
  const int32_t* inf = a.info + 4 * tile;
  const int32_t seg0 = ld_uniform(inf), rec0 = ld_uniform(inf + 1), ncols = ld_uniform(inf + 2) & 0xffff,
                nodes_segs = ld_uniform(inf + 3);
  const int32_t nnodes = nodes_segs & 0xffff;
  const int32_t seg1 = seg0 + (int32_t)((uint32_t)nodes_segs >> 16);
  const uint32_t colB = (uint32_t)klc * R::kCin * (uint32_t)sizeof(S);   // LDS column stride (this chunk)
  uint32_t ctr = 0;
  dma_copy(a.rec + (size_t)rec0 * R::kBytes, buf, 0, (uint32_t)nnodes * R::kBytes, wave, W, lane, ctr);
  const size_t gcol = (size_t)a.L * R::kCin * sizeof(S);                 // global column bytes
  const char* in = static_cast<const char*>(a.in);
  uint32_t p = 0, i = 0;
  if constexpr (sizeof(S) == 2) {
    // BF16 columns may start 2 bytes into a dword: each segment is copied as
    // the dword-aligned span around it, placed so that LDS and memory agree
    // mod 4, and its columns' LDS offsets go to a table after the records.
    const uint32_t tab = (uint32_t)nnodes * R::kBytes;
    uint32_t cur = tab + (((uint32_t)ncols * 4u + 15u) & ~15u);
    for_pairs(a.segs, seg0, seg1, [&](int32_t first, int32_t cnt) {
      const size_t g0 = (size_t)first * gcol;
      const uint32_t mis = (uint32_t)(g0 & 3u);
      const uint32_t nb = (uint32_t)((((g0 + (size_t)cnt * colB) + 3u) & ~(size_t)3u) - (g0 - mis));
      if ((i & (uint32_t)(W - 1)) == (uint32_t)wave) {
        uint32_t own = 0;
        dma_copy(in + (g0 - mis), buf, cur, nb, 0, 1, lane, own);
        for (int32_t c = lane; c < cnt; c += 64)
          *reinterpret_cast<uint32_t*>(buf + tab + 4 * (p + (uint32_t)c)) = cur + mis + (uint32_t)c * colB;
      }
      cur += nb;
      p += (uint32_t)cnt;
      ++i;
    });
  } else {
    const uint32_t data_off = (uint32_t)nnodes * R::kBytes;
    for_pairs(a.segs, seg0, seg1, [&](int32_t first, int32_t cnt) {
      if ((i & (uint32_t)(W - 1)) == (uint32_t)wave) {
        uint32_t own = 0;
        if (a.KL == a.L)
          dma_copy(in + (size_t)first * gcol, buf, data_off + p * colB, (uint32_t)cnt * colB, 0, 1, lane, own);
        else
          dma_copy_strided(in + (size_t)first * gcol + (size_t)k0 * R::kCin * sizeof(S), gcol, (uint32_t)cnt, colB,
                           buf, data_off + p * colB, 0, 1, lane, own);
      }
      p += (uint32_t)cnt;
      ++i;
    });
  }
}

// LDS offsets of a node's stencil columns from their tile positions: a
// fixed stride for FP32/FP64, the offset table for BF16.
template <class S, int N>
__device__ __forceinline__ void tile_offsets(const char* lds, uint32_t tab, uint32_t data_off, uint32_t colB,
                                             const uint32_t* pos, uint32_t self, uint32_t* so, uint32_t& xo) {
  if constexpr (sizeof(S) == 2) {
#pragma unroll
    for (int q = 0; q < N; ++q) so[q] = uni(lds_ld<uint32_t>(lds, tab + 4 * pos[q]));
    xo = uni(lds_ld<uint32_t>(lds, tab + 4 * self));
  } else {
#pragma unroll
    for (int q = 0; q < N; ++q) so[q] = data_off + pos[q] * colB;
    xo = data_off + self * colB;
  }
}

// One node of a tile (record tn) by one wave, 64 lanes over the levels of
// the chunk: positions and coefficients from the record, then the stencil.
template <class S, int OP, int U>
__device__ __forceinline__ void tile_eval(const TileArgs& a, const char* lds, int32_t tn, uint32_t data_off,
                                          uint32_t colB, int k0, int klc, int lane) {
  using R = TileRec<S, OP>;
  using C = typename Traits<S>::C;
  using C2 = typename Traits<S>::C2;
  const uint32_t ro = (uint32_t)tn * R::kBytes;
  const uint32_t obase = uni((uint32_t)lds_ld<int32_t>(lds, ro + R::kIdOff)) * (uint32_t)a.L + (uint32_t)k0;
  uint32_t pos[R::kEntries - 1], self;
  int ne;
  tile_positions<R::kEntries>(lds, ro + R::kCoefB, pos, self, ne);
  uint32_t so[R::kEntries - 1], xo;
  if constexpr (R::kRing2) {
    C w[R::kEntries - 1];
#pragma unroll
    for (int q = 0; q < R::kEntries - 1; ++q) w[q] = lds_ld<C>(lds, ro + q * (uint32_t)sizeof(C));
    if constexpr (R::kGrad) {
      C2 cf[7];
#pragma unroll
      for (int q = 0; q < 7; ++q) cf[q] = lds_ld<C2>(lds, ro + R::kLapB + q * (uint32_t)sizeof(C2));
      if (ne <= 18) {
        tile_offsets<S, 18>(lds, data_off, data_off, colB, pos, self, so, xo);
        tile_node2g<S, U, 18>(a, lds, so, xo, w, cf, obase, klc, lane);
      } else {
        tile_offsets<S, R::kEntries - 1>(lds, data_off, data_off, colB, pos, self, so, xo);
        tile_node2g<S, 1, R::kEntries - 1>(a, lds, so, xo, w, cf, obase, klc, lane);
      }
    } else if (ne <= 18) {
      tile_offsets<S, 18>(lds, data_off, data_off, colB, pos, self, so, xo);
      tile_node2<S, U, 18>(a, lds, so, xo, w, obase, klc, lane);
    } else {
      tile_offsets<S, R::kEntries - 1>(lds, data_off, data_off, colB, pos, self, so, xo);
      tile_node2<S, 1, R::kEntries - 1>(a, lds, so, xo, w, obase, klc, lane);
    }
  } else {
    C2 cf[7];
#pragma unroll
    for (int q = 0; q < 7; ++q) cf[q] = lds_ld<C2>(lds, ro + q * (uint32_t)sizeof(C2));
    const C2 dg = lds_ld<C2>(lds, ro + 7 * (uint32_t)sizeof(C2));
    tile_offsets<S, 7>(lds, data_off, data_off, colB, pos, self, so, xo);
    if constexpr (R::kDual) {
      C2 cf2[7];
#pragma unroll
      for (int q = 0; q < 7; ++q) cf2[q] = lds_ld<C2>(lds, ro + (8 + q) * (uint32_t)sizeof(C2));
      const C2 dg2 = lds_ld<C2>(lds, ro + 15 * (uint32_t)sizeof(C2));
      switch (ne) {
        case 6: tile_node1d<S, U, 6>(a, lds, so, xo, cf, dg, cf2, dg2, obase, klc, lane); break;
        case 5: tile_node1d<S, 1, 5>(a, lds, so, xo, cf, dg, cf2, dg2, obase, klc, lane); break;
        case 7: tile_node1d<S, 1, 7>(a, lds, so, xo, cf, dg, cf2, dg2, obase, klc, lane); break;
        case 4: tile_node1d<S, 1, 4>(a, lds, so, xo, cf, dg, cf2, dg2, obase, klc, lane); break;
        default: tile_node1d<S, 1, 3>(a, lds, so, xo, cf, dg, cf2, dg2, obase, klc, lane); break;
      }
      return;
    }
    switch (ne) {
      case 6: tile_node1<S, OP, U, 6>(a, lds, so, xo, cf, dg, obase, klc, lane); break;
      case 5: tile_node1<S, OP, 1, 5>(a, lds, so, xo, cf, dg, obase, klc, lane); break;
      case 7: tile_node1<S, OP, 1, 7>(a, lds, so, xo, cf, dg, obase, klc, lane); break;
      case 4: tile_node1<S, OP, 1, 4>(a, lds, so, xo, cf, dg, obase, klc, lane); break;
      default: tile_node1<S, OP, 1, 3>(a, lds, so, xo, cf, dg, obase, klc, lane); break;
    }
  }
}

// Nodes of a block (0: no blocks) and slices in registers at a time (see
// tile_block), for UT slices per step.  The FP32 divergence pairs run without
// blocks and the BF16 ones only on columns of one slice: with 16 waves a
// workgroup, two of them fit a CU within 64 registers a lane only, where a
// block's columns leave no room for both coefficient rows.
template <class S, int OP>
constexpr int kBlkN = OP == OP_DIVCURL               ? (sizeof(S) == 4 ? 0 : 2)
                      : sizeof(S) == 8 && OP == OP_GRADLAP ? 2
                      : sizeof(S) == 4 && OP == OP_LAP ? 4
                      : sizeof(S) == 2 && TileRec<S, OP>::kCin == 2 ? 2 : 3;
template <class S, int OP>
constexpr int kBlkU = (sizeof(S) == 8 && TileRec<S, OP>::kRing2) || (sizeof(S) == 2 && OP == OP_DIVCURL) ? 1 : 2;
template <class S, int OP, int UT>
constexpr bool kUseBlk = kBlkN<S, OP> > 0 && !(sizeof(S) == 2 && OP == OP_DIVCURL && UT > 1);

// A block: NB consecutive nodes of a row whose stencils have the regular
// shape (two consecutive neighbours above, left, right, two consecutive
// below, and the two-ring around them), each column one further from a node
// to the next; records r0 .. r0 + NB - 1.  One wave evaluates the block from
// the columns its nodes read together, each read from LDS once: 3 NB + 4
// instead of 7 NB (1-ring), 5 NB + 14 instead of 19 NB (two-ring), with one
// address a column and BF16 widened once.  The columns of a row lie next to
// each other in LDS, so five row positions (three for the 1-ring), from the
// first node's record, give all addresses.  What bounds the kernels this
// serves is the evaluation inside the tile (address arithmetic, LDS reads,
// BF16 widening), and for ragged columns the cache lines a column's last
// levels share with their neighbours: a block writes its remainder levels
// right after the whole slices, before those lines leave L2.  O640, one node
// a wave -> blocks: BF16 Laplacian 588 -> 448 us (137 levels), 587 -> 371
// (91), 415 -> 236 (60); BF16 gradient 371 -> 330, 332 -> 243, 221 -> 164;
// FP32 Laplacian 635 -> 580, 501 -> 428, 328 -> 275; FP32 gradient and
// Laplacian 938 -> 915, 757 -> 661, 458 -> 419; FP64 Laplacian 1422 -> 1303.
template <class S, int OP, int UT, int NB>
__device__ __forceinline__ void tile_block(const TileArgs& a, const char* lds, int32_t r0, uint32_t data_off,
                                           uint32_t colB, int k0, int klc, int rem, int tj, int tt, int lane) {
  using R = TileRec<S, OP>;
  using C = typename Traits<S>::C;
  using C2 = typename Traits<S>::C2;
  using X = typename WinT<S, R::kRing2 ? (int)OP_GRAD : OP>::X;
  constexpr int U = UT < kBlkU<S, OP> ? UT : kBlkU<S, OP>;
  constexpr uint32_t kEl = (uint32_t)sizeof(S) * R::kCin;
  constexpr uint32_t kOut = kTwoOut<OP> ? 2 : 1;
  constexpr int ring = R::kRing2 ? 2 : 1;
  const uint32_t ro = (uint32_t)r0 * R::kBytes;
  const uint32_t obase = uni((uint32_t)lds_ld<int32_t>(lds, ro + R::kIdOff)) * (uint32_t)a.L + (uint32_t)k0;
  auto pos = [&](int s) -> uint32_t { return uni(lds_ld<uint16_t>(lds, ro + R::kCoefB + 2 * s)); };
  auto at = [&](uint32_t p) -> uint32_t {
    if constexpr (sizeof(S) == 2) return uni(lds_ld<uint32_t>(lds, data_off + 4 * p));
    else return data_off + p * colB;
  };
  const uint32_t lo = (uint32_t)lane * kEl;
  // LDS address of the lane's first level in column 0 of each row: the
  // nodes' own at ring, rows above before it and below after it
  uint32_t row[2 * ring + 1];
  row[ring] = at(pos(R::kEntries - 1) & ((1u << kLocCountShift) - 1));
  row[ring - 1] = at(pos(0));
  row[ring + 1] = at(pos(4));
  if constexpr (R::kRing2) {
    row[0] = at(pos(6));
    row[4] = at(pos(15));
  }
  S* __restrict__ out = static_cast<S*>(a.out) + (size_t)kOut * (obase + (uint32_t)lane);
  S* __restrict__ out2 = static_cast<S*>(a.out2) + (size_t)(OP == OP_GRADLAP ? 2 : 1) * (obase + (uint32_t)lane);
  for (int kb = 0; kb < klc; kb += 64 * U) {
    const uint32_t ko = (uint32_t)kb * kEl + lo;
    // column x of a row (relative to its column 0)
    auto get = [&](int r, int x, X* v) {
      const uint32_t o = row[r] + (uint32_t)x * colB + ko;
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = lds_elem<S, X>(lds, o + 64u * kEl * u);
    };
    auto store = [&](int b, const C* r, const C* q, const C* z) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (kb + 64 * u + lane < klc) {
          const uint32_t o = (uint32_t)(b * a.L + kb + 64 * u);
          if constexpr (OP == OP_GRADLAP) {
            if (a.nt) {
              st1<true>(out + o, r[u]);
              st2<true>(out2 + 2 * (size_t)o, q[u], z[u]);
            } else {
              st1<false>(out + o, r[u]);
              st2<false>(out2 + 2 * (size_t)o, q[u], z[u]);
            }
          } else if constexpr (OP == OP_LAP) {
            if (a.nt) st1<true>(out + o, r[u]);
            else st1<false>(out + o, r[u]);
          } else {
            tile_store<S, OP>(a, out, o, r[u], q[u]);
            if constexpr (R::kDual) win_store<S, OP>(out2, o, a.nt, z[u], 0);
          }
        }
    };
    if constexpr (!R::kRing2) {
      X up[NB + 1][U], mi[NB + 2][U], dn[NB + 1][U];
#pragma unroll
      for (int x = 0; x < NB + 1; ++x) get(0, x, up[x]);
#pragma unroll
      for (int x = 0; x < NB + 2; ++x) get(1, x - 1, mi[x]);
#pragma unroll
      for (int x = 0; x < NB + 1; ++x) get(2, x, dn[x]);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const uint32_t rc = ro + (uint32_t)b * R::kBytes;
        C2 cf[6], dg = {0, 0}, cg[6], dg2;
#pragma unroll
        for (int q = 0; q < 6; ++q) cf[q] = lds_ld<C2>(lds, rc + q * (uint32_t)sizeof(C2));
        if constexpr (OP != OP_GRAD) dg = lds_ld<C2>(lds, rc + 7 * (uint32_t)sizeof(C2));
        if constexpr (R::kDual) {
#pragma unroll
          for (int q = 0; q < 6; ++q) cg[q] = lds_ld<C2>(lds, rc + (8 + q) * (uint32_t)sizeof(C2));
          dg2 = lds_ld<C2>(lds, rc + 15 * (uint32_t)sizeof(C2));
        }
        C r0v[U], r1v[U], z0[U], unused;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const X v[6] = {up[b][u], up[b + 1][u], mi[b][u], mi[b + 2][u], dn[b][u], dn[b + 1][u]};
          win_combine<S, OP, 6>(mi[b + 1][u], v, cf, dg, r0v[u], r1v[u]);
          keep(r0v[u]);
          if constexpr (kOut == 2) keep(r1v[u]);
          if constexpr (R::kDual) {
            win_combine<S, OP, 6>(mi[b + 1][u], v, cg, dg2, z0[u], unused);
            keep(z0[u]);
          }
        }
        store(b, r0v, r1v, z0);
      }
    } else {
      C tt[NB + 2][U], up[NB + 3][U], mi[NB + 4][U], dn[NB + 3][U], bb[NB + 2][U];
#pragma unroll
      for (int x = 0; x < NB + 2; ++x) get(0, x, tt[x]);
#pragma unroll
      for (int x = 0; x < NB + 3; ++x) get(1, x - 1, up[x]);
#pragma unroll
      for (int x = 0; x < NB + 4; ++x) get(2, x - 2, mi[x]);
#pragma unroll
      for (int x = 0; x < NB + 3; ++x) get(3, x - 1, dn[x]);
#pragma unroll
      for (int x = 0; x < NB + 2; ++x) get(4, x, bb[x]);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const uint32_t rc = ro + (uint32_t)b * R::kBytes;
        C w[18];
        C2 cf[6];
#pragma unroll
        for (int q = 0; q < 18; ++q) w[q] = lds_ld<C>(lds, rc + q * (uint32_t)sizeof(C));
        if constexpr (R::kGrad) {
#pragma unroll
          for (int q = 0; q < 6; ++q) cf[q] = lds_ld<C2>(lds, rc + R::kLapB + q * (uint32_t)sizeof(C2));
        }
        C ac[U], ax[U], ay[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const C v[18] = {up[b + 1][u], up[b + 2][u], mi[b + 1][u], mi[b + 3][u], dn[b + 1][u], dn[b + 2][u],
                           tt[b][u], tt[b + 1][u], tt[b + 2][u], up[b][u], up[b + 3][u], mi[b][u], mi[b + 4][u],
                           dn[b][u], dn[b + 3][u], bb[b][u], bb[b + 1][u], bb[b + 2][u]};
          const C x0 = mi[b + 2][u];
          ac[u] = ax[u] = ay[u] = 0;
#pragma unroll
          for (int q = 0; q < 18; ++q) {
            const C d = v[q] - x0;
            ac[u] = fma(w[q], d, ac[u]);
            if constexpr (R::kGrad) {
              if (q < 6) {
                ax[u] = fma(cf[q].x, d, ax[u]);
                ay[u] = fma(cf[q].y, d, ay[u]);
              }
            }
          }
          keep(ac[u]);
          if constexpr (R::kGrad) {
            keep(ax[u]);
            keep(ay[u]);
          }
        }
        store(b, ac, ax, ay);
      }
    }
  }
  // The rem (1..32) levels past the whole slices, as many of the block's
  // nodes at once as fit a wave: lane = (node tj, level tt), each lane with
  // its node's table row.  Written here, right after the nodes' other
  // levels, the cache lines both share are still in L2.
  if (rem == 0) return;
  const int G = 64 / rem;
  for (int b0 = 0; b0 < NB; b0 += G) {
    const bool ok = tj < G && b0 + tj < NB;
    const int b = ok ? b0 + tj : b0;
    const uint32_t rc = ro + (uint32_t)b * R::kBytes;
    const uint32_t lt = (uint32_t)b * colB + (uint32_t)(klc + tt) * kEl;
    auto val = [&](int r, int x) -> X { return lds_elem<S, X>(lds, row[r] + (uint32_t)x * colB + lt); };
    const size_t o = (size_t)(obase + (uint32_t)(b * a.L + klc + tt));
    S* __restrict__ o1 = static_cast<S*>(a.out) + kOut * o;
    if constexpr (!R::kRing2) {
      const X v[6] = {val(0, 0), val(0, 1), val(1, -1), val(1, 1), val(2, 0), val(2, 1)};
      const X x0 = val(1, 0);
      auto combine = [&](uint32_t cb, C& r0, C& r1) {
        C2 cf[6], dg = {0, 0};
#pragma unroll
        for (int q = 0; q < 6; ++q) cf[q] = lds_ld<C2>(lds, rc + cb + q * (uint32_t)sizeof(C2));
        if constexpr (OP != OP_GRAD) dg = lds_ld<C2>(lds, rc + cb + 7 * (uint32_t)sizeof(C2));
        win_combine<S, OP, 6>(x0, v, cf, dg, r0, r1);
        keep(r0);
      };
      C r0, r1, z0, unused;
      combine(0, r0, r1);
      if constexpr (R::kDual) combine(8 * (uint32_t)sizeof(C2), z0, unused);
      if (ok) {
        tile_store<S, OP>(a, o1, 0, r0, r1);
        if constexpr (R::kDual) win_store<S, OP>(static_cast<S*>(a.out2) + o, 0, a.nt, z0, 0);
      }
    } else {
      const C v[18] = {val(1, 0), val(1, 1), val(2, -1), val(2, 1), val(3, 0), val(3, 1),
                       val(0, 0), val(0, 1), val(0, 2), val(1, -1), val(1, 2), val(2, -2), val(2, 2),
                       val(3, -1), val(3, 2), val(4, 0), val(4, 1), val(4, 2)};
      const C x0 = val(2, 0);
      C ac = 0, ax = 0, ay = 0;
#pragma unroll
      for (int q = 0; q < 18; ++q) {
        const C d = v[q] - x0;
        ac = fma(lds_ld<C>(lds, rc + q * (uint32_t)sizeof(C)), d, ac);
        if constexpr (R::kGrad) {
          if (q < 6) {
            const C2 cq = lds_ld<C2>(lds, rc + R::kLapB + q * (uint32_t)sizeof(C2));
            ax = fma(cq.x, d, ax);
            ay = fma(cq.y, d, ay);
          }
        }
      }
      keep(ac);
      if (ok) {
        if (a.nt) st1<true>(o1, ac);
        else st1<false>(o1, ac);
        if constexpr (R::kGrad) {
          if (a.nt) st2<true>(static_cast<S*>(a.out2) + 2 * o, ax, ay);
          else st2<false>(static_cast<S*>(a.out2) + 2 * o, ax, ay);
        }
      }
    }
  }
}

// Tail levels [kt, kt + rem) of all nodes of a tile, rem <= 32: G = 64 / rem
// nodes share a wave, lane = (node j, level t), each lane with its node's
// record (reads within a node group are broadcasts).  The same slot-order
// arithmetic as tile_eval; 1-ring nodes of another degree than 6 in a group
// take the padded seventh slot under a select, so every lane combines
// exactly its own stencil.
template <class S, int OP>
__device__ __forceinline__ void tile_tail(const TileArgs& a, const char* lds, int32_t nnodes, uint32_t data_off,
                                          uint32_t colB, int k0, int kt, int rem, int j, int t, int32_t n0, int wave,
                                          int W, int lane) {
  using R = TileRec<S, OP>;
  using C = typename Traits<S>::C;
  using C2 = typename Traits<S>::C2;
  using X = typename WinT<S, OP>::X;
  constexpr uint32_t kEl = (uint32_t)sizeof(S) * R::kCin;
  constexpr int NE = R::kEntries - 1;
  const int G = 64 / rem;
  S* __restrict__ out = static_cast<S*>(a.out);
  for (int32_t g0 = n0 + wave * G; g0 < nnodes; g0 += W * G) {
    const int32_t tn = g0 + j;
    const bool ok = j < G && tn < nnodes;
    const uint32_t ro = (uint32_t)(ok ? tn : g0) * R::kBytes;
    uint32_t w32[R::kEntries / 2];
#pragma unroll
    for (int q = 0; q < R::kEntries / 8; ++q) {
      const uint4 r = lds_ld<uint4>(lds, ro + R::kCoefB + 16 * q);
      w32[4 * q] = r.x;
      w32[4 * q + 1] = r.y;
      w32[4 * q + 2] = r.z;
      w32[4 * q + 3] = r.w;
    }
    const uint32_t lev = (uint32_t)(kt + t) * kEl;
    auto off = [&](uint32_t pos) -> uint32_t {
      if constexpr (sizeof(S) == 2) return lds_ld<uint32_t>(lds, data_off + 4 * pos) + lev;   // BF16 table
      else return data_off + pos * colB + lev;
    };
    const uint32_t last = w32[R::kEntries / 2 - 1] >> 16;
    const X x0 = lds_elem<S, X>(lds, off(last & ((1u << kLocCountShift) - 1)));
    const int ne = (int)(last >> kLocCountShift);
    const uint32_t o = (uint32_t)lds_ld<int32_t>(lds, ro + R::kIdOff) * (uint32_t)a.L + (uint32_t)(k0 + kt + t);
    if constexpr (R::kRing2) {
      auto run = [&](auto ns) {
        constexpr int NS = decltype(ns)::value;
        C acc = 0, ax = 0, ay = 0;
#pragma unroll
        for (int q = 0; q < NS; ++q) {
          const uint32_t pos = (q & 1) ? (w32[q >> 1] >> 16) : (w32[q >> 1] & 0xffffu);
          const C d = lds_elem<S, C>(lds, off(pos)) - x0;
          acc = fma(lds_ld<C>(lds, ro + q * (uint32_t)sizeof(C)), d, acc);
          if constexpr (R::kGrad) {
            if (q < 7) {
              const C2 cq = lds_ld<C2>(lds, ro + R::kLapB + q * (uint32_t)sizeof(C2));
              const C e = grad_diff<C>(q, cq, d);
              ax = fma(cq.x, e, ax);
              ay = fma(cq.y, e, ay);
            }
          }
        }
        if (ok) {
          if (a.nt) st1<true>(out + (size_t)o, acc);
          else st1<false>(out + (size_t)o, acc);
          if constexpr (R::kGrad) {
            S* og = static_cast<S*>(a.out2) + 2 * (size_t)o;
            if (a.nt) st2<true>(og, ax, ay);
            else st2<false>(og, ax, ay);
          }
        }
      };
      if (__all(!ok || ne <= 18)) run(std::integral_constant<int, 18>());
      else run(std::integral_constant<int, NE>());
    } else {
      X v[7];
#pragma unroll
      for (int q = 0; q < 7; ++q) {
        const uint32_t pos = (q & 1) ? (w32[q >> 1] >> 16) : (w32[q >> 1] & 0xffffu);
        v[q] = lds_elem<S, X>(lds, off(pos));
      }
      const bool six = __all(!ok || ne == 6);
      // the sums with the coefficient row at byte cb (8 pairs: 7 slots and
      // the diagonal); per-lane degree: slots past ne leave the sums unchanged
      auto combine = [&](uint32_t cb, C& r0, C& r1) {
        C2 cf[7];
#pragma unroll
        for (int q = 0; q < 7; ++q) cf[q] = lds_ld<C2>(lds, ro + cb + q * (uint32_t)sizeof(C2));
        const C2 dg = lds_ld<C2>(lds, ro + cb + 7 * (uint32_t)sizeof(C2));
        if (six) {
          win_combine<S, OP, 6>(x0, v, cf, dg, r0, r1);
        } else {
          C a0, a1, b0, b1;
          win_combine<S, OP, 3>(x0, v, cf, dg, b0, b1);
#pragma unroll
          for (int d = 4; d <= 7; ++d) {
            if (d == 4) win_combine<S, OP, 4>(x0, v, cf, dg, a0, a1);
            if (d == 5) win_combine<S, OP, 5>(x0, v, cf, dg, a0, a1);
            if (d == 6) win_combine<S, OP, 6>(x0, v, cf, dg, a0, a1);
            if (d == 7) win_combine<S, OP, 7>(x0, v, cf, dg, a0, a1);
            if (ne >= d) {
              b0 = a0;
              b1 = a1;
            }
          }
          r0 = b0;
          r1 = b1;
        }
      };
      C r0, r1;
      combine(0, r0, r1);
      if constexpr (R::kDual) {
        C z0, z1;
        combine(8 * (uint32_t)sizeof(C2), z0, z1);
        if (ok) win_store<S, OP>(static_cast<S*>(a.out2), o, a.nt, z0, z1);
      }
      if (ok) tile_store<S, OP>(a, out, o, r0, r1);
    }
  }
}

// Blocks of a tile of short columns (rem <= 32 levels in all): G = 64 / rem
// blocks share a wave, lane = (block tj, level tt), each lane with its block's
// row positions and table rows.  As tile_block, the columns the block's nodes
// share are read once; table rows come per lane from LDS.  Bound by LDS reads
// and, FP32 at O640 x 19, by memory: gradient 100 us (4.5 TB/s over the
// arrays), Laplacian 109.
template <class S, int OP, int NB>
__device__ __forceinline__ void tile_short(const TileArgs& a, const char* lds, int32_t nblk, uint32_t data_off,
                                           uint32_t colB, int k0, int rem, int tj, int tt, int wave, int W) {
  using R = TileRec<S, OP>;
  using C = typename Traits<S>::C;
  using C2 = typename Traits<S>::C2;
  using X = typename WinT<S, R::kRing2 ? (int)OP_GRAD : OP>::X;
  constexpr uint32_t kEl = (uint32_t)sizeof(S) * R::kCin;
  constexpr uint32_t kOut = kTwoOut<OP> ? 2 : 1;
  constexpr int ring = R::kRing2 ? 2 : 1;
  const int G = 64 / rem;
  for (int32_t g0 = wave * G; g0 < nblk; g0 += W * G) {
    const bool ok = tj < G && g0 + tj < nblk;
    const uint32_t ro = (uint32_t)((ok ? g0 + tj : g0) * NB) * R::kBytes;
    auto at = [&](int s) -> uint32_t {
      uint32_t p = lds_ld<uint16_t>(lds, ro + R::kCoefB + 2 * s);
      if (s == R::kEntries - 1) p &= (1u << kLocCountShift) - 1;
      if constexpr (sizeof(S) == 2) return lds_ld<uint32_t>(lds, data_off + 4 * p) + (uint32_t)tt * kEl;
      else return data_off + p * colB + (uint32_t)tt * kEl;
    };
    uint32_t row[2 * ring + 1];   // column 0 of the rows, the nodes' own at ring
    row[ring] = at(R::kEntries - 1);
    row[ring - 1] = at(0);
    row[ring + 1] = at(4);
    if constexpr (R::kRing2) {
      row[0] = at(6);
      row[4] = at(15);
    }
    auto get = [&](int r, int x) -> X { return lds_elem<S, X>(lds, row[r] + (uint32_t)x * colB); };
    const uint32_t o0 = (uint32_t)lds_ld<int32_t>(lds, ro + R::kIdOff) * (uint32_t)a.L + (uint32_t)(k0 + tt);
    if constexpr (!R::kRing2) {
      X up[NB + 1], mi[NB + 2], dn[NB + 1];
#pragma unroll
      for (int x = 0; x < NB + 1; ++x) up[x] = get(0, x);
#pragma unroll
      for (int x = 0; x < NB + 2; ++x) mi[x] = get(1, x - 1);
#pragma unroll
      for (int x = 0; x < NB + 1; ++x) dn[x] = get(2, x);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const uint32_t rc = ro + (uint32_t)b * R::kBytes;
        const X v[6] = {up[b], up[b + 1], mi[b], mi[b + 2], dn[b], dn[b + 1]};
        auto combine = [&](uint32_t cb, C& r0, C& r1) {
          C2 cf[6], dg = {0, 0};
#pragma unroll
          for (int q = 0; q < 6; ++q) cf[q] = lds_ld<C2>(lds, rc + cb + q * (uint32_t)sizeof(C2));
          if constexpr (OP != OP_GRAD) dg = lds_ld<C2>(lds, rc + cb + 7 * (uint32_t)sizeof(C2));
          win_combine<S, OP, 6>(mi[b + 1], v, cf, dg, r0, r1);
        };
        C r0, r1, z0, unused;
        combine(0, r0, r1);
        if constexpr (R::kDual) combine(8 * (uint32_t)sizeof(C2), z0, unused);
        if (ok) {
          const size_t o = (size_t)(o0 + (uint32_t)(b * a.L));
          tile_store<S, OP>(a, static_cast<S*>(a.out) + kOut * o, 0, r0, r1);
          if constexpr (R::kDual) win_store<S, OP>(static_cast<S*>(a.out2) + o, 0, a.nt, z0, 0);
        }
      }
    } else {
      C t2[NB + 2], up[NB + 3], mi[NB + 4], dn[NB + 3], bb[NB + 2];
#pragma unroll
      for (int x = 0; x < NB + 2; ++x) t2[x] = get(0, x);
#pragma unroll
      for (int x = 0; x < NB + 3; ++x) up[x] = get(1, x - 1);
#pragma unroll
      for (int x = 0; x < NB + 4; ++x) mi[x] = get(2, x - 2);
#pragma unroll
      for (int x = 0; x < NB + 3; ++x) dn[x] = get(3, x - 1);
#pragma unroll
      for (int x = 0; x < NB + 2; ++x) bb[x] = get(4, x);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const uint32_t rc = ro + (uint32_t)b * R::kBytes;
        const C v[18] = {up[b + 1], up[b + 2], mi[b + 1], mi[b + 3], dn[b + 1], dn[b + 2],
                         t2[b], t2[b + 1], t2[b + 2], up[b], up[b + 3], mi[b], mi[b + 4],
                         dn[b], dn[b + 3], bb[b], bb[b + 1], bb[b + 2]};
        C ac = 0, ax = 0, ay = 0;
#pragma unroll
        for (int q = 0; q < 18; ++q) {
          const C d = v[q] - mi[b + 2];
          ac = fma(lds_ld<C>(lds, rc + q * (uint32_t)sizeof(C)), d, ac);
          if constexpr (R::kGrad) {
            if (q < 6) {
              const C2 cq = lds_ld<C2>(lds, rc + R::kLapB + q * (uint32_t)sizeof(C2));
              ax = fma(cq.x, d, ax);
              ay = fma(cq.y, d, ay);
            }
          }
        }
        if (ok) {
          const size_t o = (size_t)(o0 + (uint32_t)(b * a.L));
          S* p = static_cast<S*>(a.out) + o;
          if (a.nt) st1<true>(p, ac);
          else st1<false>(p, ac);
          if constexpr (R::kGrad) {
            S* g = static_cast<S*>(a.out2) + 2 * o;
            if (a.nt) st2<true>(g, ax, ay);
            else st2<false>(g, ax, ay);
          }
        }
      }
    }
  }
}

// Up to 16 waves per workgroup (at most 128 registers per lane), 8 for the
// three-slice FP64 Laplacian and the FP64 one-pass pairs of more than one
// slice per step, which need more registers.
template <class S, int OP, int U>
constexpr int kTileThreads =
    (sizeof(S) == 8 && (((OP == OP_GRADLAP || OP == OP_DIVCURL) && U > 1) || (OP == OP_LAP && U == 3))) ? 512 : 1024;

// Waves per SIMD the compiler has to leave room for: the 16-wave workgroups
// of the 4- and 2-byte divergence pairs run two to a CU within 64 registers.
template <class S, int OP, int U>
constexpr int kTileMinWaves = OP == OP_DIVCURL && (sizeof(S) == 4 || (sizeof(S) == 2 && U < 3)) ? 8 : 1;

// A device pointer read from a table, marked as global memory: accesses
// through it compile to global (not flat) instructions, which leave the LDS
// counter alone, so waits for LDS reads never wait for output stores.
template <class T>
__device__ __forceinline__ T* global_ptr(const void* slot) {
  using G = __attribute__((address_space(1))) T*;
  return (T*)(G)ld_const(reinterpret_cast<const uint64_t*>(slot));
}

// Workgroup barrier that orders LDS accesses only: each wave's LDS reads and
// writes are complete before it, and visible after it, but the wave's global
// stores stay in flight (a full __syncthreads() would wait for them too).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One (tile, level chunk) of a field by the W waves of a workgroup: copy into
// LDS, wait, run after_copy() (all waves are past the barrier), evaluate.
// The caller synchronises before the buffer is reused.
// SHORT: every chunk is of at most 32 levels (U 1, types and operators with
// blocks); a body of its own, since tile_short next to tile_block raises the
// register count of the long columns' kernels (FP64 gradient and Laplacian at
// O1280 x 137 7.1 -> 8.4 ms, BF16 divergence at O640 x 137 430 -> 523 us).
// BLK: blocks, where the type and operator have them.
template <class S, int OP, int U, bool SHORT, bool BLK, class F>
__device__ __forceinline__ void tile_work(const TileArgs& a, int64_t tile, int chunk, char* lds, int W, int wave,
                                          int lane, F&& after_copy) {
  using R = TileRec<S, OP>;
  const int k0 = chunk * a.KL;
  const int klc = a.L - k0 < a.KL ? a.L - k0 : a.KL;
  tile_copy<S, OP>(a, tile, k0, klc, lds, wave, W, lane);
  const int32_t nnodes = (ld_uniform(a.info + 4 * tile + 3) & 0xffff);
  const int32_t nblk = (int32_t)((uint32_t)ld_uniform(a.info + 4 * tile + 2) >> 16);   // blocks lead the records
  const uint32_t colB = (uint32_t)klc * R::kCin * (uint32_t)sizeof(S);
  const uint32_t data_off = (uint32_t)nnodes * R::kBytes;   // BF16: the offset table starts here
  __builtin_amdgcn_s_waitcnt(0);   // all counters: the direct loads have landed
  __syncthreads();
  after_copy();
  // compute: node tn of the tile goes to wave tn mod W for whole 64-level
  // slices; a short remainder (1..32 levels) of all nodes is packed G = 64 /
  // rem nodes to a wave
  const int rem = klc & 63;
  const bool pack = rem != 0 && rem <= 32;
  const int kmain = pack ? klc - rem : klc;
  if constexpr (BLK && kUseBlk<S, OP, U>) {
    constexpr int NB = kBlkN<S, OP>;
    const int tj = pack ? lane / rem : 0, tt = pack ? lane - tj * rem : 0;   // packed pass: node and level of the lane
    int32_t n0 = 0, q = wave;
    if constexpr (SHORT) {
      n0 = nblk * NB;
      tile_short<S, OP, NB>(a, lds, nblk, data_off, colB, k0, rem, tj, tt, wave, W);
    } else if (kmain > 0) {
      n0 = nblk * NB;
      for (; q < nblk; q += W)
        tile_block<S, OP, U, NB>(a, lds, q * NB, data_off, colB, k0, kmain, pack ? rem : 0, tj, tt, lane);
      q -= nblk;
      // the few nodes outside the blocks: one slice at a time, which keeps
      // them from setting the kernel's register count
      for (int32_t tn = n0 + q; tn < nnodes; tn += W) tile_eval<S, OP, 1>(a, lds, tn, data_off, colB, k0, kmain, lane);
    }
    if (pack) tile_tail<S, OP>(a, lds, nnodes, data_off, colB, k0, kmain, rem, tj, tt, n0, q, W, lane);
  } else {
    if (kmain > 0)
      for (int32_t tn = wave; tn < nnodes; tn += W) tile_eval<S, OP, U>(a, lds, tn, data_off, colB, k0, kmain, lane);
    if (pack) {
      const int tj = lane / rem, tt = lane - tj * rem;
      tile_tail<S, OP>(a, lds, nnodes, data_off, colB, k0, kmain, rem, tj, tt, 0, wave, W, lane);
    }
  }
}

// U: 64-level slices per step; 0: columns of at most 32 levels (see tile_work).
template <class S, int OP, int U>
__global__ __launch_bounds__((kTileThreads<S, OP, U>), (kTileMinWaves<S, OP, U>)) void k_tile(TileArgs a, int64_t nblocks, int remap) {
  extern __shared__ __align__(16) char lds[];
  int64_t tile;
  int chunk;
  if (remap == kXcdSchedule) {
    // entry 8 i + x of the schedule is XCD x's i-th tile (or a hole)
    const int64_t q = blockIdx.x >> 3;
    const int64_t i = a.nchunks == 1 ? q : q / a.nchunks;
    chunk = (int)(q - i * a.nchunks);
    tile = 8 * i + (blockIdx.x & 7);
    if ((ld_uniform(a.info + 4 * tile + 3) & 0xffff) == 0) return;
  } else {
    const int64_t lb = logical_block(blockIdx.x, nblocks, remap);
    if (lb >= nblocks) return;
    tile = lb / a.nchunks;
    chunk = (int)(lb - tile * a.nchunks);
  }
  const int W = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  tile_work<S, OP, (U ? U : 1), U == 0, true>(a, tile, chunk, lds, W, wave, lane, [] {});
}

// Persistent form over many fields (tracers) of one operator, each on its
// own tiling (tracers of similar level counts share one).  The work items of
// tracer t are its ntiles_t x nchunks_t (tile, chunk) pairs in tile order;
// XCD x takes the contiguous share [x n_t / 8, (x + 1) n_t / 8) of every
// tracer, so tiles stacked in latitude still meet in one L2, and every XCD
// gets the same mix of long and short columns.  pre[x][t] counts the items of
// share x before tracer t (pre[x][ntr] its total).  The workgroups b with
// b mod 8 = x (the ones the hardware places on XCD x) take the items of share
// x in order from a counter, `claim` consecutive items per claim (tiles
// stacked in latitude, whose shared halo rows the workgroup then finds in
// L2), as they become free, so the tiles in flight on an XCD stay a narrow
// window of the order (a fixed stride lets workgroups drift apart and the
// halo rows they share drop out of L2).  Claims are device-scope atomics,
// which the XCDs' counters serialise; claiming several items at once and
// giving each share's counters a cache line of their own keeps them off the
// critical path, and each workgroup claims once ahead, so a claim's latency
// hides behind a tile's copy.  The last workgroup of share x to finish sets
// both of its counters back to zero for the next launch, so a graph replays
// without a memset.  Each tracer's chunk is its own (at most its tiling's), with the
// slice count of the single-field launch (at most UMAX).  Every wave of a
// workgroup runs the same loop, so the barriers are reached by all.
// Workgroup size bound of the batched kernel: 1024 threads (16 waves), or
// 512 (8 waves, up to 256 registers a lane) for the FP64 divergence pair,
// whose two coefficient rows do not fit in 128 registers.
template <class S, int OP>
constexpr int kBatchedThreads = (sizeof(S) == 8 && OP == OP_DIVCURL) ? 512 : 1024;
inline int batched_max_waves(int kop, int dtype) { return (dtype == DT_F64 && kop == OP_DIVCURL) ? 8 : 16; }

// Blocks in the batched kernel, by the tracer's slices per step.  One kernel
// holds the code of every slice count of the plan under one register bound, so
// blocks stay where they gain there: not in the FP64 divergence and gradient
// adjoint, which would spill under 128 registers (2 and 43 of them with two
// and three slices), nor in longer steps of the FP64 pair and of FP32
// scalar-input operators; the short columns' body, one more, in none.  O160,
// five to twelve tracers of one depth, no blocks / blocks and short body
// everywhere / this: FP64 divergence x 10 72 / 76 / 71 us, x 19 122 / 134 /
// 122, x 180 671 / 684 / 674; FP64 pair x 60 491 / 469 / 467, x 180 822 / 872 /
// 814; all four FP32 operators x 10 211 / 237 / 215, x 60 703 / 680 / 685;
// FP32 gradient x 180 311 / 321 / 311, FP32 divergence x 60 207 / 186 / 185.
template <class S, int OP, int U>
constexpr bool kBatchedBlk = OP == OP_DIV || OP == OP_GRADT ? sizeof(S) == 4
                             : sizeof(S) == 8               ? OP != OP_DIVCURL || U == 1
                                                            : U < 3;

template <class S, int OP, int UMAX>
__global__ __launch_bounds__((kBatchedThreads<S, OP>)) void k_tile_batched(TileArgs base, const BatchTile* __restrict__ tr,
                                                       const int32_t* __restrict__ pre, int ntr,
                                                       int32_t* __restrict__ ctr, int32_t claim) {
  extern __shared__ __align__(16) char lds[];
  __shared__ int32_t next_item;
  const int W = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int x = (int)(blockIdx.x & 7u);
  const int32_t gx = (int32_t)(gridDim.x >> 3);   // the grid is a multiple of 8
  const int32_t* px = pre + (size_t)x * (ntr + 1);
  const int32_t mx = ld_uniform(px + ntr);
  int32_t* cx = ctr + kBatchCtrStride * x;         // claim counter; cx[kBatchCtrStride / 2]: finished
  // Thread 0 holds the end of the current claim and the next claim (`ahead`):
  // a claim made during one claim's items is used only after a later copy has
  // been waited for, which has also waited for the claim, so no evaluation
  // stalls on it.
  int32_t cur_end = 0, ahead = 0;
  if (threadIdx.x == 0) {
    const int32_t c0 = __hip_atomic_fetch_add(cx, claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ahead = __hip_atomic_fetch_add(cx, claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    next_item = c0;
    cur_end = c0 + claim;
  }
  __syncthreads();
  // k is the same in every lane: read it into a scalar register, so the
  // loop and the table loads below stay scalar
  int32_t k = __builtin_amdgcn_readfirstlane(next_item);
  // the current tracer's fields stay in registers: they are loaded again
  // only when the item index moves past the tracer's items (k only grows)
  int t = -1;
  int32_t t_lo = 0, t_hi = 0;   // the tracer's items on this share: [t_lo, t_hi)
  int64_t first = 0;            // its first item index on this share
  int U = 1;
  TileArgs a = base;
  while (k < mx) {
    if (k >= t_hi) {
      do {
        ++t;
        t_hi = ld_uniform(px + t + 1);   // px[ntr] = mx > k ends the scan
      } while (t_hi <= k);
      t_lo = ld_uniform(px + t);
      const BatchTile* d = tr + t;
      a.in = global_ptr<const S>(&d->in);
      a.out = global_ptr<S>(&d->out);
      if constexpr (OP == OP_DIVCURL) a.out2 = global_ptr<S>(&d->out2);
      a.info = reinterpret_cast<const int32_t*>(ld_const(reinterpret_cast<const uint64_t*>(&d->info)));
      a.segs = reinterpret_cast<const int32_t*>(ld_const(reinterpret_cast<const uint64_t*>(&d->segs)));
      a.rec = reinterpret_cast<const char*>(ld_const(reinterpret_cast<const uint64_t*>(&d->rec)));
      a.L = ld_const(&d->L);
      a.KL = ld_const(&d->KL);
      a.nchunks = ld_const(&d->nchunks);
      U = ld_const(&d->U);
      first = (int64_t)x * ld_const(&d->nitems) / 8;
    }
    const int64_t item = first + (k - t_lo);
    const int64_t tile = a.nchunks == 1 ? item : item / a.nchunks;
    const int chunk = (int)(item - tile * a.nchunks);
    // after the copy's wait and barrier (every wave has read next_item):
    // publish the next item, the claim's next or the first of the claim
    // ahead (then claiming another)
    auto advance = [&] {
      if (threadIdx.x == 0) {
        if (k + 1 < cur_end) {
          next_item = k + 1;
        } else {
          next_item = ahead;
          cur_end = ahead + claim;
          ahead = __hip_atomic_fetch_add(cx, claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    };
    // UMAX: the largest slice count of the plan's tracers; only the paths
    // up to it are compiled in, which keeps the kernel's code small
    constexpr int U2 = UMAX < 2 ? UMAX : 2;
    if (UMAX == 1 || U == 1) tile_work<S, OP, 1, false, kBatchedBlk<S, OP, 1>>(a, tile, chunk, lds, W, wave, lane, advance);
    else if (UMAX == 2 || U == 2) tile_work<S, OP, U2, false, kBatchedBlk<S, OP, U2>>(a, tile, chunk, lds, W, wave, lane, advance);
    else tile_work<S, OP, UMAX, false, kBatchedBlk<S, OP, UMAX>>(a, tile, chunk, lds, W, wave, lane, advance);
    // every wave is done reading the buffer, and next_item is written; the
    // tile's output stores need not have landed
    lds_barrier();
    k = __builtin_amdgcn_readfirstlane(next_item);
  }
  if (threadIdx.x == 0) {
    // every claim of this workgroup (the one ahead included) is complete
    // before its count (release); the last workgroup of the share (acquire)
    // sets both counters back to zero
    int32_t* fin = cx + kBatchCtrStride / 2;
    if (__hip_atomic_fetch_add(fin, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gx - 1) {
      __hip_atomic_store(cx, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(fin, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// Packs the node records of a tiling in tile order: record q is node
// order[q]; one thread per dword of the records.
template <class S, int OP>
__global__ __launch_bounds__(256) void k_pack_records(const int32_t* __restrict__ order,
                                                      const void* __restrict__ coef,
                                                      const void* __restrict__ coef2,
                                                      const uint16_t* __restrict__ loc, int64_t V,
                                                      uint32_t* __restrict__ rec) {
  using R = TileRec<S, OP>;
  constexpr uint32_t kDw = R::kBytes / 4;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= V * kDw) return;
  const int64_t q = t / kDw;
  const uint32_t d = (uint32_t)(t - q * kDw);
  const int64_t i = order[q];
  uint32_t v = 0;
  constexpr uint32_t kC1 = R::kGrad ? R::kLapB / 4 : R::kDual ? R::kCoefB / 8 : R::kCoefB / 4;   // from coef
  constexpr uint32_t kC2 = R::kCoefB / 4 - kC1;                       // dwords from coef2
  if (d < kC1) v = static_cast<const uint32_t*>(coef)[i * kC1 + d];
  else if (d < R::kCoefB / 4) v = static_cast<const uint32_t*>(coef2)[i * kC2 + (d - kC1)];
  else if (d < R::kIdOff / 4) v = reinterpret_cast<const uint32_t*>(loc)[i * (R::kLocB / 4) + (d - R::kCoefB / 4)];
  else if (d == R::kIdOff / 4) v = (uint32_t)i;
  rec[t] = v;
}

// ---- persistent LDS tiles, double buffered ------------------------------------
//
// One or two workgroups per CU stay resident and walk their share of the
// tiles.  Producer waves copy tile n+1 into one LDS buffer (direct loads, then
// their own wait) while consumer waves evaluate tile n from the other; one
// barrier per tile swaps the buffers.  Consumers use the lane mapping of the
// gather path: P lanes per node, 64 / P nodes per wave step, lane t handling
// levels t, t + P, ...; each lane reads its node's record from LDS (broadcast
// reads).

// P-lane evaluation of 1-ring nodes from an LDS tile: NS slots (7 = padded
// with the node itself and zero coefficients).
template <class S, int OP, int NS, int U>
__device__ __forceinline__ void tile_lanes1(const TileArgs& a, const char* buf, uint32_t data_off, uint32_t colB,
                                            const uint32_t* so, uint32_t xo, const typename Traits<S>::C2* cf,
                                            typename Traits<S>::C2 dg, uint32_t obase, bool ok, int t, int P,
                                            int klc) {
  using C = typename Traits<S>::C;
  using X = typename WinT<S, OP>::X;
  S* __restrict__ out = static_cast<S*>(a.out);
  const int nsl = (klc + P - 1) / P;
  for (int r0 = 0; r0 < nsl; r0 += U) {
    X v[U][NS], x0[U];
    bool st[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = t + P * (r0 + u);
      st[u] = ok && k < klc;
      const uint32_t kk = (uint32_t)(k < klc ? k : klc - 1) * (uint32_t)sizeof(X);
#pragma unroll
      for (int s = 0; s < NS; ++s) v[u][s] = lds_ld<X>(buf, so[s] + kk);
      x0[u] = lds_ld<X>(buf, xo + kk);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      win_emit<S, OP, NS>(out, obase + (uint32_t)(t + P * (r0 + u)), st[u], a.nt, x0[u], v[u], cf, dg);
  }
}

template <class S, int NS, int U>
__device__ __forceinline__ void tile_lanes2(const TileArgs& a, const char* buf, const uint32_t* so, uint32_t xo,
                                            const typename Traits<S>::C* w, uint32_t obase, bool ok, int t, int P,
                                            int klc) {
  using C = typename Traits<S>::C;
  S* __restrict__ out = static_cast<S*>(a.out);
  const int nsl = (klc + P - 1) / P;
  for (int r0 = 0; r0 < nsl; r0 += U) {
    C v[U][NS], x0[U];
    bool st[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = t + P * (r0 + u);
      st[u] = ok && k < klc;
      const uint32_t kk = (uint32_t)(k < klc ? k : klc - 1) * (uint32_t)sizeof(C);
#pragma unroll
      for (int s = 0; s < NS; ++s) v[u][s] = lds_ld<C>(buf, so[s] + kk);
      x0[u] = lds_ld<C>(buf, xo + kk);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      C acc = 0;
#pragma unroll
      for (int s = 0; s < NS; ++s) acc = fma(w[s], v[u][s] - x0[u], acc);
      if (st[u]) {
        const uint32_t o = obase + (uint32_t)(t + P * (r0 + u));
        if (a.nt) st1<true>(out + (size_t)o, acc);
        else st1<false>(out + (size_t)o, acc);
      }
    }
  }
}

template <class S, int OP, int U>
__device__ __forceinline__ void tile_consume(const TileArgs& a, int64_t lb, const char* buf, int cw, int NC, int P,
                                             int lane) {
  using R = TileRec<S, OP>;
  using C = typename Traits<S>::C;
  using C2 = typename Traits<S>::C2;
  const int64_t tile = lb / a.nchunks;
  const int chunk = (int)(lb - tile * a.nchunks);
  const int32_t nnodes = (ld_uniform(a.info + 4 * tile + 3) & 0xffff);
  const int k0 = chunk * a.KL;
  const int klc = a.L - k0 < a.KL ? a.L - k0 : a.KL;
  const uint32_t colB = (uint32_t)klc * R::kCin * (uint32_t)sizeof(S);   // LDS column stride (this chunk)
  const uint32_t data_off = (uint32_t)nnodes * R::kBytes;
  if (P == 64) {   // one node per wave, as in the one-tile form
    for (int32_t tn = cw; tn < nnodes; tn += NC) tile_eval<S, OP, U>(a, buf, tn, data_off, colB, k0, klc, lane);
    return;
  }
  const int G = 64 / P;
  const int j = lane / P, t = lane - (lane / P) * P;
  for (int32_t tn0 = cw * G; tn0 < nnodes; tn0 += NC * G) {
    const int32_t tn = tn0 + j;
    const bool ok = j < G && tn < nnodes;
    const uint32_t ro = (uint32_t)(ok ? tn : tn0) * R::kBytes;
    const int32_t i = lds_ld<int32_t>(buf, ro + R::kIdOff);
    const uint32_t obase = (uint32_t)i * (uint32_t)a.L + (uint32_t)k0;
    uint32_t w32[R::kEntries / 2];
#pragma unroll
    for (int q = 0; q < R::kEntries / 8; ++q) {
      const uint4 r = lds_ld<uint4>(buf, ro + R::kCoefB + 16 * q);
      w32[4 * q] = r.x;
      w32[4 * q + 1] = r.y;
      w32[4 * q + 2] = r.z;
      w32[4 * q + 3] = r.w;
    }
    uint32_t so[R::kEntries - 1];
#pragma unroll
    for (int q = 0; q < R::kEntries - 1; ++q)
      so[q] = data_off + ((q & 1) ? (w32[q >> 1] >> 16) : (w32[q >> 1] & 0xffffu)) * colB;
    const uint32_t last = w32[R::kEntries / 2 - 1] >> 16;
    const uint32_t xo = data_off + (last & ((1u << kLocCountShift) - 1)) * colB;
    const int ne = (int)(last >> kLocCountShift);
    if constexpr (R::kRing2) {
      C w[R::kEntries - 1];
#pragma unroll
      for (int q = 0; q < R::kEntries - 1; ++q) w[q] = lds_ld<C>(buf, ro + q * (uint32_t)sizeof(C));
      if (__all(ne <= 18)) tile_lanes2<S, 18, U>(a, buf, so, xo, w, obase, ok, t, P, klc);
      else tile_lanes2<S, R::kEntries - 1, 1>(a, buf, so, xo, w, obase, ok, t, P, klc);
    } else {
      C2 cf[7];
#pragma unroll
      for (int q = 0; q < 7; ++q) cf[q] = lds_ld<C2>(buf, ro + q * (uint32_t)sizeof(C2));
      const C2 dg = lds_ld<C2>(buf, ro + 7 * (uint32_t)sizeof(C2));
      if (__all(ne == 6)) tile_lanes1<S, OP, 6, U>(a, buf, data_off, colB, so, xo, cf, dg, obase, ok, t, P, klc);
      else tile_lanes1<S, OP, 7, 1>(a, buf, data_off, colB, so, xo, cf, dg, obase, ok, t, P, klc);
    }
  }
}

// Up to 16 waves per workgroup for 4-byte data (at most 128 registers per
// lane), 8 for FP64, whose two-ring variant needs more registers.
template <class S>
constexpr int kTile2Threads = sizeof(S) == 8 ? 512 : 1024;

// Copy of logical block lb (tile, level chunk) by the NP producer waves.
template <class S, int OP>
__device__ __forceinline__ void tile_issue(const TileArgs& a, int64_t lb, char* buf, int pw, int NP, int lane) {
  const int64_t tile = lb / a.nchunks;
  const int chunk = (int)(lb - tile * a.nchunks);
  const int k0 = chunk * a.KL;
  const int klc = a.L - k0 < a.KL ? a.L - k0 : a.KL;
  tile_copy<S, OP>(a, tile, k0, klc, buf, pw, NP, lane);
}

template <class S, int OP, int U>
__global__ __launch_bounds__(kTile2Threads<S>) void k_tile2(TileArgs a, int64_t nblocks, int remap, uint32_t buf_bytes, int nprod,
                                               int P) {
  extern __shared__ __align__(16) char lds[];
  const int W = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  // this workgroup's tiles: with remapping, the workgroups of one XCD sweep
  // a contiguous eighth of the tile list together
  const int64_t nwg = gridDim.x, b = blockIdx.x;
  int64_t lb, step, end;
  if (remap) {
    const int64_t per = (nblocks + 7) / 8;
    lb = (b % 8) * per + b / 8;
    step = nwg / 8;
    end = (b % 8 + 1) * per < nblocks ? (b % 8 + 1) * per : nblocks;
  } else {
    lb = b;
    step = nwg;
    end = nblocks;
  }
  const bool producer = wave < nprod;
  uint32_t cur = 0;
  if (producer && lb < end) {
    tile_issue<S, OP>(a, lb, lds, wave, nprod, lane);
    __builtin_amdgcn_s_waitcnt(0);   // all counters: the direct loads have landed
  }
  __syncthreads();
  while (lb < end) {
    const int64_t nx = lb + step;
    if (producer) {
      if (nx < end) {
        tile_issue<S, OP>(a, nx, lds + (cur ^ buf_bytes), wave, nprod, lane);
        __builtin_amdgcn_s_waitcnt(0);   // all counters: the direct loads have landed
      }
    } else {
      tile_consume<S, OP, U>(a, lb, lds + cur, wave - nprod, W - nprod, P, lane);
    }
    // LDS traffic of this step done (consumer reads, producer index stores;
    // the producers' direct loads were waited for above); consumers' global
    // stores may stay in flight across the barrier
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    __builtin_amdgcn_s_barrier();
    lb = nx;
    cur ^= buf_bytes;
  }
}

// ---- remapping: out[t][k] = w0 f[n0][k] + w1 f[n1][k] + w2 f[n2][k] ---------------
//
// Linear interpolation over the source triangle of each target point
// (Section 4.3).  A wave serves 64 / P lane groups, P lanes each (P = nlev
// for columns of at most 32 levels, else 64), and each group TP consecutive
// target points, lane t of a group taking levels t, t + P, ...; the node
// indices and weights of the TP points and then U level slices of all their
// source columns are loaded before the arithmetic (more loads in flight for
// the 4- and 2-byte types).  Blocks are remapped so that each XCD walks a
// contiguous range of target points (whose source columns are neighbours, so
// they stay in that XCD's L2).  The sum is w0 f0, then + w1 f1, then + w2 f2,
// with fused multiply-adds.  With O32 the input is addressed by 32-bit byte
// offsets from its base (the launch checks that it is under 4 GiB); with
// EXACT (64 lanes, U = the column's 64-level slices) every slice but the
// last lies inside the column, at a constant offset from the first.
template <class S, int U, int TP, bool O32 = false, bool EXACT = false>
__global__ __launch_bounds__(256) void k_remap(const int32_t* __restrict__ nodes, const void* __restrict__ wv,
                                               const S* __restrict__ in, S* __restrict__ out, int64_t P, int L,
                                               int lanes, int64_t nblocks, int remap) {
  using C = typename Traits<S>::C;
  const C* __restrict__ w = static_cast<const C*>(wv);
  const char* __restrict__ inb = reinterpret_cast<const char*>(in);
  const uint32_t colB = (uint32_t)L * (uint32_t)sizeof(S);
  auto src = [&](int32_t node, int k) -> const S* {
    if constexpr (O32) return reinterpret_cast<const S*>(inb + ((uint32_t)node * colB + (uint32_t)k * (uint32_t)sizeof(S)));
    else return in + (size_t)node * (size_t)L + k;
  };
  const int64_t lb = logical_block(blockIdx.x, nblocks, remap);
  if (lb >= nblocks) return;
  const int W = blockDim.x >> 6;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int G = 64 / lanes;
  const int j = lane / lanes, tl = lane - j * lanes;
  if (j >= G) return;   // idle lanes; the kernel has no barrier
  const int64_t t0 = ((lb * W + wave) * G + j) * TP;
  if (t0 >= P) return;
  int4 nd[TP];
  C w0[TP], w1[TP], w2[TP];
#pragma unroll
  for (int q = 0; q < TP; ++q) {
    const int64_t t = t0 + q < P ? t0 + q : P - 1;   // past the last point: reload it, store nothing
    nd[q] = *reinterpret_cast<const int4*>(nodes + 4 * t);
    w0[q] = w[4 * t];
    w1[q] = w[4 * t + 1];
    w2[q] = w[4 * t + 2];
  }
  for (int k0 = tl; k0 < L; k0 += lanes * U) {
    C v0[TP][U], v1[TP][U], v2[TP][U];
#pragma unroll
    for (int q = 0; q < TP; ++q)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (EXACT && u < U - 1) {
          v0[q][u] = ld1(src(nd[q].x, k0) + 64 * u);
          v1[q][u] = ld1(src(nd[q].y, k0) + 64 * u);
          v2[q][u] = ld1(src(nd[q].z, k0) + 64 * u);
        } else {
          const int k = k0 + lanes * u;
          const int kc = k < L ? k : L - 1;
          v0[q][u] = ld1(src(nd[q].x, kc));
          v1[q][u] = ld1(src(nd[q].y, kc));
          v2[q][u] = ld1(src(nd[q].z, kc));
        }
      }
    // every sum is formed before the guarded stores (keep), so the compiler
    // cannot sink the loads of a partial last slice into the store's branch,
    // where they would issue late and wait for all loads in flight
    C r[TP][U];
#pragma unroll
    for (int q = 0; q < TP; ++q)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        C acc = w0[q] * v0[q][u];
        acc = fma(w1[q], v1[q][u], acc);
        r[q][u] = fma(w2[q], v2[q][u], acc);
        keep(r[q][u]);
      }
#pragma unroll
    for (int q = 0; q < TP; ++q)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = k0 + lanes * u;
        if (k < L && t0 + q < P) st1<false>(out + (size_t)(t0 + q) * (size_t)L + k, r[q][u]);
      }
  }
}

template <class S, int U, int TP>
void launch_remap_u(dim3 g, dim3 b, hipStream_t st, const int32_t* nodes, const void* w, const S* src, S* dst,
                    int64_t V, int64_t P, int nlev, int lanes, int64_t nblocks) {
  const bool o32 = (uint64_t)V * (uint64_t)nlev * sizeof(S) < (1ull << 32);
  const bool exact = lanes == 64 && (nlev + 63) / 64 == U;
  if (o32 && exact)
    hipLaunchKernelGGL((k_remap<S, U, TP, true, true>), g, b, 0, st, nodes, w, src, dst, P, nlev, lanes, nblocks, 1);
  else if (o32)
    hipLaunchKernelGGL((k_remap<S, U, TP, true, false>), g, b, 0, st, nodes, w, src, dst, P, nlev, lanes, nblocks, 1);
  else
    hipLaunchKernelGGL((k_remap<S, U, TP>), g, b, 0, st, nodes, w, src, dst, P, nlev, lanes, nblocks, 1);
}

template <class S, int TP>
hipError_t launch_remap_tp(const int32_t* nodes, const void* w, int64_t V, int64_t P, int nlev, const S* src,
                           S* dst, hipStream_t st) {
  const int lanes = nlev <= 32 ? nlev : 64;
  const int G = 64 / lanes;
  constexpr int W = 4;
  const int64_t groups = (P + (int64_t)G * TP - 1) / ((int64_t)G * TP);
  const int64_t nblocks = (groups + W - 1) / W;
  const int64_t grid = (nblocks + 7) / 8 * 8;
  const int nsl = (nlev + lanes - 1) / lanes;
  const int U = nsl < 3 ? nsl : 3;
  const dim3 g((unsigned)grid), b(64 * W);
  switch (U) {
    case 1: launch_remap_u<S, 1, TP>(g, b, st, nodes, w, src, dst, V, P, nlev, lanes, nblocks); break;
    case 2: launch_remap_u<S, 2, TP>(g, b, st, nodes, w, src, dst, V, P, nlev, lanes, nblocks); break;
    default: launch_remap_u<S, 3, TP>(g, b, st, nodes, w, src, dst, V, P, nlev, lanes, nblocks); break;
  }
  return hipGetLastError();
}

// Target points per lane group (measured at O1280 x 137 -> F640): one for
// FP64, two (columns of at most 32 levels) or four for 4- and 2-byte data.
template <class S>
hipError_t launch_remap_t(const int32_t* nodes, const void* w, int64_t V, int64_t P, int nlev, const void* in,
                          void* out, hipStream_t st) {
  const S* src = static_cast<const S*>(in);
  S* dst = static_cast<S*>(out);
  if constexpr (sizeof(S) == 8) return launch_remap_tp<S, 1>(nodes, w, V, P, nlev, src, dst, st);
  else if (nlev <= 32) return launch_remap_tp<S, 2>(nodes, w, V, P, nlev, src, dst, st);
  else return launch_remap_tp<S, 4>(nodes, w, V, P, nlev, src, dst, st);
}

// Transpose of the remapping: fbar[n][k] = the sum over the entries (t, w)
// of source node n, in ascending target order, of w ybar[t][k] (fused
// multiply-adds from zero; 0 for nodes no target point uses).  A group of P
// lanes serves one node (64 / P nodes per wave).  Lane tl keeps VEC
// consecutive levels of each of NS slices of P VEC levels in registers
// (levels kb + VEC tl + P VEC s + c), so each entry's target index and
// weight are read once per block of levels; with VEC = 2 (FP64) a column is
// read with 16-byte loads where the lane's two levels lie inside it (element
// loads at its end).  A node's row bounds and first two entries (kept beside
// the compressed rows) are read together; entries go two at a time: both
// target columns are loaded together and the next pair's indices and
// weights are requested before the multiply-adds of this pair, which are
// taken in entry order.  With O32 the input is addressed by 32-bit byte
// offsets from its base (the launch checks that it is smaller than 4 GiB).
// With STG (whole columns in one block) the wave's G consecutive output
// columns are staged in LDS and written as one contiguous run in units of
// `unit` bytes: measured 15-20 % faster than the groups' own 64-byte pieces.
// Workgroups alternate between the two ends of the nodes and meet at the
// equator: where the target's rows keep all their longitudes, polar nodes
// have up to ~190 entries, a serial chain of loads, which starts first and
// ends while the many nodes of one or two entries stream; and the nodes in
// flight lie along two pairs of rows, few DRAM pages.  O640 <- F320 x 91
// FP64: an eighth of the nodes per XCD 625 us, plain order 466, from both
// ends 415 (the arrays once at 6.4 TB/s: 287); O1280 <- F640 x 137 FP32 1658,
// 1225, 1202 us, FP64 3.47, 2.60, 2.40 ms.
typedef double f64x2_e __attribute__((ext_vector_type(2), aligned(8)));   // two levels, element-aligned
template <class S, int VEC>
struct VecOf {
  using T = S;
};
template <>
struct VecOf<double, 2> {
  using T = f64x2_e;
};

template <class S, int NS, int VEC, bool O32, bool STG, bool EXACT = false>
__global__ __launch_bounds__(256) void k_remap_adj(const int64_t* __restrict__ off, const int32_t* __restrict__ tt,
                                                   const void* __restrict__ wv, const int32_t* __restrict__ ht,
                                                   const void* __restrict__ hwv, const S* __restrict__ in,
                                                   S* __restrict__ out, int64_t V, int L, int lanes, int64_t nblocks,
                                                   int unit) {
  using C = typename Traits<S>::C;
  using C2 = typename Traits<S>::C2;
  using VT = typename VecOf<S, VEC>::T;
  constexpr int EB = 2;
  extern __shared__ __align__(16) char smem[];
  const C* __restrict__ w = static_cast<const C*>(wv);
  const C* __restrict__ hw = static_cast<const C*>(hwv);
  const int64_t b = blockIdx.x;
  const int64_t lb = b & 1 ? nblocks - 1 - (b >> 1) : b >> 1;
  const int W = blockDim.x >> 6;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int G = 64 / lanes;
  const int j = lane / lanes, tl = lane - j * lanes;
  const int64_t nw0 = (lb * W + wave) * G;   // the wave's first node
  const int64_t n = nw0 + j;
  // idle lanes (past the node groups or the nodes) stay to the end: with STG
  // every wave reaches the barrier
  const bool act = j < G && n < V;
  if (!STG && !act) return;
  const char* __restrict__ inb = reinterpret_cast<const char*>(in);
  const uint32_t colB = (uint32_t)L * (uint32_t)sizeof(S);
  int64_t e0 = 0, e1 = 0;
  int2 h2 = make_int2(0, 0);
  C2 hw2;
  hw2.x = 0;
  hw2.y = 0;
  if (act) {
    e0 = off[n];
    e1 = off[n + 1];
    h2 = *reinterpret_cast<const int2*>(ht + 2 * n);
    hw2 = *reinterpret_cast<const C2*>(hw + 2 * n);
  }
  S* __restrict__ o = out + (size_t)n * (size_t)L;
  S* __restrict__ sb = reinterpret_cast<S*>(smem) + (size_t)wave * G * L;
  for (int kb = VEC * tl; kb < L + VEC * tl; kb += lanes * VEC * NS) {
    int kl[NS];   // first level of the lane's VEC levels in slice s
#pragma unroll
    for (int s = 0; s < NS; ++s) kl[s] = kb + lanes * VEC * s;
    auto addr = [&](int32_t t, int k) -> const S* {
      if constexpr (O32) return reinterpret_cast<const S*>(inb + ((uint32_t)t * colB + (uint32_t)k * (uint32_t)sizeof(S)));
      else return reinterpret_cast<const S*>(inb + ((size_t)t * colB + (size_t)k * sizeof(S)));
    };
    // the lane's VEC levels of slice s of column t: one 16-byte load inside
    // the column, else element loads (past the column: its last level, not
    // stored)
    auto load = [&](int32_t t, int s, C* v) {
      const int k = kl[s];
      if (EXACT && s < NS - 1) {
        // EXACT: 16 lanes and NS = ceil(L / (16 VEC)), so every slice but the
        // last lies inside the column; its address is the first slice's plus
        // a constant (an immediate offset of the load)
        const S* p0 = addr(t, kb) + 16 * VEC * s;
        if constexpr (VEC == 1) {
          v[0] = ld1(p0);
        } else {
          const VT x = *reinterpret_cast<const VT*>(p0);
          v[0] = x.x;
          v[1] = x.y;
        }
      } else if (VEC == 1 || k + VEC <= L) {
        if constexpr (VEC == 1) {
          v[0] = ld1(addr(t, k < L ? k : L - 1));
        } else {
          const VT x = *reinterpret_cast<const VT*>(addr(t, k));
          v[0] = x.x;
          v[1] = x.y;
        }
      } else {
#pragma unroll
        for (int c = 0; c < VEC; ++c) v[c] = ld1(addr(t, k + c < L ? k + c : L - 1));
      }
    };
    C acc[NS][VEC];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int c = 0; c < VEC; ++c) acc[s][c] = 0;
    int32_t tn[EB] = {h2.x, h2.y};
    C wn[EB] = {hw2.x, hw2.y};
    for (int64_t e = e0; e < e1; e += EB) {
      int32_t t[EB];
      C wq[EB];
#pragma unroll
      for (int q = 0; q < EB; ++q) {
        t[q] = tn[q];
        wq[q] = wn[q];
      }
      C v[EB][NS][VEC];
#pragma unroll
      for (int q = 0; q < EB; ++q)
        if (e + q < e1) {
#pragma unroll
          for (int s = 0; s < NS; ++s) load(t[q], s, v[q][s]);
        }
      if (e + EB < e1) {
#pragma unroll
        for (int q = 0; q < EB; ++q) {
          const int64_t eq = e + EB + q < e1 ? e + EB + q : e1 - 1;
          tn[q] = tt[eq];
          wn[q] = w[eq];
        }
      }
#pragma unroll
      for (int q = 0; q < EB; ++q)
        if (e + q < e1) {
#pragma unroll
          for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int c = 0; c < VEC; ++c) acc[s][c] = fma(wq[q], v[q][s][c], acc[s][c]);
        }
    }
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int c = 0; c < VEC; ++c) {
        const int k = kl[s] + c;
        if constexpr (STG) {
          if (act && k < L) st1<false>(sb + j * L + k, acc[s][c]);
        } else {
          if (k < L) st1<false>(o + k, acc[s][c]);
        }
      }
  }
  if constexpr (STG) {
    __syncthreads();
    const int cnt = (V - nw0 < G ? (int)(V - nw0) : G) * L;   // elements of the wave's run
    S* __restrict__ ob = out + (size_t)nw0 * (size_t)L;
    // whole units of `unit` bytes (16, 8 or 4; both ends of every full run
    // and the output are aligned to it), then the elements past the last one
    auto copy = [&](auto tag) {
      using T = decltype(tag);
      const int nu = cnt * (int)sizeof(S) / (int)sizeof(T);
      T* __restrict__ d = reinterpret_cast<T*>(ob);
      const T* __restrict__ q = reinterpret_cast<const T*>(sb);
      for (int i = lane; i < nu; i += 64) d[i] = q[i];
      return nu * (int)sizeof(T) / (int)sizeof(S);
    };
    int done;
    if (unit == 16) done = copy(uint4());
    else if (unit == 8) done = copy(uint2());
    else if (unit == 4) done = copy(uint32_t());
    else done = copy(S());
    for (int i = done + lane; i < cnt; i += 64) ob[i] = sb[i];
  }
}

template <class S, int NS, int VEC>
hipError_t launch_remap_adj_ns(const int64_t* off, const int32_t* tt, const void* w, const int32_t* ht, const void* hw,
                               int64_t V, int64_t P, int nlev, int lanes, const S* src, S* dst, hipStream_t st) {
  const int G = 64 / lanes;
  constexpr int W = 4;
  const int64_t groups = (V + G - 1) / G;
  const int64_t nblocks = (groups + W - 1) / W;
  const bool o32 = (uint64_t)P * (uint64_t)nlev * sizeof(S) < (1ull << 32);
  const size_t lds = (size_t)W * G * nlev * sizeof(S);
  const bool stage = nlev <= lanes * VEC * NS && lds <= 32768;
  // the widest store unit that divides a full run's bytes and the output's alignment
  const uint64_t run = (uint64_t)G * nlev * sizeof(S), addr = (uint64_t)(uintptr_t)dst;
  int unit = (int)sizeof(S);
  for (int u : {16, 8, 4})
    if (u > unit && run % u == 0 && addr % u == 0) {
      unit = u;
      break;
    }
  const dim3 g((unsigned)nblocks), b(64 * W);
  // 16 lanes with exactly the slices the column needs: constant slice
  // offsets (4- and 2-byte data; measured 3 % and 8 % faster at O1280 x 137
  // <- F640, but 6 % slower for the FP64 16-byte loads)
  const bool exact = VEC == 1 && lanes == 16 && (nlev + 15) / 16 == NS;
#define RADJ_LAUNCH(O, T)                                                                                             \
  hipLaunchKernelGGL((k_remap_adj<S, NS, VEC, O, T>), g, b, T ? lds : 0, st, off, tt, w, ht, hw, src, dst, V, nlev, \
                     lanes, nblocks, unit)
  if (o32 && stage && exact) {
    hipLaunchKernelGGL((k_remap_adj<S, NS, VEC, true, true, true>), g, b, lds, st, off, tt, w, ht, hw, src, dst, V,
                       nlev, lanes, nblocks, unit);
  } else if (o32) {
    if (stage) RADJ_LAUNCH(true, true);
    else RADJ_LAUNCH(true, false);
  } else {
    if (stage) RADJ_LAUNCH(false, true);
    else RADJ_LAUNCH(false, false);
  }
#undef RADJ_LAUNCH
  return hipGetLastError();
}

// One node per 16 lanes (fewer columns of at most 16 levels: one lane per
// level); FP64 columns of more than 32 levels are read two levels per lane
// (16-byte loads; FP32 columns, only 4-byte aligned, measured slower that
// way).  Measured at O1280 x 137 <- F640.
template <class S>
hipError_t launch_remap_adj_t(const int64_t* off, const int32_t* tt, const void* w, const int32_t* ht, const void* hw,
                              int64_t V, int64_t P, int nlev, const void* in, void* out, hipStream_t st) {
  const int lanes = nlev <= 16 ? nlev : 16;
  const S* src = static_cast<const S*>(in);
  S* dst = static_cast<S*>(out);
  if constexpr (sizeof(S) == 8) {
    if (nlev > 32) {
      const int ns = (nlev + 2 * lanes - 1) / (2 * lanes);
      if (ns <= 2) return launch_remap_adj_ns<S, 2, 2>(off, tt, w, ht, hw, V, P, nlev, lanes, src, dst, st);
      if (ns == 3) return launch_remap_adj_ns<S, 3, 2>(off, tt, w, ht, hw, V, P, nlev, lanes, src, dst, st);
      return launch_remap_adj_ns<S, 5, 2>(off, tt, w, ht, hw, V, P, nlev, lanes, src, dst, st);
    }
  }
  const int ns = (nlev + lanes - 1) / lanes;
  if (ns <= 1) return launch_remap_adj_ns<S, 1, 1>(off, tt, w, ht, hw, V, P, nlev, lanes, src, dst, st);
  if (ns == 2) return launch_remap_adj_ns<S, 2, 1>(off, tt, w, ht, hw, V, P, nlev, lanes, src, dst, st);
  if (ns == 3) return launch_remap_adj_ns<S, 3, 1>(off, tt, w, ht, hw, V, P, nlev, lanes, src, dst, st);
  if (ns <= 5) return launch_remap_adj_ns<S, 5, 1>(off, tt, w, ht, hw, V, P, nlev, lanes, src, dst, st);
  return launch_remap_adj_ns<S, 9, 1>(off, tt, w, ht, hw, V, P, nlev, lanes, src, dst, st);
}

// out += base over n numbers, for divergence adjoints with an addend off the
// LDS tiles.
template <class S>
__global__ __launch_bounds__(256) void k_add(const S* __restrict__ base, S* __restrict__ out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    st1<false>(out + i, ld1(out + i) + ld1(base + i));
}

// ---- conservation: fixed-order FP64 sums of V_i div_ik --------------------------
//
// Workgroup b reduces nodes [b*chunk, (b+1)*chunk) for every level.  Wave w
// takes nodes w, w + W, ... of the chunk and reads each node's column in one
// go (lane = level within a 256-level block, four 64-level slices), so every
// column is fetched once; waves are then combined in order through LDS and a
// second pass sums the workgroup partials in order.  Deterministic by
// construction.

constexpr int kConsWaves = 4;
constexpr int kConsBlockLevels = 256;

template <class S, int NSL>
__global__ __launch_bounds__(64 * kConsWaves) void k_cons_partial(const S* __restrict__ div,
                                                                  const double* __restrict__ vol, int64_t V,
                                                                  int L, int64_t chunk, double* __restrict__ part) {
  // NSL: 64-level slices of a 256-level block that hold levels (the last
  // block of a short column needs fewer); nodes are read four at a time and
  // added in node order, so every sum keeps its order
  constexpr int kNodes = 4;
  __shared__ double red[kConsWaves][kConsBlockLevels][2];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t n0 = (int64_t)blockIdx.x * chunk;
  const int64_t n1 = n0 + chunk < V ? n0 + chunk : V;
  for (int kb = 0; kb < L; kb += kConsBlockLevels) {
    double s[4] = {0.0, 0.0, 0.0, 0.0}, ab[4] = {0.0, 0.0, 0.0, 0.0};
    bool in[4];
    int kc[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = kb + lane + 64 * r;
      in[r] = k < L;
      kc[r] = k < L ? k : L - 1;
    }
    // slices this block needs (all four unless it is the column's last)
    const int nsl = L - kb >= kConsBlockLevels ? 4 : NSL;
    int64_t i = n0 + wave;
    for (; i + (kNodes - 1) * kConsWaves < n1; i += kNodes * kConsWaves) {
      double p[kNodes][4];
#pragma unroll
      for (int q = 0; q < kNodes; ++q) {
        const int64_t nd = i + q * kConsWaves;
        const double v = vol[nd];
        const S* col = div + nd * (int64_t)L;
#pragma unroll
        for (int r = 0; r < 4; ++r) p[q][r] = r < nsl ? v * (double)ld1(col + kc[r]) : 0.0;
      }
#pragma unroll
      for (int q = 0; q < kNodes; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (r < nsl && in[r]) {
            s[r] += p[q][r];
            ab[r] += fabs(p[q][r]);
          }
    }
    for (; i < n1; i += kConsWaves) {
      const double v = vol[i];
      const S* col = div + i * (int64_t)L;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (r < nsl && in[r]) {
          const double p = v * (double)ld1(col + kc[r]);
          s[r] += p;
          ab[r] += fabs(p);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      red[wave][lane + 64 * r][0] = s[r];
      red[wave][lane + 64 * r][1] = ab[r];
    }
    __syncthreads();
    const int k = kb + (int)threadIdx.x;
    if (threadIdx.x < kConsBlockLevels && k < L) {
      double ts = red[0][threadIdx.x][0], ta = red[0][threadIdx.x][1];
      for (int w = 1; w < kConsWaves; ++w) {
        ts += red[w][threadIdx.x][0];
        ta += red[w][threadIdx.x][1];
      }
      part[((int64_t)blockIdx.x * L + k) * 2] = ts;
      part[((int64_t)blockIdx.x * L + k) * 2 + 1] = ta;
    }
    __syncthreads();
  }
}

// Columns of at most kConsFlatLevels levels: the field as one run of numbers.
// A workgroup's step covers kConsUnroll groups of g consecutive nodes; thread
// t owns numbers t * VEC ... of every group (16 bytes; FP64 32), and as g * L
// is a multiple of VEC these keep their levels and their node of the group
// from step to step, whatever the column's length.  So every lane has work
// (94 % at 137 levels, where 64-level slices fill 71 % of theirs, and 19
// levels 30 %), every load is 16 bytes, and the groups in flight on the GPU
// are one run of memory.  At the end the g sums of a level are combined in
// node order, in two stages.  ALN: the field is 16-byte aligned; else the
// same numbers are loaded one at a time.  Bound by memory reads; one
// workgroup of 8 waves per CU (BF16, with twice the numbers a load to widen, of
// 16 where its part of the field has eight groups or more), which keeps the
// partial sums few (512 workgroups: O640 x 19 FP32 27.4 us, 256: 25.9) and the
// groups short: of 16 waves FP32 and FP64 are slower throughout, the more so
// where a step of all groups is 256 bytes short of 64 KiB (60 and 120 levels:
// O640 x 120 FP32 204 us against 138, 165 in slices).  BF16 with 8 waves O100 x
// 137 12.6 -> 11.0 us, O640 x 137 92 -> 139.  Slices of 64 levels -> this:
// O1280 x 137 FP32 692 -> 633 us (5.7 TB/s), FP64 1.23 -> 1.12 ms, BF16 615 ->
// 337 us, O640 x 91 FP32 152 -> 111, x 19 110 -> 26, FP64 x 60 154 -> 131, O320
// x 60 FP64 41 -> 34.
constexpr int kConsFlatLevels = 1024;
constexpr int kConsFlatThreads = 1024;
constexpr int kConsFlatParts = 256;   // most workgroups: one per CU

template <class S>
constexpr int kConsVec = sizeof(S) == 8 ? 4 : 16 / (int)sizeof(S);
template <class S>
constexpr int kConsUnroll = sizeof(S) == 4 ? 4 : 2;

template <class S, bool ALN>
__global__ __launch_bounds__(kConsFlatThreads) void k_cons_flat(const S* __restrict__ div, const double* __restrict__ vol,
                                                                int64_t V, int L, int g, double* __restrict__ part) {
  constexpr int VEC = kConsVec<S>, U = kConsUnroll<S>;
  struct alignas(16) Pack {
    S x[VEC];
  };
  __shared__ double red[kConsFlatThreads * VEC];
  const int t = threadIdx.x;
  const int per = g * L / VEC;   // vectors of a group
  double s[VEC], ab[VEC];
#pragma unroll
  for (int c = 0; c < VEC; ++c) s[c] = ab[c] = 0.0;
  if (t < per) {
    // the group's nodes of the first and the last number, and how many numbers
    // belong to the first; columns shorter than a vector may span more
    const int na = t * VEC / L, nb = (t * VEC + VEC - 1) / L, m = (na + 1) * L - t * VEC;
    const bool two = L >= VEC;
    const int64_t step = (int64_t)gridDim.x * U * g;
    auto load = [&](int64_t n0, Pack& x, double& va, double& vb) {
      const S* p = div + n0 * (int64_t)L + t * VEC;
      if constexpr (ALN) {
        x = *reinterpret_cast<const Pack*>(p);
      } else {
#pragma unroll
        for (int c = 0; c < VEC; ++c) x.x[c] = p[c];
      }
      va = vol[n0 + na];
      vb = vol[n0 + nb];
    };
    auto add = [&](int64_t n0, const Pack& x, double va, double vb) {
#pragma unroll
      for (int c = 0; c < VEC; ++c) {
        double w = c < m ? va : vb;
        if (!two) w = vol[n0 + (t * VEC + c) / L];
        const double q = w * (double)ld1(&x.x[c]);
        s[c] += q;
        ab[c] += fabs(q);
      }
    };
    int64_t n = (int64_t)blockIdx.x * U * g;
    for (; n + U * g <= V; n += step) {
      Pack x[U];
      double va[U], vb[U];
#pragma unroll
      for (int u = 0; u < U; ++u) load(n + u * g, x[u], va[u], vb[u]);
#pragma unroll
      for (int u = 0; u < U; ++u) add(n + u * g, x[u], va[u], vb[u]);
    }
    // the last groups: the mesh ends at a multiple of VEC numbers, so a vector
    // whose last number is there is there
    for (int u = 0; u < U; ++u, n += g)
      if (n + nb < V) {
        Pack x;
        double va, vb;
        load(n, x, va, vb);
        add(n, x, va, vb);
      }
  }
  // red[j * L + k]: level k's sum over node j of the groups.  Thread (r, k)
  // adds nodes r, r + R, ..., thread k the R sums.
  int R = (int)blockDim.x / L;
  R = R < 32 ? R : 32;
  if (R > g) R = g;
  const int r = t / L, k = t - r * L;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    __syncthreads();
    if (t < per) {
#pragma unroll
      for (int c = 0; c < VEC; ++c) red[t * VEC + c] = which ? ab[c] : s[c];
    }
    __syncthreads();
    double a = 0.0;
    if (r < R)
      for (int j = r; j < g; j += R) a += red[j * L + k];
    __syncthreads();
    if (r < R) red[t] = a;
    __syncthreads();
    if (t < L) {
      a = red[t];
      for (int j = 1; j < R; ++j) a += red[j * L + t];
      part[((int64_t)blockIdx.x * L + t) * 2 + which] = a;
    }
  }
}

// One workgroup per level: thread t sums partials t, t + 256, ... in order,
// then a fixed binary tree combines the 256 thread sums.
__global__ __launch_bounds__(256) void k_cons_final(const double* __restrict__ part, int nparts, int L,
                                                    double* __restrict__ out_sum, double* __restrict__ out_abs) {
  __shared__ double red[256][2];
  const int k = blockIdx.x;
  double s = 0.0, a = 0.0;
  for (int p = threadIdx.x; p < nparts; p += 256) {
    s += part[((int64_t)p * L + k) * 2];
    a += part[((int64_t)p * L + k) * 2 + 1];
  }
  red[threadIdx.x][0] = s;
  red[threadIdx.x][1] = a;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      red[threadIdx.x][0] += red[threadIdx.x + w][0];
      red[threadIdx.x][1] += red[threadIdx.x + w][1];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out_sum[k] = red[0][0];
    out_abs[k] = red[0][1];
  }
}

// ---- dispatch ---------------------------------------------------------------

Args make_args(int op, const DevTables& t, const NodeOrder& ord, int64_t V, int nlev, const void* in, void* out,
               const Shape& sh) {
  Args a;
  a.order = ord.order;
  a.runs = ord.runs;
  a.nruns = ord.nruns;
  if (op == OP_LAP) {
    a.nbr = t.lap_nbr;
    a.coef = t.lap_w;
  } else {
    a.nbr = t.nbr8;
    a.coef = t.coef[op];
  }
  a.in = in;
  a.out = out;
  a.V = V;
  a.L = nlev;
  a.P = lanes_per_node(nlev, sh);
  a.npw = sh.nodes_per_wave;
  a.nt = nt_of(sh) ? 1 : 0;
  return a;
}

template <class S, int OP>
hipError_t launch_win(const Args& a, int U, dim3 g, dim3 b, int64_t nblocks, int remap, hipStream_t st) {
  switch (U) {
    case 1: hipLaunchKernelGGL((k_win<S, OP, 1>), g, b, 0, st, a, nblocks, remap); break;
    case 2: hipLaunchKernelGGL((k_win<S, OP, 2>), g, b, 0, st, a, nblocks, remap); break;
    default: hipLaunchKernelGGL((k_win<S, OP, 3>), g, b, 0, st, a, nblocks, remap); break;
  }
  return hipGetLastError();
}

template <class S, int OP>
hipError_t launch_u(const Args& a, int U, dim3 g, dim3 b, int64_t nblocks, int remap, hipStream_t st) {
  switch (U) {
    case 1: hipLaunchKernelGGL((k_op<S, OP, 1>), g, b, 0, st, a, nblocks, remap); break;
    case 2: hipLaunchKernelGGL((k_op<S, OP, 2>), g, b, 0, st, a, nblocks, remap); break;
    default: hipLaunchKernelGGL((k_op<S, OP, 3>), g, b, 0, st, a, nblocks, remap); break;
  }
  return hipGetLastError();
}

// Whether chunks of KL levels run in the short columns' body (U = 0).
template <class S, int OP>
constexpr bool short_body(int KL) {
  return kUseBlk<S, OP, 1> && KL <= 32;
}

template <class S, int OP>
hipError_t launch_tile_u(const TileArgs& a, int U, dim3 g, dim3 b, uint32_t lds, int64_t nblocks, int remap,
                         hipStream_t st) {
  if constexpr (kUseBlk<S, OP, 1>) {
    if (short_body<S, OP>(a.KL)) {
      const void* fn = reinterpret_cast<const void*>(&k_tile<S, OP, 0>);
      if ((int)b.x > kTileThreads<S, OP, 0>) b.x = kTileThreads<S, OP, 0>;
      if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
      }
      hipLaunchKernelGGL((k_tile<S, OP, 0>), g, b, lds, st, a, nblocks, remap);
      return hipGetLastError();
    }
  }
  const int maxt = U == 1 ? kTileThreads<S, OP, 1> : U == 2 ? kTileThreads<S, OP, 2> : kTileThreads<S, OP, 3>;
  if ((int)b.x > maxt) b.x = (unsigned)maxt;
  if (lds > 65536) {
    const void* fn = U == 1 ? reinterpret_cast<const void*>(&k_tile<S, OP, 1>)
                     : U == 2 ? reinterpret_cast<const void*>(&k_tile<S, OP, 2>)
                              : reinterpret_cast<const void*>(&k_tile<S, OP, 3>);
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  switch (U) {
    case 1: hipLaunchKernelGGL((k_tile<S, OP, 1>), g, b, lds, st, a, nblocks, remap); break;
    case 2: hipLaunchKernelGGL((k_tile<S, OP, 2>), g, b, lds, st, a, nblocks, remap); break;
    default: hipLaunchKernelGGL((k_tile<S, OP, 3>), g, b, lds, st, a, nblocks, remap); break;
  }
  return hipGetLastError();
}

template <class S, int OP>
hipError_t launch_tile2_u(const TileArgs& a, int U, dim3 g, dim3 b, uint32_t buf_bytes, uint32_t lds,
                          int64_t nblocks, int remap, int nprod, int P, hipStream_t st) {
  const void* fn = U == 1 ? reinterpret_cast<const void*>(&k_tile2<S, OP, 1>)
                   : U == 2 ? reinterpret_cast<const void*>(&k_tile2<S, OP, 2>)
                            : reinterpret_cast<const void*>(&k_tile2<S, OP, 3>);
  if (lds > 65536) {
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  switch (U) {
    case 1: hipLaunchKernelGGL((k_tile2<S, OP, 1>), g, b, lds, st, a, nblocks, remap, buf_bytes, nprod, P); break;
    case 2: hipLaunchKernelGGL((k_tile2<S, OP, 2>), g, b, lds, st, a, nblocks, remap, buf_bytes, nprod, P); break;
    default: hipLaunchKernelGGL((k_tile2<S, OP, 3>), g, b, lds, st, a, nblocks, remap, buf_bytes, nprod, P); break;
  }
  return hipGetLastError();
}

template <class S, int OP, int UMAX>
hipError_t launch_tb(const TileArgs& a, const BatchTile* tr, const int32_t* pre, int ntr, int32_t* ctr, int32_t claim,
                     uint32_t lds, int waves, int64_t grid, hipStream_t st) {
  const void* fn = reinterpret_cast<const void*>(&k_tile_batched<S, OP, UMAX>);
  if (lds > 65536) {
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  const dim3 g((unsigned)grid), b((unsigned)(64 * waves));
  hipLaunchKernelGGL((k_tile_batched<S, OP, UMAX>), g, b, lds, st, a, tr, pre, ntr, ctr, claim);
  return hipGetLastError();
}

template <class S, int OP>
const void* tb_fn_u(int umax) {
  return umax == 1   ? reinterpret_cast<const void*>(&k_tile_batched<S, OP, 1>)
         : umax == 2 ? reinterpret_cast<const void*>(&k_tile_batched<S, OP, 2>)
                     : reinterpret_cast<const void*>(&k_tile_batched<S, OP, 3>);
}

template <class S, int OP>
hipError_t launch_tb_u(const TileArgs& a, const BatchTile* tr, const int32_t* pre, int ntr, int32_t* ctr,
                       int32_t claim, uint32_t lds, int waves, int64_t grid, int umax, hipStream_t st) {
  switch (umax) {
    case 1: return launch_tb<S, OP, 1>(a, tr, pre, ntr, ctr, claim, lds, waves, grid, st);
    case 2: return launch_tb<S, OP, 2>(a, tr, pre, ntr, ctr, claim, lds, waves, grid, st);
    default: return launch_tb<S, OP, 3>(a, tr, pre, ntr, ctr, claim, lds, waves, grid, st);
  }
}

}  // namespace

// Launches of one element type, instantiated by a compilation of this file of
// their own per type (ATLAS_KERNEL_TYPE), so that the types build in parallel.

template <class S>
hipError_t launch_op_t(int op, const Args& a, int U, int64_t nblocks, bool window, const Shape& sh,
                       hipStream_t st) {
  const int64_t grid = sh.xcd_remap ? (nblocks + 7) / 8 * 8 : nblocks;
  const dim3 g((unsigned)grid), b((unsigned)(64 * sh.waves_per_block));
  if (window) {
    switch (op) {
      case OP_GRAD: return launch_win<S, OP_GRAD>(a, U, g, b, nblocks, sh.xcd_remap, st);
      case OP_DIV: return launch_win<S, OP_DIV>(a, U, g, b, nblocks, sh.xcd_remap, st);
      case OP_GRADT: return launch_win<S, OP_GRADT>(a, U, g, b, nblocks, sh.xcd_remap, st);
      case OP_DIVT: return launch_win<S, OP_DIVT>(a, U, g, b, nblocks, sh.xcd_remap, st);
      default: return hipErrorInvalidValue;
    }
  }
  switch (op) {
    case OP_GRAD: return launch_u<S, OP_GRAD>(a, U, g, b, nblocks, sh.xcd_remap, st);
    case OP_DIV: return launch_u<S, OP_DIV>(a, U, g, b, nblocks, sh.xcd_remap, st);
    case OP_GRADT: return launch_u<S, OP_GRADT>(a, U, g, b, nblocks, sh.xcd_remap, st);
    case OP_DIVT: return launch_u<S, OP_DIVT>(a, U, g, b, nblocks, sh.xcd_remap, st);
    case OP_LAP: return launch_u<S, OP_LAP>(a, U, g, b, nblocks, sh.xcd_remap, st);
    default: return hipErrorInvalidValue;
  }
}

template <class S>
hipError_t launch_tiles2_t(int op, const TileArgs& a, int U, uint32_t buf_bytes, uint32_t lds, int nprod, int ncons,
                           int per_cu, int num_cus, int P, const Shape& sh, hipStream_t st) {
  const int64_t nblocks = a.ntiles * a.nchunks;
  int64_t grid = (int64_t)per_cu * num_cus;
  if (grid > nblocks) grid = nblocks;
  const int remap = (sh.xcd_remap && grid % 8 == 0) ? 1 : 0;
  const dim3 g((unsigned)grid), b((unsigned)(64 * (nprod + ncons)));
  switch (op) {
    case OP_GRAD: return launch_tile2_u<S, OP_GRAD>(a, U, g, b, buf_bytes, lds, nblocks, remap, nprod, P, st);
    case OP_DIV: return launch_tile2_u<S, OP_DIV>(a, U, g, b, buf_bytes, lds, nblocks, remap, nprod, P, st);
    case OP_GRADT: return launch_tile2_u<S, OP_GRADT>(a, U, g, b, buf_bytes, lds, nblocks, remap, nprod, P, st);
    case OP_DIVT: return launch_tile2_u<S, OP_DIVT>(a, U, g, b, buf_bytes, lds, nblocks, remap, nprod, P, st);
    case OP_LAP: return launch_tile2_u<S, OP_LAP>(a, U, g, b, buf_bytes, lds, nblocks, remap, nprod, P, st);
    default: return hipErrorInvalidValue;
  }
}

template <class S>
hipError_t launch_tiles_t(int op, const TileArgs& a, int U, uint32_t lds, const Shape& sh, hipStream_t st) {
  const int64_t nblocks = a.ntiles * a.nchunks;   // scheduled tiles: a multiple of 8
  const int64_t grid = sh.xcd_remap == 1 ? (nblocks + 7) / 8 * 8 : nblocks;
  const dim3 g((unsigned)grid), b((unsigned)(64 * sh.waves_per_block));
  switch (op) {
    case OP_GRAD: return launch_tile_u<S, OP_GRAD>(a, U, g, b, lds, nblocks, sh.xcd_remap, st);
    case OP_DIV: return launch_tile_u<S, OP_DIV>(a, U, g, b, lds, nblocks, sh.xcd_remap, st);
    case OP_GRADT: return launch_tile_u<S, OP_GRADT>(a, U, g, b, lds, nblocks, sh.xcd_remap, st);
    case OP_DIVT:
      if (a.out2) return launch_tile_u<S, OP_DIVTA>(a, U, g, b, lds, nblocks, sh.xcd_remap, st);
      return launch_tile_u<S, OP_DIVT>(a, U, g, b, lds, nblocks, sh.xcd_remap, st);
    case OP_LAP: return launch_tile_u<S, OP_LAP>(a, U, g, b, lds, nblocks, sh.xcd_remap, st);
    case OP_GRADLAP: return launch_tile_u<S, OP_GRADLAP>(a, U, g, b, lds, nblocks, sh.xcd_remap, st);
    case OP_DIVCURL: return launch_tile_u<S, OP_DIVCURL>(a, U, g, b, lds, nblocks, sh.xcd_remap, st);
    default: return hipErrorInvalidValue;
  }
}

template <class S>
const void* tb_fn(int op, int umax) {
  switch (op) {
    case OP_GRAD: return tb_fn_u<S, OP_GRAD>(umax);
    case OP_DIV: return tb_fn_u<S, OP_DIV>(umax);
    case OP_GRADT: return tb_fn_u<S, OP_GRADT>(umax);
    case OP_DIVT: return tb_fn_u<S, OP_DIVT>(umax);
    case OP_DIVCURL: return tb_fn_u<S, OP_DIVCURL>(umax);
    default: return nullptr;
  }
}

template <class S>
hipError_t launch_tb_t(int op, const TileArgs& a, const BatchTile* tr, const int32_t* pre, int ntr, int32_t* ctr,
                       int32_t claim, uint32_t lds, int waves, int64_t grid, int umax, hipStream_t st) {
  switch (op) {
    case OP_GRAD: return launch_tb_u<S, OP_GRAD>(a, tr, pre, ntr, ctr, claim, lds, waves, grid, umax, st);
    case OP_DIV: return launch_tb_u<S, OP_DIV>(a, tr, pre, ntr, ctr, claim, lds, waves, grid, umax, st);
    case OP_GRADT: return launch_tb_u<S, OP_GRADT>(a, tr, pre, ntr, ctr, claim, lds, waves, grid, umax, st);
    case OP_DIVT: return launch_tb_u<S, OP_DIVT>(a, tr, pre, ntr, ctr, claim, lds, waves, grid, umax, st);
    case OP_DIVCURL: return launch_tb_u<S, OP_DIVCURL>(a, tr, pre, ntr, ctr, claim, lds, waves, grid, umax, st);
    default: return hipErrorInvalidValue;
  }
}

#define ATLAS_FIELD_LAUNCHES(KW, S)                                                                                   \
  KW template hipError_t launch_op_t<S>(int, const Args&, int, int64_t, bool, const Shape&, hipStream_t);             \
  KW template hipError_t launch_tiles_t<S>(int, const TileArgs&, int, uint32_t, const Shape&, hipStream_t);
#define ATLAS_PERSISTENT_LAUNCHES(KW, S)                                                                              \
  KW template hipError_t launch_tiles2_t<S>(int, const TileArgs&, int, uint32_t, uint32_t, int, int, int, int, int,   \
                                            const Shape&, hipStream_t);                                               \
  KW template const void* tb_fn<S>(int, int);                                                                         \
  KW template hipError_t launch_tb_t<S>(int, const TileArgs&, const BatchTile*, const int32_t*, int, int32_t*,        \
                                        int32_t, uint32_t, int, int64_t, int, hipStream_t);

#ifdef ATLAS_KERNEL_TYPE
ATLAS_FIELD_LAUNCHES(, ATLAS_KERNEL_TYPE)
#ifndef ATLAS_KERNEL_FIELD_ONLY
ATLAS_PERSISTENT_LAUNCHES(, ATLAS_KERNEL_TYPE)
#endif
#else
ATLAS_FIELD_LAUNCHES(extern, double)
ATLAS_FIELD_LAUNCHES(extern, float)
ATLAS_FIELD_LAUNCHES(extern, bf16_t)
ATLAS_PERSISTENT_LAUNCHES(extern, double)
ATLAS_PERSISTENT_LAUNCHES(extern, float)

bool uses_window(int op, int nlev, const Shape& sh) {
  return op != OP_LAP && nlev > 32 && sh.row_window != 2;
}

int lanes_per_node(int nlev, const Shape& sh) {
  if (nlev <= 32) return nlev;
  if (sh.lanes_per_node > 0) return sh.lanes_per_node;
  // best lane utilisation nlev / (P * ceil(nlev / P)); ties go to the wider P
  int best = 64;
  double bu = -1.0;
  for (int p : {64, 32, 16}) {
    const int nsl = (nlev + p - 1) / p;
    const double u = (double)nlev / (double)(p * nsl);
    if (u > bu + 1e-12) {
      bu = u;
      best = p;
    }
  }
  return best;
}

int slices_per_iter(int nlev, const Shape& sh) {
  const int P = lanes_per_node(nlev, sh);
  const int nsl = (nlev + P - 1) / P;
  int U = sh.slices_per_iter > 0 ? sh.slices_per_iter : 3;
  if (U > 3) U = 3;
  return U < nsl ? U : nsl;
}

int64_t blocks_for(int op, const NodeOrder& ord, int64_t V, int nlev, const Shape& sh) {
  if (uses_window(op, nlev, sh)) {
    const int64_t per_block = (int64_t)sh.waves_per_block * sh.nodes_per_wave;
    return (ord.nruns + per_block - 1) / per_block;
  }
  const int G = 64 / lanes_per_node(nlev, sh);
  const int64_t per_block = (int64_t)sh.waves_per_block * sh.nodes_per_wave * G;
  return (V + per_block - 1) / per_block;
}

hipError_t launch_op(int op, int dtype, const DevTables& t, const NodeOrder& ord, int64_t V, int nlev,
                     const void* in, void* out, const Shape& shape_in, hipStream_t stream) {
  Shape shape = shape_in;
  if (shape.waves_per_block > 4) shape.waves_per_block = 4;   // 8 applies to LDS tiles only
  if (op == OP_LAP && t.lap_stride != kLapStride) return hipErrorInvalidValue;
  const Args a = make_args(op, t, ord, V, nlev, in, out, shape);
  const bool window = uses_window(op, nlev, shape);
  const int U = window ? window_slices(nlev, shape) : slices_per_iter(nlev, shape);
  const int64_t nblocks = blocks_for(op, ord, V, nlev, shape);
  switch (dtype) {
    case DT_F64: return launch_op_t<double>(kernel_op(op), a, U, nblocks, window, shape, stream);
    case DT_F32: return launch_op_t<float>(kernel_op(op), a, U, nblocks, window, shape, stream);
    case DT_BF16: return launch_op_t<bf16_t>(kernel_op(op), a, U, nblocks, window, shape, stream);
    default: return hipErrorInvalidValue;
  }
}

namespace {

Shape resolve_path(int op, int dtype, int nlev, int64_t V, const Shape& sh) {
  Shape e = sh;
  if (e.lds_tiles != 0) return e;
  if (nlev <= 32) {
    // Columns of at most 32 levels: the gather gives a wave 64 / nlev nodes
    // and reads each neighbour's column from L2, in pieces of less than a
    // cache line; the tiles read every column once, in whole tiles.  19
    // levels, gather -> tiles: O640 FP32 gradient 253 -> 100 us, divergence
    // 303 -> 107, Laplacian 443 -> 109, divergence and curl 603 -> 146; FP64
    // divergence 426 -> 186, BF16 Laplacian 373 -> 88; 32 levels FP32
    // Laplacian 639 -> 143.  Below eight levels the tables, not the columns,
    // are most of the traffic, and a tile's are larger (O640 x 2 FP32
    // divergence 33 -> 40 us, O320 x 4 FP64 Laplacian 30 -> 36); at eight the
    // two are level for the slowest operators (O320 BF16 divergence 17.8 ->
    // 16.1) and the others gain (FP32 Laplacian 34 -> 26).  In small fields a tile's
    // start (tables, then data, then arithmetic: 5-10 us) shows: BF16
    // divergence at 10 levels 7.3 -> 10.2 us at O160, 10.2 -> 11.2 at O200
    // (1.7 million values), 23.3 -> 17.3 at O320 (4.2 million).  A shape that sets a parameter of
    // the gather's keeps it.
    const Shape def;
    if (nlev < kShortTileLevels || V * nlev < kShortTileValues || e.row_window || e.lanes_per_node ||
        e.band_rows || e.run_nodes || e.slices_per_iter || e.nodes_per_wave != def.nodes_per_wave ||
        e.waves_per_block != def.waves_per_block) {
      e.lds_tiles = 2;
      return e;
    }
    e.short_tiles = true;
  }
  // Measured defaults at O1280 x 137 (rows: mode, KiB, tile rows, computing
  // and copying waves of the persistent form): scalar-input 1-ring operators,
  // vector-input ones, the two-ring Laplacian.
  // (mode, KiB, tile rows, computing waves, copying waves, lanes per node,
  // waves per workgroup of the one-tile form)
  struct Def { int mode, kb, rows, cw, pw, lanes, wpb; };
  const bool vec_in = kernel_op(op) == OP_DIV || kernel_op(op) == OP_GRADT || kernel_op(op) == OP_DIVCURL;
  const bool lap = op == OP_LAP || op == OP_GRADLAP;   // the fused form takes the Laplacian's
  // the divergence paired with the curl or the gradient adjoint in one pass
  // (its records hold two coefficient rows)
  const bool dual = kernel_op(op) == OP_DIVCURL;
  Def d;
  if (dtype == DT_F32)
    d = lap    ? Def{3, 80, 4, 0, 0, 0, 8}
        : dual ? Def{3, 80, 4, 0, 0, 0, 16}
        : vec_in ? Def{3, 64, 4, 0, 0, 0, 8}
                 : Def{3, 40, 4, 0, 0, 0, 8};
  else if (dtype == DT_BF16)
    d = lap ? Def{3, 53, 4, 0, 0, 0, 8} : vec_in ? Def{3, 80, 4, 0, 0, 0, 16} : Def{3, 64, 4, 0, 0, 0, 16};
  else
    d = lap    ? Def{3, 160, op == OP_LAP && V * nlev >= kTallTileValues ? 6 : 4, 0, 0, 0, 16}
        : dual ? Def{3, 160, 4, 0, 0, 0, 8}
        : vec_in ? Def{3, 80, 4, 0, 0, 0, 8}
                 : Def{3, 64, 3, 0, 0, 0, 8};
  // (FP64 Laplacian: tiles of six rows, 1.24 ms at O640 x 137, against 1.30
  // with four, O160 x 91 64.6 us against 66.2; but on small fields, where they
  // leave CUs without a tile, 10.7 against 9.5 at O32 x 91, 40.6 against 39.5 at
  // O100 x 137)
  e.lds_tiles = d.mode;
  if (d.mode == 2) return e;
  if (!e.tile_kb) e.tile_kb = d.kb;
  if (!e.band_rows) e.band_rows = d.rows;
  if (!e.tile_waves) e.tile_waves = d.cw;
  if (!e.producer_waves) e.producer_waves = d.pw;
  if (!e.lanes_per_node) e.lanes_per_node = d.lanes;
  if (d.wpb && e.waves_per_block == Shape().waves_per_block) e.waves_per_block = d.wpb;
  // FP64 one-pass gradient and Laplacian: one slice per step fits 16 waves
  // in 128 registers (7.1 ms against 7.7 ms with two slices and 8 waves)
  if (op == OP_GRADLAP && dtype == DT_F64 && !e.slices_per_iter) e.slices_per_iter = 1;
  return e;
}

}  // namespace

// Order of the work over the XCDs, where the caller does not fix it.  The
// one-tile form goes around one band of rows at a time, so the tiles in
// flight on the whole GPU lie side by side along a few rows and their reads
// and writes fall into few DRAM pages; halo rows come from the 256 MiB cache
// behind the L2s when they have left an XCD's own.  A contiguous eighth of
// the order per XCD keeps halo rows in its L2 but has eight times as many
// rows open: a plain kernel reading 1 and writing 2 bytes over rows visited
// that way drops from 6.3 to 5.1 TB/s.  O640 x 137 FP32, eighths of 8-band
// sweeps -> plain order of single bands: gradient 614 -> 552 us, divergence
// 647 -> 602, Laplacian 657 -> 630, gradient and Laplacian 994 -> 936,
// divergence and curl 859 -> 806; O1280 gradient 2.41 -> 2.22 ms; BF16 and
// FP64 4-13 %.
// Within a band each XCD takes an eighth of the longitude (schedule_tiles),
// so tiles side by side share their halo columns in one L2, where that halo
// is wide: two columns each side (the two-ring operators: FP32 Laplacian 580
// -> 553 us, gradient and Laplacian 915 -> 872) or two
// components (divergence 599 -> 571 us FP32, 1.35 -> 1.31 ms FP64; BF16 376 ->
// 363, Laplacian 441 -> 429, gradient 329 -> 319).  The FP32 and FP64
// scalar-input 1-ring operators gain by it while the GPU's caches still hold
// much of the field (FP64 gradient O100 x 200 48.3 -> 39.1 us, O320 x 200, 0.67
// GB, 439 -> 429; FP32 O200 x 97 40.7 -> 35.6, O640 x 91, 0.6 GB, 371 -> 362) and
// lose on larger ones (FP64 O640 x 60, 0.8 GB, 474 -> 491, x 137 1.10 -> 1.14
// ms; FP32 O1280 x 137 2.18 -> 2.26): those keep the plain order.
// The FP64 one-pass gradient and Laplacian, one 160 KiB tile per CU, keeps the
// eighths and 8-band sweeps: O640 x 137 1837 us against 1931 with the schedule
// and 1984 in plain order (all with its blocks of two nodes; x 60 827 against
// 837 and 924).
// Shapes that name the form and no order take the same; a sweep of several
// bands (run_nodes) in plain order or by the schedule only changes where the
// tiles are cut, and is ahead of eighths of it too (64 KiB tiles of four rows,
// 8 waves, sweeps of eight: gradient 589 us against 629, divergence 588
// against 643; single bands 565 and 578).
// The other paths, without a tile's reuse of its own halo, keep the eighths.
Shape resolve_shape(int op, int dtype, int nlev, int64_t V, const Shape& sh) {
  Shape e = resolve_path(op, dtype, nlev, V, sh);
  const bool one_tile = e.lds_tiles == 3 && uses_tiles(op, dtype, nlev, e);
  if (one_tile && !e.run_nodes && (sh.lds_tiles == 0 || e.xcd_remap < 0))
    e.run_nodes = op == OP_GRADLAP && dtype == DT_F64 ? kDefaultTileSweep : 1;
  if (e.xcd_remap >= 0) return e;
  const int k = kernel_op(op);
  if (!one_tile) e.xcd_remap = 1;
  else if (op == OP_GRADLAP && dtype == DT_F64) e.xcd_remap = 1;
  else if (dtype == DT_BF16 || (k != OP_GRAD && k != OP_DIVT)) e.xcd_remap = kXcdSchedule;
  else e.xcd_remap = V * nlev * (dtype == DT_F64 ? 8 : 4) <= kScheduleBytes ? kXcdSchedule : 0;
  return e;
}

bool uses_tiles(int op, int dtype, int nlev, const Shape& sh) {
  (void)op;
  if (nlev <= 32 && !sh.short_tiles) return false;
  if (dtype == DT_BF16) return sh.lds_tiles == 3;   // BF16: one-tile form only
  return (dtype == DT_F32 || dtype == DT_F64) && (sh.lds_tiles == 1 || sh.lds_tiles == 3);
}

TileGeom tile_geom(int op, int dtype, int nlev, const Shape& sh) {
  TileGeom g;
  const int64_t es = dtype == DT_F64 ? 8 : dtype == DT_BF16 ? 2 : 4;
  const int64_t cin = (kernel_op(op) == OP_DIV || kernel_op(op) == OP_GRADT || kernel_op(op) == OP_DIVCURL) ? 2 : 1;
  g.ring = (op == OP_LAP || op == OP_GRADLAP) ? 2 : 1;
  g.row_bytes = tile_record_bytes(op, dtype);
  g.block = tile_block_nodes(op, dtype);
  g.budget = (int64_t)(sh.tile_kb > 0 ? sh.tile_kb : kDefaultTileKB) * 1024;
  // the read-past tail behind a workgroup's buffers (one, or two for the
  // persistent form) must not cost a workgroup per CU: with n = LDS / (nb
  // budget) workgroups per CU, the budget leaves room for the largest tail
  // (3 x 64 levels)
  if (sh.lds_tiles == 3 || sh.lds_tiles == 1) {
    const int64_t nb = sh.lds_tiles == 1 ? 2 : 1;
    const int64_t n = (int64_t)kLdsPerCu / (nb * g.budget) > 1 ? (int64_t)kLdsPerCu / (nb * g.budget) : 1;
    const int64_t cap = (((int64_t)kLdsPerCu / n - 3 * 64 * cin * es) / nb) & ~(int64_t)15;
    if (g.budget > cap) g.budget = cap;
  }
  if (dtype == DT_BF16) {
    // whole columns only; per column the data, its offset-table entry and up
    // to 8 bytes of alignment padding, plus 16 bytes of table alignment
    g.budget -= 16;
    const int64_t stencil = g.ring == 2 ? kLapStride : 8;
    g.col_bytes = (int64_t)nlev * cin * es + kBf16ColExtra;
    if (stencil * g.col_bytes + (stencil / 2) * g.row_bytes > g.budget) return g;   // KL = 0: no tiles
    g.KL = nlev;
    g.nchunks = 1;
    return g;
  }
  // Column chunk: whole columns if a tile of `want` columns (and half as many
  // nodes' table rows) fits, else the largest equal chunks that do; if even
  // that fails, fall back to the minimum of one node's stencil.
  const int64_t stencil = g.ring == 2 ? kLapStride : 8;
  const int64_t wants[2] = {g.ring == 2 ? 96 : 48, stencil};
  g.KL = 0;
  if (sh.tile_levels > 0) {
    // asked-for chunk, if one node's stencil fits with it
    const int64_t k = sh.tile_levels < nlev ? sh.tile_levels : nlev;
    if (stencil * k * cin * es + (stencil / 2) * g.row_bytes <= g.budget) {
      g.KL = (int)k;
      g.nchunks = (nlev + g.KL - 1) / g.KL;
      g.col_bytes = (int64_t)g.KL * cin * es;
      return g;
    }
  }
  for (int64_t want : wants) {
    const int64_t per_col = (g.budget - (want / 2) * g.row_bytes) / want;
    const int64_t kl = per_col / (cin * es);
    if (kl < 1) continue;
    // equal chunks, rounded up to whole 16-byte units when that still fits
    const int64_t nch = (nlev + kl - 1) / kl;
    const int64_t m = 16 / (cin * es) > 1 ? 16 / (cin * es) : 1;
    int64_t k = (nlev + nch - 1) / nch;
    if ((k + m - 1) / m * m <= kl) k = (k + m - 1) / m * m;
    g.KL = (int)(k < nlev ? k : nlev);
    break;
  }
  if (g.KL < 1) return g;   // no tile geometry fits the budget
  g.nchunks = (nlev + g.KL - 1) / g.KL;
  g.col_bytes = (int64_t)g.KL * cin * es;
  return g;
}

int tile_slices(int KL, const Shape& sh) {
  // whole 64-level slices of a chunk: a remainder of 1..32 levels goes to the
  // packed tail pass
  const int rem = KL & 63;
  const int kmain = rem != 0 && rem <= 32 ? KL - rem : KL;
  const int nsl = (kmain + 63) / 64 > 0 ? (kmain + 63) / 64 : 1;
  const int u = sh.slices_per_iter > 0 ? sh.slices_per_iter : 3;
  return u < nsl ? u : nsl;
}

int64_t tile_tail_bytes(int op, int dtype, int KL, int nlev, int U, TileForm form) {
  const int64_t es = dtype == DT_F64 ? 8 : dtype == DT_BF16 ? 2 : 4;
  const int64_t cin = (kernel_op(op) == OP_DIV || kernel_op(op) == OP_GRADT || kernel_op(op) == OP_DIVCURL) ? 2 : 1;
  // a step reads 64 levels a slice (U slices, blocks at most kBlkU, other nodes
  // down to one) from level 0 on, without the levels of the packed pass of the
  // forms that have one
  const int64_t step = 64 * (int64_t)tile_step_slices(op, dtype, U, form);
  auto past = [&](int64_t k) -> int64_t {
    const int64_t rem = k & 63, kmain = form != TileForm::kPersistent && rem != 0 && rem <= 32 ? k - rem : k;
    const int64_t end = (kmain + step - 1) / step * step;
    return end > k ? end - k : 0;
  };
  const int64_t last = nlev - (int64_t)((nlev - 1) / KL) * KL;
  const int64_t t0 = past(KL), t1 = past(last);
  return (t0 > t1 ? t0 : t1) * cin * es;
}

// f(element type, kernel operator's tag): the block constants of an operator.
namespace {
template <class F>
int with_block_op(int op, int dtype, F&& f) {
  auto pick = [&](auto tag) -> int {
    switch (kernel_op(op)) {
      case OP_LAP: return f(tag, std::integral_constant<int, OP_LAP>());
      case OP_GRADLAP: return f(tag, std::integral_constant<int, OP_GRADLAP>());
      case OP_DIVCURL: return f(tag, std::integral_constant<int, OP_DIVCURL>());
      case OP_DIV:
      case OP_GRADT: return f(tag, std::integral_constant<int, OP_DIV>());
      default: return f(tag, std::integral_constant<int, OP_GRAD>());
    }
  };
  return dtype == DT_F64 ? pick(double()) : dtype == DT_F32 ? pick(float()) : pick(bf16_t());
}
}  // namespace

int tile_step_slices(int op, int dtype, int U, TileForm form) {
  if (form == TileForm::kPersistent) return U;
  return with_block_op(op, dtype, [&](auto tag, auto k) -> int {
    using S = decltype(tag);
    constexpr int OP = decltype(k)::value;
    bool blocks = U > 1 ? kUseBlk<S, OP, 2> : kUseBlk<S, OP, 1>;
    if (form == TileForm::kBatched)
      blocks &= U == 1 ? kBatchedBlk<S, OP, 1> : U == 2 ? kBatchedBlk<S, OP, 2> : kBatchedBlk<S, OP, 3>;
    return blocks && U > kBlkU<S, OP> ? kBlkU<S, OP> : U;
  });
}

int tile_block_nodes(int op, int dtype) {
  return with_block_op(op, dtype, [](auto tag, auto k) -> int { return kBlkN<decltype(tag), decltype(k)::value>; });
}

int64_t tile_record_bytes(int op, int dtype) {
  switch (op * 2 + (dtype == DT_F64 ? 1 : 0)) {
    case OP_LAP * 2: return TileRec<float, OP_LAP>::kBytes;
    case OP_LAP * 2 + 1: return TileRec<double, OP_LAP>::kBytes;
    case OP_GRADLAP * 2: return TileRec<float, OP_GRADLAP>::kBytes;
    case OP_GRADLAP * 2 + 1: return TileRec<double, OP_GRADLAP>::kBytes;
    case OP_DIVCURL * 2:
    case OP_DIVGRADT * 2: return TileRec<float, OP_DIVCURL>::kBytes;
    case OP_DIVCURL * 2 + 1:
    case OP_DIVGRADT * 2 + 1: return TileRec<double, OP_DIVCURL>::kBytes;
    default: return dtype == DT_F64 ? TileRec<double, OP_GRAD>::kBytes : TileRec<float, OP_GRAD>::kBytes;
  }
}

hipError_t pack_tile_records(int op, int dtype, const DevTables& t, const int32_t* order, const uint16_t* loc,
                             int64_t V, void* rec, hipStream_t stream) {
  const int64_t n = V * (tile_record_bytes(op, dtype) / 4);
  const dim3 g((unsigned)((n + 255) / 256)), b(256);
  const bool dual = op == OP_DIVCURL || op == OP_DIVGRADT;   // divergence rows, then the second operator's
  const void* coef = (op == OP_LAP || op == OP_GRADLAP) ? t.lap_w : dual ? t.coef[OP_DIV] : t.coef[op];
  const void* coef2 = op == OP_GRADLAP ? t.coef[OP_GRAD]
                      : op == OP_DIVCURL ? t.coef[OP_CURL]
                      : op == OP_DIVGRADT ? t.coef[OP_GRADT]
                                          : nullptr;
  uint32_t* r = static_cast<uint32_t*>(rec);
  const bool f64 = dtype == DT_F64;
  if (op == OP_LAP) {
    if (f64) hipLaunchKernelGGL((k_pack_records<double, OP_LAP>), g, b, 0, stream, order, coef, coef2, loc, V, r);
    else hipLaunchKernelGGL((k_pack_records<float, OP_LAP>), g, b, 0, stream, order, coef, coef2, loc, V, r);
  } else if (op == OP_GRADLAP) {
    if (f64) hipLaunchKernelGGL((k_pack_records<double, OP_GRADLAP>), g, b, 0, stream, order, coef, coef2, loc, V, r);
    else hipLaunchKernelGGL((k_pack_records<float, OP_GRADLAP>), g, b, 0, stream, order, coef, coef2, loc, V, r);
  } else if (dual) {
    if (f64) hipLaunchKernelGGL((k_pack_records<double, OP_DIVCURL>), g, b, 0, stream, order, coef, coef2, loc, V, r);
    else hipLaunchKernelGGL((k_pack_records<float, OP_DIVCURL>), g, b, 0, stream, order, coef, coef2, loc, V, r);
  } else {
    if (f64) hipLaunchKernelGGL((k_pack_records<double, OP_GRAD>), g, b, 0, stream, order, coef, coef2, loc, V, r);
    else hipLaunchKernelGGL((k_pack_records<float, OP_GRAD>), g, b, 0, stream, order, coef, coef2, loc, V, r);
  }
  return hipGetLastError();
}

hipError_t launch_tiles(int op, int dtype, const DevTiles& dt, const void* rec, int nlev, const void* in,
                        void* out, const Shape& shape, int num_cus, hipStream_t stream, void* out2) {
  // the tiling's LDS footprint must be the one the kernel lays out
  const bool bf = dtype == DT_BF16;
  const int64_t es = dtype == DT_F64 ? 8 : bf ? 2 : 4;
  const int64_t cin = (kernel_op(op) == OP_DIV || kernel_op(op) == OP_GRADT || kernel_op(op) == OP_DIVCURL) ? 2 : 1;
  const int64_t row = tile_record_bytes(op, dtype);
  const int64_t colb = (int64_t)dt.KL * cin * es + (bf ? kBf16ColExtra : 0);
  const int U3 = tile_slices(dt.KL, shape);
  // one tile per workgroup: lanes past a column's last level read into a
  // tail behind the buffer
  const uint32_t lds_need =
      dt.lds_bytes + (bf ? 16u : 0u) +
      (shape.lds_tiles == 3 && dt.KL >= 1 ? (uint32_t)tile_tail_bytes(op, dtype, dt.KL, nlev, U3) : 0u);
  if (dt.KL < 1 || dt.KL > nlev || dt.nchunks != (nlev + dt.KL - 1) / dt.KL || lds_need > kLdsPerCu ||
      dt.col_bytes != colb || dt.row_bytes != row || (bf && (dt.KL != nlev || shape.lds_tiles != 3)))
    return hipErrorInvalidValue;
  TileArgs a;
  a.info = dt.info;
  a.segs = dt.segs;
  a.rec = static_cast<const char*>(rec);
  a.in = in;
  a.out = out;
  a.out2 = out2;
  const bool two = op == OP_GRADLAP || kernel_op(op) == OP_DIVCURL;
  const bool second = two || (kernel_op(op) == OP_DIVT && out2);   // with an addend
  if (second != (out2 != nullptr) || (second && shape.lds_tiles != 3))
    return hipErrorInvalidValue;   // the one-pass forms: one-tile workgroups, both outputs
  a.ntiles = dt.ntiles;
  if (shape.lds_tiles == 3 && shape.xcd_remap == kXcdSchedule) {
    a.info = dt.sched;
    a.ntiles = dt.nsched;
  }
  a.L = nlev;
  a.KL = dt.KL;
  a.nchunks = dt.nchunks;
  a.nt = nt_of(shape) ? 1 : 0;
  if (shape.lds_tiles == 3) {
    const int U = U3;
    switch (dtype) {
      case DT_F64: return launch_tiles_t<double>(kernel_op(op), a, U, lds_need, shape, stream);
      case DT_F32: return launch_tiles_t<float>(kernel_op(op), a, U, lds_need, shape, stream);
      case DT_BF16: return launch_tiles_t<bf16_t>(kernel_op(op), a, U, lds_need, shape, stream);
      default: return hipErrorInvalidValue;
    }
  }
  // persistent double-buffered form
  const int nprod = shape.producer_waves > 0 ? shape.producer_waves : 2;
  const int ncons = shape.tile_waves > 0 ? shape.tile_waves : 6;
  if (nprod + ncons > (dtype == DT_F64 ? 8 : 16) || (nprod & (nprod - 1))) return hipErrorInvalidValue;
  const uint32_t buf_bytes = (dt.lds_bytes + 15u) & ~15u;
  const int P = lanes_per_node(dt.KL, shape);
  const int nsl = (dt.KL + P - 1) / P;
  int U = shape.slices_per_iter > 0 ? shape.slices_per_iter : 3;
  if (U > nsl) U = nsl;
  // whole-wave nodes read past a column's last level, as in the one-tile form
  const uint32_t lds = 2 * buf_bytes + (P == 64 ? (uint32_t)tile_tail_bytes(op, dtype, dt.KL, nlev, U, TileForm::kPersistent) : 0u);
  // workgroups per CU as asked, as far as their two buffers fit the CU's LDS
  int per_cu = shape.tile_wgs_per_cu > 0 ? shape.tile_wgs_per_cu : 1;
  while (per_cu > 1 && (uint64_t)lds * per_cu > kLdsPerCu) --per_cu;
  if (lds > kLdsPerCu) return hipErrorInvalidValue;
  switch (dtype) {
    case DT_F64:
      return launch_tiles2_t<double>(kernel_op(op), a, U, buf_bytes, lds, nprod, ncons, per_cu, num_cus, P, shape,
                                     stream);
    case DT_F32:
      return launch_tiles2_t<float>(kernel_op(op), a, U, buf_bytes, lds, nprod, ncons, per_cu, num_cus, P, shape,
                                    stream);
    default: return hipErrorInvalidValue;
  }
}

void kernel_label(int op, int dtype, int nlev, const Shape& sh, char* buf, int len) {
  const char* ty = dtype == DT_F64 ? "double" : dtype == DT_F32 ? "float" : "unsigned short";
  const char* name = nullptr;
  int U = 1;
  if (uses_tiles(op, dtype, nlev, sh)) {
    const TileGeom g = tile_geom(op, dtype, nlev, sh);
    if (g.KL > 0) {
      if (sh.lds_tiles == 3) {
        const bool is_short = with_block_op(op, dtype, [&](auto tag, auto k) -> int {
          return short_body<decltype(tag), decltype(k)::value>(g.KL);
        });
        U = is_short ? 0 : tile_slices(g.KL, sh);
      } else {
        const int P = lanes_per_node(g.KL, sh);
        const int nsl = (g.KL + P - 1) / P;
        U = sh.slices_per_iter > 0 ? sh.slices_per_iter : 3;
        if (U > nsl) U = nsl;
      }
      name = sh.lds_tiles == 3 ? "k_tile" : "k_tile2";
    }
  }
  if (!name) {
    if (op != OP_LAP && uses_window(op, nlev, sh)) {
      name = "k_win";
      U = window_slices(nlev, sh);
    } else {
      name = "k_op";
      U = slices_per_iter(nlev, sh);
    }
  }
  snprintf(buf, (size_t)len, "%s<%s, %d, %d>", name, ty, kernel_op(op), U);
}

int window_slices(int nlev, const Shape& sh) {
  const int nsl = (nlev + 63) / 64;
  int U = sh.slices_per_iter > 0 ? sh.slices_per_iter : 3;
  if (U > 3) U = 3;
  return U < nsl ? U : nsl;
}

hipError_t launch_add(int dtype, int64_t n, const void* base, void* out, hipStream_t st) {
  const dim3 g((unsigned)std::min<int64_t>((n + 255) / 256, 65536)), b(256);
  if (dtype == DT_F64)
    hipLaunchKernelGGL((k_add<double>), g, b, 0, st, static_cast<const double*>(base), static_cast<double*>(out), n);
  else if (dtype == DT_F32)
    hipLaunchKernelGGL((k_add<float>), g, b, 0, st, static_cast<const float*>(base), static_cast<float*>(out), n);
  else if (dtype == DT_BF16)
    hipLaunchKernelGGL((k_add<bf16_t>), g, b, 0, st, static_cast<const bf16_t*>(base), static_cast<bf16_t*>(out), n);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

int conservation_parts(int64_t V, int nlev) {
  (void)nlev;
  const int64_t p = (V + 63) / 64;
  return (int)(p < 4096 ? p : 4096);
}

hipError_t launch_conservation(int dtype, const double* vol, int64_t V, int nlev, const void* div, double* scratch,
                               double* out_sum, double* out_abs, hipStream_t stream) {
  int parts = conservation_parts(V, nlev);
  const int64_t es = dtype == DT_F64 ? 8 : dtype == DT_F32 ? 4 : 2;
  const int64_t vec = es == 2 ? 8 : 4;
  if (nlev <= kConsFlatLevels && V % vec == 0) {
    if (parts > kConsFlatParts) parts = kConsFlatParts;
    // nodes of a group: as many as 8 waves hold (BF16 16 where the part has
    // eight such groups), no more than a workgroup's part, in steps that keep
    // whole vectors
    int64_t q = vec;
    while (q > 1 && (q / 2) * nlev % vec == 0) q /= 2;
    const int64_t part = ((V + parts - 1) / parts + q - 1) / q * q;
    auto fit = [&](int64_t threads) {
      int64_t n = threads * vec / nlev / q * q;
      if (n < q) n = q;
      return n < part ? n : part;
    };
    int64_t gn = fit(kConsFlatThreads);
    if (es != 2 || part < 8 * gn) gn = fit(kConsFlatThreads / 2);
    const int64_t thr = (gn * nlev / vec + 63) / 64 * 64;
    const int threads = (int)(thr > (nlev + 63) / 64 * 64 ? thr : (nlev + 63) / 64 * 64);
    const bool aln = ((uintptr_t)div & 15u) == 0;
#define ATLAS_CONS(DT, S)                                                                                           \
  case DT:                                                                                                          \
    if (aln)                                                                                                        \
      hipLaunchKernelGGL((k_cons_flat<S, true>), dim3(parts), dim3(threads), 0, stream, static_cast<const S*>(div), \
                         vol, V, nlev, (int)gn, scratch);                                                           \
    else                                                                                                            \
      hipLaunchKernelGGL((k_cons_flat<S, false>), dim3(parts), dim3(threads), 0, stream,                            \
                         static_cast<const S*>(div), vol, V, nlev, (int)gn, scratch);                               \
    break;
    switch (dtype) {
      ATLAS_CONS(DT_F64, double) ATLAS_CONS(DT_F32, float) ATLAS_CONS(DT_BF16, bf16_t)
#undef ATLAS_CONS
      default: return hipErrorInvalidValue;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_cons_final, dim3(nlev), dim3(256), 0, stream, scratch, parts, nlev, out_sum, out_abs);
    return hipGetLastError();
  }
  const int64_t chunk = (V + parts - 1) / parts;
  const dim3 g(parts), b(64 * kConsWaves);
  // slices of the column's last 256-level block
  const int rem = nlev % kConsBlockLevels;
  const int nsl = rem == 0 ? 4 : (rem + 63) / 64;
  switch (dtype * 4 + (nsl - 1)) {
#define ATLAS_CONS(DT, S, N)                                                                                   \
  case DT * 4 + (N - 1):                                                                                       \
    hipLaunchKernelGGL((k_cons_partial<S, N>), g, b, 0, stream, static_cast<const S*>(div), vol, V, nlev, chunk, \
                       scratch);                                                                               \
    break;
    ATLAS_CONS(DT_F64, double, 1) ATLAS_CONS(DT_F64, double, 2) ATLAS_CONS(DT_F64, double, 3)
    ATLAS_CONS(DT_F64, double, 4) ATLAS_CONS(DT_F32, float, 1) ATLAS_CONS(DT_F32, float, 2)
    ATLAS_CONS(DT_F32, float, 3) ATLAS_CONS(DT_F32, float, 4) ATLAS_CONS(DT_BF16, bf16_t, 1)
    ATLAS_CONS(DT_BF16, bf16_t, 2) ATLAS_CONS(DT_BF16, bf16_t, 3) ATLAS_CONS(DT_BF16, bf16_t, 4)
#undef ATLAS_CONS
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_cons_final, dim3(nlev), dim3(256), 0, stream, scratch, parts, nlev, out_sum, out_abs);
  return hipGetLastError();
}

// Partial sums of the allocation-free conservation call: one array per GPU,
// held by the library until the process ends.  In host code `scratch` names
// a host-side stand-in, never the device memory: kernels and copies take the
// address hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) double scratch[kScratchBytes / sizeof(double)];

namespace {
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxScratchDevices] = {};
}  // namespace

hipError_t scratch_address(int device, double** ptr) {
  if (device < 0 || device >= kMaxScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void* p = nullptr;
    // the caller has made `device` current
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = static_cast<double*>(p);
  }
  *ptr = g_scratch_ptr[device];
  return hipSuccess;
}

int tiles_batched_per_cu(int op, int dtype, uint32_t lds, int waves, int umax) {
  const int kop = kernel_op(op);
  const void* fn = dtype == DT_F64 ? tb_fn<double>(kop, umax) : dtype == DT_F32 ? tb_fn<float>(kop, umax) : nullptr;
  if (!fn || waves < 1 || waves > batched_max_waves(kop, dtype) || lds > kLdsPerCu || umax < 1 || umax > 3) return 0;
  if (lds > 65536 && hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, 64 * waves, lds) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return n;
}

hipError_t launch_tiles_batched(int op, int dtype, const BatchTile* tr, const int32_t* pre, int ntr, int32_t* ctr,
                                int32_t claim, uint32_t lds, int waves, int64_t grid, int umax,
                                hipStream_t stream) {
  const int kop = kernel_op(op);
  // the four batchable operators and the divergence and gradient adjoint
  // pair (each tracer's out2 set)
  if (kop != OP_GRAD && kop != OP_DIV && kop != OP_GRADT && kop != OP_DIVT && op != OP_DIVGRADT)
    return hipErrorInvalidValue;
  // the grid is a multiple of 8 workgroups (one share per XCD)
  if (ntr < 1 || !ctr || claim < 1 || claim > 64 || grid < 8 || grid % 8 != 0 || grid > INT32_MAX || waves < 1 ||
      waves > batched_max_waves(kop, dtype) || lds > kLdsPerCu || umax < 1 || umax > 3)
    return hipErrorInvalidValue;
  TileArgs a;   // fields, tiling and level chunking per tracer in the kernel
  a.info = nullptr;
  a.segs = nullptr;
  a.rec = nullptr;
  a.in = nullptr;
  a.out = nullptr;
  a.out2 = nullptr;
  a.ntiles = 0;
  a.L = a.KL = a.nchunks = 1;
  a.nt = 0;
  switch (dtype) {
    case DT_F64: return launch_tb_t<double>(kop, a, tr, pre, ntr, ctr, claim, lds, waves, grid, umax, stream);
    case DT_F32: return launch_tb_t<float>(kop, a, tr, pre, ntr, ctr, claim, lds, waves, grid, umax, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_remap(int dtype, const int32_t* nodes, const void* w, int64_t V, int64_t P, int nlev,
                        const void* in, void* out, hipStream_t stream) {
  if (V < 1 || P < 1 || nlev < 1 || (P + 15) / 16 > (int64_t)INT32_MAX) return hipErrorInvalidValue;
  switch (dtype) {
    case DT_F64: return launch_remap_t<double>(nodes, w, V, P, nlev, in, out, stream);
    case DT_F32: return launch_remap_t<float>(nodes, w, V, P, nlev, in, out, stream);
    case DT_BF16: return launch_remap_t<bf16_t>(nodes, w, V, P, nlev, in, out, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_remap_adjoint(int dtype, const int64_t* off, const int32_t* tt, const void* w, const int32_t* ht,
                                const void* hw, int64_t V, int64_t P, int nlev, const void* in, void* out,
                                hipStream_t stream) {
  if (V < 1 || P < 1 || nlev < 1 || (V + 15) / 16 > (int64_t)INT32_MAX) return hipErrorInvalidValue;
  switch (dtype) {
    case DT_F64: return launch_remap_adj_t<double>(off, tt, w, ht, hw, V, P, nlev, in, out, stream);
    case DT_F32: return launch_remap_adj_t<float>(off, tt, w, ht, hw, V, P, nlev, in, out, stream);
    case DT_BF16: return launch_remap_adj_t<bf16_t>(off, tt, w, ht, hw, V, P, nlev, in, out, stream);
    default: return hipErrorInvalidValue;
  }
}

#endif  // ATLAS_KERNEL_TYPE

}  // namespace atlasnabla
