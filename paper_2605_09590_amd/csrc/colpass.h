// Column transforms of planes [rows][Gx] (kernel templates).
//
// A workgroup owns 16 adjacent columns of one plane.  A column of N = LA VA
// points is transformed in two in-register steps with one LDS exchange between
// them (layouts A and B of TwoStep), and the steps are dealt to threads as
// (column, task): thread t works on column t mod 16, in layout A on task
// a = t / 16 < LA (points a + LA m), in layout B on task k = t / 16 < VA
// (frequencies k + VA r).  Sixteen lanes of a wavefront then read or write 16
// neighbouring columns of one row, 128 contiguous bytes of a complex64 plane,
// so a column goes from memory to registers and back with no staging tile; a
// wavefront with no task in a step skips it instead of idling lanes; and a
// forward transform followed by an inverse one stays in layout B's registers.
#pragma once

#include <atomic>
#include <type_traits>

#include "fft.h"
#include "runtime.h"

namespace pico {

constexpr int kStrip = 16;   // columns per workgroup; every built line length is a multiple of 16

// C: the values' type; FP64 strips are half as wide (the same bytes)
template <int LA_, int VA_, class C = float2>
struct ColPlan {
  static constexpr int LA = LA_, VA = VA_, N = LA * VA;
  static constexpr int L = LA > VA ? LA : VA;
  static constexpr int ST = kStrip * (int)sizeof(float2) / (int)sizeof(C);
  static constexpr int THREADS = ST * L;
  // exchange: Y[a][k] of column j at k KS + ST (a ^ (k mod 2)) + j, 128 bytes per
  // task: consecutive tasks of a wavefront are on alternating halves of the LDS
  // banks in both layouts, with no padding (LA even: the swap stays inside LA)
  static_assert(LA % 2 == 0, "pairs of tasks swap");
  static constexpr int KS = ST * LA;
  static constexpr size_t LDS = (size_t)VA * KS * sizeof(C);
  using Fp64 = ColPlan<LA, VA, double2>;
};

// plane values: complex64, or bfloat16 pairs widened and rounded at the edges
__device__ __forceinline__ float2 widen(float2 v) { return v; }
__device__ __forceinline__ float2 widen(uint32_t v) { return unpack_bf16x2(v); }
__device__ __forceinline__ void narrow(float2& d, float2 v) { d = v; }
__device__ __forceinline__ void narrow(uint32_t& d, float2 v) { d = pack_bf16x2(v); }

// Layout A -> exchange: DFT over m of points a + LA m, then W^{a k} (tw).
// ODD: the points first take the factor W_{2 VA}^m (with tw = W_{2N}^{a (2k+1)}
// the transform yields the odd frequencies of the zero-padded 2N-point line)
template <class CP, bool INV, bool ODD, class C>
__device__ __forceinline__ void col_a_out(const C (&x)[CP::VA], const C (&tw)[CP::VA], C* ex, int a) {
  C v[CP::VA];
  static_for<0, CP::VA>([&](auto m) {
    if constexpr (ODD) v[m] = ctwiddle<m, 2 * CP::VA, INV>(x[m]);
    else v[m] = x[m];
  });
  dft<CP::VA, INV>(v);
#pragma unroll
  for (int k = 0; k < CP::VA; ++k) {
    const C w = INV ? cmake(tw[k].x, -tw[k].y) : tw[k];
    ex[k * CP::KS + CP::ST * (a ^ (k & 1))] = (ODD || k) ? cmul(v[k], w) : v[k];
  }
}

// exchange -> layout A of the reversed chain (INV names the sign of this transform)
template <class CP, bool INV, bool ODD, class C>
__device__ __forceinline__ void col_a_in(C (&x)[CP::VA], const C (&tw)[CP::VA], const C* ex, int a) {
  C v[CP::VA];
#pragma unroll
  for (int k = 0; k < CP::VA; ++k) {
    const C z = ex[k * CP::KS + CP::ST * (a ^ (k & 1))];
    const C w = INV ? cmake(tw[k].x, -tw[k].y) : tw[k];
    v[k] = (ODD || k) ? cmul(z, w) : z;
  }
  dft<CP::VA, INV>(v);
  static_for<0, CP::VA>([&](auto m) {
    if constexpr (ODD) x[m] = ctwiddle<m, 2 * CP::VA, INV>(v[m]);
    else x[m] = v[m];
  });
}

template <class CP, class C>
__device__ __forceinline__ void col_b_load(C (&v)[CP::LA], const C* ex, int k) {
#pragma unroll
  for (int a = 0; a < CP::LA; ++a) v[a] = ex[k * CP::KS + CP::ST * (a ^ (k & 1))];
}
template <class CP, class C>
__device__ __forceinline__ void col_b_store(const C (&v)[CP::LA], C* ex, int k) {
#pragma unroll
  for (int a = 0; a < CP::LA; ++a) ex[k * CP::KS + CP::ST * (a ^ (k & 1))] = v[a];
}

// Strip of workgroup b: workgroups go to the eight XCDs in turn, and workgroup
// b takes strip (b mod 8) ceil(W / 8) + b / 8 of the order (plane, strip), so
// each XCD runs a contiguous run of strips; -1: padding
__device__ __forceinline__ long strip_of(long b, long W) {
  const long per = (W + 7) / 8, v = (b % 8) * per + b / 8;
  return v < W ? v : -1;
}
inline unsigned strip_grid(long W) { return (unsigned)(8 * ((W + 7) / 8)); }

// ---------------------------------------------------------------- plans
// Both steps hold their points in registers: at most 32 per thread.
template <class F>
static hipError_t with_col(int n, F&& f) {
  switch (n) {
    case 32: return f(ColPlan<8, 4>{});
    case 48: return f(ColPlan<8, 6>{});
    case 64: return f(ColPlan<8, 8>{});
    case 80: return f(ColPlan<10, 8>{});
    case 96: return f(ColPlan<12, 8>{});
    case 128: return f(ColPlan<16, 8>{});
    case 144: return f(ColPlan<12, 12>{});
    case 160: return f(ColPlan<16, 10>{});
    case 192: return f(ColPlan<16, 12>{});
    case 256: return f(ColPlan<16, 16>{});
    case 288: return f(ColPlan<18, 16>{});
    case 320: return f(ColPlan<20, 16>{});
    case 384: return f(ColPlan<24, 16>{});
    case 512: return f(ColPlan<32, 16>{});
    case 576: return f(ColPlan<24, 24>{});
    case 640: return f(ColPlan<32, 20>{});
    case 768: return f(ColPlan<32, 24>{});
    default: return hipErrorInvalidValue;
  }
}

// Dynamic LDS above 64 KiB has to be allowed per kernel and device: allowed, one per
// kernel, has a bit for each device where it has been (the first 64; others ask again)
inline hipError_t allow_lds(const void* kernel, size_t bytes, std::atomic<uint64_t>& allowed) {
  if (bytes <= 64 * 1024) return hipSuccess;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0;
  if (allowed.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e == hipSuccess) allowed.fetch_or(bit, std::memory_order_release);
  return e;
}

}  // namespace pico
