// Kernels of the normal operator on a 2-D frequency grid, shared by Cartesian
// 2-D masks and the non-Cartesian Toeplitz embedding (templates; each storage
// kind is instantiated in a translation unit of its own):
//
//   q = lam p + sum_c conj(S_c) . crop( G2^-1( W . G2( pad(S_c . p) ) ) )
//
// where G2 is the unnormalised 2-D DFT on a Gy x Gx grid and W a real
// weight, [Gy][Gx] in memory:
//  * Cartesian 2-D mask: Gy x Gx = ny x nx, W = mask / (ny nx), maps folded
//    with (-1)^(y+x) (the centred DFT is (-1)^((ny+nx)/2) D F D, D = (-1)^(y+x),
//    so the centred-order mask applies unchanged; Sec. 2.1 Eq. (6));
//  * spiral, Toeplitz form (Sec. 3.2.2, 3.3): Gy x Gx = 2ny x 2nx,
//    W = DFT(circulant embedding of the point-spread function) / (4 ny nx),
//    real because the PSF is Hermitian; the product is the exact NUDFT
//    normal operator A^H A.
//
// Three kernels per application, all per-probe fields row-major [K][ny][nx]:
//  rows_fwd  per image row: CG update / probe draw, then per coil S_c p,
//            zero-pad to Gx, row FFT -> T[k][c][y][Gx] (only the ny
//            non-zero rows of the padded grid are stored);
//  cols      per strip of 16 grid columns of one (k, c) plane (colpass.h):
//            zero-pad to Gy, column FFT, times W, inverse column FFT, keep
//            rows < ny;
//  rows_inv  per image row: per coil inverse row FFT, crop to nx,
//            conj(S_c) times it, summed over coils; q written with the FP64
//            partial dots of the CG step.
#pragma once

#include <algorithm>
#include <type_traits>

#include "colpass.h"
#include "fft.h"
#include "runtime.h"

namespace pico {
// Coil map value i as stored (complex64, or for ST >= 1 a packed bfloat16
// pair) and widened; prefetched values stay in storage form until use, so
// the loads are not waited on at the point of issue
template <int ST> using MapElem = std::conditional_t<(ST >= 1), uint32_t, float2>;
template <int ST>
__device__ __forceinline__ MapElem<ST> map_raw(const Grid2dArgs& a, size_t i) {
  if constexpr (ST >= 1) return a.maps_bf[i];
  else return a.maps[i];
}
template <int ST>
__device__ __forceinline__ float2 map_at(const Grid2dArgs& a, size_t i) { return widen(map_raw<ST>(a, i)); }


// Direct global -> LDS copy of one row of n elements of E per column group of
// the wavefront: group gi's row, from src(gi), goes to the start of its
// transform tile.  Each lane loads 16 bytes per instruction and the hardware
// places them at tile + lane * 16 bytes, so the loads hold no registers.
// The row kernels use it to fetch the next coil's row into the tile, which is
// idle between two transforms; wait_lds_loads() precedes the first LDS read
// of the row.  Rows are 16-byte aligned (n and the row pitch multiples of
// 16 / E).
template <class CF, class E, int GS, class F>
__device__ __forceinline__ void dma_rows(E* dst, int n, F&& src) {
  constexpr int G = 64 / CF::L, PER = 16 / (int)sizeof(E), CH = 64 * PER;
  wait_lds_reads();
  const int lo = (int)(threadIdx.x % 64) * PER;   // this lane's first element of every chunk
#pragma unroll
  for (int gi = 0; gi < G; ++gi) {
    const E* s = src(gi) + lo;
    E* d = dst + gi * GS;
#pragma unroll
    for (int j = 0; j * CH < CF::N; ++j)   // rows are at most N elements
      if (j * CH + lo < n)
        __builtin_amdgcn_global_load_lds((const void*)(s + j * CH),
                                         (__attribute__((address_space(3))) void*)(d + j * CH), 16, 0, 0);
  }
}

// Wavefronts per workgroup of the row kernels where a launch has few rows (at most
// kFewRowGroups wavefronts of them): all work on the same rows, wavefront w on coils
// w, w + NW, ..., and their sums meet in LDS.  Each forms p itself, which costs the
// fields' reads NW times over.  Four where their tiles fit 64 KiB of LDS, else two.
template <class CF>
constexpr int kRowWaves = 4 * ((64 + CF::L - 1) / CF::L * CF::SPAN + (CF::kRowsDma ? 0 : 64 / CF::L * CF::N)) * 8 <= 60 * 1024 ? 4 : 2;

// Where the line lies, solves of 192 x 160 (8 coils), 256 x 256 (12) and 320 x 320 (15)
// with one / NW wavefronts per row group: 192-256 groups 726 / 528, 1262 / 939 and
// 1613 / 986 us, 768-853 groups 934 / 793, 1620 / 1506 and 2371 / 2303 us, 1024-1152
// groups 1088 / 1069, 1817 / 2030 and 2685 / 2854 us.
constexpr long kFewRowGroups = 3 * 256;

// sum over a lane group of L lanes, in lane order, by every lane's own wavefront
template <int L>
__device__ __forceinline__ double group_reduce2(double v, double* red, int tid, int lane) {
  red[tid] = v;
  wave_sync();
  double s = 0.0;
  if (lane == 0) {
    for (int i = 0; i < L; ++i) s += red[tid + i];
  }
  wave_sync();
  return s;
}

// ---------------------------------------------------------------- row pass 1
template <class CF, int MODE, int ST, bool HALF, int NW>
__global__ __launch_bounds__(64 * NW) void k_rows_fwd(Grid2dArgs a) {
  constexpr int L = CF::L, G = 64 / L, NG = (64 + L - 1) / L;
  constexpr int VA = CF::VA, VB = CF::VB;
  // HALF (the Toeplitz grids, nx = Gx / 2): values m >= VA / 2 lie past the
  // image row, so they are compile-time zeros in the forward transform
  constexpr int VAH = HALF ? VA / 2 : VA;
  __shared__ float2 lds_waves[NW * NG * CF::SPAN];
  __shared__ double red[64 + L];   // lane 0 of a partial last group reads L entries
  const int wave = NW > 1 ? threadIdx.x / 64 : 0, tid = NW > 1 ? threadIdx.x % 64 : threadIdx.x;
  float2* lds_all = lds_waves + wave * NG * CF::SPAN;
  const int g = tid / L, lane = tid % L;
  const long gid = (long)blockIdx.x * G + g;
  const bool active = g < G && gid < (long)a.K * a.ny;
  const long gg = active ? gid : 0;
  const int k = (int)(gg / a.ny), y = (int)(gg % a.ny);
  const bool inA = CF::inA(lane), inB = CF::inB(lane);
  float2* lds = lds_all + g * CF::SPAN;
  typename CF::Tw tw;
  CF::load_tw(tw, a.twx, lane);
  // two-step rows (256 points and more): coil 0's map rows go into the
  // transform tiles while the CG update runs (later coils': see the coil loop)
  constexpr bool DMA = CF::kRowsDma, PF = !DMA && CF::N >= 384;
  using ME = MapElem<ST>;
  auto map_rows = [&](int c) {
    dma_rows<CF, ME, CF::SPAN * (int)(sizeof(float2) / sizeof(ME))>(reinterpret_cast<ME*>(lds_all), a.nx, [&](int gi) {
      const long gq = (long)blockIdx.x * G + gi;
      const long gr = gq < (long)a.K * a.ny ? gq : 0;
      const size_t moff = ((size_t)c * a.ny + (int)(gr % a.ny)) * a.nx;
      if constexpr (ST >= 1) return (const ME*)(a.maps_bf + moff);
      else return (const ME*)(a.maps + moff);
    });
  };
  if constexpr (DMA) if (wave < a.nc) map_rows(wave);

  const size_t rowoff = ((size_t)k * a.ny + y) * a.nx;
  // the per-probe fields never alias one another: restrict lets every load of
  // the row go out before the first store
  float2* __restrict__ X = a.x;
  float2* __restrict__ R = a.r;
  float2* __restrict__ P = a.p;
  const float2* __restrict__ Q = a.q;
  const float2* __restrict__ SRC = a.src;
  float2 pv[CF::VMAX];
  double d0 = 0.0;
  float alpha = 0.f, beta = 0.f;
  if constexpr (MODE == C1_ITER) {
    alpha = (float)a.alpha[k];
    beta = (float)a.beta[k];
  }
  // every wavefront forms p of the rows from the old fields; once all have read
  // them, the wavefronts write x, r and p, a share of the elements each
#pragma unroll
  for (int m = 0; m < VA; ++m) {
    if (HALF && m >= VAH) {   // past the image row
      pv[m] = make_float2(0.f, 0.f);
      continue;
    }
    const int xx = CF::posA(lane, m);
    const bool ok = inA && xx < a.nx;
    const size_t i = rowoff + (ok ? xx : 0);   // in-bounds address for every lane
    float2 val = make_float2(0.f, 0.f);
    if constexpr (MODE == C1_FIRST_PROBE) {
      val = draw_probe(arg_seed(a), arg_first(a) + a.k0 + k, (uint32_t)(y * a.nx + xx), 0u, a.dist);
      if (!ok) val = make_float2(0.f, 0.f);
      if (active && ok && m % NW == wave) { R[i] = val; P[i] = val; }
      d0 += (double)val.x * val.x + (double)val.y * val.y;
    } else if constexpr (MODE == C1_FIRST_BUF) {
      // loads go out on every lane (the address is in bounds) and lanes
      // outside the row are zeroed by a factor: a load under a lane
      // condition (or as an operand of a select) gets a branch and a wait
      // of its own
      val = cscale(R[i], ok ? 1.f : 0.f);
      if (active && ok && m % NW == wave) P[i] = val;
      d0 += (double)val.x * val.x + (double)val.y * val.y;
    } else if constexpr (MODE == C1_ITER) {
      val = make_float2(0.f, 0.f);
      if constexpr (NW > 1) {   // p of iteration i; the fields are updated below
        const float2 rn = cfma(R[i], -alpha, Q[i]);
        val = cfma(rn, beta, P[i]);
        if (!ok) val = make_float2(0.f, 0.f);
        else d0 += (double)rn.x * rn.x + (double)rn.y * rn.y;
      }
    } else {  // C1_APPLY
      val = cscale(SRC[i], ok ? a.scale : 0.f);
    }
    pv[m] = val;
  }
  if constexpr (MODE == C1_ITER) {
    // finish iteration i-1 and start i: x += alpha p, r -= alpha q, p = r + beta p,
    // a share of the elements for each wavefront.  In chunks of H elements, every
    // load of a chunk is issued before its first store.
    constexpr int S = (VAH + NW - 1) / NW, H = S > 8 ? 8 : S;
    if constexpr (NW > 1) __syncthreads();
    const bool xz = a.x_zero != 0;
#pragma unroll
    for (int m0 = 0; m0 < S; m0 += H) {
      float2 po[H], qo[H], ro[H], xo[H];
#pragma unroll
      for (int h = 0; h < H; ++h) {
        if (m0 + h >= S) break;
        const int m = NW > 1 ? min(wave * S + m0 + h, VAH - 1) : m0 + h, xx = CF::posA(lane, m);
        const size_t i = rowoff + ((inA && xx < a.nx) ? xx : 0);
        po[h] = P[i];
        qo[h] = Q[i];
        ro[h] = R[i];
        xo[h] = X[i];
      }
#pragma unroll
      for (int h = 0; h < H; ++h) {
        if (m0 + h >= S) break;
        const int m = wave * S + m0 + h, xx = CF::posA(lane, m);
        const bool ok = inA && m < VAH && xx < a.nx;
        const size_t i = rowoff + (ok ? xx : 0);
        const float2 rn = ok ? cfma(ro[h], -alpha, qo[h]) : make_float2(0.f, 0.f);
        const float2 pn = ok ? cfma(rn, beta, po[h]) : make_float2(0.f, 0.f);
        if (active && ok) {
          X[i] = cfma(xz ? make_float2(0.f, 0.f) : xo[h], alpha, po[h]);
          R[i] = rn;
          P[i] = pn;
        }
        if constexpr (NW == 1) {
          pv[m0 + h] = pn;
          d0 += (double)rn.x * rn.x + (double)rn.y * rn.y;
        }
      }
    }
  }
  if constexpr (MODE != C1_APPLY) {
    if (wave == 0) {
      d0 = group_reduce2<L>(d0, red, tid, lane);
      if (active && lane == 0) a.part[((size_t)k * a.ny + y) * 4] = d0;
    }
  }

  float2* __restrict__ T = a.T;
  uint32_t* __restrict__ Tb = a.Tb;
  // Stockham rows of 512 and 768 points: the map row of coil c + 1 is loaded
  // into registers while coil c is transformed (measured: 512-point spiral
  // rows 6.63 -> 5.53 ms per application).  The two-step rows get their map
  // rows straight into the transform tiles, coil c + 1's once coil c's
  // transform is done; the short Stockham plans keep direct loads (their
  // many groups per wavefront would need more address registers than they
  // have).
  MapElem<ST> svn[CF::VMAX];
  auto load_maps = [&](int c) {
    const size_t moff = ((size_t)c * a.ny + y) * a.nx;
#pragma unroll
    for (int m = 0; m < VA; ++m) {
      if (HALF && m >= VAH) continue;   // past the image row (zero)
      const int xx = CF::posA(lane, m);
      svn[m] = map_raw<ST>(a, moff + ((inA && xx < a.nx) ? xx : 0));
    }
  };
  if constexpr (PF) if (wave < a.nc) load_maps(wave);
  for (int c = wave; c < a.nc; c += NW) {
    float2 v[CF::VMAX];
    if constexpr (PF) {
#pragma unroll
      for (int m = 0; m < VA; ++m) {
        if (HALF && m >= VAH) {   // past the image row
          v[m] = make_float2(0.f, 0.f);
          continue;
        }
        v[m] = cmul(widen(svn[m]), pv[m]);   // pv is 0 outside the row
      }
      if (c + NW < a.nc) load_maps(c + NW);
    } else if constexpr (DMA) {
      wait_lds_loads();
      const ME* mrow = reinterpret_cast<const ME*>(lds);
#pragma unroll
      for (int m = 0; m < VA; ++m) {
        if (HALF && m >= VAH) {   // past the image row
          v[m] = make_float2(0.f, 0.f);
          continue;
        }
        const int xx = CF::posA(lane, m);
        const bool ok = inA && xx < a.nx;
        v[m] = cmul(widen(mrow[ok ? xx : 0]), pv[m]);   // pv is 0 outside the row
      }
    } else {
      const size_t moff = ((size_t)c * a.ny + y) * a.nx;
#pragma unroll
      for (int m = 0; m < VA; ++m) {
        if (HALF && m >= VAH) {   // past the image row
          v[m] = make_float2(0.f, 0.f);
          continue;
        }
        const int xx = CF::posA(lane, m);
        const bool ok = inA && xx < a.nx;
        v[m] = cmul(map_at<ST>(a, moff + (ok ? xx : 0)), pv[m]);   // pv is 0 outside the row
      }
    }
    CF::template forward<false>(v, lds, lane, tw);
    if constexpr (DMA) {
      if (c + NW < a.nc) map_rows(c + NW);
    }
    if (active && inB) {
      const size_t off = (((size_t)k * a.nc + c) * a.ny + y) * a.Gx;
      if constexpr (ST == 2) {
#pragma unroll
        for (int r = 0; r < VB; ++r) Tb[off + CF::posB(lane, r)] = pack_bf16x2(v[r]);
      } else {
#pragma unroll
        for (int r = 0; r < VB; ++r) T[off + CF::posB(lane, r)] = v[r];
      }
    }
  }
}

// ---------------------------------------------------------------- column pass
// Unpadded 320-point columns are held to 128 registers (8 values spilled): three
// workgroups of five wavefronts share a CU instead of two (solves of 96 probes, 16
// coils: complex64 23.3 -> 23.1 ms, bfloat16 planes 19.7 -> 17.5 ms).
template <class CP, bool PAD>
constexpr int kColWaves = CP::N == 320 && !PAD ? 4 : 1;

// Per column of a (k, c) plane: transform along y, weights, inverse transform,
// in place.  PAD (the Toeplitz grids, Gy = 2 ny): the column is the first half
// of a line of 2 ny points, zero past it, and only the first half of the
// result is kept, so the line is never formed: its even and odd frequencies
// are two ny-point transforms of the column (times W_{2 ny}^y for the odd
// ones), and the two inverse transforms add up to the kept half.
// a.w is [Gy][Gx]; PAD: rows 0..ny-1 the even frequencies, ny..2ny-1 the odd.
// Bound by the planes' traffic, read and written once each: 2 x 256 padded
// columns of 256 x 16 coils x 128 probes (4.3 GB) take 1.06 ms, 4.1 TB/s,
// against 4.4 TB/s for a plain in-place pass over buffers of that size; the
// staged 512-point transforms this replaces took 1.26 ms with the VALU 93 % busy.
template <class CP, bool TB, bool PAD>
__global__ __launch_bounds__(CP::THREADS, (kColWaves<CP, PAD>)) void k_cols(Grid2dArgs a) {
  constexpr int LA = CP::LA, VA = CP::VA, N = CP::N;
  extern __shared__ float2 dyn[];
  using E = std::conditional_t<TB, uint32_t, float2>;
  const int S = a.Gx / kStrip;
  const long vb = strip_of(blockIdx.x, (long)S * a.K * a.nc);
  if (vb < 0) return;
  const int col = threadIdx.x % kStrip, t = threadIdx.x / kStrip;
  const int xc = (int)(vb % S) * kStrip + col;
  E* __restrict__ pl;
  if constexpr (TB) pl = a.Tb;
  else pl = a.T;
  pl += (size_t)(vb / S) * N * a.Gx + xc;
  float2* ex = dyn + col;
  const float2* __restrict__ twy = a.twy;
  const bool inA = LA == CP::L || t < LA, inB = VA == CP::L || t < VA;
  E raw[VA];
  float2 tw[VA];
  if (inA) {
#pragma unroll
    for (int m = 0; m < VA; ++m) raw[m] = pl[(size_t)(t + LA * m) * a.Gx];
#pragma unroll
    for (int k = 0; k < VA; ++k) tw[k] = twy[t * k * (PAD ? 2 : 1)];
  }
  const float* __restrict__ w = a.w + (size_t)t * a.Gx + xc;   // row of layout B's task
  float2 x[VA], out[VA];
  if (inA) {
#pragma unroll
    for (int m = 0; m < VA; ++m) x[m] = widen(raw[m]);
  }
  auto weigh = [&](int s) {
    if (inB) {
      float wr[LA];
#pragma unroll
      for (int r = 0; r < LA; ++r) wr[r] = w[(size_t)(s * N + VA * r) * a.Gx];
      float2 v[LA];
      col_b_load<CP>(v, ex, t);
      dft<LA, false>(v);
#pragma unroll
      for (int r = 0; r < LA; ++r) v[r] = cscale(v[r], wr[r]);
      dft<LA, true>(v);
      col_b_store<CP>(v, ex, t);   // the task's own values: no barrier in between
    }
  };
  if (inA) col_a_out<CP, false, false>(x, tw, ex, t);
  __syncthreads();
  weigh(0);
  __syncthreads();
  if (inA) col_a_in<CP, true, false>(out, tw, ex, t);
  if constexpr (PAD) {
    if (inA) {   // this task's values of the exchange have been read: no barrier
#pragma unroll
      for (int k = 0; k < VA; ++k) tw[k] = twy[t * (2 * k + 1)];
      col_a_out<CP, false, true>(x, tw, ex, t);
    }
    __syncthreads();
    weigh(1);
    __syncthreads();
    if (inA) {
      col_a_in<CP, true, true>(x, tw, ex, t);
#pragma unroll
      for (int m = 0; m < VA; ++m) out[m] = cadd(out[m], x[m]);
    }
  }
  if (inA) {
#pragma unroll
    for (int m = 0; m < VA; ++m) narrow(pl[(size_t)(t + LA * m) * a.Gx], out[m]);
  }
}

// The same through an LDS tile, for the lengths of staged_cols: 256 / L adjacent columns
// of a plane are loaded (batches of 8 loads per thread), transformed as lines of Gy
// points by groups of L lanes, a column each, and stored.  PAD: both layouts place
// values m < VA / 2 and r < VB / 2 in the first half, so the zeros and the unused
// outputs fold out of the first and last steps.  a.w is [Gx][Gy].
// The register form holds three sets of VA values at once when PAD (x, out and the
// twiddles: 190-200 registers at 288 and 320 points) and 32 values a task at 512, so
// few wavefronts are left to hide its loads.  Maps of 12 coils, 8 CG iterations, 0.9 GB
// of planes, ms, registers / tile: padded 288 points 9.30 / 8.40 (bfloat16 planes 8.24 /
// 7.21), 320 9.44 / 8.09 (8.21 / 7.22), unpadded 512 7.64 / 6.95 (6.18 / 5.96); the
// others are as fast or faster in registers: padded 256 6.58 / 7.43 (5.65 / 6.58), 384
// 9.49 / 9.39 (7.73 / 8.16), unpadded 576 9.00 / 8.98 (6.44 / 6.51), 640 9.32 / 9.27
// (6.52 / 6.57), 768 8.78 / 8.86 (6.23 / 7.17).
template <class CF, bool TB, bool PAD>
__global__ __launch_bounds__(256) void k_cols_staged(Grid2dArgs a) {
  constexpr int L = CF::L, NC = 256 / L, VA = CF::VA, VB = CF::VB, TS = NC + 1, B = 8;
  constexpr int NY = PAD ? CF::N / 2 : CF::N, TOTAL = NY * NC;
  static_assert(64 % L == 0, "a group stays within its wavefront");
  static_assert(!PAD || (VA % 2 == 0 && VB % 2 == 0), "halves of a lane's values");
  static_assert(TOTAL % 256 == 0, "whole rounds of loads");
  using E = std::conditional_t<TB, uint32_t, float2>;
  extern __shared__ float2 dyn[];   // [NY][TS] tile; between the loads and the stores, the groups' exchanges
  const int S = a.Gx / NC;
  const long vb = strip_of(blockIdx.x, (long)S * a.K * a.nc);
  if (vb < 0) return;
  const int x0 = (int)(vb % S) * NC, g = threadIdx.x / L, lane = threadIdx.x % L;
  E* __restrict__ pl;
  if constexpr (TB) pl = a.Tb;
  else pl = a.T;
  pl += (size_t)(vb / S) * NY * a.Gx + x0;
#pragma unroll
  for (int i0 = 0; i0 < TOTAL; i0 += B * 256) {
    E v[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int i = i0 + u * 256 + (int)threadIdx.x;
      if (i0 + u * 256 < TOTAL) v[u] = pl[(size_t)(i / NC) * a.Gx + i % NC];
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int i = i0 + u * 256 + (int)threadIdx.x;
      if (i0 + u * 256 < TOTAL) dyn[i / NC * TS + i % NC] = widen(v[u]);
    }
  }
  __syncthreads();
  const bool inA = CF::inA(lane), inB = CF::inB(lane);
  typename CF::Tw tw;
  CF::load_tw(tw, a.twy, lane);
  float2 v[CF::VMAX];
#pragma unroll
  for (int m = 0; m < VA; ++m) {
    if (PAD && m >= VA / 2) v[m] = make_float2(0.f, 0.f);
    else v[m] = inA ? dyn[CF::posA(lane, m) * TS + g] : make_float2(0.f, 0.f);
  }
  __syncthreads();
  float2* ex = dyn + g * CF::SPAN;
  CF::template forward<false>(v, ex, lane, tw);
  const float* __restrict__ w = a.w + (size_t)(x0 + g) * a.Gy;
  if (inB) {
#pragma unroll
    for (int r = 0; r < VB; ++r) v[r] = cscale(v[r], w[CF::posB(lane, r)]);
  }
  CF::template inverse<true>(v, ex, lane, tw);
  __syncthreads();
  if (inA) {
#pragma unroll
    for (int m = 0; m < (PAD ? VA / 2 : VA); ++m) dyn[CF::posA(lane, m) * TS + g] = v[m];
  }
  __syncthreads();
#pragma unroll 8
  for (int i = threadIdx.x; i < TOTAL; i += 256) narrow(pl[(size_t)(i / NC) * a.Gx + i % NC], dyn[i / NC * TS + i % NC]);
}

// ---------------------------------------------------------------- row pass 2
template <class CF, int MODE, int ST, bool HALF, int NW>
__global__ __launch_bounds__(64 * NW) void k_rows_inv(Grid2dArgs a) {
  constexpr int L = CF::L, G = 64 / L, NG = (64 + L - 1) / L;
  constexpr int VA = CF::VA, VB = CF::VB;
  // HALF (the Toeplitz grids, nx = Gx / 2): only values m < VA / 2 of the
  // inverse transform lie in the image row
  constexpr int VAH = HALF ? VA / 2 : VA;
  __shared__ float2 lds_waves[NW * NG * CF::SPAN];
  __shared__ double red[NW * 3 * (64 + L)];   // the sums of a partial last group read past the wavefront
  const int wave = NW > 1 ? threadIdx.x / 64 : 0, tid = NW > 1 ? threadIdx.x % 64 : threadIdx.x;
  float2* lds_all = lds_waves + wave * NG * CF::SPAN;
  const int g = tid / L, lane = tid % L;
  const long gid = (long)blockIdx.x * G + g;
  const bool active = g < G && gid < (long)a.K * a.ny;
  const long gg = active ? gid : 0;
  const int k = (int)(gg / a.ny), y = (int)(gg % a.ny);
  const bool inA = CF::inA(lane), inB = CF::inB(lane);
  float2* lds = lds_all + g * CF::SPAN;
  typename CF::Tw tw;
  CF::load_tw(tw, a.twx, lane);
  const size_t rowoff = ((size_t)k * a.ny + y) * a.nx;

  const float2* __restrict__ P = a.p;
  const float2* __restrict__ R = a.r;
  const float2* __restrict__ SRC = a.src;
  const float2* __restrict__ T = a.T;
  float2* __restrict__ Qo = a.q;
  constexpr bool DMA = CF::kRowsDma, PF = !DMA && CF::N >= 384;
  using TE = std::conditional_t<ST == 2, uint32_t, float2>;
  // two-step rows: coil c + 1's transformed rows go straight into the
  // transform tiles once coil c's inverse transform is done
  auto t_rows = [&](int c) {
    dma_rows<CF, TE, CF::SPAN * (int)(sizeof(float2) / sizeof(TE))>(reinterpret_cast<TE*>(lds_all), a.Gx, [&](int gi) {
      const long gq = (long)blockIdx.x * G + gi;
      const long gr = gq < (long)a.K * a.ny ? gq : 0;
      const size_t off = (((size_t)(gr / a.ny) * a.nc + c) * a.ny + (int)(gr % a.ny)) * a.Gx;
      if constexpr (ST == 2) return (const TE*)(a.Tb + off);
      else return (const TE*)(T + off);
    });
  };
  if constexpr (DMA) if (wave < a.nc) t_rows(wave);
  // Stockham rows of 512 and 768 points: each coil's map rows come through LDS (a
  // buffer of their own, fetched when the coil starts and read after its
  // inverse transform); with the transformed row of the next coil already in
  // registers, the combine's own loads would be serialised for want of them
  using ME = MapElem<ST>;
  __shared__ ME mapbufs[PF ? NW * G * CF::N : 1];
  ME* mapbuf = mapbufs + (PF ? wave * G * CF::N : 0);
  auto map_rows = [&](int c) {
    dma_rows<CF, ME, CF::N>(mapbuf, a.nx, [&](int gi) {
      const long gq = (long)blockIdx.x * G + gi;
      const long gr = gq < (long)a.K * a.ny ? gq : 0;
      const size_t moff = ((size_t)c * a.ny + (int)(gr % a.ny)) * a.nx;
      if constexpr (ST >= 1) return (const ME*)(a.maps_bf + moff);
      else return (const ME*)(a.maps + moff);
    });
  };
  float2 qa[CF::VMAX];   // sum over this wavefront's coils
#pragma unroll
  for (int m = 0; m < VAH; ++m) qa[m] = make_float2(0.f, 0.f);
  // Stockham rows of 512 and 768 points: the transformed row of coil c + 1 is loaded
  // while coil c is inverted (raw storage form, unconditional loads from
  // in-row addresses; lanes outside layout B get zeros at use)
  TE tn[CF::VMAX];
  auto load_row = [&](int c) {
    const size_t off = (((size_t)k * a.nc + c) * a.ny + y) * a.Gx;
#pragma unroll
    for (int r = 0; r < VB; ++r) {
      const size_t j = off + (inB ? CF::posB(lane, r) : 0);
      if constexpr (ST == 2) tn[r] = a.Tb[j];
      else tn[r] = T[j];
    }
  };
  if constexpr (PF) if (wave < a.nc) load_row(wave);
  for (int c = wave; c < a.nc; c += NW) {
    float2 v[CF::VMAX];
    if constexpr (PF) {
#pragma unroll
      for (int r = 0; r < VB; ++r) v[r] = widen(tn[r]);   // unused outside layout B
      map_rows(c);
      if (c + NW < a.nc) load_row(c + NW);
    } else if constexpr (DMA) {
      wait_lds_loads();
      const TE* trow = reinterpret_cast<const TE*>(lds);
#pragma unroll   // lanes outside layout B read tile padding, unused by the transform
      for (int r = 0; r < VB; ++r) v[r] = widen(trow[CF::posB(lane, r)]);
    } else {
      const size_t off = (((size_t)k * a.nc + c) * a.ny + y) * a.Gx;
      if constexpr (ST == 2) {
#pragma unroll
        for (int r = 0; r < VB; ++r) v[r] = unpack_bf16x2(a.Tb[off + (inB ? CF::posB(lane, r) : 0)]);
      } else {
#pragma unroll
        for (int r = 0; r < VB; ++r) v[r] = T[off + (inB ? CF::posB(lane, r) : 0)];   // unused outside layout B
      }
    }
    CF::template inverse<true>(v, lds, lane, tw);
    if constexpr (DMA) {
      if (c + NW < a.nc) t_rows(c + NW);
    }
    // the combine is unconditional (lanes outside the row are never stored
    // or summed)
    if constexpr (PF) {
      wait_lds_loads();
      const ME* mrow = mapbuf + (g < G ? g : 0) * CF::N;
#pragma unroll
      for (int m = 0; m < VA; ++m) {
        if (HALF && m >= VAH) continue;   // past the image row (zero)
        const int xx = CF::posA(lane, m);
        const bool ok = inA && xx < a.nx;
        qa[m] = cadd(qa[m], cmulc(widen(mrow[ok ? xx : 0]), v[m]));
      }
    } else {
      const size_t moff = ((size_t)c * a.ny + y) * a.nx;
#pragma unroll
      for (int m = 0; m < VA; ++m) {
        if (HALF && m >= VAH) continue;   // past the image row (zero)
        const int xx = CF::posA(lane, m);
        const bool ok = inA && xx < a.nx;
        qa[m] = cadd(qa[m], cmulc(map_at<ST>(a, moff + (ok ? xx : 0)), v[m]));
      }
    }
  }
  // the wavefronts' sums meet in their tiles; each takes a share of the elements
  // (added in wavefront order), with lam p, q's store and the dots
  static_assert(NW == 1 || VAH * 64 <= NG * CF::SPAN, "a wavefront's sums fit its tile");
  constexpr int H = (VAH + NW - 1) / NW;
  if constexpr (NW > 1) {
#pragma unroll
    for (int m = 0; m < VAH; ++m) lds_all[m * 64 + tid] = qa[m];
  }
  float2 pa[H], ra[H];   // p (or scale * src) and r of the share
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int m = min(wave * H + h, VAH - 1), xx = CF::posA(lane, m);
    const bool ok = inA && xx < a.nx;
    const size_t i = rowoff + (ok ? xx : 0);
    const float2 raw = MODE == C1_APPLY ? SRC[i] : P[i];
    pa[h] = cscale(raw, ok ? (MODE == C1_APPLY ? a.scale : 1.f) : 0.f);
    ra[h] = MODE == C1_ITER ? R[i] : pa[h];
  }
  if constexpr (NW > 1) __syncthreads();
  double d[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int m = wave * H + h, xx = CF::posA(lane, m);
    if (m >= VAH || !inA || xx >= a.nx) continue;
    float2 q = a.lam != 0.f ? cscale(pa[h], a.lam) : make_float2(0.f, 0.f);
#pragma unroll
    for (int w = 0; w < NW; ++w) q = cadd(q, NW > 1 ? lds_waves[w * NG * CF::SPAN + m * 64 + tid] : qa[m % VAH]);
    if (active) Qo[rowoff + xx] = q;
    d[0] += (double)pa[h].x * q.x + (double)pa[h].y * q.y;
    d[1] += (double)q.x * q.x + (double)q.y * q.y;
    d[2] += (double)ra[h].x * q.x + (double)ra[h].y * q.y;
  }
#pragma unroll
  for (int j = 0; j < 3; ++j) red[(wave * 3 + j) * (64 + L) + tid] = d[j];
  __syncthreads();
  static_assert(L >= 3, "one lane per sum");
  if (wave == 0 && active && lane < 3) {   // the three sums of the row, wavefronts and lanes in order
    double t = 0.0;
    for (int w = 0; w < NW; ++w)
      for (int i = 0; i < L; ++i) t += red[(w * 3 + lane) * (64 + L) + tid - lane + i];
    a.part[((size_t)k * a.ny + y) * 4 + 1 + lane] = t;
  }
}

// ---------------------------------------------------------------- plans
// Every row and column kernel holds at most two waves per SIMD here, so the
// plan per length is the one whose kernels fit 256 VGPRs without spilling:
// two-step plans (one LDS transpose per transform) where LA + VA values per
// lane fit, 32-lane groups for 576 and 640 points, and a 64-lane Stockham
// plan for 768 points (12 values per lane; the 32-lane plans of 768 points
// spill).  Measured per normal-operator application against the 16- and
// 32-lane Stockham plans they replace: 288-point grid 6.87 -> 2.55 ms (30
// coils, K = 128), 576 x 576 6.23 -> 3.54 ms and 640 x 640 4.82 -> 3.26 ms
// (spiral, K = 64), 768 x 768 13.4 -> 6.6 ms (32 coils, K = 32); 160- and
// 192-point grids (16 coils, K = 256) 1.03 -> 0.86 and 1.44 -> 1.15 ms.  The
// 64-lane plan of 512 points (8 x 8 x 8) measured 2 % slower than the 32-lane
// one, and the two-step plans of 96 and 128 points 5-15 % slower than the
// Stockham ones kept there.
using L64 = TwoStep<8, 8>;
using L96 = StockhamCol<FFTPlan<96, 8, 12, 4, 2>>;
using L128 = StockhamCol<FFTPlan<128, 16, 8, 4, 4>>;
using L160 = TwoStep<16, 10>;
using L192 = TwoStep<16, 12>;
using L256 = TwoStep<16, 16>;
using L288 = TwoStep<18, 16>;
using L320 = TwoStep<20, 16>;
using L384 = TwoStep<24, 16>;
using L512 = StockhamCol<FFTPlan<512, 32, 16, 16, 2>>;
using L576 = TwoStep<32, 18>;
using L640 = TwoStep<32, 20>;
using L768 = StockhamCol<FFTPlan<768, 64, 12, 4, 4, 4>>;

template <class F>
static hipError_t with_line(int n, F&& f) {
  switch (n) {
    case 64: return f(L64{});
    case 96: return f(L96{});
    case 128: return f(L128{});
    case 160: return f(L160{});
    case 192: return f(L192{});
    case 256: return f(L256{});
    case 288: return f(L288{});
    case 320: return f(L320{});
    case 384: return f(L384{});
    case 512: return f(L512{});
    case 576: return f(L576{});
    case 640: return f(L640{});
    case 768: return f(L768{});
    default: return hipErrorInvalidValue;
  }
}

template <class CF, int ST, bool HALF, int NW>
static hipError_t rows_fwd_h(int mode, const Grid2dArgs& a, hipStream_t s) {
  constexpr int G = 64 / CF::L;
  const long rows = (long)a.K * a.ny;
  dim3 grid((unsigned)((rows + G - 1) / G)), block(64 * NW);
  switch (mode) {
    case C1_FIRST_PROBE: hipLaunchKernelGGL((k_rows_fwd<CF, C1_FIRST_PROBE, ST, HALF, NW>), grid, block, 0, s, a); break;
    case C1_FIRST_BUF: hipLaunchKernelGGL((k_rows_fwd<CF, C1_FIRST_BUF, ST, HALF, NW>), grid, block, 0, s, a); break;
    case C1_ITER: hipLaunchKernelGGL((k_rows_fwd<CF, C1_ITER, ST, HALF, NW>), grid, block, 0, s, a); break;
    case C1_APPLY: hipLaunchKernelGGL((k_rows_fwd<CF, C1_APPLY, ST, HALF, NW>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <class CF, int ST, bool HALF, int NW>
static hipError_t rows_inv_h(int mode, const Grid2dArgs& a, hipStream_t s) {
  constexpr int G = 64 / CF::L;
  const long rows = (long)a.K * a.ny;
  dim3 grid((unsigned)((rows + G - 1) / G)), block(64 * NW);
  switch (mode) {
    case C1_FIRST_PROBE: case C1_FIRST_BUF:
      hipLaunchKernelGGL((k_rows_inv<CF, C1_FIRST_BUF, ST, HALF, NW>), grid, block, 0, s, a); break;
    case C1_ITER: hipLaunchKernelGGL((k_rows_inv<CF, C1_ITER, ST, HALF, NW>), grid, block, 0, s, a); break;
    case C1_APPLY: hipLaunchKernelGGL((k_rows_inv<CF, C1_APPLY, ST, HALF, NW>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// the half-row variants when the image row is the first half of the grid row
// (the Toeplitz grids, nx = Gx / 2)
template <class CF, int ST>
static hipError_t rows_fwd(int mode, const Grid2dArgs& a, hipStream_t s) {
  constexpr int G = 64 / CF::L;
  const bool few = ((long)a.K * a.ny + G - 1) / G <= kFewRowGroups;
  if constexpr (CF::VA % 2 == 0) {
    if (2 * a.nx == a.Gx)
      return few ? rows_fwd_h<CF, ST, true, kRowWaves<CF>>(mode, a, s) : rows_fwd_h<CF, ST, true, 1>(mode, a, s);
  }
  return few ? rows_fwd_h<CF, ST, false, kRowWaves<CF>>(mode, a, s) : rows_fwd_h<CF, ST, false, 1>(mode, a, s);
}

template <class CF, int ST>
static hipError_t rows_inv(int mode, const Grid2dArgs& a, hipStream_t s) {
  constexpr int G = 64 / CF::L;
  const bool few = ((long)a.K * a.ny + G - 1) / G <= kFewRowGroups;
  if constexpr (CF::VA % 2 == 0) {
    if (2 * a.nx == a.Gx)
      return few ? rows_inv_h<CF, ST, true, kRowWaves<CF>>(mode, a, s) : rows_inv_h<CF, ST, true, 1>(mode, a, s);
  }
  return few ? rows_inv_h<CF, ST, false, kRowWaves<CF>>(mode, a, s) : rows_inv_h<CF, ST, false, 1>(mode, a, s);
}

template <class CP, bool TB, bool PAD>
static hipError_t cols(const Grid2dArgs& a, hipStream_t s) {
  static std::atomic<uint64_t> allowed{0};
  const hipError_t e = allow_lds((const void*)k_cols<CP, TB, PAD>, CP::LDS, allowed);
  if (e != hipSuccess) return e;
  const long W = (long)(a.Gx / kStrip) * a.K * a.nc;
  hipLaunchKernelGGL((k_cols<CP, TB, PAD>), dim3(strip_grid(W)), dim3(CP::THREADS), CP::LDS, s, a);
  return hipGetLastError();
}


template <class CF, bool TB, bool PAD>
static hipError_t cols_staged(const Grid2dArgs& a, hipStream_t s) {
  constexpr int NC = 256 / CF::L, NY = PAD ? CF::N / 2 : CF::N;
  constexpr size_t lds = std::max((size_t)NY * (NC + 1), (size_t)NC * CF::SPAN) * sizeof(float2);
  static_assert(lds <= 64 * 1024, "without leave");
  const long W = (long)(a.Gx / NC) * a.K * a.nc;
  hipLaunchKernelGGL((k_cols_staged<CF, TB, PAD>), dim3(strip_grid(W)), dim3(256), lds, s, a);
  return hipGetLastError();
}

// One application of the normal operator (three passes) with storage ST:
// 0 complex64, 1 bfloat16 maps, 2 bfloat16 maps and planes
template <int ST>
static hipError_t grid_passes(int mode, const Grid2dArgs& a, hipStream_t s) {
  hipError_t e = with_line(a.Gx, [&](auto cf) { return rows_fwd<decltype(cf), ST>(mode, a, s); });
  if (e != hipSuccess) return e;
  if (staged_cols(a.ny, a.Gy == 2 * a.ny)) {
    e = with_line(a.Gy, [&](auto cf) {
      using CF = decltype(cf);
      if constexpr (staged_cols(CF::N / 2, true)) {
        if (a.Gy == 2 * a.ny) return cols_staged<CF, ST == 2, true>(a, s);
      }
      if constexpr (staged_cols(CF::N, false)) {
        if (a.Gy == a.ny) return cols_staged<CF, ST == 2, false>(a, s);
      }
      return hipErrorInvalidValue;
    });
  } else e = with_col(a.ny, [&](auto cp) {
    using CP = decltype(cp);
    // padded lines have 64 to 768 points, unpadded ones (2-D masks) too
    if constexpr (CP::N <= 384 && !staged_cols(CP::N, true)) {
      if (a.Gy == 2 * a.ny) return cols<CP, ST == 2, true>(a, s);
    }
    if constexpr (CP::N >= 64 && CP::N != 80 && CP::N != 144 && !staged_cols(CP::N, false)) {
      if (a.Gy == a.ny) return cols<CP, ST == 2, false>(a, s);
    }
    return hipErrorInvalidValue;
  });
  if (e != hipSuccess) return e;
  return with_line(a.Gx, [&](auto cf) { return rows_inv<decltype(cf), ST>(mode, a, s); });
}

// Probes per pass.  The planes cross memory four times an iteration (written, column
// pass in place, read); a set of probes whose planes fit the last-level cache (256 MiB,
// less the fields that pass through) goes through all three passes while they are
// there, and every set reuses the same stretch of T.  Of the sets of 96 MiB (below,
// the gaps between the shorter launches show) to 216 MiB that one takes whose row
// launches need the fewest rounds of the chip in all (2048 wavefronts: two per SIMD,
// 256 CUs), the smallest on a tie.
// Solves, one pass / sets of about 208 MiB: 256 x 256 spiral (16 coils, K = 64)
// 18.3 / 15.9 ms, 128 x 128 spiral (20 coils, K = 128) 11.2 / 9.3, 256 x 256 masked (12 coils,
// K = 128) 13.7 / 11.2, 288 x 288 masked (20, K = 64) 15.8 / 14.5; 1706 wavefronts / 3413:
// 160 x 160 spiral (8 coils) 7.2 / 7.5 ms, 320 x 320 masked (8) 13.3 / 13.9; sets of
// 64 MiB are slower than one pass (20.8, 11.6, 17.2, 17.0 ms).
// One pass after all, maps of 10 CG iterations, ms, one pass / sets:
// - planes of up to 256 MiB whose rows are one round: sets only halve the launches (spiral
//   160 x 128, 17 coils, K = 43: 2.32 / 2.72, K = 50, 265 MiB: 2.85 / 2.82; 256 x 256, 16, 14:
//   2.19 / 2.59; masked 192 x 192, 24, 33: 2.13 / 2.40);
// - unpadded lines of 320 points and more that need 1.25 times the rounds in sets (320 x
//   320, 32 coils, K = 32: 9.65 / 10.12; 384, 32, 24: 11.15 / 11.71; 576, 24, 14: 10.96 /
//   12.92; 640, 12, 22: 10.84 / 11.60; 768, 32, 6: 11.17 / 12.46; with fewer rounds 384, 24,
//   24: 8.46 / 8.06; shorter lines 256, 24, 40: 5.37 / 4.83; padded 256, 32, 24: 8.23 / 6.95
//   and 320, 32, 14: 9.56 / 8.88).
inline int grid_chunk(int K, int ny, int group, size_t plane, int line, bool pad) {
  const size_t most = 216u << 20, least = 96u << 20;
  if (K * plane <= most) return K;
  const auto rounds = [&](long k) { return (k * ny + group * 2048L - 1) / (group * 2048L); };
  if (K * plane <= (size_t)256 << 20 && rounds(K) == 1) return K;
  const size_t fit = std::max<size_t>(1, most / plane);
  long best = -1;
  int set = (int)fit;
  for (long n = (K + fit - 1) / fit; n <= K; ++n) {
    const long c = (K + n - 1) / n, full = K / c, rest = K - full * c;
    if (best >= 0 && c * plane < least) break;
    const long all = full * rounds(c) + rounds(rest);
    if (best < 0 || all <= best) {
      best = all;
      set = (int)c;
    }
  }
  if (!pad && line >= 320 && 4 * best >= 5 * rounds(K)) return K;
  return set;
}

template <int ST>
static hipError_t grid_normal(int mode, const Grid2dArgs& all, hipStream_t s) {
  const size_t plane = (size_t)all.nc * all.ny * all.Gx * (ST == 2 ? 4 : 8), n = (size_t)all.ny * all.nx;
  int chunk = 0;
  const hipError_t known = with_line(all.Gx, [&](auto cf) {
    chunk = grid_chunk(all.K, all.ny, 64 / decltype(cf)::L, plane, all.Gx, all.Gy == 2 * all.ny);
    return hipSuccess;
  });
  if (known != hipSuccess) return known;
  for (int k0 = 0; k0 < all.K; k0 += chunk) {
    Grid2dArgs a = all;
    a.k0 = k0;
    a.K = std::min(chunk, all.K - k0);
    for (float2** f : {&a.x, &a.r, &a.p, &a.q})
      if (*f) *f += k0 * n;
    if (a.src) a.src += k0 * n;
    if (a.alpha) a.alpha += k0;
    if (a.beta) a.beta += k0;
    if (a.part) a.part += (size_t)k0 * a.ny * 4;
    const hipError_t e = grid_passes<ST>(mode, a, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace pico
