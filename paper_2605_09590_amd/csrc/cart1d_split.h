// Phase-encode normal operator, split by residue classes of the frequencies:
// kernel templates, one translation unit per split factor.  Conventions as in
// cart1d_normal.h: one plain transform along y per image column and coil, weight
// mask[k] / ny, maps with (-1)^y folded in.
//
// Split factor S.  Frequencies k = S j + rho form S classes, and class rho of
// the transform of x is the ny/S-point transform of the fold
//   z[y'] = sum_t W_ny^{rho (y' + t ny/S)} x[y' + t ny/S],   y' < ny/S.
// Parallel-imaging masks (every R-th line plus a calibration block) leave few
// classes partly sampled.  An empty class contributes nothing.  A fully sampled
// one needs no transform: fold and unfold give
//   q[y' + t ny/S] += sum_t' g[t - t'] (sum_c conj(S_c) S_c)(t, t') p[y' + t' ny/S],
// an S x S Hermitian block per y'.  Only the partly sampled class goes through
// transforms, and the operator's maps carry its phase W_ny^{rho y} (in the blocks it
// turns g by a constant).  R = 2 with a calibration block is one 160-point pair per
// coil instead of a 320-point one, and uniform sampling none.
//
// The blocks are not held in memory (8 S ny nx bytes beyond the operator's described
// size): every workgroup sums its column's over the coils, in FP64, into the LDS that
// the maps took.  With transforms the sums are taken from the staged maps as they
// pass; the wavefronts of a workgroup share them.  Blocks held in memory and this, ms
// (map of 20 CG iterations, K = 96, 12 coils, 128 columns): R = 2 + 24 lines 1.78 / 1.79
// (320 points), 0.55 / 0.57 (64), uniform R = 2 0.98 / 1.06 and 0.26 / 0.29.  Summed by
// every wavefront for itself, from memory, 320 x 320 x 15 with K = 256 took 1.08 times
// as long as with held blocks (now 1.02).
//
// Layout: every per-probe field is stored column-major, [K][nx][ny], so a
// column is one contiguous line; maps are [nx][nc][ny].  A wavefront works on 64 / LA
// probes of one image column, whose maps it stages through LDS.  A transform of N = LA VA points runs as in colpass.h, in two register
// steps with one LDS exchange, dealt to lanes as tasks: LA per probe in layout A
// (points a + LA m), VA in layout B (frequencies k + VA r), where the forward and
// inverse transforms meet in registers.
//
// Bound by the vector ALU (FP32, not packed) with the CG fields' traffic close
// behind: 320 x 320 x 15 coils, R = 2 + 24 calibration lines, K = 256, one CG
// iteration 0.55 ms (VALU instructions issued in 92 % of the cycles; the eight
// fields read and written, 1.7 GB, take 0.36 ms at the copy rate) against 0.79 ms
// unsplit.
#pragma once

#include <type_traits>

#include "colpass.h"
#include "fft.h"
#include "runtime.h"

namespace pico {

// probes per wavefront
template <class CP> constexpr int kFoldProbes = 64 / CP::LA;

// Map column of N values into an LDS buffer, straight from global memory (16
// bytes per lane and instruction, no registers held; N even, so whole pairs);
// wait_lds_loads() comes before the first read
template <int N>
__device__ __forceinline__ void stage_column(const float2* src, float2* dst) {
  wait_lds_reads();
  const int lo = 2 * (int)(threadIdx.x % 64);
#pragma unroll
  for (int j = 0; j < N; j += 128)
    if (j + lo < N)
      __builtin_amdgcn_global_load_lds((const void*)(src + j + lo),
                                       (__attribute__((address_space(3))) void*)(dst + j), 16, 0, 0);
}

// FULL: 0 without a fully sampled class, else the wavefronts that share a workgroup's
// blocks; TR: with a class to transform
template <class CP, int S, int MODE, int FULL, bool TR>
__global__ __launch_bounds__(64 * (FULL > 1 ? FULL : 1), S * CP::VA <= 20 && (FULL != 1 || !TR) ? 3 : 2) void k_cart1d_split(Cart1dArgs a) {
  constexpr int NW = FULL > 1 ? FULL : 1;
  constexpr int LA = CP::LA, VA = CP::VA, N = CP::N, NY = N * S, G = kFoldProbes<CP>;
  static_assert(LA >= VA && LA <= 32, "layout B's tasks fit the lanes, their frequencies a word of mask bits");
  constexpr int STR = LA + 1, SPAN = VA * STR;   // exchange: Y[a][k] at k STR + a (STR odd: conflict-free)
  constexpr int V = S * VA;                      // column values per lane
  constexpr size_t EX = (size_t)G * SPAN * sizeof(float2), RED = 64 * 4 * sizeof(double);
  __shared__ __attribute__((aligned(16))) char ex_raw[NW][(EX > RED ? EX : RED) + 15 & ~15];
  // two map columns a wavefront; then, in the first one's, the blocks: [high, low][S S][N] floats
  __shared__ __attribute__((aligned(16))) float2 map_cols[NW][(S > 2 ? S : 2) * NY];
  const int wave = NW > 1 ? threadIdx.x / 64 : 0, tid = NW > 1 ? threadIdx.x % 64 : threadIdx.x;
  const int la = tid % LA, col = blockIdx.y, k0 = ((int)blockIdx.x * NW + wave) * G, k = k0 + tid / LA;
  float2* ex = reinterpret_cast<float2*>(ex_raw[wave]);
  double* red = reinterpret_cast<double*>(ex_raw[wave]);
  float2* maps = map_cols[wave];
  const bool active = tid < G * LA && k < a.K;
  // layout B's task of this lane
  const int kb = tid % VA;
  const bool activeB = tid < G * VA && k0 + tid / VA < a.K;
  float2* exA = ex + tid / LA * SPAN + la;
  float2* exB = ex + tid / VA * SPAN + kb * STR;

  const int nc = TR && a.rho >= 0 && k0 < a.K ? a.nc : 0;   // coils to transform
  const float2* mcol = a.maps + (size_t)col * a.nc * NY;
  auto stage = [&](int c) { stage_column<NY>(mcol + (size_t)c * NY, maps + (c & 1) * NY); };
  if (nc > 0) stage(0);

  // fully sampled classes: block of y' = y, per row t the real diagonal, then re and im
  // of the columns u > t, summed over the coils for RB values of y per thread: from the
  // staged maps, or from memory where no coil is staged (C coils' loads at once, the
  // first ones' ahead of the CG fields if none is)
  constexpr int T = 64 * NW, RB = (N + T - 1) / T, C = S * RB > 6 ? 2 : S * RB > 3 ? 4 : 8;
  double blk[RB][S * S];
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int j = 0; j < S * S; ++j) blk[r][j] = 0.0;
  auto block_add = [](double (&b)[S * S], const float2 (&m)[S]) {
    int j = 0;
#pragma unroll
    for (int t = 0; t < S; ++t) {
      const double x = m[t].x, y = m[t].y;
      b[j++] += x * x + y * y;
#pragma unroll
      for (int u = t + 1; u < S; ++u, j += 2) {
        b[j] += x * m[u].x + y * m[u].y;
        b[j + 1] += x * m[u].y - y * m[u].x;
      }
    }
  };

  float2 bm[C][RB][S];
  auto block_maps = [&](int c0) {   // in-bounds loads on every lane; a coil past the last is not used
#pragma unroll
    for (int h = 0; h < C; ++h)
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int t = 0; t < S; ++t)
          bm[h][r][t] = mcol[(size_t)min(c0 + h, a.nc - 1) * NY + t * N + min((int)threadIdx.x + T * r, N - 1)];
  };
  if constexpr (FULL && !TR) block_maps(0);

  float2 tw[VA];
#pragma unroll
  for (int j = 0; j < VA; ++j) tw[j] = a.twt[S * la * j];

  // value i = t VA + m of this lane: y = la + LA m + t N
  auto pos = [&](int i) { return la + LA * (i % VA) + (i / VA) * N; };
  const size_t base = ((size_t)(active ? k : 0) * a.nx + col) * NY;
  float2* __restrict__ X = a.x;
  float2* __restrict__ R = a.r;
  float2* __restrict__ P = a.p;
  const float2* __restrict__ Q = a.q;
  float2 pv[V];
  double d[4] = {0.0, 0.0, 0.0, 0.0};
  if (active) {
    if constexpr (MODE == C1_FIRST_PROBE) {
#pragma unroll
      for (int i = 0; i < V; ++i) {
        pv[i] = draw_probe(arg_seed(a), arg_first(a) + k, (uint32_t)(pos(i) * a.nx + col), 0u, a.dist);
        R[base + pos(i)] = pv[i];
        P[base + pos(i)] = pv[i];
      }
    } else if constexpr (MODE == C1_FIRST_BUF) {
#pragma unroll
      for (int i = 0; i < V; ++i) pv[i] = R[base + pos(i)];
#pragma unroll
      for (int i = 0; i < V; ++i) P[base + pos(i)] = pv[i];
    } else if constexpr (MODE == C1_ITER) {
      // finish iteration i-1 and start iteration i: x += alpha p, r -= alpha q,
      // p = r + beta p; every load of a chunk of H elements goes out before the
      // chunk's first store
      const float alpha = (float)a.alpha[k], beta = (float)a.beta[k];
      const bool xz = a.x_zero != 0;
      constexpr int H = V > 8 ? 8 : V;
#pragma unroll
      for (int i0 = 0; i0 < V; i0 += H) {
        float2 po[H], qo[H], ro[H], xo[H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
          if (i0 + h >= V) break;
          const size_t i = base + pos(i0 + h);
          po[h] = P[i];
          qo[h] = Q[i];
          ro[h] = R[i];
          xo[h] = X[i];
        }
#pragma unroll
        for (int h = 0; h < H; ++h) {
          if (i0 + h >= V) break;
          const size_t i = base + pos(i0 + h);
          const float2 rn = cfma(ro[h], -alpha, qo[h]);
          pv[i0 + h] = cfma(rn, beta, po[h]);
          X[i] = cfma(xz ? make_float2(0.f, 0.f) : xo[h], alpha, po[h]);
          R[i] = rn;
          P[i] = pv[i0 + h];
          d[0] += (double)rn.x * rn.x + (double)rn.y * rn.y;
        }
      }
    } else {  // C1_APPLY
#pragma unroll
      for (int i = 0; i < V; ++i) pv[i] = cscale(a.src[base + pos(i)], a.scale);
    }
    if constexpr (MODE == C1_FIRST_PROBE || MODE == C1_FIRST_BUF) {
#pragma unroll
      for (int i = 0; i < V; ++i) d[0] += (double)pv[i].x * pv[i].x + (double)pv[i].y * pv[i].y;
    }
  }

  float2 qa[V];   // coil sum of the transforms, unscaled
#pragma unroll
  for (int i = 0; i < V; ++i) qa[i] = make_float2(0.f, 0.f);
  wait_lds_loads();
  wave_sync();
  int on = 0;   // sampled frequencies of layout B's task
  if (nc > 0) {
#pragma unroll
    for (int r = 0; r < LA; ++r) on |= (a.maskw[S * (kb + VA * r) + a.rho] != 0.f ? 1 : 0) << r;
  }
  for (int c = 0; c < nc; ++c) {
    if (c + 1 < nc) stage(c + 1);   // the buffer of map c - 1, whose last use is behind
    const float2* mv = maps + (c & 1) * NY;
    if constexpr (FULL) {
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const int y = (int)threadIdx.x + T * r;
        if (y >= N) break;
        float2 m[S];
#pragma unroll
        for (int t = 0; t < S; ++t) m[t] = mv[t * N + y];
        block_add(blk[r], m);
      }
    }
    asm volatile("" : "+v"(on));   // opaque: LA unpacked masks held over the loop would spill
    if (active) {
      float2 z[VA];
#pragma unroll
      for (int m = 0; m < VA; ++m) {
        z[m] = cmul(mv[pos(m)], pv[m]);
#pragma unroll
        for (int t = 1; t < S; ++t) z[m] = cadd(z[m], cmul(mv[pos(t * VA + m)], pv[t * VA + m]));
      }
      dft<VA, false>(z);
#pragma unroll
      for (int j = 0; j < VA; ++j) exA[j * STR] = j ? cmul(z[j], tw[j]) : z[j];
    }
    wave_sync();
    if (activeB) {
      float2 b[LA];
#pragma unroll
      for (int i = 0; i < LA; ++i) b[i] = exB[i];
      dft<LA, false>(b);
#pragma unroll
      for (int r = 0; r < LA; ++r) {   // off the mask: zero, whatever the value
        const int m = __builtin_amdgcn_sbfe(on, r, 1);
        b[r].x = __int_as_float(__float_as_int(b[r].x) & m);
        b[r].y = __int_as_float(__float_as_int(b[r].y) & m);
      }
      dft<LA, true>(b);
#pragma unroll
      for (int i = 0; i < LA; ++i) exB[i] = b[i];   // the task's own values
    }
    wait_lds_loads();
    wave_sync();
    if (active) {
      float2 z[VA];
#pragma unroll
      for (int j = 0; j < VA; ++j) z[j] = j ? cmulc(tw[j], exA[j * STR]) : exA[0];
      dft<VA, true>(z);
#pragma unroll
      for (int i = 0; i < V; ++i) qa[i] = cadd(qa[i], cmulc(mv[pos(i)], z[i % VA]));
    }
  }

  if constexpr (FULL) {
    if (nc == 0) {
      for (int c0 = 0; c0 < a.nc; c0 += C) {
        if (TR || c0 > 0) block_maps(c0);
#pragma unroll
        for (int h = 0; h < C; ++h) {
          if (c0 + h >= a.nc) break;
#pragma unroll
          for (int r = 0; r < RB; ++r) block_add(blk[r], bm[h][r]);
        }
      }
    }
    __syncthreads();   // every wavefront is done with its maps
    float* blocks = reinterpret_cast<float*>(map_cols[0]);
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const int y = (int)threadIdx.x + T * r;
      if (y >= N) break;
      int j = 0;
      auto put = [&](double v) {
        const float hi = (float)v;
        blocks[j * N + y] = hi;
        blocks[(S * S + j) * N + y] = (float)(v - (double)hi);
        ++j;
      };
#pragma unroll
      for (int t = 0; t < S; ++t) {
        put(a.full[0].x * blk[r][j]);
#pragma unroll
        for (int u = t + 1; u < S; ++u) {   // t - u < 0: the conjugate of the weight at u - t
          const double2 g = a.full[u - t];
          const double re = blk[r][j], im = blk[r][j + 1];
          put(g.x * re + g.y * im);
          put(g.x * im - g.y * re);
        }
      }
    }
    __syncthreads();
  }
  if (active) {
    // q = lam p + transforms / ny + the fully sampled classes
    constexpr float inv = 1.0f / NY;
#pragma unroll
    for (int i = 0; i < V; ++i) qa[i] = cfma(cscale(qa[i], inv), a.lam, pv[i]);
    if constexpr (FULL) {
      // blocks as high and low words: one rounded block per pixel would not
      // average out as the transforms' errors do (FP64 products spill)
#pragma unroll
      for (int m = 0; m < VA; ++m)
#pragma unroll
        for (int w = 1; w >= 0; --w) {
          const float* b = reinterpret_cast<float*>(map_cols[0]) + w * (S * S) * N + la + LA * m;
          int j = 0;
#pragma unroll
          for (int t = 0; t < S; ++t) {
            qa[t * VA + m] = cfma(qa[t * VA + m], b[j++ * N], pv[t * VA + m]);
#pragma unroll
            for (int u = t + 1; u < S; ++u) {   // B[t][u] and its conjugate B[u][t]
              const float2 g = make_float2(b[j * N], b[(j + 1) * N]);
              j += 2;
              qa[t * VA + m] = cadd(qa[t * VA + m], cmul(g, pv[u * VA + m]));
              qa[u * VA + m] = cadd(qa[u * VA + m], cmulc(g, pv[t * VA + m]));
            }
          }
        }
    }
#pragma unroll
    for (int i = 0; i < V; ++i) {
      a.q[base + pos(i)] = qa[i];
      d[1] += (double)pv[i].x * qa[i].x + (double)pv[i].y * qa[i].y;
      d[2] += (double)qa[i].x * qa[i].x + (double)qa[i].y * qa[i].y;
    }
    if constexpr (MODE == C1_ITER) {
      // r for Re r^H q is read again: held through the coil loop it would cost
      // the third wavefront per SIMD
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const float2 r = R[base + pos(i)];
        d[3] += (double)r.x * qa[i].x + (double)r.y * qa[i].y;
      }
    } else if constexpr (MODE != C1_APPLY) {
      d[3] = d[1];   // r = p
    }
  }
  // sums over the probe's LA lanes, each in lane order
  wave_sync();
#pragma unroll
  for (int j = 0; j < 4; ++j) red[tid * 4 + j] = d[j];
  wave_sync();
  if (active && la < 4) {
    double s = 0.0;
    for (int i = 0; i < LA; ++i) s += red[(tid - la + i) * 4 + la];
    a.part[((size_t)k * a.nx + col) * 4 + la] = s;
  }
}

// ------------------------------------------------------------ dispatch
// Wavefronts that share a column's blocks: as many as have rows of them (64 each), up to
// what fits 64 KiB of LDS
template <class CP, int S>
constexpr int kBlockWaves = CP::N <= 64 ? 1 : CP::N <= 128 ? 2 :
    (kFoldProbes<CP> * CP::VA * (CP::LA + 1) + (S > 2 ? S : 2) * S * CP::N) * 8 * 4 <= 64 * 1024 ? 4 : 2;

template <int S, class CP, int FULL, bool TR>
static hipError_t split_modes(int mode, const Cart1dArgs& a, hipStream_t s) {
  constexpr int NW = FULL > 1 ? FULL : 1, G = kFoldProbes<CP> * NW;
  const dim3 grid((a.K + G - 1) / G, a.nx), block(64 * NW);
  switch (mode) {
    case C1_FIRST_PROBE: hipLaunchKernelGGL((k_cart1d_split<CP, S, C1_FIRST_PROBE, FULL, TR>), grid, block, 0, s, a); break;
    case C1_FIRST_BUF: hipLaunchKernelGGL((k_cart1d_split<CP, S, C1_FIRST_BUF, FULL, TR>), grid, block, 0, s, a); break;
    case C1_ITER: hipLaunchKernelGGL((k_cart1d_split<CP, S, C1_ITER, FULL, TR>), grid, block, 0, s, a); break;
    case C1_APPLY: hipLaunchKernelGGL((k_cart1d_split<CP, S, C1_APPLY, FULL, TR>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int S, class CP>
static hipError_t split_launch(int mode, const Cart1dArgs& a, hipStream_t s) {
  static_assert(CP::LA == split_lanes(S, S * CP::N), "the plan of this length");
  constexpr int NW = kBlockWaves<CP, S>;
  if (a.full[0].x == 0.0) return split_modes<S, CP, 0, true>(mode, a, s);
  const bool share = a.K > kFoldProbes<CP> * (NW - 1);   // a workgroup's wavefronts all have probes
  if (a.rho < 0) return share ? split_modes<S, CP, NW, false>(mode, a, s) : split_modes<S, CP, 1, false>(mode, a, s);
  if constexpr (S > 1) return share ? split_modes<S, CP, NW, true>(mode, a, s) : split_modes<S, CP, 1, true>(mode, a, s);
  return hipErrorInvalidValue;   // S = 1 has a single class
}

}  // namespace pico
