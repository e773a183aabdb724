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
// an S x S Hermitian block per y' summed over the coils once per operator
// (fgram).  Only partly sampled classes go through transforms, on maps that carry
// W_ny^{rho y} (fmaps).  R = 2 with a calibration block is one 160-point pair per
// coil instead of a 320-point one, and uniform sampling none.
//
// Layout: every per-probe field is stored column-major, [K][nx][ny], so a
// column is one contiguous line; maps are [nx][nc][ny].  A workgroup is one
// wavefront on 64 / LA probes of one image column, whose maps it stages through
// LDS.  A transform of N = LA VA points runs as in colpass.h, in two register
// steps with one LDS exchange, dealt to lanes as tasks: LA per probe in layout A
// (points a + LA m), VA in layout B (frequencies k + VA r), where the forward and
// inverse transforms meet in registers.
//
// Bound by the vector ALU (FP32, not packed) with the CG fields' traffic close
// behind: 320 x 320 x 15 coils, R = 2 + 24 calibration lines, K = 256, one CG
// iteration 0.53 ms (VALU 82 % busy; the eight fields read and written, 1.7 GB,
// take 0.36 ms at the copy rate) against 0.79 ms unsplit.
#pragma once

#include <type_traits>

#include "colpass.h"
#include "fft.h"
#include "runtime.h"

namespace pico {

// probes per workgroup of one wavefront
template <class CP> constexpr int kFoldProbes = 64 / CP::LA;

// Map column of N values into an LDS buffer, straight from global memory (16
// bytes per lane and instruction, no registers held; N even, so whole pairs);
// wait_lds_loads() and a barrier come before the first read
template <int N>
__device__ __forceinline__ void stage_column(const float2* src, float2* dst) {
  wait_lds_reads();
  const int lo = 2 * (int)threadIdx.x;
#pragma unroll
  for (int j = 0; j < N; j += 128)
    if (j + lo < N)
      __builtin_amdgcn_global_load_lds((const void*)(src + j + lo),
                                       (__attribute__((address_space(3))) void*)(dst + j), 16, 0, 0);
}

template <class CP, int S, int MODE>
__global__ __launch_bounds__(64, S * CP::VA <= 20 ? 3 : 2) void k_cart1d_split(Cart1dArgs a) {
  constexpr int LA = CP::LA, VA = CP::VA, N = CP::N, NY = N * S, G = kFoldProbes<CP>;
  static_assert(LA >= VA && LA <= 32, "layout B's tasks fit the lanes, their frequencies a word of mask bits");
  constexpr int STR = LA + 1, SPAN = VA * STR;   // exchange: Y[a][k] at k STR + a (STR odd: conflict-free)
  constexpr int V = S * VA;                      // column values per lane
  constexpr size_t EX = (size_t)G * SPAN * sizeof(float2), RED = 64 * 4 * sizeof(double);
  __shared__ __attribute__((aligned(16))) char ex_raw[EX > RED ? EX : RED];
  __shared__ __attribute__((aligned(16))) float2 maps[2 * NY];   // two deep
  float2* ex = reinterpret_cast<float2*>(ex_raw);
  double* red = reinterpret_cast<double*>(ex_raw);
  const int tid = threadIdx.x, la = tid % LA, col = blockIdx.y;
  const int k = blockIdx.x * G + tid / LA;
  const bool active = tid < G * LA && k < a.K;
  // layout B's task of this lane
  const int kb = tid % VA;
  const bool activeB = tid < G * VA && (int)blockIdx.x * G + tid / VA < a.K;
  float2* exA = ex + tid / LA * SPAN + la;
  float2* exB = ex + tid / VA * SPAN + kb * STR;

  const int nc = a.rho >= 0 ? a.nc : 0;   // coils to transform
  auto stage = [&](int c) { stage_column<NY>(a.fmaps + ((size_t)col * a.nc + c) * NY, maps + (c & 1) * NY); };
  if (nc > 0) stage(0);

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
  __syncthreads();
  int on = 0;   // sampled frequencies of layout B's task
  if (nc > 0) {
#pragma unroll
    for (int r = 0; r < LA; ++r) on |= (a.maskw[S * (kb + VA * r) + a.rho] != 0.f ? 1 : 0) << r;
  }
  for (int c = 0; c < nc; ++c) {
    if (c + 1 < nc) stage(c + 1);   // the buffer of map c - 1, whose last use is behind
    const float2* mv = maps + (c & 1) * NY;
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
    __syncthreads();
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
    __syncthreads();
    if (active) {
      float2 z[VA];
#pragma unroll
      for (int j = 0; j < VA; ++j) z[j] = j ? cmulc(tw[j], exA[j * STR]) : exA[0];
      dft<VA, true>(z);
#pragma unroll
      for (int i = 0; i < V; ++i) qa[i] = cadd(qa[i], cmulc(mv[pos(i)], z[i % VA]));
    }
  }

  if (active) {
    // q = lam p + transforms / ny + the fully sampled classes
    constexpr float inv = 1.0f / NY;
#pragma unroll
    for (int i = 0; i < V; ++i) qa[i] = cfma(cscale(qa[i], inv), a.lam, pv[i]);
    if (a.fgram) {
      // blocks as high and low words: one rounded block per pixel would not
      // average out as the transforms' errors do (FP64 products spill)
#pragma unroll
      for (int m = 0; m < VA; ++m)
#pragma unroll
        for (int w = 1; w >= 0; --w) {
          const float* b = a.fgram + ((size_t)col * 2 + w) * (S * S) * N + la + LA * m;
          int j = 0;
#pragma unroll
          for (int t = 0; t < S; ++t) {
            qa[t * VA + m] = cfma(qa[t * VA + m], b[(size_t)j++ * N], pv[t * VA + m]);
#pragma unroll
            for (int u = t + 1; u < S; ++u) {   // B[t][u] and its conjugate B[u][t]
              const float2 g = make_float2(b[(size_t)j * N], b[(size_t)(j + 1) * N]);
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
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j) red[tid * 4 + j] = d[j];
  __syncthreads();
  if (active && la < 4) {
    double s = 0.0;
    for (int i = 0; i < LA; ++i) s += red[(tid - la + i) * 4 + la];
    a.part[((size_t)k * a.nx + col) * 4 + la] = s;
  }
}

// ------------------------------------------------------------ dispatch
template <int S, class CP>
static hipError_t split_launch(int mode, const Cart1dArgs& a, hipStream_t s) {
  constexpr int G = kFoldProbes<CP>;
  const dim3 grid((a.K + G - 1) / G, a.nx), block(64);
  switch (mode) {
    case C1_FIRST_PROBE: hipLaunchKernelGGL((k_cart1d_split<CP, S, C1_FIRST_PROBE>), grid, block, 0, s, a); break;
    case C1_FIRST_BUF: hipLaunchKernelGGL((k_cart1d_split<CP, S, C1_FIRST_BUF>), grid, block, 0, s, a); break;
    case C1_ITER: hipLaunchKernelGGL((k_cart1d_split<CP, S, C1_ITER>), grid, block, 0, s, a); break;
    case C1_APPLY: hipLaunchKernelGGL((k_cart1d_split<CP, S, C1_APPLY>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace pico
