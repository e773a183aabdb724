// FP64 normal operator of the compressed-sensing primal (2-D Cartesian masks):
//   M y = sum_c conj(S_c) F^H P F S_c y,
// F the centred orthonormal 2-D DFT.  For even sizes F = (-1)^((ny+nx)/2) D G D /
// sqrt(ny nx), D = diag((-1)^(y+x)) and G the plain DFT: the maps carry D, the
// centred-order mask applies unchanged, and the scale goes into the last pass.
// Three passes of in-register two-step transforms (colpass.h): row transforms of
// S_c y, column transforms with the mask between forward and inverse, inverse row
// transforms with the coil sum.
//
// Bound by the passes over the coil planes (in the last-level cache for a few
// replicas) and by launches: 160 x 160, 8 coils, 8 images take 30 us per
// application; dense DFT products, which this replaces, took four 52 us
// matrix products and 19 us of elementwise passes.
#include "colpass.h"
#include "runtime.h"

namespace pico {

namespace {

// U[b][c][y][.] = row transform of S_c y[b]; one wavefront per 64 / LA rows
template <class CP>
__global__ __launch_bounds__(64) void k_rows64_fwd(const double2* __restrict__ img, const double2* __restrict__ S,
                                                   double2* __restrict__ U, long lines, int nc, int ny,
                                                   const double2* __restrict__ twx) {
  constexpr int LA = CP::LA, VA = CP::VA, N = CP::N, G = 64 / LA, STR = LA + 1, SPAN = VA * STR;
  __shared__ double2 ex[G * SPAN];
  const int tid = threadIdx.x, la = tid % LA, kb = tid % VA;
  const long l0 = (long)blockIdx.x * G, lineA = l0 + tid / LA, lineB = l0 + tid / VA;
  if (tid < G * LA && lineA < lines) {
    const long pl = lineA / ny;   // plane (b, c)
    const int y = (int)(lineA % ny);
    const double2* s = S + ((size_t)(pl % nc) * ny + y) * N + la;
    const double2* x = img + ((size_t)(pl / nc) * ny + y) * N + la;
    double2 v[VA];
#pragma unroll
    for (int m = 0; m < VA; ++m) v[m] = cmul(s[LA * m], x[LA * m]);
    dft<VA, false>(v);
#pragma unroll
    for (int k = 0; k < VA; ++k) ex[tid / LA * SPAN + k * STR + la] = k ? cmul(v[k], twx[la * k]) : v[0];
  }
  __syncthreads();
  if (tid < G * VA && lineB < lines) {
    double2 v[LA];
#pragma unroll
    for (int a = 0; a < LA; ++a) v[a] = ex[tid / VA * SPAN + kb * STR + a];
    dft<LA, false>(v);
    double2* u = U + (size_t)lineB * N + kb;
#pragma unroll
    for (int r = 0; r < LA; ++r) u[VA * r] = v[r];
  }
}

// columns of the planes [planes][ny][nx] in place: forward, mask, inverse, or
// (!PAIR) the inverse transform alone
template <class CP, bool PAIR>
__global__ __launch_bounds__(CP::THREADS) void k_cols64(double2* __restrict__ U, const uint8_t* __restrict__ mask,
                                                        long planes, int nx, const double2* __restrict__ twy) {
  constexpr int LA = CP::LA, VA = CP::VA, N = CP::N, ST = CP::ST;
  extern __shared__ double2 dyn64[];
  const int strips = nx / ST;
  const long vb = strip_of(blockIdx.x, strips * planes);
  if (vb < 0) return;
  const int col = threadIdx.x % ST, t = threadIdx.x / ST;
  const int xc = (int)(vb % strips) * ST + col;
  double2* __restrict__ pl = U + (size_t)(vb / strips) * N * nx + xc;
  double2* ex = dyn64 + col;
  const bool inA = LA == CP::L || t < LA, inB = VA == CP::L || t < VA;
  double2 tw[VA];
  if (inA) {
    double2 x[VA];
#pragma unroll
    for (int m = 0; m < VA; ++m) x[m] = pl[(size_t)(t + LA * m) * nx];
#pragma unroll
    for (int k = 0; k < VA; ++k) tw[k] = twy[t * k];
    col_a_out<CP, !PAIR, false>(x, tw, ex, t);
  }
  __syncthreads();
  if (inB) {
    double2 v[LA];
    col_b_load<CP>(v, ex, t);
    dft<LA, !PAIR>(v);
    if constexpr (PAIR) {
#pragma unroll
      for (int r = 0; r < LA; ++r)
        if (!mask[(size_t)(t + VA * r) * nx + xc]) v[r] = make_double2(0.0, 0.0);
      dft<LA, true>(v);
      col_b_store<CP>(v, ex, t);
    } else {
#pragma unroll
      for (int r = 0; r < LA; ++r) pl[(size_t)(t + VA * r) * nx] = v[r];
    }
  }
  if constexpr (PAIR) {
    __syncthreads();
    if (inA) {
      double2 x[VA];
      col_a_in<CP, true, false>(x, tw, ex, t);
#pragma unroll
      for (int m = 0; m < VA; ++m) pl[(size_t)(t + LA * m) * nx] = x[m];
    }
  }
}

// out[b][y][.] = scale sum_c conj(S_c) (inverse row transform of U[b][c][y]); 64 /
// LA image rows per workgroup, its wavefronts taking every fourth (long rows: every
// second) coil, their sums added in order
template <class CP> constexpr int kRows64Waves = CP::N <= 192 ? 4 : 2;   // LDS below 64 KiB
template <class CP>
__global__ __launch_bounds__(64 * kRows64Waves<CP>) void k_rows64_inv(const double2* __restrict__ U, const double2* __restrict__ S,
                                                    double2* __restrict__ out, long lines, int nc, int ny, double scale,
                                                    const double2* __restrict__ twx) {
  constexpr int LA = CP::LA, VA = CP::VA, N = CP::N, G = 64 / LA, STR = LA + 1, SPAN = VA * STR, NW = kRows64Waves<CP>;
  __shared__ double2 ex_all[NW * G * SPAN];
  const int wave = threadIdx.x / 64, tid = threadIdx.x % 64, la = tid % LA, kb = tid % VA;
  double2* ex = ex_all + wave * G * SPAN;
  const long l0 = (long)blockIdx.x * G, lineA = l0 + tid / LA, lineB = l0 + tid / VA;
  const bool inA = tid < G * LA && lineA < lines, inB = tid < G * VA && lineB < lines;
  const size_t n = (size_t)ny * N;
  const double2* u = U + (size_t)((inA ? lineA : 0) / ny) * nc * n + (size_t)((inA ? lineA : 0) % ny) * N + la;
  const double2* sB = S + (size_t)((inB ? lineB : 0) % ny) * N + kb;
  double2 acc[LA];
#pragma unroll
  for (int r = 0; r < LA; ++r) acc[r] = make_double2(0.0, 0.0);
  double2 tw[VA];
#pragma unroll
  for (int k = 0; k < VA; ++k) tw[k] = twx[la * k];
  for (int c0 = 0; c0 < nc; c0 += NW) {
    const int c = c0 + wave;
    double2 m[LA];   // the coil's maps are on their way during the first step
    if (inB && c < nc) {
#pragma unroll
      for (int r = 0; r < LA; ++r) m[r] = sB[c * n + VA * r];
    }
    if (inA && c < nc) {
      double2 v[VA];
#pragma unroll
      for (int i = 0; i < VA; ++i) v[i] = u[c * n + LA * i];
      dft<VA, true>(v);
#pragma unroll
      for (int k = 0; k < VA; ++k) ex[tid / LA * SPAN + k * STR + la] = k ? cmulc(tw[k], v[k]) : v[0];
    }
    __syncthreads();
    if (inB && c < nc) {
      double2 v[LA];
#pragma unroll
      for (int a = 0; a < LA; ++a) v[a] = ex[tid / VA * SPAN + kb * STR + a];
      dft<LA, true>(v);
#pragma unroll
      for (int r = 0; r < LA; ++r) acc[r] = cadd(acc[r], cmulc(m[r], v[r]));
    }
    __syncthreads();
  }
  // rows of G N values per wavefront, in the exchange's place
  static_assert(N <= SPAN, "a row's sums fit its exchange");
  if (inB) {
#pragma unroll
    for (int r = 0; r < LA; ++r) ex[tid / VA * N + kb + VA * r] = acc[r];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < G * N; i += 64 * NW) {
    if (l0 + i / N >= lines) break;
    double2 s = ex_all[i];
    for (int w = 1; w < NW; ++w) s = cadd(s, ex_all[w * G * SPAN + i]);
    out[(size_t)l0 * N + i] = cscale(s, scale);
  }
}

template <class F>
hipError_t with_line64(int n, F&& f) {   // the grid lengths of a 2-D mask
  return with_col(n, [&](auto cp) {
    using CP = decltype(cp);
    if constexpr (CP::N >= 64 && CP::N != 80 && CP::N != 144) return f(typename CP::Fp64{});
    return hipErrorInvalidValue;
  });
}

template <bool PAIR>
hipError_t cols64(const Cs64& o, long planes, hipStream_t s) {
  return with_line64(o.ny, [&](auto cp) {
    using CP = decltype(cp);
    static std::atomic<uint64_t> allowed{0};
    const hipError_t e = allow_lds((const void*)k_cols64<CP, PAIR>, CP::LDS, allowed);
    if (e != hipSuccess) return e;
    const dim3 grid(strip_grid(planes * (o.nx / CP::ST))), block(CP::THREADS);
    hipLaunchKernelGGL((k_cols64<CP, PAIR>), grid, block, CP::LDS, s, o.U, o.mask, planes, o.nx, o.twy);
    return hipGetLastError();
  });
}

hipError_t rows64_inv(const Cs64& o, int B, double scale, double2* out, hipStream_t s) {
  return with_line64(o.nx, [&](auto cp) {
    using CP = decltype(cp);
    constexpr int G = 64 / CP::LA;
    const long lines = (long)B * o.ny;
    hipLaunchKernelGGL((k_rows64_inv<CP>), dim3((unsigned)((lines + G - 1) / G)), dim3(64 * kRows64Waves<CP>), 0, s, o.U, o.S, out, lines,
                       o.nc, o.ny, scale, o.twx);
    return hipGetLastError();
  });
}

}  // namespace

// q[b] = M y[b] for B images
hipError_t cs64_normal(const Cs64& o, int B, const double2* y, double2* q, hipStream_t s) {
  const long planes = (long)B * o.nc;
  hipError_t e = with_line64(o.nx, [&](auto cp) {
    using CP = decltype(cp);
    constexpr int G = 64 / CP::LA;
    const long lines = planes * o.ny;
    hipLaunchKernelGGL((k_rows64_fwd<CP>), dim3((unsigned)((lines + G - 1) / G)), dim3(64), 0, s, y, o.S, o.U, lines,
                       o.nc, o.ny, o.twx);
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  if ((e = cols64<true>(o, planes, s)) != hipSuccess) return e;
  return rows64_inv(o, B, 1.0 / ((double)o.ny * o.nx), q, s);
}

// out[b] = sum_c conj(S_c) F^H of the k-space times (-1)^(ky+kx) held in o.U [B][nc]
// (overwritten)
hipError_t cs64_adjoint_u(const Cs64& o, int B, double2* out, hipStream_t s) {
  hipError_t e = cols64<false>(o, (long)B * o.nc, s);
  if (e != hipSuccess) return e;
  const double sg = (((o.ny + o.nx) / 2) & 1) ? -1.0 : 1.0;
  return rows64_inv(o, B, sg / sqrt((double)o.ny * o.nx), out, s);
}

}  // namespace pico
