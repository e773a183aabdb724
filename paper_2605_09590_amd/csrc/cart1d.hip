// Separable Cartesian SENSE: launch of the normal operator (kernels in
// cart1d_normal.h, with cart1d_bf16.hip holding the bfloat16-map instantiation,
// and cart1d_split.h) and the CG building blocks of the column-major layout.
#include "cart1d_normal.h"

#include <cmath>

namespace pico {

bool cart1d_supported(int ny) {
  switch (ny) {
    case 64: case 96: case 128: case 160: case 192: case 256: case 288: case 320: case 384: case 512:
      return true;
    default:
      return false;
  }
}

// Launches with fewer split wavefronts than SIMDs (1024) whose class to transform makes
// them slower than whole columns, which put more lanes on a probe: one wavefront's
// time counts then.  Maps of 20 CG iterations, 12 coils, R = 2 (384*: R = 4, S = 1) + 24
// lines, 128 columns, us, whole columns / split, K in brackets:
// - a last wavefront at most half full: 64 [1] 404 / 433, [4] 416 / 440, [5] 413 / 402; 192
//   [2] 636 / 679, [3] 634 / 604; 256 (S = 1) [2] 768 / 883, [3] 774 / 754, [6] 780 / 865; 288
//   [2] 829 / 879, [3] 834 / 782; 320 [2] 790 / 891, [4] 800 / 793, [5] 805 / 859; 384 [2]
//   860 / 970, [4] 870 / 864, [5] 905 / 936;
// - any: 128 [8] 559 / 573, [32] 614 / 639, [48: 768 wavefronts] 714 / 696; 160 [12] 647 / 673,
//   [16] 655 / 690, [48: 1024] 842 / 786; 384* [2] 859 / 906, [16: 1024] 1042 / 1051, [32] 1293 /
//   1272; 512 [1] 526 / 1273, [16] 812 / 1176, [28: 896] 1361 / 1385, [40] 1564 / 1529.
static bool whole_columns(const Cart1dArgs& a) {
  if (a.rho < 0 || a.split == 3 || a.ny == 96) return false;   // 96: 937 / 532 at [4]
  const int probes = 64 / split_lanes(a.split, a.ny), last = a.K % probes;
  const long waves = (long)a.nx * ((a.K + probes - 1) / probes);
  if (waves >= 1024) return false;
  if (last > 0 && 2 * last <= probes) return true;
  if (a.split == 1) return a.ny == 384;
  return a.ny == 160 || a.ny == 512 || (a.ny == 128 && waves <= 512);
}

hipError_t launch_cart1d(int mode, const Cart1dArgs& a, hipStream_t s) {
  if (mode != C1_PMR_RHS && !((a.split > 1 || unsplit_in_split_kernel(a.ny)) && whole_columns(a))) {
    if (a.split == 2) return launch_cart1d_split2(mode, a, s);
    if (a.split == 3) return launch_cart1d_split3(mode, a, s);
    if (unsplit_in_split_kernel(a.ny)) return launch_cart1d_split1(mode, a, s);
  }
  if (a.maps_bf) return launch_cart1d_bf16(mode, a, s);
  return cart1d_dispatch<false>(mode, a, s);
}

// ------------------------------------------------------------ split factor
// The split with the least transform work, at most one partly sampled class
// (whose phase the maps carry): none where every class is full or empty,
// else one class of ny / S frequencies.  Measured per noise map (12 coils, 128
// columns, K = 96, CG 20, ms): R = 2 + 24 calibration lines, S = 2, against
// unsplit 2.37 -> 1.79 (320 points), 2.02 -> 1.50 (256), 3.36 -> 2.36 (384),
// 1.12 -> 0.90 (128), 0.65 -> 0.57 (64); uniform R = 2 2.46 -> 1.06 (320), 0.64
// -> 0.29 (64).  Few probes gain least: 320 points, K = 32 1.19 -> 1.03, K = 12 0.88 ->
// 0.89.  R = 3 with calibration lines leaves two classes of S = 3, which
// ran slower than unsplit (CG 6: 192 points 0.88 -> 1.17, 288 1.51 -> 1.54).
Fold fold_of(const uint8_t* mask, int ny) {
  Fold best;
  for (int s = 1; s <= 3; ++s) {
    if (ny % s || (s == 3 && ny != 96 && ny != 192 && ny != 288 && ny != 384)) continue;   // built splits
    Fold f;
    f.split = s;
    for (int rho = 0; rho < s; ++rho) {
      int on = 0;
      for (int k = rho; k < ny; k += s) on += mask[k] != 0;
      if (on == ny / s) f.full.push_back(rho);
      else if (on > 0) f.part.push_back(rho);
    }
    // a later split is better if it leaves fewer frequencies to transform
    if (f.part.size() > 1) continue;
    if (s == 1 || f.part.size() * (size_t)(ny / s) < best.part.size() * (size_t)(ny / best.split)) best = f;
  }
  return best;
}

double2 Fold::full_weight(int d) const {
  const int at = part.empty() ? 0 : part[0];
  double2 g = make_double2(0.0, 0.0);
  for (int rho : full) {
    const double ang = 2.0 * kPi * (double)((rho - at) * d % split) / split;
    g.x += std::cos(ang) / split;
    g.y += std::sin(ang) / split;
  }
  return g;
}

// ------------------------------------------------------------ map preparation
__device__ __forceinline__ void class_phase(int rho, int y, int ny, double& c, double& s) {   // W_ny^{rho y}
  sincospi(-2.0 * (double)((long)rho * y % ny) / ny, &s, &c);
}

// out[col][c][y] = (-1)^y W_ny^{rho y} sum_d Linv[c][d] maps[d][y][col]  (whitening,
// Sec. 2.1 Eq. (3); the factor of the split form, rounded once with the rest)
__global__ void k_prep_maps_cart1d(const float2* __restrict__ maps, const double* __restrict__ linv,
                                   float2* __restrict__ out, int nc, int ny, int nx, int rho) {
  const int y = blockIdx.x * blockDim.x + threadIdx.x;
  const int col = blockIdx.y;
  if (y >= ny) return;
  const double sg = (y & 1) ? -1.0 : 1.0;
  double pc = 1.0, ps = 0.0;
  if (rho > 0) class_phase(rho, y, ny, pc, ps);
  for (int c = 0; c < nc; ++c) {
    double re = 0.0, im = 0.0;
    for (int d = 0; d <= c; ++d) {
      const double lr = linv[2 * (c * nc + d)], li = linv[2 * (c * nc + d) + 1];
      const float2 m = maps[((size_t)d * ny + y) * nx + col];
      re += lr * m.x - li * m.y;
      im += lr * m.y + li * m.x;
    }
    if (rho > 0) {
      const double t = re * pc - im * ps;
      im = re * ps + im * pc;
      re = t;
    }
    out[((size_t)col * nc + c) * ny + y] = make_float2((float)(sg * re), (float)(sg * im));
  }
}

hipError_t launch_prep_maps_cart1d(const float2* maps, const double* linv, float2* out, int nc,
                                   int ny, int nx, int rho, hipStream_t s) {
  dim3 grid((ny + 63) / 64, nx), block(64);
  hipLaunchKernelGGL(k_prep_maps_cart1d, grid, block, 0, s, maps, linv, out, nc, ny, nx, rho);
  return hipGetLastError();
}

__global__ void k_phase_maps_cart1d(float2* __restrict__ maps, long total, int ny, int rho) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  double c, s;
  class_phase(rho, (int)(i % ny), ny, c, s);
  const double re = maps[i].x, im = maps[i].y;
  maps[i] = make_float2((float)(re * c - im * s), (float)(re * s + im * c));
}

hipError_t launch_phase_maps_cart1d(float2* maps, int nc, int ny, int nx, int rho, hipStream_t s) {
  const long total = (long)nx * nc * ny;
  hipLaunchKernelGGL(k_phase_maps_cart1d, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, maps, total, ny, rho);
  return hipGetLastError();
}

// ------------------------------------------------------------ power-method start
__global__ void k_power_start(float2* __restrict__ p, int ny, int nx) {
  const int y = blockIdx.x * blockDim.x + threadIdx.x;
  const int col = blockIdx.y;
  if (y >= ny) return;
  const float s = rsqrtf((float)ny * (float)nx);
  const float2 v = draw_probe(0, 0, (uint32_t)(y * nx + col), 3u, 0);
  p[(size_t)col * ny + y] = cscale(v, s);
}

hipError_t launch_power_start(float2* p, int ny, int nx, hipStream_t s) {
  dim3 grid((ny + 63) / 64, nx), block(64);
  hipLaunchKernelGGL(k_power_start, grid, block, 0, s, p, ny, nx);
  return hipGetLastError();
}

// ------------------------------------------------------------ exact diagonal by row probing
// For a phase-encode mask Sigma is block diagonal over image columns, so the
// probe that is 1 on image row y0 + k of every column returns column x's
// Sigma_x e_(y0+k): its entry on that row is diag(Sigma) there.
__global__ void k_unit_rows(float2* __restrict__ r, int y0, int ny, int nx) {
  const int y = blockIdx.x * blockDim.x + threadIdx.x;
  const int col = blockIdx.y, k = blockIdx.z;
  if (y >= ny) return;
  r[((size_t)k * nx + col) * ny + y] = make_float2(y == y0 + k ? 1.f : 0.f, 0.f);
}

__global__ void k_extract_rows(const float2* __restrict__ x, double* __restrict__ var, int K, int y0,
                               int ny, int nx) {
  const int col = blockIdx.x * blockDim.x + threadIdx.x;
  const int k = blockIdx.y;
  if (col >= nx || k >= K) return;
  const int y = y0 + k;
  var[(size_t)y * nx + col] = (double)x[((size_t)k * nx + col) * ny + y].x;
}

hipError_t launch_unit_rows(float2* r, int K, int y0, int ny, int nx, hipStream_t s) {
  dim3 grid((ny + 63) / 64, nx, K), block(64);
  hipLaunchKernelGGL(k_unit_rows, grid, block, 0, s, r, y0, ny, nx);
  return hipGetLastError();
}

hipError_t launch_extract_rows(const float2* x, double* var, int K, int y0, int ny, int nx,
                               hipStream_t s) {
  dim3 grid((nx + 63) / 64, K), block(64);
  hipLaunchKernelGGL(k_extract_rows, grid, block, 0, s, x, var, K, y0, ny, nx);
  return hipGetLastError();
}

// ------------------------------------------------------------ layout changes
// v [K][ny][nx] (row-major images) -> out [K][nx][ny]
__global__ void k_transpose_in(const float2* __restrict__ v, float2* __restrict__ out, int ny, int nx) {
  __shared__ float2 tile[32][33];
  const int k = blockIdx.z;
  const int x0 = blockIdx.x * 32, y0 = blockIdx.y * 32;
  const float2* vk = v + (size_t)k * ny * nx;
  float2* ok = out + (size_t)k * ny * nx;
  for (int i = threadIdx.y; i < 32; i += 8) {
    const int y = y0 + i, x = x0 + threadIdx.x;
    if (y < ny && x < nx) tile[i][threadIdx.x] = vk[(size_t)y * nx + x];
  }
  __syncthreads();
  for (int i = threadIdx.y; i < 32; i += 8) {
    const int x = x0 + i, y = y0 + threadIdx.x;
    if (y < ny && x < nx) ok[(size_t)x * ny + y] = tile[threadIdx.x][i];
  }
}

// x [K][nx][ny] -> u [K][ny][nx]
__global__ void k_transpose_out(const float2* __restrict__ x, float2* __restrict__ u, int ny, int nx) {
  __shared__ float2 tile[32][33];
  const int k = blockIdx.z;
  const int x0 = blockIdx.x * 32, y0 = blockIdx.y * 32;
  const float2* xk = x + (size_t)k * ny * nx;
  float2* uk = u + (size_t)k * ny * nx;
  for (int i = threadIdx.y; i < 32; i += 8) {
    const int x = x0 + i, y = y0 + threadIdx.x;
    if (y < ny && x < nx) tile[i][threadIdx.x] = xk[(size_t)x * ny + y];
  }
  __syncthreads();
  for (int i = threadIdx.y; i < 32; i += 8) {
    const int y = y0 + i, xx = x0 + threadIdx.x;
    if (y < ny && xx < nx) uk[(size_t)y * nx + xx] = tile[threadIdx.x][i];
  }
}

hipError_t launch_transpose_in(const float2* v, float2* out, int K, int ny, int nx, hipStream_t s) {
  dim3 grid((nx + 31) / 32, (ny + 31) / 32, K), block(32, 8);
  hipLaunchKernelGGL(k_transpose_in, grid, block, 0, s, v, out, ny, nx);
  return hipGetLastError();
}

hipError_t launch_transpose_out(const float2* x, float2* u, int K, int ny, int nx, hipStream_t s) {
  dim3 grid((nx + 31) / 32, (ny + 31) / 32, K), block(32, 8);
  hipLaunchKernelGGL(k_transpose_out, grid, block, 0, s, x, u, ny, nx);
  return hipGetLastError();
}

}  // namespace pico
