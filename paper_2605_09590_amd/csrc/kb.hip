// Kaiser-Bessel gridding NUFFT for non-Cartesian operators (Sec. 3.2.2, 3.3):
// the data path (A x and A^H y per coil; PMR replicas) and, on request, the
// gridding normal operator A^H A of the CG solves.
//
// Grid G = sigma N per axis, image placed at grid index r mod G (r centred),
// plain 2-D FFT on the grid, W x W separable Kaiser-Bessel taps per sample at
// k = floor(kappa) - W/2 + 1 + t (kappa = w G / 2 pi), de-apodisation by the
// kernel's Fourier transform at r / G, scale N^-1/2.  The adjoint is the
// exact adjoint: spread with the same weights, inverse FFT, crop.
//
// Spread (A^H): every 8 x 8 tile of the grid has a list, made once per operator,
// of the samples whose W x W footprints reach it, and is the contraction of the
// tile's tap weights [64 points][samples] with the sample values [samples]
// [planes], run on the FP32 matrix cores for 16 planes at a time (k_kb_spread).
// Each grid point is written once, by its own tile, and every sum has a fixed
// order, so the spread is deterministic and needs no atomics.  Interpolation (A)
// gathers from an LDS window of the bin's neighbourhood (k_kb_interp).  Around
// both, the row transforms run on the image rows alone and several coils share
// a launch.
//
// Normal operator (A^H A): interpolation followed by the spread is P^H P on
// the grid, a real symmetric operator whose row for grid point g has
// nonzeros only at offsets d in [-(W-1), W-1]^2: S[g][d] = sum_m w_m(g)
// w_m(g + d).  It is built once per operator in FP64 (from the same tap
// tables) and applied per 16 x 16 grid tile with the input window (tile plus
// a W - 1 halo) in LDS and the tile's stencil in registers, for a run of
// probes; tiles that no sample's footprint reaches are written as zeros.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <numeric>
#include <vector>

#include "arena.h"
#include "device_common.h"
#include "runtime.h"

namespace pico {

// ------------------------------------------------------------------ host tables
namespace {

double bessel_i0(double x) {   // power series sum ((x/2)^2)^k / (k!)^2
  const double q = 0.25 * x * x;
  double term = 1.0, s = 1.0;
  for (int k = 1; k < 500; ++k) {
    term *= q / ((double)k * k);
    s += term;
    if (term <= 1e-17 * s) break;
  }
  return s;
}

double kb_phi(double u, int W, double beta) {
  const double a = 1.0 - (2.0 * u / W) * (2.0 * u / W);
  return a >= 0.0 ? bessel_i0(beta * std::sqrt(a)) : 0.0;
}

double kb_phi_hat(double nu, int W, double beta) {   // continuous transform of kb_phi
  const double z2 = beta * beta - (M_PI * W * nu) * (M_PI * W * nu);
  if (z2 > 1e-12) {
    const double z = std::sqrt(z2);
    return W * std::sinh(z) / z;
  }
  if (z2 < -1e-12) {
    const double z = std::sqrt(-z2);
    return W * std::sin(z) / z;
  }
  return W;
}

}  // namespace

double kb_beta(double sigma, int W) {
  return M_PI * std::sqrt((W / sigma) * (W / sigma) * (sigma - 0.5) * (sigma - 0.5) - 0.8);
}

size_t KbLayout::bytes_of(size_t i) const { return sizes[i]; }

KbLayout kb_layout(long M, int W, int ny, int nx, int Gy, int Gx, int K, bool normal) {
  KbLayout L;
  const size_t nb = (size_t)(Gy / kKbTile) * (Gx / kKbTile);
  const size_t s[KbLayout::kParts] = {
      (size_t)M * 4,                       // sky0
      (size_t)M * 4,                       // skx0
      (size_t)M * W * 4,                   // swy
      (size_t)M * W * 4,                   // swx
      (size_t)M * 4,                       // perm
      (nb + (size_t)M / kKbUnit) * 8,      // units: every bin ends at most one short unit
      (size_t)ny * 4,                      // dy
      (size_t)nx * 4,                      // dx
      (size_t)Gx * 8,                      // twiddles x
      (size_t)Gy * 8,                      // twiddles y
      (size_t)K * Gy * Gx * 8,             // grid [K][Gy][Gx]
      normal ? (size_t)K * Gy * Gx * 8 : 0,   // grid2 [K][Gy][Gx]
      normal ? OffsetArena::round_up((size_t)(Gy / kKbStencilTile) * (Gx / kKbStencilTile) * 4) +  // tile list
                   (size_t)Gy * Gx * (2 * W - 1) * (2 * W - 1) * 4                               // stencil
             : 0,
      (size_t)4 * M * 8,                   // tile_ent
      (nb + 1) * 4,                        // tile_ptr
      nb * 4,                              // tile_ord
      ((size_t)M / (kKbSeg / 8) + 1) * 8,  // segs: a cut list has more than kKbSeg entries
      nb * 4,                              // seg0
  };
  for (int i = 0; i < KbLayout::kParts; ++i) L.sizes[i] = s[i];
  return L;
}

void kb_build_host(const float* traj_h, long M, int W, double sigma, int ny, int nx, int Gy, int Gx, KbTables& t) {
  const double beta = kb_beta(sigma, W);
  std::vector<int> ky0(M), kx0(M);
  std::vector<float> wy((size_t)M * W), wx((size_t)M * W);
  auto taps = [&](double w, int G, int& k0m, float* wt) {
    const double kappa = w * G / (2.0 * M_PI);
    const long k0 = (long)std::floor(kappa) - W / 2 + 1;
    for (int i = 0; i < W; ++i) wt[i] = (float)kb_phi(kappa - (double)(k0 + i), W, beta);
    k0m = (int)(((k0 % G) + G) % G);
  };
  for (long m = 0; m < M; ++m) {
    taps((double)traj_h[2 * m], Gy, ky0[m], &wy[(size_t)m * W]);
    taps((double)traj_h[2 * m + 1], Gx, kx0[m], &wx[(size_t)m * W]);
  }
  // counting sort by bin of the first tap (stable: sample order within a bin)
  const int nbx = Gx / kKbTile, nby = Gy / kKbTile, nb = nby * nbx;
  auto bin_of = [&](long m) { return (ky0[m] / kKbTile) * nbx + kx0[m] / kKbTile; };
  std::vector<int> bin_ptr((size_t)nb + 1, 0);
  for (long m = 0; m < M; ++m) ++bin_ptr[bin_of(m) + 1];
  for (int b = 0; b < nb; ++b) bin_ptr[b + 1] += bin_ptr[b];
  std::vector<int> fill(bin_ptr.begin(), bin_ptr.end() - 1);
  t.perm.resize(M);
  t.sky0.resize(M);
  t.skx0.resize(M);
  t.swy.resize((size_t)M * W);
  t.swx.resize((size_t)M * W);
  for (long m = 0; m < M; ++m) {
    const int j = fill[bin_of(m)]++;
    t.perm[j] = (int)m;
    t.sky0[j] = ky0[m];
    t.skx0[j] = kx0[m];
    for (int i = 0; i < W; ++i) {
      t.swy[(size_t)j * W + i] = wy[(size_t)m * W + i];
      t.swx[(size_t)j * W + i] = wx[(size_t)m * W + i];
    }
  }
  // interpolation units: runs of up to kKbUnit samples of one bin
  for (int b = 0; b < nb; ++b)
    for (int j = bin_ptr[b]; j < bin_ptr[b + 1]; j += kKbUnit)
      t.units.push_back(make_int2(j, std::min(kKbUnit, bin_ptr[b + 1] - j)));
  // tiles that each sample's footprint reaches: its bin's and, where the last
  // tap lies past it, the next one's along each axis
  auto reach = [&](int j, auto&& f) {
    const int ty0 = t.sky0[j] / kKbTile, tx0 = t.skx0[j] / kKbTile;
    const int cy = t.sky0[j] % kKbTile + W > kKbTile, cx = t.skx0[j] % kKbTile + W > kKbTile;
    for (int a = 0; a <= cy; ++a)
      for (int c = 0; c <= cx; ++c) f((ty0 + a) % nby * nbx + (tx0 + c) % nbx);
  };
  t.tile_ptr.assign((size_t)nb + 1, 0);
  for (long j = 0; j < M; ++j) reach((int)j, [&](int tile) { ++t.tile_ptr[tile + 1]; });
  for (int b = 0; b < nb; ++b) t.tile_ptr[b + 1] += t.tile_ptr[b];
  fill.assign(t.tile_ptr.begin(), t.tile_ptr.end() - 1);
  t.tile_ent.resize(t.tile_ptr[nb]);
  for (long j = 0; j < M; ++j) reach((int)j, [&](int tile) { t.tile_ent[fill[tile]++] = make_int2((int)j, t.perm[j]); });
  // long lists first, then the others, both in tile order
  auto len = [&](int tile) { return t.tile_ptr[tile + 1] - t.tile_ptr[tile]; };
  t.tile_ord.resize(nb);
  std::iota(t.tile_ord.begin(), t.tile_ord.end(), 0);
  t.n_heavy = (int)(std::stable_partition(t.tile_ord.begin(), t.tile_ord.end(), [&](int a) { return len(a) > kKbSeg; }) -
                    t.tile_ord.begin());
  for (int slot = 0; slot < t.n_heavy; ++slot) {
    t.seg0.push_back((int)t.segs.size());
    const int tile = t.tile_ord[slot];
    for (int e = t.tile_ptr[tile]; e < t.tile_ptr[tile + 1]; e += kKbSeg) t.segs.push_back(make_int2(slot, e));
  }
  t.dy.resize(ny);
  t.dx.resize(nx);
  for (int y = 0; y < ny; ++y) t.dy[y] = (float)(1.0 / kb_phi_hat((double)(y - ny / 2) / Gy, W, beta));
  for (int x = 0; x < nx; ++x) t.dx[x] = (float)(1.0 / kb_phi_hat((double)(x - nx / 2) / Gx, W, beta));
}

void kb_build_stencil(const std::vector<int>& sky0, const std::vector<int>& skx0, const std::vector<float>& swy,
                      const std::vector<float>& swx, long M, int W, int Gy, int Gx, std::vector<int>& tile_list,
                      int& n_active, std::vector<float>& stencil) {
  // S[g][d] = sum_m w_m(g) w_m(g + d): the weight of input grid point g + d
  // in output point g of P^H P, d in [-(W-1), W-1]^2, w_m the sample's taps
  constexpr int T = kKbStencilTile;
  const int D = 2 * W - 1, nty = Gy / T, ntx = Gx / T, ntiles = nty * ntx;
  std::vector<int> slot(ntiles, -1);
  for (long m = 0; m < M; ++m)   // tiles any footprint reaches are active
    for (int a = 0; a < W; ++a)
      for (int b = 0; b < W; ++b) {
        const int gy = (sky0[m] + a) % Gy, gx = (skx0[m] + b) % Gx;
        slot[(gy / T) * ntx + gx / T] = 0;
      }
  tile_list.clear();
  for (int t = 0; t < ntiles; ++t)
    if (slot[t] == 0) {
      slot[t] = (int)tile_list.size();
      tile_list.push_back(t);
    }
  n_active = (int)tile_list.size();
  for (int t = 0; t < ntiles; ++t)
    if (slot[t] < 0) tile_list.push_back(t);
  std::vector<double> acc((size_t)n_active * D * D * T * T, 0.0);
  for (long m = 0; m < M; ++m) {
    const float* wy = &swy[(size_t)m * W];
    const float* wx = &swx[(size_t)m * W];
    for (int a1 = 0; a1 < W; ++a1) {
      const int gy = (sky0[m] + a1) % Gy;
      for (int b1 = 0; b1 < W; ++b1) {
        const int gx = (skx0[m] + b1) % Gx;
        const int t = slot[(gy / T) * ntx + gx / T];
        const size_t pt = (size_t)(gy % T) * T + gx % T;
        const double w1 = (double)wy[a1] * wx[b1];
        double* base = &acc[(size_t)t * D * D * T * T + pt];
        for (int a2 = 0; a2 < W; ++a2) {
          const double w12 = w1 * wy[a2];
          const int dy = a2 - a1 + W - 1;
          for (int b2 = 0; b2 < W; ++b2) base[((size_t)dy * D + (b2 - b1 + W - 1)) * T * T] += w12 * wx[b2];
        }
      }
    }
  }
  stencil.resize(acc.size());
  for (size_t i = 0; i < acc.size(); ++i) stencil[i] = (float)acc[i];
}

// ------------------------------------------------------------------ kernels

enum KbSrc : int { KB_READ = 0, KB_NOISE = 1 };

typedef float floatx16 __attribute__((ext_vector_type(16)));

// Planes of a data pass: plane p of the launch is image p / cg, coil c0 + p mod cg
struct KbPlanes {
  int planes, cg, c0, nc;
  __device__ __forceinline__ int line(int p) const { return p / cg * nc + c0 + p % cg; }   // of K nc <= 2^22
};

// Spread of 16 planes onto 8 x 8 tiles: per tile D[64 points][32 columns (16
// planes, re and im)] = sum over the list's samples of wy wx [64][samples] times
// the values [samples][32], with v_mfma_f32_32x32x2f32 (two row blocks of 32
// points, two samples an instruction), 32 samples a step.  A wavefront stages a
// step's values and per-axis tile weights in LDS (the next step's loads are in
// flight during the products) and forms the weights' outer product as it feeds
// them.  The samples of a spiral crowd at the centre (a tenth of them within
// eight cells), so lists of more than kKbSeg entries are cut into segments, whose
// sums k_kb_join adds in list order; every wavefront then has at most kKbSeg / 32
// steps.  Without room for the segments' sums (nseg = 0) a long list stays with
// one wavefront.  192^2, 73728 samples, W 6, 12 coils x 6 probes: two launches of
// 57 us against 12 of 980 us for a scan of each tile's samples by one wavefront
// (uncut lists on one workgroup of 8 or 16 wavefronts: 99 and 92 us, the centre
// tiles' products then run on four of the chip's compute units).
//   KB_READ    src[line(p) M + m] (m the sample's index),
//   KB_NOISE   CN(0, 1) Philox draw (stream 1, element c M + m, draw first + image).
template <int W, int SRC>
__global__ __launch_bounds__(256) void k_kb_spread(KbOp o, KbPlanes pp, const float2* __restrict__ src, uint64_t seed,
                                                   uint64_t first, float2* __restrict__ gout, int nseg,
                                                   float2* __restrict__ part) {
  constexpr int T = kKbTile, ST = 32, VS = 34, WS = 17, P = 16;
  static_assert(T == 8, "64 points: two row blocks of 32");
  __shared__ float sv_all[4 * ST * VS];   // values [sample][plane, component]
  __shared__ float sw_all[4 * ST * WS];   // weights of the tile's rows, then columns, per sample
  const int wave = threadIdx.x / 64, l = threadIdx.x % 64, q = l % 32, h = l / 32;
  const int ntiles = o.nby * o.nbx, groups = (pp.planes + P - 1) / P;
  // items: the segments, then the tiles that are not cut; a tile's plane groups together
  const int item = (int)blockIdx.x * 4 + wave;
  const int idx = item / groups, pl0 = item % groups * P;
  const bool seg = idx < nseg;
  const int slot = seg ? o.segs[idx].x : idx - nseg + (nseg ? o.n_heavy : 0);
  if (slot >= ntiles) return;   // wavefronts work alone: no barriers
  const int tile = o.tile_ord[slot], p0 = seg ? o.segs[idx].y : o.tile_ptr[tile];
  const int p1 = seg ? min(p0 + kKbSeg, o.tile_ptr[tile + 1]) : o.tile_ptr[tile + 1];
  const int y0 = tile / o.nbx * T, x0 = tile % o.nbx * T;
  float* sv = sv_all + wave * ST * VS;
  float* sw = sw_all + wave * ST * WS;
  // this lane's sample (q) and planes pl0 + 8 h + u of a step; its axis is h (0: y, 1: x)
  const int* __restrict__ tap0 = h ? o.skx0 : o.sky0;
  const float* __restrict__ taps = h ? o.swx : o.swy;
  const int org = h ? x0 : y0, G = h ? o.Gx : o.Gy;
  int line[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) line[u] = pp.line(min(pl0 + 8 * h + u, pp.planes - 1));
  int2 ent = make_int2(0, -1), nxt = ent;   // entry of this step, of the next
  int d = 0;
  float wt[W];
  float2 v[8];
  auto entry = [&](int e) { return e < p1 ? o.tile_ent[e] : make_int2(0, -1); };
  auto load = [&](int2 en) {   // sample 0 past the list, not used
    d = tap0[en.x] - org;
#pragma unroll
    for (int t = 0; t < W; ++t) wt[t] = taps[(size_t)en.x * W + t];
    if constexpr (SRC == KB_READ) {
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = src[(size_t)line[u] * o.M + max(en.y, 0)];
    }
  };
  floatx16 acc[2] = {};
  if (p0 < p1) {
    ent = entry(p0 + q);
    nxt = entry(p0 + ST + q);
    load(ent);
  }
  const int py = q / T, px = q % T;
  for (int e = p0; e < p1; e += ST) {
    const bool on = ent.y >= 0;
    float* w8 = sw + q * WS + h * T;
#pragma unroll
    for (int i = 0; i < T; ++i) w8[i] = 0.f;
    d -= d >= T ? G : 0;   // the footprint wraps into this tile
#pragma unroll
    for (int t = 0; t < W; ++t)
      if (on && (unsigned)(d + t) < (unsigned)T) w8[d + t] = wt[t];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const bool use = on && pl0 + 8 * h + u < pp.planes;
      float2 val = make_float2(0.f, 0.f);
      if constexpr (SRC == KB_READ) {
        val = use ? v[u] : val;
      } else {
        if (use) {
          const int p = pl0 + 8 * h + u;
          val = draw_probe(seed, first + p / pp.cg, (uint32_t)((size_t)(pp.c0 + p % pp.cg) * o.M + ent.y), 1u, 3);
        }
      }
      *reinterpret_cast<float2*>(sv + q * VS + 2 * (8 * h + u)) = val;
    }
    ent = nxt;
    load(ent);
    nxt = entry(e + 2 * ST + q);
    wave_sync();
#pragma unroll 4
    for (int s = 0; s < ST / 2; ++s) {
      const float* ws = sw + (2 * s + h) * WS;
      const float b = sv[(2 * s + h) * VS + q], wx = ws[T + px];
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(ws[py] * wx, b, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(ws[4 + py] * wx, b, acc[1], 0, 0, 0);
    }
    wave_sync();
  }
  // accumulator i of lane l: row 8 (i / 4) + 4 (l / 32) + i mod 4 of its block,
  // column l mod 32; staged as [plane][32 points], padded
  constexpr int OS = 66;
  static_assert(P * OS <= ST * VS, "the output reuses the values' LDS");
  const size_t ps = seg ? (size_t)nseg * (T * T) : (size_t)o.Gy * o.Gx;   // from plane to plane
  const int rs = seg ? T : o.Gx;                                          // from tile row to tile row
  float2* __restrict__ to = seg ? part + (size_t)idx * (T * T) : gout + (size_t)y0 * o.Gx + x0;
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
#pragma unroll
    for (int i = 0; i < 16; ++i) sv[(q / 2) * OS + 2 * (8 * (i / 4) + 4 * h + i % 4) + q % 2] = acc[rb][i];
    wave_sync();
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int p = 2 * u + h;
      if (pl0 + p < pp.planes)
        to[(pl0 + p) * ps + (size_t)(4 * rb + py) * rs + px] = *reinterpret_cast<float2*>(sv + p * OS + 2 * q);
    }
    wave_sync();
  }
}

// grid points of the cut tiles: their segments' sums added in list order (one
// wavefront per tile, blockIdx.x, and plane, blockIdx.y)
__global__ __launch_bounds__(64) void k_kb_join(KbOp o, int nseg, const float2* __restrict__ part,
                                                float2* __restrict__ gout) {
  constexpr int T = kKbTile;
  const int slot = blockIdx.x, tile = o.tile_ord[slot];
  const int n = (o.tile_ptr[tile + 1] - o.tile_ptr[tile] + kKbSeg - 1) / kKbSeg;
  const float2* __restrict__ pt = part + ((size_t)blockIdx.y * nseg + o.seg0[slot]) * (T * T) + threadIdx.x;
  float2 acc = make_float2(0.f, 0.f);
#pragma unroll 8
  for (int i = 0; i < n; ++i) acc = cadd(acc, pt[(size_t)i * (T * T)]);
  const int y = tile / o.nbx * T + (int)threadIdx.x / T, x = tile % o.nbx * T + (int)threadIdx.x % T;
  gout[(size_t)blockIdx.y * o.Gy * o.Gx + (size_t)y * o.Gx + x] = acc;
}

// P^H P by its stencil, one 16 x 16 tile (a slot of the tile list) and a run
// of kc probes per workgroup.  Work items (probe run, slot), slots fastest,
// go to the eight XCDs in contiguous runs (workgroup b on XCD b mod 8 takes
// item (b mod 8) * ceil(total / 8) + b / 8), so tiles that share window
// halos meet in one L2; the padding workgroups return at once.
template <int W>
__global__ __launch_bounds__(256) void k_kb_stencil(KbOp o, const float2* __restrict__ gin, float2* __restrict__ gout,
                                                    int K, int kc, int slots) {
  constexpr int T = kKbStencilTile, D = 2 * W - 1, WIN = T + D - 1;
  static_assert(T * T == 256, "one output point per thread");
  __shared__ float2 win[WIN * WIN];
  const long total = (long)slots * ((K + kc - 1) / kc), per = (total + 7) / 8;
  const long item = (long)(blockIdx.x % 8) * per + blockIdx.x / 8;
  if (item >= total) return;
  const int slot = (int)(item % slots), tile = o.tile_list[slot], ntx = o.Gx / T;
  const int y0 = (tile / ntx) * T, x0 = (tile % ntx) * T, wy0 = y0 - (W - 1), wx0 = x0 - (W - 1);
  const int py = threadIdx.x / T, px = threadIdx.x % T;
  const int k0 = (int)(item / slots) * kc, k1 = min(K, k0 + kc);
  const long G2 = (long)o.Gy * o.Gx;
  float2* outp = gout + (size_t)(y0 + py) * o.Gx + x0 + px;
  if (slot >= o.n_active) {   // no sample reaches this tile
    for (int k = k0; k < k1; ++k) outp[(size_t)k * G2] = make_float2(0.f, 0.f);
    return;
  }
  // window points of this thread (NW per thread), and the next probe's values
  // loaded while the current probe is computed (W <= 6: at W = 8 the 225
  // stencil weights leave no registers for them)
  constexpr int NW = (WIN * WIN + 255) / 256;
  constexpr bool PF = W <= 6;
  auto goff = [&](int i) {
    int gy = wy0 + i / WIN, gx = wx0 + i % WIN;   // the window spans less than one period
    gy += gy < 0 ? o.Gy : 0;
    gy -= gy >= o.Gy ? o.Gy : 0;
    gx += gx < 0 ? o.Gx : 0;
    gx -= gx >= o.Gx ? o.Gx : 0;
    return (long)gy * o.Gx + gx;
  };
  float2 nxt[NW];
  auto load_win = [&](int k) {
    const float2* gk = gin + (size_t)k * G2;
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      const int i = threadIdx.x + 256 * j;
      if (i < WIN * WIN) nxt[j] = gk[goff(i)];
    }
  };
  if (PF && k0 < k1) load_win(k0);
  float st[D * D];
  const float* sp = o.stencil + (size_t)slot * D * D * T * T + threadIdx.x;
#pragma unroll
  for (int i = 0; i < D * D; ++i) st[i] = sp[(size_t)i * T * T];
  for (int k = k0; k < k1; ++k) {
    __syncthreads();   // every thread is done with the previous window
    if constexpr (PF) {
#pragma unroll
      for (int j = 0; j < NW; ++j)
        if (threadIdx.x + 256 * j < WIN * WIN) win[threadIdx.x + 256 * j] = nxt[j];
    } else {
      const float2* gk = gin + (size_t)k * G2;
      for (int i = threadIdx.x; i < WIN * WIN; i += 256) win[i] = gk[goff(i)];
    }
    __syncthreads();
    if (PF && k + 1 < k1) load_win(k + 1);
    float2 acc = make_float2(0.f, 0.f);
#pragma unroll
    for (int dy = 0; dy < D; ++dy)
#pragma unroll
      for (int dx = 0; dx < D; ++dx) acc = cfma(acc, st[dy * D + dx], win[(py + dy) * WIN + px + dx]);
    outp[(size_t)k * G2] = acc;
  }
}

// out[line(p) M + m] = sum_{a, t} wy[a] wx[t] grid[p][ky0 + a][kx0 + t].  One
// wavefront per unit of up to 32 samples of one bin and a run of planes, two
// planes at a time (one per half wave): the bin's window of grid points is read
// once per plane into LDS (the next pair's while this one is summed) and the
// samples' weights stay in registers over the run.  Bound by the LDS window
// reads (W^2 per sample and plane); gathering from the grid in L2 with one
// plane per thread took 30.6 us per coil (256^2, 98304 samples, W 6, 8 planes),
// 490 us for 16 coils; now two launches of 85 us.
template <int W>
__global__ __launch_bounds__(256) void k_kb_interp(KbOp o, KbPlanes pp, const float2* __restrict__ grid,
                                                   float2* __restrict__ out, int run) {
  constexpr int T = kKbTile, WIN = T + W - 1, W2 = WIN * WIN, NL = (2 * W2 + 63) / 64;
  __shared__ float2 win_all[4][2 * W2];
  const int wave = threadIdx.x / 64, l = threadIdx.x % 64, q = l % 32, h = l / 32;
  const int u = (int)blockIdx.x * 4 + wave;
  if (u >= o.n_units) return;   // wavefronts work alone: no barriers
  float2* win = win_all[wave];
  const int2 un = o.units[u];
  const int j = un.x + min(q, un.y - 1), m = o.perm[j];
  const int y0 = o.sky0[un.x] / T * T, x0 = o.skx0[un.x] / T * T;
  const float2* __restrict__ wq = win + h * W2 + (o.sky0[j] - y0) * WIN + (o.skx0[j] - x0);
  float wy[W], wx[W];
#pragma unroll
  for (int t = 0; t < W; ++t) {
    wy[t] = o.swy[(size_t)j * W + t];
    wx[t] = o.swx[(size_t)j * W + t];
  }
  const long G2 = (long)o.Gy * o.Gx;
  const int pa = (int)blockIdx.y * run, pb = min(pp.planes, pa + run);
  int off[NL];        // window points of this lane within a plane (bounded by the grid: below 2^31)
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int w = (l + 64 * i) % W2;
    int gy = y0 + w / WIN, gx = x0 + w % WIN;
    gy -= gy >= o.Gy ? o.Gy : 0;
    gx -= gx >= o.Gx ? o.Gx : 0;
    off[i] = gy * o.Gx + gx;
  }
  float2 nxt[NL];
  auto load = [&](int p) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int pl = min(p + (l + 64 * i) / W2, pb - 1);   // past the run: any plane, not used
      nxt[i] = grid[pl * G2 + off[i]];
    }
  };
  if (pa < pb) load(pa);
  for (int p = pa; p < pb; p += 2) {
#pragma unroll
    for (int i = 0; i < NL; ++i)
      if (l + 64 * i < 2 * W2) win[l + 64 * i] = nxt[i];
    wave_sync();
    if (p + 2 < pb) load(p + 2);
    float2 acc = make_float2(0.f, 0.f);
#pragma unroll
    for (int a = 0; a < W; ++a) {
      float2 row = make_float2(0.f, 0.f);
#pragma unroll
      for (int t = 0; t < W; ++t) row = cfma(row, wx[t], wq[a * WIN + t]);
      acc = cfma(acc, wy[a], row);
    }
    if (q < un.y && p + h < pb) out[(size_t)pp.line(p + h) * o.M + m] = acc;
    wave_sync();
  }
}

template <int SRC>
static hipError_t spread(const KbOp& o, const KbPlanes& pp, const float2* src, uint64_t seed, uint64_t first,
                         float2* gout, float2* part, hipStream_t s) {
  const int nseg = part ? o.n_seg : 0;
  const long items = ((long)nseg + (long)o.nby * o.nbx - (nseg ? o.n_heavy : 0)) * ((pp.planes + 15) / 16);
  const dim3 grid((unsigned)((items + 3) / 4)), block(256);
  switch (o.W) {
    case 2: hipLaunchKernelGGL((k_kb_spread<2, SRC>), grid, block, 0, s, o, pp, src, seed, first, gout, nseg, part); break;
    case 4: hipLaunchKernelGGL((k_kb_spread<4, SRC>), grid, block, 0, s, o, pp, src, seed, first, gout, nseg, part); break;
    case 6: hipLaunchKernelGGL((k_kb_spread<6, SRC>), grid, block, 0, s, o, pp, src, seed, first, gout, nseg, part); break;
    case 8: hipLaunchKernelGGL((k_kb_spread<8, SRC>), grid, block, 0, s, o, pp, src, seed, first, gout, nseg, part); break;
    default: return hipErrorInvalidValue;
  }
  if (nseg)
    hipLaunchKernelGGL(k_kb_join, dim3((unsigned)o.n_heavy, (unsigned)pp.planes), dim3(64), 0, s, o, nseg, part, gout);
  return hipGetLastError();
}

// Probes per workgroup: a workgroup loads its tile's (2W-1)^2 stencil weights
// once (124 KB at W = 6) for its run of probes, so runs grow from 16 while
// the active tiles still give at least 2048 workgroups.
static hipError_t stencil(const KbOp& o, int K, const float2* gin, float2* gout, hipStream_t s) {
  const int slots = (o.Gy / kKbStencilTile) * (o.Gx / kKbStencilTile);
  int kc = 16;
  while (kc < 128 && (long)std::max(o.n_active, 1) * ((K + 2 * kc - 1) / (2 * kc)) >= 2048) kc *= 2;
  const long total = (long)slots * ((K + kc - 1) / kc);
  const dim3 grid((unsigned)(8 * ((total + 7) / 8))), block(256);
  switch (o.W) {
    case 2: hipLaunchKernelGGL(k_kb_stencil<2>, grid, block, 0, s, o, gin, gout, K, kc, slots); break;
    case 4: hipLaunchKernelGGL(k_kb_stencil<4>, grid, block, 0, s, o, gin, gout, K, kc, slots); break;
    case 6: hipLaunchKernelGGL(k_kb_stencil<6>, grid, block, 0, s, o, gin, gout, K, kc, slots); break;
    case 8: hipLaunchKernelGGL(k_kb_stencil<8>, grid, block, 0, s, o, gin, gout, K, kc, slots); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Planes per wavefront: the unit's weights and window offsets are set up once per
// run, so runs grow from 8 while the units still give 8192 wavefronts (eight per
// SIMD).
static hipError_t interp(const KbOp& o, const KbPlanes& pp, const float2* grid, float2* out, hipStream_t s) {
  int run = 8;
  while (run < 64 && (long)o.n_units * ((pp.planes + 2 * run - 1) / (2 * run)) >= 8192) run *= 2;
  const dim3 g((unsigned)((o.n_units + 3) / 4), (unsigned)((pp.planes + run - 1) / run)), block(256);
  switch (o.W) {
    case 2: hipLaunchKernelGGL(k_kb_interp<2>, g, block, 0, s, o, pp, grid, out, run); break;
    case 4: hipLaunchKernelGGL(k_kb_interp<4>, g, block, 0, s, o, pp, grid, out, run); break;
    case 6: hipLaunchKernelGGL(k_kb_interp<6>, g, block, 0, s, o, pp, grid, out, run); break;
    case 8: hipLaunchKernelGGL(k_kb_interp<8>, g, block, 0, s, o, pp, grid, out, run); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Coils per launch for K images: as many as the scratch holds grids for, dealt
// evenly; for the spread (seg), with room for the segments' sums in the idle grid
// buffer or behind the grids, whichever lets more coils share a launch
struct CoilGroups {
  int step;
  float2* part;   // segments' sums, or NULL: no room
};
static CoilGroups coil_groups(const KbOp& o, int nc, int K, const KbScratch& sc, bool seg) {
  const size_t G2 = (size_t)o.Gy * o.Gx, sums = (size_t)o.n_seg * kKbTile * kKbTile;   // per plane
  const size_t grids = sc.room / (K * G2);
  size_t fit = grids;
  int where = 0;   // 0: no segments, 1: beside, 2: behind
  if (seg && sums) {
    const size_t beside = std::min(grids, sc.room2 / (K * sums)), behind = sc.room / (K * (G2 + sums));
    if (beside || behind) {
      where = beside >= behind ? 1 : 2;
      fit = std::max(beside, behind);
    }
  }
  const int most = (int)std::max<size_t>(1, std::min<size_t>(nc, fit)), n = (nc + most - 1) / most;
  const int step = (nc + n - 1) / n;
  return {step, where == 1 ? sc.buf2 : where == 2 ? sc.buf + (size_t)K * step * G2 : nullptr};
}

// out[K][ny][nx] = A^H of K multi-coil sample arrays: src [K][nc][M] (whitened),
// or Philox CN(0, 1) noise (src == nullptr; stream 1, element c M + m).  Per
// group of coils: spread onto their grids, inverse column transforms back to the
// image rows (in place), inverse row transforms cropped and combined.
hipError_t kb_adjoint(const KbOp& o, const float2* maps, int nc, int K, const float2* src, uint64_t seed,
                      uint64_t first, float2* out, const KbScratch& sc, hipStream_t s) {
  const long n = (long)o.ny * o.nx, G2 = (long)o.Gy * o.Gx;
  const float scale = (float)(1.0 / std::sqrt((double)n));
  const auto [step, part] = coil_groups(o, nc, K, sc, true);
  float2* scratch = sc.buf;
  for (int c = 0; c < nc; c += step) {
    const int cg = std::min(step, nc - c);
    const KbPlanes pp{K * cg, cg, c, nc};
    hipError_t e = src ? spread<KB_READ>(o, pp, src, 0, 0, scratch, part, s)
                       : spread<KB_NOISE>(o, pp, nullptr, seed, first, scratch, part, s);
    if (e != hipSuccess) return e;
    if ((e = launch_fft_cols_crop(scratch, scratch, G2, G2, pp.planes, o.ny, o.Gy, o.Gx, true, o.twy, s)) != hipSuccess)
      return e;
    if ((e = launch_kbn_rows(true, scratch, maps + (size_t)c * n, o.dy, o.dx, out, K, cg, G2, o.ny, o.nx, o.Gx, scale,
                             c > 0 ? 1 : 0, o.twx, s)) != hipSuccess)
      return e;
  }
  return hipSuccess;
}

// out[K][nc][M] = A x for K images x [K][ny][nx]: per group of coils, the image
// rows expanded and row-transformed, column transforms to the full grids (in
// place), interpolation
hipError_t kb_forward(const KbOp& o, const float2* maps, int nc, int K, const float2* x, float2* out,
                      const KbScratch& sc, hipStream_t s) {
  const long n = (long)o.ny * o.nx, G2 = (long)o.Gy * o.Gx;
  const float scale = (float)(1.0 / std::sqrt((double)n));
  const int step = coil_groups(o, nc, K, sc, false).step;
  float2* scratch = sc.buf;
  for (int c = 0; c < nc; c += step) {
    const int cg = std::min(step, nc - c);
    const KbPlanes pp{K * cg, cg, c, nc};
    hipError_t e = launch_kbn_rows(false, x, maps + (size_t)c * n, o.dy, o.dx, scratch, K, cg, G2, o.ny, o.nx, o.Gx,
                                   scale, 0, o.twx, s);
    if (e != hipSuccess) return e;
    if ((e = launch_fft_cols_crop(scratch, scratch, G2, G2, pp.planes, o.ny, o.Gy, o.Gx, false, o.twy, s)) != hipSuccess)
      return e;
    if ((e = interp(o, pp, scratch, out, s)) != hipSuccess) return e;
  }
  return hipSuccess;
}

// ------------------------------------------------------------------ gridding normal operator

// double sum over a 256-thread block, fixed order
__device__ double block_sum256(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int o2 = 128; o2 > 0; o2 >>= 1) {
    if ((int)threadIdx.x < o2) red[threadIdx.x] += red[threadIdx.x + o2];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

// p of the CG step per image row (blockIdx.x = y, blockIdx.y = k), as the grid
// path's first row kernel forms it, with |r|^2 of the row in part[k][y][0]
template <int MODE>
__global__ __launch_bounds__(256) void k_kbn_pro(Grid2dArgs a) {
  __shared__ double red[256];
  const int y = blockIdx.x, k = blockIdx.y;
  const size_t row = ((size_t)k * a.ny + y) * a.nx;
  float alpha = 0.f, beta = 0.f;
  if constexpr (MODE == C1_ITER) {
    alpha = (float)a.alpha[k];
    beta = (float)a.beta[k];
  }
  double d0 = 0.0;
  for (int x = threadIdx.x; x < a.nx; x += 256) {
    const size_t i = row + x;
    if constexpr (MODE == C1_FIRST_PROBE) {
      const float2 v = draw_probe(arg_seed(a), arg_first(a) + k, (uint32_t)(y * a.nx + x), 0u, a.dist);
      a.r[i] = v;
      a.p[i] = v;
      d0 += (double)v.x * v.x + (double)v.y * v.y;
    } else if constexpr (MODE == C1_FIRST_BUF) {
      const float2 v = a.r[i];
      a.p[i] = v;
      d0 += (double)v.x * v.x + (double)v.y * v.y;
    } else if constexpr (MODE == C1_ITER) {
      const float2 po = a.p[i], qo = a.q[i], ro = a.r[i];
      const float2 xo = a.x_zero ? make_float2(0.f, 0.f) : a.x[i];
      const float2 rn = cfma(ro, -alpha, qo);
      a.x[i] = cfma(xo, alpha, po);
      a.r[i] = rn;
      a.p[i] = cfma(rn, beta, po);
      d0 += (double)rn.x * rn.x + (double)rn.y * rn.y;
    }
  }
  d0 = block_sum256(d0, red);
  if (threadIdx.x == 0) a.part[((size_t)k * a.ny + y) * 4] = d0;
}

// q = (coil sum already in q) + lam p_in, and the partial dots Re p^H q, |q|^2,
// Re r^H q of the row (r = p_in outside C1_ITER)
template <int MODE>
__global__ __launch_bounds__(256) void k_kbn_epi(Grid2dArgs a) {
  __shared__ double red[256];
  const int y = blockIdx.x, k = blockIdx.y;
  const size_t row = ((size_t)k * a.ny + y) * a.nx;
  double d1 = 0.0, d2 = 0.0, d3 = 0.0;
  for (int x = threadIdx.x; x < a.nx; x += 256) {
    const size_t i = row + x;
    const float2 pin = MODE == C1_APPLY ? cscale(a.src[i], a.scale) : a.p[i];
    const float2 q = cfma(a.q[i], a.lam, pin);
    a.q[i] = q;
    const float2 rv = MODE == C1_ITER ? a.r[i] : pin;
    d1 += (double)pin.x * q.x + (double)pin.y * q.y;
    d2 += (double)q.x * q.x + (double)q.y * q.y;
    d3 += (double)rv.x * q.x + (double)rv.y * q.y;
  }
  d1 = block_sum256(d1, red);
  d2 = block_sum256(d2, red);
  d3 = block_sum256(d3, red);
  if (threadIdx.x == 0) {
    double* pp = a.part + ((size_t)k * a.ny + y) * 4;
    pp[1] = d1;
    pp[2] = d2;
    pp[3] = d3;
  }
}

hipError_t launch_kb_normal(int mode, const Grid2dArgs& a, const KbOp& o, hipStream_t s) {
  if (!o.grid2 || !o.stencil) return hipErrorInvalidValue;
  const dim3 rows((unsigned)a.ny, a.K), block(256);
  switch (mode) {
    case C1_FIRST_PROBE: hipLaunchKernelGGL(k_kbn_pro<C1_FIRST_PROBE>, rows, block, 0, s, a); break;
    case C1_FIRST_BUF: hipLaunchKernelGGL(k_kbn_pro<C1_FIRST_BUF>, rows, block, 0, s, a); break;
    case C1_ITER: hipLaunchKernelGGL(k_kbn_pro<C1_ITER>, rows, block, 0, s, a); break;
    case C1_APPLY: break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const long n = (long)o.ny * o.nx, G2 = (long)o.Gy * o.Gx, rows_n = (long)o.ny * o.Gx;
  const float scale = (float)(1.0 / std::sqrt((double)n));
  const float2* xin = mode == C1_APPLY ? a.src : a.p;
  const float in_scale = mode == C1_APPLY ? scale * a.scale : scale;
  // per coil: image rows expanded and row-transformed ([K][ny][Gx] in
  // grid2), column transforms to the full grid, stencil, inverse column
  // transforms back to the image rows (in grid), inverse row transforms
  // cropped and combined into q
  for (int c = 0; c < a.nc; ++c) {
    const float2* Sc = a.maps + (size_t)c * n;
    if ((e = launch_kbn_rows(false, xin, Sc, o.dy, o.dx, o.grid2, a.K, 1, rows_n, o.ny, o.nx, o.Gx, in_scale, 0, o.twx,
                             s)) != hipSuccess)
      return e;
    if ((e = launch_fft_cols_crop(o.grid2, o.grid, rows_n, G2, a.K, o.ny, o.Gy, o.Gx, false, o.twy, s)) != hipSuccess)
      return e;
    if ((e = stencil(o, a.K, o.grid, o.grid2, s)) != hipSuccess) return e;
    if ((e = launch_fft_cols_crop(o.grid2, o.grid, G2, rows_n, a.K, o.ny, o.Gy, o.Gx, true, o.twy, s)) != hipSuccess)
      return e;
    if ((e = launch_kbn_rows(true, o.grid, Sc, o.dy, o.dx, a.q, a.K, 1, rows_n, o.ny, o.nx, o.Gx, scale, c > 0 ? 1 : 0,
                             o.twx, s)) != hipSuccess)
      return e;
  }
  switch (mode) {
    case C1_FIRST_PROBE: hipLaunchKernelGGL(k_kbn_epi<C1_FIRST_PROBE>, rows, block, 0, s, a); break;
    case C1_FIRST_BUF: hipLaunchKernelGGL(k_kbn_epi<C1_FIRST_BUF>, rows, block, 0, s, a); break;
    case C1_ITER: hipLaunchKernelGGL(k_kbn_epi<C1_ITER>, rows, block, 0, s, a); break;
    default: hipLaunchKernelGGL(k_kbn_epi<C1_APPLY>, rows, block, 0, s, a); break;
  }
  return hipGetLastError();
}

}  // namespace pico
