"""GPU parity of the batched gridding data path (matrix-core spread, windowed
interpolation, several coils a launch) against the FP64 oracle, where the
kernels can go wrong: every kernel width, one sample, a footprint that wraps
the grid's edge, more than one list step per tile, tiles long enough for eight
wavefronts, planes that do not fill a group of 16, coils that need several
launches.

Tolerance: tap weights are stored in FP32 and multiplied (1.2e-7), the
transforms lose about eps log2(G^2) <= 6e-8 * 16 = 1e-6, and a grid point sums
up to n <= 2000 samples with an error of about eps sqrt(n) = 2.7e-6 (relative,
2-norm); together below 5e-6.
"""
import numpy as np
import pytest

import workloads
from oracle import kbnufft as okb
from oracle import sense

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

TOL = 5e-6


def _traj(kind, M, rng):
    if kind == "edge":      # around the grid's corners: taps wrap in both axes
        w = rng.choice([-np.pi, np.pi - 1e-3], size=(M, 2)) + rng.uniform(0, 1e-3, size=(M, 2))
    elif kind == "crowd":   # nearly all within a few cells of the centre
        w = rng.standard_normal((M, 2)) * 0.05
        w[: M // 8] = rng.uniform(-np.pi, np.pi, size=(M // 8, 2))
    else:
        w = rng.uniform(-np.pi, np.pi, size=(M, 2))
    return np.clip(w, -np.pi, np.nextafter(np.float32(np.pi), np.float32(0))).astype(np.float32)


@pytest.mark.parametrize("kind,M,ny,nx,nc,k,sigma,W", [
    ("spread", 1, 32, 32, 1, 1, 2.0, 6),        # one sample, one plane
    ("edge", 700, 32, 48, 3, 2, 2.0, 8),        # wrapped footprints; one coil a launch
    ("spread", 3001, 64, 48, 5, 3, 2.0, 2),     # three launches of 2, 2 and 1 coils
    ("crowd", 6000, 32, 32, 9, 5, 2.0, 6),      # heavy tiles; 20 planes: a group of 16 and one of 4
    ("crowd", 2500, 48, 64, 33, 1, 2.0, 4),     # 16 planes a launch, then one
    ("spread", 900, 128, 256, 2, 3, 1.25, 4),   # oversampling 1.25
])
def test_batched_data_path(kind, M, ny, nx, nc, k, sigma, W):
    from paper_2605_09590_amd import pico as lib
    print(f"case: {kind}, {M} samples, {ny}x{nx}, {nc} coils, {k} images, sigma {sigma}, W {W}", flush=True)
    rng = np.random.default_rng(M + W)
    traj = _traj(kind, M, rng)
    maps = workloads.coil_maps(ny, nx, nc, rng).astype(np.complex64)
    psi = workloads.noise_cov(nc, rng)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    h = lib.pico_init(ny, nx, dev(maps), psi, None, sampling=lib.PICO_NONCART, traj=dev(traj), nsamples=M,
                      cg_iters=1, probe_tile=k, oversamp=sigma, kb_width=W)
    g = okb.KBGridding(traj.astype(np.float64), ny, nx, sigma, W)
    S = sense.whiten_maps(maps.astype(np.complex128), psi)
    cn = lambda *s: (rng.standard_normal(s) + 1j * rng.standard_normal(s)).astype(np.complex64)  # noqa: E731
    x, y = cn(k, ny, nx), cn(k, nc, M)
    out_f = torch.empty(k, nc, M, dtype=torch.complex64, device="cuda:0")
    out_a = torch.empty(k, ny, nx, dtype=torch.complex64, device="cuda:0")
    lib.pico_apply_nufft(h, 0, dev(x), out_f, k)
    lib.pico_apply_nufft(h, 1, dev(y), out_a, k)
    torch.cuda.synchronize()
    lib.pico_destroy(h)
    ref_f = np.stack([np.stack([g.forward(S[c] * x[b]) for c in range(nc)]) for b in range(k)])
    ref_a = np.stack([sum(np.conj(S[c]) * g.adjoint(y[b, c].astype(np.complex128)) for c in range(nc)) for b in range(k)])
    for name, got, ref in (("forward", out_f, ref_f), ("adjoint", out_a, ref_a)):
        err = np.linalg.norm(got.cpu().numpy() - ref) / np.linalg.norm(ref)
        print(f"  {name}: rel err {err:.2e}", flush=True)
        assert err < TOL
