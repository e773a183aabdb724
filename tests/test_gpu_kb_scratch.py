"""Gridding data path against the FP64 oracle for each place that the sums of cut
tile lists can have: none (one or two coils: the planes are no larger than a grid, a
crowded list stays with one wavefront), beside the grids, and behind them (more sums
than a grid has points).  Tolerance as in the batched data path's test: 5e-6.
"""
import numpy as np
import pytest

import workloads
from oracle import kbnufft as okb
from oracle import sense

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

TOL = 5e-6


@pytest.mark.parametrize("place,M,nc,k,spread", [
    ("none", 3000, 1, 2, 0.05),
    ("none", 3000, 2, 3, 0.05),
    ("beside", 3000, 5, 2, 0.05),
    ("behind", 20000, 20, 2, 1.5),        # 64 tiles, about 260 segments of 64 sums
    ("behind", 20000, 45, 1, 1.5),
])
def test_places_of_the_sums(place, M, nc, k, spread):
    from paper_2605_09590_amd import pico as lib
    ny = nx = 32
    print(f"case: sums {place}, {M} samples, {ny}x{nx}, {nc} coils, {k} images", flush=True)
    rng = np.random.default_rng(M + nc)
    traj = (rng.standard_normal((M, 2)) * spread).clip(-3.1, 3.1).astype(np.float32)
    maps = workloads.coil_maps(ny, nx, nc, rng).astype(np.complex64)
    psi = workloads.noise_cov(nc, rng)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    h = lib.pico_init(ny, nx, dev(maps), psi, None, sampling=lib.PICO_NONCART, traj=dev(traj), nsamples=M,
                      cg_iters=1, probe_tile=k, oversamp=2.0, kb_width=6)
    g = okb.KBGridding(traj.astype(np.float64), ny, nx, 2.0, 6)
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
