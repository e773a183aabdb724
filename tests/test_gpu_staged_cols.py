"""Columns that go through an LDS tile (padded 288 and 320 points, unpadded 512), with
the coil planes in bfloat16, against the same operator with complex64 planes (whose
parity with the oracle the column and probe-set tests check).

Tolerance: the planes are rounded to 8 significand bits twice an application, so a
product is off by about 2^-9 sqrt(2) = 2.8e-3 of its norm, and the regularised solves
(lambda 0.1: condition number <= 11) pass on at most that multiple: 3e-2.
"""
import numpy as np
import pytest

import workloads

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,ny,nx", [("spiral", 288, 48), ("spiral", 320, 32), ("cart2d", 512, 96)])
def test_bfloat16_planes(kind, ny, nx):
    from paper_2605_09590_amd import pico as lib
    K, nc = 3, 3
    print(f"case: {kind} {ny}x{nx}, {nc} coils, {K} probes, bfloat16 planes", flush=True)
    rng = np.random.default_rng(ny + nx)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    maps = dev(workloads.coil_maps(ny, nx, nc, rng).astype(np.complex64))
    psi = workloads.noise_cov(nc, rng)
    kw = dict(lam=0.1, cg_iters=4, probe_tile=K)
    if kind == "spiral":
        traj = workloads.spiral_traj(max(ny, nx), 1, 12, 256).astype(np.float32)
        kw.update(mask=None, sampling=lib.PICO_NONCART, traj=dev(traj), nsamples=traj.shape[0])
    else:
        kw.update(mask=dev((rng.uniform(size=(ny, nx)) < 0.5).astype(np.uint8)), sampling=lib.PICO_CART_2D)
    v = torch.randn(K, ny, nx, dtype=torch.complex64, device="cuda:0")
    u = {}
    for storage in (1, 2):
        h = lib.pico_init(ny, nx, maps, psi, storage=storage, **kw)
        u[storage] = torch.empty_like(v)
        lib.pico_apply_cov(h, v, u[storage], K)
        torch.cuda.synchronize()
        lib.pico_destroy(h)
    for k in range(K):
        err = float((u[2][k] - u[1][k]).norm() / u[1][k].norm())
        print(f"  probe {k}: rel diff {err:.2e}", flush=True)
        assert 0 < err < 3e-2
