"""Grid path with coil planes of more than 108 MiB a probe: 768 x 288 points and 64 coils,
where a set holds one probe and has few enough rows for the form with several
wavefronts, and 768 x 768 with 32 coils, which go through in one pass.  Against the
FP64 oracle, two unregularised CG iterations (no power method).  Tolerance: a transform pair and the coil sum are off by eps (log2(Ny Nx) +
nc) <= 6e-8 * 82 = 4.9e-6 an application; two of them and the vector updates, below 2e-5.
"""
import numpy as np
import pytest

import workloads
from oracle import pico as opico

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nc", [(288, 64), (768, 32)])
def test_large_planes(nx, nc):
    from paper_2605_09590_amd import pico as lib
    ny, K, cg = 768, 3, 2
    print(f"case: cart2d {ny}x{nx}, {nc} coils, {K} probes, lambda 0, CG {cg}", flush=True)
    rng = np.random.default_rng(ny + nx)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    maps = workloads.coil_maps(ny, nx, nc, rng).astype(np.complex64)
    psi = workloads.noise_cov(nc, rng)
    mask = (rng.uniform(size=(ny, nx)) < 0.5).astype(np.uint8)
    h = lib.pico_init(ny, nx, dev(maps), psi, dev(mask), sampling=lib.PICO_CART_2D, lam=0.0, cg_iters=cg, probe_tile=K)
    v = (rng.standard_normal((K, ny, nx)) + 1j * rng.standard_normal((K, ny, nx))).astype(np.complex64)
    vt = dev(v)
    ut = torch.empty_like(vt)
    lib.pico_apply_cov(h, vt, ut, K)
    torch.cuda.synchronize()
    lib.pico_destroy(h)
    cov = opico.Covariance(opico.cartesian(maps.astype(np.complex128), psi, mask), 0.0, cg)
    for k in (0, K - 1):
        ref = cov.apply(v[k].astype(np.complex128))
        err = np.linalg.norm(ut[k].cpu().numpy() - ref) / np.linalg.norm(ref)
        print(f"  probe {k}: rel err {err:.2e}", flush=True)
        assert err < 2e-5
