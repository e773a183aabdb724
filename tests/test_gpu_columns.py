"""GPU parity of the grid path's column pass at the line lengths that the other
grid tests do not reach (the shortest and longest padded lines, and the
unpadded ones of 64, 128 and 512 to 768 points), against the FP64 oracle.

Tolerance: an FP32 transform pair and coil sum is off by about
eps (log2(Ny Nx) + nc) <= 6e-8 * 22 = 1.3e-6; the regularised solves
(lambda 0.1: condition number <= 11) pass on at most that multiple: 1.5e-5,
rounded up to 2e-5.
"""
import numpy as np
import pytest

import workloads
from oracle import nufft as onufft
from oracle import pico as opico

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

TOL = 2e-5


@pytest.mark.parametrize("kind,ny,nx", [
    ("spiral", 32, 48),     # shortest padded column
    ("spiral", 48, 32),
    ("spiral", 64, 80),
    ("spiral", 80, 32),
    ("spiral", 384, 32),    # longest padded column
    ("cart2d", 64, 96),
    ("cart2d", 128, 64),
    ("cart2d", 512, 64),
    ("cart2d", 576, 64),
    ("cart2d", 640, 64),
    ("cart2d", 768, 64),    # longest column
])
def test_column_lengths(kind, ny, nx):
    from paper_2605_09590_amd import pico as lib
    K, nc, cg = 3, 2, 4
    print(f"case: {kind} {ny}x{nx}, {nc} coils, {K} probes, lambda 0.1, CG {cg}", flush=True)
    rng = np.random.default_rng(ny * 1000 + nx)
    maps = workloads.coil_maps(ny, nx, nc, rng)
    psi = workloads.noise_cov(nc, rng)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    kw = dict(lam=0.1, cg_iters=cg, probe_tile=K)
    if kind == "spiral":
        traj = workloads.spiral_traj(max(ny, nx), 1, 12, 256).astype(np.float32)
        h = lib.pico_init(ny, nx, dev(maps.astype(np.complex64)), psi, None, sampling=lib.PICO_NONCART,
                          traj=dev(traj), nsamples=traj.shape[0], **kw)
        op = onufft.NonCartOp(maps, psi, traj.astype(np.float64))
    else:
        mask = (rng.uniform(size=(ny, nx)) < 0.5).astype(np.uint8)
        h = lib.pico_init(ny, nx, dev(maps.astype(np.complex64)), psi, dev(mask), sampling=lib.PICO_CART_2D, **kw)
        op = opico.cartesian(maps, psi, mask)
    v = (rng.standard_normal((K, ny, nx)) + 1j * rng.standard_normal((K, ny, nx))).astype(np.complex64)
    vt = dev(v)
    ut = torch.empty_like(vt)
    lib.pico_apply_cov(h, vt, ut, K)
    torch.cuda.synchronize()
    lib.pico_destroy(h)
    cov = opico.Covariance(op, 0.1, cg)
    u = ut.cpu().numpy()
    for k in range(K):
        ref = cov.apply(v[k].astype(np.complex128))
        err = np.linalg.norm(u[k] - ref) / np.linalg.norm(ref)
        print(f"  probe {k}: rel err {err:.2e}", flush=True)
        assert err < TOL
