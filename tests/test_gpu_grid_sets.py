"""GPU parity of the grid path where its launches change form, against the FP64
oracle: few rows (several wavefronts on the same rows, a share of the coils each,
down to fewer coils than wavefronts), the first launch with one wavefront per row
group, and planes beyond the last-level cache (the probes go through in sets, the
last one smaller).

Tolerances: products as in the column pass's test, an FP32 transform pair and coil
sum off by eps (log2(Ny Nx) + nc) <= 6e-8 * 22 = 1.3e-6 times the condition number
11 of lambda 0.1, rounded up to 2e-5; maps, where a pixel's sum of products is
smaller than its terms, the 1e-4 of the other grid tests.
"""
import numpy as np
import pytest

import workloads
from oracle import nufft as onufft
from oracle import pico as opico

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

CG = 3


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _operator(lib, kind, ny, nx, nc, tile):
    rng = np.random.default_rng(ny * 1000 + nx + nc)
    maps = workloads.coil_maps(ny, nx, nc, rng)
    psi = workloads.noise_cov(nc, rng)
    kw = dict(lam=0.1, cg_iters=CG, probe_tile=tile)
    if kind == "spiral":
        traj = workloads.spiral_traj(max(ny, nx), 1, 12, 256).astype(np.float32)
        h = lib.pico_init(ny, nx, _dev(maps.astype(np.complex64)), psi, None, sampling=lib.PICO_NONCART,
                          traj=_dev(traj), nsamples=traj.shape[0], **kw)
        return h, opico.Covariance(onufft.NonCartOp(maps, psi, traj.astype(np.float64)), 0.1, CG)
    mask = (rng.uniform(size=(ny, nx)) < 0.5).astype(np.uint8)
    h = lib.pico_init(ny, nx, _dev(maps.astype(np.complex64)), psi, _dev(mask), sampling=lib.PICO_CART_2D, **kw)
    return h, opico.Covariance(opico.cartesian(maps, psi, mask), 0.1, CG)


@pytest.mark.parametrize("kind,ny,nx,nc,K,check", [
    ("cart2d", 192, 160, 1, 3, (0, 2)),             # one coil: three wavefronts of four have none
    ("cart2d", 192, 160, 5, 16, (0, 15)),           # 768 row groups, the last with several wavefronts
    ("cart2d", 192, 160, 5, 17, (0, 16)),           # the first with one
    ("cart2d", 96, 64, 6, 3, (0, 2)),
    ("cart2d", 64, 288, 3, 2, (0, 1)),              # three rows a group, lanes left over
    ("cart2d", 64, 576, 5, 2, (0, 1)),
    ("cart2d", 64, 768, 3, 2, (0, 1)),              # two wavefronts
    ("spiral", 64, 256, 3, 2, (0, 1)),              # 512 points, half rows
    ("spiral", 80, 32, 7, 3, (0, 2)),
    ("cart2d", 256, 256, 7, 71, (0, 35, 36, 70)),   # 249 MiB of planes: sets of 36 and 35
    ("spiral", 288, 32, 3, 2, (0, 1)),              # padded columns with a plan of their own
    ("spiral", 320, 48, 2, 2, (0, 1)),
])
def test_products(kind, ny, nx, nc, K, check):
    from paper_2605_09590_amd import pico as lib
    print(f"case: {kind} {ny}x{nx}, {nc} coils, {K} probes, lambda 0.1, CG {CG}", flush=True)
    h, cov = _operator(lib, kind, ny, nx, nc, K)
    rng = np.random.default_rng(K)
    v = (rng.standard_normal((K, ny, nx)) + 1j * rng.standard_normal((K, ny, nx))).astype(np.complex64)
    vt = _dev(v)
    ut = torch.empty_like(vt)
    lib.pico_apply_cov(h, vt, ut, K)
    torch.cuda.synchronize()
    lib.pico_destroy(h)
    for k in check:
        ref = cov.apply(v[k].astype(np.complex128))
        err = np.linalg.norm(ut[k].cpu().numpy() - ref) / np.linalg.norm(ref)
        print(f"  probe {k}: rel err {err:.2e}", flush=True)
        assert err < 2e-5


@pytest.mark.parametrize("ny,nx,nc,K", [
    (192, 160, 3, 4),      # several wavefronts on the same rows
    (256, 256, 7, 35),     # one wavefront, one set
    (256, 256, 7, 71),     # sets: every probe drawn from its own index
])
def test_drawn_probes(ny, nx, nc, K):
    from paper_2605_09590_amd import pico as lib
    print(f"case: map of {ny}x{nx}, {nc} coils, {K} probes, lambda 0.1, CG {CG}", flush=True)
    h, cov = _operator(lib, "cart2d", ny, nx, nc, K)
    runs = []
    for _ in range(4):     # the same bits every time: no tile is overwritten while it is read
        acc_t = [torch.zeros(ny * nx, dtype=torch.float64, device="cuda:0") for _ in range(3)]
        lib.pico_noise_map(h, 5, 2, K, 0, lib.make_accum(*acc_t), None)
        torch.cuda.synchronize()
        runs.append(acc_t[0].cpu().numpy())
    lib.pico_destroy(h)
    ref = opico.noise_map(cov, 5, 2, K)["sum"].ravel()
    err = np.linalg.norm(runs[0] - ref) / np.linalg.norm(ref)
    print(f"  rel err {err:.2e}", flush=True)
    assert err < 1e-4
    assert all(np.array_equal(runs[0], r) for r in runs[1:])
