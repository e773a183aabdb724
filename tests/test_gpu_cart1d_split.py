"""GPU parity of the split phase-encode normal operator against the FP64 oracle:
every column length of each split, with a class to transform and without (full
and empty classes only), ragged probe counts, each entry into the CG (probe
draw, right-hand side in memory, plain application), and the mask rule itself.

Tolerance: a transform pair and the coil sum are off by about
eps (log2(ny) + nc) <= 6e-8 * 15 = 9e-7; the regularised solves (lambda 0.1:
condition number <= 11) pass on at most that multiple: 1e-5.
"""
import numpy as np
import pytest

import workloads
from oracle import pico as opico

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

TOL = 1e-5
LENGTHS = (64, 96, 128, 160, 192, 256, 288, 320, 384, 512)


def _mask(kind, ny, rng):
    j = np.arange(ny)
    if kind == "acs2":          # one class full, one partly sampled
        return workloads.cart_mask_1d(ny, 2, 12)
    if kind == "odd2":          # one class empty, one partly sampled
        return ((j % 2 == 1) & (rng.uniform(size=ny) < 0.6)).astype(np.uint8)
    if kind == "uniform3":      # one of three full
        return workloads.cart_mask_1d(ny, 3)
    if kind == "two3":          # two of three full, the third partly sampled
        return ((j % 3 != 1) | (rng.uniform(size=ny) < 0.3)).astype(np.uint8)
    if kind == "all":           # nothing to transform, no split
        return np.ones(ny, np.uint8)
    return (rng.uniform(size=ny) < 0.5).astype(np.uint8)


@pytest.mark.parametrize("kind,ny,K", [
    *[("acs2", n, 5) for n in LENGTHS],
    *[("uniform2", n, 3) for n in (64, 320)],
    *[("odd2", n, 9) for n in (64, 160, 320)],
    *[("uniform3", n, 7) for n in (96, 384)],
    *[("two3", n, 4) for n in (96, 192, 288, 384)],
    *[("random", n, 6) for n in (96, 256, 384)],
    ("all", 128, 2),
])
def test_split_lengths(kind, ny, K):
    from paper_2605_09590_amd import pico as lib
    nx, nc, cg = 6, 4, 4
    print(f"case: {kind} {ny}x{nx}, {nc} coils, {K} probes, lambda 0.1, CG {cg}", flush=True)
    rng = np.random.default_rng(ny + K)
    mask = workloads.cart_mask_1d(ny, 2) if kind == "uniform2" else _mask(kind, ny, rng)
    maps = workloads.coil_maps(ny, nx, nc, rng)
    psi = workloads.noise_cov(nc, rng)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    h = lib.pico_init(ny, nx, dev(maps.astype(np.complex64)), psi, dev(mask), lam=0.1, cg_iters=cg, probe_tile=K)
    v = (rng.standard_normal((K, ny, nx)) + 1j * rng.standard_normal((K, ny, nx))).astype(np.complex64)
    ut = torch.empty(K, ny, nx, dtype=torch.complex64, device="cuda:0")
    lib.pico_apply_cov(h, dev(v), ut, K)
    acc_t = [torch.zeros(ny * nx, dtype=torch.float64, device="cuda:0") for _ in range(3)]
    lib.pico_noise_map(h, 3, 1, K, 0, lib.make_accum(*acc_t))
    torch.cuda.synchronize()
    lib.pico_destroy(h)
    cov = opico.Covariance(opico.cartesian(maps, psi, mask), 0.1, cg)
    u = ut.cpu().numpy()
    errs = [np.linalg.norm(u[k] - r) / np.linalg.norm(r)
            for k in range(K) for r in [cov.apply(v[k].astype(np.complex128))]]
    ref = opico.noise_map(cov, 3, 1, K)["sum"].ravel()
    errs.append(np.linalg.norm(acc_t[0].cpu().numpy() - ref) / np.linalg.norm(ref))
    print(f"  rel err up to {max(errs):.2e}", flush=True)
    assert max(errs) < TOL
