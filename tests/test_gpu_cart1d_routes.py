"""Phase-encode operator on both sides of the rules that choose its kernel by the launch's
size, against the FP64 oracle: whole columns on maps that carry a class phase (few
probes), and the split kernel with one wavefront a workgroup, with several (which share
the fully sampled classes' blocks, the last workgroup ragged) and with no class to
transform.

Tolerance as in the split operator's test: 1e-5.
"""
import numpy as np
import pytest

import workloads
from oracle import pico as opico

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

TOL = 1e-5


def _mask(kind, ny, rng):
    j = np.arange(ny)
    if kind == "acs2":          # one class full, the odd one partly sampled
        return workloads.cart_mask_1d(ny, 2, 12)
    if kind == "odd2":          # one class empty, the odd one partly sampled
        return ((j % 2 == 1) & (rng.uniform(size=ny) < 0.6)).astype(np.uint8)
    if kind == "two3":          # two of three full, the last partly sampled
        return ((j % 3 != 2) | (rng.uniform(size=ny) < 0.3)).astype(np.uint8)
    if kind == "random":        # no split
        return (rng.uniform(size=ny) < 0.5).astype(np.uint8)
    return workloads.cart_mask_1d(ny, int(kind[-1]))      # uniform2, uniform3


@pytest.mark.parametrize("kind,ny,nx,K,storage", [
    # whole columns, the class phase on the maps (none on packed bfloat16 ones)
    ("acs2", 64, 6, 3, 0), ("acs2", 192, 6, 2, 0), ("acs2", 288, 6, 2, 0), ("acs2", 320, 6, 6, 0), ("acs2", 384, 6, 5, 0),
    ("acs2", 256, 6, 1, 1), ("odd2", 512, 6, 9, 0), ("random", 256, 6, 6, 0), ("random", 384, 6, 3, 0),
    # split, one wavefront a workgroup
    ("acs2", 64, 6, 8, 0), ("acs2", 128, 66, 63, 0), ("odd2", 320, 6, 7, 0), ("acs2", 320, 6, 4, 1), ("random", 256, 6, 4, 0),
    # split, several
    ("acs2", 160, 128, 48, 0), ("acs2", 192, 6, 14, 0), ("acs2", 256, 6, 8, 1), ("acs2", 288, 6, 19, 0),
    ("acs2", 320, 6, 31, 0), ("acs2", 384, 6, 16, 0), ("acs2", 512, 256, 15, 0),
    ("two3", 96, 6, 9, 0), ("two3", 288, 6, 11, 0), ("two3", 384, 6, 9, 0),
    # no class to transform
    ("uniform2", 64, 6, 17, 0), ("uniform2", 256, 6, 3, 0), ("uniform2", 256, 6, 9, 0), ("uniform2", 320, 6, 18, 1),
    ("uniform2", 512, 6, 7, 0), ("uniform3", 288, 6, 12, 0),
])
def test_routes(kind, ny, nx, K, storage):
    from paper_2605_09590_amd import pico as lib
    nc, cg = 4, 4
    print(f"case: {kind} {ny}x{nx}, {nc} coils, {K} probes, storage {storage}, lambda 0.1, CG {cg}", flush=True)
    rng = np.random.default_rng(ny + K)
    mask = _mask(kind, ny, rng)
    maps = workloads.coil_maps(ny, nx, nc, rng)
    psi = np.eye(nc, dtype=np.complex128) if storage else workloads.noise_cov(nc, rng)
    if storage:       # maps that bfloat16 holds exactly (unwhitened), so the oracle has the same operator
        ri = np.stack([maps.real, maps.imag], -1).astype(np.float32)
        ri = torch.from_numpy(ri).to(torch.bfloat16).double().numpy()
        maps = ri[..., 0] + 1j * ri[..., 1]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    h = lib.pico_init(ny, nx, dev(maps.astype(np.complex64)), psi, dev(mask), lam=0.1, cg_iters=cg, probe_tile=K,
                      storage=storage)
    v = (rng.standard_normal((K, ny, nx)) + 1j * rng.standard_normal((K, ny, nx))).astype(np.complex64)
    ut = torch.empty(K, ny, nx, dtype=torch.complex64, device="cuda:0")
    lib.pico_apply_cov(h, dev(v), ut, K)
    torch.cuda.synchronize()
    lib.pico_destroy(h)
    cov = opico.Covariance(opico.cartesian(maps, psi, mask), 0.1, cg)
    u = ut.cpu().numpy()
    errs = [np.linalg.norm(u[k] - r) / np.linalg.norm(r)
            for k in sorted({0, K // 2, K - 1}) for r in [cov.apply(v[k].astype(np.complex128))]]
    print(f"  rel err up to {max(errs):.2e}", flush=True)
    assert max(errs) < TOL
