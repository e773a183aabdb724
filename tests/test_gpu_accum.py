"""GPU parity of the accumulation over probe slices (fewer probes than slices, a
count that they do not divide, both slice counts, both field layouts), against the
FP64 oracle: sum, imaginary sum and sum of squares.

Tolerance: the sums are FP64; what is off is the FP32 solve behind them, eps times
(log2(Ny Nx) + nc) <= 6e-8 * 22 = 1.3e-6 at the condition number 11 of lambda 0.1,
on terms that a sum of a few probes may cancel by a factor of a few: the 1e-4 of
the other map tests.
"""
import numpy as np
import pytest

import workloads
from oracle import pico as opico

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout,n,K", [
    ("cart1d", 64, 1), ("cart1d", 64, 5), ("cart1d", 64, 37),      # sixteen slices at most
    ("cart1d", 192, 3), ("cart1d", 192, 6),                        # four
    ("cart2d", 64, 1), ("cart2d", 64, 37), ("cart2d", 192, 6),
])
def test_accumulated_moments(layout, n, K):
    from paper_2605_09590_amd import pico as lib
    print(f"case: {layout} {n}x{n}, 3 coils, {K} probes, lambda 0.1, CG 3", flush=True)
    rng = np.random.default_rng(n + K)
    maps = workloads.coil_maps(n, n, 3, rng)
    psi = workloads.noise_cov(3, rng)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    mask = (rng.uniform(size=n if layout == "cart1d" else (n, n)) < 0.5).astype(np.uint8)
    mask[n // 2] = 1
    kw = dict(sampling=lib.PICO_CART_2D) if layout == "cart2d" else {}
    h = lib.pico_init(n, n, dev(maps.astype(np.complex64)), psi, dev(mask), lam=0.1, cg_iters=3, probe_tile=K, **kw)
    acc = [torch.zeros(n * n, dtype=torch.float64, device="cuda:0") for _ in range(3)]
    lib.pico_noise_map(h, 7, 1, K, 0, lib.make_accum(*acc), None)
    torch.cuda.synchronize()
    lib.pico_destroy(h)
    mask2 = mask if layout == "cart2d" else np.repeat(mask[:, None], n, axis=1)
    ref = opico.noise_map(opico.Covariance(opico.cartesian(maps, psi, mask2), 0.1, 3), 7, 1, K)
    for t, key in zip(acc, ("sum", "sum_im", "sumsq")):
        r = ref[key].ravel()
        err = np.linalg.norm(t.cpu().numpy() - r) / np.linalg.norm(r)
        print(f"  {key}: rel err {err:.2e}", flush=True)
        assert err < 1e-4
