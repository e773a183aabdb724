"""The FP64 primal of compressed sensing over its line lengths: the
reconstruction of every built row and column length against the FP64 oracle,
one and more wavelet levels, and the replica batch against it.

Tolerance: both sides run the same FP64 iteration, differing by the rounding of
their transforms (1e-15 a step, a few steps); pico_recon hands the image out in
FP32, so 6e-8 per value remains: 2e-7.  The replica noise is drawn in FP32
(6e-8 a draw times a few ulp of its logarithm and sine), which the difference
quotient passes on: 2e-6.
"""
import numpy as np
import pytest

import workloads
from oracle import cs as ocs
from oracle import pico as opico

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nx,nc,levels,nrep", [
    (64, 128, 3, 2, 3),
    (128, 96, 5, 3, 2),       # coils that do not fill the last round of wavefronts
    (96, 160, 1, 1, 2),
    (160, 64, 4, 4, 5),
    (192, 256, 2, 2, 2),
    (256, 64, 2, 6, 2),       # levels down to blocks of 4 x 1
    (288, 64, 2, 1, 2),
    (64, 288, 2, 1, 2),
    (384, 64, 2, 1, 2),
    (64, 384, 3, 1, 2),
    (512, 64, 2, 1, 2),
    (64, 512, 2, 1, 2),
    (576, 64, 1, 1, 2),
    (64, 640, 2, 1, 2),
    (768, 64, 1, 1, 2),
    (64, 768, 2, 1, 2),
])
def test_primal_lengths(ny, nx, nc, levels, nrep):
    from paper_2605_09590_amd import pico as lib
    T, lam, sigma = 4, 1e-3, 1e-2
    print(f"case: {ny}x{nx}, {nc} coils, {levels} levels, FISTA {T}, {nrep} replicas", flush=True)
    rng = np.random.default_rng(ny + 7 * nx)
    maps = workloads.coil_maps(ny, nx, nc, rng)
    psi = workloads.noise_cov(nc, rng)
    mask = (rng.uniform(size=(ny, nx)) < 0.6).astype(np.uint8)
    k = (rng.standard_normal((nc, ny, nx)) + 1j * rng.standard_normal((nc, ny, nx))).astype(np.complex64) * mask
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    h = lib.pico_init(ny, nx, dev(maps.astype(np.complex64)), psi, dev(mask), sampling=lib.PICO_CART_2D, probe_tile=nrep,
                      recon=lib.PICO_CS_FISTA_L1WAV, kdata=dev(k), fista_iters=T, cs_lambda=lam, wavelet_levels=levels)
    x = torch.empty(ny, nx, dtype=torch.complex64, device="cuda:0")
    lib.pico_recon(h, x)
    acc_t = [torch.zeros(ny, nx, dtype=torch.float64, device="cuda:0") for _ in range(3)]
    lib.pico_pmr_cs(h, 11, 0, nrep, sigma, lib.make_accum(*acc_t))
    torch.cuda.synchronize()
    lib.pico_destroy(h)
    op = opico.cartesian(maps.astype(np.complex64).astype(np.complex128), psi, mask)
    f = ocs.FistaL1Wavelet(op, lam, T, levels)
    Li = np.linalg.inv(np.linalg.cholesky(psi))
    bw = np.tensordot(Li, k.astype(np.complex128), axes=1) * mask
    ref = f.recon(bw)
    err = np.linalg.norm(x.cpu().numpy() - ref) / np.linalg.norm(ref)
    acc = ocs.pmr_cs(f, bw, 11, 0, nrep, sigma)
    errs = [np.linalg.norm(t.cpu().numpy() - acc[n]) / np.linalg.norm(acc[n])
            for t, n in zip(acc_t, ("sum", "sum_im", "sumsq"))]
    print(f"  recon rel err {err:.2e}, replica sums {max(errs):.2e}", flush=True)
    assert err < 2e-7
    assert max(errs) < 2e-6
