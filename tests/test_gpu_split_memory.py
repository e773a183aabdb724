"""The split phase-encode operator lives within the bytes that pico_estimate_bytes
describes: every block that it takes is reported, an allocator or a serving budget
of exactly those bytes is enough, and its results do not depend on spare room.
The maps carry the partly sampled class's phase; the pseudo-replica right-hand side,
which reads the same maps, is checked against an operator of the dense form (whose
maps carry none).

Tolerance of that check: the two operators' products and coil sums are each off by
about eps (log2(ny) + nc) <= 6e-8 * 15, and a regularised solve (lambda 0.1:
condition number <= 11) passes on at most that multiple: 2e-5 for the pair.
"""
import numpy as np
import pytest

import workloads

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

KINDS = ("acs2", "uniform2", "uniform3", "two3", "random", "all")


def _mask(kind, ny):
    j, rng = np.arange(ny), np.random.default_rng(ny)
    if kind == "acs2":          # class 0 full, class 1 partly sampled
        return workloads.cart_mask_1d(ny, 2, 12)
    if kind in ("uniform2", "uniform3"):
        return workloads.cart_mask_1d(ny, int(kind[-1]))
    if kind == "two3":          # classes 0 and 1 full, class 2 partly sampled
        return ((j % 3 != 2) | (rng.uniform(size=ny) < 0.3)).astype(np.uint8)
    if kind == "all":
        return np.ones(ny, np.uint8)
    return (rng.uniform(size=ny) < 0.5).astype(np.uint8)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _problem(kind, ny, nx=10, nc=4, **kw):
    rng = np.random.default_rng(ny + nx)
    return dict(ny=ny, nx=nx, maps=_dev(workloads.coil_maps(ny, nx, nc, rng).astype(np.complex64)),
                psi=workloads.noise_cov(nc, rng), mask=_dev(_mask(kind, ny)), lam=0.1, cg_iters=4, probe_tile=5, **kw)


@pytest.fixture(scope="module")
def lib():
    from paper_2605_09590_amd import pico as lib
    lib.load()
    yield lib
    lib.pico_set_allocator()


def _run(lib, p, fn):
    """(op_bytes, accumulators) of one call on a fresh operator."""
    h = lib.pico_init(**p)
    acc = [torch.zeros(p["ny"] * p["nx"], dtype=torch.float64, device="cuda:0") for _ in range(3)]
    try:
        by = lib.pico_op_bytes(h)
        fn(h, lib.make_accum(*acc))
        torch.cuda.synchronize()
    finally:
        lib.pico_destroy(h)
    return by, acc


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("kind,ny", [*((k, 96) for k in KINDS), ("acs2", 320)])
def test_described_bytes_are_all_it_takes(lib, kind, ny, storage):
    print(f"case: {kind} {ny}x10, storage {storage}, allocator of the described bytes", flush=True)
    p = _problem(kind, ny, storage=storage)
    noise_map = lambda h, a: lib.pico_noise_map(h, 3, 0, 7, 0, a)  # noqa: E731
    _, want = _run(lib, p, noise_map)
    d, keep = lib.make_desc(**p)
    resident, peak = lib.pico_estimate_bytes(d)
    live = {}

    def alloc(n):
        if sum(live.values()) + n > peak:
            return 0
        q = torch.cuda.caching_allocator_alloc(n)
        live[q] = n
        return q

    def free(q):
        live.pop(q)
        torch.cuda.caching_allocator_delete(q)

    lib.pico_set_allocator(alloc, free)
    h = lib.pico_init(**p)
    try:
        assert sum(live.values()) == resident == lib.pico_op_bytes(h)[0]
    finally:
        lib.pico_destroy(h)
    by, got = _run(lib, p, noise_map)
    lib.pico_set_allocator()
    assert live == {} and by == (resident, peak)
    for x, y in zip(want, got):
        assert torch.equal(x, y)


def test_served_in_exactly_the_described_bytes(lib):
    for kinds in (("acs2",), ("acs2", "two3", "uniform2")):
        ps = [_problem(k, 96) for k in kinds]
        budget = sum(lib.pico_estimate_bytes(lib.make_desc(**p)[0])[1] for p in ps)
        print(f"case: {kinds} 96x10 served in {budget} bytes", flush=True)
        want = [_run(lib, p, lambda h, a: lib.pico_noise_map(h, 3, 0, 7, 0, a))[1] for p in ps]
        srv = lib.Server(budget, len(ps), 2)
        accs = [[torch.zeros(96 * 10, dtype=torch.float64, device="cuda:0") for _ in range(3)] for _ in ps]
        torch.cuda.synchronize()
        for p, a in zip(ps, accs):
            srv.submit(3, 0, 7, lib.make_accum(*a), **p)
        srv.wait_idle(60.0)
        info = srv.poll()
        st = srv.cache_stats()
        srv.close()
        torch.cuda.synchronize()
        assert [r["status"] for r in info] == [0] * len(ps) and st["resident_ops"] == len(ps)
        for w, a in zip(want, accs):
            for x, y in zip(w, a):
                assert torch.equal(x, y)


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("kind,ny", [("acs2", 64), ("acs2", 96), ("acs2", 320), ("two3", 96), ("two3", 288), ("acs2", 512)])
def test_replica_right_hand_side(lib, kind, ny, storage):
    print(f"case: replicas, {kind} {ny}x10, storage {storage}, against the dense form", flush=True)
    pmr = lambda h, a: lib.pico_pmr_baseline(h, 5, 2, 9, a)  # noqa: E731
    _, got = _run(lib, _problem(kind, ny, storage=storage), pmr)
    _, ref = _run(lib, _problem(kind, ny, storage=storage, normal_form=2), pmr)
    err = [float((x - y).norm() / y.norm()) for x, y in zip(got, ref)]
    print(f"  rel diff {err}", flush=True)
    assert max(err) < 2e-5
