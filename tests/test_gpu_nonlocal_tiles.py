"""Edges of the nonlocal kernels' tiles against the oracle: both lane shapes
(32 x 8, and 16 x 16 where the x axis ends early), grids one voxel past a
tile, each halo, the padded feature counts (degrees 0 to 8), 2D and 3D, and
the matrix form with one and with two rows of 16 features.  FP64 fields: both
sides add the same products in another order, so the bars are those of the
existing parity tests (1e-12 of the largest entry)."""
import sys

import numpy as np
import pytest

from oracle import nonlocal_oracle as N

pytestmark = pytest.mark.gpu

CASES = [
    # (grid in array order, horizon, degree, form, nsample)
    ((9, 9, 33), 2.0, 1, 0, 1),     # 32 x 8 lanes, one voxel past the tile on every axis; smallest halo
    ((8, 17, 17), 4.5, 3, 0, 2),    # 16 x 16 lanes, one voxel past
    ((5, 33, 16), 5.5, 6, 0, 1),    # halo 5, 16 x 16
    ((12, 8, 40), 6.5, 7, 0, 1),    # halo 6, 32 x 8
    ((65, 33), 7.0, 5, 0, 2),       # 2D, one past the 32 x 64 tile, largest halo
    ((5, 5, 17), 2.5, 6, 1, 2),     # matrix form, 15 rows of features (one tile), one past 16 x 4 x 4
    ((4, 8, 16), 5.0, 7, 1, 1),     # matrix form, 19 rows (two tiles), whole tiles, largest 3D halo
    ((17, 33), 3.0, 2, 1, 2),       # matrix form, 2D
]


def say(msg):
    print(f"\n[case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("shape,delta,deg,form,ns", CASES)
def test_tile_edges(shape, delta, deg, form, ns):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_00822_amd import nonlocal_apply, nonlocal_normal_equations
    say(f"nonlocal tiles {shape} delta {delta} degree {deg} form {form} x{ns}")
    d = len(shape)
    rng = np.random.default_rng(sum(shape) + 31 * deg + form)
    us = [rng.normal(size=(d,) + shape) for _ in range(ns)]
    gs = [rng.normal(size=(d,) + shape) for _ in range(ns)]
    c = rng.normal(size=(form + 1) * (deg + 1))
    U, Gm = (torch.from_numpy(np.stack(v)).cuda() for v in (us, gs))
    G, g, gg = nonlocal_normal_equations(U, Gm, deg, delta, form)
    Gw, gw, ggw = N.normal_equations(us, gs, deg, delta, form)
    np.testing.assert_allclose(G, Gw, rtol=0, atol=1e-12 * np.abs(Gw).max())
    np.testing.assert_allclose(g, gw, rtol=0, atol=1e-12 * np.abs(Gw).max() ** 0.5 * ggw ** 0.5)
    np.testing.assert_allclose(gg, ggw, rtol=1e-13)
    out = nonlocal_apply(U, c, delta, form).cpu().numpy()
    for k in range(ns):
        want = N.apply_operator(c, us[k], delta, form)
        np.testing.assert_allclose(out[k], want, rtol=0, atol=1e-12 * np.abs(want).max(), err_msg=f"sample {k}")


def test_threads_share_no_scratch():
    """Calls that overlap in time, from threads with streams of their own, give the
    bits that they give one after another."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import threading
    from paper_2601_00822_amd import nonlocal_apply, nonlocal_normal_equations
    say("nonlocal calls from three threads")
    jobs = []
    for k, (shape, delta, deg, form) in enumerate([((16, 16, 32), 3.0, 4, 0), ((8, 16, 16), 2.5, 6, 1), ((64, 65), 4.0, 3, 1)]):
        rng = np.random.default_rng(k)
        d = len(shape)
        U, Gm = (torch.from_numpy(rng.normal(size=(2, d) + shape)).cuda() for _ in range(2))
        jobs.append((U, Gm, deg, delta, form, rng.normal(size=(form + 1) * (deg + 1))))

    def run(job):
        U, Gm, deg, delta, form, c = job
        G, g, gg = nonlocal_normal_equations(U, Gm, deg, delta, form)
        return np.array(G), np.array(g), gg, nonlocal_apply(U, c, delta, form).cpu().numpy()

    alone = [run(j) for j in jobs]
    torch.cuda.synchronize()
    bad = []

    def worker(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(10):
                got = run(jobs[k])
                if not all(np.array_equal(a, b) for a, b in zip(got, alone[k])):
                    bad.append(k)

    threads = [threading.Thread(target=worker, args=(k,)) for k in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
