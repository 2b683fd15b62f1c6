"""What a program chooses for the x and y passes runs, also on grids whose planes are
otherwise transformed in one launch: by hand, by the cache and by the tuner.  Timed
plans run the passes as chosen, so an untimed plan has to give their bits; the other
radix orders (variant 2) give other bits than the defaults."""
import json
import os
import sys

import numpy as np
import pytest

from oracle import lsfft_oracle as O
import gen

pytestmark = pytest.mark.gpu

LAME10 = O.lame_from_young(gen.Material.two_phase(1.0, 10.0).table())
SHAPE = (48, 64, 64)
K_YPASS = 1


def say(msg):
    print(f"\n[case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def solve(torch, plan):
    rng = np.random.default_rng(5)
    phase = torch.from_numpy((rng.random(SHAPE) < 0.3).astype(np.uint8)).cuda()
    f = torch.from_numpy(rng.normal(size=(3,) + SHAPE).astype(np.float32)).cuda()
    out, rep = plan.solve(phase, LAME10, f, tol=1e-12, max_iter=4)
    torch.cuda.synchronize()
    return out["eps"], rep.residual


def run(torch, choices=(), cache=None, tmp_path=None, timing=False):
    from paper_2601_00822_amd import Plan
    if cache is not None:
        path = tmp_path / "tune.json"
        path.write_text(json.dumps(cache))
        os.environ["LSFFT_TUNE_CACHE"] = str(path)
    try:
        plan = Plan([SHAPE], prec="f32", timing=timing)
    finally:
        os.environ.pop("LSFFT_TUNE_CACHE", None)
    say(f"{SHAPE} choices {choices} cache {cache} timed {timing}")
    for kind, n, v in choices:
        plan.set_schedule(kind, n, v)
        assert plan.schedule(kind, n)[0] == v
    out = solve(torch, plan) + (plan.iteration_bytes(K_YPASS) == 0,)
    plan.close()
    return out


def same(torch, a, b):
    return torch.equal(a[0], b[0]) and a[1] == b[1]


@pytest.mark.parametrize("kind,n", [("x", 64), ("y", 64)])
def test_chosen_variants_run(torch, tmp_path, kind, n):
    default = run(torch)
    assert default[2]
    for v in (1, 2):
        want = run(torch, [(kind, n, v)], timing=True)
        for got in (run(torch, [(kind, n, v)]), run(torch, cache={f"f32/3d/{kind}/{n}": v}, tmp_path=tmp_path)):
            assert same(torch, got, want) and not got[2]
    assert not torch.equal(want[0], default[0])
    # back to the default; a tuner's choice of the plane launch, and its end by hand
    assert same(torch, run(torch, [(kind, n, 2), (kind, n, 0)]), default)
    tuned = {f"f32/3d/{kind}/{n}": 2, "f32/3d/plane/64x64x48": 1}
    assert run(torch, cache=tuned, tmp_path=tmp_path)[2]
    got = run(torch, [(kind, n, 2)], cache=tuned, tmp_path=tmp_path)
    assert same(torch, got, want) and not got[2]
    tuned = {"f32/3d/plane/64x64x48": 0}
    got = run(torch, cache=tuned, tmp_path=tmp_path)
    assert same(torch, got, default) and not got[2]


def test_tuner_times_what_runs(torch, tmp_path):
    """One grid that may take the plane launch, alone and with one that shares its
    lengths but runs the passes; plans made from the cache run what the tuner chose."""
    from paper_2601_00822_amd import Plan
    for shapes in ([SHAPE], [SHAPE, (4, 64, 256), (4, 256, 64)]):
        cache = tmp_path / f"tune{len(shapes)}.json"
        say(f"autotune {shapes}")
        plan = Plan(shapes, prec="f32", max_batch=2)
        table = plan.autotune(iters=6, cache_path=str(cache))
        got = json.loads(cache.read_text())
        take = got["f32/3d/plane/64x64x48"]
        assert take in (0, 1) and "f32/3d/plane/256x64x4" not in got
        us = {(e["kind"], e["len"]): e["us"] for e in table if e["chosen"]}
        if len(shapes) == 1:
            # per iteration: the x, two y and the outer launches, or less by the plane launch
            passes = us["x", 64] + 2 * us["y", 64] + us["outer", 48]
            assert us["layout", 0] <= passes * (1 + 1e-9)
            assert (us["layout", 0] < passes * (1 - 1e-9)) == bool(take)
        tuned = solve(torch, plan)
        assert (plan.iteration_bytes(K_YPASS) == 0) == bool(take)
        plan.close()
        os.environ["LSFFT_TUNE_CACHE"] = str(cache)
        try:
            again = Plan(shapes, prec="f32", max_batch=2)
        finally:
            del os.environ["LSFFT_TUNE_CACHE"]
        assert same(torch, solve(torch, again), tuned)
        assert (again.iteration_bytes(K_YPASS) == 0) == bool(take)
        again.close()


def test_default_y_variant_is_reported(torch):
    from paper_2601_00822_amd import Plan
    for shapes, want in (([(32, 256, 256)], 1), ([(4, 256, 16)], 0), ([(4, 256, 16), (32, 256, 256)], 1)):
        say(f"schedule of {shapes}")
        plan = Plan(shapes, prec="f32")
        assert plan.schedule("y", 256)[0] == want
        plan.set_schedule("y", 256, 0)
        assert plan.schedule("y", 256)[0] == 0
        plan.close()
