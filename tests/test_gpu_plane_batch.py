"""Planes in one pass where a batch has more planes than the GPU has CUs (48 x 96
points have a variant of their own there): bit for bit the three passes, which timed
plans keep, and the same as a batch that takes the other variant."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LAME3 = np.array([[1.0, 1.0], [4.0, 2.0], [0.5, 3.0]])


def say(msg):
    print(f"\n[case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("nx,ny", [(48, 96), (96, 48)])
def test_many_planes(nx, ny, layout):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_00822_amd import Plan
    shape, n, k = (16, ny, nx), 9, 4          # 288 work items; two solves: 64
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(nx)
    probs = [dict(grid=0, phase=torch.from_numpy(rng.integers(0, 3, size=shape).astype(np.uint8)).to(dev), lame=LAME3,
                  f=torch.from_numpy(rng.normal(size=(3,) + shape).astype(np.float32)).to(dev)) for _ in range(n)]
    outs = []
    for timing, batch in ((False, n), (False, 2), (True, n)):
        say(f"{n} solves of {shape} layout {layout}, {batch} at once, timed {timing}")
        plan = Plan([shape], prec="f32", max_batch=batch, timing=timing)
        plan.set_schedule("layout", 0, layout)
        out, reps, _ = plan.solve_batch(probs, tol=1e-12, max_iter=k)
        torch.cuda.synchronize()
        outs.append((out, [r.residual for r in reps]))
        plan.close()
    for out, res in outs[1:]:
        assert res == outs[0][1]
        for a, b in zip(out, outs[0][0]):
            for name in a:
                assert torch.equal(a[name], b[name]), name
