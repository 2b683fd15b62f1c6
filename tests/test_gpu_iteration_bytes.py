"""lsfft_iteration_bytes by the kernels that a plan runs: the passes' streams of timed
plans, whole planes in one launch, and small 2D solves whose spectra stay in LDS."""
import sys

import pytest

pytestmark = pytest.mark.gpu

GREEN, X, Y, REDUCE, CGUPD = 2, 0, 1, 3, 4


def say(msg):
    print(f"\n[case] {msg}", flush=True)
    sys.stdout.flush()


def bytes_of(shape, **kw):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_00822_amd import Plan
    say(f"iteration bytes {shape} {kw}")
    plan = Plan([shape], **kw)
    got = [plan.iteration_bytes(k) for k in (X, Y, GREEN, REDUCE, CGUPD)]
    plan.close()
    n = 1
    for v in shape:
        n *= v
    return got, n, n // 2 * (16 if kw["prec"] == "f64" else 8)   # voxels, one half-spectrum stream


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_2d(prec):
    got, n, c = bytes_of((64, 64), prec=prec)
    assert got == [0, 0, 6 * c, 0, 0]
    for shape, kw in (((64, 64), dict(timing=True)), ((96, 64), {}), ((64, 12), {})):
        got, n, c = bytes_of(shape, prec=prec, **kw)
        assert got[:3] == [6 * c + n, 0, 12 * c] and got[3] > 0 and got[4] == 0
    got, n, c = bytes_of((64, 64), prec=prec, scheme="cg")
    assert got[0] == 6 * c + n and got[4] == 12 * c


def test_3d():
    for kw, y in (({}, 0), (dict(timing=True), 24)):
        got, n, c = bytes_of((16, 48, 64), prec="f32", **kw)
        assert got[:3] == [12 * c + n, y * c, 21 * c] and got[3] > 0
