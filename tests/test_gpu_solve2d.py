"""Small 2D solves, which one workgroup iterates: iterate for iterate against the
FP64 oracle at the edges of its range (one row tile and many, odd factors, rounds
of rows or columns per wave, 4096 points and just above, more iterations than one
launch makes).

Bars: FP64 relative strain error 1e-10 and the same iteration count; FP32 1e-5.
"""
import sys

import numpy as np
import pytest

from oracle import lsfft_oracle as O
import gen

pytestmark = pytest.mark.gpu

LAME10 = O.lame_from_young(gen.Material.two_phase(1.0, 10.0).table())
LAME3 = np.array([[1.0, 1.0], [4.0, 2.0], [0.5, 3.0]])
BAR = {"f64": 1e-10, "f32": 1e-5}


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def inputs(shape, nphase, seed):
    rng = np.random.default_rng(seed)
    return rng.integers(0, nphase, size=shape).astype(np.uint8), rng.normal(size=(2,) + tuple(shape))


def check(dev, shape, lame, prec, iters, phase, f):
    import torch
    from paper_2601_00822_amd import Plan
    dt = torch.float64 if prec == "f64" else torch.float32
    f = f if prec == "f64" else f.astype(np.float32).astype(np.float64)
    plan = Plan([shape], prec=prec, scheme="basic")
    for k in iters:
        print(f"\n[case] {shape} {prec} max_iter={k}", flush=True)
        sys.stdout.flush()
        ref = O.solve_basic(phase, lame, f, tol=1e-12, max_iter=k)
        out, rep = plan.solve(torch.from_numpy(phase).to(dev), lame, torch.from_numpy(f).to(dev).to(dt), tol=1e-12,
                              max_iter=k)
        torch.cuda.synchronize()
        assert rep.iters == ref.iters and rep.status == ref.status
        assert abs(rep.residual - ref.residual) <= (1e-9 if prec == "f64" else 1e-4) * ref.residual
        err = O.relative_strain_error_voigt(out["eps"].double().cpu().numpy(), O.to_voigt(ref.eps))
        assert err <= BAR[prec], err
    plan.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("shape", [(16, 16), (16, 256), (256, 16), (24, 48), (48, 24), (128, 32), (32, 128), (96, 32),
                                   (24, 96), (64, 64), (48, 96), (8, 64), (64, 12)])
def test_iterates(dev, shape, prec):
    lame = LAME3 if shape[0] < shape[1] else LAME10
    check(dev, shape, lame, prec, (0, 1, 4), *inputs(shape, len(lame), 7))


def test_more_iterations_than_a_launch(dev):
    # a block of contrast 200: neither converged nor stagnating within 700 iterations
    shape = (16, 24)
    lame = O.lame_from_young(gen.Material.two_phase(1.0, 200.0).table())
    phase = np.zeros(shape, dtype=np.uint8)
    phase[4:12, 4:16] = 1
    check(dev, shape, lame, "f64", (511, 512, 513, 700), phase, gen.bump_force(shape, (7.2, 9.9), 6.0, [0.8, -0.6]))
