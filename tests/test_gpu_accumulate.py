"""Averages over more shifts than one fetch of descriptors holds, and remainders of
the shifts summed together, against the oracle.  Both sides stop at residual 1e-10;
bar 1e-9 of the largest entry."""
import numpy as np
import pytest

from oracle import lsfft_oracle as O
import gen

pytestmark = pytest.mark.gpu

LAME = O.lame_from_young(gen.Material.two_phase(1.0, 5.0).table())


@pytest.mark.parametrize("shape,nshift", [((16, 16), 1), ((16, 16), 67), ((12, 24), 64), ((4, 6, 8), 65), ((4, 6, 8), 3)])
def test_average(shape, nshift):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_00822_amd import Plan
    print(f"\n[case] {shape} {nshift} shifts", flush=True)
    d = len(shape)
    rng = np.random.default_rng(nshift)
    phase = (rng.random(shape) < 0.3).astype(np.uint8)
    f = rng.normal(size=(d,) + shape)
    shifts = np.stack([rng.integers(0, n, size=nshift) for n in shape], axis=1).astype(np.int32)
    ref, iters = O.translate_average(phase, LAME, f, shifts, tol=1e-10)
    plan = Plan([shape], prec="f64", max_batch=128)
    avg, reps = plan.translate_average(torch.from_numpy(phase).cuda(), LAME, torch.from_numpy(f).cuda(), shifts,
                                       tol=1e-10)
    a = avg.cpu().numpy()
    plan.close()
    assert [r.iters for r in reps] == iters
    assert np.abs(a - ref).max() <= 1e-9 * np.abs(ref).max()
