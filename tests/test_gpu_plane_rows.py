"""The three plane sizes that fill a CU each, on the row layout: their wave counts, two
LDS buffers and piece mapping are their own.  Bars are those of the other planes: the
bits of the three passes, which timed plans keep, and the FP64 oracle within 1e-5."""
import pytest

from oracle import lsfft_oracle as O
import test_gpu_plane as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(96, 128), (128, 96), (128, 128)])
def test_rows(nx, ny):
    import numpy as np
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_00822_amd import Plan
    dev, shape, k = torch.device("cuda:0"), (96, ny, nx), 2
    P.say(f"{shape} rows")
    phase, f = P.problem(shape, nx + ny)
    ref = O.solve_basic(phase, P.LAME3, f.astype(np.float64), tol=1e-12, max_iter=k)
    outs = []
    for timing in (False, True):
        plan = Plan([shape], prec="f32", scheme="basic", timing=timing)
        plan.set_schedule("layout", 0, 0)
        assert (plan.iteration_bytes(1) == 0) == (not timing)      # the y passes' class
        outs.append(plan.solve(torch.from_numpy(phase).to(dev), P.LAME3, torch.from_numpy(f).to(dev), tol=1e-12,
                               max_iter=k))
        torch.cuda.synchronize()
        plan.close()
    (out, rep), (out3, rep3) = outs
    assert rep.residual == rep3.residual
    for name in out:
        assert torch.equal(out[name], out3[name]), name
    assert rep.iters == ref.iters
    assert abs(rep.residual - ref.residual) <= 1e-4 * ref.residual
    assert O.relative_strain_error_voigt(out["eps"].double().cpu().numpy(), O.to_voigt(ref.eps)) <= 1e-5
