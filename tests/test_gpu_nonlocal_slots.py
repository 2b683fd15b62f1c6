"""Normal equations of batches with more tiles than partial sums: the same as the sum of
its samples' own, which take a slot per tile.  FP64 sums of the same products in another
order: 1e-12 of the largest entry, as against the oracle."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,degree", [(0, 8), (1, 8), (1, 2)])
def test_batch_is_the_sum_of_its_samples(form, degree):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_00822_amd import nonlocal_normal_equations
    shape, delta, ns = (16, 32, 32), 2.5, 40
    print(f"\n[case] nonlocal batch of {ns} {shape} form {form} degree {degree}", flush=True)
    sys.stdout.flush()
    g = torch.Generator(device="cuda").manual_seed(degree)
    u, gam = (torch.randn((ns, 3) + shape, dtype=torch.float64, device="cuda", generator=g) for _ in range(2))
    G, b, bb = nonlocal_normal_equations(u, gam, degree, delta, form)
    parts = [nonlocal_normal_equations(u[k:k + 1].contiguous(), gam[k:k + 1].contiguous(), degree, delta, form)
             for k in range(ns)]
    Gs, bs, bbs = (sum(p[i] for p in parts) for i in range(3))
    np.testing.assert_allclose(G, Gs, rtol=0, atol=1e-12 * np.abs(Gs).max())
    np.testing.assert_allclose(b, bs, rtol=0, atol=1e-12 * np.abs(Gs).max() ** 0.5 * bbs ** 0.5)
    np.testing.assert_allclose(bb, bbs, rtol=1e-13)
