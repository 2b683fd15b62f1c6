"""The surrogate at the edges of its transform and mode kernels: every grid
size, the fewest and the most kept modes, mode counts that leave the last
group of eight half full, one sample, and one sample more than a tile of the
mode products.  Bars and reasons are those of the parity test of the whole
surrogate (fp32 sums and the rare flipped bf16 rounding)."""
import numpy as np
import pytest

from oracle import fno_oracle as F

import test_gpu_fno as T

pytestmark = pytest.mark.gpu

CASES = [
    # (n, modes, hidden, layers, cin, cout, batch)
    (8, 1, 32, 1, 3, 6, 1),       # 4 modes: half a group
    (8, 4, 64, 2, 2, 9, 3),       # most modes of the smallest grid
    (16, 5, 32, 2, 3, 6, 2),      # 500 modes: the last group half full
    (16, 8, 128, 1, 6, 3, 33),    # most modes, batch one past a tile
    (32, 7, 32, 1, 1, 1, 1),      # odd mode count, smallest channels
    (32, 16, 256, 1, 32, 32, 2),  # most modes, widest projection and channels
]


@pytest.mark.parametrize("n,modes,hidden,layers,cin,cout,batch", CASES)
def test_forward_and_gradients_at_the_edges(n, modes, hidden, layers, cin, cout, batch):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_00822_amd.fno import FnoArch, Surrogate, pack, unpack
    arch = FnoArch(n=n, modes=modes, hidden=hidden, layers=layers, cin=cin, cout=cout)
    T.say(f"surrogate edges {arch} batch {batch}")
    oa = T.oracle_arch(arch)
    p = T.random_params(arch, 11)
    rng = np.random.default_rng(12)
    x = rng.normal(size=(batch, cin) + (n,) * 3).astype(np.float32)
    t = rng.normal(size=(batch, cout) + (n,) * 3).astype(np.float32)
    s = Surrogate(arch, max_batch=batch)
    s.set_params(pack(arch, p))
    xd, td = torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda()
    y = s.forward(xd).cpu().numpy().astype(np.float64)
    yo = F.forward(p, x.astype(np.float64), oa, bf16=True)
    assert T.rel(y, yo) < 1e-3
    assert np.abs(y - yo).max() < 1e-2 * np.abs(yo).max()
    loss, g = s.loss_grad(xd, td)
    lo, go = F.backward(p, x.astype(np.float64), t.astype(np.float64), oa, bf16=True)
    assert abs(loss - lo) <= 1e-4 * abs(lo)
    gg = unpack(arch, g.cpu().numpy())
    for k in go:
        assert T.rel(gg[k], go[k]) < 5e-3, (k, T.rel(gg[k], go[k]))
        assert np.abs(gg[k] - go[k]).max() <= 3e-2 * np.abs(go[k]).max(), k
    s.close()
