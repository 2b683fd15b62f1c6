"""Calls from several threads whose kernels are the same functions with other amounts of
dynamic LDS: each gives the bits that it gives alone, and none is refused."""
import sys
import threading

import numpy as np
import pytest

from oracle import lsfft_oracle as O
import gen

pytestmark = pytest.mark.gpu

LAME10 = O.lame_from_young(gen.Material.two_phase(1.0, 10.0).table())


def say(msg):
    print(f"\n[case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def overlap(torch, makers, rounds=12):
    """Each maker returns a call; the calls alone, then all threads at once."""
    alone, bad = [], []
    for make in makers:
        call = make()
        alone.append([t.clone() for t in call()])
        torch.cuda.synchronize()

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                call = makers[k]()
                for _ in range(rounds):
                    out = call()
                    torch.cuda.current_stream().synchronize()
                    if not all(torch.equal(a, b) for a, b in zip(out, alone[k])):
                        bad.append((k, "other bits"))
        except Exception as e:   # a refused launch
            bad.append((k, repr(e)))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(makers))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad


def test_small_2d_solves(torch):
    from paper_2601_00822_amd import Plan

    def maker(shape):
        def make():
            rng = np.random.default_rng(shape[0])
            phase = torch.from_numpy((rng.random(shape) < 0.3).astype(np.uint8)).cuda()
            f = torch.from_numpy(rng.normal(size=(2,) + shape)).cuda()
            torch.cuda.synchronize()
            plan = Plan([shape], prec="f64")
            return lambda: list(plan.solve(phase, LAME10, f, tol=1e-12, max_iter=6)[0].values())
        return make

    say("2D solves of 16 x 16, 48 x 64 and 64 x 64 from three threads")
    overlap(torch, [maker((16, 16)), maker((48, 64)), maker((64, 64))])


def test_surrogates(torch):
    from paper_2601_00822_amd.fno import FnoArch, Surrogate

    def maker(modes):
        def make():
            arch = FnoArch(n=32, modes=modes, hidden=32, layers=1)
            n = sum(int(np.prod(s)) * (2 if name.startswith("r") else 1) for name, s in arch.layout())
            rng = np.random.default_rng(modes)
            params = torch.from_numpy((0.1 * rng.normal(size=n)).astype(np.float32)).cuda()
            x = torch.from_numpy(rng.normal(size=(2, arch.cin, 32, 32, 32)).astype(np.float32)).cuda()
            torch.cuda.synchronize()
            model = Surrogate(arch, max_batch=2)
            model.set_params(params)
            return lambda: [model.forward(x)]
        return make

    say("surrogates of 9, 12 and 16 modes from three threads")
    overlap(torch, [maker(9), maker(12), maker(16)])
