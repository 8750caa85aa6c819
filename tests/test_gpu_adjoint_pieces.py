"""The adjoint's pieces: every way that checkpoint intervals, step counts and
renewal points cut a trajectory, in both bounded shift tiers, gives the same
bits as one checkpoint per 20-step block, and the oracle's values."""
import ctypes

import numpy as np
import pytest

import synth_inputs as si

torch = pytest.importorskip("torch")
soax = pytest.importorskip("paper_1710_03462_amd")

pytestmark = pytest.mark.gpu

N = 259
ABC = (1.0, 0.8, 0.6)


def _run(x0, target, dt, nsteps, k):
    abc = (ctypes.c_double * 3)(*ABC)
    xT, tape = soax.forward_ckpt(x0, abc, dt, nsteps, k)
    loss, lam = soax.sqdist_loss(xT, target)
    gx, gabc = soax.adjoint(tape, lam, abc, dt, nsteps, k)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in (xT, loss, gx, gabc)]


@pytest.mark.parametrize("dt", [5e-3, 2e-2])  # shifts up to 0.012 and 0.048
@pytest.mark.parametrize("nsteps", [1, 10, 19, 20, 21, 40, 61])
def test_pieces_agree_bit_for_bit_and_with_the_oracle(ref, dt, nsteps):
    x0, target = (torch.from_numpy(a).cuda() for a in si.adjoint_inputs(N, seed=nsteps))
    want = _run(x0, target, dt, nsteps, 20)
    for k in (1, 2, 5, 7, 8, 9, 10, 11, 16, 19, 21, 33, 40, 64):
        got = _run(x0, target, dt, nsteps, k)
        for what, g, w in zip(("xT", "loss", "grad_x0", "grad_abc"), got, want):
            assert np.array_equal(g, w), (k, what)
    h = x0.cpu().numpy()
    rxT = ref.rk2_forward(h, list(ABC), dt, nsteps)
    _, lam = ref.sqdist_loss(rxT, target.cpu().numpy())
    rgx, rgabc = ref.adjoint(h, lam, list(ABC), dt, nsteps)
    assert np.abs(want[0] - rxT).max() <= 1e-12 * si.BOX_L
    assert np.abs(want[2] - rgx).max() <= 1e-6 * np.abs(rgx).max()
    assert np.all(np.abs(want[3] - rgabc) <= 1e-6 * np.abs(rgabc).max())


@pytest.mark.parametrize("dt", [5e-3, 2e-2])
@pytest.mark.parametrize("nsteps,k", [(1, 1), (20, 20), (40, 20), (61, 16), (61, 7), (100, 33)])
def test_a_small_set_equals_its_part_of_a_large_one(dt, nsteps, k):
    # up to 2^15 particles a quad of lanes takes each; a particle's results do
    # not depend on it, nor do the sums but for their order
    n = (1 << 15) + 1
    x0, target = (torch.from_numpy(a).cuda() for a in si.adjoint_inputs(n, seed=k))
    large = _run(x0, target, dt, nsteps, k)
    total = np.zeros(3)
    for part in (slice(0, n - 1), slice(n - 1, n)):
        small = _run(x0[:, part].contiguous(), target[:, part].contiguous(), dt, nsteps, k)
        assert np.array_equal(small[0], large[0][:, part])
        assert np.array_equal(small[2], large[2][:, part])
        total += small[3]
    # 2^15 terms of at most a few units each, summed twice in different orders
    assert np.abs(total - large[3]).max() <= 1e-12 * n


@pytest.mark.parametrize("parts", [1, 1023, 1024, 1025, 8192, 8193, 16384])
def test_partial_sums_of_every_batch_remainder(parts):
    # one partial sum per 256 particles; whole numbers, so every order of
    # summation gives the same exact result
    n = 256 * parts - 3
    xT = torch.arange(3 * n, device="cuda", dtype=torch.float64).remainder_(5).reshape(3, n)
    loss, lam = soax.sqdist_loss(xT, torch.zeros_like(xT))
    assert loss.item() == (xT * xT).sum().item()
    assert torch.equal(lam, 2.0 * xT)
