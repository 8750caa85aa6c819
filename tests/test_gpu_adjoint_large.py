"""The adjoint of sets of more than 2^15 particles, which take one lane each:
the straight-line kernels for k and nsteps that are multiples of 20 (segments
of one block and of several, and a shorter last one), the general ones for the
others, with positions in arrays and in records, in both bounded shift tiers.
The quads that take smaller sets give the same bits particle by particle."""
import ctypes

import pytest

import synth_inputs as si

torch = pytest.importorskip("torch")
soax = pytest.importorskip("paper_1710_03462_amd")
from paper_1710_03462_amd import autograd  # noqa: E402

pytestmark = pytest.mark.gpu

N = (1 << 15) + 1
NSTEPS = 200
ABC = (ctypes.c_double * 3)(1.0, 0.8, 0.6)


def _inputs(n, seed):
    return [torch.from_numpy(a).cuda() for a in si.adjoint_inputs(n, seed=seed)]


def _run(x0, target, dt, k):
    xT, tape = soax.forward_ckpt(x0, ABC, dt, NSTEPS, k)
    loss, lam = soax.sqdist_loss(xT, target)
    gx, gabc = soax.adjoint(tape, lam, ABC, dt, NSTEPS, k)
    return xT, loss, gx, gabc


@pytest.mark.parametrize("dt", [5e-3, 2e-2])  # shifts up to 0.012 and 0.048
def test_every_interval_gives_the_same_bits(dt):
    x0, target = _inputs(N, 11)
    want = _run(x0, target, dt, 20)
    for k in (40, 60, 80, 200, 1000, 1, 7, 10, 16, 32, 33, 50):
        for what, g, w in zip(("xT", "loss", "grad_x0", "grad_abc"), _run(x0, target, dt, k), want):
            assert torch.equal(g, w), (k, what)
    for part in (slice(0, N - 1), slice(N - 1, N)):  # taken by quads
        small = _run(x0[:, part].contiguous(), target[:, part].contiguous(), dt, 60)
        assert torch.equal(small[0], want[0][:, part])
        assert torch.equal(small[2], want[2][:, part])


@pytest.mark.parametrize("dt", [5e-3, 2e-2])
@pytest.mark.parametrize("k", [20, 60, 7, 16])
@pytest.mark.parametrize("stride,offset", [(48, 8), (24, 0)])
def test_positions_in_records(dt, k, stride, offset):
    x0, target = _inputs(N, k)
    xT, loss, gx, gabc = _run(x0, target, dt, k)

    def records(x=None):
        rec = torch.full((N, stride), 0xA5, dtype=torch.uint8, device="cuda")
        if x is not None:
            rec[:, offset:offset + 24] = x.t().contiguous().view(torch.uint8).view(N, 24)
        return rec.view(-1)

    def positions(rec):
        return rec.view(N, stride)[:, offset:offset + 24].contiguous().view(torch.float64).t()

    rec, lam, grad = records(x0), records(), records()
    tape = autograd.forward_ckpt_records(rec, rec, offset, stride, N, ABC, dt, NSTEPS, k)
    loss_r = autograd.sqdist_loss_records(rec, target, lam, offset, stride, N)
    gabc_r = autograd.adjoint_records(tape, lam, grad, offset, stride, N, ABC, dt, NSTEPS, k)
    assert torch.equal(positions(rec), xT)
    assert torch.equal(loss_r, loss)
    assert torch.equal(positions(grad), gx)
    assert torch.equal(gabc_r, gabc)
    for r in (rec, lam, grad):  # nothing but the positions is written
        r = r.view(N, stride)
        assert (r[:, :offset] == 0xA5).all() and (r[:, offset + 24:] == 0xA5).all()
