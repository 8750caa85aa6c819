"""The partial sums of the loss and the adjoint on many streams and threads
at once: every call gets its own sums."""
import ctypes
import threading

import pytest

torch = pytest.importorskip("torch")
soax = pytest.importorskip("paper_1710_03462_amd")
from paper_1710_03462_amd import _lib  # noqa: E402

pytestmark = pytest.mark.gpu


def _input(i, n):
    """A position block whose loss against zero is a known whole number."""
    x = torch.zeros((3, n), dtype=torch.float64, device="cuda")
    x[i % 3, : i + 1] = 2.0
    return x, 4.0 * (i + 1)


@pytest.mark.parametrize("n", [1, 300, 100_000, 12_000_000])  # the last takes no kept buffer
def test_many_streams_without_waiting(n):
    zero = torch.zeros((3, n), dtype=torch.float64, device="cuda")
    jobs = [_input(i % min(n, 12), n) for i in range(12)]
    streams = [torch.cuda.Stream() for _ in jobs]
    torch.cuda.synchronize()
    out = []
    for _ in range(5):
        for (x, want), s in zip(jobs, streams):
            with torch.cuda.stream(s):
                out.append((soax.sqdist_loss(x, zero, want_grad=False)[0], want))
    torch.cuda.synchronize()
    assert [t.item() for t, _ in out] == [w for _, w in out]


@pytest.mark.parametrize("shared", [True, False])
def test_many_threads(shared):
    n, per, wrong = 5000, 50, []
    zero = torch.zeros((3, n), dtype=torch.float64, device="cuda")
    common = torch.cuda.Stream()
    torch.cuda.synchronize()

    def work(i):
        x, want = _input(i, n)
        torch.cuda.synchronize()
        with torch.cuda.stream(common if shared else torch.cuda.Stream()):
            out = [soax.sqdist_loss(x, zero, want_grad=False)[0] for _ in range(per)]
            torch.cuda.current_stream().synchronize()
            wrong.extend(t.item() for t in out if t.item() != want)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(12)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


@pytest.mark.parametrize("n", [300, 100_000])
def test_beside_another_threads_capture(n):
    # a capture in the global mode is invalidated by unsafe calls of any
    # thread; the C call with memory of the caller's makes none
    zero = torch.zeros((3, n), dtype=torch.float64, device="cuda")
    x, want = _input(7, n)
    y = torch.zeros(64, device="cuda")
    loss = torch.zeros(16, dtype=torch.float64, device="cuda")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    dev = torch.cuda.current_device()
    rows = [(ctypes.c_void_p * 3)(*(t[d].data_ptr() for d in range(3))) for t in (x, zero)]
    codes = []

    def work(first, times):
        torch.cuda.set_device(dev)
        for i in range(first, first + times):
            codes.append(_lib.lib().soax_sqdist_loss(
                rows[0], rows[1], n, None, ctypes.c_void_p(loss.data_ptr() + 8 * i),
                ctypes.c_void_p(s.cuda_stream)))

    work(0, 4)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        y.add_(1.0)
        t = threading.Thread(target=work, args=(4, 8))
        t.start()
        t.join()
        y.add_(1.0)
    for k in range(3):
        g.replay()
        work(12 + k, 1)
        torch.cuda.synchronize()
        assert y.unique().tolist() == [2.0 * (k + 1)]
    assert codes == [0] * 15
    assert loss.tolist() == [want] * 15 + [0.0]
