"""The partial sums of the loss and the adjoint on many streams and threads
at once: every call gets its own sums."""
import threading

import pytest

torch = pytest.importorskip("torch")
soax = pytest.importorskip("paper_1710_03462_amd")

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
