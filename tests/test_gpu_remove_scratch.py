"""What a removal keeps of the device's memory: no more than the few buffers
that all calls share, however many sets have removed however much."""
import ctypes

import pytest

torch = pytest.importorskip("torch")
soax = pytest.importorskip("paper_1710_03462_amd")
from paper_1710_03462_amd import _lib  # noqa: E402

pytestmark = pytest.mark.gpu

USED_MEM_CURRENT = 7  # hipMemPoolAttrUsedMemCurrent
KEPT = 64 << 20       # of all kept buffers together


def _used():
    """Bytes in use of the stream-ordered memory pool, which torch does not use."""
    L = _lib.lib()
    pool, used = ctypes.c_void_p(), ctypes.c_uint64()
    dev = torch.cuda.current_device()
    assert L.hipDeviceGetDefaultMemPool(ctypes.byref(pool), ctypes.c_int(dev)) == 0
    assert L.hipMemPoolGetAttribute(pool, ctypes.c_int(USED_MEM_CURRENT), ctypes.byref(used)) == 0
    return used.value


@pytest.mark.parametrize("n,every", [(2_000_000, 2), (9_000_000, 3)])
def test_many_sets_keep_no_scratch_of_their_own(n, every):
    torch.cuda.synchronize()
    flags = (torch.arange(n, device="cuda") % every == 0).to(torch.uint8)
    sets = []
    for _ in range(12):
        ps = soax.ParticleSet([("id", "i32", 1)], n, aos=False)
        ps.array("id").copy_(torch.arange(n, dtype=torch.int32, device="cuda"))
        assert ps.remove_flagged(flags) == n - int(flags.sum())
        sets.append(ps)
    torch.cuda.synchronize()
    assert _used() <= KEPT
    for ps in sets:
        ps.close()
    assert _used() <= KEPT


# lists in one buffer with the counts, and (4.1e6 moves and more) by themselves
@pytest.mark.parametrize("n,every", [(300_000, 7), (9_000_000, 7), (9_000_000, 2)])
def test_sets_removed_from_and_closed_at_once_on_many_streams(n, every):
    # the lists of moves are still being read when a set is destroyed
    ids = torch.arange(n, dtype=torch.int32, device="cuda")
    flags = (ids % every == 0).to(torch.uint8)
    n_new = n - int(flags.sum())
    holes = torch.nonzero(flags[:n_new]).flatten()
    movers = n_new + torch.nonzero(flags[n_new:] == 0).flatten().flip(0)
    want = ids[:n_new].clone()
    want[holes] = ids[movers]
    streams = [torch.cuda.Stream() for _ in range(6)]
    torch.cuda.synchronize()
    got = []
    for i in range(24):
        with torch.cuda.stream(streams[i % 6]):
            ps = soax.ParticleSet([("id", "i32", 1)], n, aos=False)
            ps.array("id").copy_(ids)
            assert ps.remove_flagged(flags) == n_new
            got.append(ps.array("id"))
            ps.close()
    torch.cuda.synchronize()
    assert all(torch.equal(g, want) for g in got)
