"""Removal where the scan of the tile counts takes one run, just over one run
and several (runs of 4096 tiles of 16384 flags), against the closed form."""
import pytest

torch = pytest.importorskip("torch")
soax = pytest.importorskip("paper_1710_03462_amd")

pytestmark = pytest.mark.gpu

RUN = 4096 * 16384  # particles whose tile counts one run of the scan covers


@pytest.mark.parametrize("n", [RUN - 1, RUN, RUN + 1, 2 * RUN + 16384 * 3 + 17])
@pytest.mark.parametrize("every", [3, 1000])
def test_removal_matches_the_closed_form(n, every):
    ps = soax.ParticleSet([("id", "i32", 1)], n, aos=False)
    ids = torch.arange(n, dtype=torch.int32, device="cuda")
    ps.array("id").copy_(ids)
    g = torch.Generator(device="cuda")
    g.manual_seed(n + every)
    flags = (torch.randint(0, every, (n,), generator=g, device="cuda") == 0).to(torch.uint8)
    flags[-1] = 1
    n_new = n - int(flags.sum())
    assert ps.remove_flagged(flags) == n_new
    holes = torch.nonzero(flags[:n_new]).flatten()
    movers = n_new + torch.nonzero(flags[n_new:] == 0).flatten().flip(0)
    want = ids[:n_new].clone()
    want[holes] = ids[movers]
    assert torch.equal(ps.array("id"), want)
    ps.close()
