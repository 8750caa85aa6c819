"""The batch's default shape on both sides of the size from which it streams."""
import numpy as np
import pytest

import synth_inputs as si

torch = pytest.importorskip("torch")
soax = pytest.importorskip("paper_1710_03462_amd")

pytestmark = pytest.mark.gpu

EDGE = -(-(128 << 20) // 36)  # particles of f64 positions and f32 velocities that span 128 MiB


@pytest.mark.parametrize("total,per_thread", [(EDGE, 2), (EDGE - 1, 1)])
def test_default_shape_by_size_and_same_results(total, per_thread):
    sizes = [1_000_001, 3, 512, total - 1_000_516]
    dts, abc = np.array([1e-3, 1e-2, 2e-3, 8e-3]), np.full((4, 3), 1.1)
    out = []
    for mode in (soax.GRAPH, soax.PER_SET):
        sets = []
        for s, n in enumerate(sizes):
            ps = soax.ParticleSet(si.BASE_FIELDS, n, aos=False)
            ps.fill(seed=s)
            sets.append(ps)
        b = soax.Batch(sets)
        assert b.get_config() == (256, per_thread, 65536)
        b.step(dts, abc, 2, mode=mode)
        torch.cuda.synchronize()
        out.append([t.clone() for ps in sets for t in ps.soa])
        b.close()
        for ps in sets:
            ps.close()
    assert all(torch.equal(x, y) for x, y in zip(*out))
