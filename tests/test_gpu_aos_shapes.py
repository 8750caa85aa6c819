"""The staged AoS step's default tiles on sets that stream, at every record
size at which the rule changes, against the SoA step of the same particles."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
soax = pytest.importorskip("paper_1710_03462_amd")

pytestmark = pytest.mark.gpu


def _fields(extra, pos):
    f = [("pos", pos, 3), ("vel", "f32", 3), ("acc", "f32", 3)]
    return f + [(f"x{i}", "f32", 1) for i in range(extra)]


# record bytes: f32 36 + 4 extra, f64 48 (with its tail padding) + 8 per two extra
CASES = [(pos, extra, integ)
         for pos, extras, integs in (
             ("f32", (0, 7, 8, 23), ("euler", "euler_acc")),
             ("f64", (0, 4, 5, 26), ("euler", "euler_acc", "rk2_abc", "heun_abc", "rk4_abc")))
         for extra in extras for integ in integs]


@pytest.mark.parametrize("pos,extra,integ", CASES)
def test_streaming_tiles_match_the_soa_step(pos, extra, integ):
    fields = _fields(extra, pos)
    stride = soax.Schema(fields).layout()[1]
    n = (512 << 20) // stride + 37  # beyond the caches; the last tile is partial
    ps = soax.ParticleSet(fields, n)
    ps.fill(seed=extra)
    ps.soa_to_aos()
    for layout in ("soa", "aos"):
        ps.step(layout, integ, 2e-3, 2, abc=[1.0, 0.8, 0.6], wrap=pos == "f64")
    want = [t.clone() for t in ps.soa]
    ps.aos_to_soa()
    for a, (g, w) in enumerate(zip(ps.soa, want)):
        assert torch.equal(g.view(torch.uint8), w.view(torch.uint8)), (stride, a)
    ps.close()


@pytest.mark.parametrize("stride_fields", [6, 8])  # 24- and 32-byte records
def test_small_records(stride_fields):
    fields = [("pos", "f32", 3), ("vel", "f32", 3)]
    fields += [(f"t{i}", "f32", 1) for i in range(stride_fields - 6)]
    n = (128 << 20) // (4 * stride_fields) + 101
    ps = soax.ParticleSet(fields, n)
    ps.fill(seed=1)
    ps.soa_to_aos()
    for layout in ("soa", "aos"):
        ps.step(layout, "euler", 1e-3, 2, wrap=False)
    want = [t.clone() for t in ps.soa]
    ps.aos_to_soa()
    assert all(np.array_equal(g.cpu().numpy(), w.cpu().numpy()) for g, w in zip(ps.soa, want))
    ps.close()


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("extra", [0, 1, 2, 8, 9, 53, 54])  # 36 to 252 bytes
def test_streaming_transpose_round_trip(extra, packed):
    fields = [("id", "i32", 1), ("pos", "f64", 3), ("b", "u8", 1)]
    fields += [(f"x{i}", "f32", 1) for i in range(min(extra, 24))]
    fields += [(f"y{i}", "f64", 3) for i in range(max(0, extra - 49))]
    stride = soax.Schema(fields, packed).layout()[1]
    n = (128 << 20) // stride + 91
    ps = soax.ParticleSet(fields, n, packed=packed)
    ps.fill(seed=extra)
    want = [t.clone() for t in ps.soa]
    ps.soa_to_aos()
    for t in ps.soa:
        t.zero_()
    ps.aos_to_soa()
    for a, (g, w) in enumerate(zip(ps.soa, want)):
        assert torch.equal(g.view(torch.uint8), w.view(torch.uint8)), (stride, a)
    ps.close()
