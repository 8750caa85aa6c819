"""The staged AoS step's launch shapes (launch.h), compiled for the host, over
the sizes a set can have: every launch holds fewer than 2^32 threads (HIP
refuses more), its threads and its tile's staging are within the kernel's
bounds, and every tile starts on a 16-byte boundary.  No GPU is used."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1710_03462_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"

MEMORY = 288 << 30  # of one card: the largest buffer of records
MAX_N = 2 ** 31 - 1


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if not os.path.exists(HIPCC) or shutil.which("gcc") is None:
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("aos") / "aos_shape_check")
    subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-I", CSRC,
                    os.path.join(HERE, "aos_shape_check.cpp"), "-o", out],
                   check=True, capture_output=True)
    return out


@pytest.mark.parametrize("integ", range(6))  # every integrator code
@pytest.mark.parametrize("aligned", [0, 1])
def test_every_default_shape_can_be_launched(exe, integ, aligned):
    cases = []
    for stride in list(range(12, 300)) + [400, 768, 776, 1000]:
        top = min(MAX_N, MEMORY // stride)
        sizes = {1, 255, (128 << 20) // stride, (512 << 20) // stride + 1, top // 8, top // 4,
                 top // 3, top // 2, top - 1, top}
        sizes |= {min(top, (1 << 36) // stride + d) for d in (-200, -1, 0, 1, 200)}
        cases += [(integ, aligned, n, stride, 0) for n in sorted(sizes)]
    out = subprocess.run([exe], input="\n".join(" ".join(map(str, c)) for c in cases), check=True,
                         capture_output=True, text=True).stdout.split()
    assert len(out) == 2 * len(cases)
    for (_, _, n, stride, _), tile, block in zip(cases, map(int, out[0::2]), map(int, out[1::2])):
        case = (n, stride, tile, block)
        assert block % 64 == 0 and 64 <= block <= 1024, case
        assert tile % 16 == 0 and tile * stride <= 48 * 1024, case
        assert -(-n // tile) * block < 2 ** 32, case
