"""The library's fp64 sincos (csrc/trig.h) next to the multiples of pi/2,
where the reduced argument is tiny and one of the two results with it: the
relative error stays within two ulp there as elsewhere.  The reference is
exact: x - k pi/2 in integers of 400 bits and two terms of the sine's series.
No GPU is used; the check program is compiled for the host with hipcc."""
import importlib.util
import math
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1710_03462_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"
BITS = 400


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if not os.path.exists(HIPCC) or shutil.which("gcc") is None:
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("trig") / "trig_near_check")
    subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O2", "-ffp-contract=off",
                    "-I", CSRC, os.path.join(HERE, "trig_near_check.cpp"), "-o", out],
                   check=True, capture_output=True)
    return out


@pytest.fixture(scope="module")
def half_pi():
    spec = importlib.util.spec_from_file_location("gen", os.path.join(CSRC, "gen_trig_constants.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    return int(gen.pi_fraction() / 2 * 2 ** BITS)


def scaled(x):
    """x * 2^BITS as an integer, exactly (x a multiple of 2^-BITS)."""
    m, d = x.as_integer_ratio()
    return m * (2 ** BITS // d)


# Two roundings of r (half an ulp each) and none of its size after them: 1 ulp;
# 2 is what trig.h states for every argument of its range.
@pytest.mark.parametrize("k0,k1,sign", [(1, 5, 1), (1, 4097, -1), (4097, 65537, 1),
                                        (65537, 333772, 1)])
def test_two_ulp_next_to_multiples_of_half_pi(exe, half_pi, k0, k1, sign):
    step = max(1, (k1 - k0) // 40000)
    xs, ks = [], []
    for k in list(range(k0, k1, step)) + [k for k in (29, 116, 204552) if k0 <= k < k1]:
        near = float(sign) * (k * half_pi / 2 ** BITS)
        for x in (near, math.nextafter(near, -math.inf), math.nextafter(near, math.inf)):
            xs.append(x)
            ks.append(sign * k)
    out = subprocess.run([exe], input="\n".join(x.hex() for x in xs), check=True,
                         capture_output=True, text=True).stdout.split()
    assert len(out) == 2 * len(xs)
    worst, at = 0.0, None
    for x, k, s, c in zip(xs, ks, out[0::2], out[1::2]):
        r = scaled(x) - k * half_pi
        exact = r - r * r * r // (6 << (2 * BITS))  # |r| < 2^-32: the rest is below 2^-160 of it
        # sin x = (., cos r, -sin r, -cos r)[k mod 4] and so on: the tiny one
        got, neg = ((s, 0), (c, 1), (s, 1), (c, 0))[k % 4]
        got = -float.fromhex(got) if neg else float.fromhex(got)
        err = abs(scaled(got) - exact) / 2 ** BITS / math.ulp(exact / 2 ** BITS)
        if err > worst:
            worst, at = err, x
    assert worst <= 2.0, (worst, at)
