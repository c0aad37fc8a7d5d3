"""The host rule that sends fp32 contractions to the tiled kernel, compiled by itself: what it accepts can
be launched."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1811_02084_amd", "csrc")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    src, so = str(d / "rule.cpp"), str(d / "rule.so")
    with open(src, "w") as f:
        f.write('#include "einsum_folded_rule.h"\n'
                'extern "C" int fits(int64_t m, int64_t n, int64_t k, int64_t b) { return mtf::folded_fits(m, n, k, b); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, src, "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.fits.argtypes = [ctypes.c_int64] * 4
    return lib


@pytest.mark.parametrize("m,n,fits", [
    (1, 2, True), (4096, 4096, True), (262144, 262144 - 64, True),
    (262144, 262144, False),            # 2^24 tiles of 256 threads: 2^32 in x
    (600_000_000, 80, False), (80, 600_000_000, False), (2**24 * 64, 1, False), ((2**24 - 1) * 64, 1, True)])
def test_launch_limits(rule, m, n, fits):
    assert bool(rule.fits(m, n, 4, 1)) == fits
    assert not fits or ((m + 63) // 64) * ((n + 63) // 64) * 256 < 2**32
    assert not rule.fits(m, n, 4, 65536) and not rule.fits(m, n, 2**31, 1)
