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
                'extern "C" int kernel(int64_t m, int64_t n, int64_t k, int64_t b, int a_k, int b_k) {\n'
                '  return mtf::fp32_kernel(m, n, k, b, a_k, b_k); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, src, "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.kernel.argtypes = [ctypes.c_int64] * 4 + [ctypes.c_int] * 2
    return lib.kernel


GENERIC, TILE16, TILE64 = 0, 1, 2
ORDERS = [(a, b) for a in (0, 1) for b in (0, 1)]


def _tiles(m, n, t):
    return -(-m // t) * -(-n // t)


@pytest.mark.parametrize("m,n", [(1, 2), (4096, 4096), (262144, 262144 - 64), (262144, 262144), (600_000_000, 80),
                                 (80, 600_000_000), (2**24 * 64 - 64, 1), (2**30 - 1, 2), (2**31, 64), (2**40, 3)])
@pytest.mark.parametrize("k", [2, 33, 4096])
def test_launch_limits(rule, m, n, k):
    """What the tiled kernel takes can be launched: ints, grid y, fewer than 2^32 threads in x."""
    for a, b in ORDERS:
        for batch in (1, 65535):
            got = rule(m, n, k, batch, a, b)
            if got != GENERIC:
                assert max(m, n) < 2**30 and _tiles(m, n, 16 if got == TILE16 else 64) * 256 < 2**32
        assert rule(m, n, k, 65536, a, b) == GENERIC and rule(m, n, 2**31, 1, a, b) == GENERIC
    if _tiles(m, n, 64) >= 2**24:
        assert rule(m, n, k, 1, 1, 0) == GENERIC


def test_tiny_outputs_of_a_batch_stay_generic(rule):
    """Where a tile would be nearly empty the thread-per-output kernel is the faster one (measured sides in the
    rule's comment); where it would be full, the tiled ones."""
    for a, b in ORDERS:
        for m, n, k, batch in [(8, 8, 4, 16384), (2, 2, 4, 60000), (4, 4, 4, 65535), (1, 4, 32, 16384)]:
            assert rule(m, n, k, batch, a, b) == GENERIC
        assert rule(16, 16, 16, 1, a, b) == TILE16
        assert rule(64, 64, 64, 512, a, b) == TILE64
        assert rule(1024, 1024, 512, 1, a, b) == TILE64
    assert rule(2, 500000, 2, 1, 1, 0) == GENERIC and rule(1, 500000, 64, 1, 1, 0) == GENERIC
