"""The assignment kernels step along a linear path by counting the carries of
a 32-bit accumulator (start 2^31, increment F = ceil(2^32 |d_minor| / n), or
2^32 - 1 for a diagonal).  This checks, on the CPU, that the carry count after
i steps equals the path's minor-axis offset floor((2 i |d_minor| + n) / (2 n))
of Sec. II-B for every step: exhaustively for short paths, on random pairs up
to the bound n < 46340 the argument gives."""
import math

import numpy as np
import pytest


def _increment(am: int, n: int) -> int:
    if am == n:
        return 0xFFFFFFFF
    # the same double-precision expression the kernels evaluate
    return int(math.ceil(float(am) * 4294967296.0 / float(n)))


def _check(n: int, am: int) -> None:
    i = np.arange(1, n, dtype=np.uint64)
    F = np.uint64(_increment(am, n))
    carries = (np.uint64(1 << 31) + i * F) >> np.uint64(32)
    exact = (2 * i.astype(np.int64) * am + n) // (2 * n)
    assert (carries.astype(np.int64) == exact).all(), (n, am)


def test_exhaustive_short_paths():
    for n in range(2, 257):
        for am in range(0, n + 1):
            _check(n, am)


@pytest.mark.parametrize("seed", range(4))
def test_random_long_paths(seed):
    rng = np.random.default_rng(seed)
    for n in rng.integers(257, 46340, 40):
        n = int(n)
        for am in (0, 1, n // 3, n // 2, n - 1, n, int(rng.integers(0, n + 1))):
            _check(n, am)


def test_ties_round_toward_the_endpoint():
    # n = 4, |d_minor| = 2: the segment passes exactly between two pixels at
    # i = 1 and i = 3 (i s = 1/2, 3/2); offsets floor((4 i + 4) / 8) = 1, 1, 2
    # take the pixel nearer the endpoint
    F = _increment(2, 4)
    assert [((1 << 31) + i * F) >> 32 for i in (1, 2, 3)] == [1, 1, 2]


f32 = np.float32


def _short_increment(am, n, ulps):
    """The rule for n < 1023: an FP32 reciprocal that may be `ulps` off, a product, a
    bound below 2^32 (what it converts to an integer is in range) and a saturating sum."""
    with np.errstate(divide="ignore", invalid="ignore"):
        r = f32(1.0) / n.astype(f32)
        r = (r.view(np.int32) + np.int32(ulps)).view(f32)
        v = (am.astype(f32) * r) * f32(2.0 ** 32)
    v = np.fmin(v, f32(float.fromhex("0x1.fffffep31")))
    assert (v >= 0).all() and (v < 2.0 ** 32).all()
    return np.minimum(v.astype(np.uint64) + np.uint64(1025), np.uint64(0xFFFFFFFF))


@pytest.mark.parametrize("ulps", [-1, 0, 1])
def test_short_paths_by_the_reciprocal(ulps):
    """Every (minor, major) extent below 1023, at every step."""
    for n in range(1, 1023):
        am = np.arange(0, n + 1)
        F = _short_increment(am, np.full(n + 1, n), ulps)
        i = np.arange(1, n, dtype=np.uint64)
        carries = (np.uint64(1 << 31) + i[None, :] * F[:, None]) >> np.uint64(32)
        exact = (2 * i.astype(np.int64)[None, :] * am[:, None] + n) // (2 * n)
        assert (carries.astype(np.int64) == exact).all(), n
    # no steps: 0 times an infinite reciprocal is bounded, too
    assert _short_increment(np.array([0]), np.array([0]), 0)[0] == 0xFFFFFFFF


def test_kernel_source_bounds_the_conversion():
    """A float of 2^32 or more, or NaN, must not reach the conversion to an integer."""
    import os
    import re
    from paper_1903_07149_amd import build
    text = open(os.path.join(build.CSRC, "scalp_device.h")).read()
    body = re.search(r"unsigned step_increment\(int am, int n\) \{.*?\n\}", text, re.S).group(0)
    assert "(unsigned)(sf" not in body and "fminf(sf * 4294967296.0f, 0x1.fffffep31f)" in body
