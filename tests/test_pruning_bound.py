"""The lower bound behind the assignment's exact pruning, checked on the CPU.

For candidate k of pixel p, D of Eq. (3) is evaluated in FP32 as
  A = fl(fl(lambda dcp) + fl((1 - lambda) fl(sc / np)))      (Eq. (1))
  B = fl(1 + fl(gamma fl(sw / np)))                           (Eq. (2))
  D = fl(fl(A B) + fl(ds spw))                                (Eq. (3))
with sc >= dcp >= 0 (sums of colour distances, p itself first), sw >= 0,
lambda in [0, 1], gamma >= 0, spw >= 0.  The kernel skips the walk when
LB = fl(fl(lambda dcp) + fl(ds spw)) cannot beat the best D so far; that is
exact only if LB <= D for every such operand, which holds because FP32
rounding is monotone.  These draws cover ordinary, tiny, huge and tied
operands; numpy's float32 operations round like the kernel's.
"""
import numpy as np
import pytest

f32 = np.float32


def _d_and_lb(dcp, sc, sw, n, ds, lam, gamma, spw):
    with np.errstate(over="ignore", invalid="ignore"):
        np1 = (n + 1).astype(f32)
        qc = sc / np1
        qw = sw / np1
        A = lam * dcp + (f32(1.0) - lam) * qc
        B = f32(1.0) + gamma * qw
        D = A * B + ds * spw
        LB = lam * dcp + ds * spw
    return D, LB


def _draw(rng, size, scale):
    dcp = (rng.random(size) * scale).astype(f32)
    sc = (dcp + (rng.random(size) * scale * 40).astype(f32)).astype(f32)
    sw = (rng.random(size) * 40).astype(f32)
    n = rng.integers(0, 2000, size)
    ds = (rng.random(size) * 5000).astype(f32)
    return dcp, sc, sw, n, ds


@pytest.mark.parametrize("scale", [1e-30, 1e-6, 1.0, 1e4, 1e30])
@pytest.mark.parametrize("lam,gamma,spw", [(0.5, 64.0, 0.0961), (0.0, 64.0, 0.0961), (1.0, 0.0, 0.0961),
                                          (0.3, 7.0, 0.0), (0.5, 0.0, 0.25), (1.0, 50.0, 1e-3)])
def test_lower_bound_never_exceeds_d(scale, lam, gamma, spw):
    rng = np.random.default_rng(7)
    dcp, sc, sw, n, ds = _draw(rng, 200_000, scale)
    D, LB = _d_and_lb(dcp, sc, sw, n, ds, f32(lam), f32(gamma), f32(spw))
    finite = np.isfinite(D)
    assert finite.any()
    assert (LB[finite] <= D[finite]).all()
    # an infinite D is still >= its bound
    assert (LB[~finite & ~np.isnan(D)] <= D[~finite & ~np.isnan(D)]).all()


def test_bound_is_tight_without_path_and_contour_terms():
    """With lambda = 1 (or sc = 0) and sw = 0 the bound is D itself: ties between
    a bound and the best D really occur, which is why a tied bound is skipped
    only for a higher slot."""
    rng = np.random.default_rng(3)
    dcp, sc, sw, n, ds = _draw(rng, 10_000, 10.0)
    D, LB = _d_and_lb(dcp, sc, np.zeros_like(sw), n, ds, f32(1.0), f32(64.0), f32(0.1))
    assert (D == LB).all()


# ---- the bound as the kernels evaluate it: fused operations, the low 4 bits of its
# FP32 pattern replaced by the slot, compared as integers with threshold(best)

def _fma(a, b, c):
    return (a.astype(np.float64) * b.astype(np.float64) + np.asarray(c, np.float64)).astype(f32)


def _bits(v):
    return np.ascontiguousarray(v, f32).view(np.uint32)


def _threshold(best):
    return np.maximum(best * f32(1.0 + 2.0 ** -16), f32(2.0 ** -70))


def _candidate(rng, size, scale, reach, lam, gamma, spw):
    """Texels, centres and pixels; D of Eq. (3) for path sums that begin with the pixel
    itself, and the key of bound_keys (slot 8, the largest)."""
    f = (rng.normal(0, 1, (size, 3)) * scale).astype(f32)
    c = (f + rng.normal(0, 1, (size, 3)) * scale * rng.choice([0.0, 1e-6, 0.1, 1.0], (size, 1))).astype(f32)
    px, py = rng.integers(0, 5000, (2, size)).astype(f32)
    cx = (px + rng.uniform(-reach, reach, size)).astype(f32)
    cy = (py + rng.uniform(-reach, reach, size)).astype(f32)
    with np.errstate(over="ignore", invalid="ignore", under="ignore"):
        d = (f - c).astype(f32)
        ax, ay = px - cx, py - cy
        dcp = (d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2]
        # sums over the path: the pixel's own term, and others that are often nothing
        n = rng.integers(0, 1500, size)
        more = (rng.random(size) * rng.choice([0.0, 0.0, 1.0, 100.0], size)).astype(f32)
        sc = dcp + more * dcp
        sw = (rng.random(size) * n * rng.choice([0.0, 0.0, 1.0], size)).astype(f32)
        np1 = (n + 1).astype(f32)
        A = lam * dcp + (f32(1.0) - lam) * (sc / np1)
        B = f32(1.0) + gamma * (sw / np1)
        D = A * B + (ax * ax + ay * ay) * spw
        fused = _fma(d[:, 2], d[:, 2], _fma(d[:, 1], d[:, 1], d[:, 0] * d[:, 0]))
        lb = _fma(ax * ax + ay * ay, np.full(size, spw, f32), lam * fused)
    return D, (_bits(lb) & np.uint32(0xFFFFFFF0)) | np.uint32(8)


@pytest.mark.parametrize("scale", [1e-22, 1e-18, 1e-6, 1.0, 60.0, 1e15])
@pytest.mark.parametrize("lam,gamma,spw", [(0.5, 64.0, 0.0961), (0.0, 64.0, 0.0961), (1.0, 0.0, 0.0961),
                                          (1.0, 0.0, 0.0), (0.3, 7.0, 0.0), (0.5, 0.0, 1e-30)])
def test_fused_key_leaves_no_winner_out(scale, lam, gamma, spw):
    """A candidate is left out when its key exceeds threshold(best) with the low bits
    set.  With best = D itself, the smallest best that D does not beat, it never is."""
    rng = np.random.default_rng(11)
    for reach in (0.5, 40.0, 3000.0):
        D, key = _candidate(rng, 60_000, scale, reach, f32(lam), f32(gamma), f32(spw))
        ok = np.isfinite(D)
        assert ok.any()
        limit = _bits(_threshold(D[ok])) | np.uint32(15)
        assert (key[ok] <= limit).all()
        # and the margin is small: twice D's bound is above D's limit where it is normal
        big = ok & (D > 1e-20) & (D < 1e30)
        above = _bits((key & np.uint32(0xFFFFFFF0)).view(f32)[big] * f32(2.0))
        tight = (key & np.uint32(0xFFFFFFF0)).view(f32)[big] > f32(0.6) * D[big]
        assert (above[tight] > (_bits(_threshold(D[big])) | np.uint32(15))[tight]).all()


def test_keys_order_like_bounds_and_never_reach_the_outside_mark():
    """Integers compare like the bounds; infinity stays below a NaN and both below the
    mark of a slot outside the grid, which exceeds every limit."""
    v = np.array([0.0, 1e-45, 1e-20, 1.0, 3.4e38, np.inf], f32)
    keys = (_bits(v) & np.uint32(0xFFFFFFF0)) | np.uint32(0)
    assert (np.diff(keys.astype(np.int64)) >= 0).all()
    limit_inf = _bits(_threshold(f32(np.inf))) | np.uint32(15)
    assert (keys <= limit_inf).all() and 0x7FC00000 > limit_inf
    assert 0xFFFFFFFF > 0x7FFFFFFF >= limit_inf          # the limit without pruning
