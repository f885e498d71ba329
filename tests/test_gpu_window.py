"""Window form of the assignment (the candidate rule of Algorithm 1) on the GPU against
the oracle: one pass bit-exact (labels, with uncovered pixels keeping theirs),
whole runs bit-exact against the fixed-point-mean oracle and >= 99.9 % label
agreement against the FP64-mean oracle.  Also reports how far the window form
and the 3x3 grid form end up from each other."""
import os

import numpy as np
import pytest

from paper_1903_07149_amd import synth
from paper_1903_07149_amd._lib import ASSIGN_WINDOW
from gpu_util import dev, host, needs_gpu, perturbed_state, say, torch

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.fixture(scope="module", autouse=True)
def _threads(orc):
    orc.set_threads(min(16, os.cpu_count() or 1))


def _scalp(W, H, k, **kw):
    from paper_1903_07149_amd.scalp import Scalp
    return Scalp(W, H, k, assign_mode=ASSIGN_WINDOW, **kw)


CASES = [(97, 61, 30), (481, 321, 250), (37, 5, 7), (1, 1, 1), (64, 64, 4096), (300, 200, 2)]
TUNINGS = [dict(), dict(lds_pixels=1), dict(wg_size=256, lds_pixels=900)]


@pytest.mark.parametrize("tune", range(len(TUNINGS)))
@pytest.mark.parametrize("W,H,k", CASES)
def test_window_assign_bit_exact(orc, W, H, k, tune):
    img = synth.make_image(W, H, max(2, W * H // 4000), 10.0, 13)
    g = orc.grid(W, H, k)
    c, e = perturbed_state(orc, g, img.lab, seed=W + 3 * H, jitter=0.3 * g.r + 1)
    prev = np.random.default_rng(1).integers(0, g.num_sp, (H, W)).astype(np.int32)
    s = _scalp(W, H, k, **TUNINGS[tune])
    say("window assign", W, H, k, TUNINGS[tune])
    lbl = host(s.assign(dev(img.lab), dev(img.contour), dev(c), dev(e), labels=dev(prev)))
    ol, _ = orc.assign_window(g, img.lab, orc.wmap(img.contour), c, e, prev)
    assert (lbl == ol).all(), f"{int((lbl != ol).sum())} labels differ"


def _clumped(g, lab, rng, spread):
    """Every barycenter within `spread` pixels of one point, endpoints anywhere."""
    K = g.num_sp
    c = np.empty((K, 5), np.float32)
    ys, xs = rng.integers(0, g.height, K), rng.integers(0, g.width, K)
    c[:, :3] = lab[ys, xs]
    c[:, 3] = np.clip(0.6 * g.width + rng.uniform(-spread, spread, K), 0, g.width - 1)
    c[:, 4] = np.clip(0.4 * g.height + rng.uniform(-spread, spread, K), 0, g.height - 1)
    e = np.stack([rng.integers(0, g.width, K), rng.integers(0, g.height, K)], 1).astype(np.int32)
    return c, e


@pytest.mark.parametrize("prune", [1, 0])
@pytest.mark.parametrize("W,H,k,spread", [
    (16, 16, 4, 30.0), (17, 33, 6, 30.0), (95, 15, 13, 60.0),   # whole, one over, one short of tiles
    (96, 80, 14, 4.0),      # 12 candidates and more: the last that fit and those beyond
    (96, 80, 200, 2.0),     # 200 candidates in few tiles: many batches
    (96, 80, 800, 1.5),     # lists overflow: all clusters are tested, in turns
])
def test_window_tiles_and_lists(orc, W, H, k, spread, prune):
    img = synth.make_image(W, H, 5, 10.0, 17)
    g = orc.grid(W, H, k)
    rng = np.random.default_rng(W + H + k)
    c, e = _clumped(g, img.lab, rng, spread)
    prev = rng.integers(0, g.num_sp, (H, W)).astype(np.int32)
    s = _scalp(W, H, k, exact_pruning=prune)
    say("window lists", W, H, k, spread, prune)
    lab, con = dev(img.lab), dev(img.contour)
    ol, _ = orc.assign_window(g, img.lab, orc.wmap(img.contour), c, e, prev)
    for rep in range(2):                     # the second pass meets counts left at zero
        lbl = host(s.assign(lab, con, dev(c), dev(e), labels=dev(prev)))
        assert (lbl == ol).all(), f"{rep}: {int((lbl != ol).sum())} labels differ"


@pytest.mark.parametrize("W,H,k,spread", [(96, 80, 14, 4.0), (96, 80, 200, 2.0), (96, 80, 800, 1.5)])
def test_window_sums_of_long_lists(orc, W, H, k, spread):
    """A stepped pass with the update's sums: several batches of bins, overflowed
    lists, and pixels that no window contains (their sums go to their old label)."""
    img = synth.make_image(W, H, 5, 10.0, 18)
    g = orc.grid(W, H, k)
    rng = np.random.default_rng(W + H + k)
    c, e = _clumped(g, img.lab, rng, spread)
    prev = rng.integers(0, g.num_sp, (H, W)).astype(np.int32)
    ol, _ = orc.assign_window(g, img.lab, orc.wmap(img.contour), c, e, prev)
    oc, on = orc.update(g, img.lab, ol, c, mode=orc.MEAN_FIXED)
    s = _scalp(W, H, k)
    say("window sums", W, H, k, spread)
    lab, con = dev(img.lab), dev(img.contour)
    C, E, L = dev(c), dev(e), dev(prev)
    N = torch.zeros(g.num_sp, dtype=torch.int32, device="cuda")
    s.prepare(lab, con)
    s.assign_accumulate(C, E, L)
    s.finalize(L, C, E, N)
    assert (host(L) == ol).all()
    assert (host(C) == oc).all() and (host(N) == on).all()


def test_window_paths_beyond_carry_range(orc):
    """W + H beyond 46340: the walks with 64-bit indexes."""
    W, H, k = 46400, 2, 8
    rng = np.random.default_rng(5)
    lab = rng.normal(0, 20, (H, W, 3)).astype(np.float32)
    con = rng.random((H, W)).astype(np.float32)
    g = orc.grid(W, H, k)
    c, e = _clumped(g, lab, rng, 500.0)
    e[:, 0] = np.clip(c[:, 3] + rng.integers(-3000, 3000, g.num_sp), 0, W - 1)
    e[0, 0] = 0
    prev = np.zeros((H, W), np.int32)
    s = _scalp(W, H, k)
    say("window wide", W, H, k)
    lbl = host(s.assign(dev(lab), dev(con), dev(c), dev(e), labels=dev(prev)))
    ol, _ = orc.assign_window(g, lab, orc.wmap(con), c, e, prev)
    assert (lbl == ol).all()


def _compare(orc, img, k, iters):
    H, W = img.contour.shape
    s = _scalp(W, H, k)
    say("window run", W, H, k, iters)
    r = s.run(dev(img.lab), dev(img.contour), iterations=iters)
    lbl, c, e = host(r.labels), host(r.centers), host(r.endpoints)
    fixed = orc.run_window(img.lab, img.contour, k, iterations=iters, mode=orc.MEAN_FIXED)
    assert (lbl == fixed.labels).all(), f"{int((lbl != fixed.labels).sum())} labels differ"
    assert (c == fixed.centres).all() and (e == fixed.endpoints).all()
    plain = orc.run_window(img.lab, img.contour, k, iterations=iters, mode=orc.MEAN_PLAIN)
    assert (lbl == plain.labels).mean() >= 0.999
    grid3 = orc.run(img.lab, img.contour, k, iterations=iters, mode=orc.MEAN_FIXED)
    agree = float((lbl == grid3.labels).mean())
    print(f"{W}x{H} k={k}: window form vs 3x3 form label agreement {agree:.4f}")
    return agree


@pytest.mark.parametrize("W,H,k", [(97, 61, 30), (160, 120, 48)])
def test_window_run_small(orc, W, H, k):
    _compare(orc, synth.make_image(W, H, 6, 10.0, 21), k, 10)


def test_window_run_bsd_shape(orc):
    _compare(orc, synth.workload_image(synth.BSD_SHAPE), 250, 10)


def test_window_run_hd(orc):
    _compare(orc, synth.workload_image(synth.HD), synth.HD.k, 10)


def test_window_graph_replays(orc):
    img = synth.make_image(200, 150, 8, 10.0, 3)
    s = _scalp(200, 150, 60)
    lab, con = dev(img.lab), dev(img.contour)
    say("window graph")
    ref = s.run(lab, con)
    refs = [host(t) for t in (ref.labels, ref.centers, ref.endpoints)]
    c, e, l = s.init_grid(lab, con)
    n = torch.empty_like(ref.counts)
    gr = s.graph(c, e, l, n)
    for rep in range(3):
        s.init_grid(lab, con, out=(c, e, l))
        torch.cuda.synchronize()
        gr.launch()
        for a, b in zip((host(l), host(c), host(e)), refs):
            assert (a == b).all(), rep
    gr.close()


def test_window_mode_rejected_where_unsupported():
    from paper_1903_07149_amd import _lib as L
    from paper_1903_07149_amd.scalp import ScalpBatch
    from paper_1903_07149_amd.soft import SoftScalp
    b = ScalpBatch([(40, 30, 12)], assign_mode=ASSIGN_WINDOW)
    lab = torch.zeros((1200, 3), device="cuda")
    con = torch.zeros((1200,), device="cuda")
    with pytest.raises(L.ScalpError) as ei:
        b.run(lab, con)
    assert ei.value.code == L.SCALP_ERR_UNSUPPORTED
    eng = SoftScalp(32, 32, 16, 1, assign_mode=ASSIGN_WINDOW)
    with pytest.raises(L.ScalpError):
        eng.forward(torch.zeros((1, 32, 32, 3), device="cuda"), torch.zeros((1, 32, 32), device="cuda"))


@pytest.mark.parametrize("W,H,k", [
    (97, 61, 300), (9, 9, 81), (9, 1, 9), (256, 256, 300),    # tiles of 8 with lists, at most 1024
    (264, 256, 300), (17, 17, 289), (1, 700, 350),            # one more; few ids per tile
])
def test_window_runs_of_small_tiles(orc, W, H, k):
    img = synth.make_image(W, H, 5, 10.0, 19)
    s = _scalp(W, H, k)
    say("window small tiles", W, H, k)
    lab, con = dev(img.lab), dev(img.contour)
    ref = orc.run_window(img.lab, img.contour, k, iterations=4, mode=orc.MEAN_FIXED)
    for rep in range(2):
        r = s.run(lab, con, iterations=4)
        assert (host(r.labels) == ref.labels).all(), rep
        assert (host(r.centers) == ref.centres).all() and (host(r.endpoints) == ref.endpoints).all()
