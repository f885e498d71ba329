"""Images that 32-bit texel offsets or step counters do not serve as a whole (W + H
from 46340 on): work items whose box they serve, and items with an endpoint far
across the image beside them, in every form, with the update's sums."""
import os

import numpy as np
import pytest

from paper_1903_07149_amd import synth
from paper_1903_07149_amd._lib import ASSIGN_GRID3X3, ASSIGN_WINDOW
from gpu_util import dev, host, needs_gpu, perturbed_state, say, torch

pytestmark = [pytest.mark.gpu, needs_gpu]

WIDE = [(46400, 3, 60), (60000, 1, 400), (2, 46338, 90)]


@pytest.fixture(scope="module", autouse=True)
def _threads(orc):
    orc.set_threads(min(16, os.cpu_count() or 1))


def _image(W, H, seed):
    rng = np.random.default_rng(seed)
    step = np.repeat(np.repeat(rng.normal(0, 30, (-(-H // 7), -(-W // 50), 3)), 7, 0), 50, 1)
    lab = (step[:H, :W] + rng.normal(0, 4, (H, W, 3))).astype(np.float32)
    return np.ascontiguousarray(lab), (rng.random((H, W)) ** 4).astype(np.float32)


@pytest.mark.parametrize("mode", [ASSIGN_GRID3X3, ASSIGN_WINDOW])
@pytest.mark.parametrize("prune", [1, 0])
@pytest.mark.parametrize("W,H,k", WIDE)
def test_runs(orc, W, H, k, prune, mode):
    from paper_1903_07149_amd.scalp import Scalp
    lab, con = _image(W, H, 3)
    say("far run", W, H, k, prune, mode)
    r = Scalp(W, H, k, iterations=2, assign_mode=mode, exact_pruning=prune).run(dev(lab), dev(con))
    run = orc.run_window if mode == ASSIGN_WINDOW else orc.run
    ref = run(lab, con, k, iterations=2, mode=orc.MEAN_FIXED)
    assert (host(r.labels) == ref.labels).all()
    assert (host(r.centers) == ref.centres).all() and (host(r.endpoints) == ref.endpoints).all()


@pytest.mark.parametrize("wg", [256, 1024])
@pytest.mark.parametrize("W,H,k", WIDE)
def test_items_with_a_far_endpoint(orc, W, H, k, wg):
    """Every 7th endpoint lies at the other end of the image: beside the items of
    that candidate, which take the 64-bit walks, all others keep the near ones."""
    from paper_1903_07149_amd.scalp import Scalp
    lab, con = _image(W, H, 4)
    g = orc.grid(W, H, k)
    c, e = perturbed_state(orc, g, lab, seed=7, jitter=0.3 * g.r)
    e = e.copy()
    e[::7] = (W - 1, H - 1) - e[::7]
    e[::21] = (-5, H + 3)                                # clamped into the image
    s = Scalp(W, H, k, wg_size=wg)
    say("far endpoints", W, H, k, wg)
    l, cn = dev(lab), dev(con)
    labels = torch.empty((H, W), dtype=torch.int32, device="cuda")
    C, E, N = dev(c), dev(e), torch.zeros(g.num_sp, dtype=torch.int32, device="cuda")
    s.init_grid(l, cn)                                   # packs; the sums are left at zero
    s.assign_accumulate(C, E, labels)
    s.finalize(labels, C, E, N, project=0)
    clamped = np.clip(e, 0, (W - 1, H - 1)).astype(np.int32)
    ol, _, _ = orc.assign(g, lab, orc.wmap(con), c, clamped)
    assert (host(labels) == ol).all()
    oc, on = orc.update(g, lab, ol, c, mode=orc.MEAN_FIXED)
    assert (host(C) == oc).all() and (host(N) == on).all()


def test_batch_with_a_wide_image(orc):
    from paper_1903_07149_amd.scalp import ScalpBatch
    shapes = [(97, 61, 30), (46400, 3, 60), (160, 120, 48)]
    data = [_image(w, h, 10 + i) for i, (w, h, _) in enumerate(shapes)]
    say("far batch")
    for wg in (256, 512, 1024):
        b = ScalpBatch(shapes, iterations=2, wg_size=wg)
        _, _, l, _ = b.run(dev(np.concatenate([d[0].reshape(-1, 3) for d in data])),
                           dev(np.concatenate([d[1].reshape(-1) for d in data])))
        l = host(l)
        for (p0, p1, H, W), (w, h, k), (lab, con) in zip(b.pixel_slices(), shapes, data):
            ref = orc.run(lab, con, k, iterations=2, mode=orc.MEAN_FIXED)
            assert (l[p0:p1].reshape(H, W) == ref.labels).all(), (wg, w, h)


@pytest.mark.parametrize("T", [0.5, 5.0])
def test_soft(orc, T):
    from paper_1903_07149_amd.soft import SoftScalp
    from test_gpu_soft import assert_grads, compare_forward
    W, H, k, iters = 46400, 3, 60, 2
    lab, con = (a[None] for a in _image(W, H, 6))
    say("far soft", T)
    e = SoftScalp(W, H, k, 1, temperature=T, iterations=iters)
    ct, q, saved = e.forward(dev(lab), dev(con))
    th_o, q_o, _ = orc.soft_forward(lab, con, k, iterations=iters, T=T, d32=True)
    assert compare_forward(host(ct), host(q), th_o, q_o, W, H) == iters
    rng = np.random.default_rng(2)
    gq = rng.normal(0, 1, (1, 9, H, W)).astype(np.float32)
    gt = rng.normal(0, 1, (1, e.K, 5)).astype(np.float32)
    glab, gcon = e.backward(dev(lab), dev(con), ct, q, saved, dev(gq), dev(gt))
    assert_grads(orc, lab, con, k, gq, gt, iters, T, host(glab), host(gcon))
