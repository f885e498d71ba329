"""Calls whose time must keep up with that of a like call: images that differ only
in a property that should cost little.  The limits leave about half as much again
for noise as a correct build needs; what they guard against was far outside."""
import numpy as np
import pytest

from gpu_util import needs_gpu, say, torch

pytestmark = [pytest.mark.gpu, needs_gpu]


def _image(W, H, seed=1):
    """Blocks of colour with noise, and a contour map that is nowhere quite 0."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    lo = torch.rand((H // 40 + 1, W // 40 + 1, 3), generator=g, device="cuda") * 60
    lab = lo.repeat_interleave(40, 0).repeat_interleave(40, 1)[:H, :W]
    lab = (lab + 4 * torch.randn((H, W, 3), generator=g, device="cuda")).contiguous()
    return lab, torch.rand((H, W), generator=g, device="cuda") ** 4


def _time(fn, target=30.0):
    """Least of five averages, in ms."""
    def once(n):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(n):
            fn()
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) / n
    once(2)
    n = max(2, int(target / once(2)))
    return min(once(n) for _ in range(5))


def _run(W, H, k, data=None, **params):
    from paper_1903_07149_amd.scalp import Scalp
    lab, con = data if data is not None else _image(W, H)
    s = Scalp(W, H, k, **params)
    out = s.new_state()
    return _time(lambda: s.run(lab, con, out=out))


@pytest.mark.parametrize("mode", [0, 1])
def test_far_images_keep_up_with_near_ones(mode):
    """60000x80 against 30000x160, the same pixels and cells."""
    say("far against near", mode)
    far = _run(60000, 80, 4800, iterations=5, assign_mode=mode)
    near = _run(30000, 160, 4800, iterations=5, assign_mode=mode)
    print(f"far {far:.3f} ms, near {near:.3f} ms")
    assert far < 1.5 * near


def test_every_candidate_walked_keeps_up():
    """exact_pruning = 0 walks nine times as many paths, in about 2.3 times the time."""
    lab, _ = _image(1920, 1080)
    data = lab, torch.zeros(lab.shape[:2], device="cuda")
    say("every candidate against the pruned walks")
    full = _run(1920, 1080, 2000, data, iterations=5, exact_pruning=0)
    pruned = _run(1920, 1080, 2000, data, iterations=5)
    print(f"all {full:.3f} ms, pruned {pruned:.3f} ms")
    assert full < 4.0 * pruned


def test_soft_backward_of_large_cells_keeps_up():
    """512x512 in 16 cells at T = 5: the backward takes about as long as the forward."""
    from paper_1903_07149_amd.soft import SoftScalp
    lab, con = (a[None].contiguous() for a in _image(512, 512))
    e = SoftScalp(512, 512, 16, 1, temperature=5.0, iterations=2)
    gq, gt = torch.ones((1, 9, 512, 512), device="cuda"), torch.ones((1, e.K, 5), device="cuda")
    gq[:, 4] = -1.0
    say("soft large cells, time")
    ct, q, saved = e.forward(lab, con)
    fwd = _time(lambda: e.forward(lab, con))
    bwd = _time(lambda: e.backward(lab, con, ct, q, saved, gq, gt))
    print(f"forward {fwd:.3f} ms, backward {bwd:.3f} ms")
    assert bwd < 4.0 * fwd


def test_noise_keeps_up():
    """An image of noise, which bounds tell little about, against one of regions."""
    lab, _ = _image(1920, 1080)
    zero = torch.zeros(lab.shape[:2], device="cuda")
    say("noise against regions")
    easy = _run(1920, 1080, 2000, (lab, zero), iterations=5)
    g = torch.Generator(device="cuda").manual_seed(3)
    hard = _run(1920, 1080, 2000, (30 * torch.randn(lab.shape, generator=g, device="cuda"),
                                   torch.rand(zero.shape, generator=g, device="cuda")), iterations=5)
    print(f"noise {hard:.3f} ms, regions {easy:.3f} ms")
    assert hard < 6.5 * easy


def test_many_pairs_of_large_cells_keep_up():
    """One colour at m = 0 lists every candidate: cells of 3000 pixels against 1000, whose
    paths have 1.7 times the samples."""
    say("large cells, every candidate listed")
    data = torch.full((1080, 1920, 3), 50.0, device="cuda"), torch.zeros((1080, 1920), device="cuda")
    small, large = (_run(1920, 1080, k, data, iterations=5, m=0.0) for k in (2000, 700))
    print(f"700 cells {large:.3f} ms, 2000 {small:.3f} ms")
    assert large < 3.5 * small


def test_many_pairs_of_short_items_keep_up():
    """One colour at m = 0: cells of 500 pixels, in items of 192, against 1000."""
    say("short items, every candidate listed")
    data = torch.full((1080, 1920, 3), 50.0, device="cuda"), torch.zeros((1080, 1920), device="cuda")
    whole, short = (_run(1920, 1080, k, data, iterations=5, m=0.0) for k in (2000, 4000))
    print(f"4000 cells {short:.3f} ms, 2000 {whole:.3f} ms")
    assert short < 1.5 * whole


def test_metrics_of_few_labels_keep_up():
    """One label everywhere against many, 3840x2160."""
    from paper_1903_07149_amd.metrics import Metrics
    H, W = 2160, 3840
    y, x = torch.arange(H, device="cuda")[:, None], torch.arange(W, device="cuda")[None]
    many = ((y // 29) * (W // 29 + 1) + x // 29).int().contiguous()
    region = ((y // 97) * (W // 93 + 1) + x // 93).int().contiguous()
    one = torch.zeros_like(many)
    m, n = Metrics(W, H, int(many.max()) + 1, int(region.max()) + 1), Metrics(W, H, 4, 4)
    say("metrics of one label, time")
    a, b = _time(lambda: m.run(many, region)), _time(lambda: n.run(one, one))
    print(f"many labels {a:.4f} ms, one {b:.4f} ms")
    assert b < 1.3 * a
