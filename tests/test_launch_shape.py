"""Launch shapes of the hard assignment, from the library's own header compiled
for the host: work items cover their cells, and a single image's launch stays
below the 2^32 lanes of one, for every workgroup size."""
import os
import subprocess

import numpy as np
import pytest

from paper_1903_07149_amd import _lib as L
from paper_1903_07149_amd import build

SOURCE = r"""
#include <cstdio>
#include "scalp_internal.h"
using namespace scalp;
int main() {
    long long W, H, nx, ny;
    int wg;
    while (scanf("%lld %lld %lld %lld %d", &W, &H, &nx, &ny, &wg) == 5) {
        const int px = item_pixels(W, H, nx * ny, wg);
        const int bpx = batch_item_pixels(W * H, W, H, nx * ny, wg);
        printf("%d %d %d %d\n", px, assign_slices((int)W, (int)H, (int)nx, (int)ny, px,
                                                  fill_slices(nx * ny)),
               bpx, assign_slices((int)W, (int)H, (int)nx, (int)ny, bpx, 1));
    }
}
"""


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    d = tmp_path_factory.mktemp("shape")
    src, exe = str(d / "shape.cpp"), str(d / "shape")
    with open(src, "w") as f:
        f.write(SOURCE)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include",
                    f"-I{build.CSRC}", src, "-o", exe], check=True)

    def ask(rows):
        text = "".join("%d %d %d %d %d\n" % r for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]

    return ask


def _grid(W, H, k):
    g = L.make_grid(W, H, k)
    return g.nx, g.ny


@pytest.mark.parametrize("wg", [256, 512, 1024])
def test_large_cells_stay_below_a_launch(shapes, wg):
    """Cells above 48 x 48 pixels (shorter items) on images up to the largest
    accepted: fewer than 2^32 lanes, as without shorter items."""
    sizes = [(23171, 23171), (32768, 32768), (32768, 32760), (46340, 46340), (30000, 18000),
             (2 ** 29, 3), (20000, 50000), (16384, 16384)]
    rows = []
    for W, H in sizes:
        for px in (2305, 2500, 3600, 10 ** 4, 10 ** 6, W * H):
            nx, ny = _grid(W, H, max(1, W * H // px))
            if W * H > 2304 * nx * ny:
                rows.append((W, H, nx, ny, wg))
    assert len(rows) > 30
    for (W, H, nx, ny, _), (px, spl, *_) in zip(rows, shapes(rows)):
        assert nx * ny * spl * wg < 1 << 32, (W, H, nx, ny, px, spl)


@pytest.mark.parametrize("wg", [256, 512, 1024])
def test_items_cover_their_cells(shapes, wg):
    rng = np.random.default_rng(wg)
    rows = []
    for _ in range(400):
        W, H = (int(np.exp(v)) for v in rng.uniform(0, np.log(9000), 2))
        rows.append((W, H, *_grid(W, H, int(rng.integers(1, W * H + 1))), wg))
        rows.append((W, H, *_grid(W, H, max(1, int(W * H / rng.uniform(1, 20000)))), wg))
    for (W, H, nx, ny, _), (px, spl, *_) in zip(rows, shapes(rows)):
        assert 64 <= px <= wg and px % 64 == 0
        chunks = -(-(-(-W // nx) * -(-H // ny)) // 64)      # of the largest cell
        assert 1 <= spl <= chunks
        # chunks split evenly over the slices: none has more than px pixels, nor than the lanes
        assert -(-chunks // spl) * 64 <= px, (W, H, nx, ny, px, spl)


@pytest.mark.parametrize("wg", [256, 512, 1024])
def test_items_of_small_batches_grow_with_the_workgroup(shapes, wg):
    """At least a quarter of a workgroup's lanes have a pixel where the cells have
    that many, and no item has more pixels than lanes."""
    rng = np.random.default_rng(wg)
    rows = []
    for _ in range(300):
        W, H = (int(v) for v in rng.integers(16, 900, 2))
        rows.append((W, H, *_grid(W, H, max(1, int(W * H / rng.uniform(1, 20000)))), wg))
    for (W, H, nx, ny, _), (_, _, px, spl) in zip(rows, shapes(rows)):
        assert wg // 4 <= px <= wg, (W, H, nx, ny, px)
        chunks = -(-(-(-W // nx) * -(-H // ny)) // 64)
        assert -(-chunks // spl) * 64 <= px
