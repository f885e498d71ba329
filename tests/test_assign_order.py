"""Host replay of the integer and FP32 rules of the 3x3 assignment's walk
order: invariant division, the pixel enumeration built on it, the enumeration
of candidates by key, and the bound that cuts a walk short."""
import numpy as np
import pytest

M32 = 1 << 32


def fast_div(d, limit):
    return (M32 + d - 1) // d if d > 1 and limit < M32 // d else 0


def fdiv(v, d, m):
    return (v * m) >> 32 if m else v // d


@pytest.mark.parametrize("n,length", [(60, 1920), (34, 1080), (1, 97), (64, 64), (133, 3840),
                                      (7, 61), (9, 65535), (1000, 65535)])
def test_cell_boundaries_by_multiplication(n, length):
    """cell_lo(i) = ceil(i len / n) as one high multiplication, for every cell."""
    m = fast_div(n, n * (length + 1))
    for i in range(n + 1):
        v = i * length + n - 1
        assert v < M32
        assert fdiv(v, n, m) == -(-i * length // n)


LAST_STRIP = [0, 0, 0x80000000, 0x55555556, 0x40000000, 0x33333334, 0x2aaaaaab, 0x24924925]


@pytest.mark.parametrize("cw,ch", [(32, 32), (33, 31), (7, 40), (1, 900), (23, 15), (160, 161),
                                   (1920, 8), (8, 1), (15, 2)])
def test_pixel_enumeration_by_multiplication(cw, ch):
    """Every pixel of the cell exactly once, in 8-wide serpentine strips."""
    per = 8 * ch
    m = fast_div(per, (cw + 1) * ch)
    if m == 0:
        pytest.skip("divided, not multiplied")
    full = (cw >> 3) * per
    seen = np.zeros((ch, cw), int)
    for t in range(cw * ch):
        if t < full:
            s = fdiv(t, per, m)
            r = t - s * per
            row, x = r >> 3, 8 * s + (r & 7)
        else:
            wr, r, s = cw & 7, t - full, cw >> 3
            row = (r * LAST_STRIP[wr]) >> 32 if wr > 1 else r
            x = 8 * s + r - row * wr
        y = ch - 1 - row if s & 1 else row
        assert s == x // 8
        seen[y, x] += 1
    assert (seen == 1).all()


def next_key(keys, cur):
    c1 = (cur + 1) % M32
    low = min((k - c1) % M32 for k in keys)
    return low + c1 if low + c1 < M32 else M32 - 1


@pytest.mark.parametrize("span", [12, 1 << 20, M32])
def test_candidates_come_in_ascending_order_once(span):
    rng = np.random.default_rng(span % 1000)
    for _ in range(2000):
        keys = [(int(v) & ~15) | j for j, v in enumerate(rng.integers(0, span, 9))]
        for j in np.flatnonzero(rng.random(9) < 0.3):
            keys[j] = M32 - 1                    # a slot outside the grid
        got, cur = [], M32 - 1
        for _ in range(10):
            cur = next_key(keys, cur)
            if cur == M32 - 1:
                break
            got.append(cur)
        assert got == sorted(k for k in keys if k != M32 - 1)


@pytest.mark.parametrize("scale", [1.0, 1e-9, 1e-19, 1e12])
def test_a_cut_walk_could_not_have_won(scale):
    """Where the partial sums' value exceeds best (1 + 2^-16), so does the FP32
    D of the whole path (the reciprocal may be off by an ulp either way)."""
    f = np.float32
    rng = np.random.default_rng(5)
    cuts = 0
    for _ in range(3000):
        n = int(rng.integers(1, 60))
        d = (rng.gamma(0.7, 60.0, n + 1) * scale).astype(f)
        w = np.where(rng.random(n + 1) < 0.8, 0.0, rng.random(n + 1)).astype(f)
        lam, gamma, dsp = f(rng.choice([0.0, 0.3, 0.5, 1.0])), f(rng.choice([0.0, 64.0, 3e5])), \
            f(rng.random() * 50 * scale)
        oml = f(1) - lam
        sc = sw = f(0)
        part = []
        for i in range(n + 1):
            sc, sw = f(sc + d[i]) if i else d[0], f(sw + w[i]) if i else w[0]
            part.append((sc, sw))
        A = f(f(lam * d[0]) + f(oml * f(sc / f(n + 1))))
        D = f(f(A * f(f(1) + f(gamma * f(sw / f(n + 1))))) + dsp)
        # every value of best that D does not exceed
        best = np.nextafter(D, f(np.inf)) if rng.random() < 0.5 else f(D * f(1 + rng.random()))
        best = max(best, D)
        thr = max(f(best * f(1 + 2.0 ** -16)), f(2.0 ** -70))
        for ulp in (-1, 0, 1):
            r = f(1) / f(n + 1)
            r = f(np.nextafter(r, f(ulp * np.inf))) if ulp else r
            a0, fr, g = f(lam * d[0]), f(oml * r), f(gamma * r)
            for (s, t) in part:
                assert not f(f(f(a0 + f(fr * s)) * f(f(1) + f(g * t))) + dsp) > thr
        # and it does cut losers
        low = f(D * f(0.5))
        cuts += any(f(f(f(a0 + f(fr * s)) * f(f(1) + f(g * t))) + dsp) >
                    max(f(low * f(1 + 2.0 ** -16)), f(2.0 ** -70)) for (s, t) in part)
    assert cuts > 1000 or scale < 1e-10
