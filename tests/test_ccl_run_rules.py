"""CPU replay of the GPU CCL's run rules (64 x 64 tiles: local unions between
the runs of adjacent rows, the left-border and first-row merges) against
scipy's labelling, on small images cut into small tiles, so that every rule
meets tile corners often. Only the forest entries the kernels define are
used: reading any other raises."""
import numpy as np
import pytest
from scipy import ndimage


def _label_by_rules(fg, conn, side):
    H, W = fg.shape
    F = {}

    def find(a):
        while F[a] != a:
            a = F[a]
        return a

    def union(a, b):
        a, b = find(a), find(b)
        F[max(a, b)] = min(a, b)

    def start(y, x, x0):
        while x > x0 and fg[y, x - 1]:
            x -= 1
        return y * W + x

    tiles = [(y0, min(y0 + side, H), x0, min(x0 + side, W))
             for y0 in range(0, H, side) for x0 in range(0, W, side)]
    for y0, y1, x0, x1 in tiles:  # local phase, on the tile's own forest
        P = {start(y, x, x0): start(y, x, x0) for y in range(y0, y1) for x in range(x0, x1) if fg[y, x]}

        def pfind(a):
            while P[a] != a:
                a = P[a]
            return a

        def on(y, x):
            return x0 <= x < x1 and y >= y0 and bool(fg[y, x])
        for y in range(y0 + 1, y1):
            for x in range(x0, x1):
                if not fg[y, x]:
                    continue
                aL, aC, aR, first = on(y - 1, x - 1), on(y - 1, x), on(y - 1, x + 1), not on(y, x - 1)
                take = []
                if conn == 4:
                    if aC and not (aL and not first):
                        take = [x]
                else:
                    if first and (aL or aC):
                        take.append(x - 1 if aL else x)
                    if aR and not aC:
                        take.append(x + 1)
                for k in take:
                    a, b = pfind(start(y, x, x0)), pfind(start(y - 1, k, x0))
                    P[max(a, b)] = min(a, b)
        for y in range(y0, y1):
            for x in range(x0, x1):
                if fg[y, x] and (start(y, x, x0) == y * W + x or y in (y0, y1 - 1) or x == x0 + side - 1):
                    F[y * W + x] = pfind(start(y, x, x0))

    def at(y, x):
        return 0 <= y < H and 0 <= x < W and bool(fg[y, x])
    for y0, y1, x0, x1 in tiles:  # merges
        if x0 > 0:
            for y in range(y0, y1):
                c, l = at(y, x0), at(y, x0 - 1)
                cu, lu = (at(y - 1, x0), at(y - 1, x0 - 1)) if y > y0 else (False, False)
                p = y * W + x0
                if c and l and not (cu and lu):
                    union(p, p - 1)
                if conn == 8 and c and lu and not l and not cu:
                    union(p, p - W - 1)
                if conn == 8 and l and cu and not c and not lu:
                    union(p - 1, p - W)
        if y0 > 0:
            for x in range(x0, x1):
                if not fg[y0, x]:
                    continue
                first = x == x0 or not fg[y0, x - 1]
                aL, aC, aR = at(y0 - 1, x - 1), at(y0 - 1, x), at(y0 - 1, x + 1)
                p = y0 * W + x
                if conn == 4:
                    if aC and not (not first and aL):
                        union(p, p - W)
                else:
                    if first and aL:
                        union(p, p - W - 1)
                    if first and aC and not aL:
                        union(p, p - W)
                    if aR and not aC:
                        union(p, p - W + 1)
    out = np.zeros((H, W), np.int64)
    for y0, y1, x0, x1 in tiles:
        for y in range(y0, y1):
            for x in range(x0, x1):
                if fg[y, x]:
                    out[y, x] = find(start(y, x, x0)) + 1
    return out


@pytest.mark.parametrize("conn", [4, 8])
@pytest.mark.parametrize("side", [2, 3, 8])
@pytest.mark.parametrize("p", [0.35, 0.5, 0.65, 0.8])
def test_run_rules_label_like_scipy(conn, side, p):
    rng = np.random.default_rng(side * 100 + conn + int(100 * p))
    for H, W in ((1, 1), (1, 17), (17, 1), (2 * side, 2 * side), (3 * side + 1, 4 * side + 1), (26, 31)):
        fg = rng.random((H, W)) < p
        lab, n = ndimage.label(fg, ndimage.generate_binary_structure(2, 1 if conn == 4 else 2))
        want = np.zeros((H, W), np.int64)
        for k in range(1, n + 1):
            want[lab == k] = np.flatnonzero(lab == k).min() + 1
        assert np.array_equal(_label_by_rules(fg, conn, side), want)
