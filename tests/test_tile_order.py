"""The D2Q9 tile passes keep one copy of a tile's populations and have one
barrier a step, so between two barriers no node may write a slot that another
node reads or writes.  The schedule of test_tile_schedule.py run in place, the
nodes of a step in a random order, with the slots of each step recorded."""
import numpy as np
import pytest

from test_tile_schedule import EX, EY, OPP, collide, plain_step


def tile_pass_in_place(f, solid, x0, y0, cols, core_rows, T, W, rng):
    """{(y, x): nine values} of the core after T steps."""
    ny, nx = solid.shape
    halo, rows = T - 1, core_rows + 2 * (T - 1)
    pad = W + 8
    plane = W * rows + pad
    lds = np.zeros(9 * plane + pad, dtype=np.int64)
    core = {}

    def node(n):
        return (y0 - halo + n // W) % ny, (x0 - halo + n % W) % nx

    def back(n, i):
        y, x = node(n)
        return bool(solid[(y - EY[i]) % ny, (x - EX[i]) % nx])

    for n in rng.permutation(rows * W):
        y, x = node(n)
        h = [f[OPP[i], y, x] if i and back(n, i) else f[i, (y - EY[i]) % ny, (x - EX[i]) % nx] for i in range(9)]
        for i, v in enumerate(collide(h)):
            lds[i * plane + pad + n] = v
    for s in range(2, T + 1):
        readers, writers = {}, {}
        for n in rng.permutation(np.arange((s - 1) * W, (rows - s + 1) * W)):
            y, x = node(n)
            own = [OPP[i] * plane + pad + n for i in range(9)]
            slot = own if s % 2 else [own[i] if i and back(n, i) else i * plane + pad + n - (EY[i] * W + EX[i])
                                      for i in range(9)]
            for a in slot:
                readers.setdefault(a, set()).add(n)
            h = collide([lds[a] for a in slot])
            if solid[y, x]:
                continue
            col, row = n % W, n // W
            if s == T:
                if halo <= col < halo + cols:
                    core[(y0 + row - halo, x)] = h
                continue
            for i in range(9):
                a = slot[OPP[i]] if s % 2 == 0 else i * plane + pad + n
                writers.setdefault(a, set()).add(n)
                lds[a] = h[i]
        # columns that hold values of the region in this step
        valid = {n for n in range((s - 1) * W, (rows - s + 1) * W) if s - 1 <= n % W < cols + 2 * halo - s + 1}
        for a, w in writers.items():
            users = (w | {n for n in readers.get(a, ()) if not solid[node(n)]}) & valid
            assert not users or users == w, "a slot written by one node is used by another in the same step"
    return core


@pytest.mark.parametrize("T", [2, 3, 4, 5, 8])
@pytest.mark.parametrize("ny,nx,cols,core_rows", [(13, 17, 6, 3), (4, 5, 5, 4), (9, 40, 11, 2), (1, 6, 6, 1)])
@pytest.mark.parametrize("density", [0.0, 0.1, 0.4])
def test_any_order_between_barriers(T, ny, nx, cols, core_rows, density):
    rng = np.random.default_rng([T, nx, int(10 * density)])
    solid = rng.random((ny, nx)) < density
    f = rng.integers(-2**40, 2**40, (9, ny, nx))
    want = f
    with np.errstate(over="ignore"):
        for _ in range(T):
            want = plain_step(want, solid)
        W = cols + 2 * (T - 1) + 3
        for y0 in range(0, ny, core_rows):
            for x0 in range(0, nx, cols):
                c, r = min(cols, nx - x0), min(core_rows, ny - y0)
                got = tile_pass_in_place(f, solid, x0, y0, c, r, T, W, rng)
                for y in range(y0, y0 + r):
                    for x in range(x0, x0 + c):
                        if not solid[y, x]:
                            assert got[(y, x)] == list(want[:, y, x])
