"""The schedule of the D2Q9 tile passes, emulated with exact integers: one
copy of a tile's nine populations, every step writing where it read, regions
that shrink by one node a step, bounce-back through the node's own slot.  A
pass of T steps equals T plain steps at every fluid node of the core, and no
slot that a later step reads is used by two nodes in one step."""
import numpy as np
import pytest

EX = (0, 1, 0, -1, 0, 1, -1, -1, 1)
EY = (0, 0, 1, 0, -1, 1, 1, -1, -1)
OPP = (0, 3, 4, 1, 2, 7, 8, 5, 6)


def collide(h):
    """Any map that mixes all nine values and tells them apart (wrapping int64)."""
    s = sum((i + 3) * h[i] for i in range(9))
    return [h[i] * (2 * i + 5) ^ (s + (i << 7)) for i in range(9)]


def plain_step(f, solid):
    """f[9][ny][nx] post-collision -> the next post-collision state."""
    out = []
    for i in range(9):
        src = np.roll(f[i], (EY[i], EX[i]), (0, 1))
        back = np.roll(solid, (EY[i], EX[i]), (0, 1))
        out.append(np.where(back, f[OPP[i]], src))
    return np.array(collide(out))


def tile_pass(f, solid, x0, y0, cols, core_rows, T, W):
    """{(y, x): nine values} of the core after T steps, as one workgroup does it."""
    ny, nx = solid.shape
    halo, rows = T - 1, core_rows + 2 * (T - 1)
    pad = W + 8
    plane = W * rows + pad
    lds = np.zeros(9 * plane + pad, dtype=np.int64)
    core, flags = {}, {}

    def node(n):
        return (y0 - halo + n // W) % ny, (x0 - halo + n % W) % nx

    def back(n, i):
        y, x = node(n)
        return solid[(y - EY[i]) % ny, (x - EX[i]) % nx]

    for n in range(rows * W):
        y, x = node(n)
        flags[n] = [bool(back(n, i)) for i in range(9)]
        h = [f[OPP[i], y, x] if flags[n][i] and i else f[i, (y - EY[i]) % ny, (x - EX[i]) % nx]
             for i in range(9)]
        for i, v in enumerate(collide(h)):
            lds[i * plane + pad + n] = v
    for s in range(2, T + 1):
        even, used = s % 2 == 0, {}
        new = lds.copy()
        for n in range((s - 1) * W, (rows - s + 1) * W):
            y, x = node(n)
            own = [OPP[i] * plane + pad + n for i in range(9)]
            slot = own
            if even:
                slot = [own[i] if i and flags[n][i] else i * plane + pad + n - (EY[i] * W + EX[i])
                        for i in range(9)]
            h = collide([lds[a] for a in slot])
            if solid[y, x]:
                continue
            col, row = n % W, n // W
            if s == T:
                if halo <= col < halo + cols:
                    core[(y0 + row - halo, x)] = h
                continue
            valid = s - 1 <= col < cols + 2 * halo - s + 1
            for i in range(9):
                a = slot[OPP[i]] if even else i * plane + pad + n
                assert not valid or a not in used, "two nodes write one slot"
                if valid:
                    used[a] = n
                new[a] = h[i]
        lds = new
    return core


@pytest.mark.parametrize("T", [2, 3, 4, 5, 8])
@pytest.mark.parametrize("ny,nx,cols,core_rows", [(13, 17, 6, 3), (4, 5, 5, 4), (9, 40, 11, 2), (1, 6, 6, 1)])
@pytest.mark.parametrize("density", [0.0, 0.1, 0.4])
def test_tile_pass_equals_plain_steps(T, ny, nx, cols, core_rows, density):
    rng = np.random.default_rng(T * 100 + nx)
    solid = rng.random((ny, nx)) < density
    f = rng.integers(-2**40, 2**40, (9, ny, nx))
    want = f
    with np.errstate(over="ignore"):
        for _ in range(T):
            want = plain_step(want, solid)
        W = cols + 2 * (T - 1) + 3  # columns past the region hold no meaning
        for y0 in range(0, ny, core_rows):
            for x0 in range(0, nx, cols):
                c, r = min(cols, nx - x0), min(core_rows, ny - y0)
                got = tile_pass(f, solid, x0, y0, c, r, T, W)
                for y in range(y0, y0 + r):
                    for x in range(x0, x0 + c):
                        if not solid[y, x]:
                            assert got[(y, x)] == list(want[:, y, x])
