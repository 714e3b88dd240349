"""The schedule of the D3Q19 march with solids (csrc/march3d.hpp), emulated
with exact integers: first steps of a workgroup's rows plane by plane into the
LDS slots of their direction classes (1, 2 and 3 planes for e_z = -1, 0, 1),
values that bounce back put into the slots of the solids, second steps that
read all slots alike.  Between two barriers the threads run in a random
order, so a slot that two of them use without a barrier between them shows.
A column's core equals two plain steps at every fluid node."""
import numpy as np
import pytest

E = [(0, 0, 0)]
for _v in [(1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (1, -1, 0), (1, 0, 1), (1, 0, -1), (0, 1, 1), (0, 1, -1)]:
    E += [_v, tuple(-c for c in _v)]
OPP = [E.index(tuple(-c for c in v)) for v in E]
CLS = [v[2] + 1 for v in E]
SLOTS = [1, 2, 3]


def collide(h):
    """Any map that mixes all nineteen values and tells them apart (wrapping int64)."""
    s = sum((i + 3) * h[i] for i in range(19))
    return [h[i] * (2 * i + 5) ^ (s + (i << 7)) for i in range(19)]


def plain_step(f, solid):
    """f[19][nz][ny][nx] post-collision -> the next post-collision state."""
    out = []
    for i, (ex, ey, ez) in enumerate(E):
        back = np.roll(solid, (ez, ey, ex), (0, 1, 2))
        out.append(np.where(back, f[OPP[i]], np.roll(f[i], (ez, ey, ex), (0, 1, 2))))
    return np.array(collide(out))


def march(f, solid, x0, y0, cols, BY, zs, ze, rng):
    """{(z, y, x): nineteen values} of the core, as one workgroup does it."""
    nz, ny, nx = solid.shape
    threads = [(w, l) for w in range(BY + 2) for l in range(cols + 2)]
    lds, out, values = {}, {}, {}

    def node(t, k):
        return k % nz, (y0 - 1 + t[0]) % ny, (x0 - 1 + t[1]) % nx

    def flags(t, k):
        z, y, x = node(t, k)
        return [bool(solid[z, y, x])] + [bool(solid[(z - E[i][2]) % nz, (y - E[i][1]) % ny, (x - E[i][0]) % nx])
                                         for i in range(1, 19)]

    def core(t):
        return 1 <= t[0] <= BY and 1 <= t[1] <= cols and x0 - 1 + t[1] < nx

    def slot(i, it, t, shift=(0, 0)):
        return i, it % SLOTS[CLS[i]], t[0] - shift[1], t[1] - shift[0]

    def first(t, k, it):
        z, y, x = node(t, k)
        fl, fp = flags(t, k), flags(t, k - 1)
        h = collide([f[OPP[i], z, y, x] if i and fl[i] else
                     f[i, (z - E[i][2]) % nz, (y - E[i][1]) % ny, (x - E[i][0]) % nx] for i in range(19)])
        if not fl[0]:
            for i in range(19):
                lds[slot(i, it, t)] = h[i]
        if it == 0 or not core(t):
            return
        for i in range(1, 19):
            if CLS[i] and fl[i] and not fl[0]:
                lds[slot(i, it + 1 - CLS[i], t, E[i])] = h[OPP[i]]
            if CLS[i] == 0 and fp[i] and not fp[0]:
                lds[slot(i, it, t, E[i])] = lds.get(slot(OPP[i], it - 1, t))

    def second(t, k, it):
        if not core(t):
            return
        z, y, x = node(t, k - 1)
        got = [lds.get(slot(i, it - CLS[i], t, E[i])) for i in range(19)]
        if not solid[z, y, x]:
            out[z, y, x] = collide(got)

    def phase(*work):
        """Each thread runs the work in its order, the threads interleaved at random."""
        left = {t: list(work) for t in threads}
        while left:
            t = list(left)[rng.integers(len(left))]
            left[t].pop(0)(t)
            if not left[t]:
                del left[t]

    phase(lambda t: first(t, zs - 1, 0), lambda t: first(t, zs, 1))
    phase(lambda t: first(t, zs + 1, 2))
    k, it = zs + 1, 2
    while True:
        phase(lambda t: second(t, k, it))
        if k == ze:
            return out
        phase(lambda t: first(t, k + 1, it + 1))
        k, it = k + 1, it + 1


@pytest.mark.parametrize("nz,ny,nx,cols,BY,zc", [(4, 5, 6, 3, 2, 2), (3, 4, 5, 5, 3, 3), (1, 6, 4, 4, 2, 1),
                                               (5, 2, 3, 3, 3, 4)])
@pytest.mark.parametrize("density", [0.0, 0.1, 0.4])
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_march_equals_two_plain_steps(nz, ny, nx, cols, BY, zc, density, seed):
    rng = np.random.default_rng([seed, nx, int(10 * density)])
    solid = rng.random((nz, ny, nx)) < density
    f = rng.integers(-2**40, 2**40, (19, nz, ny, nx))
    with np.errstate(over="ignore"):
        want = plain_step(plain_step(f, solid), solid)
        seen = set()
        for zs in range(0, nz, zc):
            for y0 in range(0, ny, BY):
                for x0 in range(0, nx, cols):
                    got = march(f, solid, x0, y0, cols, BY, zs, min(zs + zc, nz), rng)
                    for (z, y, x), h in got.items():
                        assert h == list(want[:, z, y, x]), (z, y, x)
                        seen.add((z, y, x))
    assert len(seen) == int((~solid).sum())
