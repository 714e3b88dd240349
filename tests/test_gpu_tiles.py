"""D2Q9 passes of several steps on tiles in LDS (calls of eight steps and
more) and the D3Q19 march: the populations equal those of one step per pass bit for bit, for
every storage type, with solids, open x, Scheme I and in a batch.  The sizes
put the lattice edge, the periodic wrap, solids and the open boundaries at
every place of a tile, down to lattices smaller than a tile's halo."""
import numpy as np
import pytest

import lbm_inputs as I
from conftest import print_case

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2602_06686_amd.ptrt")

STORAGE = ["f64", "f32", "f16", "bf16", "f16sr", "bf16sr"]


def _mask(kind, ny, nx):
    m = np.zeros((1, ny, nx), dtype=np.uint8)
    if kind == "none":
        return None
    if kind == "walls":
        m[0, 0] = m[0, -1] = 1
    if kind == "block":
        m[0, ny // 3:ny // 3 + max(1, ny // 6), nx // 2:nx // 2 + max(1, nx // 5)] = 1
    if kind == "seam":      # across the periodic corner, and single nodes next to each other
        m[0, :2, :3] = m[0, -2:, -2:] = 1
        m[0, ny // 2, nx // 2] = m[0, ny // 2 + 1, nx // 2 + 1] = 1
    if kind == "random":
        m[0] = np.random.default_rng(ny).random((ny, nx)) < 0.15
    return m


def _populations(shape, storage, calls, spp, mask=None, open_x=None, forcing="scheme2", passes=None):
    ny, nx = shape
    rho, u = I.random_fields(np.random.default_rng(nx), (1, ny, nx), umax=0.04)
    if open_x is not None:
        u[0] += open_x[0]
    with P.Lattice(P.PTRT_D2Q9, nx, ny, 1, 0.64, 0.2, force=[3e-6, -1e-6, 0.0], solid_mask=mask,
                   storage=storage, open_x=open_x, forcing=forcing, steps_per_pass=spp) as G:
        G.init_equilibrium(rho, u[:2])
        for n in calls:
            G.step(n)
            if passes is not None:
                passes.append(G.last_pass()[0])
        assert G.t == sum(calls)
        return G.populations()


def _same(shape, storage, calls, mask=None, **options):
    print_case("tile passes against single steps", shape, storage, calls, options)
    one = _populations(shape, storage, calls, 1, mask, **options)
    passes = []
    two = _populations(shape, storage, calls, 2, mask, passes=passes, **options)
    fluid = np.broadcast_to(True if mask is None else mask == 0, one.shape)
    assert np.array_equal(one[fluid], two[fluid])
    # an even call ends with a pass of two steps, an odd one with a single step
    assert all(p == 2 - n % 2 for n, p in zip(calls, passes) if n >= 8)


# smaller than a halo, around one tile, a few tiles with short last ones, and
# the large-lattice shapes (64 x 32 regions in 32 bits, 32 x 32 in 64)
SHAPES = [(1, 1), (1, 40), (33, 2), (7, 9), (16, 16), (31, 97), (64, 64), (130, 61), (381, 509)]


@pytest.mark.parametrize("storage", STORAGE)
@pytest.mark.parametrize("shape", SHAPES)
def test_periodic(shape, storage):
    _same(shape, storage, [8, 9, 21, 40])


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_periodic_large(storage):
    _same((1501, 1403), storage, [11, 24])


@pytest.mark.parametrize("storage", STORAGE)
@pytest.mark.parametrize("kind", ["walls", "block", "seam", "random"])
@pytest.mark.parametrize("shape", [(12, 9), (31, 97), (64, 64), (200, 333)])
def test_solids(shape, kind, storage):
    _same(shape, storage, [10, 17], _mask(kind, *shape))


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("kind", ["none", "walls", "block", "random"])
@pytest.mark.parametrize("shape", [(9, 2), (20, 5), (31, 97), (150, 264)])
def test_open_x(shape, kind, storage):
    _same(shape, storage, [10, 17], _mask(kind, *shape), open_x=(0.03, 1.01))


@pytest.mark.parametrize("storage", STORAGE)
@pytest.mark.parametrize("kind", ["none", "block"])
def test_scheme1(kind, storage):
    _same((45, 83), storage, [10, 17], _mask(kind, 45, 83), forcing="guo")


@pytest.mark.parametrize("storage", STORAGE)
@pytest.mark.parametrize("sizes", [[(5, 3), (1, 20), (40, 33), (97, 31), (64, 64)],
                                   [(300, 250), (33, 512), (511, 40)] * 12])
def test_batch(sizes, storage):
    print_case("batch tile passes against single steps", len(sizes), storage)
    kinds = ["none", "walls", "block", "random"]
    specs = [{"nx": nx, "ny": ny, "tau_plus": 0.6 + 0.05 * (k % 7), "Lambda": 0.2,
              "g": (1e-6 * k, -1e-6, 0.0), "mask": _mask(kinds[k % 4], ny, nx)}
             for k, (nx, ny) in enumerate(sizes)]
    got = []
    for spp in (1, 2):
        b = P.ptrt_batch_create(specs, storage)
        try:
            P.ptrt_batch_set_steps_per_pass(b, spp)
            for k, (nx, ny) in enumerate(sizes):
                rho, u = I.random_fields(np.random.default_rng(k), (1, ny, nx), umax=0.04)
                P.ptrt_batch_init_equilibrium(b, k, rho, u[:2])
            for n in (8, 23, 3, 12):
                P.ptrt_batch_step(b, n)
            got.append([P.ptrt_batch_get_populations(b, k) for k in range(len(sizes))])
        finally:
            P.ptrt_batch_destroy(b)
    for k, s in enumerate(specs):
        fluid = np.broadcast_to(True if s["mask"] is None else s["mask"] == 0, got[0][k].shape)
        assert np.array_equal(got[0][k][fluid], got[1][k][fluid]), f"instance {k}"


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("count", [1, 2, 9])
def test_batch_diagnostics_equal_single(count, storage):
    """Mass and energy of all lattices from one launch: bit for bit those of
    each lattice alone (same blocks, same order of sums)."""
    print_case("batch diagnostics against single lattices", count, storage)
    kinds = ["walls", "none", "random", "block"]
    sizes = [(70, 9), (1, 1), (64, 4), (65, 5), (3, 200), (200, 3), (130, 61), (300, 333), (16, 16)][:count]
    specs = [{"nx": nx, "ny": ny, "tau_plus": 0.7, "Lambda": 0.2, "g": (1e-5, -2e-6 * k, 0.0),
              "mask": _mask(kinds[k % 4], ny, nx)} for k, (nx, ny) in enumerate(sizes)]
    b = P.ptrt_batch_create(specs, storage)
    try:
        fields = [I.random_fields(np.random.default_rng(k), (1, ny, nx), umax=0.04)
                  for k, (nx, ny) in enumerate(sizes)]
        for k, (rho, u) in enumerate(fields):
            P.ptrt_batch_init_equilibrium(b, k, rho, u[:2])
        P.ptrt_batch_step(b, 5)
        mass, energy = P.ptrt_batch_diagnostics(b)
    finally:
        P.ptrt_batch_destroy(b)
    for k, s in enumerate(specs):
        with P.Lattice(P.PTRT_D2Q9, s["nx"], s["ny"], 1, 0.7, 0.2, force=s["g"], solid_mask=s["mask"],
                       storage=storage) as G:
            G.init_equilibrium(fields[k][0], fields[k][1][:2])
            G.step(5)
            assert G.diagnostics() == (mass[k], energy[k])


# D3Q19 march: one strip, two and four, with widths down to 24 columns; rows
# and chunks that end ragged; one plane; widths that are multiples of 64 below
# and above the other pass's range; four-row workgroups (FP32, large)
@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("shape", [(60, 61, 24), (47, 45, 48), (1, 1500, 62), (90, 85, 101), (41, 2, 1000),
                                   (92, 84, 100), (33, 70, 130), (30, 64, 64), (50, 100, 192),
                                   (182, 183, 186)])
def test_d3q19_march(shape, storage):
    print_case("D3Q19 march against single steps", shape, storage)
    nz, ny, nx = shape
    rho, u = I.random_fields(np.random.default_rng(nx), shape, umax=0.04)
    got = []
    for spp in (1, 2):
        with P.Lattice(P.PTRT_D3Q19, nx, ny, nz, 0.64, 0.2, force=[3e-6, -1e-6, 2e-6], storage=storage,
                       steps_per_pass=spp) as G:
            G.init_equilibrium(rho, u)
            G.step(5)
            G.step(2)
            assert G.last_pass()[0] == spp
            got.append(G.populations())
    assert np.array_equal(got[0], got[1])


# the same with solids, in calls of eight steps and more: walls on the y seam,
# a block, solids on the corner of the box, scattered ones (every kind of
# link, on every plane of a chunk and row of a workgroup)
@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("kind", ["walls", "block", "corner", "random"])
@pytest.mark.parametrize("shape", [(47, 45, 48), (3, 600, 62), (90, 85, 101), (64, 50, 64)])
def test_d3q19_march_solids(shape, kind, storage):
    print_case("D3Q19 march with solids against single steps", shape, kind, storage)
    nz, ny, nx = shape
    mask = np.zeros(shape, dtype=np.uint8)
    if kind == "walls":
        mask[:, 0] = mask[:, -1] = 1
    if kind == "block":
        mask[nz // 3:nz // 2 + 1, ny // 3:ny // 2, nx // 4:nx // 2] = 1
    if kind == "corner":
        mask[-1:, -2:, -2:] = mask[:1, :2, :1] = mask[nz // 2, ny // 2, nx // 2] = 1
    if kind == "random":
        mask[:] = np.random.default_rng(nz).random(shape) < 0.12
    rho, u = I.random_fields(np.random.default_rng(nx), shape, umax=0.04)
    got, passes = [], []
    for spp in (1, 2):
        with P.Lattice(P.PTRT_D3Q19, nx, ny, nz, 0.64, 0.2, force=[3e-6, -1e-6, 2e-6], storage=storage,
                       solid_mask=mask, steps_per_pass=spp) as G:
            G.init_equilibrium(rho, u)
            G.step(9)
            G.step(8)
            passes.append(G.last_pass()[0])
            got.append(G.populations())
    fluid = np.broadcast_to(mask == 0, got[0].shape)
    assert np.array_equal(got[0][fluid], got[1][fluid])
    # 64 x 64 x 50 falls into strips of 32 columns: one step per pass in FP32
    assert passes == [1, 1 if storage == "f32" and nx == 64 else 2]
