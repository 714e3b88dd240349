"""Calls on D3Q19 lattices with solids whose steps run partly in replayed
graphs: every pair takes the march, and the populations equal those of one
step per pass bit for bit."""
import numpy as np
import pytest

import lbm_inputs as I
from conftest import print_case

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2602_06686_amd.ptrt")


@pytest.mark.parametrize("calls", [(23,), (47,), (21, 22)])
def test_calls_beyond_the_graphs(calls):
    print_case("march with solids after graph replays", calls)
    nz, ny, nx = 47, 45, 48
    mask = (np.random.default_rng(1).random((nz, ny, nx)) < 0.05).astype(np.uint8)
    rho, u = I.random_fields(np.random.default_rng(2), (nz, ny, nx), umax=0.04)
    got = []
    for spp in (1, 2):
        with P.Lattice(P.PTRT_D3Q19, nx, ny, nz, 0.64, 0.2, force=[3e-6, -1e-6, 2e-6], storage="f64",
                       solid_mask=mask, steps_per_pass=spp) as G:
            G.init_equilibrium(rho, u)
            for n in calls:
                G.step(n)
                assert G.last_pass()[0] == (1 if spp == 1 else 2 - n % 2)
            got.append(G.populations())
    fluid = np.broadcast_to(mask == 0, got[0].shape)
    assert np.array_equal(got[0][fluid], got[1][fluid])


# FP64 with solids on lattices that fill few of a wave's lanes: rows of 32
# lanes, two a wave; one strip and several, the last one short, rows and
# chunks that end ragged, fewer rows than a workgroup's, one plane
@pytest.mark.parametrize("kind", ["walls", "block", "corner", "random"])
@pytest.mark.parametrize("shape", [(60, 61, 30), (130, 29, 31), (1, 3500, 30), (41, 100, 64), (70, 15, 90),
                                   (1500, 2, 60), (40, 43, 65), (33, 57, 79)])
def test_narrow_strips(shape, kind):
    print_case("march with solids, rows of 32 lanes", shape, kind)
    nz, ny, nx = shape
    mask = np.zeros(shape, dtype=np.uint8)
    if kind == "walls":
        mask[:, 0] = 1
        mask[:, -1, ::3] = 1
    if kind == "block":
        mask[nz // 3:nz // 2 + 1, ny // 3:ny // 2 + 1, nx // 4:nx // 2] = 1
    if kind == "corner":
        mask[-1:, -2:, -2:] = mask[:1, :2, :1] = mask[nz // 2, ny // 2, nx // 2] = 1
    if kind == "random":
        mask[:] = np.random.default_rng(nz).random(shape) < 0.12
    rho, u = I.random_fields(np.random.default_rng(nx), shape, umax=0.04)
    got, passes = [], []
    for spp in (1, 2):
        with P.Lattice(P.PTRT_D3Q19, nx, ny, nz, 0.64, 0.2, force=[3e-6, -1e-6, 2e-6], storage="f64",
                       solid_mask=mask, steps_per_pass=spp) as G:
            G.init_equilibrium(rho, u)
            G.step(9)
            G.step(10)
            passes.append(G.last_pass()[0])
            got.append(G.populations())
    fluid = np.broadcast_to(mask == 0, got[0].shape)
    assert np.array_equal(got[0][fluid], got[1][fluid])
    assert passes[0] == 1
