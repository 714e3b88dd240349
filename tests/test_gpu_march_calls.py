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
