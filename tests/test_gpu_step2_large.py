"""The D3Q19 two-step pass k_step2 on the lattices that it has to itself (nx a
multiple of 64, 800 000 nodes and more; below, the march runs): ragged ny,
one and two planes, chunks of planes, more columns than one round of resident
workgroups, the source offsets of FP32 and the general pulls.  The same
populations, bit for bit, as one step per pass.  Which kernel runs is
asserted without a GPU in test_host_paths.py."""
import numpy as np
import pytest

import lbm_inputs as I
from conftest import print_case

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2602_06686_amd.ptrt")

SHAPES = [(99, 65, 128), (128, 101, 64), (4, 3130, 64), (1, 6255, 128), (2, 3133, 128), (5, 1370, 128), (66, 67, 192)]


def _populations(shape, storage, steps, spp, first_forcing="scheme2", model="ptrt"):
    nz, ny, nx = shape
    rho, u = I.random_fields(np.random.default_rng(nx + nz), shape, umax=0.05)
    with P.Lattice(P.PTRT_D3Q19, nx, ny, nz, 0.61, 0.25, storage=storage, force=[3e-6, -1e-6, 2e-6],
                   steps_per_pass=spp, forcing=first_forcing, model=model) as G:
        G.init_equilibrium(rho, u)
        P.ptrt_set_forcing(G.h, "scheme2")
        G.step(steps)
        assert G.last_pass()[0] == (1 if spp == 1 or steps % 2 else 2)
        return G.populations()


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("steps", [2, 7])
def test_bitwise(shape, storage, steps):
    print_case("k_step2 against single steps", shape, storage, steps)
    assert np.array_equal(_populations(shape, storage, steps, 1), _populations(shape, storage, steps, 2))


@pytest.mark.parametrize("shape", SHAPES)
def test_general_pulls_in_fp32(shape):
    """A handle first initialised with Scheme I has rows that share layout
    tiles across planes: no source offsets."""
    print_case("k_step2 with general pulls against single steps", shape)
    one, two = (_populations(shape, "f32", 6, spp, "guo") for spp in (1, 2))
    assert np.array_equal(one, two)


@pytest.mark.parametrize("model", ["trt", "trt-rlb"])
def test_comparison_models(model):
    print_case("k_step2, comparison models against single steps", model)
    one, two = (_populations((99, 65, 128), "f32", 6, spp, model=model) for spp in (1, 2))
    assert np.array_equal(one, two)
