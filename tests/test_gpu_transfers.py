"""Transfers between host arrays and the state: pinned chunks read and
written by the kernels, moved by host threads.  Sizes below one chunk, with
odd last chunks and of many chunks; parts left out; FP32 crossing of the
populations against what FP64 gives; several threads and streams at once."""
import ctypes
import threading

import numpy as np
import pytest

import lbm_inputs as I
from conftest import print_case

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2602_06686_amd.ptrt")
torch = pytest.importorskip("torch")

Q = {0: 9, 1: 19, 2: 27}
# nodes of one row only, one piece, a few pieces, several chunks, the ring
# more than once over
SIZES = [(0, 1, 1, 1), (0, 7, 3, 1), (0, 517, 131, 1), (1, 33, 29, 31), (2, 64, 48, 40), (1, 127, 113, 64)]


def _mask(nz, ny, nx):
    return (np.random.default_rng(5).random((nz, ny, nx)) < 0.1).astype(np.uint8)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16sr"])
@pytest.mark.parametrize("lat,nx,ny,nz", SIZES)
@pytest.mark.parametrize("solids", [False, True])
def test_populations_round_trip(lat, nx, ny, nz, storage, solids):
    print_case("set, get populations", lat, (nz, ny, nx), storage, solids)
    e, w = P.ptrt_velocity_set(lat)
    rng = np.random.default_rng(nx)
    mask = _mask(nz, ny, nx) if solids else None
    f = w[:, None, None, None] * (1 + 0.05 * rng.uniform(-1, 1, (Q[lat], nz, ny, nx)))
    with P.Lattice(lat, nx, ny, nz, 0.8, 0.25, storage=storage, solid_mask=mask) as G:
        G.set_populations(f)
        got = G.populations()
        rho, u = G.moments()
    fluid = np.ones((nz, ny, nx), bool) if mask is None else mask == 0
    h = f - w[:, None, None, None]
    if storage == "f64":
        want = h + w[:, None, None, None]
    else:
        h32 = torch.from_numpy(h.astype(np.float32))
        kept = h32 if storage == "f32" else h32.to(torch.float16 if storage == "f16" else torch.bfloat16)
        want = kept.to(torch.float64).numpy() + w[:, None, None, None]
    assert np.array_equal(got[:, fluid], want[:, fluid])
    assert not got[:, ~fluid].any() and not rho[~fluid].any() and not u[:, ~fluid].any()
    # the moments of the same populations (sums of Q terms in FP64)
    r = want.sum(0)
    j = np.einsum("ia,izyx->azyx", e.astype(float), want)
    assert np.abs(rho - r)[fluid].max(initial=0) < 1e-13
    assert np.abs(u - j / r)[:, fluid].max(initial=0) < 1e-13


@pytest.mark.parametrize("lat,nx,ny,nz", [(0, 517, 131, 1), (1, 127, 113, 64)])
def test_parts_left_out(lat, nx, ny, nz):
    print_case("init and moments with parts left out", lat, (nz, ny, nx))
    rho, u = I.random_fields(np.random.default_rng(3), (nz, ny, nx), umax=0.04)
    if lat == 0:
        u[2] = 0
    with P.Lattice(lat, nx, ny, nz, 0.8, 0.25, storage="f64") as G:
        for r, v in ((rho, u), (rho, None), (None, u), (None, None)):
            G.init_equilibrium(r, v)
            got_r, got_u = G.moments()
            assert np.abs(got_r - (1.0 if r is None else r)).max() < 1e-13
            assert np.abs(got_u - (0.0 if v is None else v)).max() < 1e-13
            one = np.full((nz, ny, nx), np.nan)
            three = np.full((3, nz, ny, nx), np.nan)
            dp = ctypes.POINTER(ctypes.c_double)
            assert P._lib.ptrt_moments(G.h.ptr, one.ctypes.data_as(dp), None) == 0
            assert P._lib.ptrt_moments(G.h.ptr, None, three.ctypes.data_as(dp)) == 0
            assert P._lib.ptrt_moments(G.h.ptr, None, None) == 0
            assert np.array_equal(one, got_r) and np.array_equal(three, got_u)


def test_threads_and_streams():
    """Handles of several threads, each on its own stream, transfer at once."""
    print_case("transfers of six threads")
    errors = []

    def work(k):
        try:
            stream = torch.cuda.Stream()
            rng = np.random.default_rng(k)
            shape = (20 + k, 40 + 3 * k, 64 + 7 * k)
            _, w = P.ptrt_velocity_set(1)
            f = w[:, None, None, None] * (1 + 0.05 * rng.uniform(-1, 1, (19,) + shape))
            want = (f - w[:, None, None, None]) + w[:, None, None, None]
            with P.Lattice(1, shape[2], shape[1], shape[0], 0.8, 0.25, storage="f64", stream=stream) as G:
                for _ in range(5):
                    G.set_populations(f)
                    if not np.array_equal(G.populations(), want):
                        errors.append(k)
        except Exception as e:  # noqa: BLE001 (reported below)
            errors.append((k, repr(e)))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
