"""The host code of libptrt without a GPU: a stand-in for the HIP runtime
(tests/host/recorder.cpp) records which kernels a call launches, with which
grids, and makes allocations fail.  Each case is a script of its own process
(tests/host/library.py)."""
import os
import shutil
import subprocess
import sys

import pytest

from conftest import ROOT

HOST = os.path.join(ROOT, "tests", "host")
LIB = os.path.join(ROOT, "paper_2602_06686_amd", "libptrt.so")


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if not (shutil.which("g++") and os.path.exists(LIB)):
        pytest.skip("needs g++ and the built library")
    out = tmp_path_factory.mktemp("host")
    recorder = str(out / "recorder.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-pthread",
                    os.path.join(HOST, "recorder.cpp"), "-o", recorder], check=True)

    def script(text, timeout=120):
        path = str(out / "script.py")
        with open(path, "w") as fh:
            fh.write(text)
        res = subprocess.run([sys.executable, os.path.join(HOST, "library.py"), recorder, LIB, path],
                             capture_output=True, text=True, timeout=timeout)
        assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
        return res.stdout

    return script


@pytest.mark.parametrize("boundary", ["solids", "open"])
def test_storage_after_a_failed_allocation(run, boundary):
    """Whichever allocation of the first init fails, the handle then takes
    another storage type and runs the passes of that type: no tile pass of the
    failed attempt's plan, which would not know of solids and open x."""
    run(f"""
mask = bytearray(2048 * 2048)
mask[0] = 1
for k in range(1, 20):
    h = create(D2Q9, 2048, 2048, 1, F64, bytes(mask) if {boundary == "solids"} else None)
    if {boundary == "open"}:
        ok(L.ptrt_set_open_x(h, C.c_double(0.01), C.c_double(1.0)), h)
    R.rec_fail_device(k)
    rc = L.ptrt_init_equilibrium(h, None, None)
    R.rec_fail_device(0)
    if rc == 0:
        break
    assert rc in (ENOMEM, EDEVICE)
    assert L.ptrt_set_storage(h, F16_SR) == 0
    init(h)
    assert set(kernels(h, 10)) == {{"k_step"}}, (k, launches())
    ok(L.ptrt_destroy(h), h)
assert k > 5
# the same handle without a failure: tile passes, with the flags of their tiles
ok(L.ptrt_destroy(h), h)
h = create(D2Q9, 2048, 2048, 1, F64, bytes(mask))
init(h)
assert set(kernels(h, 10)) == {{"k_tile_2d"}}
assert all(R.rec_pointer(i, 4) for i in range(R.rec_launches()))
""")


@pytest.mark.parametrize("steps", [8, 9, 20, 21, 23, 27, 47])
def test_march_covers_the_remainder_after_graph_replays(run, steps):
    """A call of eight steps or more on a D3Q19 lattice with solids takes the
    march for all its pairs, those after the replayed graphs of 20 steps too."""
    run(f"""
h = create(D3Q19, 48, 45, 47, F64, bytes([1]) + bytes(48 * 45 * 47 - 1))
init(h)
assert kernels(h, {steps}) == ["k_march3d"] * {steps // 2} + ["k_step"] * {steps % 2}
assert last_pass(h) == {2 - steps % 2}
assert kernels(h, 7) == ["k_step"] * 7 and last_pass(h) == 1
""")


def test_march_between_divergence_checks(run):
    """The check splits a call; its pieces are still parts of a long call."""
    run("""
h = create(D3Q19, 48, 45, 47, F64, bytes([1]) + bytes(48 * 45 * 47 - 1))
init(h)
ok(L.ptrt_set_divergence_check(h, 4), h)
assert kernels(h, 12) == ["k_march3d", "k_march3d", "k_check_finite"] * 3
assert kernels(h, 4) == ["k_step"] * 4 + ["k_check_finite"]
""")


@pytest.mark.parametrize("storage", ["F32", "F64", "F16"])
def test_no_launch_beyond_the_thread_limit(run, storage):
    """Rows so long and few that a tile per core would need 2^32 threads or
    more in a launch: the passes of before run."""
    run(f"""
for nx, ny in ((300000000, 7), (400000000, 5), (470000000, 4)):
    h = C.c_void_p()
    ok(L.ptrt_create(D2Q9, nx, ny, 1, C.c_double(0.7), C.c_double(0.25), None, None, C.byref(h)), None)
    if L.ptrt_set_storage(h, {storage}) == 0:
        init(h)
        step(h, 10)
    ok(L.ptrt_destroy(h), h)
""")


def test_batch_diagnostics_beyond_one_launch(run):
    """Blocks of a batch whose one launch would have 2^32 threads or more
    (lattices of one column: 64 times the threads of their nodes) are taken
    in several, each block once."""
    run("""
rc, b = batch([(1, 262140)] * 257, F16)
assert rc == 0, L.ptrt_batch_last_error(None)
mass, energy = (C.c_double * 257)(), (C.c_double * 257)()
R.rec_reset()
assert L.ptrt_batch_diagnostics(b, mass, energy) == 0, L.ptrt_batch_last_error(b)
gather = [l for l in launches() if l[0] == "k_batch_gather"]
assert sum(l[2][0] for l in gather) == 257 * 65535
assert [l[2][0] for l in launches() if l[0] == "k_batch_finalize"] == [257]
L.ptrt_batch_destroy(b)
""")


def test_handle_freed_in_a_forked_child(run):
    """The host threads of the transfers do not exist in a forked child:
    freeing the inherited handle there returns, and so does a read-back."""
    run("""
import os, time
h = create(D3Q19, 128, 128, 96)
init(h)
rho = (C.c_double * (128 * 128 * 96))()
for _ in range(4):
    ok(L.ptrt_moments(h, rho, None), h)
pid = os.fork()
if pid == 0:
    ok(L.ptrt_moments(h, rho, None), h)
    ok(L.ptrt_moments(h, rho, None), h)
    L.ptrt_destroy(h)
    os._exit(7)
for _ in range(100):
    done, status = os.waitpid(pid, os.WNOHANG)
    if done:
        break
    time.sleep(0.1)
else:
    os.kill(pid, 9)
    os.waitpid(pid, 0)
assert done and os.WEXITSTATUS(status) == 7
ok(L.ptrt_moments(h, rho, None), h)
L.ptrt_destroy(h)
""")


def test_threads_and_pinned_memory_for_what_is_moved(run):
    """A small handle that is read a few times starts no thread and pins no
    more than it moves at once, at most 4 MB; handles that move much, as many
    threads as their pieces keep busy and at most 64 MB a ring."""
    run("""
import os
threads = lambda: len(os.listdir("/proc/self/task")) - 1
most = min(15, len(os.sched_getaffinity(0)) - 1)

def arrays(n):
    return (C.c_double * n)(), (C.c_double * (3 * n))()

rho, u = arrays(32 ** 3)
h = create(D3Q19, 32, 32, 32)
ok(L.ptrt_init_equilibrium(h, rho, u), h)       # 1 MB, four pieces
for _ in range(5):
    ok(L.ptrt_moments(h, rho, u), h)
assert threads() == 0 and R.rec_host_most() == 1 << 20
for _ in range(30):
    ok(L.ptrt_moments(h, rho, u), h)
assert threads() == min(3, most), threads()
L.ptrt_destroy(h)
assert threads() == 0 and R.rec_host_now() == 0
rho, u = arrays(64 ** 3)
h = create(D3Q19, 64, 64, 64)
ok(L.ptrt_init_equilibrium(h, rho, u), h)       # 8 MB
ok(L.ptrt_moments(h, rho, u), h)
assert R.rec_host_most() == 4 << 20 and threads() == min(7, most)
L.ptrt_destroy(h)
rho, u = arrays(128 ** 3)
h = create(D3Q19, 128, 128, 128)
for _ in range(40):                             # 2.7 GB
    ok(L.ptrt_moments(h, rho, u), h) if _ else ok(L.ptrt_init_equilibrium(h, rho, u), h)
assert threads() == most
assert 64 << 20 <= R.rec_host_now() <= 128 << 20 and R.rec_host_most() <= 192 << 20
L.ptrt_destroy(h)
assert threads() == 0 and R.rec_host_now() == 0
""")


def test_few_rows_keep_the_earlier_passes(run):
    """Long lattices of few rows, and batches of them, whose tiles would be
    mostly halo take the passes of one and two steps; short ones, those of
    more rows and 16-bit batches take tile passes."""
    run("""
def kind(nx, ny, storage, open_x=False, forcing=0):
    h = create(D2Q9, nx, ny, 1, storage)
    if open_x:
        ok(L.ptrt_set_open_x(h, C.c_double(0.01), C.c_double(1.0)), h)
    init(h)
    ok(L.ptrt_set_forcing(h, forcing), h)
    k = set(kernels(h, 10))
    ok(L.ptrt_destroy(h), h)
    assert len(k) == 1, k
    return k.pop()

for storage, few, earlier in ((F32, 6, "k_step2_2d"), (F64, 6, "k_step2_2d"), (F16, 12, "k_step")):
    for nx in (100000, 1000000):
        for ny in (1, 2, 3):
            assert kind(nx, ny, storage) == earlier, (nx, ny, storage)
    assert kind(1000000, few - 2, storage) == earlier
    for nx, ny in ((100, 1), (10000, 1), (10000, 3), (1000000, 16), (7, 200000), (509, 381)):
        assert kind(nx, ny, storage) == "k_tile_2d", (nx, ny, storage)
assert kind(70000, 4, F32) == kind(1000000, 8, F32) == "k_tile_2d"
# the earlier pass of open x and of Scheme I is one of a single step
for storage in (F32, F64):
    assert kind(100000, 3, storage, open_x=True) == kind(100000, 3, storage, forcing=2) == "k_tile_2d"
    assert kind(1000000, 4, storage, open_x=True) == "k_step2_2d"
assert kind(1000000, 10, F16, open_x=True) == kind(1000000, 10, F16, forcing=2) == "k_step"

def batch_kind(sizes, storage):
    rc, b = batch(sizes, storage)
    assert rc == 0
    R.rec_reset()
    assert L.ptrt_batch_step(b, 10) == 0
    k = {l[0] for l in launches()}
    L.ptrt_batch_destroy(b)
    assert len(k) == 1, k
    return k.pop()

thin = [(200, 4), (210, 5)] * 500
assert batch_kind(thin, F64) == batch_kind(thin, F32) == "k_batch_step2"
assert batch_kind(thin, F16) == "k_batch_tile"
for storage in (F64, F32, F16):
    assert batch_kind(thin[:20], storage) == "k_batch_tile"
    assert batch_kind(thin[:50] + [(300, 200)] * 20, storage) == "k_batch_tile"
""")


def test_layout_of_whole_planes_only_for_passes_that_need_it(run):
    """Odd ny: rows share tiles (the buffer holds a multiple of the tile's
    rows) in every kernel of one step per pass, and have one row a tile where
    the march or k_step2's source offsets run."""
    run("""
SCHEME2, SCHEME2_G, GUO = 0, 1, 2
PTRT, RLB, TRT, EXACT = 0, 1, 2, 3

def rows(lattice, nx, ny, nz, storage, mask=None, forcing=SCHEME2, model=PTRT):
    h = create(lattice, nx, ny, nz, storage, mask)
    ok(L.ptrt_set_model(h, model), h)
    ok(L.ptrt_set_forcing(h, forcing), h)
    R.rec_reset()
    init(h)
    elem = {F64: 8, F32: 4}.get(storage, 2)
    line = 128 // elem
    pitch = (nx + line - 1) // line * line
    n, q = R.rec_device_size(0), {D3Q19: 19, D3Q27: 27}[lattice]
    ok(L.ptrt_destroy(h), h)
    assert n % (q * pitch * elem) == 0
    return n // (q * pitch * elem)

def solid(nx, ny, nz):
    return bytes([1]) + bytes(nx * ny * nz - 1)

S = (60, 61, 61)
whole = 61 * 61
for storage in (F32, F64):
    assert rows(D3Q19, *S, storage) == whole
    assert rows(D3Q19, *S, storage, solid(*S)) == whole          # march with solids
    for option in ({"forcing": GUO}, {"forcing": SCHEME2_G}, {"model": RLB}, {"model": TRT}, {"model": EXACT}):
        assert rows(D3Q19, *S, storage, **option) > whole, option
    assert rows(D3Q27, *S, storage) > whole
for storage in (F16, BF16_SR):
    assert rows(D3Q19, *S, storage) > whole and rows(D3Q27, *S, storage) > whole
T = (128, 99, 99)                       # k_step2: source offsets in FP32 only
assert rows(D3Q19, *T, F32) == rows(D3Q19, *T, F32, model=TRT) == 99 * 99
assert rows(D3Q19, *T, F64) > 99 * 99
U = (64, 99, 99)                        # FP32 with solids, strips of 32 columns: one step per pass
assert rows(D3Q19, *U, F32, solid(*U)) > 99 * 99
# a forcing chosen after the first init: the passes that the layout allows
h = create(D3Q19, *S, F64)
ok(L.ptrt_set_forcing(h, GUO), h)
init(h)
ok(L.ptrt_set_forcing(h, SCHEME2), h)
assert set(kernels(h, 8)) == {"k_step"}
h = create(D3Q19, *S, F64)
init(h)
assert set(kernels(h, 8)) == {"k_march3d"}
ok(L.ptrt_set_forcing(h, GUO), h)
assert set(kernels(h, 8)) == {"k_step"}
ok(L.ptrt_set_forcing(h, SCHEME2), h)
assert set(kernels(h, 8)) == {"k_march3d"}
""")


def test_march_with_solids_rows_of_32_lanes(run):
    """FP64 with solids: rows of 32 lanes where strips of 64 have at most 40
    columns and need more rounds, never in FP32 or without solids."""
    run("""
def shape(nx, ny, nz, storage, solids=True):
    h = create(D3Q19, nx, ny, nz, storage, bytes([1]) + bytes(nx * ny * nz - 1) if solids else None)
    init(h)
    (l,) = set(step(h, 8))
    ok(L.ptrt_destroy(h), h)
    strips = {"64": 62, "32": 30}
    if l[0] != "k_march3d":
        return l[0]
    args = l[1].split("<")[1].split(">")[0].split(", ")   # storage, rows, lanes
    lanes, rows = int(args[2]), int(args[1])
    assert l[3] == (lanes * (rows + 2), 1, 1)
    n = -(-nx // (lanes - 2))
    assert l[2][0] == -(-nx // -(-nx // n)) and l[2][1] == -(-ny // rows)
    return lanes

for nx in (24, 30, 64, 65, 80):
    assert shape(nx, 100, 102, F64) == 32, nx
    assert shape(nx, 100, 102, F64, False) == 64
    assert shape(nx, 100, 102, F32) == "k_step"
for nx in (48, 62, 96, 126, 128):  # 42 columns and more
    assert shape(nx, 100, 102, F64) == 64, nx
assert shape(50, 100, 102, F32) == 64
""")


@pytest.mark.parametrize("storage", ["F32", "F64"])
def test_kernel_of_a_pair_of_steps_in_3d(run, storage):
    """k_step2 from 800 000 nodes on where nx is a multiple of 64 (one launch
    per round of resident workgroups), the march below; source offsets in
    FP32, the general pulls for a handle first initialised with Scheme I."""
    run(f"""
def pair(nx, ny, nz, forcing=0):
    h = create(D3Q19, nx, ny, nz, {storage})
    ok(L.ptrt_set_forcing(h, forcing), h)
    init(h)
    ok(L.ptrt_set_forcing(h, 0), h)
    out = step(h, 2)
    ok(L.ptrt_destroy(h), h)
    assert len({{l[0] for l in out}}) == 1
    return out

f32 = {storage} == F32
for nx, ny, nz in ((128, 65, 99), (64, 101, 128), (64, 3130, 4), (128, 6255, 1), (128, 3133, 2), (128, 1370, 5),
                   (192, 67, 66)):
    out = pair(nx, ny, nz)
    assert out[0][0] == "k_step2" and out[0][1].endswith("true" if f32 else "false"), out[0]
    assert sum(l[2][1] for l in out) == -(-ny // 4)
    ragged = pair(nx, ny, nz, 2)
    assert ragged[0][0] == "k_step2"
    if ny % 2:
        assert ragged[0][1].endswith("false")
assert len(pair(64, 3130, 4)) == 2                    # rows of workgroups in two rounds
for nx, ny, nz in ((64, 64, 64), (128, 64, 64), (128, 60, 100), (192, 64, 64)):
    assert pair(nx, ny, nz)[0][0] == "k_march3d"
assert pair(64, 64, 64)[0][0] == pair(100, 84, 92)[0][0] == "k_march3d"
""")


@pytest.mark.parametrize("mask", [False, True])
def test_out_of_host_memory_is_reported(run, mask):
    """Whichever host allocation of a first init or of a batch's creation
    fails: a status and a message, no exception past the C interface, nothing
    left behind, and the next attempt succeeds."""
    run(f"""
m = bytes([1]) + bytes(300 * 200 - 1) if {mask} else None
h = create(D2Q9, 300, 200, 1, F32, m)
for k in range(1, 200):
    R.rec_fail_new(k)
    rc = L.ptrt_init_equilibrium(h, None, None)
    R.rec_fail_new(0)
    if rc == 0:
        break
    assert rc == ENOMEM and L.ptrt_last_error(h), (k, rc)
    assert R.rec_blocks() == 0
assert rc == 0 and 2 < k < 150, k
assert set(kernels(h, 10)) == {{"k_tile_2d"}}
ok(L.ptrt_destroy(h), h)
assert R.rec_blocks() == 0

sizes = [(40 + k, 30 + k) for k in range(5)]
for k in range(1, 400):
    R.rec_fail_new(k)
    rc, b = batch(sizes, F32)
    R.rec_fail_new(0)
    if rc == 0:
        break
    assert rc == ENOMEM and not b and L.ptrt_batch_last_error(None), (k, rc)
    assert R.rec_blocks() == 0, k
assert rc == 0 and k > 10, k
L.ptrt_batch_destroy(b)
""")


def test_little_pinned_memory(run):
    """Where less pinned memory can be had than a transfer asks for, it runs in
    smaller chunks; none at all is an error that leaves the handle usable."""
    run("""
n = 32 * 32 * 32
rho, u = (C.c_double * n)(*([1.0] * n)), (C.c_double * (3 * n))()
for limit in (1 << 20, 256 << 10, 64 << 10):
    h = create(D3Q19, 32, 32, 32)
    R.rec_limit_host(limit)
    R.rec_reset()
    ok(L.ptrt_init_equilibrium(h, rho, u), h)
    fills = [l for l in launches() if l[0] == "k_init_eq"]
    assert len(fills) >= (1 << 20) // limit and sum(l[2][0] * 256 for l in fills) >= n
    R.rec_reset()
    ok(L.ptrt_moments(h, rho, u), h)
    assert sum(l[2][0] * 256 for l in launches()) >= n
    R.rec_limit_host((1 << 64) - 1)
    ok(L.ptrt_destroy(h), h)
h = create(D3Q19, 32, 32, 32)
R.rec_limit_host(1024)
assert L.ptrt_init_equilibrium(h, rho, u) in (ENOMEM, EDEVICE)
R.rec_limit_host((1 << 64) - 1)
ok(L.ptrt_init_equilibrium(h, rho, u), h)
ok(L.ptrt_destroy(h), h)
assert R.rec_blocks() == 0
""")


def test_where_solids_take_the_march(run):
    """Sizes on both sides of the rule for D3Q19 with solids: columns, nodes,
    strips, few rows."""
    run("""
def kind(nx, ny, nz, storage, solids=True):
    h = create(D3Q19, nx, ny, nz, storage, bytes([1]) + bytes(nx * ny * nz - 1) if solids else None)
    init(h)
    k = set(kernels(h, 8))
    ok(L.ptrt_destroy(h), h)
    assert len(k) == 1, k
    return k.pop() == "k_march3d"

for size in ((24, 100, 102), (50, 50, 40), (64, 50, 64), (96, 12, 220), (126, 14, 200), (48, 45, 47)):
    assert kind(*size, F64), size
for size in ((23, 100, 102), (56, 40, 40), (64, 40, 40), (96, 8, 220), (64, 16, 180), (96, 13, 220)):
    assert not kind(*size, F64), size
for size in ((48, 45, 47), (50, 14, 200), (100, 84, 92), (180, 150, 150), (145, 150, 150)):
    assert kind(*size, F32), size
for size in ((47, 60, 61), (60, 40, 40), (100, 40, 40), (96, 16, 180), (200, 100, 102), (128, 96, 96), (180, 190, 180)):
    assert not kind(*size, F32), size
for storage in (F16, BF16):
    assert not kind(100, 84, 92, storage)
# without solids: few rows and planes
for size in ((125, 2, 600), (200, 5, 300), (125, 6, 300), (200, 10, 200), (62, 1500, 1), (300, 1000, 2)):
    assert kind(*size, F64, False) and kind(*size, F32, False), size
for size in ((125, 1, 1000), (125, 7, 300), (200, 8, 220)):
    assert not kind(*size, F64, False) and not kind(*size, F32, False), size
for size in ((300, 1000, 1), (125, 4, 600)):
    assert not kind(*size, F64, False) and kind(*size, F32, False), size
assert not kind(100, 1000, 2, F64) and kind(100, 1000, 2, F32)
""")
