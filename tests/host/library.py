"""libptrt with recorder.cpp in place of the HIP runtime, as a script of its
own uses it:  python library.py RECORDER LIBPTRT SCRIPT  runs SCRIPT with the
names defined here."""
import ctypes as C
import re
import sys

R = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
L = C.CDLL(sys.argv[2])
R.rec_name.restype = C.c_char_p
R.rec_limit_host.argtypes = [C.c_size_t]
for name in ("rec_host_now", "rec_host_most", "rec_device_size"):
    getattr(R, name).restype = C.c_size_t
L.ptrt_last_error.restype = L.ptrt_batch_last_error.restype = C.c_char_p

D2Q9, D3Q19, D3Q27 = 0, 1, 2
F64, F32, F16, BF16, F16_SR, BF16_SR = range(6)
ENOMEM, EDEVICE = -3, -4


class Desc(C.Structure):
    _fields_ = [("nx", C.c_int), ("ny", C.c_int), ("tau_plus", C.c_double), ("Lambda", C.c_double),
                ("force", C.c_double * 3), ("solid_mask", C.c_char_p)]


def create(lattice, nx, ny, nz=1, storage=F32, mask=None):
    """A handle (not initialised); mask: bytes of the nodes, or None."""
    h = C.c_void_p()
    rc = L.ptrt_create(lattice, nx, ny, nz, C.c_double(0.7), C.c_double(0.25), None, mask, C.byref(h))
    assert rc == 0, L.ptrt_last_error(None)
    assert L.ptrt_set_storage(h, storage) == 0
    return h


def batch(sizes, storage=F32):
    b = C.c_void_p()
    d = (Desc * len(sizes))(*[Desc(nx, ny, 0.7, 0.25, (C.c_double * 3)(), None) for nx, ny in sizes])
    return L.ptrt_batch_create(len(sizes), d, storage, C.byref(b)), b


def ok(rc, h):
    assert rc == 0, (rc, L.ptrt_last_error(h))


def init(h):
    ok(L.ptrt_init_equilibrium(h, None, None), h)


def step(h, n):
    """The launches of one call: [(kernel, template arguments, grid, block)]."""
    R.rec_reset()
    ok(L.ptrt_step(h, n), h)
    return launches()


def launches():
    out = []
    for k in range(R.rec_launches()):
        name = R.rec_name(k).decode()
        m = re.match(r"(?:void )?(?:ptrt|\(anonymous namespace\))::(\w+)(?:<(.*)>)?\(", name)
        # types that the demangler does not know
        m_raw = re.match(r"_ZN(?:4ptrt|12_GLOBAL__N_1)(\d+)(.*)", name)
        shape = (C.c_uint * 6)()
        R.rec_shape(k, shape)
        if m:
            kernel, args = m.group(1), m.group(2) or ""
        elif m_raw:
            n = int(m_raw.group(1))
            kernel, args = m_raw.group(2)[:n], m_raw.group(2)[n:]
        else:
            kernel, args = name, ""
        out.append((kernel, args, tuple(shape[:3]), tuple(shape[3:])))
    return out


def kernels(h, n):
    return [l[0] for l in step(h, n)]


def last_pass(h):
    s, b = C.c_int(), C.c_double()
    ok(L.ptrt_last_pass(h, C.byref(s), C.byref(b)), h)
    return s.value


exec(compile(open(sys.argv[3]).read(), sys.argv[3], "exec"))
