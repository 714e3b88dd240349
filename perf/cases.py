"""Work that a user of this library has it do, as cases to be timed.

A program that simulates a flow keeps a handle, advances it by some steps,
reads the state back and goes on: one pass is a number of steps followed by
the read-back that such a program makes (density and velocity, the mass and
energy monitor, the drag, a checkpoint).  The handle and the initial state
are what it has in hand before the call.

The steps between two read-backs are what sampling a flow takes: a few
hundred on an ordinary lattice, ten where a small flow is watched closely.
"""
import math

import numpy as np
import torch

from paper_2602_06686_amd import ptrt as P

LATTICE = {"d2q9": P.PTRT_D2Q9, "d3q19": P.PTRT_D3Q19, "d3q27": P.PTRT_D3Q27}
Q = {"d2q9": 9, "d3q19": 19, "d3q27": 27}
# operations of one node update of the method (moments, equilibrium, ghost
# removal, relaxation)
UPDATE_FLOPS = {"d2q9": 130, "d3q19": 290, "d3q27": 480}
STORED = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}


def single(name, lattice, nx, ny, nz, storage, steps, **options):
    case = {"name": name, "kind": "single", "lattice": lattice, "nx": nx, "ny": ny, "nz": nz,
            "storage": storage, "steps": steps, "solids": "none", "forced": False, "open": False,
            "forcing": "scheme2", "read": "moments"}
    case.update(options)
    return case


def listed():
    return [
        # the decaying vortex on its usual small lattice, in FP64: many steps between two samples
        single("vortex2d 64x64 f64", "d2q9", 64, 64, 1, "f64", 1000),
        # a small driven channel watched closely: few steps a call, where latency counts
        single("channel2d 97x31 f32", "d2q9", 97, 31, 1, "f32", 10, solids="walls", forced=True),
        # an ordinary two-dimensional lattice of odd sizes with a body force
        single("driven2d 509x381 f32", "d2q9", 509, 381, 1, "f32", 200, forced=True,
               read="moments+diagnostics"),
        # the double shear layer at the resolution that its stability study uses
        single("shear2d 2048x2048 f32", "d2q9", 2048, 2048, 1, "f32", 500),
        # the square cylinder between velocity inlet and pressure outlet, drag every 200 steps
        single("cylinder2d 1050x1050 f64", "d2q9", 1050, 1050, 1, "f64", 200, solids="block",
               open=True, read="moments+drag"),
        # a parameter sweep of uneven channels and obstacles, monitored as a whole
        {"name": "sweep 512 f32", "kind": "batch", "count": 512, "lo": 32, "hi": 512,
         "storage": "f32", "steps": 200, "read": "diagnostics", "mix": 0},
        # a small sweep in FP64 whose fields are all read
        {"name": "sweep 24 f64", "kind": "batch", "count": 24, "lo": 32, "hi": 200,
         "storage": "f64", "steps": 100, "read": "moments", "mix": 1},
        # the three-dimensional vortex at the headline size
        single("vortex3d 256^3 f32", "d3q19", 256, 256, 256, "f32", 400,
               read="moments+diagnostics"),
        # a three-dimensional box of sizes that no tile divides, with a body force
        single("driven3d 100x84x92 f32", "d3q19", 100, 84, 92, "f32", 200, forced=True),
        # the cubic correction of the forcing scheme
        single("cubic3d 128^3 f32", "d3q19", 128, 128, 128, "f32", 200, forced=True,
               forcing="scheme2+g"),
        # a duct with a block in it, in FP64
        single("duct3d 128x96x96 f64", "d3q19", 128, 96, 96, "f64", 200, solids="walls+block",
               forced=True, read="moments+drag"),
        # resumed from a checkpoint and written to the next one, in FP16 storage
        single("restart3d 96^3 f16", "d3q27", 96, 96, 96, "f16", 200, read="restart"),
    ]


def spread(rng, lo, hi):
    """A whole number in [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    family = rng.choice(["plane", "plane", "channel", "cylinder", "sweep", "box", "box", "duct",
                         "restart"])
    storage = rng.choice(["f32", "f32", "f64", "f16", "bf16"])
    if family == "sweep":
        count, lo = spread(rng, 8, 400), spread(rng, 16, 64)
        hi = spread(rng, 2 * lo, 400)
        case = {"kind": "batch", "count": count, "lo": lo, "hi": hi, "storage": rng.choice(["f32", "f64"]),
                "steps": spread(rng, 10, 200), "read": "moments" if count <= 30 else "diagnostics",
                "mix": rng.randrange(1, 1000)}
    elif family in ("plane", "channel", "cylinder"):
        nx, ny = spread(rng, 24, 2000), spread(rng, 24, 2000)
        steps = spread(rng, 10, max(10, min(1000, int(1e9 / (nx * ny)))))
        if family == "plane":
            case = single("", "d2q9", nx, ny, 1, storage, steps, forced=rng.random() < 0.5,
                          forcing=rng.choice(["scheme2", "scheme2", "scheme2", "guo", "scheme2+g"]),
                          read=rng.choice(["moments", "moments+diagnostics", "restart"]))
        elif family == "channel":
            case = single("", "d2q9", nx, ny, 1, storage, steps, forced=True,
                          solids=rng.choice(["walls", "block", "walls+block"]),
                          read=rng.choice(["moments", "moments+drag"]))
        else:
            case = single("", "d2q9", max(nx, 64), max(ny, 64), 1, storage, steps, solids="block",
                          open=True, read="moments+drag")
    else:
        nx, ny, nz = (spread(rng, 24, 200) for _ in range(3))
        if rng.random() < 0.4:  # a multiple of the wave width, as many users choose
            nx = max(64, nx // 64 * 64)
        lattice = "d3q27" if rng.random() < 0.3 else "d3q19"
        steps = spread(rng, 10, max(10, min(400, int(4e8 / (nx * ny * nz)))))
        if family == "box":
            case = single("", lattice, nx, ny, nz, storage, steps, forced=rng.random() < 0.5,
                          forcing=rng.choice(["scheme2", "scheme2", "scheme2", "guo", "scheme2+g"]),
                          read=rng.choice(["moments", "moments+diagnostics"]))
        elif family == "duct":
            case = single("", lattice, nx, ny, nz, storage, steps, forced=True,
                          solids=rng.choice(["walls", "block", "walls+block"]), read="moments+drag")
        else:
            case = single("", lattice, min(nx, 128), min(ny, 128), min(nz, 128), storage, steps,
                          read="restart")
    case.pop("name", None)
    return case


# ------------------------------------------------------------------ inputs

def solid_mask(case, ny, nx, nz=1):
    """Walls at both ends of y, a block in the middle, or both; None without solids."""
    kind = case["solids"]
    if kind == "none":
        return None
    m = np.zeros((nz, ny, nx), dtype=np.uint8)
    if "walls" in kind:
        m[:, 0, :] = m[:, -1, :] = 1
    if "block" in kind:
        side = max(2, min(nx, ny) // (50 if case["open"] else 8))
        x0, y0 = (nx - side) // 2, (ny - side) // 2
        z0, zs = ((nz - side) // 2, side) if nz > side else (0, nz)
        m[z0:z0 + zs, y0:y0 + side, x0:x0 + side] = 1
    return m


def flow(rng, nx, ny, nz, u0):
    """A vortex field whose phases come from the seed, with a smaller one across it:
    rho [nz,ny,nx] and u [2 or 3,nz,ny,nx]."""
    def waves(n, k):
        a = 2 * np.pi * k * (np.arange(n) + rng.uniform(0, n)) / n
        return np.sin(a), np.cos(a)

    sx, cx = (v[None, None, :] for v in waves(nx, 1))
    sy, cy = (v[None, :, None] for v in waves(ny, 1))
    sz, cz = (v[:, None, None] for v in (waves(nz, 1) if nz > 1 else (np.zeros(1), np.ones(1))))
    tx, ty = waves(nx, 2)[0][None, None, :], waves(ny, 2)[0][None, :, None]
    tz = waves(nz, 2)[0][:, None, None] if nz > 1 else np.ones((1, 1, 1))
    rho = np.empty((nz, ny, nx))
    u = np.empty((3 if nz > 1 else 2, nz, ny, nx))
    np.multiply(u0 * u0 * (cx * cy), cz, out=rho)
    rho += 1.0
    np.multiply(u0 * (sx * cy), cz, out=u[0])
    np.multiply(-u0 * (cx * sy), cz, out=u[1])
    u[0] += 0.2 * u0 * (ty * tz)
    u[1] += 0.2 * u0 * (tx * tz)
    if nz > 1:
        u[2] = 0.2 * u0 * (tx * ty)
    return rho, u


def single_inputs(case, seed):
    """tau+, Lambda, force, mask, (u_in, rho_out) or None, rho, u of a single lattice."""
    rng = np.random.default_rng([int(seed), 1])
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    tau = float(rng.uniform(0.56, 0.62)) if case["solids"] == "none" else float(rng.uniform(0.7, 0.9))
    lam = 0.25 if case["solids"] == "none" else 3.0 / 16.0
    force = None
    if case["forced"]:
        g = 10.0 ** rng.uniform(-6.5, -6.0)
        force = [float(g), float(0.2 * g) if case["solids"] == "none" else 0.0, 0.0]
    mask = solid_mask(case, ny, nx, nz)
    if case["open"]:
        u_in = float(rng.uniform(0.02, 0.04))
        rho = np.ones((nz, ny, nx))
        u = np.zeros((2, nz, ny, nx))
        u[0] = u_in
        return tau, lam, force, mask, (u_in, 1.0), rho, u
    rho, u = flow(rng, nx, ny, nz, 0.04)
    return tau, lam, force, mask, None, rho, u


def batch_inputs(case, seed):
    """Channels (walls at both ends of y) and boxes around a square, of uneven sizes: the
    sizes belong to the case, the relaxation times, forces and fields come from the seed."""
    sizes = np.random.default_rng([case["mix"], case["count"]])
    rng = np.random.default_rng([int(seed), 2])
    specs, fields = [], []
    for k in range(case["count"]):
        nx, ny = (int(sizes.integers(case["lo"], case["hi"] + 1)) for _ in range(2))
        m = np.zeros((1, ny, nx), dtype=np.uint8)
        if k % 2 == 0:
            m[0, 0] = m[0, -1] = 1
        else:
            side = max(1, min(nx, ny) // 8)
            m[0, (ny - side) // 2:(ny - side) // 2 + side, (nx - side) // 2:(nx - side) // 2 + side] = 1
        specs.append({"nx": nx, "ny": ny, "tau_plus": float(rng.uniform(0.6, 1.5)),
                      "Lambda": 3.0 / 16.0, "g": (float(10.0 ** rng.uniform(-7, -6)), 0.0, 0.0),
                      "mask": m})
        # a small sweep starts each lattice from a field of its own; a large one from rest
        fields.append(flow(rng, nx, ny, 1, 0.03) if case["read"] == "moments" else None)
    return specs, fields


def prepare(case, seed):
    if case["kind"] == "batch":
        specs, fields = batch_inputs(case, seed)
        b = P.ptrt_batch_create(specs, case["storage"])
        for k, f in enumerate(fields):
            if f is not None:
                P.ptrt_batch_init_equilibrium(b, k, f[0], f[1])
        return {"case": case, "batch": Owner(b)}
    tau, lam, force, mask, ends, rho, u = single_inputs(case, seed)
    lat = P.Lattice(LATTICE[case["lattice"]], case["nx"], case["ny"], case["nz"], tau, lam,
                    force=force, solid_mask=mask, storage=case["storage"], open_x=ends,
                    forcing=case["forcing"])
    lat.init_equilibrium(rho, u)
    state = {"case": case, "lattice": lat}
    if case["read"] == "restart":
        state["checkpoint"] = lat.populations()
    return state


class Owner:
    """Frees a batch with the state that holds it."""

    def __init__(self, handle):
        self.handle = handle

    def __del__(self):
        P.ptrt_batch_destroy(self.handle)


def run(state):
    case = state["case"]
    if case["kind"] == "batch":
        b = state["batch"].handle
        P.ptrt_batch_step(b, case["steps"])
        if case["read"] == "diagnostics":
            return P.ptrt_batch_diagnostics(b)
        return [P.ptrt_batch_moments(b, k) for k in range(case["count"])]
    lat = state["lattice"]
    if case["read"] == "restart":
        lat.set_populations(state["checkpoint"])
        lat.step(case["steps"])
        return lat.populations()
    lat.step(case["steps"])
    out = {}
    if "diagnostics" in case["read"]:
        out["mass"], out["energy"] = lat.diagnostics()
    if "drag" in case["read"]:
        out["drag"] = lat.momentum_exchange()
    out["rho"], out["u"] = lat.moments()
    return out


def work(case):
    stored = STORED[case["storage"]]
    if case["kind"] == "batch":
        specs, _ = batch_inputs({**case, "read": "diagnostics"}, 0)
        n, q, lattice = sum(s["nx"] * s["ny"] for s in specs), 9, "d2q9"
        back = 4 * 8 * n if case["read"] == "moments" else 16 * case["count"]
    else:
        n, lattice = case["nx"] * case["ny"] * case["nz"], case["lattice"]
        q = Q[lattice]
        back = 2 * q * 8 * n if case["read"] == "restart" else 4 * 8 * n
    # the state read once and written once, the fields that are handed over
    return {"bytes": 2.0 * q * stored * n + back, "flops": float(UPDATE_FLOPS[lattice]) * n * case["steps"]}


# ------------------------------------------------- the same in 64 bits, plainly

def velocities(lattice):
    """e [Q,3] and w [Q] in the order of the populations."""
    if lattice == "d2q9":
        e = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (-1, 0, 0), (0, -1, 0),
             (1, 1, 0), (-1, 1, 0), (-1, -1, 0), (1, -1, 0)]
        return np.array(e), np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)
    e = [(0, 0, 0)]
    for v in [(1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (1, -1, 0), (1, 0, 1), (1, 0, -1),
              (0, 1, 1), (0, 1, -1)]:
        e += [v, tuple(-c for c in v)]
    if lattice == "d3q19":
        return np.array(e), np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)
    for v in [(1, 1, 1), (1, 1, -1), (1, -1, 1), (-1, 1, 1)]:
        e += [v, tuple(-c for c in v)]
    return np.array(e), np.array([8 / 27] + [2 / 27] * 6 + [1 / 54] * 12 + [1 / 216] * 8)


class Plain:
    """Nodes of one or several lattices side by side, updated in FP64: collide every node,
    then take each population from the node it comes from."""

    def __init__(self, lattice, shapes, masks, taus, lams, forces, ends=None, cubic=False, guo=False):
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        e, w = velocities(lattice)
        self.e, self.w, self.Q, self.D = e, w, len(w), 2 if lattice == "d2q9" else 3
        self.opp = [int(np.where((e == -v).all(1))[0][0]) for v in e]
        self.ends, self.cubic, self.guo, self.dev = ends, cubic, guo, dev
        self.N = sum(int(np.prod(s)) for s in shapes)
        starts = np.cumsum([0] + [int(np.prod(s)) for s in shapes])

        def joined(make):
            return torch.cat([make(k, s, int(starts[k])).reshape(-1) for k, s in enumerate(shapes)])

        def number(k, s, start):
            return torch.arange(start, start + int(np.prod(s)), device=dev).reshape(s)

        def shifted(v):  # node number of x - v at x
            return joined(lambda k, s, start: torch.roll(number(k, s, start), (int(v[2]), int(v[1]), int(v[0])), (0, 1, 2)))

        self.solid = joined(lambda k, s, start: torch.zeros(s, dtype=torch.bool, device=dev) if masks[k] is None
                            else torch.from_numpy(masks[k] != 0).to(dev))
        here = torch.arange(self.N, device=dev)
        self.source = []
        for i in range(self.Q):
            src = shifted(e[i])
            self.source.append(torch.where(self.solid[src], self.opp[i] * self.N + here, i * self.N + src))
        shifts = {}

        def neighbour(v):
            key = tuple(int(c) for c in v)
            if key not in shifts:
                shifts[key] = shifted(key)
            return shifts[key]

        self.neighbour = neighbour

        def constant(values):
            return values[0] if len(shapes) == 1 else joined(
                lambda k, s, start: torch.full(s, values[k], dtype=torch.float64, device=dev))

        self.tau = constant(taus)
        self.ap = constant([1 - 1 / t for t in taus])
        self.am = constant([1 - 1 / (0.5 + m / (t - 0.5)) for t, m in zip(taus, lams)])
        self.g = [constant([float(f[a]) if f is not None else 0.0 for f in forces]) for a in range(3)]
        if ends:
            nx = shapes[0][2]
            self.first, self.last = here[::nx], here[nx - 1::nx]
        # projection onto the second-order Hermite modes, orthogonal under 1/w
        modes = []
        for a in range(self.D):
            for b in range(a, self.D):
                modes.append(w * (e[:, a] * e[:, b] - (1 / 3 if a == b else 0.0)))
        B = np.array(modes).T
        Bw = B.T / w[None, :]
        self.stress = torch.from_numpy(B @ np.linalg.solve(Bw @ B, Bw)).to(dev)

    def field(self, arrays):
        return torch.cat([torch.from_numpy(np.ascontiguousarray(a)).reshape(-1) for a in arrays]).to(self.dev)

    def dot(self, i, v):
        r = None
        for a in range(self.D):
            if self.e[i, a]:
                t = v[a] if self.e[i, a] == 1 else -v[a]
                r = t if r is None else r + t
        return r

    def equilibrium(self, i, rho, u, uu):
        eu = self.dot(i, u)
        if eu is None:
            return self.w[i] * rho * (1 - 1.5 * uu)
        return self.w[i] * rho * (1 + 3 * eu + 4.5 * eu * eu - 1.5 * uu + 4.5 * eu * (eu * eu - uu))

    def start(self, rho, u):
        uu = sum(c * c for c in u)
        self.f = torch.stack([self.equilibrium(i, rho, u, uu) for i in range(self.Q)])
        if self.ends:
            self.outlet()

    def outlet(self):
        f, x = self.f, self.last
        ru = f[0, x] + f[2, x] + f[4, x] + 2 * (f[1, x] + f[5, x] + f[8, x]) - self.ends[1]
        d = 0.5 * (f[2, x] - f[4, x])
        f[3, x] = f[1, x] - 2 / 3 * ru
        f[7, x] = f[5, x] + d - ru / 6
        f[6, x] = f[8, x] - d - ru / 6

    def moments(self):
        rho = self.f.sum(0)
        u = []
        for a in range(self.D):
            j = sum(float(self.e[i, a]) * self.f[i] for i in range(self.Q) if self.e[i, a])
            u.append(j / rho + 0.5 * self.g[a])
        return rho, u

    def step(self):
        rho, u = self.moments()
        uu = sum(c * c for c in u)
        eq = torch.stack([self.equilibrium(i, rho, u, uu) for i in range(self.Q)])
        neq = self.f - eq
        post = torch.matmul(self.stress, neq)
        post *= self.ap
        post += eq
        del eq
        if self.cubic:
            phi = [torch.where(self.solid, 0.0, rho * c * c * c) for c in u]
            slope = []
            for a in range(self.D):
                v = [0, 0, 0]
                v[a] = 1
                slope.append(0.5 * (phi[a][self.neighbour([-c for c in v])] - phi[a][self.neighbour(v)]))
        b = 1 - 0.5 / self.tau
        ug = sum(u[a] * self.g[a] for a in range(self.D))
        for i in range(self.Q):
            j = self.opp[i]
            eg = self.dot(i, self.g)
            if eg is not None:
                drive = 1.5 * self.w[i] * rho * eg
                post[i] += self.am * (0.5 * (neq[i] - neq[j]) + drive) + drive
            if self.cubic:
                s = sum(float(self.e[i, a] ** 2 - 1 / 3) * slope[a] for a in range(self.D))
                post[i] += -4.5 * b * self.w[i] * s
            if self.guo:
                t = -3 * ug if eg is None else 9 * self.dot(i, u) * eg - 3 * ug
                post[i] += b * self.w[i] * rho * t
        del neq
        post[:, self.solid] = torch.from_numpy(self.w).to(self.dev)[:, None]
        self.post = post
        flat = post.reshape(-1)
        for i in range(self.Q):
            torch.take(flat, self.source[i], out=self.f[i])
        if self.ends:
            for i in range(self.Q):
                if self.e[i, 0] == 1:
                    self.f[i, self.first] = post[self.opp[i], self.first] + 6 * self.w[i] * self.ends[0]
            self.outlet()

    def drag(self):
        total = np.zeros(3)
        fluid = ~self.solid
        for i in range(1, self.Q):
            link = fluid & self.solid[self.neighbour([-c for c in self.e[i]])]
            if self.ends:
                link[self.first if self.e[i, 0] == -1 else self.last] &= bool(self.e[i, 0] == 0)
            total += 2.0 * self.e[i] * float(self.post[i][link].sum())
        return total


def exact(case, seed):
    if case["kind"] == "batch":
        specs, fields = batch_inputs(case, seed)
        shapes = [s["mask"].shape for s in specs]
        m = Plain("d2q9", shapes, [s["mask"] for s in specs], [s["tau_plus"] for s in specs],
                  [s["Lambda"] for s in specs], [s["g"] for s in specs])
        if fields[0] is None:
            one = torch.ones(m.N, dtype=torch.float64, device=m.dev)
            m.start(one, [torch.zeros_like(one)] * 2)
        else:
            m.start(m.field([f[0] for f in fields]), [m.field([f[1][a] for f in fields]) for a in range(2)])
    else:
        tau, lam, force, mask, ends, rho, u = single_inputs(case, seed)
        shapes = [rho.shape]
        m = Plain(case["lattice"], shapes, [mask], [tau], [lam], [force], ends,
                  case["forcing"] == "scheme2+g", case["forcing"] == "guo")
        m.start(m.field([rho]), [m.field([c]) for c in u])
    for _ in range(case["steps"]):
        m.step()
    if case["read"] == "restart":
        f = m.f.clone()
        f[:, m.solid] = 0.0
        return f.reshape((m.Q,) + shapes[0]).cpu().numpy()
    rho, u = m.moments()
    rho, u = (torch.where(m.solid, 0.0, v) for v in (rho, torch.stack(u + [torch.zeros_like(rho)] * (3 - m.D))))
    cut = np.cumsum([0] + [int(np.prod(s)) for s in shapes])
    if case["kind"] == "batch" and case["read"] == "diagnostics":
        energy = 0.5 * rho * (u * u).sum(0)
        parts = [(float(rho[a:b].sum()), float(energy[a:b].sum())) for a, b in zip(cut, cut[1:])]
        return np.array([p[0] for p in parts]), np.array([p[1] for p in parts])
    read = [(rho[a:b].reshape(s).cpu().numpy(), u[:, a:b].reshape((3,) + s).cpu().numpy())
            for a, b, s in zip(cut, cut[1:], shapes)]
    if case["kind"] == "batch":
        return read
    out = {"rho": read[0][0], "u": read[0][1]}
    if "diagnostics" in case["read"]:
        out["mass"], out["energy"] = float(rho.sum()), float((0.5 * rho * (u * u).sum(0)).sum())
    if "drag" in case["read"]:
        out["drag"] = m.drag()
    return out
