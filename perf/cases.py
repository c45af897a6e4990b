"""The calls whose speed is followed, and how each is set up.

A case names one call of the public interface on a synthetic mesh of the shapes
that the benchmark, the tests and the workload generators use: split-square
triangulations of a 10 km square in Hilbert order, extruded in sigma layers or
in flat z-levels (ragged columns, several members), with 1 to 4 tracer fields
and the precision forms of the library.  ``exact`` computes the same outputs in
64 bits with plain torch operations, straight from the definitions.

A case is a dict:
  op      "step", "graph", "rhs", "stage", "solve", "dv" or "gradient"
  mesh    "sigma" (every column has ``layers`` layers) or "zlevel" (5 up to
          ``layers`` layers of 5 m, by a smooth depth field)
  n       squares per side (2 n^2 columns per member); members: their number
  fields  tracer fields (for "dv": components); prec "f64", "f32state", "f32"
  scheme  "lie" or "imex"; okubo: horizontal diffusion scale (0: off)
  w       whether the vertical velocity is read; tune: launch shape measured
          by autotune before the first call, else the library's default
  steps   time steps per call (for "dv": the system, 0 = D_vu, 1 = D_vd)
"""

from __future__ import annotations

import functools
import math

import numpy as np
import torch

SIDE = 10_000.0
DEV = "cuda" if torch.cuda.is_available() else "cpu"


def _case(name, op, mesh, n, layers, fields, prec="f64", scheme="lie", okubo=0.0, w=False, tune=False, steps=1,
          members=1):
    c = dict(op=op, mesh=mesh, n=n, layers=layers, members=members, fields=fields, prec=prec, scheme=scheme,
             okubo=okubo, w=w, tune=tune, steps=steps)
    return dict(c, name=name) if name else c


def listed():
    return [
        # A first try of the library or a unit test: one step of a mesh that fills half a
        # wavefront's cell.  Launches and the column solve's serial chain are all there is.
        _case("tiny_step", "step", "sigma", 4, 7, 2),
        # The plain rotating-blob run: 1,800 columns x 10 layers, one field, ten steps a call.
        _case("blob_10_steps", "step", "sigma", 30, 10, 1, steps=10),
        # The benchmark: a time step of the four-field ocean, 5,991,360 prisms, launch shape tuned.
        _case("ocean_step", "step", "sigma", 316, 30, 4, tune=True),
        # The same with float state and the double column solve.
        _case("ocean_step_f32state", "step", "sigma", 316, 30, 4, "f32state", tune=True),
        # The other time scheme with horizontal diffusion and vertical velocity, an odd mesh.
        _case("ocean_imex_hdiff", "step", "sigma", 173, 41, 3, scheme="imex", okubo=1.0, w=True, tune=True),
        # The batched form: several members of ragged z-level columns, captured step
        # replayed, with the mass diagnostic that a run prints.
        _case("ensemble_graph_mass", "graph", "zlevel", 96, 60, 4, tune=True, steps=2, members=5),
        # Differentiation at the size of the gradient workload (49,928 x 20), default shape.
        _case("gradient_lie", "gradient", "sigma", 158, 20, 1, steps=4),
        # A small inverse problem with the other scheme, two fields and horizontal diffusion.
        _case("gradient_imex", "gradient", "sigma", 47, 13, 2, scheme="imex", okubo=1.0, steps=6),
        # The explicit operator alone (a user's own time stepper), default shape.  In double: a
        # float tendency is mostly the rounding of terms that cancel.
        _case("rhs_w", "rhs", "sigma", 101, 17, 3, w=True),
        # The column solve alone on ragged columns, float everywhere.
        _case("solve_f32_ragged", "solve", "zlevel", 150, 60, 2, "f32"),
        # The pressure-gradient columns, two components, at the benchmark's mesh.
        _case("dv_vu_ocean", "dv", "sigma", 316, 30, 2, steps=0),
        # One SSP-RK3 stage in float on a mid-sized mesh that was not tuned.
        _case("stage_f32", "stage", "sigma", 119, 25, 2, "f32state"),
    ]


def draw(rng):
    op = rng.choice(["step", "step", "step", "graph", "rhs", "stage", "solve", "solve", "dv", "gradient", "gradient"])
    mesh = rng.choice(["sigma", "sigma", "zlevel"])
    layers = rng.randint(3, 60) if mesh == "sigma" else rng.randint(8, 60)
    fields = rng.randint(1, 4) if op != "gradient" else rng.randint(1, 2)
    prec = rng.choice(["f64", "f64", "f32state", "f32"]) if op not in ("gradient", "rhs") else "f64"
    steps = {"step": rng.randint(1, 4), "graph": rng.randint(1, 4), "gradient": rng.randint(2, 6),
             "dv": rng.randint(0, 1)}.get(op, 1)
    members = rng.randint(1, 6) if mesh == "zlevel" else 1
    # from 18 columns to 3 million prisms a call over all its steps, spread over the logarithm
    prisms = math.exp(rng.uniform(math.log(18.0 * layers), math.log(3.0e6 / max(steps, 1))))
    n = max(3, min(300, round(math.sqrt(prisms / (2.0 * layers * members)))))
    return _case("", op, mesh, n, layers, fields, prec, rng.choice(["lie", "lie", "imex"]),
                 rng.choice([0.0, 0.0, 1.0]) if op != "solve" else 0.0, rng.random() < 0.3,
                 op in ("step", "graph") and prisms > 2.0e5 and rng.random() < 0.7, steps, members)


# ---------------------------------------------------------------------------
# Meshes and inputs
# ---------------------------------------------------------------------------
def _hilbert(px, py, bits=16):
    n = 1 << bits
    span = max(np.ptp(px), np.ptp(py), 1e-300)
    x = np.minimum(((px - px.min()) / span * (n - 1)).astype(np.int64), n - 1)
    y = np.minimum(((py - py.min()) / span * (n - 1)).astype(np.int64), n - 1)
    d = np.zeros_like(x)
    s = n // 2
    while s:
        rx, ry = ((x & s) > 0).astype(np.int64), ((y & s) > 0).astype(np.int64)
        d += s * s * ((3 * rx) ^ ry)
        flip = (ry == 0) & (rx == 1)
        x, y = np.where(flip, n - 1 - x, x), np.where(flip, n - 1 - y, y)
        x, y = np.where(ry == 0, y, x), np.where(ry == 0, x, y)
        s //= 2
    return np.argsort(d, kind="stable")


def _square(n, seed):
    """Jittered split squares in Hilbert order: vertices, triangles, neighbours, neighbours' edges."""
    h = SIDE / n
    ii, jj = np.meshgrid(np.arange(n + 1), np.arange(n + 1), indexing="ij")
    vid = (ii * (n + 1) + jj).astype(np.int32)
    vxy = np.stack([ii.ravel() * h, jj.ravel() * h], axis=1).astype(np.float64)
    inner = ((ii > 0) & (ii < n) & (jj > 0) & (jj < n)).ravel()
    vxy[inner] += np.random.default_rng(seed).uniform(-0.2, 0.2, size=vxy.shape)[inner] * h
    bl, br, tr, tl = (v.ravel() for v in (vid[:-1, :-1], vid[1:, :-1], vid[1:, 1:], vid[:-1, 1:]))
    tri = np.concatenate([np.stack([bl, br, tr], 1), np.stack([bl, tr, tl], 1)]).astype(np.int32)
    mid = vxy[tri].mean(axis=1)
    tri = tri[_hilbert(mid[:, 0], mid[:, 1])]
    a, b = tri.astype(np.int64), np.roll(tri, -1, axis=1).astype(np.int64)
    key = (np.minimum(a, b) * len(vxy) + np.maximum(a, b)).ravel()
    order = np.argsort(key, kind="stable")
    pair = key[order[1:]] == key[order[:-1]]
    i, j = order[:-1][pair], order[1:][pair]
    other = np.full(key.size, -1, dtype=np.int64)
    other[i], other[j] = j, i
    other = other.reshape(-1, 3)
    return vxy, tri, np.where(other < 0, -1, other // 3).astype(np.int32), np.where(other < 0, 0, other % 3)


@functools.lru_cache(maxsize=2)
def _mesh(kind, n, layers, members):
    """Host arrays of a mesh, its columns padded to the deepest one in ``z`` (C, N + 1, 3)."""
    parts, moff = [], [0]
    for m in range(members):
        parts.append(_square(max(3, n - 7 * m % max(n // 2, 1)) if m else n, 1000 + m))
        moff.append(moff[-1] + len(parts[-1][1]))
    voff = np.concatenate([[0], np.cumsum([len(p[0]) for p in parts])])
    vxy = np.concatenate([p[0] for p in parts])
    tri = np.concatenate([p[1] + voff[m] for m, p in enumerate(parts)]).astype(np.int32)
    nbr = np.concatenate([np.where(p[2] >= 0, p[2] + moff[m], -1) for m, p in enumerate(parts)]).astype(np.int32)
    edge = np.concatenate([p[3] for p in parts])
    C = len(tri)
    if kind == "sigma":
        nl = np.full(C, layers, dtype=np.int32)
        h = 20.0 + 10.0 * np.sin(np.pi * vxy[:, 0] / SIDE) * np.sin(np.pi * vxy[:, 1] / SIDE)
        z = -(np.arange(layers + 1) / layers)[None, :, None] * h[tri][:, None, :]
    else:
        mid = vxy[tri].mean(axis=1)
        rng = np.random.default_rng(7)
        g = np.zeros(C)
        for _ in range(3):
            kx, ky = rng.integers(1, 4, size=2)
            px, py = rng.uniform(0, 2 * np.pi, size=2)
            g += np.cos(np.pi * kx * mid[:, 0] / SIDE + px) * np.cos(np.pi * ky * mid[:, 1] / SIDE + py)
        g = (g - g.min()) / max(np.ptp(g), 1e-300)
        nl = np.clip(np.ceil(5 + (layers - 5) * g), 5, layers).astype(np.int32)
        z = np.broadcast_to((-5.0 * np.arange(layers + 1))[None, :, None], (C, layers + 1, 3))
    N = int(nl.max())
    z = np.ascontiguousarray(z[:, :N + 1], dtype=np.float64)
    deep = np.zeros(-(-C // 64) * 64, dtype=np.int64)
    deep[:C] = nl
    deep = deep.reshape(-1, 64).max(axis=1)
    base = 64 * np.concatenate([[0], np.cumsum(deep)])
    live = np.arange(N)[None, :] < nl[:, None]
    slot = (base[np.arange(C) // 64] + np.arange(C) % 64)[:, None] + 64 * np.arange(N)[None, :]
    p = vxy[tri]
    sides = [np.hypot(*(p[:, k] - p[:, (k + 1) % 3]).T) for k in range(3)]
    area2 = ((p[:, 1, 0] - p[:, 0, 0]) * (p[:, 2, 1] - p[:, 0, 1]) - (p[:, 2, 0] - p[:, 0, 0]) * (p[:, 1, 1] - p[:, 0, 1]))
    return dict(vxy=vxy, tri=tri, nbr=nbr, edge=edge, nl=nl, z=z, live=live, slots=slot[live], n_slots=int(base[-1]),
                zlev=np.ascontiguousarray(z[np.arange(N + 1)[None, :] <= nl[:, None]]), N=N, C=C,
                moff=np.asarray(moff, dtype=np.int32), dt=float(0.3 * (2.0 * area2 / sum(sides)).min() / 0.75))


def _mesh_of(case):
    return _mesh(case["mesh"], case["n"], case["layers"], case["members"])


def _kappa(N):
    return 10.0 ** (-2.0 - 3.0 * torch.arange(N, dtype=torch.float64, device=DEV) / max(N - 1, 1))


EXTERIOR = (0.0, 0.0, 17.5, 35.0)


def _inputs(case, seed):
    """Velocity (3, 6, C, N) and fields (F, 6, C, N): a sheared rotation about a centre drawn from
    the seed, its components, a temperature that falls with depth and a salinity, both with noise;
    for "dv" unit normal right-hand sides.  One field: the temperature."""
    m = _mesh_of(case)
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    rand = lambda *s: torch.rand(*s, dtype=torch.float64, device=DEV, generator=gen)  # noqa: E731
    C, N, F = m["C"], m["N"], case["fields"]
    if case["op"] == "dv":
        return None, torch.randn(F, 6, C, N, dtype=torch.float64, device=DEV, generator=gen)
    xy = torch.as_tensor(m["vxy"], device=DEV)[torch.as_tensor(m["tri"], device=DEV).long()]       # (C, 3, 2)
    z = torch.as_tensor(m["z"], device=DEV)
    zn = torch.cat([z[:, :-1], z[:, 1:]], dim=2).permute(2, 0, 1)                                    # (6, C, N)
    x, y = (torch.cat([xy[..., d], xy[..., d]], dim=1).T[:, :, None] for d in (0, 1))                # (6, C, 1)
    c = 0.5 * SIDE + 500.0 * (rand(2) - 0.5)
    om = 0.5 * math.sqrt(2.0) / SIDE
    rel = zn / -float(z.min())
    shear = 1.0 + 0.2 * rel
    U = torch.stack([-om * (y - c[1]) * shear, om * (x - c[0]) * shear,
                     1e-3 * torch.sin(math.pi * x / SIDE) * torch.sin(math.pi * y / SIDE) * (1.0 + rel) if case["w"]
                     else torch.zeros_like(rel)])
    temp = 25.0 + 15.0 * rel + 3.0 * torch.exp(-((x - 7000.0) ** 2 + (y - 5000.0) ** 2) / 2.0e6) + 0.2 * rand(6, C, N)
    salt = 34.5 + rand(6, C, N)
    return U, torch.stack([[temp], [U[0], temp], [U[0], temp, salt], [U[0], U[1], temp, salt]][F - 1])


def _exterior(case):
    return [(17.5,), (0.0, 17.5), (0.0, 17.5, 35.0), EXTERIOR][case["fields"] - 1]


def _to_slots(m, dense, dtype):
    """(K, 6, C, N) values -> (K, 6, n_slots) storage, zero where no prism is."""
    out = torch.zeros(dense.shape[0], 6, m["n_slots"], dtype=dtype, device=DEV)
    out[:, :, torch.as_tensor(m["slots"], device=DEV)] = dense[:, :, torch.as_tensor(m["live"], device=DEV)].to(dtype)
    return out


def prepare(case, seed):
    import paper_2605_16082_amd as P

    m = _mesh_of(case)
    prec = {"f64": P.SDG_FP64, "f32": P.SDG_FP32, "f32state": P.SDG_FP32_STATE_FP64_SOLVE}[case["prec"]]
    s = P.SlimDG(P.Mesh(m["vxy"], m["tri"], m["nbr"], m["nl"], m["zlev"], case["fields"], prec,
                        m["moff"] if case["members"] > 1 else None))
    U, T = _inputs(case, seed)
    st = {"case": case, "s": s, "P": P, "T": _to_slots(m, T, s.dtype)}
    del T
    if case["op"] == "dv":
        return dict(st, out=s.zeros(case["fields"]))
    st["U"] = _to_slots(m, U, s.dtype)
    st["kappa"] = _kappa(m["N"])
    s.set_params(m["dt"], _exterior(case), w_is_zero=not case["w"], okubo_scale=case["okubo"],
                 time_scheme=P.SDG_SCHEME_SPLIT_IMEX if case["scheme"] == "imex" else P.SDG_SCHEME_SSPRK3_LIE)
    s.set_velocity(st["U"])
    s.set_diffusivity(st["kappa"])
    if case["op"] in ("step", "graph"):
        s.set_fields(st["T"])
        if case["tune"]:
            s.autotune(reps=2)
        if case["op"] == "graph":
            s.graph_capture_step()
    elif case["op"] != "gradient":
        st["out"] = s.new_state()
        st["Tn"] = st["T"].clone() if case["op"] == "stage" else None
    return st


def run(st):
    case, s, T = st["case"], st["s"], st["T"]
    op = case["op"]
    if op == "step":
        s.step(case["steps"])
        return T
    if op == "graph":
        s.graph_launch(case["steps"])
        return {"state": T, "mass": s.mass(T)}
    if op == "rhs":
        return s.rhs_3d(T, st["out"])
    if op == "stage":
        return s.rk_stage(1, st["Tn"], T, st["out"])
    if op == "solve":
        return s.vertical_implicit_solve(T, st["out"])
    if op == "dv":
        return s.column_dv_solve(case["steps"], T, st["out"])
    T0 = T.detach().requires_grad_(True)
    kap = st["kappa"].detach().requires_grad_(True)
    J = st["P"].MNorm.apply(st["P"].TracerSteps.apply(T0, kap, s, case["steps"], 3), s)
    J.backward()
    return {"J": J.detach(), "T0": T0.grad, "kappa": kap.grad}


def work(case):
    m = _mesh_of(case)
    prisms, F, es = int(m["nl"].sum()), case["fields"], 8 if case["prec"] == "f64" else 4
    state = 6.0 * F * prisms * es
    vel = 6.0 * (3 if case["w"] else 2) * prisms * es
    mesh = 3.0 * (prisms + m["C"]) * es + m["C"] * (6 * es + 12.0)
    # multiply-adds count two: an explicit evaluation's factors and fields, a column solve's layers
    explicit, solve = (1400.0 + 450.0 * F) * prisms, (1100.0 + 330.0 * F) * prisms
    if case["okubo"]:
        explicit += (150.0 + 350.0 * F) * prisms
    evals = 2 if case["scheme"] == "imex" else 3
    # one step: state in and out, velocity and mesh, each once
    step = {"bytes": 2 * state + vel + mesh, "flops": evals * explicit + solve}
    op, k = case["op"], max(case["steps"], 1)
    if op in ("step", "graph"):
        return {"bytes": k * step["bytes"] + (state if op == "graph" else 0), "flops": k * step["flops"]}
    if op in ("rhs", "stage"):
        return {"bytes": (2 + (op == "stage")) * state + vel + mesh, "flops": explicit}
    if op == "solve":
        return {"bytes": 2 * state + mesh, "flops": solve}
    if op == "dv":
        return {"bytes": 2 * state + 12.0 * m["C"], "flops": 40.0 * F * prisms}
    # forward and reverse steps (the reverse reads the forward state too)
    return {"bytes": k * (2 * step["bytes"] + state), "flops": 2 * k * step["flops"]}


# ---------------------------------------------------------------------------
# The same outputs in 64 bits
# ---------------------------------------------------------------------------
_A1, _W1 = 0.44594849091596488631832925388305199, 0.22338158967801146569500700843312280
_A2, _W2 = 0.091576213509770743459571463402201508, 0.10995174365532186763832632490021053
_TRI = [(lam, 0.5 * w) for a, w in ((_A1, _W1), (_A2, _W2))
        for lam in ((1 - 2 * a, a, a), (a, 1 - 2 * a, a), (a, a, 1 - 2 * a))]
_ZETA = [((1 + s / math.sqrt(3.0)) / 2, (1 - s / math.sqrt(3.0)) / 2) for s in (-1.0, 1.0)]   # top, bottom weight
_EDGE = [(0.5 + s * math.sqrt(0.15), w / 18.0) for s, w in ((-1, 5), (0, 8), (1, 5))]


def _at(lam, t, b, v):
    """Value of nodal data v (K, 6, ...) at barycentric ``lam`` and vertical weights (t, b)."""
    return sum(lam[a] * (t * v[:, a] + b * v[:, a + 3]) for a in range(3) if lam[a])


def _eliminate(A, rhs):
    """A^-1 rhs for small matrices A (n, n, ...), rhs (n, k, ...), by Gauss-Jordan elimination."""
    n = len(A)
    rows = [torch.cat([A[i], rhs[i]]) for i in range(n)]
    for k in range(n):
        rows[k] = rows[k] / rows[k][k].clone()
        rows = [r if i == k else r - r[k] * rows[k] for i, r in enumerate(rows)]
    return torch.stack([r[n:] for r in rows])


def _mul(A, B):
    """(i, j, ...) x (j, k, ...) -> (i, k, ...)."""
    return sum(A[:, j, None] * B[j][None] for j in range(A.shape[1]))


class _Exact:
    def __init__(self, case):
        m = _mesh_of(case)
        dev = lambda v: torch.as_tensor(v, device=DEV)  # noqa: E731
        xy, z = dev(m["vxy"])[dev(m["tri"]).long()], dev(m["z"])
        self.m, self.case, self.N, self.nl = m, case, m["N"], dev(m["nl"]).long()
        self.live = dev(m["live"])
        self.nbr, self.edge = dev(m["nbr"]).long(), dev(m["edge"]).long()
        self.lay = torch.arange(self.N, device=DEV)
        self.zn = torch.cat([z[:, :-1], z[:, 1:]], dim=2).permute(2, 0, 1)
        self.dz = self.zn[:3] - self.zn[3:]
        d1, d2 = xy[:, 1] - xy[:, 0], xy[:, 2] - xy[:, 0]
        self.xxi, self.yxi, self.xet, self.yet = (v[:, None] for v in (d1[:, 0], d1[:, 1], d2[:, 0], d2[:, 1]))
        self.J = self.xxi * self.yet - self.xet * self.yxi                     # (C, 1)
        # gradients of the barycentric functions, edge normals and lengths
        g1, g2 = (self.yet / self.J, -self.xet / self.J), (-self.yxi / self.J, self.xxi / self.J)
        self.gl = [(-g1[0] - g2[0], -g1[1] - g2[1]), g1, g2]
        e = [xy[:, (k + 1) % 3] - xy[:, k] for k in range(3)]
        self.len = [torch.hypot(v[:, 0], v[:, 1])[:, None] for v in e]
        self.nrm = [(v[:, 1, None] / L, -v[:, 0, None] / L) for v, L in zip(e, self.len)]
        self.Mz = torch.zeros(3, 3, *self.dz.shape[1:], dtype=torch.float64, device=DEV)
        for lam, w in _TRI:
            c = w * 0.5 * sum(lam[a] * self.dz[a] for a in range(3)) * self.J
            for a in range(3):
                for b in range(3):
                    self.Mz[a, b] += lam[a] * lam[b] * c
        self.Mz = self.Mz * 2.0                                                # J int l_a l_b dz
        self.dt, self.text = m["dt"], _exterior(case)
        self.kh = case["okubo"] * 0.0103 * 100.0 ** 1.15 * 1e-4 * self.J ** 0.575

    def mass(self, T):
        """M T: M = [2 1; 1 2] / 6 x (J int l_a l_b dz)."""
        t, b = _mul(self.Mz, T[:, :3].transpose(0, 1)), _mul(self.Mz, T[:, 3:].transpose(0, 1))
        return torch.cat([2 * t + b, t + 2 * b]).transpose(0, 1) / 6.0

    def mass_inv(self, R):
        R = R.transpose(0, 1)
        x = _eliminate(self.Mz, torch.cat([R[:3], R[3:]], dim=1))
        t, b = x[:, :R.shape[1]], x[:, R.shape[1]:]
        return torch.cat([4 * t - 2 * b, 4 * b - 2 * t]).transpose(0, 1)

    def neighbour(self, V, e):
        """V's values (K, 4, C, N) at the neighbour's nodes A top, B top, A bottom, B bottom."""
        nb, k = self.nbr[:, e].clamp(min=0), self.edge[:, e]
        a, b = (k + 1) % 3, k
        return torch.stack([V[:, i, nb] for i in (a, b, a + 3, b + 3)], dim=1)

    def masks(self, e):
        inner = self.nbr[:, e, None] >= 0
        wall = inner & (self.lay[None] >= self.nl[self.nbr[:, e].clamp(min=0), None])
        return inner & ~wall, wall

    def advect(self, U, T):
        R = [0.0] * 6
        for lam, w in _TRI:
            zz = 0.5 * sum(lam[a] * self.dz[a] for a in range(3))
            for t, b in _ZETA:
                u, Tq = _at(lam, t, b, U), _at(lam, t, b, T)
                zx = t * (self.zn[1] - self.zn[0]) + b * (self.zn[4] - self.zn[3])
                ze = t * (self.zn[2] - self.zn[0]) + b * (self.zn[5] - self.zn[3])
                al, be = self.yet * u[0] - self.xet * u[1], self.xxi * u[1] - self.yxi * u[0]
                fx, fe, fz = w * zz * al * Tq, w * zz * be * Tq, w * (self.J * u[2] - zx * al - ze * be) * Tq
                for a, (gx, ge) in enumerate(((-1, -1), (1, 0), (0, 1))):
                    R[a] = R[a] + t * (gx * fx + ge * fe) + 0.5 * lam[a] * fz
                    R[a + 3] = R[a + 3] + b * (gx * fx + ge * fe) - 0.5 * lam[a] * fz
        text = torch.tensor(self.text, dtype=torch.float64, device=DEV)[:, None, None]
        upwind = lambda q, i, o: torch.where(q > 0, q * i, q * o)  # noqa: E731
        for e in range(3):
            A, B = e, (e + 1) % 3
            own = [A, B, A + 3, B + 3]
            alive, wall = self.masks(e)
            Un, To = self.neighbour(U[:2], e), self.neighbour(T, e)
            To = torch.where(alive, To, text[:, None])
            Um = torch.where(alive, 0.5 * (U[:2][:, own] + Un), U[:2][:, own])
            un = self.nrm[e][0] * Um[0] + self.nrm[e][1] * Um[1]
            Ti = T[:, own]
            for s, w in _EDGE:
                dS = w * self.len[e] * 0.5 * ((1 - s) * self.dz[A] + s * self.dz[B])
                for t, b in _ZETA:
                    c = ((1 - s) * t, s * t, (1 - s) * b, s * b)
                    f = upwind(sum(c[i] * un[i] for i in range(4)) * dS, sum(c[i] * Ti[:, i] for i in range(4)),
                               sum(c[i] * To[:, i] for i in range(4)))
                    f = torch.where(wall, 0.0, f)
                    for i, node in enumerate(own):
                        R[node] = R[node] - c[i] * f
        # horizontal faces 0 (surface) .. N: the prisms below and above each
        last = self.lay[None] == self.nl[:, None] - 1
        pad = lambda v, where: torch.cat([v, v[..., :1]], -1) if where else torch.cat([v[..., :1], v], -1)  # noqa: E731
        zf = torch.cat([self.zn[:3], self.zn[3:, :, -1:]], -1)
        zx, ze = zf[1] - zf[0], zf[2] - zf[0]
        jx, jy = zx * self.yet - ze * self.yxi, ze * self.xxi - zx * self.xet
        has_lo = torch.cat([torch.ones_like(last[:, :1]), ~last], -1)
        has_up = torch.ones_like(has_lo)
        has_up[:, 0] = False
        side = lambda v: self.J * v[2] - jx * v[0] - jy * v[1]  # noqa: E731
        nu, nlo = side(pad(U[:, 3:], False)), side(pad(U[:, :3], True))
        un = torch.where(has_up & has_lo, 0.5 * (nu + nlo), torch.where(has_up, nu, nlo))
        Tu = torch.where(has_up, pad(T[:, 3:], False), text[:, None])
        Tl = torch.where(has_lo, pad(T[:, :3], True), text[:, None])
        for lam, w in _TRI:
            q = w * sum(lam[a] * un[a] for a in range(3))
            f = upwind(q, *(sum(lam[a] * V[:, a] for a in range(3)) for V in (Tl, Tu)))
            for a in range(3):
                R[a] = R[a] - lam[a] * f[..., :-1]
                R[a + 3] = R[a + 3] + lam[a] * f[..., 1:]
        return torch.stack(R, dim=1)

    def diffuse(self, T):
        """Along-layer symmetric interior penalty diffusion."""
        R = [0.0] * 6
        grad = lambda V, gl, t, b: [sum(gl[a][d] * (t * V[:, a] + b * V[:, a + 3]) for a in range(3)) for d in (0, 1)]  # noqa: E731
        vol = self.kh * self.J * self.dz.sum(0) / 12.0
        for t, b in _ZETA:
            g = grad(T, self.gl, t, b)
            for a in range(3):
                f = vol * (self.gl[a][0] * g[0] + self.gl[a][1] * g[1])
                R[a], R[a + 3] = R[a] - t * f, R[a + 3] - b * f
        for e in range(3):
            A, B = e, (e + 1) % 3
            alive, _ = self.masks(e)
            nb = self.nbr[:, e].clamp(min=0)
            n, L = self.nrm[e], self.len[e]
            gn = [(g[0][nb], g[1][nb]) for g in self.gl]
            kn, Tn, To = self.kh[nb], T[:, :, nb], self.neighbour(T, e)
            sig = 4.0 * 0.5 * (self.kh + kn) / (torch.minimum(self.J, self.J[nb]) / L)
            for t, b in _ZETA:
                gi, go = grad(T, self.gl, t, b), grad(Tn, gn, t, b)
                mean = 0.5 * (self.kh * (gi[0] * n[0] + gi[1] * n[1]) + kn * (go[0] * n[0] + go[1] * n[1]))
                for s, w in _EDGE:
                    dS = torch.where(alive, w * L * 0.5 * ((1 - s) * self.dz[A] + s * self.dz[B]), 0.0)
                    jump = ((1 - s) * (t * (T[:, A] - To[:, 0]) + b * (T[:, A + 3] - To[:, 2]))
                            + s * (t * (T[:, B] - To[:, 1]) + b * (T[:, B + 3] - To[:, 3])))
                    flux = dS * (mean - sig * jump)
                    for a, wt in ((A, 1 - s), (B, s)):
                        R[a], R[a + 3] = R[a] + wt * t * flux, R[a + 3] + wt * b * flux
                    sym = dS * 0.5 * self.kh * jump
                    for a in range(3):
                        d = self.gl[a][0] * n[0] + self.gl[a][1] * n[1]
                        R[a], R[a + 3] = R[a] + t * d * sym, R[a + 3] + b * d * sym
        return torch.stack(R, dim=1)

    def rhs(self, U, T):
        R = self.advect(U, T)
        if self.case["okubo"]:
            R = R + self.diffuse(T)
        return torch.where(self.live, self.mass_inv(R), 0.0)

    def solve(self, T, kappa, dt):
        """(M - dt A) x = M T by block elimination down each column."""
        C = T.shape[2]
        S = (self.J[:, 0] / 24.0) * (torch.ones(3, 3, 1, device=DEV, dtype=torch.float64)
                                    + torch.eye(3, device=DEV, dtype=torch.float64)[:, :, None])
        Kv = torch.zeros(3, 3, C, self.N, dtype=torch.float64, device=DEV)
        for lam, w in _TRI:
            c = w * self.J / sum(lam[a] * self.dz[a] for a in range(3))
            for a in range(3):
                for b in range(3):
                    Kv[a, b] += lam[a] * lam[b] * c
        hbar = self.dz.mean(0)
        MT = self.mass(T)
        two = lambda a, b: torch.cat([a, b], dim=1)  # noqa: E731
        zero = torch.zeros(3, 3, C, dtype=torch.float64, device=DEV)
        K = [0.5 * dt * kappa[l] * Kv[..., l] for l in range(self.N)]
        on = [self.nl > l for l in range(self.N)]
        sig = [zero[0, 0]] + [torch.where(on[l], dt * 4.0 * 0.5 * (kappa[l - 1] + kappa[l])
                                          / torch.minimum(hbar[:, l - 1], hbar[:, l]), 0.0) for l in range(1, self.N)]
        E, y = [], []
        for l in range(self.N):
            up = on[l] if l else torch.zeros_like(on[l])
            dn = on[l + 1] if l + 1 < self.N else torch.zeros_like(on[l])
            M = self.Mz[..., l] / 6.0
            k2 = 2 * K[l]
            ku, kd = torch.where(up, K[l], 0.0), torch.where(dn, K[l], 0.0)
            sd = sig[l + 1] * S if l + 1 < self.N else zero
            D = torch.cat([two(2 * M + k2 - ku + torch.where(up, sig[l] * S, 0.0), M - k2 + ku),
                           two(M - k2 + kd, 2 * M + k2 - kd + torch.where(dn, sd, 0.0))])
            r = MT[..., l].transpose(0, 1)
            if l:
                Bl = torch.where(up, two(-K[l - 1], K[l - 1] - sig[l] * S), 0.0)
                Cu = torch.where(up, two(K[l] - sig[l] * S, -K[l]), 0.0)
                D = torch.cat([D[:3] - _mul(_mul(Bl, E[-1]), Cu), D[3:]])
                r = torch.cat([r[:3] - _mul(Bl, y[-1]), r[3:]])
            unit = torch.cat([zero, zero + torch.eye(3, device=DEV, dtype=torch.float64)[:, :, None]])
            sol = _eliminate(D, torch.cat([unit, r], dim=1))
            E.append(sol[:, :3])
            y.append(sol[:, 3:])
        x = [None] * self.N
        x[-1] = y[-1]
        for l in range(self.N - 2, -1, -1):
            Cl = torch.where(on[l + 1], two(K[l + 1] - sig[l + 1] * S, -K[l + 1]), 0.0)
            x[l] = y[l] - _mul(E[l], _mul(Cl, x[l + 1]))
        return torch.where(self.live, torch.stack(x, dim=-1).transpose(0, 1), 0.0)

    def step(self, U, T, kappa):
        from torch.utils.checkpoint import checkpoint
        rhs = (lambda V: checkpoint(self.rhs, U, V, use_reentrant=False)) if T.requires_grad else (lambda V: self.rhs(U, V))
        dt = self.dt
        if self.case["scheme"] == "imex":
            y = T + 0.5 * dt * rhs(T)
            xh = self.solve(y, kappa, 0.5 * dt)
            return T + 2.0 * (xh - y) + dt * rhs(xh)
        T1 = T + dt * rhs(T)
        T2 = 0.75 * T + 0.25 * (T1 + dt * rhs(T1))
        return self.solve(T / 3.0 + (2.0 / 3.0) * (T2 + dt * rhs(T2)), kappa, dt)


def exact(case, seed):
    m = _mesh_of(case)
    if int(m["nl"].sum()) * case["steps"] > 1.3e7 and case["op"] in ("step", "graph"):
        return None
    x = _Exact(case)
    kind = torch.float64 if case["prec"] == "f64" else torch.float32
    U, T = _inputs(case, seed)
    if kind is torch.float32:   # the values that the call is given
        T = T.to(kind).double()
        U = None if U is None else U.to(kind).double()
    out = lambda V: _to_slots(m, V, torch.float64)  # noqa: E731
    op = case["op"]
    if op == "dv":
        T = torch.where(x.live, T, 0.0)
        f = [24.0 / x.J * (T[:, h:h + 3] - T[:, h:h + 3].sum(1, keepdim=True) / 4.0) for h in (0, 3)]   # M_h^-1 F
        total = f[0] + f[1]
        if case["steps"] == 0:
            xb = -total.cumsum(-1)
            xt = xb + 2.0 * f[1]
        else:
            xt = total.flip(-1).cumsum(-1).flip(-1)
            xb = xt - 2.0 * f[0]
        return out(torch.cat([xt, xb], dim=1))
    kappa = _kappa(m["N"])
    if op == "rhs":
        return out(x.rhs(U, T))
    if op == "stage":
        return out(0.75 * T + 0.25 * (T + x.dt * x.rhs(U, T)))
    if op == "solve":
        return out(x.solve(T, kappa, x.dt))
    if op == "gradient":
        T0, kap = T.clone().requires_grad_(True), kappa.clone().requires_grad_(True)
        V = T0
        for _ in range(case["steps"]):
            V = x.step(U, V, kap)
        J = torch.where(x.live, V * x.mass(V), 0.0).sum().sqrt()
        J.backward()
        return {"J": J.detach(), "T0": out(torch.where(x.live, T0.grad, 0.0)), "kappa": kap.grad}
    for _ in range(case["steps"]):
        T = x.step(U, T, kappa)
    if op == "step":
        return out(T)
    per = (torch.where(x.live, x.mass(T), 0.0)).sum(dim=(1, 3))                    # (F, C)
    off = m["moff"]
    sums = torch.stack([per[:, off[i]:off[i + 1]].sum(1) for i in range(len(off) - 1)])
    return {"state": out(T), "mass": sums.cpu().numpy()}
