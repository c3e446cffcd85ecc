"""The workloads whose speed this framework is judged by, each one pass
through its public entry points (``paper_2404_19751_amd.gsim``).

``listed()`` gives them by name, ``draw(rng)`` more of the same ranges,
``prepare`` what a program has in hand before the call (device tensors of
positions, a context with the mesh uploaded), ``run`` one pass, ``work`` the
bytes and operations a pass cannot do without, and ``exact`` the result in 64
bits from plain torch: straight links by unfolding faces in the plane of
their root, shortest chains of links over the bend vertices, and a walk in
the faces' own frames.

Every pass starts from positions handed in as device tensors
(``particles_set_dev``), so that a pass is the same work each time.
"""
import functools
import math

import numpy as np
import torch

from paper_2404_19751_amd import gsim
from paper_2404_19751_amd import workloads as W

DEV = "cuda" if torch.cuda.is_available() else "cpu"
F64 = torch.float64


# ------------------------------------------------------------------- cases
def listed():
    return [
        # one force evaluation of a small system: latency and launches only
        dict(name="forces_sphere_64", kind="forces", mesh="sphere", size=3, n=64, range=0.5, potential="harmonic"),
        # overdamped relaxation of an ordinary system on a curved surface with
        # saddles: fewer particles than the device has wavefront slots
        dict(name="steps_bumpy_1000", kind="steps", mesh="bumpy", size=5, n=1000, range=0.15, potential="harmonic",
             integrator="overdamped", steps=20),
        # Brownian dynamics on a large open height field (199,712 faces)
        dict(name="steps_height_20000", kind="steps", mesh="height", size=316, n=20000, range=0.11,
             potential="harmonic", integrator="brownian", steps=10),
        # neighbour distances and tangents for a program that goes on in torch
        dict(name="pairs_height_7001", kind="pairs", mesh="height", size=211, n=7001, range=0.23),
        # sixteen independent surfaces of all sizes in one batch, both
        # precisions (FP32 trajectories of longer runs part by themselves)
        dict(name="batch16_fp64", kind="batch", first=0, count=16, steps=20, precision="fp64"),
        dict(name="batch16_fp32", kind="batch", first=0, count=16, steps=6, precision="fp32_mixed"),
        # molecular dynamics on the benchmark torus: tens, then hundreds of
        # neighbours per particle
        dict(name="nve_torus_8192_58", kind="steps", mesh="torus", size=28, n=8192, range=0.5, potential="harmonic",
             integrator="verlet", steps=10),
        dict(name="nve_torus_8192_232", kind="steps", mesh="torus", size=28, n=8192, range=1.0, potential="harmonic",
             integrator="verlet", steps=3),
        # charges on a sphere of 81,920 faces, every pair: one FIRE iteration
        dict(name="fire_sphere_2000", kind="fire", mesh="sphere", size=6, n=2000),
        # distances between a hundred landmarks across a whole mesh
        dict(name="allpairs_torus_100", kind="pairs", mesh="torus", size=24, n=100, range=0.0),
        # coordination numbers of a particle packing (host arrays)
        dict(name="voronoi_torus_500", kind="voronoi", mesh="torus", size=28, n=500),
        # a hundred thousand tracers moved straight across faces
        dict(name="walk_height_100000", kind="walk", mesh="height", size=316, n=100000, length=0.08),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["forces", "steps", "steps", "pairs", "batch", "dense", "fire", "allpairs", "voronoi", "walk"])
    if kind in ("forces", "steps", "pairs"):
        mesh = rng.choice(["sphere", "bumpy", "height", "torus"])
        size = {"sphere": rng.randint(3, 5), "bumpy": rng.randint(4, 5), "height": int(_log(rng, 40, 316)),
                "torus": int(_log(rng, 20, 90))}[mesh]
        m = _mesh(mesh, size)
        r = rng.uniform(2.0, 4.5) * _edge(mesh, size)
        n = int(min(20000, max(64, _log(rng, 2.0, 12.0) * _area(mesh, size) / (math.pi * r * r))))
        n = min(n, 2 * m.nf)
        c = dict(kind=kind, mesh=mesh, size=size, n=n, range=round(r, 4))
        if kind != "pairs":
            c["potential"] = rng.choice(["harmonic", "gaussian"])
        if kind == "steps":
            c.update(integrator=rng.choice(["overdamped", "brownian", "verlet"]), steps=rng.randint(1, 10))
        return c
    if kind == "batch":
        count = rng.randint(2, 16)
        prec = rng.choice(["fp64", "fp64", "fp32_mixed"])
        return dict(kind="batch", first=rng.randint(0, 16 - count), count=count,
                    steps=rng.randint(2, 20 if prec == "fp64" else 6), precision=prec)
    if kind == "dense":
        r = rng.choice([0.5, 0.7, 1.0])
        return dict(kind="steps", mesh="torus", size=rng.randint(20, 32), n=int(_log(rng, 1000, 8192)), range=r,
                    potential="harmonic", integrator="verlet", steps=rng.randint(1, 4))
    if kind == "fire":
        return dict(kind="fire", mesh="sphere", size=rng.randint(3, 5), n=int(_log(rng, 60, 1500)))
    if kind == "allpairs":
        return dict(kind="pairs", mesh=rng.choice(["torus", "bumpy"]), size=rng.choice([12, 17, 24, 34]),
                    n=int(_log(rng, 50, 400)), range=0.0) if rng.random() < 0.6 else \
            dict(kind="pairs", mesh="sphere", size=rng.randint(3, 4), n=int(_log(rng, 50, 800)), range=0.0)
    if kind == "voronoi":
        return dict(kind="voronoi", mesh="torus", size=rng.randint(20, 48), n=int(_log(rng, 200, 1000)))
    return dict(kind="walk", mesh="height", size=int(_log(rng, 60, 316)), n=int(_log(rng, 1000, 100000)),
                length=round(rng.uniform(0.02, 0.2), 3))


@functools.lru_cache(maxsize=8)
def _mesh(mesh, size):
    if mesh == "sphere":
        return W.icosphere(size)
    if mesh == "bumpy":
        return W.bumpy_sphere(min(size, 5))
    if mesh == "height":
        return W.height_field(size)
    return W.torus(3.0, 1.0, 83 if size == 28 else 3 * size, size)  # 28: the benchmark torus, 4648 faces


@functools.lru_cache(maxsize=64)
def _edge(mesh, size):
    return W.mean_edge_length(_mesh(mesh, size))


@functools.lru_cache(maxsize=64)
def _area(mesh, size):
    return W.surface_area(_mesh(mesh, size))


@functools.lru_cache(maxsize=1)
def _batch_surfaces():
    """(mesh, range, particles) of the sixteen surfaces: icospheres and tori
    at packing fraction 0.3, range two mean edges."""
    out = []
    for m in [W.icosphere(lv) for lv in (3, 4, 5, 6)] + [W.torus(1.0, 0.3, a, b) for a, b in W.C3_TORI]:
        r = 2.0 * W.mean_edge_length(m)
        out.append((m, r, W.packing_count(m, r)))
    return out


def _surfaces(case):
    """(mesh, particles, potential, integrator) of each surface of a case."""
    if case["kind"] == "batch":
        return [(m, n, dict(kind="harmonic", k=1.0, sigma=r, cutoff=r),
                 dict(kind="overdamped", dt=0.01 * r * r, mobility=1.0))
                for m, r, n in _batch_surfaces()[case["first"]:case["first"] + case["count"]]]
    m = _mesh(case["mesh"], case["size"])
    r = case.get("range", 0.0)
    pot, integ = None, None
    if case["kind"] == "fire":
        pot = dict(kind="coulomb", k=1.0, sigma=1.0, cutoff=math.inf)
        le = _edge(case["mesh"], case["size"])
        integ = dict(kind="fire", dt=0.1 * le, max_disp=0.5 * le)
    elif "potential" in case:
        s = r if case["potential"] == "harmonic" else r / 3.0
        pot = dict(kind=case["potential"], k=1.0, sigma=s, cutoff=r)
    if case["kind"] == "steps":
        integ = dict(overdamped=dict(kind="overdamped", dt=0.05 * r * r, mobility=1.0),
                     brownian=dict(kind="brownian", dt=0.4 * r * r, kT=0.1, friction=1.0, seed=3),
                     verlet=dict(kind="verlet", dt=0.005 * r))[case["integrator"]]
    return [(m, case["n"], pot, integ)]


def _inputs(case, seed):
    """Host arrays of each surface's positions, and of the walk's
    displacements and velocities."""
    out = []
    for k, (m, n, _, _) in enumerate(_surfaces(case)):
        face, bary = W.random_particles(m.nf, n, 1000 * (seed + 1) + k)
        disp = vel = None
        if case["kind"] == "walk":
            rng = np.random.default_rng(seed)
            disp = rng.normal(size=(n, 3)) * case["length"] / math.sqrt(2.0)
            vel = rng.normal(size=(n, 3))
        out.append((face, bary, disp, vel))
    return out


def _capacity(case):
    """Pairs that the buffers of a pairs case hold: every pair, or the
    expected number with room (random positions crowd here and there)."""
    n, r = case["n"], case["range"]
    if r == 0.0:
        return n * (n - 1)
    return int(n * (2.0 * n * math.pi * r * r / _area(case["mesh"], case["size"]) + 8))


def prepare(case, seed):
    kind = case["kind"]
    stream = torch.cuda.Stream()
    prec = case.get("precision", "fp64")
    ctx = gsim.Context(0, prec, stream=stream)
    st = dict(case=case, ctx=ctx, stream=stream, f32=prec != "fp64", surf=[])

    def dev(a):
        return None if a is None else torch.from_numpy(a).cuda()

    for (m, n, pot, integ), (face, bary, disp, vel) in zip(_surfaces(case), _inputs(case, seed)):
        mid = ctx.mesh_upload(m.V, m.T)
        s = dict(mid=mid, n=n, face=dev(face), bary=dev(bary), disp=dev(disp), vel=dev(vel),
                 out_face=torch.empty(n, dtype=torch.int32, device="cuda"),
                 out_bary=torch.empty(n, 3, dtype=F64, device="cuda"),
                 out_vel=torch.empty(n, 3, dtype=F64, device="cuda"))
        if pot:
            s["pot"] = gsim.potential(**pot)
        if integ:
            s["integ"] = gsim.integrator(**integ)
        if kind == "forces":
            s["force"], s["energy"] = torch.empty(n, 3, dtype=F64, device="cuda"), torch.empty(1, dtype=F64, device="cuda")
        if kind == "pairs":
            r = case["range"]
            cap = _capacity(case)
            s["pairs"] = dict(off=torch.zeros(n + 1, dtype=torch.int64, device="cuda"),
                              nbr=torch.zeros(cap, dtype=torch.int32, device="cuda"),
                              dist=torch.zeros(cap, dtype=F64, device="cuda"),
                              tan=torch.zeros(cap, 3, dtype=F64, device="cuda"),
                              flags=torch.zeros(cap, dtype=torch.uint8, device="cuda"))
        if kind == "voronoi":
            s["table"] = np.zeros(12 * n, np.int32)
        st["surf"].append(s)
    return st


def run(st):
    case, ctx, kind = st["case"], st["ctx"], st["case"]["kind"]
    for s in st["surf"]:
        ctx.particles_set_dev(s["mid"], s["face"], s["bary"], s["vel"])
    s = st["surf"][0]
    if kind == "forces":
        ctx.compute_forces_dev(s["mid"], s["pot"], s["force"], s["energy"])
        return dict(force=s["force"], energy=s["energy"])
    if kind == "pairs":
        p = s["pairs"]
        count = ctx.geodesic_pairs_dev(s["mid"], case["range"] or math.inf, **p)
        return dict(p, count=count)
    if kind == "voronoi":
        off, nbr = ctx.voronoi_neighbours(s["mid"])
        s["table"][:len(nbr)] = nbr
        return dict(off=off, nbr=s["table"])
    if kind == "walk":
        stats = ctx.displace_on_surface_dev(s["mid"], s["disp"])
        ctx.particles_get_dev(s["mid"], s["out_face"], s["out_bary"], s["out_vel"])
        return dict(face=s["out_face"], bary=s["out_bary"], vel=s["out_vel"], crossings=stats["crossings"])
    if kind == "batch":
        ctx.step_batched([s["mid"] for s in st["surf"]], [s["pot"] for s in st["surf"]],
                         [s["integ"] for s in st["surf"]], case["steps"])
    else:
        ctx.step(s["mid"], s["pot"], s["integ"], case.get("steps", 1))
    out = []
    with torch.cuda.stream(st["stream"]):
        for s in st["surf"]:
            ctx.particles_get_dev(s["mid"], s["out_face"], s["out_bary"], s["out_vel"])
            # the FP32-mixed mode computes with the accuracy of FP32, so its
            # program keeps the coordinates in that type
            b = s["out_bary"].float() if st["f32"] else s["out_bary"]
            o = dict(face=s["out_face"], bary=b)
            if kind != "batch":
                o["vel"] = s["out_vel"]
            out.append(o)
    return out if kind == "batch" else out[0]


def work(case):
    nbytes = flops = 0.0
    steps = case.get("steps", 1)
    for m, n, pot, integ in _surfaces(case):
        mesh = 24.0 * m.nv + 12.0 * m.nf
        state = 52.0 * n  # face, barycentrics, velocity
        r = case.get("range", 0.0) if case["kind"] != "batch" else pot["cutoff"]
        finite = case["kind"] not in ("fire", "voronoi", "walk") and r > 0.0
        area = W.surface_area(m)
        near = n * math.pi * r * r / area if finite else n - 1.0
        # windows of the exact method: about four a face within the range,
        # 0.17 nf^1.5 over a whole surface; 90 operations each
        windows = 4.0 * m.nf * min(1.0, math.pi * r * r / area) if finite else 0.17 * m.nf ** 1.5
        if case["kind"] == "voronoi":
            nbytes += mesh + state + 4.0 * 6 * n + 8.0 * n
            flops += 60.0 * 10 * m.nf
        elif case["kind"] == "walk":
            nbytes += 2 * state + 24.0 * n + 96.0 * n
            flops += 150.0 * n * (1.0 + case["length"] / _edge(case["mesh"], case["size"]))
        else:
            out = 37.0 * near * n + 8.0 * n if case["kind"] == "pairs" else 24.0 * n if case["kind"] == "forces" else state
            nbytes += steps * (min(mesh, 36.0 * windows * n) + state + out)
            flops += steps * n * (90.0 * windows + 20.0 * near)
    return dict(bytes=nbytes, flops=flops)


# ------------------------------------------------- the exact result in 64 bits
class _Surface:
    """Half-edge tables of a mesh in torch: half-edge h = 3f + k runs from
    vertex k of face f to vertex k + 1."""

    def __init__(self, m):
        V, T = np.asarray(m.V), np.asarray(m.T).astype(np.int64)
        nf, nv = m.nf, m.nv
        A, B, C = T.reshape(-1), np.roll(T, -1, 1).reshape(-1), np.roll(T, -2, 1).reshape(-1)
        key, back = A * nv + B, B * nv + A
        order = np.argsort(key)
        at = np.minimum(np.searchsorted(key[order], back), 3 * nf - 1)
        twin = np.where(key[order][at] == back, order[at], -1)
        e, w = V[B] - V[A], V[C] - V[A]
        L = np.linalg.norm(e, axis=1)
        cx = (w * e).sum(1) / L
        cy = np.linalg.norm(np.cross(e, w), axis=1) / L
        ang = np.arctan2(cy, cx)
        total = np.bincount(A, ang, nv)
        border = np.zeros(nv, bool)
        border[A[twin < 0]] = border[B[twin < 0]] = True
        normal = np.cross(V[T[:, 1]] - V[T[:, 0]], V[T[:, 2]] - V[T[:, 0]])
        normal /= np.linalg.norm(normal, axis=1, keepdims=True)
        ex = e[0::3] / L[0::3, None]

        def t(a):
            return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)

        self.nv, self.nf = nv, nf
        self.V, self.T, self.twin, self.tail, self.opp = t(V), t(T), t(twin), t(A), t(C)
        self.L, self.cx, self.cy = t(L), t(cx), t(cy)
        self.bend = t(border | (total >= 2 * np.pi - 1e-9))
        self.ex, self.normal = t(ex), t(normal)
        self.ey = torch.cross(self.normal, self.ex, dim=1)
        # the corners of every face in its own frame (vertex 0 at the origin, vertex 1 on the x axis)
        P = np.zeros((nf, 3, 2))
        P[:, 1, 0], P[:, 2, 0], P[:, 2, 1] = L[0::3], cx[0::3], cy[0::3]
        self.P = t(P)

    def lift(self, face, v2):
        """2D components in the faces' frames as 3D vectors."""
        return v2[:, :1] * self.ex[face] + v2[:, 1:] * self.ey[face]

    def flat(self, face, v3):
        return torch.stack([(v3 * self.ex[face]).sum(1), (v3 * self.ey[face]).sum(1)], 1)


def _cross(a, b):
    return a[:, 0] * b[:, 1] - a[:, 1] * b[:, 0]


def _unit(a):
    return a / a.norm(dim=1, keepdim=True)


def _expand(start, count):
    """Row index and position of every entry of ragged ranges."""
    row = torch.repeat_interleave(torch.arange(len(count), device=DEV), count)
    first = torch.cumsum(count, 0) - count
    return row, start[row] + (torch.arange(len(row), device=DEV) - first[row])


def _least(key, d, *more):
    """The entry of smallest d for each key, keys ascending."""
    o = torch.argsort(d)
    o = o[torch.argsort(key[o], stable=True)]
    k = key[o]
    first = torch.ones_like(k, dtype=torch.bool)
    first[1:] = k[1:] != k[:-1]
    o = o[first]
    return [x[o] for x in (key, d) + more]


def _links(S, cut, faces, root, he, a, b):
    """Every straight link shorter than `cut` from a root (at the origin of
    its plane) through entry half-edges `he` whose ends lie at a (left, seen
    from the root) and b: to particles, (root, particle, length, direction),
    and to bend vertices. faces: (particle order, first, count, bary)."""
    order, first, count, bary = faces
    rl, rr = _unit(a), _unit(b)
    to_p, to_v = [], []
    while len(root):
        f, k = he // 3, he % 3
        e = (b - a) / S.L[he][:, None]
        c = a + S.cx[he][:, None] * e + S.cy[he][:, None] * torch.stack([-e[:, 1], e[:, 0]], 1)
        w, at = _expand(first[f], count[f])
        if len(w):
            j = order[at]
            bj, kk = bary[j], k[w][:, None]
            q = (bj.gather(1, kk) * a[w] + bj.gather(1, (kk + 1) % 3) * b[w] + bj.gather(1, (kk + 2) % 3) * c[w])
            d = q.norm(dim=1)
            u = q / d[:, None]
            ok = (d < cut) & (_cross(rr[w], u) >= -1e-13) & (_cross(u, rl[w]) >= -1e-13)
            to_p.append((root[w][ok], j[ok], d[ok], u[ok]))
        d = c.norm(dim=1)
        u = c / d[:, None]
        sl, sr = _cross(u, rl), _cross(rr, u)
        ok = S.bend[S.opp[he]] & (d < cut) & (sl >= -1e-13) & (sr >= -1e-13)
        to_v.append((root[ok], S.opp[he][ok], d[ok], u[ok]))
        prev, nxt = he - k + (k + 2) % 3, he - k + (k + 1) % 3
        parts = []
        for tw, keep, ca, cb, cl, cr in (
                (S.twin[prev], sl > 0, a, c, rl, torch.where((sr > 0)[:, None], u, rr)),
                (S.twin[nxt], sr > 0, c, b, torch.where((sl > 0)[:, None], u, rl), rr)):
            # the part of the edge between the two rays, and its distance
            s = cb - ca
            keep = keep & (tw >= 0) & (_cross(cr, cl) > 1e-14)
            ends = []
            for ray in (cl, cr):
                den = _cross(s, ray)
                x = torch.where(den != 0, -_cross(ca, ray) / den, torch.zeros_like(den)).clamp(0, 1)
                ends.append(ca + x[:, None] * s)
            g = ends[1] - ends[0]
            x = (-(ends[0] * g).sum(1) / (g * g).sum(1).clamp_min(1e-300)).clamp(0, 1)
            keep &= (ends[0] + x[:, None] * g).norm(dim=1) < cut
            parts.append((root[keep], tw[keep], ca[keep], cb[keep], cl[keep], cr[keep]))
        root, he, a, b, rl, rr = (torch.cat(x) for x in zip(*parts))
    return [torch.cat(x) for x in zip(*to_p)] if to_p else None, [torch.cat(x) for x in zip(*to_v)]


def _pairs(S, face, bary, cut):
    """Exact geodesic pairs (i, j, d, tangent in i's face frame), sorted."""
    n = len(face)
    order = torch.argsort(face)
    count = torch.bincount(face, minlength=S.nf)
    faces = (order, torch.cumsum(count, 0) - count, count, bary)
    P = (bary[:, :, None] * S.P[face]).sum(1)
    chunk = 1 << 13
    pp, pv, vp, vv = [], [], [], []
    for i0 in range(0, n, chunk):  # from the particles
        i = torch.arange(i0, min(n, i0 + chunk), device=DEV)
        corner = S.P[face[i]] - P[i][:, None, :]
        w, at = _expand(faces[1][face[i]], count[face[i]])
        j = order[at]
        w, j = w[j != i[w]], j[j != i[w]]
        d = (P[j] - P[i[w]]).norm(dim=1)
        ok = d < cut
        pp.append((i[w][ok], j[ok], d[ok], ((P[j] - P[i[w]]) / d[:, None])[ok]))
        for k in range(3):
            v, d = S.T[face[i], k], corner[:, k].norm(dim=1)
            ok = S.bend[v] & (d < cut)
            pv.append((i[ok], v[ok], d[ok], (corner[:, k] / d[:, None])[ok]))
            tw = S.twin[3 * face[i] + k]
            ok = tw >= 0
            p, v = _links(S, cut, faces, i[ok], tw[ok], corner[ok, (k + 1) % 3], corner[ok, k])
            if p:
                pp.append(p)
            pv.append(v)
    fan = torch.nonzero(S.bend[S.tail])[:, 0]
    for h0 in range(0, len(fan), chunk):  # from the bend vertices, one fan edge at a time
        h = fan[h0:h0 + chunk]
        v, f, k = S.tail[h], h // 3, h % 3
        u1 = torch.stack([S.L[h], torch.zeros_like(S.L[h])], 1)
        u2 = torch.stack([S.cx[h], S.cy[h]], 1)
        w, at = _expand(faces[1][f], count[f])
        if len(w):
            j, kk = order[at], k[w][:, None]
            d = (bary[j].gather(1, (kk + 1) % 3) * u1[w] + bary[j].gather(1, (kk + 2) % 3) * u2[w]).norm(dim=1)
            ok = d < cut
            vp.append((v[w][ok], j[ok], d[ok]))
        for end, at2 in ((S.tail[h - k + (k + 1) % 3], u1), (S.opp[h], u2)):
            d = at2.norm(dim=1)
            ok = S.bend[end] & (d < cut)
            vv.append((v[ok], end[ok], d[ok]))
        tw = S.twin[h - k + (k + 1) % 3]
        ok = tw >= 0
        p, q = _links(S, cut, faces, v[ok], tw[ok], u2[ok], u1[ok])
        if p:
            vp.append(p[:3])
        vv.append(q[:3])
    none = (torch.zeros(0, dtype=torch.int64, device=DEV),) * 2 + (torch.zeros(0, dtype=F64, device=DEV),)
    pp = [torch.cat(x) for x in zip(*pp)]
    vp = [torch.cat(x) for x in zip(*(vp or [none]))]
    vv = [torch.cat(x) for x in zip(*(vv or [none]))]
    pv = [torch.cat(x) for x in zip(*pv)]

    def rows(v, w, d, nw):  # the shortest link of each (v, w), as rows by v
        key, d = _least(v * nw + w, d)
        v, w = key // nw, key % nw
        c = torch.bincount(v, minlength=S.nv)
        return w, d, torch.cumsum(c, 0) - c, c

    vv, vp = rows(*vv, S.nv), rows(*vp, n)
    best = [[] for _ in range(4)]
    chunk = 1 << 10
    for i0 in range(0, n, chunk):  # chains of links: source, vertices, target
        mine = (pv[0] >= i0) & (pv[0] < i0 + chunk)
        key, d, t = _least(pv[0][mine] * S.nv + pv[1][mine], pv[2][mine], pv[3][mine])
        fresh = torch.ones_like(key, dtype=torch.bool)
        while bool(fresh.any()):
            fk, fd, ft = key[fresh], d[fresh], t[fresh]
            w, at = _expand(vv[2][fk % S.nv], vv[3][fk % S.nv])
            nd = fd[w] + vv[1][at]
            ok = nd < cut
            nk = fk[w][ok] // S.nv * S.nv + vv[0][at][ok]
            old = torch.cat([torch.ones_like(key), torch.zeros_like(nk)])
            nkey, nd, t, old = _least(torch.cat([key, nk]), torch.cat([d, nd[ok]]), torch.cat([t, ft[w][ok]]), old)
            # a vertex goes on when its distance fell by more than rounding
            was = torch.full_like(nd, math.inf)
            was[torch.searchsorted(nkey, key)] = d
            fresh = (old == 0) & (nd < was * (1 - 1e-15))
            key, d = nkey, nd
        w, at = _expand(vp[2][key % S.nv], vp[3][key % S.nv])
        dd = d[w] + vp[1][at]
        ok = dd < cut
        i, j, dd, tt = (key // S.nv)[w][ok], vp[0][at][ok], dd[ok], t[w][ok]
        mine = (pp[0] >= i0) & (pp[0] < i0 + chunk)
        i, j, dd, tt = (torch.cat([x[mine], y]) for x, y in zip(pp, (i, j, dd, tt)))
        ok = i != j
        key, dd, tt = _least(i[ok] * n + j[ok], dd[ok], tt[ok])
        for x, y in zip(best, (key // n, key % n, dd, tt)):
            x.append(y)
    return [torch.cat(x) for x in best]


def _forces(S, face, bary, pot):
    i, _, d, t = _pairs(S, face, bary, pot["cutoff"])
    k, s = pot["k"], pot["sigma"]
    if pot["kind"] == "harmonic":
        x = (1.0 - d / s).clamp_min(0.0)
        U, dU = 0.5 * k * x * x, -(k / s) * x
    else:
        U = k * torch.exp(-d * d / (2.0 * s * s))
        dU = -(d / (s * s)) * U
    F = torch.zeros(len(face), 3, dtype=F64, device=DEV).index_add_(0, i, dU[:, None] * S.lift(face[i], t))
    return F, 0.5 * U.sum()


def _walk(S, face, bary, disp, vel):
    """Each particle straight across faces by `disp`, velocities carried
    along; reflected at boundary edges. Returns face, bary, vel, crossings."""
    face, bary = face.clone(), bary.clone()
    D, v = S.flat(face, disp), S.flat(face, vel)
    rem = D.norm(dim=1)
    u = D / rem.clamp_min(1e-300)[:, None]
    shut = torch.full_like(face, -1)
    live = torch.nonzero(rem > 0)[:, 0]
    crossings = 0
    while len(live):
        f, b = face[live], bary[live]
        P = S.P[f]
        E = P.roll(-2, 1) - P.roll(-1, 1)  # the edge opposite each corner
        area2 = P[:, 1, 0] * P[:, 2, 1]
        # a coordinate grows along the edge's inward normal
        rate = (E[:, :, 0] * u[live][:, None, 1] - E[:, :, 1] * u[live][:, None, 0]) / area2[:, None]
        s = torch.where(rate < 0, (-b / rate).clamp_min(0.0), torch.full_like(b, math.inf))
        s[torch.arange(len(live), device=DEV), shut[live].clamp_min(0)] = torch.where(
            shut[live] >= 0, torch.full_like(s[:, 0], math.inf),
            s.gather(1, shut[live].clamp_min(0)[:, None])[:, 0])
        s1, k1 = s.min(1)
        ends = rem[live] <= s1
        bary[live] = b + torch.where(ends, rem[live], s1)[:, None] * rate
        go = live[~ends]
        k1, s1, f = k1[~ends], s1[~ends], f[~ends]
        rem[go] -= s1
        row = torch.arange(len(go), device=DEV)
        e = _unit(E[~ends][row, k1])
        out = torch.stack([e[:, 1], -e[:, 0]], 1)
        tw = S.twin[3 * f + (k1 + 1) % 3]
        wall = tw < 0
        q, g = tw.clamp_min(0) % 3, tw.clamp_min(0) // 3
        ge = _unit(S.P[g][row, q] - S.P[g][row, (q + 1) % 3])  # the same edge in the next face
        gout = torch.stack([ge[:, 1], -ge[:, 0]], 1)
        for x in (u, v):
            along, across = (x[go] * e).sum(1, keepdim=True), (x[go] * out).sum(1, keepdim=True)
            x[go] = torch.where(wall[:, None], along * e - across * out, along * ge + across * gout)
        b = bary[go]
        b[row, k1] = 0.0
        nb = torch.zeros_like(b)
        nb[row, q] = b[row, (k1 + 2) % 3]
        nb[row, (q + 1) % 3] = b[row, (k1 + 1) % 3]
        bary[go] = torch.where(wall[:, None], b, nb)
        face[go] = torch.where(wall, f, g)
        shut[go] = torch.where(wall, k1, (q + 2) % 3)
        crossings += int((~wall).sum())
        live = go
    return face, bary, S.lift(face, v), crossings


def _noise(seed, step, n):
    """Two unit normals per particle: Philox4x32-10 (Salmon et al. 2011) with
    counter (particle, step, 0) and key seed, then Box-Muller."""
    M = np.uint64(0xFFFFFFFF)
    c = [np.arange(n, dtype=np.uint64), np.full(n, step & 0xFFFFFFFF, np.uint64), np.full(n, step >> 32, np.uint64),
         np.zeros(n, np.uint64)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & M, (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & M]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    c = [x.astype(np.int64) for x in c]
    u1, u2 = (((x >> 5) * 67108864 + (y >> 6)) / 9007199254740992.0 for x, y in ((c[0], c[1]), (c[2], c[3])))
    r = np.sqrt(-2.0 * np.log(1.0 - u1))
    return torch.from_numpy(np.stack([r * np.cos(2 * np.pi * u2), r * np.sin(2 * np.pi * u2)], 1)).to(DEV)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("fire", "voronoi", "batch") or (kind == "pairs" and case["range"] == 0.0):
        return None  # whole-mesh unfolding without trimming, or hundreds of passes, take too long; whole numbers
    (m, n, pot, integ), (face, bary, disp, vel) = _surfaces(case)[0], _inputs(case, seed)[0]
    S = _Surface(m)
    face, bary = torch.from_numpy(face).to(DEV).long(), torch.from_numpy(bary).to(DEV)
    if kind == "walk":
        f, b, v, _ = _walk(S, face, bary, torch.from_numpy(disp).to(DEV), torch.from_numpy(vel).to(DEV))
        return dict(face=None, bary=b, vel=v, crossings=None)
    if kind == "forces":
        F, E = _forces(S, face, bary, pot)
        return dict(force=F, energy=E.reshape(1))
    if kind == "pairs":
        i, j, d, t = _pairs(S, face, bary, case["range"])
        dist, tan = torch.zeros(_capacity(case), dtype=F64), torch.zeros(_capacity(case), 3, dtype=F64)
        dist[:len(d)], tan[:len(d)] = d, S.lift(face[i], t)
        return dict(off=None, nbr=None, dist=dist, tan=tan, flags=None, count=None)
    v = torch.zeros(n, 3, dtype=F64, device=DEV)
    for step in range(case["steps"]):
        F, _ = _forces(S, face, bary, pot)
        if integ["kind"] == "verlet":
            v = v + integ["dt"] * F
            D = integ["dt"] * v
        elif integ["kind"] == "overdamped":
            D = integ["mobility"] * integ["dt"] * F
        else:
            lam, dt = integ["friction"], integ["dt"]
            D = dt / lam * F + math.sqrt(2.0 * integ["kT"] * lam * dt) / lam * S.lift(face, _noise(integ["seed"], step, n))
        face, bary, v, _ = _walk(S, face, bary, D, v)
    return dict(face=None, bary=bary, vel=v)
