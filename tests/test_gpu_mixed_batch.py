"""A batch of sparse and dense surfaces: each kind goes its own way, so that
every surface's steps equal, bit for bit, those it takes alone (whatever the
order, the integrators, and with or without graphs), and the results of the
batch's calls come back to the surfaces in the caller's order."""
import math

import numpy as np
import pytest

from paper_2404_19751_amd import gsim, workloads as W

pytestmark = pytest.mark.gpu


def surfaces():
    """(mesh, particles, mean candidates, integrator)"""
    return [(W.icosphere(4), 700, 8.0, "overdamped"), (W.torus(3.0, 1.0, 48, 16), 900, 150.0, "verlet"),
            (W.bumpy_sphere(3, 0.2), 400, 12.0, "brownian"), (W.icosphere(3), 600, 60.0, "overdamped"),
            (W.torus(3.0, 1.0, 40, 12), 1500, 20.0, "fire"), (W.flat_grid(20, 20), 800, 90.0, "verlet")]


def parts(which):
    out = []
    for k in which:
        m, n, mean, kind = surfaces()[k]
        f, b = W.random_particles(m.nf, n, 10 + k)
        r = math.sqrt(mean * W.surface_area(m) / (math.pi * n))
        dt = dict(overdamped=0.01 * r * r, brownian=0.01 * r * r, verlet=0.01 * r, fire=0.01 * r)[kind]
        out.append((m, f, b, gsim.potential("harmonic", 1.0, r), gsim.integrator(kind, dt=dt, kT=0.1, seed=k, max_disp=0.1 * r)))
    return out


@pytest.mark.parametrize("prec", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("which", [(0, 1), (1, 0, 3, 2), (0, 1, 2, 3, 4, 5), (5, 4, 3, 2, 1, 0)])
def test_batch_equals_each_surface_alone(which, prec):
    P = parts(which)
    steps = 5
    alone = []
    for m, f, b, pot, integ in P:
        ctx = gsim.Context(0, prec)
        mid = ctx.mesh_upload(m.V, m.T)
        ctx.particles_set(mid, f, b)
        ctx.step(mid, pot, integ, steps)
        alone.append(ctx.particles_get(mid))
        ctx.close()
    for graphs in (50, 0):
        ctx = gsim.Context(0, prec)
        ctx.tune(graph_steps=graphs)
        mids = [ctx.mesh_upload(p[0].V, p[0].T) for p in P]
        for mid, p in zip(mids, P):
            ctx.particles_set(mid, p[1], p[2])
        ctx.step_batched(mids, [p[3] for p in P], [p[4] for p in P], steps)
        c = ctx.counters()
        assert c["limited"] == 0 and c["cum_passes"] == steps
        for k, mid in enumerate(mids):
            same = [bool(np.array_equal(x, y)) for x, y in zip(ctx.particles_get(mid), alone[k])]
            if prec == "fp64":
                assert all(same), (which[k], graphs, same)
            else:
                # grouping, and with it the sums, follows the batch's size
                assert np.abs(ctx.particles_get(mid)[3] - alone[k][3]).max() <= 1e-6
        ctx.close()
