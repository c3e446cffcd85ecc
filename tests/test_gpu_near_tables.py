"""The tables that near passes keep from call to call: after a call that found
no room for larger ones, after calls of other layouts (meshes and particle
counts in turn), every array of a call equals a fresh context's bit for bit."""
import math

import numpy as np
import pytest

from paper_2404_19751_amd import gsim, workloads as W

pytestmark = pytest.mark.gpu


def dense(m, n, mean):
    f, b = W.random_particles(m.nf, n, n)
    return f, b, math.sqrt(mean * W.surface_area(m) / (math.pi * n))


def fresh(m, f, b, cutoff, prec="fp64"):
    ctx = gsim.Context(0, prec)
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    g = ctx.geodesic_pairs(mid, cutoff)
    ctx.close()
    return g


def same(g, h):
    return {k: bool(np.array_equal(g[k], h[k])) for k in g}


def test_after_a_call_without_room():
    torch = pytest.importorskip("torch")
    m = W.torus(3.0, 1.0, 83, 28)
    f, b, cutoff = dense(m, 4096, 60.0)
    f2, b2, cutoff2 = dense(m, 24576, 60.0)
    want = fresh(m, f, b, cutoff)
    ctx = gsim.Context(0, "fp64")
    mid = ctx.mesh_upload(m.V, m.T)
    big = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    ctx.particles_set(big, f2, b2)
    assert all(same(ctx.geodesic_pairs(mid, cutoff), want).values())
    # room for the larger call's rows, but not for its near tables
    free, _ = torch.cuda.mem_get_info()
    hold = torch.empty(max(free - (700 << 20), 0), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    try:
        ctx.geodesic_pairs(big, cutoff2)
    except gsim.GsimError as e:
        assert e.status in (gsim.E_OOM, gsim.E_LIMIT)
    del hold
    torch.cuda.empty_cache()
    for _ in range(2):
        ok = same(ctx.geodesic_pairs(mid, cutoff), want)
        assert all(ok.values()), ok
    ctx.close()
