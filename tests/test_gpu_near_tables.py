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


@pytest.mark.parametrize("prec", ["fp64", "fp32_mixed"])
def test_layouts_in_turn(prec):
    """Meshes with and without bend vertices, particle counts and numbers of
    wavefronts in turn in one context; FP32-mixed results repeat bit for bit
    here too (every source runs alone)."""
    cases = [(W.torus(3.0, 1.0, 48, 16), 1200, 60.0), (W.icosphere(4), 900, 150.0), (W.bumpy_sphere(3, 0.2), 2500, 50.0),
             (W.torus(3.0, 1.0, 48, 16), 1500, 200.0), (W.icosphere(3), 300, 250.0)]
    ins = [(m, *dense(m, n, mean)) for m, n, mean in cases]
    want = [fresh(*x, prec) for x in ins]
    ctx = gsim.Context(0, prec)
    mids = [ctx.mesh_upload(x[0].V, x[0].T) for x in ins]
    for turn in range(3):
        for k in (0, 1, 2, 3, 4, 0, 2, 1):
            ctx.tune(max_slots=[65536, 64, 777][turn])
            m, f, b, cutoff = ins[k]
            ctx.particles_set(mids[k], f, b)
            ok = same(ctx.geodesic_pairs(mids[k], cutoff), want[k])
            assert all(ok.values()), (turn, k, ok)
    ctx.close()
