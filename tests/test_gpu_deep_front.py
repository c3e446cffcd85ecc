"""Cutoffs many edges wide with many targets: the windows that wait at once are a
whole front, far more than in depth-first passes. Compared with the whole-mesh
pass pruned at the same cutoff (neighbour sets equal, FP64 distances within
1e-12, FP32-mixed within 1e-5: the tolerances of the parity tests)."""
import math

import numpy as np
import pytest

from paper_2404_19751_amd import gsim, workloads as W

pytestmark = pytest.mark.gpu

SURFACES = {"height": lambda: W.height_field(100), "bumpy": lambda: W.bumpy_sphere(5, 0.2),
            "torus": lambda: W.torus(3.0, 1.0, 180, 60), "sphere": lambda: W.icosphere(6)}


@pytest.mark.parametrize("prec", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("name,n,share", [("height", 200, 0.55), ("bumpy", 150, 0.55), ("torus", 200, 0.3),
                                          ("sphere", 300, 0.52)])
def test_deep_fronts(name, n, share, prec):
    """share: of the surface's area in a flat disc of the cutoff."""
    m = SURFACES[name]()
    f, b = W.random_particles(m.nf, n, 2)
    cutoff = math.sqrt(share * W.surface_area(m) / math.pi)
    ctx = gsim.Context(0, prec)
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    g = ctx.geodesic_pairs(mid, cutoff)
    depth = ctx.counters()["max_stack_depth"]
    ctx.close()
    ctx = gsim.Context(0, "fp64")
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    ctx.tune(whole_mesh=1)
    h = ctx.geodesic_pairs(mid, cutoff)
    ctx.close()
    print(f"{name} {prec}: {len(g['nbr']) / n:.0f} targets a source, depth {depth}")
    assert np.array_equal(g["off"], h["off"]) and np.array_equal(g["nbr"], h["nbr"])
    assert np.abs(g["dist"] / h["dist"] - 1.0).max() <= (1e-12 if prec == "fp64" else 1e-5)
