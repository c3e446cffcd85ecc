"""Whole-mesh passes in which several wavefronts share a source, at the edges
of the rule that picks 8, 4, 2 or 1 of them (here by a limit on the resident
wavefronts, and once by the device's own), on surfaces with saddle and boundary
vertices, structured ties and sources on edges. Distances and tangents are held
to the enumeration oracle with the FP64 tolerance of the other parity tests
(1e-12 relative: links of a few dozen unfoldings, each exact to rounding), and
the two largest counts to the same passes with one wavefront a source."""
import math

import numpy as np
import pytest

import oracle as orc
from paper_2404_19751_amd import gsim, workloads as W

from .test_gpu_parity import compare_pairs

pytestmark = pytest.mark.gpu

SURFACES = {
    "cone_saddle": lambda: W.cone_fan(2.5 * math.pi, 12),
    "l_shape": lambda: W.l_shape(3),
    "cube": lambda: W.cube(3),
    "torus": lambda: W.torus(3.0, 1.0, 18, 6),
    "bumpy": lambda: W.bumpy_sphere(2, 0.2),
}


def particles(m, n, seed):
    """Random places, every fourth one moved onto an edge of its face."""
    f, b = W.random_particles(m.nf, n, seed)
    for k in range(0, n, 4):
        b[k, k % 3] = 0.0
        b[k] /= b[k].sum()
    return f, b


@pytest.mark.parametrize("name", list(SURFACES))
@pytest.mark.parametrize("n", [2, 8, 9, 16, 17, 32, 33])
def test_teams_against_enumeration(name, n):
    m = SURFACES[name]()
    f, b = particles(m, n, 7 + n)
    ctx = gsim.Context(0, "fp64")
    ctx.tune(max_slots=64)  # 8 wavefronts a source up to 8 sources, 4 up to 16, 2 up to 32
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    g = ctx.geodesic_pairs(mid, math.inf)
    assert ctx.counters()["limited"] == 0
    o = orc.geodesic_pairs(orc.OracleMesh(m.V, m.T), f, b, math.inf)
    compare_pairs(g, o, W.mean_edge_length(m), label=f"{name} {n}")
    ctx.close()


@pytest.mark.parametrize("n", [256, 257])
def test_teams_against_one_wavefront(n):
    m = W.torus(3.0, 1.0, 36, 12)
    f, b = particles(m, n, 3)
    ctx = gsim.Context(0, "fp64")
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    g = ctx.geodesic_pairs(mid, math.inf)
    ctx.tune(max_slots=n)
    h = ctx.geodesic_pairs(mid, math.inf)
    assert np.array_equal(g["nbr"], h["nbr"])
    assert np.array_equal(g["flags"], h["flags"])
    assert np.abs(g["dist"] / h["dist"] - 1.0).max() <= 1e-12
    one = h["flags"] == 0  # a tied pair may take any of its directions
    assert np.abs(g["tan"] - h["tan"])[one].max() <= 1e-12
    ctx.close()


def test_steps_repeat_bit_for_bit():
    """Time steps do not share sources: a run repeats exactly."""
    m = W.torus(3.0, 1.0, 18, 6)
    f, b = W.random_particles(m.nf, 40, 5)
    out = []
    for _ in range(2):
        ctx = gsim.Context(0, "fp64")
        mid = ctx.mesh_upload(m.V, m.T)
        ctx.particles_set(mid, f, b)
        ctx.step(mid, gsim.potential("coulomb", 1.0, 1.0, math.inf), gsim.integrator("overdamped", 1e-3), 5)
        out.append(ctx.particles_get(mid))
        ctx.close()
    for x, y in zip(out[0], out[1]):
        assert np.array_equal(x, y)
