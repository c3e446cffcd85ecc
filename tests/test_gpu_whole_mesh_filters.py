"""The whole-mesh kernel's window filters and stacks where they can go wrong:
surfaces whose windows split at saddle and boundary vertices (one angle, one
split), exact symmetries with tied paths, and particle counts around the
64-lane batches of targets and buffered windows. Distances and tangents are
held to the enumeration oracle with the FP64 tolerance of the other parity
tests (1e-12 relative: links of a few dozen unfoldings, each exact to
rounding)."""
import math

import numpy as np
import pytest

import oracle as orc
from paper_2404_19751_amd import gsim, workloads as W

from .test_gpu_parity import compare_pairs

pytestmark = pytest.mark.gpu

SURFACES = {
    "cone_saddle": lambda: W.cone_fan(2.5 * math.pi, 12),
    "cone_steep": lambda: W.cone_fan(3.2 * math.pi, 16),
    "l_shape": lambda: W.l_shape(3),
    "prism": lambda: W.prism(7, nz=3),
    "cube": lambda: W.cube(3),
    "torus": lambda: W.torus(3.0, 1.0, 18, 6),
    "bumpy": lambda: W.bumpy_sphere(2, 0.2),
}


@pytest.mark.parametrize("name", list(SURFACES))
@pytest.mark.parametrize("n", [2, 63, 65])
def test_filters_against_enumeration(name, n):
    m = SURFACES[name]()
    f, b = W.random_particles(m.nf, n, 31 + n)
    ctx = gsim.Context(0, "fp64")
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    g = ctx.geodesic_pairs(mid, math.inf)
    assert ctx.counters()["limited"] == 0
    o = orc.geodesic_pairs(orc.OracleMesh(m.V, m.T), f, b, math.inf)
    compare_pairs(g, o, W.mean_edge_length(m), label=name)
    ctx.close()


def test_symmetric_ties_keep_their_flags():
    """Opposite face centres of a cube: four tied paths of different
    directions, none of which a filter may drop."""
    m = W.cube(2)
    c = m.V[m.T].mean(1)
    lo, hi = np.argmin(np.abs(c - [0.5, 0.5, 0.0]).sum(1)), np.argmin(np.abs(c - [0.5, 0.5, 1.0]).sum(1))
    # the points of those faces nearest to the square's centre, moved along the diagonal by rounding-free steps
    f = np.array([lo, hi], np.int32)
    b = np.full((2, 3), 0.125)
    for k, (face, z) in enumerate(((lo, 0.0), (hi, 1.0))):
        v = np.argmin(np.abs(m.V[m.T[face]] - [0.5, 0.5, z]).sum(1))
        b[k, v] = 0.75
    ctx = gsim.Context(0, "fp64")
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    g = ctx.geodesic_pairs(mid, math.inf)
    o = orc.geodesic_pairs(orc.OracleMesh(m.V, m.T), f, b, math.inf)
    compare_pairs(g, o, W.mean_edge_length(m), label="cube ties")
    ctx.close()
