"""Many lanes updating one table entry at once: particles crowded into few
faces, so that neighbouring windows meet the same targets, and fans of
launched bend vertices meeting in shared neighbours. 20 particles take the
grouped or single cutoff kernel, 100 nearly fill its target table, 300 need
the near pass; every count also runs as a whole-mesh pass. Against the
enumeration oracle with the FP64 tolerance of the other parity tests (1e-12
relative: links of a few unfoldings, each exact to rounding)."""
import numpy as np
import pytest

import oracle as orc
from paper_2404_19751_amd import gsim, workloads as W

from .test_gpu_parity import compare_pairs

pytestmark = pytest.mark.gpu


def crowd(m, n, seed):
    """n particles in the faces around vertex 0 (and a few elsewhere)."""
    faces = np.nonzero((m.T == m.T[0, 0]).any(1))[0]
    _, b = W.random_particles(m.nf, n, seed)
    u = W.uniforms(seed + 1, n)
    f = faces[np.minimum((u * len(faces)).astype(int), len(faces) - 1)].astype(np.int32)
    return f, b


@pytest.mark.parametrize("whole", [0, 1])
@pytest.mark.parametrize("n", [20, 100, 300])
@pytest.mark.parametrize("name", ["bumpy", "flat"])
def test_crowded_faces(name, n, whole):
    m = W.bumpy_sphere(2, 0.2) if name == "bumpy" else W.flat_grid(6, 6)
    f, b = crowd(m, n, 17 + n)
    cutoff = 1.5 * W.mean_edge_length(m)
    ctx = gsim.Context(0, "fp64")
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    ctx.tune(whole_mesh=whole)
    g = ctx.geodesic_pairs(mid, cutoff)
    assert ctx.counters()["limited"] == 0
    o = orc.geodesic_pairs(orc.OracleMesh(m.V, m.T), f, b, cutoff)
    compare_pairs(g, o, W.mean_edge_length(m), label=name)
    ctx.close()
