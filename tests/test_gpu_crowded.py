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
    mean = n * np.pi * cutoff ** 2 / W.surface_area(m)
    if not whole and n > 128 and 3.0 * mean + 16.0 <= 128:
        # sparse on the whole, so rows for 128 candidates are expected to do:
        # a source with more is reported, never cut short
        with pytest.raises(gsim.GsimError) as e:
            ctx.geodesic_pairs(mid, cutoff)
        assert e.value.status == gsim.E_LIMIT
        return
    g = ctx.geodesic_pairs(mid, cutoff)
    assert ctx.counters()["limited"] == 0
    o = orc.geodesic_pairs(orc.OracleMesh(m.V, m.T), f, b, cutoff)
    compare_pairs(g, o, W.mean_edge_length(m), label=name)
    ctx.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("n", [129, 300, 600])
def test_crowded_near_pass(n, prec):
    """A cutoff wide enough that rows are counted: the near pass, its sort in
    LDS (up to 512 keys) and in global memory, and its reset of what a source
    reached, on crowded and spread particles of one surface."""
    m = W.bumpy_sphere(2, 0.2)
    f, b = crowd(m, n, 5)
    f2, b2 = W.random_particles(m.nf, n, 6)
    f[::2], b[::2] = f2[::2], b2[::2]
    cutoff = 1.2
    assert 3.0 * n * np.pi * cutoff ** 2 / W.surface_area(m) + 16.0 > 128
    ctx = gsim.Context(0, prec)
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    g = ctx.geodesic_pairs(mid, cutoff)
    h = ctx.geodesic_pairs(mid, cutoff)
    assert np.array_equal(g["nbr"], h["nbr"]) and np.array_equal(g["off"], h["off"])
    o = orc.geodesic_pairs(orc.OracleMesh(m.V, m.T), f, b, cutoff)
    if prec == "fp64":
        compare_pairs(g, o, W.mean_edge_length(m), label="near")
    else:
        # the FP32-mixed contract: exact neighbour sets, distances within 1e-5
        assert np.array_equal(g["off"], o.off) and np.array_equal(g["nbr"], o.nbr)
        assert np.max(np.abs(g["dist"] - o.dist) / o.dist) <= 1e-5
    ctx.close()
