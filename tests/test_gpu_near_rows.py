"""Near passes: rows at the edges of their sort (512 keys in LDS, more in global
memory, up to a few thousand), and tables whose epochs run out after a few
sources, in which case they are cleared and start over."""
import math

import numpy as np
import pytest

import oracle as orc
from paper_2404_19751_amd import gsim, workloads as W

from .test_gpu_parity import compare_pairs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("n", [510, 511, 512, 513, 514, 1025, 2100])
def test_long_rows(n, prec):
    """Every other particle of a small patch is a target."""
    m = W.bumpy_sphere(2, 0.2)
    faces = np.nonzero((m.T == m.T[0, 0]).any(1))[0]
    _, b = W.random_particles(m.nf, n, 5)
    f = faces[np.minimum((W.uniforms(6, n) * len(faces)).astype(int), len(faces) - 1)].astype(np.int32)
    cutoff = 0.9
    assert 3.0 * n * math.pi * cutoff ** 2 / W.surface_area(m) + 16.0 > 128
    ctx = gsim.Context(0, prec)
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    g = ctx.geodesic_pairs(mid, cutoff)
    o = orc.geodesic_pairs(orc.OracleMesh(m.V, m.T), f, b, cutoff)
    assert np.diff(o.off).max() == n - 1
    if prec == "fp64":
        compare_pairs(g, o, W.mean_edge_length(m), label=str(n))
    else:
        # the FP32-mixed contract: exact neighbour sets, distances within 1e-5
        assert np.array_equal(g["off"], o.off) and np.array_equal(g["nbr"], o.nbr)
        some = o.dist > 1e-3 * W.mean_edge_length(m)
        assert np.max(np.abs(g["dist"] - o.dist)[some] / o.dist[some]) <= 1e-5
    ctx.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("epochs", [1, 2, 3, 50])
def test_epochs_run_out(epochs, prec):
    m = W.torus(3.0, 1.0, 36, 12)
    n = 700
    f, b = W.random_particles(m.nf, n, 3)
    cutoff = math.sqrt(90.0 * W.surface_area(m) / (math.pi * n))
    out = []
    for e in (None, epochs):
        ctx = gsim.Context(0, prec)
        ctx.tune(max_slots=16)
        if e:
            ctx.tune(near_epochs=e)
        mid = ctx.mesh_upload(m.V, m.T)
        ctx.particles_set(mid, f, b)
        for _ in range(2):
            out.append(ctx.geodesic_pairs(mid, cutoff))
        ctx.close()
    for g in out[1:]:
        assert all(np.array_equal(g[k], out[0][k]) for k in g)
