"""Cutoff passes on both sides of the density from which near passes run (43
and 46 expected candidates a source): pairs against the oracle in both
precisions, and below it, where the rows are counted first, the fused update
against the separate one bit for bit (the timed stages tell which ran)."""
import math

import numpy as np
import pytest

import oracle as orc
from paper_2404_19751_amd import gsim, workloads as W

from .test_gpu_fp32 import compare32
from .test_gpu_parity import compare_pairs
from .util import oracle_band

pytestmark = pytest.mark.gpu


def system(n, mean):
    m = W.benchmark_torus()
    f, b = W.random_particles(m.nf, n, 9)
    r = math.sqrt(mean * W.surface_area(m) / (math.pi * n))
    assert (mean + 3.0 * math.sqrt(mean) > 64.0) == (mean > 44.0) and 3.0 * mean + 16.0 > 128.0
    return m, f, b, r


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("mean", [43.0, 46.0])
def test_pairs(mean, prec):
    m, f, b, r = system(1000, mean)
    o = orc.geodesic_pairs(orc.OracleMesh(m.V, m.T), f, b, r, **oracle_band(prec))
    ctx = gsim.Context(0, prec)
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    g = ctx.geodesic_pairs(mid, r)
    assert ctx.counters()["limited"] == 0
    if prec == "fp64":
        compare_pairs(g, o, W.mean_edge_length(m), label=str(mean))
    else:
        compare32(g, o, W.mean_edge_length(m), str(mean))
    ctx.close()


@pytest.mark.parametrize("mean,fused", [(43.0, True), (46.0, False)])
def test_fused_equals_separate(mean, fused):
    m, f, b, r = system(900, mean)
    pot, integ = gsim.potential("harmonic", 1.0, r), gsim.integrator("verlet", 0.01 * r)
    out = []
    for fuse in (1, 0):
        ctx = gsim.Context(0, "fp64")
        ctx.tune(fuse_update=fuse)
        mid = ctx.mesh_upload(m.V, m.T)
        ctx.particles_set(mid, f, b)
        ctx.timing(True)
        ctx.step(mid, pot, integ, 4)
        assert ctx.timing_get("commit")[1] == (1 if fuse and fused else 0)
        assert ctx.timing_get("update")[1] == (0 if fuse and fused else 4)
        out.append(ctx.particles_get(mid))
        ctx.close()
    assert all(np.array_equal(x, y) for x, y in zip(*out))
