"""Positions and cells by a launch of their own (a surface with more than 1024
particles) and inside the binning workgroup (all others), at the edges of that
rule, alone and beside a small surface in a batch. Pairs are held to the
enumeration oracle with the FP64 tolerance of the other parity tests (1e-12
relative); the batch to the same surfaces stepped alone, bit for bit (each
particle's step depends on its own row only)."""
import numpy as np
import pytest

import oracle as orc
from paper_2404_19751_amd import gsim, workloads as W

from .test_gpu_parity import compare_pairs

pytestmark = pytest.mark.gpu

SIZES = [1, 1023, 1024, 1025, 2049]


@pytest.mark.parametrize("n", SIZES)
def test_pairs_at_the_edges(n):
    m = W.bumpy_sphere(3, 0.2)
    f, b = W.random_particles(m.nf, n, 60 + n)
    ctx = gsim.Context(0, "fp64")
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    g = ctx.geodesic_pairs(mid, 0.15)
    compare_pairs(g, orc.geodesic_pairs(orc.OracleMesh(m.V, m.T), f, b, 0.15), W.mean_edge_length(m), label=str(n))
    ctx.close()


@pytest.mark.parametrize("n", SIZES)
def test_batch_equals_alone(n):
    ms = [W.bumpy_sphere(3, 0.2), W.icosphere(2)]
    ns = [n, 40]
    pot, ig = gsim.potential("harmonic", 1.0, 0.15, 0.15), gsim.integrator("overdamped", 0.01)

    def run(groups):
        ctx = gsim.Context(0, "fp64")
        ids = []
        for m, k in zip(ms, ns):
            ids.append(ctx.mesh_upload(m.V, m.T))
            ctx.particles_set(ids[-1], *W.random_particles(m.nf, k, 9 + k))
        for g in groups:
            ctx.step_batched([ids[i] for i in g], [pot] * len(g), [ig] * len(g), 3)
        out = [ctx.particles_get(i) for i in ids]
        ctx.close()
        return out

    for x, y in zip(run([[0, 1]]), run([[0], [1]])):
        for u, v in zip(x, y):
            assert np.array_equal(u, v)
