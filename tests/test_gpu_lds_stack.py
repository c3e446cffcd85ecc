"""Every depth of the LDS window stack with few sources, where each workgroup's
LDS is padded up to its share of a compute unit's: the launch asks for no more
than there is, whatever the kernel itself holds. Against the enumeration oracle
with the tolerances of the other parity tests (FP64 1e-12, FP32-mixed 1e-5)."""
import numpy as np
import pytest

import oracle as orc
from paper_2404_19751_amd import gsim, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("kb", [4, 8, 16])
def test_padded_launches(kb, prec):
    m = W.icosphere(3)
    cutoff = 0.4
    pot, integ = gsim.potential("harmonic", 1.0, cutoff), gsim.integrator("overdamped", 1e-3)
    for n in (2, 200, 257, 600):
        f, b = W.random_particles(m.nf, n, n)
        ctx = gsim.Context(0, prec)
        ctx.tune(lds_stack_kb=kb)
        mid = ctx.mesh_upload(m.V, m.T)
        ctx.particles_set(mid, f, b)
        print(f"n={n} kb={kb} {prec}", flush=True)
        g = ctx.geodesic_pairs(mid, cutoff)
        o = orc.geodesic_pairs(orc.OracleMesh(m.V, m.T), f, b, cutoff)
        assert np.array_equal(g["off"], o.off) and np.array_equal(g["nbr"], o.nbr)
        assert len(o.dist) == 0 or np.max(np.abs(g["dist"] - o.dist) / o.dist) <= (1e-12 if prec == "fp64" else 1e-5)
        ctx.step(mid, pot, integ, 3)
        assert ctx.counters()["limited"] == 0
        ctx.close()


def test_autotuner_with_few_sources():
    m = W.icosphere(3)
    f, b = W.random_particles(m.nf, 100, 1)
    pot, integ = gsim.potential("harmonic", 1.0, 0.4), gsim.integrator("overdamped", 1e-3)
    for cutoff_kb in (4, 16):
        ctx = gsim.Context(0, "fp64")
        ctx.tune(lds_stack_kb=cutoff_kb)
        mid = ctx.mesh_upload(m.V, m.T)
        ctx.particles_set(mid, f, b)
        assert ctx.autotune([mid], [pot], [integ], reps=1)["best_ms"] > 0.0
        ctx.close()
