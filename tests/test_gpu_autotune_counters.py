"""The counters of a call are that call's own: what the autotuner's update
launches counted (crossings, pairs, non-finite particles) does not show up in
the next call. Counts are whole numbers and compared exactly with those of a
context that was never tuned."""
import pytest

from paper_2404_19751_amd import gsim, workloads as W

pytestmark = pytest.mark.gpu


def test_counters_start_from_zero_after_the_autotuner():
    m = W.icosphere(3)
    f, b = W.random_particles(m.nf, 200, 1)
    # displacements of several edges, so that the scratch moves cross edges
    pot, integ = gsim.potential("harmonic", 1.0, 0.5), gsim.integrator("overdamped", 1.0)
    got = []
    for tuned in (False, True):
        ctx = gsim.Context(0, "fp64")
        mid = ctx.mesh_upload(m.V, m.T)
        ctx.particles_set(mid, f, b)
        if tuned:
            ctx.autotune([mid], [pot], [integ], reps=1)
        ctx.compute_forces(mid, pot)
        got.append({k: ctx.counters()[k] for k in ("nbr_pairs", "crossings", "nonfinite")})
        ctx.step(mid, pot, integ, 1)
        got[-1]["step"] = ctx.counters()["crossings"]
        ctx.close()
    assert got[0]["step"] > 0 and got[0]["crossings"] == 0
    assert got[1] == got[0]
