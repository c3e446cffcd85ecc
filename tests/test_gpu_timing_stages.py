"""Stage timings count a pairs call once: one pass, one compaction, in host and
device calls, with and without pairs."""
import math

import pytest

from paper_2404_19751_amd import gsim, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cutoff", [0.4, 1e-6, math.inf])
def test_one_stage_a_call(cutoff):
    torch = pytest.importorskip("torch")
    m = W.icosphere(3)
    n = 200
    f, b = W.random_particles(m.nf, n, 1)
    ctx = gsim.Context(0, "fp64")
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    P = len(ctx.geodesic_pairs(mid, cutoff)["nbr"])
    dev = dict(off=torch.zeros(n + 1, dtype=torch.int64, device="cuda"),
               nbr=torch.zeros(P + 1, dtype=torch.int32, device="cuda"),
               dist=torch.zeros(P + 1, dtype=torch.float64, device="cuda"),
               tan=torch.zeros(P + 1, 3, dtype=torch.float64, device="cuda"))
    torch.cuda.synchronize()
    for k in (1, 2, 3):
        ctx.timing(True)
        for _ in range(k):
            assert ctx.geodesic_pairs_dev(mid, cutoff, **dev) == P
        for stage in ("prefilter", "geodesic", "compact"):
            ms, launches = ctx.timing_get(stage)
            assert launches == k and 0.0 < ms < 1e4, stage
        ctx.timing(False)
    ctx.close()
