"""A call that finds no device memory says so, and the next one starts clean; a
near pass with little memory left makes do with fewer wavefronts (results equal
bit for bit: a source's do not depend on where it runs)."""
import numpy as np
import pytest

from paper_2404_19751_amd import gsim, workloads as W

pytestmark = pytest.mark.gpu


def test_the_call_after_one_without_room():
    torch = pytest.importorskip("torch")
    m = W.icosphere(5)
    f, b = W.random_particles(m.nf, 20000, 1)
    ctx = gsim.Context(0, "fp64")
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    free, _ = torch.cuda.mem_get_info()
    hold = torch.empty(max(free - (40 << 20), 0), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    with pytest.raises(gsim.GsimError) as e:
        ctx.geodesic_pairs(mid, 0.05)  # rows of 128 candidates: 95 MB
    assert e.value.status == gsim.E_OOM
    del hold
    torch.cuda.empty_cache()
    g = ctx.geodesic_pairs(mid, 0.05)
    ctx.close()
    ctx = gsim.Context(0, "fp64")
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    h = ctx.geodesic_pairs(mid, 0.05)
    assert all(np.array_equal(g[k], h[k]) for k in h)
    ctx.close()


def test_near_pass_beside_a_full_device():
    torch = pytest.importorskip("torch")
    m = W.torus(3.0, 1.0, 83, 28)
    f, b = W.random_particles(m.nf, 8192, 1)
    out = []
    for hold_gib in (None, 3.4):
        ctx = gsim.Context(0, "fp64")
        mid = ctx.mesh_upload(m.V, m.T)
        ctx.particles_set(mid, f, b)
        hold = None
        if hold_gib:
            free, _ = torch.cuda.mem_get_info()
            hold = torch.empty(max(free - int(hold_gib * 2 ** 30), 0), dtype=torch.uint8, device="cuda")
            torch.cuda.synchronize()
        out.append(ctx.geodesic_pairs(mid, 1.0))
        ctx.close()
        del hold
        torch.cuda.empty_cache()
    assert all(np.array_equal(out[0][k], out[1][k]) for k in out[0])
