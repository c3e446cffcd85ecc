"""Device calls whose output arrays a kernel must not write: ordinary host
memory, and device addresses that are not multiples of the element's size. The
results arrive as in aligned device memory, bit for bit."""
import math

import numpy as np
import pytest

from paper_2404_19751_amd import gsim, workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def host(dtype, *shape):
    return torch.zeros(*shape, dtype=dtype)


def odd(dtype, *shape):
    """A device array two bytes past an aligned address."""
    size = math.prod(shape) * torch.empty(0, dtype=dtype).element_size()
    raw = torch.zeros(size + 16, dtype=torch.uint8, device="cuda")

    class At:
        def __init__(self):
            self.shape = shape

        def data_ptr(self):
            return raw.data_ptr() + 2

        def cpu(self):
            return raw[2:2 + size].cpu().clone().view(dtype).reshape(shape)
    return At()


def device(dtype, *shape):
    return torch.zeros(*shape, dtype=dtype, device="cuda")


def results(make):
    m = W.icosphere(3)
    n, cutoff = 300, 0.5
    f, b = W.random_particles(m.nf, n, 1)
    ctx = gsim.Context(0, "fp64")
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    F, E = make(torch.float64, n, 3), make(torch.float64, 1)
    torch.cuda.synchronize()
    ctx.compute_forces_dev(mid, gsim.potential("harmonic", 1.0, cutoff), F, E)
    cap = 40 * n
    p = dict(off=device(torch.int64, n + 1), nbr=make(torch.int32, cap), dist=make(torch.float64, cap),
             tan=make(torch.float64, cap, 3), flags=make(torch.uint8, cap))
    torch.cuda.synchronize()
    P = ctx.geodesic_pairs_dev(mid, cutoff, **p)
    s = [make(torch.int32, n), make(torch.float64, n, 3), make(torch.float64, n, 3)]
    torch.cuda.synchronize()
    ctx.particles_get_dev(mid, *s)
    ctx.synchronize()
    torch.cuda.synchronize()
    ctx.close()
    return [F.cpu(), E.cpu(), p["off"].cpu()] + [p[k].cpu()[:P] for k in ("nbr", "dist", "tan", "flags")] + [x.cpu() for x in s]


@pytest.mark.parametrize("make", [host, odd])
def test_outputs_that_no_kernel_writes(make):
    for x, y in zip(results(make), results(device)):
        assert torch.equal(x, y)
