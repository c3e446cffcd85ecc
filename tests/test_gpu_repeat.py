"""Calls repeat bit for bit: pairs without a cutoff of few sources (several
wavefronts share each), pairs of many targets within a cutoff, and time steps
over them, on surfaces whose symmetry makes paths of equal length meet at many
targets (several in one face). Twelve calls each; every array of each equals
the first call's exactly."""
import math

import numpy as np
import pytest

from paper_2404_19751_amd import gsim, workloads as W

pytestmark = pytest.mark.gpu

LATTICE = np.array([[1, 1, 1], [2, 1, 1], [1, 2, 1], [1, 1, 2], [2, 2, 1], [1, 2, 2]], float)


def lattice(m, per_face, seed=3):
    """per_face particles at the same few places of every face, in random order."""
    f = np.repeat(np.arange(m.nf), per_face)
    b = np.tile(LATTICE[:per_face] / LATTICE[:per_face].sum(1, keepdims=True), (m.nf, 1))
    o = np.random.default_rng(seed).permutation(len(f))
    return f[o].astype(np.int32), b[o]


def repeats(m, f, b, cutoff, calls=12, **tune) -> dict:
    ctx = gsim.Context(0, "fp64")
    ctx.tune(**tune)
    mid = ctx.mesh_upload(m.V, m.T)
    ctx.particles_set(mid, f, b)
    first = ctx.geodesic_pairs(mid, cutoff)
    bad = {}
    for _ in range(calls - 1):
        g = ctx.geodesic_pairs(mid, cutoff)
        for k in first:
            if not np.array_equal(first[k], g[k]):
                bad[k] = bad.get(k, 0) + 1
    ctx.close()
    return bad


@pytest.mark.parametrize("name", ["cube", "torus", "bumpy"])
def test_pairs_of_few_sources(name):
    m = {"cube": lambda: W.cube(4), "torus": lambda: W.torus(3.0, 1.0, 36, 12),
         "bumpy": lambda: W.bumpy_sphere(3, 0.2)}[name]()
    if name == "cube":
        f, b = lattice(m, 1)
    else:
        f, b = W.random_particles(m.nf, 100, 4)
    bad = repeats(m, f[:200], b[:200], math.inf)
    assert not bad


@pytest.mark.parametrize("name", ["flat", "torus", "cube", "bumpy"])
def test_pairs_of_many_targets(name):
    m = {"flat": lambda: W.flat_grid(24, 24), "torus": lambda: W.torus(3.0, 1.0, 48, 16), "cube": lambda: W.cube(8),
         "bumpy": lambda: W.bumpy_sphere(3, 0.2)}[name]()
    f, b = lattice(m, 6)
    cutoff = math.sqrt(150.0 * W.surface_area(m) / (math.pi * len(f)))
    bad = repeats(m, f, b, cutoff)
    assert not bad


def test_steps_of_many_targets():
    """Two runs of the same time steps, as a resumed run promises."""
    m = W.cube(8)
    f, b = lattice(m, 6)
    r = math.sqrt(150.0 * W.surface_area(m) / (math.pi * len(f)))
    out = []
    for _ in range(3):
        ctx = gsim.Context(0, "fp64")
        mid = ctx.mesh_upload(m.V, m.T)
        ctx.particles_set(mid, f, b)
        ctx.step(mid, gsim.potential("harmonic", 1.0, r), gsim.integrator("overdamped", 1e-3 * r * r), 4)
        out.append(ctx.particles_get(mid))
        ctx.close()
    for k in range(1, 3):
        same = [bool(np.array_equal(x, y)) for x, y in zip(out[0], out[k])]
        assert all(same)
