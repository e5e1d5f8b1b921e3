"""Particles that leave their tile over its upper face between sorts, on axes
shorter than two tiles: they stay within the margin of the tile's LDS regions,
so none takes the global-memory path, and the step is that of particles
sorted in every step."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FP64, FP32C = (1e-12, 1e-12), (1e-4, 1e-5)
CASES = [  # dims, cells of the short axis, options, tolerances
    (3, 9, {}, FP64), (3, 13, {}, FP64), (3, 15, {}, FP64), (3, 12, {}, FP64), (3, 14, {}, FP64),
    (3, 11, dict(precision="fp32c"), FP32C), (3, 13, dict(precision="fp32c"), FP32C),
    (3, 13, dict(order=2), FP64), (3, 10, dict(order=2), FP64),
    (3, 13, dict(interp="conventional"), FP64), (3, 9, dict(interp="conventional"), FP64),
    (2, 17, {}, FP64), (2, 24, {}, FP64), (2, 30, {}, FP64), (2, 31, {}, FP64), (2, 24, dict(precision="fp32c"), FP32C),
    (2, 24, dict(order=2), FP64), (2, 24, dict(interp="conventional"), FP64)]


def _run(n, dims, x, w, weight, sort_every, steps, options):
    from paper_1101_0809_amd import Sim
    sim = Sim(*n, 0.4, dims=dims, sort_every=sort_every, **options)
    sim.add_species(-1.0, 1.0, weight.size)
    sim.load(0, x, w, weight)
    sim.step(steps)
    fractions = sim.fallback_fraction(), sim.migrant_fraction()
    F = sim.fields_numpy()
    return fractions, F, sim.particles(0)


@pytest.mark.parametrize("dims,length,options,tols,axis", [c + (axis,) for c in CASES for axis in range(c[0])])
@pytest.mark.parametrize("tile", ["first", "last"])
def test_upper_margin_of_a_short_axis(dims, length, options, tols, axis, tile):
    """A beam along the short axis from the last cell of the axis's first or last
    tile into the cells above it: one in 3D (where the field margin is one cell),
    two in 2D3V."""
    T, M = (8, 1) if dims == 3 else (16, 2)
    n = [10, 11, 12 if dims == 3 else 1]
    n[axis] = length
    rng = np.random.Generator(np.random.PCG64(83))
    rest, beam = 300, 100
    x = rng.uniform(0, 1, (3, rest + beam)) * np.array(n, dtype=float)[:, None]
    w = rng.normal(0, 0.01, (3, rest + beam))
    v = 0.75
    w[:, rest:] = 0.0
    w[axis, rest:] = v / np.sqrt(1.0 - v * v)  # 0.3 cells per step
    face = T if tile == "first" else length
    x[axis, rest:] = face - 0.35 + rng.uniform(0, 0.04, beam)
    # the last step starts in the margin's last cell (the path is the start cell's)
    steps = int((M + 0.3) / 0.3) + 1
    last = x[axis, rest:] + (steps - 1) * 0.3
    assert np.all(np.floor(last) == face - 1 + M)
    weight = np.full(rest + beam, 1e-5)
    (fallback, migrant), F, (px, pw, _, _) = _run(n, dims, x, w, weight, 0, steps, options)
    _, G, (qx, qw, _, _) = _run(n, dims, x, w, weight, 1, steps, options)
    assert np.linalg.norm(F - G) <= tols[0] * np.linalg.norm(G)
    for a in range(dims):
        d = px[a] - qx[a]
        assert np.max(np.abs(d - n[a] * np.round(d / n[a]))) <= tols[1] * n[a]
    assert np.max(np.abs(pw - qw)) <= tols[1] * np.max(np.abs(qw))
    if not (dims == 2 and options.get("interp")):  # which reports no such count
        assert fallback == 0.0 and migrant == 0.0
