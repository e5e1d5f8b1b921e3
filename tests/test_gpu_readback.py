"""Sim.particles: id order whatever the ids, and arrays of their own."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sim(counts, precision="fp64"):
    from paper_1101_0809_amd import Sim
    rng = np.random.Generator(np.random.PCG64(41))
    sim = Sim(24, 20, 1, 0.4, dims=2, precision=precision, sort_every=0)
    sim.add_species(-1.0, 1.0, sum(counts))
    for n in counts:
        sim.load(0, rng.uniform(0, 20, (3, n)), rng.normal(0, 0.1, (3, n)), rng.uniform(0.5, 1.5, n))
    return sim


@pytest.mark.parametrize("precision", ["fp64", "fp32c"])
@pytest.mark.parametrize("keep", [1, 300, 500])
def test_particles_of_a_lowered_count(keep, precision):
    """A count set below the loaded one leaves ids of any size among the
    particles kept: they come in the order of their ids all the same."""
    sim = _sim((200, 300), precision)
    sim.sort()
    hs = sim.host_state()
    hs.n[0] = keep
    sim.set_host_state(hs)
    x, w, weight, ids = sim.particles(0, raw=True)
    order = np.argsort(ids)
    for a, b in zip(sim.particles(0), (x[:, order], w[:, order], weight[order], ids[order])):
        assert a.dtype == b.dtype and np.array_equal(a, b)
    if keep < 500:
        assert ids.max() >= keep


@pytest.mark.parametrize("raw", [False, True])
def test_particle_arrays_own_their_memory(raw):
    """Each array returned holds its own bytes and no others, so that keeping
    one does not keep the rest."""
    import torch
    for a in _sim((1000,)).particles(0, raw=raw):
        root = a
        while isinstance(root, np.ndarray) and root.base is not None:
            root = root.base
        held = root.untyped_storage().nbytes() if isinstance(root, torch.Tensor) else root.nbytes
        assert held == a.nbytes and a.flags.c_contiguous and a.flags.writeable


def test_particles_of_an_empty_species():
    """No particles: empty arrays of the usual shapes and types."""
    sim = _sim(())
    x, w, weight, ids = sim.particles(0)
    assert x.shape == w.shape == (3, 0) and weight.shape == ids.shape == (0,) and ids.dtype == np.int64
