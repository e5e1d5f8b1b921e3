"""Particles that fill a few tiles of many: the kernels whose work split depends
on a tile's own count."""
import numpy as np
import pytest

import picgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("box,counts", [
    # particles in the whole box, and in a corner of one tile: a tile far above
    # the mean, one at about twice the mean, some of a few particles and none
    ((64, 48, 1), (300, 4000)), ((272, 272, 1), (2000, 1500)), ((24, 17, 9), (200, 3000)),
    ((48, 40, 40), (0, 2500)), ((40, 40, 48), (3000, 60)), ((16, 8, 8), (500, 1400))])
def test_reverse_step_of_clustered_particles(box, counts):
    """One reverse step with shares of a tile by its own count: against the
    one-step reference, as test_reverse_step_shares_a_tile."""
    import torch
    from oracle import adjoint as ad
    from paper_1101_0809_amd import Sim
    dims = 2 if box[2] == 1 else 3
    dt = 0.5 if dims == 2 else 0.45
    n = sum(counts)
    shape = (box[2], box[1], box[0])
    x, w, weight = picgen.beams(box, n, 71, w_th=0.3, drift=0.2, dims=dims)
    edge = 16.0 if dims == 2 else 8.0
    for a in range(dims):
        x[a, counts[0]:] *= edge / box[a]  # the rest into the first tile
    rng = np.random.Generator(np.random.PCG64(73))
    f = np.zeros((9,) + shape)
    f[:6] = rng.normal(0.0, 0.05, (6,) + shape)
    lam = [rng.normal(size=(3,) + shape), rng.normal(size=(3,) + shape), rng.normal(size=(3, n)), rng.normal(size=(3, n))]
    if dims == 2:
        lam[2][2] = 0.0
    bext = (0.03, -0.02, 0.05)
    ref = ad.step_vjp(ad.Grid(*box, dt), f[:3], f[3:6], x, w, weight, -1.0, 1.0, bext, *lam)
    sim = Sim(nx=box[0], ny=box[1], nz=box[2], dt=dt, dims=dims, bext=bext, fields=f)
    sim.add_species(-1.0, 1.0, capacity=n)
    sim.load(0, x, w, weight)
    sim.sort()
    dev = torch.device("cuda:0")
    lf = torch.tensor(np.concatenate([lam[0], lam[1]]).reshape(-1), device=dev)
    lx, lw = torch.tensor(lam[2], device=dev), torch.tensor(lam[3], device=dev)
    lb = torch.zeros(3, dtype=torch.float64, device=dev)
    sim.adjoint_step(lf, [lx], [lw], lb)
    got = lf.cpu().numpy().reshape((6,) + shape)
    for a, b in ((got[:3], ref[0]), (got[3:], ref[1]), (lx.cpu().numpy()[:dims], ref[2][:dims]),
                 (lw.cpu().numpy(), ref[3]), (lb.cpu().numpy(), ref[4])):
        assert np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b))


@pytest.mark.parametrize("box,counts", [
    ((13, 14, 15), (2000, 0)), ((8, 8, 8), (70, 0)), ((24, 20, 17), (300, 2500)), ((48, 40, 41), (4000, 3000)),
    ((17, 16, 1), (150, 0)), ((32, 32, 1), (400, 3000)), ((100, 70, 1), (5000, 900))])
def test_density_shares_at_order_2(box, counts):
    """The order-2 1/2 charge density of a sorted species, by shares of a tile,
    against that of the same species unsorted (every contribution its own global
    add), cell by cell: the Gauss drift between two diagnostics with a sort in
    between is their difference.  Two sums of n terms of one sign differ by 2 n
    roundings at most."""
    from paper_1101_0809_amd import Sim
    dims = 2 if box[2] == 1 else 3
    n = sum(counts)
    x, w, weight = picgen.beams(box, n, 79, w_th=0.3, drift=0.2, dims=dims)
    for a in range(dims):  # the rest into the first tile
        x[a, counts[0]:] *= (16.0 if dims == 2 else 8.0) / box[a]
    sim = Sim(*box, 0.4, dims=dims, order=2, sort_every=0)
    sim.add_species(-1.0, 1.0, n)
    sim.load(0, x, w, weight)
    before = sim.diagnostics()
    sim.sort()
    after = sim.diagnostics()
    bound = 2 * n * 2.0 ** -53
    assert after["gauss_abs"] <= bound * after["rho_mobile_max"]
    assert abs(after["charge"] - before["charge"]) <= bound * abs(before["charge"])
