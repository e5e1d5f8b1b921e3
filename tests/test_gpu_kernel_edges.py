"""Edges of the step kernels' work splits against the FP64 oracle: grids and
particle counts around the sizes at which a kernel changes how it divides its
work.  Tolerances as in test_gpu_parity.py: the split changes only the order of
FP64 sums."""
import picgen
import pytest

from test_gpu_parity import _compare, _run_pair

pytestmark = pytest.mark.gpu

FP64 = (1e-12, 1e-12, 1e-12)
FP32C = (1e-3, 1e-5, 1e-6)


@pytest.mark.parametrize("precision,tols", [("fp64", FP64), ("fp32c", FP32C)])
@pytest.mark.parametrize("nx,ny,ppc", [(16, 16, 1), (17, 16, 2), (33, 18, 3), (40, 24, 9), (64, 48, 20)])
def test_2d_step_shares_a_tile(nx, ny, ppc, precision, tols):
    """2D3V: a tile's particles shared by one workgroup or several, with fewer
    particles than threads, a partly filled last share and tiles of a few
    cells; hot, so that particles leave their tile between the sorts."""
    wl = picgen.WORKLOADS["2d3v_32x32_fp64"].scaled(nx=nx, ny=ny, ppc=ppc, w_th=(0.3,) * 3, omega_pe=0.1,
                                                    bext=(0.0, 0.0, 0.05))
    sim, st, _ = _run_pair(wl, precision, 24, sort_every=12)
    _compare(sim, st, wl, *tols)


@pytest.mark.parametrize("precision,tols", [("fp64", FP64), ("fp32c", FP32C)])
@pytest.mark.parametrize("nx,ny,ppc", [(368, 369, 2), (128, 128, 9), (48, 33, 60), (250, 200, 6)])
def test_2d_step_widths(nx, ny, ppc, precision, tols):
    """2D3V: one workgroup of 256 threads to a tile, and shares of 512 threads
    as many as, half as many as and more than half as many as those of 256."""
    wl = picgen.WORKLOADS["2d3v_32x32_fp64"].scaled(nx=nx, ny=ny, ppc=ppc, w_th=(0.3,) * 3, omega_pe=0.1,
                                                    bext=(0.0, 0.0, 0.05))
    sim, st, _ = _run_pair(wl, precision, 6, sort_every=4)
    _compare(sim, st, wl, *tols)


@pytest.mark.parametrize("precision,tols", [("fp64", FP64), ("fp32c", FP32C)])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_3d_crossings_along_one_axis(axis, precision, tols):
    """3D: nearly every particle crosses cells along one axis (0.32 cells per
    step), so that one section of the crossing pass holds nearly all of its
    blocks; tiles of very different fill (a slab of 10 of 20 cells)."""
    w_th = [0.02] * 3
    wl = picgen.WORKLOADS["3d_64cube_8ppc"].scaled(nx=20, ny=16, nz=16, ppc=7, w_th=tuple(w_th), slab=(3, 13))
    e = picgen.electrons(wl)
    e.w[axis] += 1.0
    import oracle
    from paper_1101_0809_amd import Sim
    sim = Sim(wl.nx, wl.ny, wl.nz, wl.dt, precision=precision, sort_every=4)
    sim.add_species(e.q, e.m, e.n)
    sim.load(0, e.x, e.w, e.weight)
    st = oracle.State(oracle.Grid(wl.nx, wl.ny, wl.nz, wl.dt), [oracle.Species(e.x, e.w, e.weight, q=e.q, m=e.m)])
    sim.step(10)
    st.step(10)
    _compare(sim, st, wl, *tols)


@pytest.mark.parametrize("precision,tols", [("fp64", FP64), ("fp32c", FP32C)])
@pytest.mark.parametrize("n,ppc", [((8, 8, 8), 1), ((9, 8, 16), 3), ((13, 14, 17), 3), ((24, 9, 8), 30), ((20, 14, 17), 60)])
def test_3d_step_shares_a_tile(n, ppc, precision, tols):
    """3D grids of few tiles, whose particles several workgroups share: shares
    of less than a wave's chunk, empty shares, and more than one chunk per
    wave; hot, so that particles cross cells and leave their tiles."""
    wl = picgen.WORKLOADS["3d_64cube_8ppc"].scaled(nx=n[0], ny=n[1], nz=n[2], ppc=ppc, w_th=(0.4,) * 3)
    sim, st, _ = _run_pair(wl, precision, 8, sort_every=4)
    _compare(sim, st, wl, *tols)


@pytest.mark.parametrize("precision,tols", [("fp64", FP64), ("fp32c", FP32C)])
@pytest.mark.parametrize("n,slab", [((64, 48, 56), (20, 44)), ((65, 41, 67), (0, 9)), ((64, 64, 40), None)])
def test_3d_more_tiles_than_workgroups(n, slab, precision, tols):
    """3D grids of more tiles than the chip has CUs, two species: with tiles
    without particles (also the ones that a workgroup begins with), with all
    particles in one XCD's share of the tiles or two, and filled evenly."""
    import oracle
    from paper_1101_0809_amd import Sim
    wl = picgen.WORKLOADS["3d_64cube_8ppc"].scaled(nx=n[0], ny=n[1], nz=n[2], ppc=1, w_th=(0.2,) * 3, slab=slab)
    e = picgen.electrons(wl)
    sim = Sim(*n, wl.dt, precision=precision, sort_every=3)
    parts = []
    for k, (q, m) in enumerate([(e.q, e.m), (-e.q, 2.0 * e.m)]):
        sim.add_species(q, m, e.n)
        x, w, weight = e.x.copy(), e.w * (1 - 2 * k), e.weight * (1 - 0.5 * k)
        sim.load(k, x, w, weight)
        parts.append(oracle.Species(x, w, weight, q=q, m=m))
    st = oracle.State(oracle.Grid(*n, wl.dt), parts)
    sim.step(5)
    st.step(5)
    _compare(sim, st, wl, *tols)


@pytest.mark.parametrize("precision", ["fp64", "fp32c"])
@pytest.mark.parametrize("n,count", [((16, 8, 8), 80_000), ((168, 168, 168), 300_000), ((9, 17, 8), 7),
                                     ((32, 16, 1), 80_000), ((1040, 1040, 1), 300_000), ((17, 16, 1), 5)])
def test_sort_moves_particles_whole(n, count, precision):
    """The sort with more particles in a tile than its histogram holds in
    registers, with more groups of tiles than a workgroup has threads, and with
    nearly no particles, from a fresh load and after the particles have moved:
    every particle keeps its values, tiles are in order, and the order inside a
    tile is that of test_sort_order (lane classes in as many home slots as the
    counts allow in 3D, rank levels in 2D)."""
    import numpy as np
    from paper_1101_0809_amd import Sim
    dims = 2 if n[2] == 1 else 3
    T = 16 if dims == 2 else 8
    rng = np.random.Generator(np.random.PCG64(23))
    x = rng.uniform(0, 1, (3, count)) * np.array(n, dtype=float)[:, None]
    w, weight = rng.normal(0, 0.4, (3, count)), rng.uniform(0.5, 1.5, count) * 1e-6
    sim = Sim(*n, 0.4, dims=dims, precision=precision, sort_every=0)
    sim.add_species(-1.0, 1.0, count)
    sim.load(0, x, w, weight)
    for moves in range(2):
        before = sim.particles(0)
        sim.sort()
        after = sim.particles(0)
        for a, b in zip(before, after):
            assert np.array_equal(a, b)
        xs, _, _, ids = sim.particles(0, raw=True)
        assert np.array_equal(np.sort(ids), np.arange(count))
        cell = np.floor(xs).astype(np.int64)
        if dims == 2:
            cell[2] = 0
        nt = [-(-k // T) for k in n]
        tile = ((cell[2] // T) * nt[1] + cell[1] // T) * nt[0] + cell[0] // T
        assert np.all(np.diff(tile) >= 0)
        l = cell % T
        for t in np.unique(tile)[:40]:
            sel = tile == t
            n_t, slot = int(sel.sum()), np.arange(int(sel.sum()))
            if dims == 3:
                C, row, plane, o = (16, 14, 168, 2) if precision == "fp64" else (32, 18, 216, 4)
                k = ((l[0] + o) + row * (l[1] + 2) + plane * (l[2] + 2))[sel] % C
                counts, rows = np.bincount(k, minlength=C), (n_t - np.arange(C) + C - 1) // C
                assert (k == slot % C).sum() == np.minimum(counts, rows).sum()
            else:
                local = (l[1] * T + l[0])[sel]
                level = np.concatenate([[0], np.cumsum(np.diff(local) <= 0)])
                counts = np.bincount(local, minlength=T * T)
                assert np.array_equal(np.bincount(level), [(counts > v).sum() for v in range(counts.max())])
        sim.step(2)


@pytest.mark.parametrize("precision,tols", [("fp64", FP64), ("fp32c", FP32C)])
@pytest.mark.parametrize("axis,ppc", [(0, 0.5), (1, 2), (2, 12)])
def test_3d_migrant_buckets(axis, ppc, precision, tols):
    """3D: a fast drift along one axis without a sort in between, so that a
    tile's bucket of migrants grows through the sizes at which they are taken
    from global memory, in order of arrival and in class rows, up to several
    chunks of rows."""
    import numpy as np
    import oracle
    from paper_1101_0809_amd import Sim
    wl = picgen.WORKLOADS["3d_64cube_8ppc"].scaled(nx=24, ny=25, nz=24, ppc=1, w_th=(0.05,) * 3)
    e = picgen.electrons(wl)
    rng = np.random.Generator(np.random.PCG64(31))
    count = int(e.n * ppc)
    x = rng.uniform(0, 1, (3, count)) * np.array([[wl.nx], [wl.ny], [wl.nz]], dtype=float)
    w = rng.normal(0, 0.05, (3, count))
    w[axis] += 3.0
    weight = np.full(count, float(e.weight[0]) / ppc)
    sim = Sim(wl.nx, wl.ny, wl.nz, wl.dt, precision=precision, sort_every=30)
    sim.add_species(e.q, e.m, count)
    sim.load(0, x, w, weight)
    st = oracle.State(oracle.Grid(wl.nx, wl.ny, wl.nz, wl.dt), [oracle.Species(x, w, weight, q=e.q, m=e.m)])
    sim.step(12)
    st.step(12)
    assert sim.migrant_fraction() > 0  # the mean over the steps: the first ones have none
    _compare(sim, st, wl, *tols)


@pytest.mark.parametrize("n,options", [
    ((13, 10, 11), dict()), ((9, 15, 14), dict(precision="fp32c")), ((13, 10, 11), dict(order=2)),
    ((13, 10, 11), dict(interp="conventional")), ((17, 31, 1), dict()), ((25, 19, 1), dict(precision="fp32c")),
    ((17, 25, 1), dict(order=2))])
def test_short_axes_stay_on_the_tiles(n, options):
    """On an axis shorter than two tiles every particle lies inside its tile's
    LDS region right after a sort: none takes the global-memory path (the
    2D3V conventional step reports no such count)."""
    from paper_1101_0809_amd import Sim
    dims = 2 if n[2] == 1 else 3
    wl = picgen.WORKLOADS["3d_64cube_8ppc"].scaled(nx=n[0], ny=n[1], nz=n[2], dims=dims, ppc=5, w_th=(0.02,) * 3)
    e = picgen.electrons(wl)
    sim = Sim(*n, 0.4, dims=dims, sort_every=1, **options)
    sim.add_species(e.q, e.m, e.n)
    sim.load(0, e.x, e.w, e.weight)
    sim.step(3)
    assert sim.fallback_fraction() == 0.0 and sim.migrant_fraction() == 0.0


@pytest.mark.parametrize("n", [(3, 5, 2), (64, 64, 64), (65, 64, 64), (67, 129, 96), (513, 512, 1)])
def test_poisson_cells_per_thread(n):
    """The conjugate-gradient kernels at one cell per thread or fewer, exactly
    one for every thread (64^3), one more, and several: against the FFT solve
    of the same charge density (the field bar of test_gpu_poisson.py)."""
    import numpy as np
    import oracle
    from oracle import poisson
    from paper_1101_0809_amd import Sim
    dims = 2 if n[2] == 1 else 3
    rng = np.random.Generator(np.random.PCG64(17))
    count = 4000
    x = rng.uniform(0, 1, (3, count)) * np.array(n, dtype=float)[:, None]
    w, weight = np.zeros((3, count)), np.full(count, 1e-3)
    sim = Sim(*n, 0.4, dims=dims)
    sim.add_species(-1.0, 1.0, count)
    sim.load(0, x, w, weight)
    it, res = sim.solve_poisson(neutralize=True)
    assert res <= 1e-13 and it > 0
    g = oracle.Grid(*n, 0.4)
    rho = oracle.State(g, [oracle.Species(x, w, weight, q=-1.0, m=1.0)]).rho()
    E = poisson.e_of_phi(g, poisson.solve(g, rho))
    assert np.linalg.norm(sim.fields_numpy()[:3] - E) <= 1e-9 * np.linalg.norm(E)


@pytest.mark.parametrize("scheme", ["order2", "conventional"])
@pytest.mark.parametrize("n,ppc,w_th,sort_every", [
    ((8, 8, 8), 9, 0.05, 3),      # one tile, more particles than one ordered chunk
    ((9, 8, 17), 1, 0.1, 2),      # shares of a few particles and none
    ((13, 14, 17), 6, 0.5, 0),    # unsorted and hot: off the fields' region and off the current's
    ((24, 8, 9), 20, 0.2, 4)])
def test_two_pass_steps_in_class_rows(scheme, n, ppc, w_th, sort_every):
    """The two-pass 3D steps (order 2 1/2, conventional): class rows over
    several chunks and shares of a tile, particles that stay, cross, and leave
    either LDS region."""
    import test_gpu_conventional
    import test_gpu_order2
    mod = test_gpu_order2 if scheme == "order2" else test_gpu_conventional
    wl = picgen.WORKLOADS["3d_64cube_8ppc"].scaled(nx=n[0], ny=n[1], nz=n[2], ppc=ppc, w_th=(w_th,) * 3,
                                                  sort_every=sort_every)
    sim, st = mod._run_pair(wl, 9)
    mod._compare(sim, st, wl)


@pytest.mark.parametrize("scheme", ["order2", "conventional"])
@pytest.mark.parametrize("n,ppc", [((16, 16, 16), 42), ((16, 16, 16), 48), ((20, 15, 16), 60)])
def test_two_pass_full_shares(scheme, n, ppc):
    """The two-pass steps with shares of a tile just below and above the size
    from which the current pass has four waves per SIMD, and unevenly filled
    tiles; hot."""
    import test_gpu_conventional
    import test_gpu_order2
    mod = test_gpu_order2 if scheme == "order2" else test_gpu_conventional
    wl = picgen.WORKLOADS["3d_64cube_8ppc"].scaled(nx=n[0], ny=n[1], nz=n[2], ppc=ppc, w_th=(0.3,) * 3, sort_every=3)
    sim, st = mod._run_pair(wl, 5)
    mod._compare(sim, st, wl)


@pytest.mark.parametrize("precision,tols", [("fp64", FP64), ("fp32c", FP32C)])
@pytest.mark.parametrize("nx,ny,ppc,w_th", [
    (16, 16, 12, 0.2),    # one tile of a few shares
    (48, 32, 40, 0.02),   # shares of several ordered chunks, cold
    (40, 35, 30, 0.8)])   # most particles cross; many leave their tile
def test_2d_step_in_class_rows(nx, ny, ppc, w_th, precision, tols):
    """2D3V in class rows: several chunks per share, particles that stay and
    that cross on one axis or both, and particles outside the margins."""
    wl = picgen.WORKLOADS["2d3v_32x32_fp64"].scaled(nx=nx, ny=ny, ppc=ppc, w_th=(w_th,) * 3, omega_pe=0.1,
                                                    drift=0.2, bext=(0.0, 0.0, 0.05))
    sim, st, _ = _run_pair(wl, precision, 12, sort_every=6)
    _compare(sim, st, wl, *tols)


def _poisson_case(n, seed):
    import numpy as np
    import oracle
    from oracle import poisson
    from paper_1101_0809_amd import Sim
    rng = np.random.Generator(np.random.PCG64(seed))
    count = 3000
    x = rng.uniform(0, 1, (3, count)) * np.array(n, dtype=float)[:, None]
    w, weight = np.zeros((3, count)), np.full(count, 1e-3)
    sim = Sim(*n, 0.4, dims=2 if n[2] == 1 else 3)
    sim.add_species(-1.0, 1.0, count)
    sim.load(0, x, w, weight)
    g = oracle.Grid(*n, 0.4)
    return sim, poisson.e_of_phi(g, poisson.solve(g, oracle.State(g, [oracle.Species(x, w, weight, q=-1.0, m=1.0)]).rho()))


@pytest.mark.parametrize("n", [(16, 8, 8), (41, 25, 1), (7, 5, 1), (64, 64, 65), (128, 64, 64), (128, 64, 65)])
def test_poisson_one_launch(n):
    """The solve in one launch with exactly one workgroup, one cell more, a
    partly filled one, two cells per thread, its largest grid, and the next one
    (in separate launches), as in test_poisson_cells_per_thread; solved twice."""
    import numpy as np
    sim, E = _poisson_case(n, 29)
    for _ in range(2):
        it, res = sim.solve_poisson(neutralize=True)
        assert res <= 1e-13 and it % 16 == 0
        assert np.linalg.norm(sim.fields_numpy()[:3] - E) <= 1e-9 * np.linalg.norm(E)


def test_poisson_from_two_threads():
    """Two threads on streams of their own: the second of two solves at a time
    takes separate launches."""
    import threading
    import numpy as np
    import torch
    cases = [_poisson_case((48, 48, 48), 31), _poisson_case((64, 64, 64), 37)]
    torch.cuda.synchronize()
    done = [0, 0]

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(4):
                _, res = cases[k][0].solve_poisson(neutralize=True)
                done[k] += res <= 1e-13

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert done == [4, 4]
    for sim, E in cases:
        assert np.linalg.norm(sim.fields_numpy()[:3] - E) <= 1e-9 * np.linalg.norm(E)


@pytest.mark.parametrize("box,n", [((16, 16, 1), 700), ((40, 24, 1), 5000), ((272, 272, 1), 3000),
                                   ((8, 8, 8), 600), ((24, 17, 9), 2500), ((64, 40, 56), 3000)])
def test_reverse_step_shares_a_tile(box, n):
    """One reverse step with a tile's particles shared by several workgroups
    (shares of less than a workgroup's threads, empty ones) and with a tile
    each: against the one-step reference, as test_step_vjp_matches_reference."""
    import numpy as np
    import torch
    from oracle import adjoint as ad
    from paper_1101_0809_amd import Sim
    dims = 2 if box[2] == 1 else 3
    dt = 0.5 if dims == 2 else 0.45
    shape = (box[2], box[1], box[0])
    x, w, weight = picgen.beams(box, n, 61, w_th=0.3, drift=0.2, dims=dims)
    rng = np.random.Generator(np.random.PCG64(67))
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
