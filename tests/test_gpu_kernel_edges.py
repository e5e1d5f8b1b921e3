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
