"""The sort of so many tiles that their groups are scanned before them."""
import pytest

import test_gpu_kernel_edges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32c"])
@pytest.mark.parametrize("n", [(2048, 2032, 1), (2048, 2048, 1), (2048, 8224, 1), (264, 256, 256)])
def test_sort_of_scanned_groups(n, precision):
    """Grids of 1016 groups of tiles (added up by the tiles), 1024 (scanned, one
    pass), 4112 (a full pass and a second) and, in 3D, 2112: as
    test_sort_moves_particles_whole."""
    if precision == "fp32c" and n[1] > 2048:
        n = (n[0], 2048, 1)  # FP32 mode's largest axes
    test_gpu_kernel_edges.test_sort_moves_particles_whole(n, 300_000, precision)


@pytest.mark.parametrize("precision", ["fp64", "fp32c"])
@pytest.mark.parametrize("count", [15, 8191, 8192, 8193, 24_600])
def test_sort_rounds_of_a_tile(count, precision):
    """One tile whose waves hold no particle or one, just under, exactly and just
    over one round of slots, and a few rounds."""
    test_gpu_kernel_edges.test_sort_moves_particles_whole((8, 8, 8), count, precision)
