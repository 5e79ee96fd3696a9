"""Host logic of the on-line deformation (no GPU): which of its two forms smooths the fields of which images."""
import pytest

from paper_1102_0183_amd import binding


@pytest.mark.parametrize("maps,rows,cols,sigma", [(4, 27, 30, 1.3), (1, 36, 36, 0.8), (16, 29, 29, 6.0), (4, 31, 34, 2.0), (16, 34, 36, 0.6),
                                                  (1, 24, 64, 6.0), (1, 17, 17, 6.0)])
def test_narrow_gaussians_and_many_maps_keep_the_sums_over_a_line(maps, rows, cols, sigma):
    """Measured up to half as slow again on the matrix cores."""
    assert not binding.deform_on_matrix_cores(maps, rows, cols, sigma)


@pytest.mark.parametrize("maps,size", [(1, 29), (2, 48), (3, 32), (2, 96), (1, 16)])
def test_the_usual_maps_are_smoothed_on_the_matrix_cores(maps, size):
    assert binding.deform_on_matrix_cores(maps, size, size, 6.0)


@pytest.mark.parametrize("rows,cols", [(9311, 1), (1, 9311), (2, 4655), (4656, 2), (97, 95)])
def test_maps_whose_tiles_do_not_fit_in_lds_are_never_in_tiles(rows, cols):
    """Two planes of whole 16 x 16 tiles with a pitch of four floats more, beside the ring of affine maps."""
    up = lambda x: -(-x // 16) * 16
    for sigma in (0.3, 6.0, 16.0):
        if 2 * up(rows) * (up(cols) + 4) * 4 > 160 * 1024 - 768:
            assert not binding.deform_on_matrix_cores(1, rows, cols, sigma)
