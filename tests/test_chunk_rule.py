"""The derived split of the marches on grids whose cells are deep along the march, seen through the
workspace it asks for (host side only): chunks of about 16 planes where longer ones would leave the
chip idle, and no short chunks where a node row would then lie in dozens of them."""
import pytest

from paper_1804_10541_amd import mfr
from synth import GridSpec


def _size(m, my, chunk=0):
    old = mfr.get_tile_config()
    try:
        mfr.set_tile_config(32, 16, chunk, 0)
        return mfr.workspace_size(GridSpec(m=m, h=(1.0, 1.0, 1.0), my=my, tau=0.1, rho=0.1, alpha=1.0))
    finally:
        mfr.set_tile_config(**old)


@pytest.mark.parametrize("m,my", [((128, 128, 96), (65, 65, 2)), ((128, 128, 96), (65, 65, 3)),
                                  ((64, 64, 64), (5, 5, 3)), ((300, 300, 1), (5, 5, 1))])
def test_deep_cells_take_chunks_of_about_16(m, my):
    assert _size(m, my, 24) < _size(m, my) <= _size(m, my, 16)   # (longer chunks, fewer partials)


# bytes asked for when chunks had 16 rows or more
@pytest.mark.parametrize("m,my,before", [((1477, 140, 1), (1322, 3, 1), 2010000), ((357, 565, 1), (287, 6, 1), 2120000)])
def test_wide_plane_cells_keep_few_partial_slots(m, my, before):
    assert _size(m, my) <= before
