"""Which sketches are updated cell by cell along lists of each cell's coordinates: not those whose cells have so many
coordinates, or that have so many cells, that the other forms take less time.  Host only."""
import pytest

import paper_1903_04488_amd as cs

# (r, c, d, W): W = 0 is one vector into one table
SLOWER = [  # few columns: a cell's lanes are a serial chain
    (3, 64, 10**6, 1), (5, 33, 10**6, 1), (3, 32, 4 * 10**6, 1), (1, 1, 4 * 10**6, 1), (3, 3, 20_000, 4), (3, 63, 400_000, 4),
    (15, 16, 400_000, 1), (3, 100, 10**6, 1), (5, 128, 600_000, 1), (3, 256, 10**6, 1),
    # wide tables: cells without a coordinate
    (3, 1 << 20, 1000, 1), (3, 1 << 20, 30_000, 4), (3, 200_001, 60_001, 32), (3, 500_001, 150_001, 1),
    (3, 1 << 27, 1000, 25), (1, 1 << 31, 1, 1), (5, 1 << 16, 131_073, 0), (3, 1_000_001, 1000, 0)]
FASTER = [(7, 40, 784, 4), (3, 3, 2000, 32), (3, 63, 100_000, 4), (15, 33, 100_000, 32), (15, 16, 20_000, 1), (3, 64, 400_000, 1),
          (3, 256, 400_000, 1), (3, 70_001, 140_003, 4), (3, 1 << 16, 30_000, 32), (5, 20_001, 100_006, 4),
          (3, 63, 4 * 10**6, 0), (3, 16, 400_000, 0), (5, 1 << 14, 81_921, 0), (3, 200_001, 400_003, 0)]


@pytest.mark.parametrize("r, c, d, W", SLOWER)
def test_none_where_the_other_forms_take_less_time(r, c, d, W):
    assert cs.cs_cell_lists_bytes(cs.cs_params_init(r, c, 190304488, d), W, d) == 0


@pytest.mark.parametrize("r, c, d, W", FASTER)
def test_lists_where_they_take_less_time(r, c, d, W):
    assert cs.cs_cell_lists_bytes(cs.cs_params_init(r, c, 190304488, d), W, d) == 4 * r * (c + 1 + d)
