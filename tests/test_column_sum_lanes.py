"""Sums over the rows beside a row reduce: how the lanes of a wavefront that hold the same columns meet, for every number of
lanes a row, and the schedules with two slots a lane in place of three."""
import pytest

from tests.test_row_col_sums import layernorm_backward_graph, test_layernorm_backward_single_pattern_matches_oracle as matches_oracle

DIMS = [[37, 7], [1100, 8], [1, 16], [1100, 31], [37, 64], [1100, 65], [3000, 130], [1, 250], [1100, 300], [37, 520], [1100, 700],
        [4097, 150], [300, 5465], [1000, 6143]]


def test_two_slots_in_place_of_three():
    from paper_2103_05288_amd import Context
    ctx = Context(-1)
    h = ctx.register(layernorm_backward_graph())
    for dims, lanes, slots in (([2048, 140], 16, 2), ([4096, 140], 16, 2), ([4097, 140], 8, 3), ([2048, 380], 32, 2), ([2049, 380], 16, 3), ([1024, 700], 32, 3),
                               ([300, 1400], 64, 3), ([300, 5464], 512, 2), ([300, 5456], 256, 3), ([9000, 6144], 512, 2)):
        p = h.plan(dims)
        assert (p["lanes_per_row"], p["slots_per_lane"]) == (lanes, slots), dims
    ctx.close()


def test_the_workspace_of_the_most_rows_serves_fewer():
    """Up to the row of partial sums by which grids are made odd, where it was so before those schedules."""
    from paper_2103_05288_amd import Context
    ctx = Context(-1)
    h = ctx.register(layernorm_backward_graph())
    for H in (130, 300, 700, 5500, 6140):
        most = 0
        for k in range(8 * 16):
            need = h.plan([int(2 ** (k / 8)), H])["workspace_bytes"]
            assert need >= most - (2 * 4 * H if H < 5464 else 0), (k, H)
            most = max(most, need)
    ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("dims", DIMS, ids=lambda d: f"{d[0]}x{d[1]}")
def test_results(dims):
    matches_oracle(dims)
