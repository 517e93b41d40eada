"""CPU tests of how bench.py reads the library's round log: which kernels a round is put down to, and what they move."""
from types import SimpleNamespace

import pytest

import bench


@pytest.mark.parametrize("staged,lanes,launch_rounds,name", [
    (1, 16, 0.0, "k_row_update<16, 16, true>"), (0, 32, 0.0, "k_row_update<16, 32, false>"), (2, 32, 0.0, "k_row_update_pull<16, 32>"),
    (2, 0, 0.0, "k_pk_round<16>"), (3, 16, 0.0, "k_pb_scatter + k_pb_gather"), (4, 16, 7.0, "k_rounds_persistent<16, 16>"),
    (1, 16, 5.0, "k_tail_rounds<16, 16>"), (2, 32, -1.0, "k_row_product<16, 32> + k_cg_step<16>"),
    (2, 0, -1.0, "k_pk_product<16> + k_cg_step<16>"), (3, 16, -1.0, "k_pb_scatter_product + k_pb_product + k_cg_step<16>")])
def test_a_round_is_put_down_to_the_kernels_that_ran_it(staged, lanes, launch_rounds, name):
    kind = bench.round_kind(SimpleNamespace(staged=staged, group_lanes=lanes, launch_rounds=launch_rounds))
    assert bench.round_kernel(*kind, 16) == name


def test_bytes_of_the_vector_step():
    """Five arrays of the size of the label matrix per iteration, the labels both ways in every second one, and the degrees."""
    assert bench.step_bytes(10, 3) == 10 * (3 * 4 * (5 + 2 * 0.5) + 4)
