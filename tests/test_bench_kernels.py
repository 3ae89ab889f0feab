"""The benchmark names the direct-space kernel that a shape runs: the bfloat16 one for wide
blocks on the matrix cores, the float one below 64 right-hand sides whatever the mode, the
vector one for wide blocks in mode 0."""
import pytest

import bench


@pytest.mark.parametrize("shape,block,want", [
    (dict(pair_mode=1), 128, "k_pair_split<8, 2>"), (dict(pair_mode=1), 256, "k_pair_split<8, 2>"),
    (dict(pair_mode=1), 64, "k_pair_split<4, 4>"), (dict(pair_mode=2), 128, "k_pair_split<4, 4>"),
    (dict(), 16, "k_pair_mfma<float, 4, 1, 1>"),
    (dict(pair_mode=1, pair_subsets=4), 32, "k_pair_mfma<float, 4, 2, 1>"),
    (dict(), 128, "k_pair_list<float, 2, 4>"),
    (dict(pair_subsets=4), 64, "k_pair_list<float, 4, 4>"),
    (dict(pair_subsets=1), 64, "k_pair_list<float, 1, 1>")])
def test_pair_kernel_of_a_shape(shape, block, want):
    assert bench.pair_kernel_name(shape, block, 24000) == want
