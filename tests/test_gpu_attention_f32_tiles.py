"""fp32 attention at the edges of its tiles: launches large enough for the 32-query waves (at least 512 of them, more
than 48 tokens a group) in both workgroup heights, key tiles with one key left over, waves without queries; the
16-query workgroups of one wave (from 1 024 of them on) and of eight, and the first sizes on either side of their range.  v_gain 2^40: values beyond the range of the split into bf16 numbers, so that
the 32-query waves take the walk on the fp32 instructions instead.  Bound as in the other fp32 tests."""
import math

import numpy as np
import pytest

import paper_2505_14687_amd as grat
from gpu_util import assert_all_written, assert_close, nan_like, to_device, to_f64
from oracle import grat_oracle as orc
from paper_2505_14687_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("v_gain", [1.0, 2.0 ** 40])
@pytest.mark.parametrize("grid,group,pattern,radius,heads,d", [
    ((32, 64), (4, 8), "block", (1, 1), 16, 64),       # 32 tokens
    ((42, 64), (7, 7), "block", (1, 1), 12, 128),      # 49 tokens: the smallest groups of the 64-row workgroups, clipped
    ((33, 62), (7, 9), "cross", (0, 0), 16, 64),       # 63 tokens, clipped on both axes
    ((32, 60), (8, 6), "block", (1, 1), 16, 128),      # 48 tokens: the largest of the 16-row workgroups
    ((32, 64), (8, 8), "cross", (0, 0), 16, 128),      # 64-row workgroups
    ((32, 64), (16, 16), "cross", (0, 0), 16, 64),     # 128-row workgroups
    ((32, 64), (8, 12), "block", (1, 1), 16, 128),     # 96-token groups, the last column of them 4 wide
    ((24, 80), (4, 10), "block", (1, 2), 12, 64),      # 40-token groups: a key tile of 32 and one of 8
    ((35, 64), (16, 16), "block", (1, 1), 16, 128),    # 128-row workgroups, last group-row 3 of 16 rows
    ((33, 62), (3, 11), "cross", (0, 0), 16, 64),      # 33-token groups, clipped on the last axis
    ((33, 33), (1, 17), "block", (2, 1), 8, 128),      # 17 tokens: just above the packed groups
    ((32, 36), (4, 4), "block", (1, 1), 2, 128),       # 16 tokens: one block of the split kernel each
    ((33, 35), (3, 5), "block", (1, 1), 2, 64),        # 15 tokens, packed, clipped on both axes
    ((33, 35), (3, 5), "block", (1, 1), 16, 64),       # the same, one wave a workgroup
    ((20, 26), (1, 1), "cross", (0, 0), 4, 128),       # single tokens
])
def test_grouped_tiles(grid, group, pattern, radius, heads, d, v_gain):
    host = synth.make_qkv(1, heads, int(np.prod(grid)), d, "f32", 5100, q_gain=3.0)
    scale = 1.0 / math.sqrt(d)
    dev = [to_device(x) for x in host]
    dev[2] *= v_gain
    O = nan_like(dev[0])
    count, index = grat.grat_build_block_lists(grid, group, pattern, radius)
    grat.grat_attention_fwd(*dev, scale, grid, group, count, index, out=O)
    assert_all_written(O, f"{grid} {group}")
    assert_close(to_f64(O) / v_gain, orc.grat_attention(*host, grid, group, pattern, radius, scale), "f32", f"{grid} {group} {pattern}")


@pytest.mark.parametrize("v_gain", [1.0, 2.0 ** 40])
@pytest.mark.parametrize("N,heads,d", [(2050, 16, 64), (2079, 16, 128), (16, 1, 128), (17, 2, 64), (129, 3, 128),
                                       (48, 300, 128), (49, 300, 64), (64, 300, 128), (128, 130, 128), (129, 130, 64),
                                       (1, 1100, 64), (15, 300, 128)])
def test_dense_tiles(N, heads, d, v_gain):
    host = synth.make_qkv(1, heads, N, d, "f32", 5200, q_gain=3.0)
    dev = [to_device(x) for x in host]
    dev[2] *= v_gain
    O = nan_like(dev[0])
    grat.grat_dense_attention_fwd(*dev, 1.0 / math.sqrt(d), out=O)
    assert_all_written(O, f"dense {N}")
    assert_close(to_f64(O) / v_gain, orc.dense_attention(*host, 1.0 / math.sqrt(d)), "f32", f"dense N={N}")
