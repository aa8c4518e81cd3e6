"""Launches of at most one tile a compute unit (256 of them, 32 to each of the 8 dies that workgroups go to in turn).  Those that
are not ranked by list length deal every head's tiles in eighths, rounded up: no die may get more tiles than it has compute
units that way, and the workgroups that only fill up an eighth have to fit as well, or the launch takes a second round.  Host only."""
import math

import pytest
import torch

from paper_2505_14687_amd.probe import grat_probe_launch

DIES, UNITS = 8, 32


# heads, or tiles a head, that are no multiple of 8
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype,grid,group,heads,prompt", [
    (torch.bfloat16, (48, 48), (16, 16), 14, 0), (torch.float16, (48, 48), (16, 16), 13, 0), (torch.bfloat16, (80, 80), (16, 16), 5, 0),
    (torch.bfloat16, (48, 48), (16, 16), 13, 10), (torch.float32, (56, 56), (8, 8), 1, 0)])
def test_no_die_gets_more_tiles_than_units(dtype, grid, group, heads, prompt, d):
    i = grat_probe_launch(dtype, 1, heads, d, grid, group, 9, prompt)
    assert i.tiles <= DIES * UNITS and i.xcd_tiles <= UNITS


@pytest.mark.parametrize("dtype,d,grid,group,heads,prompt", [
    (torch.bfloat16, 64, (48, 48), (16, 16), 12, 86), (torch.bfloat16, 128, (16, 40), (8, 8), 24, 0), (torch.bfloat16, 128, (16, 48), (16, 16), 30, 1),
    (torch.float16, 128, (34, 46), (16, 16), 12, 0), (torch.float32, 64, (8, 56), (8, 8), 9, 0)])
def test_launches_that_fit_only_without_their_padding_are_ranked(dtype, d, grid, group, heads, prompt):
    i = grat_probe_launch(dtype, 1, heads, d, grid, group, 9, prompt)
    assert i.tiles <= DIES * UNITS and i.longest_first


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_sweep_of_small_launches(dtype):
    seen = 0
    for rows in range(1, 9):
        for cols in range(rows, 9):
            for heads in range(1, 33):
                for prompt in (0, 100) if dtype == torch.bfloat16 else (0,):
                    i = grat_probe_launch(dtype, 1, heads, 64, (16 * rows, 16 * cols), (16, 16), min(9, rows * cols), prompt)
                    if i.tiles > DIES * UNITS:
                        continue
                    seen += 1
                    # (by rank the prompt tiles and the grouped ones are each dealt in turn: one more where neither fills a row of dies)
                    assert i.xcd_tiles <= UNITS or (prompt and i.longest_first and i.xcd_tiles <= math.ceil(i.tiles / DIES) + 1)
                    tiles_per_head = rows * cols * math.ceil(256 / i.rows)
                    grouped = DIES * math.ceil(tiles_per_head / DIES) * heads
                    prompts = DIES * math.ceil(heads * math.ceil(prompt / i.rows) / DIES)
                    assert i.longest_first == (grouped + prompts > (DIES * UNITS if i.teams > 1 or rows * cols < 4 else DIES * UNITS - 1))
    assert seen > 200


# 257 to 384 tiles of 256 rows: where 128-row workgroups were measured to be faster than the mixed launch, and where they were not
@pytest.mark.parametrize("grid,group,max_kv,heads,mixed", [
    ((64, 64), (16, 16), 9, 18, False), ((64, 64), (16, 16), 7, 24, False), ((32, 32), (16, 16), 4, 72, False),
    ((32, 32), (16, 16), 3, 96, False), ((32, 48), (16, 16), 6, 64, False), ((48, 48), (16, 16), 5, 36, False),
    ((48, 64), (16, 16), 9, 32, False), ((48, 96), (16, 16), 9, 16, False),
    ((96, 96), (16, 16), 25, 8, False), ((80, 80), (16, 16), 25, 11, False), ((12, 24, 32), (4, 8, 8), 27, 8, False),
    ((64, 80), (16, 16), 9, 14, False),
    ((64, 64), (16, 16), 9, 19, True), ((64, 64), (16, 16), 7, 23, True), ((64, 64), (16, 16), 9, 24, True),
    ((64, 80), (16, 16), 9, 16, True), ((80, 80), (16, 16), 9, 12, True), ((96, 96), (16, 16), 9, 10, True),
    ((128, 128), (16, 16), 25, 6, True), ((128, 128), (16, 16), 9, 6, True), ((8, 32, 48), (4, 8, 8), 18, 7, True)])
def test_mixed_launches_where_they_gain(grid, group, max_kv, heads, mixed):
    assert (grat_probe_launch(torch.bfloat16, 1, heads, 128, grid, group, max_kv).whole_tiles > 0) == mixed


# joint sequences of more than 256 tiles: two teams only where the prompt tiles' walk is what the launch waits for
@pytest.mark.parametrize("grid,group,max_kv,heads,d,prompt,teams", [
    ((4, 8, 40), (2, 8, 8), 10, 24, 128, 88, 1), ((64, 64), (32, 32), 3, 8, 128, 835, 1), ((64, 96), (32, 32), 6, 6, 64, 18, 1),
    ((64, 32), (16, 16), 5, 20, 128, 96, 1), ((64, 64), (16, 16), 16, 8, 128, 62, 1), ((128, 128), (16, 16), 15, 12, 128, 100, 1),
    ((128, 128), (16, 16), 15, 8, 128, 100, 2), ((64, 64), (16, 16), 9, 12, 64, 256, 2), ((128, 128), (16, 16), 9, 8, 128, 512, 2),
    ((48, 48), (16, 16), 9, 12, 64, 86, 2), ((2, 32, 32), (2, 8, 8), 9, 16, 128, 127, 2), ((8, 24, 24), (2, 8, 8), 27, 10, 128, 74, 2),
    ((2, 16, 64), (2, 8, 8), 6, 28, 64, 21, 2), ((48, 48), (16, 16), 5, 16, 64, 91, 1), ((4, 24, 24), (2, 8, 8), 6, 16, 128, 87, 2), ((80, 144), (16, 16), 35, 4, 128, 21, 2), ((160, 304), (16, 16), 49, 3, 64, 56, 2)])
def test_teams_of_joint_sequences(grid, group, max_kv, heads, d, prompt, teams):
    assert grat_probe_launch(torch.bfloat16, 1, heads, d, grid, group, max_kv, prompt).teams == teams


# short lists at head_dim 128: four teams of 64 rows against undivided workgroups of 128, half as many
@pytest.mark.parametrize("grid,group,max_kv,heads,teams", [
    ((16, 32), (16, 16), 2, 27, 1), ((16, 32), (8, 16), 4, 25, 1), ((16, 32), (16, 16), 2, 15, 4), ((16, 32), (16, 16), 2, 21, 1), ((8, 112), (8, 16), 5, 15, 4), ((16, 80), (16, 16), 3, 10, 4),
    ((32, 32), (16, 16), 4, 15, 4), ((32, 32), (8, 8), 9, 16, 4)])
def test_four_teams_of_groups(grid, group, max_kv, heads, teams):
    assert grat_probe_launch(torch.bfloat16, 1, heads, 128, grid, group, max_kv).teams == teams


# 256 undivided workgroups, padding included: ranked unless their groups are too few for lists that differ
@pytest.mark.parametrize("dtype,d,grid,group,max_kv,heads,ranked", [
    (torch.bfloat16, 128, (32, 32), (32, 32), 1, 32, 0), (torch.float16, 64, (4, 24, 8), (4, 8, 8), 3, 32, 0), (torch.float32, 128, (32, 64), (32, 32), 2, 2, 0),
    (torch.bfloat16, 128, (32, 32), (16, 16), 4, 32, 1), (torch.float32, 64, (16, 64), (8, 8), 6, 16, 1)])
def test_full_launches_of_few_groups_are_not_ranked(dtype, d, grid, group, max_kv, heads, ranked):
    i = grat_probe_launch(dtype, 1, heads, d, grid, group, max_kv)
    assert i.teams <= 1 and i.longest_first == ranked
