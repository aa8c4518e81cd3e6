"""Small 16-bit launches, whose workgroups are teams of waves that share the keys (4 teams: 64-row workgroups of 32-key tiles,
2 teams: 128-row workgroups of 64-key tiles), against the float64 softmax of the same inputs: fewer tiles than teams, tiles
left over, the last tile cut short in every team, prompts, lists of unequal length, scores of -infinity."""
import math

import pytest
import torch

import paper_2505_14687_amd as grat

pytestmark = pytest.mark.gpu

# weights and result rounded once to the type, as in the other 16-bit tests: per tensor, and twice that per row
BAR = {torch.bfloat16: 1e-2, torch.float16: 1.25e-3}


def _inputs(heads, n, d, dtype, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return [torch.randn((1, heads, n, d), generator=gen, device="cuda", dtype=dtype) for _ in range(3)]


def _check(got, q, k, v, mask, dtype):
    assert bool(torch.isfinite(got).all())
    want = torch.empty_like(q, dtype=torch.float64)
    for h in range(q.shape[1]):
        s = q[0, h].double() @ k[0, h].double().T.contiguous() / math.sqrt(q.shape[3])
        want[0, h] = torch.softmax(s if mask is None else s.masked_fill(~mask, -math.inf), -1) @ v[0, h].double()
    assert float((got.double() - want).norm() / want.norm()) <= BAR[dtype]
    assert float(((got.double() - want).norm(dim=-1) / want.norm(dim=-1)).max()) <= 2 * BAR[dtype]


# head_dim 64: four teams from 384 keys on, two for 17 x 1 030; head_dim 128: four from 640 (tiles of 64 rows: eight keys each), two for 17 x 1 500
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,n", [(1, 384), (2, 385), (1, 641), (2, 672), (1, 703), (1, 1000), (3, 1279), (2, 2049), (17, 1030),
                                     (17, 1500), (16, 1601), (19, 1409)])
def test_sequences(heads, n, d):
    dtype = torch.float16 if n % 2 else torch.bfloat16
    q, k, v = _inputs(heads, n, d, dtype, 9000 + heads + n + d)
    out = torch.full_like(q, float("nan"))
    grat.grat_dense_attention_fwd(q, k, v, 1.0 / math.sqrt(d), out=out)
    _check(out, q, k, v, None, dtype)


def _group_mask(grid, group, pattern, radius):
    n = math.prod(grid)
    c = torch.stack(torch.meshgrid(*[torch.arange(t, device="cuda") // g for t, g in zip(grid, group)], indexing="ij"), -1).reshape(n, -1)
    diff = (c[:, None] - c[None]).abs()
    return (diff <= torch.tensor(radius, device="cuda")).all(-1) if pattern == "block" else (diff != 0).sum(-1) <= 1


# four teams; two (288 tiles of 64 rows); 24x8 groups have three 64-key tiles; a prompt ahead of or behind the grid: two teams
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("grid,group,pattern,heads,prompt", [
    ((24, 40), (8, 8), "block", 3, 0), ((8, 16, 16), (2, 8, 8), "cross", 1, 0), ((48, 48), (16, 16), "block", 2, 0),
    ((64, 48), (32, 16), "cross", 1, 0), ((48, 64), (16, 16), "block", 6, 0), ((72, 24), (24, 8), "block", 1, 0),
    ((48, 32), (16, 16), "block", 2, 1), ((48, 32), (16, 16), "cross", 1, 64), ((32, 32), (16, 16), "block", 3, 130),
    ((32, 48), (16, 16), "cross", 2, 200)])
def test_groups(grid, group, pattern, heads, prompt, d):
    n, dtype = math.prod(grid), torch.bfloat16 if prompt % 4 else torch.float16
    radius, first = (1,) * len(grid), heads % 2 == 1
    q, k, v = _inputs(heads, n + prompt, d, dtype, 9100 + n + prompt)
    mask = torch.ones(n + prompt, n + prompt, dtype=torch.bool, device="cuda")
    g0 = prompt if first else 0
    mask[g0:g0 + n, g0:g0 + n] = _group_mask(grid, group, pattern, radius)
    count, index = grat.grat_build_block_lists(grid, group, pattern, radius)
    out = torch.full_like(q, float("nan"))
    if prompt:
        grat.grat_attention_global_fwd(q, k, v, 1.0 / math.sqrt(d), prompt, first, grid, group, count, index, out=out)
    else:
        grat.grat_attention_fwd(q, k, v, 1.0 / math.sqrt(d), grid, group, count, index, out=out)
    _check(out, q, k, v, mask, dtype)


# 257 to 384 tiles of 256 rows: 256 whole ones, the others split between workgroups of two teams
@pytest.mark.parametrize("grid,group,pattern,heads", [((64, 64), (16, 16), "block", 17), ((64, 64), (16, 16), "cross", 24),
                                                      ((16, 48), (16, 16), "block", 86), ((8, 32, 48), (4, 8, 8), "block", 6)])
def test_mixed_launches(grid, group, pattern, heads):
    n, radius = math.prod(grid), (1,) * len(grid)
    dtype = torch.float16 if heads % 2 else torch.bfloat16
    q, k, v = _inputs(heads, n, 128, dtype, 9200 + heads)
    count, index = grat.grat_build_block_lists(grid, group, pattern, radius)
    out = torch.full_like(q, float("nan"))
    grat.grat_attention_fwd(q, k, v, 1.0 / math.sqrt(128), grid, group, count, index, out=out)
    assert bool(torch.isfinite(out).all())
    rows = torch.arange(heads % 7, n, max(1, n // 1000), device="cuda")
    mask = _group_mask(grid, group, pattern, radius)[rows]
    for h in range(heads):
        s = (q[0, h, rows].double() @ k[0, h].double().T.contiguous() / math.sqrt(128)).masked_fill(~mask, -math.inf)
        want = torch.softmax(s, -1) @ v[0, h].double()
        assert float(((out[0, h, rows].double() - want).norm(dim=-1) / want.norm(dim=-1)).max()) <= 2 * BAR[dtype]


@pytest.mark.parametrize("d", [64, 128])
def test_short_lists_among_long_ones(d):
    """A list of one group has two 32-key tiles: two of four teams have none.  And O with a layout of its own (packed)."""
    grid, group, n = (24, 24), (8, 8), 576
    count, index = grat.grat_build_block_lists(grid, group, "block", (1, 1))
    count[4] = 1                                     # group 4 attends group 0 only
    gen = torch.Generator(device="cuda")
    gen.manual_seed(77)
    qkv = torch.randn((1, n, 3, 2, d), generator=gen, device="cuda", dtype=torch.bfloat16)
    out = grat.grat_attention_packed_fwd(qkv, 1.0 / math.sqrt(d), grid, group, count, index)
    mask = _group_mask(grid, group, "block", (1, 1))
    gid = (torch.arange(24, device="cuda")[:, None] // 8 * 3 + torch.arange(24, device="cuda") // 8).reshape(-1)
    mask[gid == 4] = gid == 0
    q, k, v = (qkv[:, :, i].transpose(1, 2).contiguous() for i in range(3))
    _check(out.transpose(1, 2), q, k, v, mask, torch.bfloat16)


# four teams, two teams (both walk from the last tile), undivided
@pytest.mark.parametrize("heads,n,d", [(1, 1024, 128), (17, 1536, 128), (1, 1000, 64), (17, 1100, 64), (24, 2100, 64)])
@pytest.mark.parametrize("behind", [False, True])
def test_scores_of_minus_infinity(heads, n, d, behind):
    """Keys 32 to 127, or the last 150, score -infinity: whole tiles, among them the first of some teams, or the first that is
    walked (not the first of the sequence)."""
    q, k, v = _inputs(heads, n, d, torch.bfloat16, 31)
    q[..., 0] = q[..., 0].abs() + 0.1
    k[:, :, slice(n - 150, n) if behind else slice(32, 128), 0] = -math.inf
    out = torch.full_like(q, float("nan"))
    grat.grat_dense_attention_fwd(q, k, v, 1.0 / math.sqrt(d), out=out)
    _check(out, q, k.clamp(min=-1e6), v, None, torch.bfloat16)
