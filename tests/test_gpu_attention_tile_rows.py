"""Dense 16-bit launches at the edges of their query tiles: 128-row workgroups (head_dim 64; head_dim 128 where they
leave less of the last round idle) and 256-row workgroups, and head_dim 64 over 64-, 128- and 256-token groups, against the
float64 softmax of the same 16-bit inputs."""
import math

import pytest
import torch

import paper_2505_14687_amd as grat

pytestmark = pytest.mark.gpu

# relative L2 per tensor: weights and result rounded once to the type, as in the other 16-bit tests
BAR = {torch.bfloat16: 1e-2, torch.float16: 1.25e-3}


def _inputs(batch, heads, n, d, dtype, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return [torch.randn((batch, heads, n, d), generator=gen, device="cuda", dtype=dtype) for _ in range(3)]


def _softmax64(q, k, v, mask=None):
    # (one head at a time in float64: the products are plain two-dimensional ones)
    out = torch.empty_like(q, dtype=torch.float64)
    for b in range(q.shape[0]):
        for h in range(q.shape[1]):
            s = q[b, h].double() @ k[b, h].double().T.contiguous() / math.sqrt(q.shape[3])
            if mask is not None:
                s = s.masked_fill(~mask, -math.inf)
            out[b, h] = torch.softmax(s, -1) @ v[b, h].double()
    return out


def _check(got, want, dtype):
    assert bool(torch.isfinite(got).all())
    err = (got.double() - want).norm(dim=-1) / want.norm(dim=-1)
    assert float((got.double() - want).norm() / want.norm()) <= BAR[dtype]
    assert float(err.max()) <= 2 * BAR[dtype]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,n", [(2, 1), (3, 63), (2, 127), (2, 128), (1, 129), (1, 257), (2, 385),
                                     (384, 130), (385, 130), (193, 257), (128, 257)])   # 128 | 256 | 128 | 256 rows
def test_dense_rows(heads, n, d):
    dtype = torch.bfloat16 if n % 2 else torch.float16
    q, k, v = _inputs(1, heads, n, d, dtype, 7000 + heads + n + d)
    out = torch.full_like(q, float("nan"))
    grat.grat_dense_attention_fwd(q, k, v, 1.0 / math.sqrt(d), out=out)
    _check(out, _softmax64(q, k, v), dtype)


@pytest.mark.parametrize("grid,group", [((32, 48), (16, 16)), ((40, 35), (16, 16)), ((4, 16, 24), (2, 8, 8)),
                                        ((3, 20, 17), (2, 8, 8)), ((24, 40), (8, 8)), ((21, 30), (8, 8)),
                                        ((80, 528), (8, 8))])   # the last: 75-group lists, 64-key tiles of 2-wave workgroups
def test_head_dim_64_groups(grid, group):
    _groups(grid, group, 64)


# boxes with whole tiles, and whole workgroups of queries, outside the grid; 10x10: the only group is clipped
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("grid,group", [((40, 70), (32, 32)), ((33, 65), (32, 32)), ((49, 33), (16, 16)), ((10, 10), (16, 16)),
                                        ((1, 40), (16, 16)), ((5, 17, 9), (4, 8, 8)), ((3, 9, 20), (2, 8, 8)), ((9, 25), (8, 8))])
def test_clipped_boxes(grid, group, d):
    _groups(grid, group, d)


# one launch with workgroups that take the plain walk (nothing clipped in reach) and ones that do not, whose last token
# inside the grid is the last of a wave's 32 queries, or the next; 4 heads of 130x256: 256-row workgroups at head_dim 128
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("grid,group,heads", [((66, 48), (16, 16), 2), ((67, 48), (16, 16), 2), ((78, 70), (16, 16), 2),
                                              ((130, 256), (16, 16), 4), ((36, 24), (8, 8), 2), ((37, 44), (8, 8), 2),
                                              ((9, 20, 24), (2, 8, 8), 2), ((40, 648), (8, 8), 1)])
def test_clipped_beside_whole_groups(grid, group, heads, d):
    _groups(grid, group, d, heads)


def _groups(grid, group, d, heads=None):
    pattern = "cross" if grid in ((80, 528), (40, 648)) else "block"
    n = math.prod(grid)
    dtype = torch.bfloat16
    q, k, v = _inputs(1, heads or (1 if n > 10000 else 2), n, d, dtype, 7100 + n)
    radius = (1,) * len(grid)
    count, index = grat.grat_build_block_lists(grid, group, pattern, radius)
    out = torch.full_like(q, float("nan"))
    grat.grat_attention_fwd(q, k, v, 1.0 / math.sqrt(d), grid, group, count, index, out=out)
    coords = torch.stack(torch.meshgrid(*[torch.arange(t, device="cuda") // g for t, g in zip(grid, group)], indexing="ij"), -1)
    coords = coords.reshape(n, len(grid))
    rows = torch.arange(0, n, max(1, n // 2000), device="cuda")
    diff = (coords[rows, None, :] - coords[None, :, :]).abs()
    mask = (diff <= 1).all(-1) if pattern == "block" else (diff != 0).sum(-1) <= 1
    want = torch.empty((1, q.shape[1], len(rows), d), dtype=torch.float64, device="cuda")
    for h in range(q.shape[1]):
        s = (q[0, h, rows].double() @ k[0, h].double().T.contiguous() / math.sqrt(d)).masked_fill(~mask, -math.inf)
        want[0, h] = torch.softmax(s, -1) @ v[0, h].double()
    assert bool(torch.isfinite(out).all())
    _check(out[:, :, rows], want, dtype)
