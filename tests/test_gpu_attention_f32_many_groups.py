"""fp32 launches of more workgroups than one launch of 512 threads each may hold (2^23): single-token groups of a long
sequence, many heads.  Every query attends itself and its two neighbours, so the reference is three products."""
import math

import pytest
import torch

import paper_2505_14687_amd as grat

pytestmark = pytest.mark.gpu


def test_more_workgroups_than_one_launch_holds():
    heads, n, d = 33, 1 << 18, 64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5500)
    q, k, v = (torch.randn(1, heads, n, d, generator=gen, device="cuda") for _ in range(3))
    count, index = grat.grat_build_block_lists((n,), (1,), "block", (1,))
    O = torch.full_like(q, float("nan"))
    grat.grat_attention_fwd(q, k, v, 1.0 / math.sqrt(d), (n,), (1,), count, index, out=O)
    for h in range(heads):
        a, b, c = (t[0, h].double() for t in (q, k, v))
        s = torch.full((n, 3), -math.inf, dtype=torch.float64, device="cuda")
        s[1:, 0] = (a[1:] * b[:-1]).sum(-1)
        s[:, 1] = (a * b).sum(-1)
        s[:-1, 2] = (a[:-1] * b[1:]).sum(-1)
        w = torch.softmax(s / math.sqrt(d), -1)
        want = w[:, 1:2] * c
        want[1:] += w[1:, 0:1] * c[:-1]
        want[:-1] += w[:-1, 2:3] * c[1:]
        err = (O[0, h].double() - want).norm(dim=-1) / want.norm(dim=-1)
        assert float(err.max()) <= 1e-4, h   # (a NaN fails too)
