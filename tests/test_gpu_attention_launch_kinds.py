"""Every kind of 16-bit launch on every kind of input: undivided workgroups of 128 and 256 rows, two and four teams, mixed launches,
with prompts, several batches and token-major or packed tensors, flat, peaked and rising scores.  The kernel that a case is
meant for is pinned by name, so that a case that a changed dispatch rule takes elsewhere fails instead of testing something
else.  Against the float64 softmax of the same inputs."""
import math

import pytest
import torch

import paper_2505_14687_amd as grat
from paper_2505_14687_amd.probe import launched_kernel
from test_gpu_attention_teams import BAR, _group_mask

pytestmark = pytest.mark.gpu


def _inputs(batch, heads, n, d, dtype, scores):
    """[B, n, 3, H, d]"""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(batch + heads + n + d)
    x = torch.randn((batch, n, 3, heads, d), generator=gen, device="cuda", dtype=torch.float32)
    if scores.startswith("peaked"):       # near one-hot weights
        x[:, :, 0] *= float(scores[6:])
    elif scores == "rising":              # every KV tile beats the one before it
        sign = torch.where(x[:, :1, 0] < 0, -1.0, 1.0)
        ramp = torch.arange(n, device="cuda", dtype=torch.float32)[None, :, None, None] / n * 6.0
        x[:, :, 0] = 0.05 * x[:, :, 0] + 3.0 * sign
        x[:, :, 1] = 0.05 * x[:, :, 1] + ramp * sign
    return x.to(dtype)


def _run(kernel, dtype, batch, heads, d, grid, group, pattern, prompt, first, layout, scores):
    dense = grid is None
    n = prompt if dense else prompt + math.prod(grid)
    radius, scale = () if dense else (1,) * len(grid), 1.0 / math.sqrt(d)
    count = index = None
    if not dense:
        count, index = grat.grat_build_block_lists(grid, group, pattern, radius)
    assert launched_kernel(dtype, batch, heads, d, grid, group, 0 if dense else index.shape[1], prompt) == "grat::attn_mfma_" + kernel
    qkv = _inputs(batch, heads, n, d, dtype, scores)
    q, k, v = (qkv[:, :, i].transpose(1, 2) for i in range(3))           # [B, H, n, d] views
    if layout == "packed":
        out = torch.full((batch, n, heads, d), float("nan"), device="cuda", dtype=dtype)
        grat.grat_attention_packed_fwd(qkv, scale, grid, group, count, index, n_global=prompt, global_first=first, out=out)
        out = out.transpose(1, 2)
    else:
        a = [t.contiguous() if layout == "heads first" else t.transpose(1, 2).contiguous().transpose(1, 2) for t in (q, k, v)]
        out = torch.full_like(a[0], float("nan"))
        if dense:
            grat.grat_dense_attention_fwd(*a, scale, out=out)
        elif prompt:
            grat.grat_attention_global_fwd(*a, scale, prompt, first, grid, group, count, index, out=out)
        else:
            grat.grat_attention_fwd(*a, scale, grid, group, count, index, out=out)
    assert bool(torch.isfinite(out).all())
    mask = torch.ones(n, n, dtype=torch.bool, device="cuda")
    if not dense:
        g0 = prompt if first else 0
        m = n - prompt
        mask[g0:g0 + m, g0:g0 + m] = _group_mask(grid, group, pattern, radius)
    diff2 = want2 = 0.0
    for b in range(batch):
        for h in range(heads):
            s = (q[b, h].double() @ k[b, h].double().T.contiguous() * scale).masked_fill_(~mask, -math.inf)
            want = torch.softmax(s, -1) @ v[b, h].double()
            diff = out[b, h].double() - want
            assert float((diff.norm(dim=-1) / want.norm(dim=-1)).max()) <= 2 * BAR[dtype], (b, h)
            diff2, want2 = diff2 + float(diff.pow(2).sum()), want2 + float(want.pow(2).sum())
    assert math.sqrt(diff2 / want2) <= BAR[dtype]


DTYPES = {"false": torch.bfloat16, "true": torch.float16}


def _dtype(kernel):
    return DTYPES[kernel.split("<")[1].rstrip(">").split(", ")[3 if "," in kernel else 0]]


# undivided workgroups of 128 rows: prompt and grid in one sequence, both types and head dims
@pytest.mark.parametrize("half", ["false", "true"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,grid,group,pattern,prompt,first,layout", [
    (24, (48, 32), (16, 16), "block", 100, True, "heads first"),
    (42, (32, 32), (8, 16), "block", 65, False, "packed"),
    (33, (48, 32), (16, 16), "cross", 1, False, "token major"),
])
def test_undivided_joint_128_rows(heads, grid, group, pattern, prompt, first, layout, d, half):
    kernel = f"kernel<4, 64, 2, {half}, {d}>"
    _run(kernel, _dtype(kernel), 1, heads, d, grid, group, pattern, prompt, first, layout, "normal")


CASES = [  # kernel, batch, heads, head_dim, grid, group, pattern, prompt, prompt first, layout, scores
    # undivided, 128 rows
    ("kernel<4, 64, 0, true, 128>", 1, 24, 128, (32, 64), (8, 16), "block", 0, True, "heads first", "normal"),
    ("kernel<4, 64, 0, true, 128>", 2, 6, 128, (64, 64), (16, 16), "cross", 0, True, "token major", "peaked16"),
    ("kernel<4, 64, 0, true, 128>", 1, 12, 128, (64, 64), (16, 16), "cross", 0, True, "heads first", "rising"),
    ("kernel<4, 64, 0, false, 128>", 1, 12, 128, (64, 64), (16, 16), "block", 0, True, "heads first", "peaked4"),
    ("kernel<4, 64, 0, false, 128>", 1, 12, 128, (64, 64), (16, 16), "cross", 0, True, "packed", "rising"),
    ("kernel<4, 64, 0, true, 64>", 1, 12, 64, (64, 64), (16, 16), "block", 0, True, "heads first", "peaked16"),
    ("kernel<4, 64, 0, false, 64>", 1, 12, 64, (64, 64), (16, 16), "cross", 0, True, "heads first", "rising"),
    ("kernel<4, 64, 2, true, 128>", 1, 24, 128, (48, 32), (16, 16), "block", 100, True, "heads first", "rising"),
    ("kernel<4, 64, 2, false, 64>", 1, 24, 64, (48, 32), (16, 16), "block", 100, False, "heads first", "peaked16"),
    # undivided, 256 rows
    ("kernel<8, 64, 0, true, 128>", 2, 18, 128, (64, 64), (16, 16), "block", 0, True, "token major", "peaked16"),
    ("kernel<8, 64, 0, true, 128>", 1, 33, 128, (64, 64), (16, 16), "cross", 0, True, "heads first", "rising"),
    ("kernel<8, 64, 2, true, 128>", 1, 33, 128, (64, 64), (16, 16), "block", 40, False, "packed", "normal"),
    # undivided, 64 rows: 32-key and 64-key tiles
    ("kernel<2, 32, 0, true, 128>", 1, 24, 128, (32, 48), (8, 8), "block", 0, True, "heads first", "peaked16"),
    ("kernel<2, 32, 0, false, 128>", 2, 12, 128, (32, 48), (8, 8), "cross", 0, True, "token major", "rising"),
    ("kernel<2, 32, 0, true, 64>", 1, 24, 64, (32, 48), (8, 8), "block", 0, True, "packed", "rising"),
    ("kernel<2, 64, 0, true, 128>", 1, 4, 128, (8, 528), (8, 8), "cross", 0, True, "heads first", "rising"),
    ("kernel<2, 64, 0, false, 64>", 2, 2, 64, (8, 528), (8, 8), "cross", 0, True, "token major", "peaked16"),
    # two teams
    ("teams_kernel<4, 64, 0, true, 128, 2>", 2, 3, 128, (64, 64), (16, 16), "cross", 0, True, "token major", "rising"),
    ("teams_kernel<4, 64, 0, false, 64, 2>", 2, 4, 64, (64, 64), (16, 16), "block", 0, True, "packed", "peaked16"),
    ("teams_kernel<4, 64, 2, false, 128, 2>", 2, 1, 128, (48, 48), (16, 16), "block", 130, False, "packed", "normal"),
    ("teams_kernel<4, 64, 2, true, 64, 2>", 2, 2, 64, (32, 48), (16, 16), "cross", 77, True, "packed", "rising"),
    ("teams_kernel<4, 64, 1, false, 128, 2>", 2, 9, 128, None, None, "", 1500, True, "token major", "rising"),
    # four teams
    ("teams_kernel<2, 32, 0, false, 128, 4>", 2, 2, 128, (48, 48), (16, 16), "cross", 0, True, "token major", "rising"),
    ("teams_kernel<2, 32, 0, true, 64, 4>", 2, 1, 64, (64, 64), (16, 16), "block", 0, True, "token major", "peaked16"),
    ("teams_kernel<2, 32, 1, true, 128, 4>", 2, 1, 128, None, None, "", 1001, True, "token major", "rising"),
    ("teams_kernel<2, 32, 1, false, 64, 4>", 3, 2, 64, None, None, "", 1055, True, "token major", "peaked16"),
    # mixed
    ("mixed_kernel<false>", 2, 8, 128, (64, 80), (16, 16), "block", 0, True, "token major", "normal"),
    ("mixed_kernel<true>", 1, 16, 128, (64, 80), (16, 16), "cross", 0, True, "packed", "rising"),
    ("mixed_kernel<true>", 3, 5, 128, (4, 32, 48), (4, 8, 8), "block", 0, True, "heads first", "peaked16"),
]


@pytest.mark.parametrize("kernel,batch,heads,d,grid,group,pattern,prompt,first,layout,scores", CASES)
def test_launch_kinds(kernel, batch, heads, d, grid, group, pattern, prompt, first, layout, scores):
    _run(kernel, _dtype(kernel), batch, heads, d, grid, group, pattern, prompt, first, layout, scores)
