"""The calls a user of this framework makes, as measurable cases.

The framework is one attention path (block lists + grouped attention, forward only, as in the paper)
behind a handful of entry points.  A case is one pass through one of them:

  entry     "grid"    grat_attention_fwd         tokens of an image or video grid
            "joint"   grat_attention_global_fwd  prompt tokens and grid tokens in one sequence
            "packed"  grat_attention_packed_fwd  the same, read in place from a fused QKV projection
            "dense"   grat_dense_attention_fwd   full attention over one sequence
  build     the block lists are built in the pass too (a new resolution, and the benchmark's step);
            otherwise they are kept beside the weights, as a sampler that runs many steps does
  grid, group, radius   extents per axis, last axis fastest, "512x512"
  prompt    prompt tokens of a joint sequence, ahead of the grid tokens or behind them
  token_major  Q, K, V are [B, H, N, d] views of [B, N, H, d] tensors, as a projection leaves them

Inputs are N(0,1), which is what queries, keys and values are after the normalisation of the models
the method is applied to, and what the tests and the benchmark draw.
"""
import math

import torch

import paper_2505_14687_amd as grat

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


def _case(name, entry, grid, group, pattern, radius, *, batch=1, heads=24, head_dim=128, dtype="bf16", build=False,
          prompt=0, prompt_first=True, token_major=False):
    return {"name": name, "entry": entry, "grid": grid, "group": group, "pattern": pattern, "radius": radius,
            "batch": batch, "heads": heads, "head_dim": head_dim, "dtype": dtype, "build": build, "prompt": prompt,
            "prompt_first": prompt_first, "token_major": token_major}


def listed():
    return [
        # the first call anyone makes: the small fp32 configuration that examples and parity checks use
        _case("tiny_f32_block", "grid", "32x32", "8x8", "block", "1x1", heads=2, head_dim=64, dtype="f32", build=True),
        # one layer of a 1024^2-pixel image model in fp32: checking a model's numerics at its real size
        _case("img1024_f32_cross", "grid", "64x64", "16x16", "cross", "0x0", dtype="f32"),
        # the same layer in bf16 at a resolution not seen before: launches of a tenth of a millisecond
        _case("img1024_block", "grid", "64x64", "16x16", "block", "1x1", build=True),
        # smaller heads, several images at once, tensors as the projections leave them
        _case("img1024_d64_cross", "grid", "64x64", "16x16", "cross", "0x0", batch=4, heads=16, head_dim=64,
              token_major=True),
        # a layer of an image transformer at 2048^2 pixels: 512 prompt tokens, fused QKV read in place
        _case("img2048_prompt_packed", "packed", "128x128", "16x16", "block", "1x1", prompt=512),
        # a wide 2560x1440-pixel image, two at a time, in half precision: 90 token rows in groups of 16
        _case("img1440_ragged_f16", "grid", "90x160", "16x16", "block", "1x1", batch=2, dtype="f16"),
        # full attention over a joint sequence of odd length: what the grouped layers stand beside
        _case("dense_odd", "dense", "4429", "1", "dense", "0"),
        # video, 128-token groups: the benchmark's own shape
        _case("video_block", "grid", "30x48x80", "2x8x8", "block", "1x1x1"),
        # the paper's own video shape with its prompt tokens behind the video tokens
        _case("video_cross_prompt", "joint", "32x48x80", "4x8x8", "cross", "0x0x0", prompt=256, prompt_first=False),
        # the paper's group-size ablation at 8192^2 pixels: many small groups
        _case("img8192_g8_block", "grid", "512x512", "8x8", "block", "1x1"),
        # the headline shape at 8192^2 pixels, lists included
        _case("img8192_block", "grid", "512x512", "16x16", "block", "1x1", build=True),
        # ... and its criss-cross pattern, the largest launch
        _case("img8192_cross", "grid", "512x512", "16x16", "cross", "0x0"),
    ]


def draw(rng):
    while True:
        case = _draw_any(rng)
        flops, limit = work(case)["flops"], 0.5e12 if case["dtype"] == "f32" else 25e12
        if 1e8 <= flops <= limit:
            return case


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_any(rng):
    entry = rng.choice(["grid"] * 5 + ["joint", "packed", "packed", "dense"])
    dtype = rng.choice(["bf16"] * 6 + ["f16"] * 2 + (["f32"] * 2 if entry in ("grid", "dense") else []))
    batch, heads = rng.choice([1, 1, 1, 2, 4]), rng.choice([1, 2, 4, 8, 12, 16, 24, 24])
    head_dim = rng.choice([64, 128, 128])
    if entry == "dense":
        case = _case("", "dense", str(_log_int(rng, 64, 32768)), "1", "dense", "0", batch=batch, heads=heads,
                     head_dim=head_dim, dtype=dtype)
    else:
        if rng.random() < 0.65:   # an image
            side = rng.choice([8, 16, 16, 16, 32])
            group = [side, side]
            rows = _log_int(rng, 32, 512)
            grid = [rows, min(512, max(32, int(rows * rng.uniform(0.5, 2.0))))]
            radius = [rng.choice([1, 1, 1, 2, 3])] * 2
            pattern = rng.choice(["block", "block", "cross"])
        else:                     # a video
            group = rng.choice([[2, 8, 8], [4, 8, 8]])
            grid = [_log_int(rng, 4, 32), _log_int(rng, 16, 64), _log_int(rng, 16, 96)]
            radius = [1, rng.choice([1, 1, 2]), 1]
            pattern = rng.choice(["block", "block", "cross", "cross_planes"])
        if entry != "grid" or rng.random() < 0.6:   # whole groups (joint sequences have no others)
            grid = [max(1, round(t / g)) * g for t, g in zip(grid, group)]
        if pattern != "block":
            radius = [0] * len(group)
        prompt = 0 if entry == "grid" else _log_int(rng, 16, 1024)
        case = _case("", entry, _text(grid), _text(group), pattern, _text(radius), batch=batch, heads=heads,
                     head_dim=head_dim, dtype=dtype, build=rng.random() < 0.3, prompt=prompt,
                     prompt_first=rng.random() < 0.5, token_major=entry != "packed" and rng.random() < 0.3)
    del case["name"]
    return case


def _text(extents):
    return "x".join(str(e) for e in extents)


def _extents(text):
    return tuple(int(e) for e in text.split("x"))


def prepare(case, seed):
    grid, group, radius = (_extents(case[k]) for k in ("grid", "group", "radius"))
    B, H, d = case["batch"], case["heads"], case["head_dim"]
    L = math.prod(grid) + case["prompt"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=DTYPES[case["dtype"]])

    state = {"case": case, "grid": grid, "group": group, "radius": radius, "scale": 1.0 / math.sqrt(d)}
    if case["entry"] == "packed":
        state["qkv"] = normal(B, L, 3, H, d)
    elif case["token_major"]:
        state["q"], state["k"], state["v"] = (normal(B, L, H, d).permute(0, 2, 1, 3) for _ in range(3))
    else:
        state["q"], state["k"], state["v"] = (normal(B, H, L, d) for _ in range(3))
    if case["entry"] != "dense" and not case["build"]:
        state["lists"] = grat.grat_build_block_lists(grid, group, case["pattern"], radius)
    return state


def run(state):
    case = state["case"]
    if case["entry"] == "dense":
        return grat.grat_dense_attention_fwd(state["q"], state["k"], state["v"], state["scale"])
    grid, group = state["grid"], state["group"]
    if case["build"]:
        count, index = grat.grat_build_block_lists(grid, group, case["pattern"], state["radius"])
    else:
        count, index = state["lists"]
    if case["entry"] == "packed":
        out = grat.grat_attention_packed_fwd(state["qkv"], state["scale"], grid, group, count, index,
                                             n_global=case["prompt"], global_first=case["prompt_first"])
    elif case["entry"] == "joint":
        out = grat.grat_attention_global_fwd(state["q"], state["k"], state["v"], state["scale"], case["prompt"],
                                             case["prompt_first"], grid, group, count, index)
    else:
        out = grat.grat_attention_fwd(state["q"], state["k"], state["v"], state["scale"], grid, group, count, index)
    return (count, index, out) if case["build"] else out


def _attended_pairs(case):
    """(query, key) pairs of one head."""
    grid, group, radius = (_extents(case[k]) for k in ("grid", "group", "radius"))
    n = math.prod(grid)
    if case["pattern"] == "dense":
        return n * n
    near, same, every = [], [], []   # per axis: pairs of coordinates in near groups, in one group, at all
    for t, g, r in zip(grid, group, radius):
        size = [min(g, t - p) for p in range(0, t, g)]
        near.append(sum(s * sum(size[max(0, i - r):i + r + 1]) for i, s in enumerate(size)))
        same.append(sum(s * s for s in size))
        every.append(t * t)
    axes = range(len(grid))
    if case["pattern"] == "block":
        pairs = math.prod(near)
    elif case["pattern"] == "cross":   # all group coordinates equal, or all but one
        pairs = math.prod(same) + sum((every[k] - same[k]) * math.prod(same[j] for j in axes if j != k) for k in axes)
    else:                              # at least one equal
        pairs = math.prod(every) - math.prod(every[k] - same[k] for k in axes)
    return pairs + case["prompt"] * (2 * n + case["prompt"])


def work(case):
    rows = case["batch"] * case["heads"] * (math.prod(_extents(case["grid"])) + case["prompt"])
    nbytes = 4 * rows * case["head_dim"] * (4 if case["dtype"] == "f32" else 2)
    return {"bytes": nbytes, "flops": 4 * case["head_dim"] * case["batch"] * case["heads"] * _attended_pairs(case)}


def tolerance(case):
    # Against the same attention in 64 bits on the same inputs the whole-tensor error is 2.3e-3 in bf16
    # and 2.7e-4 in half (softmax weights and result rounded once to the type), and in fp32 5e-7 to
    # 1.1e-6 (576 to 1792 keys a row): four times that.
    return {"bf16": {"rel": 1e-2}, "f16": {"rel": 1.2e-3}, "f32": {"rel": 4e-6}}[case["dtype"]]
