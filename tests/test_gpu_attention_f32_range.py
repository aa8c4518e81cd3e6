"""fp32 attention over the range of fp32 numbers: the split into bf16 numbers covers magnitudes below 2^34, everything else
goes through the fp32 instructions, and both must come out as float64 says.  Bound: an fp32 dot product of d terms is off
by up to d/2 roundings (2^-24) of its magnitude, so a weight by |scale * q k| of that, here at most 64 * 2^-24 * 30
= 1.2e-4 and on average far less; 2e-5 for the norm of all."""
import math

import numpy as np
import pytest
import torch

import paper_2505_14687_amd as grat
from gpu_util import errors, nan_like, to_f64
from oracle import grat_oracle as orc

pytestmark = pytest.mark.gpu
D = 128


def inputs(heads, n, gains, seed=5300):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return [g * torch.randn(1, heads, n, D, generator=gen, device="cuda") for g in gains]


def reference(q, k, v):
    q, k, v = (t[0].double().cpu() for t in (q, k, v))
    return torch.stack([torch.softmax(a @ b.t() / math.sqrt(D), -1) @ c for a, b, c in zip(q, k, v)])[None].numpy()


# 2, 8 and 12 heads: either side of the launch size from which waves own 32 queries (512 waves)
@pytest.mark.parametrize("heads", [2, 8, 12])
@pytest.mark.parametrize("gains", [(1, 1, 1), (3, 1, 1e-3), (1, 1, 1e-6), (1, 1, 200), (1, 1, 1e7), (1e4, 1e-4, 1), (1e-3, 1e3, 1),
                                   (1e-30, 1, 1), (1, 1, 1e36)])
def test_magnitudes(heads, gains):
    q, k, v = inputs(heads, 1500, gains)
    O = nan_like(q)
    grat.grat_dense_attention_fwd(q, k, v, 1.0 / math.sqrt(D), out=O)
    assert errors(to_f64(O), reference(q, k, v))[1] <= 2e-5


@pytest.mark.parametrize("heads", [2, 8, 12])
def test_special_values(heads):
    """One head of huge scores, one with an infinity in V, one with an infinity in K; the others as ever."""
    q, k, v = inputs(heads, 1500, (1, 1, 1))
    k[0, 0, 700, 0] = -1e30
    v[0, 1, 900, 5] = math.inf
    want = reference(q, k, v)
    O = to_f64(grat.grat_dense_attention_fwd(q, k, v, 1.0 / math.sqrt(D)))
    assert np.isposinf(O[0, 1, :, 5]).all() and np.isposinf(want[0, 1, :, 5]).all()
    O[0, 1, :, 5] = want[0, 1, :, 5] = 0.0
    assert errors(O, want)[1] <= 2e-5
    k[0, 0] = 1.0
    q[0, 0] = 1.0
    k[0, 0, 1000, 3] = -math.inf   # this key weighs nothing, the others all the same
    O = to_f64(grat.grat_dense_attention_fwd(q, k, v, 1.0 / math.sqrt(D)))
    mean = np.delete(to_f64(v)[0, 0], 1000, axis=0).mean(0)
    assert np.abs(O[0, 0] - mean).max() <= 1e-5


# Where an infinity of V meets the padding of a key tile: sequences and groups that end inside a tile, the infinity in
# their first or last token.  (1500 = 46 * 32 + 28 = 93 * 16 + 12 tokens; groups of 3 x 11 and, clipped, 3 x 7 tokens;
# of 5 x 3 and, clipped, fewer; of 7 x 9, whose workgroups own 64 queries.)  heads: either side of the launch size from
# which waves own 32 queries.
@pytest.mark.parametrize("heads,d", [(2, 128), (12, 128), (16, 64)])
@pytest.mark.parametrize("grid,group", [((1500,), None), ((33, 62), (3, 11)), ((33, 35), (5, 3)), ((33, 62), (7, 9))])   # None: dense
@pytest.mark.parametrize("last", [True, False])
def test_infinity_beside_padding(grid, group, last, heads, d):
    n = math.prod(grid)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5310)
    q, k, v = (torch.randn(1, heads, n, d, generator=gen, device="cuda") for _ in range(3))
    first = (0,) if group is None else tuple((t - 1) // g * g for t, g in zip(grid, group))   # of the last group
    token = n - 1 if last else int(np.ravel_multi_index(first, grid))
    v[0, :, token, 5] = math.inf
    if group is None:
        O = grat.grat_dense_attention_fwd(q, k, v, 1.0 / math.sqrt(d))
        sees = np.ones(n, dtype=bool)
    else:
        count, index = grat.grat_build_block_lists(grid, group, "block", (1, 1))
        O = grat.grat_attention_fwd(q, k, v, 1.0 / math.sqrt(d), grid, group, count, index)
        sees = orc.mask_rows(np.arange(n), grid, group, "block", (1, 1))[:, token]
    O = to_f64(O)
    assert np.isposinf(O[0, :, sees, 5]).all()
    O[0, :, sees, 5] = 0.0
    assert np.isfinite(O).all()


def channel_errors(got, want):
    """worst relative L2 error of a head dim of a head"""
    return float((np.linalg.norm(got - want, axis=2) / np.linalg.norm(want, axis=2)).max())


# Small numbers beside large ones keep the accuracy of fp32, each of them: one head dim in four is as ever, the others
# are scaled.  Bound: as above for the scores; a weighted sum is as accurate relative to its own head dim's values.
@pytest.mark.parametrize("heads", [2, 12])
@pytest.mark.parametrize("small", [1e-3, 1e-6, 1e-10, 1e-20, 1e-30, 1e-36])
def test_head_dims_of_their_own_magnitude_in_v(heads, small):
    q, k, v = inputs(heads, 1500, (1, 1, 1), 5400)
    gain = torch.full((D,), small, device="cuda")
    gain[::4] = 1.0
    v = v * gain
    O = to_f64(grat.grat_dense_attention_fwd(q, k, v, 1.0 / math.sqrt(D)))
    assert channel_errors(O, reference(q, k, v)) <= 2e-5


@pytest.mark.parametrize("heads", [2, 12])
@pytest.mark.parametrize("gain", [1e3, 1e5, 1e7, 1e9, 1e12])
@pytest.mark.parametrize("big", ["q", "k"])
def test_head_dims_of_their_own_magnitude_in_scores(heads, gain, big):
    """Q large and K small in one head dim of four (or the other way round): the same scores but for roundings."""
    q, k, v = inputs(heads, 1500, (1, 1, 1), 5401)
    f = torch.ones(D, device="cuda")
    f[::4] = gain
    q, k = (q * f, k / f) if big == "q" else (q / f, k * f)
    O = to_f64(grat.grat_dense_attention_fwd(q, k, v, 1.0 / math.sqrt(D)))
    assert channel_errors(O, reference(q, k, v)) <= 2e-5


@pytest.mark.parametrize("heads", [2, 12])
def test_tokens_of_their_own_magnitude_in_v(heads):
    """Half the queries attend (all but) nothing but tokens whose values are a millionth of the others'."""
    q, k, v = inputs(heads, 1500, (1, 1, 1), 5402)
    q[:, :, 0::2, 0], q[:, :, 1::2, 0] = 60.0, -60.0
    k[:, :, 0::2, 0], k[:, :, 1::2, 0] = 12.0, -12.0
    v[:, :, 0::2] *= 1e-6
    O, want = to_f64(grat.grat_dense_attention_fwd(q, k, v, 1.0 / math.sqrt(D))), reference(q, k, v)
    for rows in (slice(0, None, 2), slice(1, None, 2)):
        assert errors(O[:, :, rows], want[:, :, rows])[1] <= 2e-5


@pytest.mark.parametrize("heads", [2, 12])
@pytest.mark.parametrize("scale", [1e-37, 1e-25, 1e25, 1e37])
def test_scales(heads, scale):
    """Scales far from 1 (and, where they are large, queries that make up for it), a tile end inside the sequence."""
    q, k, v = inputs(heads, 1500, (1e-20 if scale < 1 else 0.1 / scale, 1, 1), 5403)
    O = to_f64(grat.grat_dense_attention_fwd(q, k, v, scale))
    q, k, v = (t[0].double().cpu() for t in (q, k, v))
    want = torch.stack([torch.softmax(a @ b.t() * float(np.float32(scale)), -1) @ c for a, b, c in zip(q, k, v)])[None].numpy()
    assert errors(O, want)[1] <= 2e-5


@pytest.mark.parametrize("heads,v_gain", [(2, 1e36), (12, 1e36)])   # (the second: the walk on the fp32 instructions)
def test_weights_below_the_normal_range(heads, v_gain):
    """One token has all but 2^-120 of the weight and no value, the others weigh 2^-130 each.  Bound: their exponent, 130, is
    rounded twice (2^-17 each, times ln 2) and the weight has 19 bits left: 1.3e-5."""
    q, k, v = inputs(heads, 1500, (0, 0, v_gain), 5404)
    q[..., 0], k[..., 0] = 10.0, -13.0 / math.log2(math.e)
    k[:, :, 700], v[:, :, 700] = 0.0, 0.0
    O = to_f64(grat.grat_dense_attention_fwd(q, k, v, 1.0))
    q, k, v = (t[0].double().cpu() for t in (q, k, v))
    want = torch.stack([torch.softmax(a @ b.t(), -1) @ c for a, b, c in zip(q, k, v)])[None].numpy()
    assert errors(O, want)[1] <= 2e-5
