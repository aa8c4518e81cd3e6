"""The native part of the binding takes ordinary calls only; all others go the long way and come to the same."""
import sys

import numpy as np
import pytest
import torch

import paper_2505_14687_amd as grat
from paper_2505_14687_amd import build
from paper_2505_14687_amd import grat as binding
from paper_2505_14687_amd.build import BINDING_PATH

GRID, GROUP = (32, 32), (8, 8)


def test_what_is_not_ordinary_is_left_alone():
    grat.lib()
    n = binding._native
    x = torch.zeros(1, 2, 1024, 64)
    cnt, idx = torch.zeros(16, dtype=torch.int32), torch.zeros(16, 9, dtype=torch.int32)
    assert n.attention(x, x, x, 0.1, None, True, GRID, GROUP, cnt, idx, None, None) is None       # host tensors
    assert n.attention(None, x, x, 0.1, None, True, GRID, GROUP, cnt, idx, None, None) is None
    assert n.dense(x, x, x, 0.1, None, None) is None
    assert n.dense(x, x, x, "0.1", None, None) is None
    assert n.packed(torch.zeros(1, 1024, 3, 2, 64), 0.1, 0, True, GRID, GROUP, cnt, idx, None, None) is None
    assert n.block_lists(GRID, (8,), 0, (1, 1), None) is None
    assert n.block_lists(GRID, GROUP, 9, (1, 1), None) is None
    assert n.block_lists((1,) * 4, (1,) * 4, 3, None, None) is None
    with pytest.raises(TypeError):
        n.dense(x)


class Sub(torch.Tensor):
    pass


@pytest.mark.gpu
def test_both_ways_give_the_same_and_refuse_the_same():
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    q, k, v = (torch.randn(1, 2, 1024, 64, generator=g, device="cuda") for _ in range(3))
    cnt, idx = grat.grat_build_block_lists(GRID, GROUP, "block", (1, 1))
    c2, i2 = grat.grat_build_block_lists(np.array(GRID), GROUP, "block", (1, 1), device="cuda:0")   # the long way
    assert torch.equal(cnt, c2) and torch.equal(idx, i2)
    ints = [np.int64(t) for t in GRID]
    want = grat.grat_attention_fwd(q, k, v, 0.125, ints, GROUP, cnt, idx)                           # the long way
    assert binding._native.attention(q, k, v, 0.125, None, True, ints, GROUP, cnt, idx, None, None) is None
    n, qkv = binding._native, torch.randn(1, 1024, 3, 2, 64, generator=g, device="cuda")
    for r in (n.attention(q, k, v, 0.125, None, True, GRID, GROUP, cnt, idx, None, None), n.dense(q, k, v, 0.125, None, None),
              n.packed(qkv, 0.125, 0, True, GRID, GROUP, cnt, idx, None, None), n.block_lists(GRID, GROUP, 0, (1, 1), None)[0]):
        assert isinstance(r, torch.Tensor)                                                          # ordinary calls
    got = grat.grat_attention_fwd(q, k, v, 0.125, GRID, GROUP, cnt, idx)
    assert torch.equal(got, want) and got.stride() == want.stride()
    out = torch.full_like(q, float("nan"))
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    assert grat.grat_attention_fwd(q, k, v, 0.125, list(GRID), GROUP, cnt, idx, out=out, stream=s) is out
    s.synchronize()
    assert torch.equal(out, want)
    sub = q.as_subclass(Sub)
    assert type(grat.grat_dense_attention_fwd(sub, sub, sub, 0.125)) is Sub
    assert torch.equal(grat.grat_dense_attention_fwd(sub, sub, sub, 0.125).as_subclass(torch.Tensor),
                       grat.grat_dense_attention_fwd(q, q, q, 0.125))
    t = q.transpose(1, 2).contiguous().transpose(1, 2)
    assert grat.grat_dense_attention_fwd(t, t, t, 0.125).stride() == t.stride()
    for bad in (lambda: grat.grat_attention_fwd(q, k, t, 0.1, GRID, GROUP, cnt, idx),
                lambda: grat.grat_attention_fwd(q, k, v, 0.1, (32, 64), GROUP, cnt, idx),
                lambda: grat.grat_attention_fwd(q, k, v, 0.1, GRID, GROUP, cnt.cpu(), idx),
                lambda: grat.grat_attention_fwd(q, k, v.double(), 0.1, GRID, GROUP, cnt, idx),
                lambda: grat.grat_dense_attention_fwd(q, k, v, 0.1, out=torch.empty_like(t))):
        with pytest.raises(ValueError):
            bad()
    with pytest.raises(grat.GratError) as e:
        grat.grat_attention_fwd(q, k, v, -1.0, GRID, GROUP, cnt, idx)
    assert e.value.status == 2
    with pytest.raises(grat.GratError) as e:
        grat.grat_build_block_lists(GRID, GROUP, "block", (1, -1))
    assert e.value.status == 2
    with pytest.raises(grat.GratError):
        grat.grat_build_block_lists(GRID, GROUP, "block", (1, 1), max_kv=3)


@pytest.fixture(params=["file missing", "cannot be loaded"])
def without_native(request, monkeypatch):
    """libgrat.so there, _binding.so not built (no host compiler) or built for another torch."""
    grat.lib()
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_native", None)
    if request.param == "file missing":
        monkeypatch.setattr(binding, "BINDING_PATH", binding.BINDING_PATH + ".not-there")
    else:
        monkeypatch.setitem(sys.modules, "paper_2505_14687_amd._binding", None)


def test_without_the_native_part_calls_go_the_long_way(without_native):
    with pytest.warns(RuntimeWarning, match="_binding"):
        assert grat.grat_block_list_shape(GRID, GROUP, "block", (1, 1)) == (16, 9)
    x = torch.zeros(1, 2, 1024, 64)
    cnt, idx = torch.zeros(16, dtype=torch.int32), torch.zeros(16, 9, dtype=torch.int32)
    for call in (lambda: grat.grat_attention_fwd(x, x, x, 0.1, GRID, GROUP, cnt, idx),
                 lambda: grat.grat_attention_global_fwd(x, x, x, 0.1, 0, True, GRID, GROUP, cnt, idx),
                 lambda: grat.grat_dense_attention_fwd(x, x, x, 0.1),
                 lambda: grat.grat_attention_packed_fwd(torch.zeros(1, 1024, 3, 2, 64), 0.1, GRID, GROUP, cnt, idx)):
        with pytest.raises(ValueError, match="device memory"):
            call()


@pytest.mark.gpu
def test_without_the_native_part_results_are_the_same(without_native):
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    q, k, v = (torch.randn(1, 2, 1024, 64, generator=g, device="cuda") for _ in range(3))
    with pytest.warns(RuntimeWarning, match="_binding"):
        cnt, idx = grat.grat_build_block_lists(GRID, GROUP, "block", (1, 1))
    got = grat.grat_attention_fwd(q, k, v, 0.125, GRID, GROUP, cnt, idx), grat.grat_dense_attention_fwd(q, k, v, 0.125)
    binding._lib = None   # (the fixture puts everything back)
    sys.modules.pop("paper_2505_14687_amd._binding", None)
    binding.BINDING_PATH = BINDING_PATH
    c2, i2 = grat.grat_build_block_lists(GRID, GROUP, "block", (1, 1))
    assert isinstance(binding._native.dense(q, k, v, 0.125, None, None), torch.Tensor)
    want = grat.grat_attention_fwd(q, k, v, 0.125, GRID, GROUP, cnt, idx), grat.grat_dense_attention_fwd(q, k, v, 0.125)
    assert torch.equal(cnt, c2) and torch.equal(idx, i2) and all(torch.equal(a, b) for a, b in zip(got, want))


def test_a_failed_build_step_names_its_compiler():
    with pytest.raises(RuntimeError, match="false failed"):
        build._run(["/bin/false"], False)
