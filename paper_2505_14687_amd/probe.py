"""The probes of libgrat (grat_probe.h): the MFMA-only loop with the checksum its sink must show, and what an attention call
would launch.  Measurement aids for benchmarks and tests, not part of the attention path."""
from __future__ import annotations

import ctypes
from typing import Optional, Sequence

import numpy as np
import torch

from .grat import DTYPES, GRAT_OK, GratError, _ivec, _stream_ptr, lib

PROBE_DATA = {"ones": 0, "small_ints": 1, "normal_like": 2}


def grat_probe_mfma(dtype, data, blocks: int, iters: int, sink=None, stream=None):
    """One launch of the MFMA-only loop (grat_probe.h) on operands of kind `data` ("ones",
    "small_ints", "normal_like" or 0..2); returns the sink tensor [blocks * 256] int64."""
    if sink is None:
        sink = torch.empty(int(blocks) * 256, dtype=torch.int64, device="cuda")
    if sink.dtype != torch.int64 or not sink.is_contiguous() or sink.numel() < int(blocks) * 256:
        raise ValueError("sink: contiguous int64, at least blocks * 256 elements")
    kind = PROBE_DATA[data] if isinstance(data, str) else int(data)
    st = lib().grat_probe_mfma(DTYPES[dtype], kind, sink.data_ptr(), int(blocks), int(iters), _stream_ptr(stream))
    if st != GRAT_OK:
        raise GratError(st, "grat_probe_mfma")
    return sink


def probe_wave_sum(data, iters: int) -> int:
    """What the 64 sink values of one wave add up to (grat_probe.h)."""
    kind = PROBE_DATA[data] if isinstance(data, str) else int(data)
    if kind == 0:
        return 4 * 2 * 32 * 32 * 16 * int(iters)
    l = np.arange(64)[:, None]
    e = np.arange(8)[None, :]

    def matrix(values):   # [lane, e] -> M[l % 32][8 (l // 32) + e]
        M = np.zeros((32, 16), dtype=np.int64)
        for lane in range(64):
            M[lane % 32, 8 * (lane // 32):8 * (lane // 32) + 8] = values[lane]
        return M

    total = 0
    for v in ((0, 1, 2, 3) if kind == 1 else (3,)):
        A = matrix(((37 + 2 * v) * l + 11 * e + 5 + 3 * v) % 9 - 4)
        B = matrix(((53 + 2 * v) * l + 17 * e + 2 + 3 * v) % 9 - 4).T
        total += 2 * int((A @ B).sum())
    return total * int(iters)


class LaunchInfo(ctypes.Structure):
    """grat_launch_info"""
    _fields_ = [(n, ctypes.c_int32) for n in ("mode", "rows", "teams", "tile_keys", "whole_tiles", "key_waves", "longest_first",
                                              "tiles", "xcd_tiles")]


def grat_probe_launch(dtype, batch: int, heads: int, head_dim: int, grid: Optional[Sequence[int]] = None,
                      group: Optional[Sequence[int]] = None, max_kv: int = 0, n_global: int = 0) -> LaunchInfo:
    """What an attention call with these sizes launches (host only).  Without a grid: a dense call over n_global tokens."""
    info = LaunchInfo()
    st = lib().grat_probe_launch(DTYPES[dtype], batch, heads, head_dim, n_global, len(grid) if grid else 0, _ivec(grid), _ivec(group),
                                 max_kv, ctypes.byref(info))
    if st != GRAT_OK:
        raise GratError(st, "grat_probe_launch")
    return info


def launched_kernel(dtype, batch: int, heads: int, head_dim: int, grid: Optional[Sequence[int]] = None,
                    group: Optional[Sequence[int]] = None, max_kv: int = 0, n_global: int = 0) -> str:
    """The same as the name of a kernel with its template arguments.  attn_mfma_kernel and attn_mfma_teams_kernel: waves of a
    team, keys of an LDS tile, mode, half?, head_dim (, teams); the fp32 kernels: head_dim, dense?, waves."""
    i = grat_probe_launch(dtype, batch, heads, head_dim, grid, group, max_kv, n_global)
    if dtype == torch.float32:
        name, waves = ("attn_f32_split_kernel", i.key_waves) if i.rows == 16 else ("attn_f32_kernel", i.rows // 32)
        return "grat::%s<%d, %s, %d>" % (name, head_dim, "true" if i.mode == 1 else "false", waves)
    half = "true" if dtype == torch.float16 else "false"
    if i.whole_tiles:
        return "grat::attn_mfma_mixed_kernel<%s>" % half
    args = "%d, %d, %d, %s, %d" % (i.rows // 32, i.tile_keys, i.mode, half, head_dim)
    return "grat::attn_mfma_teams_kernel<%s, %d>" % (args, i.teams) if i.teams > 1 else "grat::attn_mfma_kernel<%s>" % args
