"""Helpers for the GPU parity tests: move seeded workloads to the device, run the C-ABI
path through the binding, run the CPU oracle per head, compare."""
from __future__ import annotations

from math import sqrt
from typing import Dict, Iterable, Optional

import numpy as np
import torch

from bsa_workloads import Workload, bf16_round, head_inputs, head_tensor
from oracle import bsa_oracle as o
from paper_2509_01085_amd import binding as B

import bench
import tolerance as T

# Deciding comparisons closer to equality than this (relative to the row's total mass) are
# within reach of the one non-reproducible step (exp of libm vs the device, summation tree
# of the scan): such a row may legitimately differ by its boundary block.
SELECT_MARGIN = 1e-10


def progress(msg: str) -> None:
    """Progress line of a long test: stdout (visible with -s) and a log file in the run's output
    folder, so that a run whose output pytest captures is still seen to be alive."""
    import os
    import time

    print(msg, flush=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    try:
        os.makedirs(os.path.join(root, "gpurun_out"), exist_ok=True)
        with open(os.path.join(root, "gpurun_out", "test_progress.log"), "a") as f:
            f.write(f"{time.strftime('%H:%M:%S')} {msg}\n")
    except OSError:
        pass


def shape_of(wl: Workload) -> B.Shape:
    return B.Shape(wl.B, wl.H, *wl.grid, *wl.block, wl.d, B.F32 if wl.dtype == "fp32" else B.BF16, *wl.window, int(wl.block_major))


def part_of(wl: Workload) -> o.Partition:
    return o.Partition(*wl.grid, *wl.block, *wl.window, wl.block_major)


def device_inputs(wl: Workload, names=("Q", "K", "V", "dO"), heads: Optional[Iterable[int]] = None) -> Dict[str, torch.Tensor]:
    """[B,H,L,d] device tensors of the workload's dtype (heads not listed stay zero)."""
    dt = torch.float32 if wl.dtype == "fp32" else torch.bfloat16
    out = {}
    for name in names:
        host = torch.zeros((wl.B, wl.H, wl.L, wl.d), dtype=dt)
        for b in range(wl.B):
            for h in (range(wl.H) if heads is None else heads):
                host[b, h] = torch.from_numpy(head_tensor(wl, name, b, h)).to(dt)  # exact: values are bf16 already
        out[name] = host.cuda()
    return out


def run_indices(wl: Workload, x: Dict[str, torch.Tensor], threshold=None, keep_ratio=None):
    shp = shape_of(wl)
    Qbar = B.pool_blocks(shp, x["Q"])
    Kbar = B.pool_blocks(shp, x["K"])
    lists = B.select_kv(shp, Qbar, Kbar, wl.threshold if threshold is None else threshold)
    keep = B.prune_q(shp, x["Q"], wl.keep_ratio if keep_ratio is None else keep_ratio)
    return shp, Qbar, Kbar, lists, keep


def lists_to_host(shp: B.Shape, lists: B.KvLists):
    torch.cuda.synchronize()
    nnz = int(lists.nnz.item())
    q2k_ptr = lists.q2k_ptr.cpu().numpy()
    assert q2k_ptr[-1] == nnz
    return dict(q2k_ptr=q2k_ptr, q2k_idx=lists.q2k_idx[:nnz].cpu().numpy(),
                k2q_ptr=lists.k2q_ptr.cpu().numpy(), k2q_idx=lists.k2q_idx[:nnz].cpu().numpy(), nnz=nnz)


def head_csr(host: dict, shp: B.Shape, b: int, h: int, which="q2k"):
    """Slice one head's CSR out of the all-rows CSR, rebased to start at 0."""
    r0 = (b * shp.H + h) * shp.N
    ptr = host[which + "_ptr"][r0:r0 + shp.N + 1]
    return (ptr - ptr[0]).astype(np.int32), host[which + "_idx"][ptr[0]:ptr[-1]]


def check_lists_against_oracle(wl: Workload, shp: B.Shape, host: dict, b: int, h: int, ix: o.HeadResult, scores=None):
    """Bit-exact CSR and transposed CSR; a row may differ only if its margin is below SELECT_MARGIN."""
    ptr, idx = head_csr(host, shp, b, h, "q2k")
    if np.array_equal(ptr, ix.q2k_ptr) and np.array_equal(idx, ix.q2k_idx):
        tptr, tidx = head_csr(host, shp, b, h, "k2q")
        assert np.array_equal(tptr, ix.k2q_ptr) and np.array_equal(tidx, ix.k2q_idx)
        return 0
    assert scores is not None, "lists differ from the oracle"
    bad = 0
    for i in range(shp.N):
        mine = idx[ptr[i]:ptr[i + 1]]
        ref = ix.q2k_idx[ix.q2k_ptr[i]:ix.q2k_ptr[i + 1]]
        if not np.array_equal(mine, ref):
            sel = o.select_row(scores[i], wl.threshold)
            assert sel.margin < SELECT_MARGIN, (i, sel.margin)
            assert abs(len(mine) - len(ref)) == 1 and len(np.setxor1d(mine, ref)) == 1
            bad += 1
    return bad


def split_plan(N: int, BH: int, n_keep: int):
    """The host-side plan of the forward and dQ launches, restated: (kind, segments, units of a head, the units whose
    walk is split).  A unit is a group of 4 query blocks (8 when n_keep <= 16); XCD x owns the contiguous range
    [x*q + min(x, r), ...) of q or q + 1 units (q, r = divmod(units, 8)).  From 40 units up, "all": no more than half of
    the chip's slots and at least 32 blocks, every unit is split; else "tail": shorter than 12 rounds of slots, the
    last n = ceil(q / 5) of every XCD in four."""
    pg = 8 if n_keep <= 16 else 4
    groups = -(-N // pg)
    units = groups * BH
    q, r = divmod(units, 8)
    slots = 256 * (1 if n_keep > 32 else 2)
    if q < 5 or not (2 * units <= slots and N >= 32 or units < 12 * slots):
        return "none", 1, groups, []
    if 2 * units <= slots and N >= 32:
        return "all", min(slots // units, 8, N // 8), groups, list(range(units))
    n, out = (q + 4) // 5, []
    for x in range(8):
        end = x * q + min(x, r) + q + (1 if x < r else 0)
        out.extend(range(end - n, end))
    return "tail", 4, groups, out


def forward_route(N: int, BH: int, n_keep: int, d: int) -> str:
    """Which of the two bf16 forward kernels a sparse call launches: "walk" (bsa_attn_fwd.hip), "pipe" (bsa_attn_pipe.hip) or
    "both", where the lists' mean length decides on the device."""
    return bench.forward_route(N, BH, n_keep, d)[0]


unit_blocks = bench.unit_blocks


def walk_split(N: int, BH: int, n_keep: int):
    """Segments of the split units of "walk", and these: the last ones of every XCD, where there is more than a round of
    units and the workspace of "pipe" has room: what is more than a round in four, or every twelfth in two."""
    _, units = unit_blocks(N, BH, n_keep)
    kind, S, groups, _ = split_plan(N, BH, n_keep)
    q, r = divmod(groups * BH, 8)
    room = 8 * {"none": 0, "tail": (q + 4) // 5, "all": q + (r > 0)}[kind] * S * (2 if n_keep > 32 else 1)
    q, r = divmod(units, 8)
    over = q + (r > 0) - 32
    n, S = (over, 4) if 0 < over < 32 and 32 * over <= room else (-(-q // 12), 2)
    if units <= 256 or 8 * n * S > room:
        return 1, []
    return S, [u for x in range(8) for end in [x * q + min(x, r) + q + (x < r)] for u in range(end - min(n, q + (x < r)), end)]


def rel_err(got: np.ndarray, ref: np.ndarray) -> float:
    """max |got - ref| / RMS(ref): the plain tolerance metric."""
    return T.figures(got, ref)["plain"]


def record(case: str, where: str, figs: dict) -> None:
    """Append the parity figures of one comparison to the run's figure log (one JSON line)."""
    import json
    import os

    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    try:
        os.makedirs(os.path.join(root, "gpurun_out"), exist_ok=True)
        with open(os.path.join(root, "gpurun_out", "parity_figures.jsonl"), "a") as f:
            f.write(json.dumps({"case": case, "where": where, **figs}) + "\n")
    except OSError:
        pass


def check_tensors(case: str, where: str, dtype: str, pairs, sigma=None, lse=None) -> dict:
    """Hold every (name, got, ref) of `pairs` to the criteria of tests/tolerance.py; `sigma`: the
    operand-rounding model's standard deviations for the bf16 gradients; `lse` = (got, ref).
    The figures are logged whether or not they pass.  Returns them."""
    figs, bad = {}, []
    for name, got, ref in pairs:
        sg = (sigma or {}).get(name) if dtype == "bf16" and name != "O" else None  # O: no operand term
        if dtype == "bf16" and name != "O":
            assert sg is not None, f"no rounding model for {name}"
        f = T.figures(got, ref, sg)
        bad += T.failures(name, f, dtype)
        figs[name] = {k: float(f"{v:.3e}") for k, v in f.items()}
    if lse is not None:
        figs["LSE"] = {"abs": float(f"{np.abs(np.asarray(lse[0], dtype=np.float64) - lse[1]).max():.3e}")}
        if not figs["LSE"]["abs"] <= T.TOL_LSE:
            bad.append(f"LSE: max-abs {figs['LSE']['abs']:.3e} > {T.TOL_LSE}")
    record(case, where, figs)
    assert not bad, (case, where, bad, figs)
    return figs


def o_storage_of(wl: Workload):
    """How the forward output is stored before the backward reads it back (None: exactly)."""
    if wl.dtype == "fp32":
        return lambda O: np.asarray(O, dtype=np.float32)
    return lambda O: bf16_round(np.asarray(O, dtype=np.float32))


def host_f64(t: torch.Tensor) -> np.ndarray:
    return t.detach().to(torch.float64).cpu().numpy()
