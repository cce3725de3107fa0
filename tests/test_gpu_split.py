"""dQ launches, and those of the forward with a barrier a tile, whose walks are split over several workgroups, all of them
or the last ones of every XCD, against the oracle: both plans with every variant of the kernels (the forward's of two tiles a block
only where the last ones are split), unit counts that leave a remainder of eight, ragged last groups, and lists so short that a walk has
fewer segments than the plan or segments without a tile.  (Walks that the other forward splits: test_gpu_fwd_walk.py.)"""
from math import sqrt

import numpy as np
import pytest
import torch

from bsa_workloads import Workload, head_inputs
from oracle import bsa_oracle as o
from paper_2509_01085_amd import binding as B

import gpu_util as U

pytestmark = pytest.mark.gpu


def case(H, N, d, keep_ratio, window=(0, 0, 0)):
    return Workload(f"split_{H}_{N}_{d}_{keep_ratio}", 1, H, d, "bf16", (4, 8, 2 * N), (4, 4, 4), threshold=0.7, keep_ratio=keep_ratio,
                    window=window)


CASES = {  # heads, blocks of a head, d, share of queries kept -> the plan and its segments
    "all_one": (case(5, 38, 128, 0.5), "all", 4),               # 50 units
    "all_one_fwd": (case(12, 44, 128, 0.5), "all", 3),          # 132 units, the forward's, too
    "all_pack_fwd": (case(12, 46, 64, 0.25), "all", 5),         # 72 units of eight blocks, the forward's, too
    "all_two": (case(5, 32, 64, 1.0), "all", 4),                # 40 units
    "all_pack": (case(9, 38, 64, 0.25, (2, 2, 2)), "all", 4),   # 45 units of eight blocks
    "all_long": (case(4, 64, 128, 0.5, (2, 2, 2)), "all", 8),   # 64 units
    "tail_two": (case(15, 36, 64, 0.75), "tail", 4),            # 135 units, more than half of 256 slots
    "tail_two_d128": (case(21, 12, 128, 1.0), "tail", 4),       # 63 units of a few blocks
    "tail_one": (case(29, 36, 64, 0.5), "tail", 4),             # 261 units, more than half of 512 slots
    "tail_pack": (case(53, 36, 128, 0.25), "tail", 4),          # 265 units
    "whole": (case(3, 48, 64, 0.5), "none", 1),                 # 36 units
}


def short_lists(N, rng):
    """Groups of rows that list one block, the same one or each its own; two or three; many."""
    rows = []
    for i in range(N):
        k = (1, 1, 3, N - 1, 2)[(i // 4) % 5]
        rows.append(np.sort(rng.choice(N, size=k, replace=False)) if (i // 4) % 5 else np.array([(i // 4) % N]))
    return rows


@pytest.mark.parametrize("lists", ["selected", "short"])
@pytest.mark.parametrize("name", list(CASES))
def test_split_walks(name, lists):
    wl, kind, segments = CASES[name]
    U.progress(f"split {name} {lists}")
    shp, part, scale = U.shape_of(wl), U.part_of(wl), 1 / sqrt(wl.d)
    N, H, nk = shp.N, wl.H, part.n_keep(wl.keep_ratio)
    got_kind, S, groups, units = U.split_plan(N, H, nk)
    assert (got_kind, S) == (kind, segments)
    assert U.forward_route(N, H, nk, wl.d) == ("pipe" if kind == "tail" or name.endswith("fwd") else "walk")
    split_heads = sorted({u // groups for u in units})
    heads = sorted({0, H - 1} | ({split_heads[0], split_heads[len(split_heads) // 2]} if kind == "tail" else set()))
    assert kind != "tail" or any(u // groups in heads for u in units)
    x = U.device_inputs(wl, heads=heads)
    if lists == "selected":
        _, _, _, kv, keep = U.run_indices(wl, x)
    else:
        rows = [r for h in range(H) for r in short_lists(N, np.random.default_rng(h))]
        cols = [r for h in range(H) for r in np.split(*_transposed(rows[h * N:(h + 1) * N], N))]
        i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
        ends = lambda l: np.cumsum([0] + [len(r) for r in l])
        kv = B.KvLists(i32(ends(rows)), i32(np.concatenate(rows)), i32(ends(cols)), i32(np.concatenate(cols)),
                       torch.tensor([len(np.concatenate(rows))], device="cuda"), torch.empty(1, dtype=torch.uint8, device="cuda"))
        keep = B.prune_q(shp, x["Q"], wl.keep_ratio)
    O, LSE = B.attn_fwd(shp, x["Q"], x["K"], x["V"], kv, keep)
    dQ, dK, dV = B.attn_bwd(shp, x["Q"], x["K"], x["V"], O, LSE, x["dO"], kv, keep)
    host = U.lists_to_host(shp, kv)
    for h in heads:
        xi = head_inputs(wl, 0, h)
        ptr, idx = U.head_csr(host, shp, 0, h)
        kptr, kidx = U.head_csr(host, shp, 0, h, "k2q")
        keep_h = keep[0, h].cpu().numpy()
        assert np.array_equal(keep_h, o.prune_q(xi["Q"], part, wl.keep_ratio)[0])
        rO, rLSE = o.attn_fwd(xi["Q"], xi["K"], xi["V"], part, ptr, idx, keep_h, scale)
        rdQ, rdK, rdV = o.attn_bwd(xi["Q"], xi["K"], xi["V"], xi["dO"], part, ptr, idx, keep_h, scale, O_in=U.o_storage_of(wl)(rO))
        sigma = U.T.rounding_sigma(xi, part, o.HeadResult(None, None, ptr, idx, kptr, kidx, keep_h, 0.0, 0.0), scale)
        U.check_tensors(f"{wl.name} {lists}", f"h{h}", "bf16",
                        [(nm, U.host_f64(t[0, h]), ref) for nm, t, ref in (("O", O, rO), ("dQ", dQ, rdQ), ("dK", dK, rdK), ("dV", dV, rdV))],
                        sigma=sigma, lse=(U.host_f64(LSE[0, h]), rLSE))


def _transposed(rows, N):
    ptr, idx = o.transpose_csr(np.cumsum([0] + [len(r) for r in rows]), np.concatenate(rows), N)
    return idx, ptr[1:-1]
