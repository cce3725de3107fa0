"""The bf16 forward with a barrier a tile (bsa_attn_pipe.hip) where it is the one that works: more than a round of the other
one's units, and short lists.  Whole walks and segments that the combine launch of both kernels merges; empty lists, lists
that begin with, and segments that hold nothing but, blocks of -inf logits; windows; both token orders."""
from math import sqrt

import numpy as np
import pytest
import torch

from bsa_workloads import Workload
from oracle import bsa_oracle as o
from paper_2509_01085_amd import binding as B

import gpu_util as U

pytestmark = pytest.mark.gpu

# heads, blocks of a head, d, share of queries kept; both: the other kernel is launched, too, and ends at once
SIZES = [(4, 323, 128, 0.5, True), (2, 259, 128, 1.0, True), (2, 257, 64, 1.0, True), (11, 197, 128, 0.25, True),
         (15, 70, 64, 0.5, False), (12, 65, 64, 1.0, False), (28, 74, 64, 0.25, False), (12, 89, 128, 0.5, False)]


def some_lists(H, N, rng):
    """Empty ones, one to five blocks, a run of even ones (-inf below) ahead of an odd one; the same for four rows or not."""
    rows = []
    for i in range(H * N):
        k = (0, 1, 3, 5, 2, 9, 4)[(i // 3) % 7]
        r = rng.choice(N, size=k, replace=False)
        if k == 9:
            r = np.append(2 * np.arange(8), N - 1 - N % 2)  # eight blocks of -inf, then an odd one
        if k and not (r % 2).any():
            r[0] += 1 if r[0] + 1 < N and r[0] + 1 not in r else -1
        rows.append(np.unique(r))
    return rows


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("H,N,d,keep_ratio,both", SIZES)
def test_short_lists(H, N, d, keep_ratio, both, masked):
    U.progress(f"short lists H={H} N={N} d={d} r={keep_ratio} masked={masked}")
    wl = Workload(f"short_{H}_{N}_{d}_{keep_ratio}_{masked}", 1, H, d, "bf16", (4, 4, 4 * N), (4, 4, 4), keep_ratio=keep_ratio,
                  window=(2, 2, 2) if masked else (0, 0, 0), block_major=masked)
    part, shp = U.part_of(wl), U.shape_of(wl)
    nk = part.n_keep(keep_ratio)
    assert U.forward_route(N, H, nk, d) == ("both" if both else "pipe")
    kind, S, groups, units = U.split_plan(N, H, nk)
    assert kind == "tail"
    heads = [0, units[0] // groups, H - 1]
    x = U.device_inputs(wl, ("Q", "K", "V"), heads=heads)
    Q, K = x["Q"], x["K"]
    Q[..., 0] = Q[..., 0].abs() + 0.5
    tok = part.block_tokens()
    if masked:
        K[:, :, torch.from_numpy(tok[::2].reshape(-1)).cuda(), 0] = float("-inf")
    rows = some_lists(H, N, np.random.default_rng(N))
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    ptr, idx = np.cumsum([0] + [len(r) for r in rows]), np.concatenate(rows)
    lists = B.KvLists(i32(ptr), i32(idx), i32(ptr), i32(idx), torch.tensor([len(idx)], device="cuda"), torch.empty(1, dtype=torch.uint8, device="cuda"))
    keep = B.prune_q(shp, Q, keep_ratio)
    O, LSE = B.attn_fwd(shp, Q, K, x["V"], lists, keep)
    assert any(u // groups in heads for u in units)
    for h in sorted(set(heads)):
        mine = rows[h * N:(h + 1) * N]
        p, ix = np.cumsum([0] + [len(r) for r in mine]), np.concatenate(mine)
        pg = 8 if nk <= 16 else 4
        split = [b for u in units if u // groups == h for b in range(u % groups * pg, min(N, u % groups * pg + pg))]
        blocks = sorted({0, 1, 2, N // 2, N - 2, N - 1, *range(15, 21), *split[:16]} & set(range(N)))
        full = [i for i in blocks if len(mine[i])]
        sel = tok[full].reshape(-1)
        rO, rL = o.attn_fwd(*[U.host_f64(t[0, h]) for t in (Q, K, x["V"])], part, p, ix, keep[0, h].cpu().numpy(), 1 / sqrt(d), q_blocks=full)
        U.check_tensors(wl.name, f"h{h}", "bf16", [("O", U.host_f64(O[0, h])[sel], rO[sel])], lse=(U.host_f64(LSE[0, h])[sel], rL[sel]))
        for i in set(blocks) - set(full):
            t = torch.from_numpy(tok[i]).cuda()
            assert (O[0, h, t] == 0).all() and (LSE[0, h, t] == float("-inf")).all(), (h, i)
