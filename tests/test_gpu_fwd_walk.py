"""The bf16 matrix-core forward where its launches can go wrong: every number of query blocks that a unit can have, units
handed out by their length, unions longer than the list a workgroup keeps, row maxima that rise along a walk."""
from math import sqrt

import numpy as np
import pytest
import torch

from bsa_workloads import Workload
from oracle import bsa_oracle as o
from paper_2509_01085_amd import binding as B

import gpu_util as U

pytestmark = pytest.mark.gpu


def check(wl, x, shp, lists, keep, heads, blocks, K=None):
    K = x["K"] if K is None else K
    O, LSE = B.attn_fwd(shp, x["Q"], K, x["V"], lists, keep)
    part, host = U.part_of(wl), U.lists_to_host(shp, lists)
    sel = part.block_tokens()[blocks].reshape(-1)
    for h in heads:
        ptr, idx = U.head_csr(host, shp, 0, h)
        rO, rL = o.attn_fwd(*[U.host_f64(t[0, h]) for t in (x["Q"], K, x["V"])], part, ptr, idx, keep[0, h].cpu().numpy(),
                            1 / sqrt(wl.d), q_blocks=blocks)
        U.check_tensors(wl.name, f"h{h}", "bf16", [("O", U.host_f64(O[0, h])[sel], rO[sel])], lse=(U.host_f64(LSE[0, h])[sel], rL[sel]))


# heads, blocks of a head, share of queries kept -> query blocks of a unit.  0: more units than workgroups, handed out by length,
# and the last ones of every XCD split in two; -1: little more units than workgroups, what is more split in four (d = 128 there
# where a block has one tile or less: with d = 64 that is the other kernel's)
SIZES = [(3, 64, 0.5, 1), (7, 64, 0.5, 2), (4, 129, 0.5, 3), (5, 170, 0.5, 4), (8, 320, 0.5, 0), (4, 320, 0.5, -1),
         (3, 64, 1.0, 1), (5, 63, 1.0, 2), (5, 263, 1.0, 0), (2, 257, 1.0, -1),
         (5, 63, 0.25, 2), (5, 130, 0.25, 4), (10, 130, 0.25, 6), (14, 133, 0.25, 8), (14, 320, 0.25, 0), (11, 197, 0.25, -1)]


@pytest.mark.parametrize("H,N,keep_ratio,blocks,d", [(*s, d) for s in SIZES for d in (64, 128) if d == 128 or s[3] > 0 or s[2] == 1.0])
def test_units(H, N, keep_ratio, blocks, d):
    part = U.part_of(Workload("", 1, H, d, "bf16", (4, 4, 4 * N), (4, 4, 4)))
    nk = part.n_keep(keep_ratio)
    got, units = U.unit_blocks(N, H, nk)
    groups = -(-N // got)
    S, split = U.walk_split(N, H, nk)
    route = U.forward_route(N, H, nk, d)
    if blocks > 0:
        assert got == blocks and units <= 256 and route == "walk"
    else:
        assert units > 256 and route == "both" and S == (2 if blocks == 0 else 4) and split
    U.progress(f"units H={H} N={N} r={keep_ratio} d={d}")
    wl = Workload(f"units_{H}_{N}_{keep_ratio}_{d}", 1, H, d, "bf16", (4, 4, 4 * N), (4, 4, 4), threshold=0.7 if blocks > 0 else 0.9, keep_ratio=keep_ratio)
    heads = sorted({0, H // 2, H - 1} | {u // groups for u in split[:1]})
    x = U.device_inputs(wl, ("Q", "K", "V"), heads=heads)
    shp, _, _, lists, keep = U.run_indices(wl, x)
    sample = {0, 1, N // 2, N - 2, N - 1} | {b for u in split[:2] for b in range(u % groups * got, min(N, u % groups * got + got))}
    check(wl, x, shp, lists, keep, heads, sorted(sample))
    if blocks <= 0:
        assert lists.nnz.item() >= {0.25: 24, 0.5: 48, 1.0: 32}[keep_ratio] * H * N  # from here on the lists are long
        # segments of a split unit that hold nothing but logits of -inf
        x["Q"][..., 0] = x["Q"][..., 0].abs() + 0.5
        x["K"][:, :, torch.from_numpy(part.block_tokens()[:int(0.6 * N)].reshape(-1)).cuda(), 0] = float("-inf")
        check(wl, x, shp, lists, keep, heads, sorted(sample))


@pytest.mark.parametrize("N", [2048, 2049, 4100])
def test_unions_longer_than_a_list(N):
    """2,048 entries stand in LDS at a time; every block listed, the last unit and the last list of entries ragged."""
    U.progress(f"long union N={N}")
    wl = Workload(f"long_union_{N}", 1, 1, 128, "bf16", (4, 4, 4 * N), (4, 4, 4), threshold=1.0, keep_ratio=0.5)
    shp = U.shape_of(wl)
    gen = torch.Generator("cuda").manual_seed(N)
    x = {k: torch.randn((1, 1, N * 64, 128), generator=gen, device="cuda").to(torch.bfloat16) for k in ("Q", "K", "V")}
    i32 = lambda a: a.to(device="cuda", dtype=torch.int32).contiguous()
    lists = B.KvLists(i32(torch.arange(N + 1) * N), i32(torch.arange(N).repeat(N)), i32(torch.arange(N + 1) * N), i32(torch.arange(N).repeat(N)),
                      torch.tensor([N * N], device="cuda"), torch.empty(1, dtype=torch.uint8, device="cuda"))
    check(wl, x, shp, lists, B.prune_q(shp, x["Q"], wl.keep_ratio), [0], [0, 5, N - 1])


@pytest.mark.parametrize("keep_ratio", [1.0, 0.5, 0.25])
@pytest.mark.parametrize("step", [3.0, 20.0, -20.0])
def test_rising_maxima(keep_ratio, step):
    """Logits that rise by `step` (or fall) from one KV block to the next: the running maximum is moved now and then, at every block, never."""
    U.progress(f"rising maxima r={keep_ratio} step={step}")
    H, N, d = 3, 16, 128
    wl = Workload(f"rising_{step}", 1, H, d, "bf16", (4, 4, 4 * N), (4, 4, 4), threshold=1.0, keep_ratio=keep_ratio)
    x = U.device_inputs(wl, ("Q", "K", "V"), heads=(0, H - 1))
    x["Q"][..., 0] = 8.0
    shp, _, _, lists, keep = U.run_indices(wl, x)
    K = x["K"].clone()
    tok = torch.from_numpy(U.part_of(wl).block_tokens()).cuda()
    for j in range(N):
        K[:, :, tok[j], 0] = torch.tensor(step * (j - N // 2) * sqrt(d) / 8, device="cuda").to(torch.bfloat16)
    check(wl, x, shp, lists, keep, [0, H - 1], [0, 13, N - 1], K=K)


@pytest.mark.parametrize("keep_ratio,limit", [(0.25, 24), (0.5, 48), (1.0, 32)])
def test_both_kernels_at_the_limit(keep_ratio, limit):
    """More than a round of units: one listed block less than the limit a row on average, and as many as it; one kernel or the
    other writes every row."""
    U.progress(f"limit r={keep_ratio}")
    H, N, d = 20, 320, 128
    wl = Workload(f"limit_{limit}", 1, H, d, "bf16", (4, 4, 4 * N), (4, 4, 4), threshold=1.0, keep_ratio=keep_ratio)
    x = U.device_inputs(wl, ("Q", "K", "V"), heads=(0, H - 1))
    shp, keep = U.shape_of(wl), B.prune_q(U.shape_of(wl), x["Q"], keep_ratio)
    rng = np.random.default_rng(limit)
    rows = [np.sort(rng.choice(N, size=limit, replace=False)) for _ in range(H * N)]
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    for short in (True, False):
        if short:
            rows[H * N // 2] = rows[H * N // 2][:-1]
        else:
            rows[H * N // 2] = np.arange(limit)
        ptr, idx = i32(np.cumsum([0] + [len(r) for r in rows])), i32(np.concatenate(rows))
        lists = B.KvLists(ptr, idx, ptr, idx, torch.tensor([len(idx)], device="cuda"), torch.empty(1, dtype=torch.uint8, device="cuda"))
        check(wl, x, shp, lists, keep, [0, H // 2, H - 1], [0, 1, N // 2, N - 1])


# heads, blocks of a head, d: more than a round of units, the kernel without a barrier, then, with fewer blocks, the other one
@pytest.mark.parametrize("H,N,d", [(5, 257, 128), (9, 65, 64), (12, 50, 128), (14, 38, 64)])
def test_dense_beyond_a_round(H, N, d):
    U.progress(f"dense H={H} N={N} d={d}")
    wl = Workload(f"dense_{H}_{N}_{d}", 1, H, d, "bf16", (4, 4, 4 * N), (4, 4, 4), keep_ratio=1.0)
    assert U.unit_blocks(N, H, 64)[1] > 256
    heads, blocks = [0, H // 2, H - 1], [0, 1, N // 2, N - 2, N - 1]
    x = U.device_inputs(wl, ("Q", "K", "V"), heads=heads)
    O, LSE = B.dense_attn_fwd(U.shape_of(wl), x["Q"], x["K"], x["V"])
    part = U.part_of(wl)
    sel = part.block_tokens()[blocks].reshape(-1)
    for h in heads:
        rO, rL = o.attn_fwd(*[U.host_f64(x[k][0, h]) for k in "QKV"], part, np.arange(N + 1) * N, np.tile(np.arange(N), N),
                            np.tile(np.arange(64), (N, 1)), 1 / sqrt(d), q_blocks=blocks)
        U.check_tensors(wl.name, f"h{h}", "bf16", [("O", U.host_f64(O[0, h])[sel], rO[sel])], lse=(U.host_f64(LSE[0, h])[sel], rL[sel]))
