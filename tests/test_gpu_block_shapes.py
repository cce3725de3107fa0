"""Attention kernels at the sizes where their tiling can go wrong, against the oracle: block sizes
around the 16- and 64-key tiles, head dimensions around the 16- and 32-channel steps, retained
queries around one and two 16-row tiles.  Infinities in V, and lists that are sets in any order."""
from math import sqrt

import numpy as np
import pytest
import torch

from bsa_workloads import Workload, head_inputs
from oracle import bsa_oracle as o
from paper_2509_01085_amd import binding as B

import gpu_util as U

pytestmark = pytest.mark.gpu

# name: (dtype, d, grid, block, keep ratio, window)
SHAPES = {
    "bk1_f32_d8": ("fp32", 8, (2, 3, 4), (1, 1, 1), 1.0, (0, 0, 0)),
    "bk15_bf16_d8": ("bf16", 8, (3, 9, 5), (1, 3, 5), 0.5, (0, 0, 0)),
    "bk16_f32_d24": ("fp32", 24, (4, 8, 8), (1, 4, 4), 0.5, (1, 2, 2)),
    "bk18_bf16_d72": ("bf16", 72, (4, 9, 6), (2, 3, 3), 0.9, (0, 0, 0)),       # 17 queries: a second tile of one row
    "bk30_bf16_d80": ("bf16", 80, (6, 4, 10), (3, 2, 5), 0.5, (0, 0, 0)),
    "bk45_bf16_d96": ("bf16", 96, (3, 6, 10), (3, 3, 5), 0.75, (0, 0, 0)),     # 34 queries, three key tiles
    "bk60_bf16_d128": ("bf16", 128, (6, 10, 8), (3, 5, 4), 0.5, (0, 0, 0)),
    "bk60_f32_d104": ("fp32", 104, (6, 10, 8), (3, 5, 4), 0.5, (0, 0, 0)),
    "bk64_bf16_d48": ("bf16", 48, (4, 8, 12), (4, 4, 4), 0.5, (2, 2, 2)),
    "bk64_bf16_d152": ("bf16", 152, (4, 8, 8), (4, 4, 4), 0.3, (0, 0, 0)),
    "bk24_bf16_d200": ("bf16", 200, (4, 6, 12), (2, 3, 4), 0.5, (0, 0, 0)),
    "bk70_bf16_d40": ("bf16", 40, (2, 10, 14), (2, 5, 7), 0.5, (0, 0, 0)),     # steps of 48 and 22 keys
    "bk128_bf16_d256": ("bf16", 256, (4, 8, 16), (4, 4, 8), 0.3, (0, 0, 0)),
    "bk256_f32_d128": ("fp32", 128, (4, 8, 16), (4, 8, 8), 0.3, (0, 0, 0)),
}

# Enough blocks that a dK/dV workgroup takes several 16-key tiles: name: (heads, tiles a workgroup, shape as above)
MANY = {
    "2_of_2_f32_d72": (64, 2, ("fp32", 72, (4, 6, 10), (2, 3, 5), 0.5, (0, 0, 0))),        # 30 keys
    "2_of_2_f32_d64": (64, 2, ("fp32", 64, (4, 6, 10), (2, 3, 5), 1.0, (0, 0, 0))),        # (no padding channels)
    "2_of_2_bf16_d80": (64, 2, ("bf16", 80, (4, 6, 8), (2, 3, 4), 0.9, (0, 0, 0))),        # 24 keys
    "2_of_2_bf16_d96": (64, 2, ("bf16", 96, (4, 6, 10), (2, 3, 5), 0.5, (0, 0, 0))),       # (no padding channels)
    "4_of_3_f32_d64": (64, 4, ("fp32", 64, (6, 6, 10), (3, 3, 5), 0.4, (0, 0, 0))),        # 45 keys: a wavefront without a tile
    "4_of_3_bf16_d104": (64, 4, ("bf16", 104, (6, 6, 10), (3, 3, 5), 0.4, (0, 0, 0))),
    "4_of_5_f32_d128": (32, 4, ("fp32", 128, (4, 10, 14), (2, 5, 7), 0.5, (0, 0, 0))),     # 70 keys: forward steps of 64 and 6
    "4_of_5_bf16_d128": (32, 4, ("bf16", 128, (4, 10, 14), (2, 5, 7), 0.3, (0, 0, 0))),
    "2_of_3_f32_d136": (32, 2, ("fp32", 136, (6, 6, 10), (3, 3, 5), 0.5, (0, 0, 0))),
    "2_of_5_bf16_d200": (22, 2, ("bf16", 200, (4, 10, 14), (2, 5, 7), 0.5, (0, 0, 0))),
}


def _run(wl, heads=None):
    x = U.device_inputs(wl, heads=heads)
    shp, _, _, lists, keep = U.run_indices(wl, x)
    O, LSE = B.attn_fwd(shp, x["Q"], x["K"], x["V"], lists, keep)
    return x, shp, lists, keep, O, LSE


def _check_shape(name, shape, H, heads):
    dtype, d, grid, block, keep_ratio, window = shape
    wl = Workload("shape_" + name, 1, H, d, dtype, grid, block, threshold=0.7, keep_ratio=keep_ratio, window=window)
    x, shp, lists, keep, O, LSE = _run(wl, heads)
    dQ, dK, dV = B.attn_bwd(shp, x["Q"], x["K"], x["V"], O, LSE, x["dO"], lists, keep)
    torch.cuda.synchronize()
    part = U.part_of(wl)
    for h in heads:
        xi = head_inputs(wl, 0, h)
        ix, rO, rL, rdQ, rdK, rdV = o.bsa_head(xi["Q"], xi["K"], xi["V"], xi["dO"], part, wl.threshold, wl.keep_ratio,
                                               o_storage=U.o_storage_of(wl))
        assert np.array_equal(keep[0, h].cpu().numpy(), ix.keep_idx)
        sg = U.T.rounding_sigma(xi, part, ix, 1 / sqrt(d)) if dtype == "bf16" else None
        U.check_tensors(name, f"h{h}", dtype, [(t, U.host_f64(got[0, h]), ref) for t, got, ref in
                                               (("O", O, rO), ("dQ", dQ, rdQ), ("dK", dK, rdK), ("dV", dV, rdV))],
                        sigma=sg, lse=(U.host_f64(LSE[0, h]), rL))
    return shp


@pytest.mark.parametrize("name", list(SHAPES))
def test_block_shape(name):
    U.progress(f"block shape {name}")
    _check_shape(name, SHAPES[name], 2, (0, 1))


@pytest.mark.parametrize("name", list(MANY))
def test_block_shape_many_blocks(name):
    U.progress(f"many blocks {name}")
    H, tiles, shape = MANY[name]
    shp = _check_shape("many_" + name, shape, H, (0, H // 2, H - 1))
    nkt = (shp.Bk + 15) // 16
    assert shp.rows * -(-nkt // tiles) >= 512 and nkt > tiles // 2  # the rule of the launch, restated


@pytest.mark.parametrize("name,value,token", [("bk30_bf16_d80", float("inf"), 7), ("bk60_bf16_d128", float("-inf"), 7),
                                              ("bk45_bf16_d96", float("inf"), -1), ("bk60_f32_d104", float("-inf"), -1)])
def test_infinity_in_v_stays_in_its_channel(name, value, token):
    """Every query lists every block here and no probability underflows, so the channel of an
    infinite V entry is infinite for every token, and nothing else is."""
    dtype, d, grid, block, keep_ratio, window = SHAPES[name]
    wl = Workload("inf_" + name, 1, 1, d, dtype, grid, block, threshold=1.0, keep_ratio=keep_ratio, window=window)
    x, shp, lists, keep, O, _ = _run(wl)
    assert torch.isfinite(O).all()
    V = x["V"].clone()
    V[0, 0, token, 5] = value  # (the last token is the last key of a block whose last key tile is partial)
    O2, _ = B.attn_fwd(shp, x["Q"], x["K"], V, lists, keep)
    assert (O2[..., 5].float() == value).all()
    rest = torch.arange(d, device=O.device) != 5
    # the finite channels: the same products, rounded to bf16 after sums in another order
    assert ((O2 - O).float()[..., rest].abs() <= 2.0 ** -7 * O.float()[..., rest].abs() + 1e-5).all()


@pytest.mark.parametrize("dtype,d", [("fp32", 72), ("fp32", 104), ("fp32", 136), ("bf16", 72)])
def test_key_at_minus_infinity_in_the_backward(dtype, d):
    """Channel 0 of one key is -inf and that channel of every query positive: its logits are -inf, its P and
    dS zero.  Only 0 * inf of dQ's own channel 0 is not finite; d leaves padding channels in the last group."""
    grid, block = (4, 6, 10), (2, 3, 5)
    wl = Workload(f"neg_inf_{dtype}_{d}", 1, 1, d, dtype, grid, block, threshold=1.0, keep_ratio=0.5)
    x = U.device_inputs(wl)
    shp, _, _, lists, keep = U.run_indices(wl, x)
    Q, K = x["Q"].clone(), x["K"].clone()
    Q[..., 0] = Q[..., 0].abs() + 0.5
    K[0, 0, 33, 0] = float("-inf")
    O, LSE = B.attn_fwd(shp, Q, K, x["V"], lists, keep)
    got = B.attn_bwd(shp, Q, K, x["V"], O, LSE, x["dO"], lists, keep)
    torch.cuda.synchronize()
    host = U.lists_to_host(shp, lists)
    part, ptr, idx = U.part_of(wl), *U.head_csr(host, shp, 0, 0)
    args = [U.host_f64(t[0, 0]) for t in (Q, K, x["V"])]
    keep_h = keep[0, 0].cpu().numpy()
    rO, _ = o.attn_fwd(*args, part, ptr, idx, keep_h, 1 / sqrt(d))
    with np.errstate(invalid="ignore"):
        ref = o.attn_bwd(*args, U.host_f64(x["dO"][0, 0]), part, ptr, idx, keep_h, 1 / sqrt(d), O_in=U.o_storage_of(wl)(rO))
    for name, a, r in zip(("O", "dQ", "dK", "dV"), (O, *got), (rO, *ref)):
        a = U.host_f64(a[0, 0])
        assert np.array_equal(np.isfinite(a), np.isfinite(r)), name
        a, r = a[np.isfinite(r)], r[np.isfinite(r)]
        f = U.T.figures(a, r)  # (these kernels round no operand: the bf16 excess needs no sigma)
        assert f["plain"] <= U.T.TOL_F32 if dtype == "fp32" else f["excess"] <= U.T.TOL_BF16, (name, f)
    assert not np.isfinite(ref[0]).all() and np.isfinite(ref[0][:, 1:]).all()


@pytest.mark.parametrize("dtype,d,block", [("fp32", 64, (2, 3, 5)), ("bf16", 72, (2, 3, 5)), ("bf16", 128, (4, 6, 5)), ("fp32", 200, (1, 3, 5))])
def test_blocks_at_minus_infinity(dtype, d, block):
    """Whole KV blocks whose logits are -inf, at every position of a list: they weigh nothing, whichever
    wavefront begins with them.  With every block masked the softmax has no value: O is NaN, LSE -inf."""
    grid = tuple(2 * b for b in block)  # eight blocks, all listed
    wl = Workload(f"masked_{dtype}_{d}", 1, 1, d, dtype, grid, block, threshold=1.0, keep_ratio=0.5)
    x = U.device_inputs(wl)
    shp, _, _, lists, keep = U.run_indices(wl, x)
    part, host = U.part_of(wl), U.lists_to_host(shp, lists)
    ptr, idx = U.head_csr(host, shp, 0, 0)
    tok, keep_h = part.block_tokens(), keep[0, 0].cpu().numpy()
    Q = x["Q"].clone()
    Q[..., 0] = Q[..., 0].abs() + 0.5
    for masked in ([1], [2, 3], [1, 3, 5, 7], [0], [0, 1, 2, 3, 4, 5, 6], list(range(8))):
        K = x["K"].clone()
        K[0, 0, torch.from_numpy(tok[masked].reshape(-1)).cuda(), 0] = float("-inf")
        O, LSE = B.attn_fwd(shp, Q, K, x["V"], lists, keep)
        if len(masked) == 8:
            assert O.isnan().all() and (LSE == float("-inf")).all()
            continue
        rO, rL = o.attn_fwd(*[U.host_f64(t[0, 0]) for t in (Q, K, x["V"])], part, ptr, idx, keep_h, 1 / sqrt(d))
        U.check_tensors(wl.name, f"blocks {masked}", dtype, [("O", U.host_f64(O[0, 0]), rO)], lse=(U.host_f64(LSE[0, 0]), rL))


@pytest.mark.parametrize("dtype,d,block", [("bf16", 72, (2, 3, 5)), ("bf16", 128, (3, 5, 4)), ("fp32", 64, (2, 3, 5))])
def test_zero_probability_keeps_any_finite_value_out(dtype, d, block):
    """A key whose probability underflows to zero adds nothing, also with V at the type's lowest value."""
    grid = tuple(2 * b for b in block)
    wl = Workload(f"lowest_{dtype}_{d}", 1, 1, d, dtype, grid, block, threshold=1.0, keep_ratio=0.5)
    x = U.device_inputs(wl)
    shp, _, _, lists, keep = U.run_indices(wl, x)
    Q, K, V = (x[n].clone() for n in ("Q", "K", "V"))
    Q[..., 0] = Q[..., 0].abs() + 0.5
    K[0, 0, 17, 0] = -1e5
    V[0, 0, 17] = torch.finfo(V.dtype).min
    O, LSE = B.attn_fwd(shp, Q, K, V, lists, keep)
    ptr, idx = U.head_csr(U.lists_to_host(shp, lists), shp, 0, 0)
    rO, rL = o.attn_fwd(*[U.host_f64(t[0, 0]) for t in (Q, K, V)], U.part_of(wl), ptr, idx, keep[0, 0].cpu().numpy(), 1 / sqrt(d))
    U.check_tensors(wl.name, "O", dtype, [("O", U.host_f64(O[0, 0]), rO)], lse=(U.host_f64(LSE[0, 0]), rL))


@pytest.mark.parametrize("dtype,d,block", [("fp32", 64, (2, 3, 5)), ("fp32", 136, (1, 3, 5)), ("bf16", 72, (2, 3, 5)), ("bf16", 128, (3, 5, 4))])
def test_nan_reaches_every_gradient(dtype, d, block):
    """One NaN in K, every block listed: no row has a softmax, and no gradient may look as if it had."""
    grid = tuple(2 * b for b in block)
    wl = Workload(f"nan_{dtype}_{d}", 1, 1, d, dtype, grid, block, threshold=1.0, keep_ratio=0.5)
    x = U.device_inputs(wl)
    shp, _, _, lists, keep = U.run_indices(wl, x)
    K = x["K"].clone()
    K[0, 0, 17, 3] = float("nan")
    O, LSE = B.attn_fwd(shp, x["Q"], K, x["V"], lists, keep)
    dQ, dK, dV = B.attn_bwd(shp, x["Q"], K, x["V"], O, LSE, x["dO"], lists, keep)
    kept = torch.zeros(shp.L, dtype=torch.bool)
    tok = U.part_of(wl).block_tokens()
    for i, ids in enumerate(keep[0, 0].cpu().numpy()):
        kept[torch.from_numpy(tok[i, ids])] = True
    assert O.isnan().all() and not LSE.isfinite().any()
    assert not dQ[0, 0].cpu()[kept].isfinite().any() and not dQ[0, 0].cpu()[~kept].any()
    assert not dK.isfinite().any() and not dV.isfinite().any()


@pytest.mark.parametrize("keep_ratio", [0.25, 0.5, 1.0])
def test_transposed_lists_are_sets(keep_ratio):
    """dK, dV of the bf16 path: order, repetition and ids out of range in a k2q list change nothing."""
    wl = Workload("sets", 1, 2, 128, "bf16", (4, 12, 20), (4, 4, 4), threshold=0.8, keep_ratio=keep_ratio)
    x, shp, lists, keep, O, LSE = _run(wl)
    run = lambda li: B.attn_bwd(shp, x["Q"], x["K"], x["V"], O, LSE, x["dO"], li, keep)
    want = run(lists)
    host = U.lists_to_host(shp, lists)
    rng = np.random.default_rng(3)
    ptr, idx = [0], []
    for r in range(shp.B * shp.H * shp.N):
        own = host["k2q_idx"][host["k2q_ptr"][r]:host["k2q_ptr"][r + 1]]
        row = np.concatenate([own, own[:2], [-1, shp.N, shp.N + 5]]).astype(np.int32)
        rng.shuffle(row)
        idx.append(row)
        ptr.append(ptr[-1] + len(row))
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    other = B.KvLists(lists.q2k_ptr, lists.q2k_idx, i32(ptr), i32(np.concatenate(idx)), lists.nnz, lists.workspace)
    for a, b in zip(run(other), want):
        assert torch.equal(a, b)


# name: (d, grid, block, keep ratio)
ROUNDING = {
    "24_keys_d72": (72, (6, 9, 16), (2, 3, 4), 0.5),
    "24_keys_d200": (200, (4, 9, 12), (2, 3, 4), 0.5),
    "30_keys_d80": (80, (6, 8, 15), (3, 2, 5), 0.5),
    "45_keys_d96": (96, (6, 9, 15), (3, 3, 5), 0.5),
    "60_keys_d128": (128, (6, 15, 16), (3, 5, 4), 0.5),
    "64_keys_d152": (152, (8, 12, 12), (4, 4, 4), 0.25),
    "128_keys_d64": (64, (8, 12, 16), (4, 4, 8), 0.5),
}


@pytest.mark.parametrize("name", list(ROUNDING))
def test_only_results_are_rounded(name):
    """bf16 tensors of other shapes: products of bf16 values are exact, and an fp32 operand is the sum of three
    bf16 parts, so a result is the bf16 rounding of an fp32 sum.  Such a sum meets the fp32 tolerance and rounds
    differently only that close to a midpoint of two bf16 values ("flip": the farthest such midpoint, in RMS).
    Most sums are within 2^-20 RMS, which is a share of about 2^-11 E[RMS / |x|] of the elements, near 1e-3
    ("differ").  An operand rounded to bf16 would move most elements, by up to 2^-9."""
    d, grid, block, keep_ratio = ROUNDING[name]
    wl = Workload("round_" + name, 1, 1, d, "bf16", grid, block, threshold=0.8, keep_ratio=keep_ratio)
    x = U.device_inputs(wl)
    shp, _, _, lists, keep = U.run_indices(wl, x)
    O, LSE = B.attn_fwd(shp, x["Q"], x["K"], x["V"], lists, keep)
    xi = head_inputs(wl, 0, 0)
    _, rO, rL, rdQ, rdK, rdV = o.bsa_head(xi["Q"], xi["K"], xi["V"], xi["dO"], U.part_of(wl), wl.threshold, wl.keep_ratio,
                                          o_storage=U.o_storage_of(wl))
    # the backward of the oracle's own stored output and LSE
    O_in = torch.from_numpy(U.o_storage_of(wl)(rO)).to(torch.bfloat16).cuda()[None, None]
    dQ, dK, dV = B.attn_bwd(shp, x["Q"], x["K"], x["V"], O_in, torch.from_numpy(rL).float().cuda()[None, None], x["dO"], lists, keep)
    figs = {"LSE": {"abs": float(f"{np.abs(U.host_f64(LSE[0, 0]) - rL).max():.2e}")}}
    for n, got, ref in (("O", O, rO), ("dQ", dQ, rdQ), ("dK", dK, rdK), ("dV", dV, rdV)):
        got = U.host_f64(got[0, 0])
        rounded = U.host_f64(torch.from_numpy(ref).to(torch.bfloat16))
        bad = got != rounded
        flip = np.abs(ref - (got + rounded) / 2)[bad].max(initial=0.0) / np.sqrt(np.mean(ref ** 2))
        figs[n] = {"differ": float(f"{bad.mean():.2e}"), "flip": float(f"{flip:.2e}"), **{k: float(f"{v:.3e}") for k, v in U.T.figures(got, ref).items()}}
    U.record("round " + name, "h0", figs)
    assert figs["LSE"]["abs"] <= 1e-5  # logits of some tens: 2^-24 of them, and the sums of up to 1e3 terms
    assert all(figs[n]["differ"] <= 2e-3 and figs[n]["flip"] <= U.T.TOL_F32 for n in ("O", "dQ", "dK", "dV")), figs


@pytest.mark.parametrize("d,grid,block", [(72, (6, 9, 16), (2, 3, 4)), (72, (8, 16, 16), (4, 4, 4)), (200, (4, 9, 12), (2, 3, 4))])
def test_lse_is_as_good_as_its_storage(d, grid, block):
    """LSE below 16 is stored to 2^-20, an rms error of at most 2^-20 / sqrt(12) = 2.8e-7.  The logarithm (1 ulp of
    up to 10 in the exp2 domain) and its scaling add 1.9e-7 and 1.4e-7, the logits (products of bf16 values,
    exact, summed in fp32) less: 3.6e-7 together.  A rounded scale would leave up to 2^-24 of the logits."""
    wl = Workload(f"lse_d{d}", 1, 1, d, "bf16", grid, block, threshold=0.8, keep_ratio=1.0)
    x = U.device_inputs(wl)
    shp, _, _, lists, keep = U.run_indices(wl, x)
    _, LSE = B.attn_fwd(shp, x["Q"], x["K"], x["V"], lists, keep)
    ptr, idx = U.head_csr(U.lists_to_host(shp, lists), shp, 0, 0)
    _, rL = o.attn_fwd(*[U.host_f64(x[n][0, 0]) for n in "QKV"], U.part_of(wl), ptr, idx, keep[0, 0].cpu().numpy(), 1 / sqrt(d))
    assert 4 < np.median(rL) and rL.max() < 16
    err = U.host_f64(LSE[0, 0]) - rL
    figs = {"LSE": {"rms": float(f"{np.sqrt(np.mean(err * err)):.2e}"), "mean": float(f"{err.mean():.2e}")}}
    U.record(wl.name, f"grid {grid}", figs)
    assert figs["LSE"]["rms"] <= 4e-7, figs
