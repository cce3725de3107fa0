"""Whole KV blocks whose logits are -inf, on the bf16 matrix-core path: wherever a walk, or a segment of a walk that
several workgroups share, begins with such a block, it weighs nothing.  An empty list gives zeros."""
from math import sqrt

import pytest
import torch

from bsa_workloads import Workload
from oracle import bsa_oracle as o
from paper_2509_01085_amd import binding as B

import gpu_util as U

pytestmark = pytest.mark.gpu


# 64, 32 and 16 retained queries a block: two wavefronts a block, one, and two blocks a wavefront
@pytest.mark.parametrize("keep_ratio", [1.0, 0.5, 0.25])
@pytest.mark.parametrize("d,H", [(64, 5), (128, 1), (128, 20)])
def test_blocks_at_minus_infinity(keep_ratio, d, H):
    """32 blocks, all listed.  One head and five: whole walks of the kernel without a barrier.  Twenty: segments of all walks, or
    of the last ones of an XCD, of the one with a barrier a tile."""
    assert U.forward_route(32, H, 64 * keep_ratio, d) == ("pipe" if H == 20 else "walk")
    U.progress(f"masked blocks r={keep_ratio} d={d} H={H}")
    wl = Workload(f"masked_{d}_{H}", 1, H, d, "bf16", (8, 16, 16), (4, 4, 4), threshold=1.0, keep_ratio=keep_ratio)
    x = U.device_inputs(wl, ("Q", "K", "V"), heads=(0, H - 1))
    shp, _, _, lists, keep = U.run_indices(wl, x)
    part, host = U.part_of(wl), U.lists_to_host(shp, lists)
    tok = part.block_tokens()
    Q = x["Q"].clone()
    Q[..., 0] = Q[..., 0].abs() + 0.5
    for masked in ([0], list(range(8)), [8], list(range(7, 17)), list(range(0, 32, 2)), list(range(31)), list(range(32))):
        K = x["K"].clone()
        K[:, :, torch.from_numpy(tok[masked].reshape(-1)).cuda(), 0] = float("-inf")
        O, LSE = B.attn_fwd(shp, Q, K, x["V"], lists, keep)
        if len(masked) == 32:  # no softmax
            assert (LSE == float("-inf")).all()
            assert (O == 0).all() if keep.shape[-1] <= 16 else O.isnan().all()
            continue
        assert torch.isfinite(O).all() and torch.isfinite(LSE).all(), masked
        for h in {0, H - 1}:
            ptr, idx = U.head_csr(host, shp, 0, h)
            blocks = [0, 13, 31]
            sel = tok[blocks].reshape(-1)
            rO, rL = o.attn_fwd(*[U.host_f64(t[0, h]) for t in (Q, K, x["V"])], part, ptr, idx, keep[0, h].cpu().numpy(),
                                1 / sqrt(d), q_blocks=blocks)
            U.check_tensors(wl.name, f"h{h} masked {masked}", "bf16", [("O", U.host_f64(O[0, h])[sel], rO[sel])],
                            lse=(U.host_f64(LSE[0, h])[sel], rL[sel]))


@pytest.mark.parametrize("keep_ratio", [1.0, 0.5, 0.25])
@pytest.mark.parametrize("N", [12, 32])
def test_empty_list(keep_ratio, N):
    """Rows that list nothing, in the same workgroup as rows that do: O is zero and LSE -inf, the others are finite.  12 blocks: the
    kernel with a barrier a tile, 32: the other one."""
    U.progress(f"empty lists r={keep_ratio} N={N}")
    wl = Workload("empty", 1, 1, 64, "bf16", (4, 4, 4 * N), (4, 4, 4), threshold=0.7, keep_ratio=keep_ratio)
    x = U.device_inputs(wl, ("Q", "K", "V"))
    shp, _, _, lists, keep = U.run_indices(wl, x)
    ptr, idx = lists.q2k_ptr.cpu(), lists.q2k_idx.cpu()
    rows = [idx[ptr[i]:ptr[i + 1]] if i % 3 else idx[:0] for i in range(N)]
    lists.q2k_ptr[:] = torch.tensor([0] + [len(r) for r in rows]).cumsum(0).int().cuda()
    lists.q2k_idx[:sum(map(len, rows))] = torch.cat(rows).cuda()
    O, LSE = B.attn_fwd(shp, x["Q"], x["K"], x["V"], lists, keep)
    tok = torch.from_numpy(U.part_of(wl).block_tokens()).cuda()
    for i in range(N):
        if i % 3:
            assert torch.isfinite(O[0, 0, tok[i]]).all() and torch.isfinite(LSE[0, 0, tok[i]]).all() and (O[0, 0, tok[i]] != 0).any()
        else:
            assert (O[0, 0, tok[i]] == 0).all() and (LSE[0, 0, tok[i]] == float("-inf")).all()
