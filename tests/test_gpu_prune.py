"""GPU parity of bsa_prune_q alone on queries that hold infinities and NaN: every window keeps exactly its
quota, the lists are the oracle's, and nothing is written past the last one."""
import numpy as np
import pytest
import torch

from oracle import bsa_oracle as o
from paper_2509_01085_amd import binding as B

import gpu_util as U

pytestmark = pytest.mark.gpu

GUARD = 256  # words behind the lists


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("block,window,keep_ratio", [((4, 4, 4), (0, 0, 0), 0.5), ((4, 4, 4), (2, 2, 2), 0.5), ((3, 2, 5), (0, 0, 0), 0.1),
                                                     ((4, 6, 5), (2, 3, 5), 0.4), ((4, 8, 8), (0, 0, 0), 0.25)])
def test_quota_holds_with_infinities(dtype, block, window, keep_ratio):
    """inf / inf is no cosine: such a token ranks behind all others, ties by id, as the oracle's sort puts NaN
    last.  In the last block (whose list ends the buffer) one token is infinite, then two, then the center of its
    window; a NaN counts as a zero vector."""
    U.progress(f"prune infinities {dtype} {block} {window}")
    d, grid = 24, tuple(2 * b for b in block)
    part = o.Partition(*grid, *block, *window)
    shp = B.Shape(1, 1, *grid, *block, d, B.F32 if dtype == "fp32" else B.BF16, *window)
    nk = B.n_keep(shp, keep_ratio)
    rng = np.random.default_rng(3)
    base = torch.from_numpy(rng.standard_normal((part.L, d)).astype(np.float32)).to(shp.torch_dtype)
    tok, cen = part.block_tokens(), part.centers()
    others = [c for c in range(part.Bk) if c not in set(int(x) for x in cen)]
    inf = float("inf")
    for bad in ({others[0]: inf}, {others[-1]: -inf, others[1]: inf}, {int(cen[0]): inf}, {int(cen[-1]): -inf, others[0]: inf},
                {others[0]: float("nan"), others[2]: inf}, {c: inf for c in range(part.Bk)}):
        Q = base.clone()
        for c, v in bad.items():
            Q[tok[-1, c], 5] = v
            Q[tok[0, c], 2] = v
        buf = torch.full((part.N * nk + GUARD,), -7, dtype=torch.int32, device="cuda")
        keep = buf[:part.N * nk].view(1, 1, part.N, nk)
        B.prune_q(shp, Q.cuda().view(1, 1, part.L, d), keep_ratio, keep)
        with np.errstate(invalid="ignore"):
            ref, _ = o.prune_q(Q.double().numpy(), part, keep_ratio)
        assert np.array_equal(keep[0, 0].cpu().numpy(), ref), bad
        assert (buf[part.N * nk:] == -7).all(), bad
