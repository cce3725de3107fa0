"""The plan of the forward and dQ launches, through the workspace sizes that follow from it (no GPU)."""
import pytest

from paper_2509_01085_amd import binding as B

import gpu_util as U


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_keep", [1, 16, 17, 32, 33, 64])
def test_workspace_follows_the_plan(d, n_keep):
    """Partial results of every segment, and none below 40 units: there a forward call takes no workspace."""
    kinds = set()
    for H in (1, 2, 3, 5, 9, 12, 17, 33, 53, 100, 300):
        for N in (1, 4, 12, 31, 32, 38, 48, 64, 156, 364):
            shp = B.Shape(1, H, 4, 4, 4 * N, 4, 4, 4, d, B.BF16)
            kind, S, _, units = U.split_plan(N, H, n_keep)
            waves, regs = (8 if n_keep > 32 else 4), d // 2
            slots = 8 * -(-len(units) // 8) * S * waves * 256  # (an XCD with a unit less leaves its place unused)
            assert B.fwd_workspace_bytes(shp, n_keep) == slots * (regs + 2), (kind, H, N)
            records = H * (-(-N // 2) if n_keep <= 16 else N * (2 if n_keep > 32 else 1)) * (64 * 2 * d + 256)
            assert B.bwd_workspace_bytes(shp, n_keep) == records + slots * regs, (kind, H, N)
            if H * -(-N // (8 if n_keep <= 16 else 4)) < 40:
                assert kind == "none"
            kinds.add(kind)
    assert kinds == {"none", "tail", "all"}
