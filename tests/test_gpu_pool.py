"""GPU parity of bsa_pool_blocks alone at the edges of its batches of rows, of the words a lane owns and of its passes:
means bit for bit the oracle's."""
import numpy as np
import pytest
import torch

from oracle import bsa_oracle as o
from paper_2509_01085_amd import binding as B

import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("block", [(1, 1, 1), (1, 7, 1), (2, 2, 2), (3, 1, 3), (4, 2, 2), (1, 17, 1), (2, 4, 4), (3, 1, 11), (5, 13, 1), (4, 8, 8)])
def test_means_are_bit_exact(dtype, block):
    U.progress(f"pool {dtype} {block}")
    grid = (block[0], 2 * block[1], 5 * block[2])
    part = o.Partition(*grid, *block)
    rng = np.random.default_rng(part.Bk)
    for d in (8, 64, 72, 128, 136, 256):
        shp = B.Shape(1, 2, *grid, *block, d, B.F32 if dtype == "fp32" else B.BF16)
        x = torch.from_numpy(rng.standard_normal((1, 2, part.L, d)).astype(np.float32)).to(shp.torch_dtype)
        got = B.pool_blocks(shp, x.cuda()).cpu().numpy()
        for h in range(2):
            assert np.array_equal(got[0, h], o.pool_blocks(x[0, h].double().numpy(), part)), (d, h)
