"""GPU parity where the preparation's grid and the bias gradient's row chunks
change shape: key-bit blocks of 64 rows and words of 32 keys (ending node),
padding queries, two slabs up to 32 (small maps), the four-heads-at-a-time
reduction and its remainder.  Bounds of test_parity_gpu."""
import pytest
import torch

from paper_2506_20686_amd import binding as B

from test_parity_gpu import full_check, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("node", [B.STARTING, B.ENDING])
@pytest.mark.parametrize("n,h,mask_kind", [(2, 4, "random"), (31, 8, "pair"), (32, 5, "random"),
                                           (65, 4, "random"), (97, 8, "none"), (128, 8, "pair"),
                                           (129, 2, "random"), (161, 6, "random")])
def test_small_maps(dtype, node, n, h, mask_kind):
    full_check(inputs(n, h, dtype, seed=40 + n + node, mask_kind=mask_kind), node, dtype)
