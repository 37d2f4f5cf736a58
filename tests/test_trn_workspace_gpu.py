"""The transition layer in a workspace of exactly the reported size: nothing
past it is written, and the results are bitwise those of a larger one."""
import pytest
import torch

from paper_2506_20686_amd import binding as B
from paper_2506_20686_amd import workloads as W

pytestmark = pytest.mark.gpu
GUARD = 4096


@pytest.mark.parametrize("m,f", [(1, 128), (300, 256), (4097, 2048)])
def test_exact_workspace(m, f):
    x = {k: v.cuda() for k, v in W.trn_inputs(m, seed=700 + m, f=f).items()}
    args = (x["x"], x["gamma"], x["beta"], x["w1"], x["w2"])
    out, mean, rstd = B.transition_fwd(*args)
    grads = B.transition_bwd(*args, mean, rstd, x["dout"])
    for size, call, ref in (
            (B.tri_transition_fwd_workspace_bytes(B.BF16, m, 128, f),
             lambda ws: B.transition_fwd(*args, workspace=ws), (out, mean, rstd)),
            (B.tri_transition_bwd_workspace_bytes(B.BF16, m, 128, f),
             lambda ws: B.transition_bwd(*args, mean, rstd, x["dout"], workspace=ws), grads)):
        ws = torch.full((size + GUARD,), 0x5A, dtype=torch.uint8, device="cuda")
        got = call(ws[:size])
        assert bool((ws[size:] == 0x5A).all())
        assert bool((ws[:size] != 0x5A).any()), "the workspace passed in was not used"
        for a, b in zip(got, ref):
            assert torch.equal(a, b)
