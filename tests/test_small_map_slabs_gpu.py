"""GPU parity of the backward of small maps, whose bias gradient keeps part of
its partial slabs in dK's place: every head width, a row range, few and many
slabs past the workspace's own, in a workspace of exactly the reported size
(nothing past it is written), one map or a batch (bitwise the same).  Bounds
of test_parity_gpu."""
import pytest
import torch

import oracle
from paper_2506_20686_amd import binding as B
from paper_2506_20686_amd import workloads as W

from test_parity_gpu import close, to_dev

pytestmark = pytest.mark.gpu
NAMES = ("dq", "dk", "dv", "dg", "dbias")
GUARD = 4096


def guarded(size):
    ws = torch.full((size + GUARD,), 0x5A, dtype=torch.uint8, device="cuda")
    return ws, ws[:size]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("node", [B.STARTING, B.ENDING])
@pytest.mark.parametrize("n,h,d", [(24, 4, 32), (32, 4, 32), (33, 4, 16), (65, 3, 64), (100, 4, 16),
                                   (100, 4, 32), (128, 4, 32), (128, 1, 64), (129, 1, 32)])
def test_backward(dtype, node, n, h, d):
    t, gen = W.make_inputs(n, h, d, dtype, seed=60 + n + d)
    t["mask"] = W.random_mask(n, 0.8, gen)
    x = to_dev(t)
    args = (x["q"], x["k"], x["v"], x["g"], x["bias"])
    out, lse = B.fwd(*args, x["mask"], node)
    code = B.BF16 if dtype == torch.bfloat16 else B.F32
    ws, use = guarded(B.tri_attn_bwd_workspace_bytes(node, code, n, h, d))
    print(f"\n[small backward {dtype} node {node} n={n} h={h} d={d}]", flush=True)
    got = B.bwd(*args, out, lse, x["dout"], x["mask"], node, workspace=use)
    again = B.bwd(*args, out, lse, x["dout"], x["mask"], node)
    ref = oracle.bwd(node, *(t[k] for k in ("q", "k", "v", "g", "bias", "dout", "mask")))
    for name, a, b, r in zip(NAMES, got, again, ref):
        close(name, a, r, dtype)
        assert torch.equal(a, b), name
    assert bool((ws[-GUARD:] == 0x5A).all()), "written past the workspace"


@pytest.mark.parametrize("n,rows", [(64, 64), (100, 30), (128, 50)])
def test_row_range(n, rows):
    h, d = 4, 32
    t, _ = W.make_inputs(n, h, d, torch.bfloat16, seed=80 + n)
    t["dout"][rows:] = 0  # the other rows then add nothing to the bias gradient
    whole = oracle.bwd(B.STARTING, *(t[k] for k in ("q", "k", "v", "g", "bias", "dout")), None)
    x = to_dev(t)
    part = [x[k][:rows].contiguous() for k in ("q", "k", "v", "g")] + [x["bias"]]
    out, lse = B.rows_fwd(*part)
    ws, use = guarded(B.tri_attn_rows_bwd_workspace_bytes(B.BF16, n, rows, h, d))
    got = B.rows_bwd(*part, out, lse, x["dout"][:rows].contiguous(), workspace=use)
    for name, a, r in zip(NAMES, got, whole):
        close(name, a, r if name == "dbias" else r[:rows], torch.bfloat16)
    assert bool((ws[-GUARD:] == 0x5A).all()), "written past the workspace"


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,d", [(32, 32), (100, 16), (100, 32), (90, 64)])
def test_batch_equals_single_maps(dtype, n, d):
    parts = [W.make_inputs(n, 4, d, dtype, seed=90 + i)[0] for i in range(3)]
    x = {k: torch.stack([p[k] for p in parts]).cuda() for k in ("q", "k", "v", "g", "bias", "dout")}
    args = [x[k] for k in ("q", "k", "v", "g", "bias")]
    out, lse = B.fwd(*args)
    got = B.bwd(*args, out, lse, x["dout"])
    code = B.BF16 if dtype == torch.bfloat16 else B.F32
    one = torch.empty(B.tri_attn_bwd_workspace_bytes(0, code, n, 4, d), dtype=torch.uint8,
                      device="cuda")
    in_turn = B.bwd(*args, out, lse, x["dout"], workspace=one)
    for i in range(3):
        s = [a[i].clone() for a in args]
        single = B.bwd(*s, out[i].clone(), lse[i].clone(), x["dout"][i].clone())
        for name, a, b, c in zip(NAMES, got, in_turn, single):
            assert torch.equal(a[i], c) and torch.equal(b[i], c), (i, name)
