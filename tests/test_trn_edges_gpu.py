"""GPU parity of the fused transition layer at the edges of its tilings (32-row
blocks, 16-row tiles of the row sums, 128- and 32-column hidden groups, row
parts that end inside a block), with the bounds of test_trn_gpu."""
import pytest

from paper_2506_20686_amd import workloads as W

from oracle import transition as OT
from test_lnl_gpu import close
from test_trn_gpu import check_sums, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,f", [(15, 128), (16, 640), (31, 256), (32, 128), (33, 384), (65, 2048),
                                 (127, 512), (2049, 128), (8193, 256)])
def test_edges(m, f):
    t = W.trn_inputs(m, seed=300 + m + f, f=f)
    print(f"\n[transition edges m={m} f={f}]", flush=True)
    out, _, _, (dx, *sums) = run(t)
    args = (t["x"], t["gamma"], t["beta"], t["w1"], t["w2"])
    close("out", out, OT.trn_fwd(*args)[0])
    ref = OT.trn_bwd(*args, t["dout"])
    close("dx", dx, ref[0])
    check_sums(sums, ref[1:])
