"""GPU parity of the fused layer-norm + linear backward where its kernels
split: two, three and four leading outputs of 128 columns, none to sixteen
further columns in one or several narrow outputs, one column more than the
one-pass kernels take, rows that end inside a 32-row unit, and workgroups with
one or several units (each instance with and without narrow outputs past a
whole turn of its ring of three, four or five units in a workgroup).  Bounds
of test_lnl_gpu."""
import pytest

import oracle
from paper_2506_20686_amd import workloads as W

from test_lnl_gpu import EPS, close, run_bwd

pytestmark = pytest.mark.gpu

C = 128


@pytest.mark.parametrize("m,cols", [
    (1, (C, C)), (31, (C, C, 4)), (33, (C, C, C)), (95, (C, C, C, 8)), (100, (C, C, C, C)),
    (2047, (C, C, C, C, 4)), (9000, (C, C, C, C, 8)), (8193, (C, C, C, C, 16)),
    (300, (C, C, 4, 8, 4)), (300, (C, C, C, C, 4, 4, 4, 4)), (300, (C, C, 20)), (640, (C, C, C, 64)),
    (24600, (C, C, C, 12)), (24611, (C, C)), (33000, (C, C)), (24611, (C, C, 4)),
    (33000, (C, C, 8, 4)), (24611, (C, C, C)), (33000, (C, C, C)), (24611, (C, C, C, C)),
    (33000, (C, C, C, C)), (33001, (C, C, C, C, 4))])
def test_backward_widths(m, cols):
    t = W.lnl_inputs(m, cols, seed=500 + m)
    print(f"\n[ln_linear backward m={m} cols={cols}]", flush=True)
    dx, dw, dg, db = run_bwd(t)
    rdx, rdw, rdg, rdb = oracle.lnl_bwd(t["x"], t["gamma"], t["beta"], t["w"], t["do2"], EPS)
    close("dx", dx, rdx)
    close("dw", dw, rdw, row_sum=True)
    close("dgamma", dg, rdg, row_sum=True)
    close("dbeta", db, rdb, row_sum=True)
