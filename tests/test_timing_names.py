"""The numbering of the timed kernels (CPU): callers hold indices, mask bits and
names, so none may move."""
from paper_2506_20686_amd import binding as B

NAMES = ["prep_bias", "prep_kbits", "fwd", "bwd_prep", "bwd_pad", "dq", "dkdv", "db", "db_reduce",
         "lnl_fwd", "lnl_bwd_dx", "lnl_bwd_g", "lnl_reduce", "lnl_finish", "trn_pack", "trn_fwd",
         "trn_bwd_dx", "trn_bwd_w", "trn_reduce", "trn_finish", "pad16"]


def test_indices_and_names():
    for i, name in enumerate(NAMES):
        got = B.tri_attn_timing_read(i)
        assert got is not None and got[0] == name, (i, got)
