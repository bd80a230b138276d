"""Batched products whose rounds change route: all in one workgroup (up to
2^8 entries), one or more GPU-wide rounds, with the steps inside the sweeps or
launches of their own (2^19 entries), head rounds that end inside the
wide part or inside the workgroup, no head rounds, no inner rounds, no rounds;
byte for byte against the oracle."""
import pytest

import oracle.bmm as ob
import workloads
from bmm_util import bmm_args
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1, 1), (2, 1, 1, 1), (1, 3, 2, 2), (8, 2, 64, 2), (16, 3, 64, 2), (32, 2, 64, 3), (3, 2, 700, 2),
          (1000, 1, 2, 1), (1025, 2, 1, 1), (1, 2, 2049, 2), (5, 2, 1000, 3), (300, 1, 700, 1)]


@pytest.mark.parametrize("shape", SHAPES)
def test_routes_match_oracle(shape):
    from paper_2508_21393_amd import binding as B
    H, d0, d1, d2 = shape
    hb = workloads.tiny_head_batch(H + d1, H, d0, d1, d2)
    proofs, digs = B.bmm_prove([bmm_args(hb, "device", to_dev)], 17)
    want = ob.prove_batch(hb, 17)
    assert proofs[0] == want[0] and digs[0] == want[1]


def test_false_statement_is_refused_in_wide_rounds():
    from paper_2508_21393_amd import binding as B
    hb = workloads.tiny_head_batch(3, 4, 2, 700, 2)
    hb.C.base.reshape(-1)[5] += 1
    with pytest.raises(B.VLError) as e:
        B.bmm_prove([bmm_args(hb, "device", to_dev)], 17)
    assert e.value.status == B.VL_ERR_FALSE_STATEMENT
