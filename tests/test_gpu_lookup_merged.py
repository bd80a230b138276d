"""Lookups whose first low round takes the last high round's step in its own
launch (tables of 2^9 to 2^15 rows), byte for byte against the oracle, on an
idle GPU and with another stream's products on its CUs."""
import pytest

import oracle.lookup as ol
import workloads
from gpu_util import to_dev
from lookup_util import lookup_args

pytestmark = pytest.mark.gpu

SEED = 7


@pytest.mark.parametrize("nL,factor,two", [(9, 3, False), (10, 2, True), (11, 5, False), (12, 2, False), (13, 2, True),
                                           (14, 2, False), (15, 2, False)])
def test_merged_first_low_round(nL, factor, two):
    import torch
    from paper_2508_21393_amd import binding as B
    N = 1 << nL
    lc = workloads.tiny_lookup(nL, factor * N - 3, N, t0=-N // 2, two_col=two, lid=2)
    want = ol.prove_case(lc, SEED)
    args = [lookup_args(lc, "device", to_dev)]
    proofs, digs = B.lookup_prove(args, SEED)
    assert proofs[0] == want[0] and digs[0] == want[1]
    a = torch.ones((2048, 2048), device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for _ in range(3):
        with torch.cuda.stream(side):
            for _ in range(8):
                c = a @ a
        proofs, digs = B.lookup_prove(args, SEED)
        assert proofs[0] == want[0] and digs[0] == want[1]
    torch.cuda.synchronize()
    assert float(c[0, 0]) == 2048.0
