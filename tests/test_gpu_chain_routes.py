"""Chained layers whose claim reductions change route (row and column tables
around 2^8 to 2^10 entries, tables of one entry, and 2^16 entries, whose steps
are launches of their own), byte for byte against the
oracle."""
import pytest

import oracle.chain as oc
import workloads
from gpu_util import to_dev

pytestmark = pytest.mark.gpu


class _Dev:
    def __init__(self, w):
        for n in ("X", "W", "A", "B", "dY", "H", "G", "Y", "C2", "C4", "dA", "dB", "dX", "UA", "UB"):
            setattr(self, n, to_dev(getattr(w, n)))
        self.F, self.eta = w.F, w.eta


@pytest.mark.parametrize("T,d_in,d_out,r", [(1, 1, 1, 1), (2, 512, 3, 1), (513, 3, 2, 2), (5, 2, 1025, 3), (257, 2, 256, 1),
                                           (1, 1, 65535, 1)])
def test_routes_match_oracle(T, d_in, d_out, r):
    from paper_2508_21393_amd import binding as B
    w = workloads.tiny_layer(T + d_in, T, d_in, d_out, r)
    proof, dig = B.lora_chain_prove(B.LayerArgs(_Dev(w)), 23)
    want = oc.chain_prove(w, 23)
    assert proof == want[0] and dig == want[1]
