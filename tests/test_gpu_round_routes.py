"""Matmul rounds at the edges of their routes, byte for byte against the
oracle: one-entry and short tables, the longest table of the one-workgroup
rounds and the shortest wide one, a later product that folds in global memory
first, and a group of eight products."""
import numpy as np
import pytest

import workloads
from oracle.zkmat import prove_workload_group
from gpu_util import device_group

pytestmark = pytest.mark.gpu

CASES = [[(2, 1, 3)], [(1, 2, 1)], [(3, 33, 2)], [(2, 64, 2)], [(2, 513, 3)], [(3, 1024, 2)], [(2, 1025, 3)],
         [(3, 2049, 2), (3, 700, 2)], [(2, 40, 2), (2, 4000, 2)], [(2, 1, 3), (2, 2, 3)] + [(2, 5, 3)] * 6]


@pytest.mark.parametrize("mode", [1, 2])
def test_routes_match_oracle_bytes(mode):
    from paper_2508_21393_amd import binding as B
    groups = []
    for k, dims in enumerate(CASES):
        g = workloads.tiny_random_group(300 + k, dims, dtype=np.int16, name=f"route{k}")
        g.group_id = k
        groups.append(g)
    proofs, digests = B.sumcheck_matmul_prove([device_group(g, B) for g in groups], 31, mode=mode)
    for g, pr, dg in zip(groups, proofs, digests):
        want, st = prove_workload_group(g, 31)[:2]
        assert pr == want, g.name
        assert dg == st, g.name
