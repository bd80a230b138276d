"""Rounds of long tables in one workgroup (persistent mode, later products of a
sum): whether a round is summed ahead of its challenge or after it, the bytes are
the oracle's, and a pair takes the seven products it needs."""
import time

import numpy as np
import pytest

import workloads
from oracle.zkmat import prove_workload_group
from gpu_util import device_group

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,mode", [([(2, 257, 2)], 2), ([(2, 1023, 2)], 2), ([(2, 1025, 2)], 2), ([(1, 8192, 2)], 2),
                                       ([(2, 3, 2), (2, 1025, 2)], 1), ([(2, 2048, 3), (2, 5000, 3)], 1),
                                       ([(2, 1100, 2), (2, 300, 2), (2, 1100, 2)], 2)])
def test_long_tables_match_oracle(dims, mode):
    from paper_2508_21393_amd import binding as B
    g = workloads.tiny_random_group(len(dims) + dims[-1][1], dims, dtype=np.int16, name="long")
    proofs, digests = B.sumcheck_matmul_prove([device_group(g, B)], 5, mode=mode)
    want = prove_workload_group(g, 5)
    assert proofs[0] == want[0] and digests[0] == want[1]


def test_time_of_a_pair():
    """2^18 entries in one workgroup: 11 ns a pair with 7 products each, 28 with the 21 that sums
    ahead of the challenge take.  The bytes are those of the rounds across the GPU."""
    import torch
    from paper_2508_21393_amd import binding as B
    n = 1 << 18
    gen = torch.Generator(device="cuda").manual_seed(3)
    a = torch.randint(-100, 100, (4, n), generator=gen, device="cuda", dtype=torch.int16)
    b = torch.randint(-100, 100, (n, 4), generator=gen, device="cuda", dtype=torch.int16)
    batch = B.GroupBatch([B.GroupArgs(0, [(a, b, False, False)], (a.double() @ b.double()).to(torch.int64))])
    ws = torch.empty(B.workspace_size(batch, 2), dtype=torch.uint8, device="cuda")
    got, best = None, 1.0
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        got = B.sumcheck_matmul_prove(batch, 5, mode=2, workspace=ws)
        best = min(best, time.perf_counter() - t)
    assert got == B.sumcheck_matmul_prove(batch, 5, mode=1)
    assert best < n * 18e-9, best
