"""Wide rounds whose blocks take more than one run of pairs (tables of 2^18
entries and more): the bytes of the rounds in one workgroup, and a proof that the
host verifier accepts with the witness."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(1 << 17) + 1, (1 << 19) - 5, 1 << 20])
def test_long_inner_dimension(n):
    import torch
    from paper_2508_21393_amd import binding as B
    rng = np.random.default_rng(n)
    a = rng.integers(-300, 300, size=(3, n)).astype(np.int16)
    b = rng.integers(-300, 300, size=(n, 2)).astype(np.int16)
    c = a.astype(np.int64) @ b.astype(np.int64)
    g = B.GroupArgs(4, [(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), False, False)], torch.from_numpy(c).cuda())
    wide = B.sumcheck_matmul_prove([g], 8, mode=1)
    assert wide == B.sumcheck_matmul_prove([g], 8, mode=2)
    ok, fr, _ = B.verify_transcript(wide[0][0], B.GroupArgs(4, [(a, b, False, False)], c), 8)
    assert ok, fr
