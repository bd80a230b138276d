"""Hyrax commitments where the kernel's slices, runs of slices and exceptional
additions can go wrong, against the oracle (exact bytes)."""
import numpy as np
import pytest

import oracle.hyrax as hy

pytestmark = pytest.mark.gpu


def _commit(B, T, M, ws_bytes=None):
    import torch
    R, m = M.shape
    need = B.hyrax_commit_workspace_size(R, m) if ws_bytes is None else ws_bytes
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    out = B.hyrax_commit(torch.from_numpy(M).cuda(), T, workspace=ws)
    torch.cuda.synchronize()
    return [bytes(r) for r in out.cpu().numpy()]


@pytest.mark.parametrize("R,m", [(1, 1), (1, 3), (65, 5), (3, 1030), (1, 1200)])
def test_slices_and_runs(R, m):
    """Up to 300 slices of a row (the last one ragged), summed with and without the pass of runs;
    a workspace of one slice per 256 columns gives the same bytes, a smaller one is refused."""
    from paper_2508_21393_amd import binding as B
    rng = np.random.default_rng([R, m])
    M = rng.integers(-300, 300, size=(R, m)).astype(np.int16)
    M[rng.random((R, m)) < 0.9] = 0       # the oracle adds the nonzero entries one by one
    gens = {j: hy.generator(j) for j in np.flatnonzero(M.any(axis=0))}
    want = []
    for i in range(R):
        acc = None
        for j in np.flatnonzero(M[i]):
            k = int(M[i, j])
            acc = hy.add(acc, hy.mul(abs(k), gens[j] if k > 0 else hy.neg(gens[j])))
        want.append(hy.encode(acc))
    T = B.HyraxTable(m, 2)
    assert _commit(B, T, M) == want
    least = (R * 192 * -(-m // 256) + 255) // 256 * 256
    assert _commit(B, T, M, least) == want
    with pytest.raises(B.VLError):
        _commit(B, T, M, least - 256)


@pytest.mark.parametrize("far", [1, 5, 64])
def test_equal_and_opposite_points(far):
    """A table whose generator `far` repeats generator 0: equal points (a doubling) and
    opposite points (infinity) inside a lane's slice, across lanes and in longer sums."""
    from paper_2508_21393_amd import binding as B
    m = 130
    T = B.HyraxTable(m, 2)
    per = 2 * 128 * 96
    T.buf[far * per:(far + 1) * per] = T.buf[:per].clone()
    G, H = hy.generator(0), hy.generator(129)
    rows = [(7, 7, 0), (7, -7, 0), (-100, -100, 0), (300, 300, 5), (300, -300, 5), (1, 2, 0), (0, 0, 0), (5, -5, 1)]
    M = np.zeros((len(rows), m), dtype=np.int16)
    want = []
    for i, (a, b, c) in enumerate(rows):
        M[i, 0], M[i, far], M[i, 129] = a, b, c
        s = a + b
        acc = hy.mul(abs(s), G if s > 0 else hy.neg(G)) if s else None
        want.append(hy.encode(hy.add(acc, hy.mul(c, H) if c else None)))
    assert _commit(B, T, M) == want
