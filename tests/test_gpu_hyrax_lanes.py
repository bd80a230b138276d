"""Commitments whose slices are shared by 4 to 64 lanes (a given split, or a
workspace for few slices), against the oracle (exact bytes): ragged rows in the
last workgroup, lanes without columns, empty rows."""
import numpy as np
import pytest

import oracle.hyrax as hy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,m,split,dtype", [
    (8191, 256, 4, "int16"), (4099, 256, 4, "int16"), (1, 130, 1, "int16"), (1, 65, 2, "int32"), (5, 300, 3, "int16"),
    (67, 129, 1, "int64"), (3, 70, 2, "int16"), (1000, 600, 1, "int16"), (4096, 300, 0, "int16"), (2, 700, 0, "int32")])
def test_shared_slices(R, m, split, dtype):
    import torch
    from paper_2508_21393_amd import binding as B
    rng = np.random.default_rng([R, m, split])
    kinds = 7       # distinct rows; the oracle adds their few nonzero entries one by one
    top = {"int16": 1 << 15, "int32": 1 << 31, "int64": 1 << 62}[dtype]
    rows = np.zeros((kinds, m), dtype=dtype)
    for i in range(1, kinds):
        cols = rng.choice(m, size=5, replace=False)
        rows[i, cols] = rng.integers(-top, top, size=5)
    rows[1, m - 1], rows[2, 0] = -top, top - 1
    gens = {j: hy.generator(j) for j in np.flatnonzero(rows.any(axis=0))}
    want = []
    for row in rows:
        acc = None
        for j in np.flatnonzero(row):
            k = int(row[j])
            acc = hy.add(acc, hy.mul(abs(k), gens[j] if k > 0 else hy.neg(gens[j])))
        want.append(hy.encode(acc))
    pick = rng.integers(0, kinds, size=R)
    T = B.HyraxTable(m, B.hyrax_windows(torch.empty(0, dtype=getattr(torch, dtype)).dtype))
    M = torch.from_numpy(rows[pick]).cuda()
    # without a split: room for one slice of a row in 256 columns
    need = B.hyrax_commit_workspace_size(R, m, split) if split else (R * 192 * -(-m // 256) + 255) // 256 * 256
    ws = torch.full((need + 256,), 0xa5, dtype=torch.uint8, device="cuda")
    got = B.hyrax_commit(M, T, workspace=ws[:need], split=split)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    assert all(bytes(got[i]) == want[pick[i]] for i in range(R))
    assert bool((ws[need:] == 0xa5).all())
