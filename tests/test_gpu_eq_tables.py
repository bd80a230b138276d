"""eq tables around a block's 2^8 entries and at the largest size, against the
product of the entry's factors (exact)."""
import random

import pytest

from oracle.field import P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [0, 1, 4, 7, 8, 9, 13, 20])
def test_entries(n):
    import torch
    from paper_2508_21393_amd import binding as B
    rng = random.Random(n)
    x = [rng.randrange(P) for _ in range(n)]
    L = 1 << n
    eq = torch.zeros((8, L), dtype=torch.int32, device="cuda")
    out = torch.zeros((L, 8), dtype=torch.int32, device="cuda")
    B.eq_table(x, B.fr_vec(eq))
    B.fr_export(B.fr_vec(eq), L, out)
    w = out.cpu().numpy().view("uint32")
    for i in {0, L - 1, L // 2} | {rng.randrange(L) for _ in range(300)}:
        v = 1
        for j in range(n):
            v = v * (x[j] if (i >> (n - 1 - j)) & 1 else 1 - x[j]) % P
        assert sum(int(w[i, k]) << (32 * k) for k in range(8)) == v, i
