"""Device field products at the values where limb arithmetic can go wrong:
zero, one, p - 1, values of all-ones 29-bit or 32-bit limbs and values next to
the limb boundaries, against Python integers (exact)."""
import random

import pytest

from oracle.field import P

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 2, P - 1, P - 2, (P + 1) // 2, (1 << 254) - 1, (1 << 255) % P] + \
    [v for k in (28, 29, 32, 58, 64, 232, 233, 253) for v in ((1 << k) - 1, 1 << k)] + \
    [sum(0x1fffffff << (29 * j) for j in range(0, 9, 2)) % P, sum(0xffffffff << (32 * j) for j in range(0, 8, 2)) % P]


@pytest.mark.parametrize("seed", range(4))
def test_products_of_edge_values(seed):
    """eq(x, .) over three variables is all products of x_j and 1 - x_j."""
    import torch
    from paper_2508_21393_amd import binding as B
    rng = random.Random(seed)
    points = [[rng.choice(EDGES) for _ in range(3)] for _ in range(24)] + [[rng.randrange(P) for _ in range(3)]]
    for x in points:
        eq = torch.zeros((8, 8), dtype=torch.int32, device="cuda")
        out = torch.zeros((8, 8), dtype=torch.int32, device="cuda")
        B.eq_table(x, B.fr_vec(eq))
        B.fr_export(B.fr_vec(eq), 8, out)
        w = out.cpu().numpy().view("uint32")
        got = [sum(int(w[i, k]) << (32 * k) for k in range(8)) for i in range(8)]
        want = []
        for i in range(8):
            v = 1
            for j in range(3):
                v = v * (x[j] if (i >> (2 - j)) & 1 else 1 - x[j]) % P
            want.append(v)
        assert got == want, x
