"""The prover's workloads as timed cases.

A LoRA fine-tuning step is proved piece by piece: matrix products (single
calls, whole layers, a whole decoder block), the chained proof of a layer,
the per-head products of attention, lookups, commitments to the weights and
openings of committed tensors.  ``listed()`` names the cases, ``draw`` makes
more of the same ranges, ``prepare`` makes a case's inputs on the GPU with the
buffers a program keeps, and ``run`` is one call through the binding.  The
verifiers are CPU code of the verifier's machine and are not among them.

Tensors are integers with the distributions of quantised training: weights
N(0, 0.02^2) and activations N(0, 1) at scale 2^12, clipped to int16.
"""
import math

import numpy as np
import torch

from paper_2508_21393_amd import binding as B

SCALE = 4096.0
P = B.FR_MODULUS


# ----------------------------------------------------------------- cases ----
def listed():
    return [
        # the smallest call: one 64x128 . 128x32 product, a latency of launches and hashing
        {"name": "product_64x128x32", "kind": "product", "D0": 64, "D1": 128, "D2": 32, "dtype": "int16",
         "trans_a": False, "trans_b": False, "bind": True},
        # an ordinary request of the proof server: a 13B-class layer's forward products, asynchronous on its own stream
        {"name": "serve_13b_q_fwd_T128", "kind": "layer", "api": "async", "T": 128, "d_in": 5120, "d_out": 5120,
         "r": 8, "part": "fwd"},
        # a training step's block, T = 2048, one blocking call: latency
        {"name": "block_7b_T2048", "kind": "block", "api": "blocking", "T": 2048, "hidden": 4096, "ffn": 11008, "r": 16},
        # the same block through a captured prove graph, a pass following the other: throughput
        {"name": "block_7b_T2048_graph", "kind": "block", "api": "graph", "T": 2048, "hidden": 4096, "ffn": 11008,
         "r": 16},
        # the FFN-up layer's forward, backward and update in one transcript
        {"name": "chain_ffn_up_T512", "kind": "chain", "T": 512, "d_in": 4096, "d_out": 11008, "r": 16},
        # the six per-head products of a 7B-class attention layer
        {"name": "attention_7b_T2048", "kind": "attention", "T": 2048, "H": 32, "dh": 128},
        # a short ragged sequence with few heads
        {"name": "attention_ragged_T333", "kind": "attention", "T": 333, "H": 5, "dh": 80},
        # range check of one activation tensor, 2048 x 4096 entries
        {"name": "lookup_range_2^23", "kind": "lookup", "D": 1 << 23, "N": 1 << 16, "two_col": False,
         "dtype": "int16"},
        # SwiGLU's input/output check of a few tokens, a ragged number of entries
        {"name": "lookup_silu_ragged", "kind": "lookup", "D": 97 * 2753, "N": 1 << 16, "two_col": True,
         "dtype": "int16"},
        # commitment to a frozen attention weight
        {"name": "commit_4096x4096", "kind": "commit", "R": 4096, "m": 4096, "dtype": "int16"},
        # commitment to a LoRA B matrix after its update
        {"name": "commit_lora_16x11008", "kind": "commit", "R": 16, "m": 11008, "dtype": "int16"},
        # opening of a layer's int64 output at the claim's row point
        {"name": "open_out_2048x11008", "kind": "open", "R": 2048, "m": 11008, "dtype": "int64"},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["product", "product", "layer", "layer", "block", "chain", "attention", "lookup", "lookup",
                       "commit", "commit", "open", "open"])
    if kind == "product":
        return {"kind": kind, "D0": _log_int(rng, 1, 2048), "D1": _log_int(rng, 16, 11008),
                "D2": _log_int(rng, 1, 5120), "dtype": rng.choice(["int16", "int16", "int32"]),
                "trans_a": rng.random() < 0.5, "trans_b": rng.random() < 0.5, "bind": rng.random() < 0.5}
    if kind == "layer":
        return {"kind": kind, "api": rng.choice(["async", "blocking", "graph"]), "T": _log_int(rng, 64, 2048),
                "d_in": _log_int(rng, 512, 5120), "d_out": _log_int(rng, 512, 11008), "r": rng.choice([8, 16, 64]),
                "part": rng.choice(["fwd", "bwd", "upd"])}
    if kind == "block":
        hidden = 64 * _log_int(rng, 8, 64)
        return {"kind": kind, "api": rng.choice(["blocking", "graph"]), "T": _log_int(rng, 128, 2048),
                "hidden": hidden, "ffn": (hidden * 43 // 16) & ~7, "r": rng.choice([8, 16])}
    if kind == "chain":
        return {"kind": kind, "T": _log_int(rng, 32, 512), "d_in": _log_int(rng, 256, 4096),
                "d_out": _log_int(rng, 256, 11008), "r": rng.choice([8, 16])}
    if kind == "attention":
        return {"kind": kind, "T": _log_int(rng, 64, 2048), "H": rng.randint(2, 32), "dh": rng.choice([64, 80, 96, 128])}
    if kind == "lookup":
        return {"kind": kind, "D": _log_int(rng, 1 << 12, 1 << 23), "N": 1 << rng.randint(10, 16),
                "two_col": rng.random() < 0.5, "dtype": rng.choice(["int16", "int16", "int32"])}
    if kind == "commit":
        return {"kind": kind, "R": _log_int(rng, 8, 2048), "m": _log_int(rng, 8, 4096),
                "dtype": rng.choice(["int16", "int16", "int32"])}
    return {"kind": "open", "R": _log_int(rng, 16, 2048), "m": _log_int(rng, 16, 11008),
            "dtype": rng.choice(["int16", "int32", "int64"])}


# ---------------------------------------------------------------- inputs ----
def _gen(seed, salt):
    return torch.Generator(device="cuda").manual_seed(1000003 * int(seed) + salt)


def _gauss(g, shape, sigma, dtype=torch.int16, top=32767):
    x = torch.randn(shape, generator=g, device="cuda") * (sigma * SCALE)
    return x.round_().clamp_(-top - 1, top).to(dtype)


def _mm(a, b):
    """Exact product: every partial sum is an integer below 2^53."""
    return (a.double() @ b.double()).to(torch.int64)


def _requant(z):
    return ((z + 2048) >> 12).clamp_(-32768, 32767).to(torch.int16)


class _Layer:
    """One LoRA-adapted linear layer: Y = X W + (X A) B and its gradients."""

    def __init__(self, g, T, d_in, d_out, r, X=None):
        self.X = _gauss(g, (T, d_in), 1.0) if X is None else X
        self.W = _gauss(g, (d_in, d_out), 0.02)
        self.A = _gauss(g, (d_in, r), 0.02)
        self.B = _gauss(g, (r, d_out), 0.02)
        self.dY = _gauss(g, (T, d_out), 1.0)
        self.C2 = _mm(self.X, self.A)
        self.C4 = _mm(self.dY, self.B.t())
        self.H = _requant(self.C2)
        self.G = _requant(self.C4)

    def groups(self, part, first):
        """vl_group arguments of the forward, backward or update products."""
        X, W, A, Bm, dY, H, G = self.X, self.W, self.A, self.B, self.dY, self.H, self.G
        out = []

        def add(C, *prods):
            out.append(B.GroupArgs(first + len(out), list(prods), C))

        if part in ("fwd", "all"):
            add(_mm(X, W), (X, W, False, False))
            add(self.C2, (X, A, False, False))
            add(_mm(H, Bm), (H, Bm, False, False))
        if part in ("bwd", "all"):
            add(self.C4, (dY, Bm, False, True))
            add(_mm(dY, W.t()) + _mm(G, A.t()), (dY, W, False, True), (G, A, False, True))
        if part in ("upd", "all"):
            add(_mm(X.t(), G), (X, G, True, False))
            add(_mm(H.t(), dY), (H, dY, True, False))
        return out


class _Bag:
    pass


def _groups_of(case, seed):
    kind = case["kind"]
    if kind == "product":
        g = _gen(seed, 1)
        d0, d1, d2 = case["D0"], case["D1"], case["D2"]
        if case["dtype"] == "int16":
            a = torch.randint(-32768, 32768, (d0, d1), generator=g, device="cuda", dtype=torch.int16)
            b = torch.randint(-32768, 32768, (d1, d2), generator=g, device="cuda", dtype=torch.int16)
        else:
            a = _gauss(g, (d0, d1), 8.0, torch.int32, (1 << 18) - 1)
            b = _gauss(g, (d1, d2), 8.0, torch.int32, (1 << 18) - 1)
        C = _mm(a, b)
        ta, tb = bool(case["trans_a"]), bool(case["trans_b"])
        A = a.t().contiguous() if ta else a
        Bm = b.t().contiguous() if tb else b
        bind = bytes((seed * 31 + 7 * i) & 255 for i in range(32)) if case["bind"] else None
        return [B.GroupArgs(0, [(A, Bm, ta, tb)], C, bind=bind)]
    if kind == "layer":
        return _Layer(_gen(seed, 2), case["T"], case["d_in"], case["d_out"], case["r"]).groups(case["part"], 0)
    g = _gen(seed, 3)
    T, hid, ffn, r = case["T"], case["hidden"], case["ffn"], case["r"]
    xa, xo, xm = (_gauss(g, (T, hid), 1.0) for _ in range(3))
    xd = _gauss(g, (T, ffn), 1.0)
    out = []
    for X, d_in, d_out in ((xa, hid, hid), (xa, hid, hid), (xa, hid, hid), (xo, hid, hid), (xm, hid, ffn),
                           (xm, hid, ffn), (xd, ffn, hid)):
        out += _Layer(g, T, d_in, d_out, r, X).groups("all", len(out))
    return out


def _attention(case, seed):
    g = _gen(seed, 4)
    T, H, dh = case["T"], case["H"], case["dh"]
    Q, K, V, dO = (_gauss(g, (T, H * dh), 1.0) for _ in range(4))
    dS = _gauss(g, (H, T, T), 1.0)
    P_ = torch.empty((H, T, T), dtype=torch.int16, device="cuda")
    S, dP = (torch.empty((H, T, T), dtype=torch.int64, device="cuda") for _ in range(2))
    O, dV, dQ, dK = (torch.empty((T, H * dh), dtype=torch.int64, device="cuda") for _ in range(4))
    for h in range(H):
        c = slice(h * dh, (h + 1) * dh)
        q, k, v, do, ds = Q[:, c].double(), K[:, c].double(), V[:, c].double(), dO[:, c].double(), dS[h].double()
        s = q @ k.t()
        S[h] = s.to(torch.int64)
        p = (torch.softmax(s / (2.0 ** 24 * math.sqrt(dh)), dim=1) * SCALE).round_()
        P_[h] = p.to(torch.int16)
        O[:, c] = (p @ v).to(torch.int64)
        dP[h] = (do @ v.t()).to(torch.int64)
        dV[:, c] = (p.t() @ do).to(torch.int64)
        dQ[:, c] = (ds @ k).to(torch.int64)
        dK[:, c] = (ds.t() @ q).to(torch.int64)
    W, n = H * dh, T * T
    wide, tall = (W, dh), (T, n)   # (leading dimension, head stride)

    def bmm(i, A, Bm, C, d1, d2, la, lb, lc, ta, tb):
        return B.BmmArgs(A, Bm, C, H, T, d1, d2, la[0], lb[0], lc[0], la[1], lb[1], lc[1], ta, tb, group_id=i)

    return [bmm(0, Q, K, S, dh, T, wide, wide, tall, False, True),
            bmm(1, P_, V, O, T, dh, tall, wide, wide, False, False),
            bmm(2, dO, V, dP, dh, T, wide, wide, tall, False, True),
            bmm(3, P_, dO, dV, T, dh, tall, wide, wide, True, False),
            bmm(4, dS, K, dQ, T, dh, tall, wide, wide, False, False),
            bmm(5, dS, Q, dK, T, dh, tall, wide, wide, True, False)]


def _lookup(case, seed):
    g = _gen(seed, 5)
    D, N = case["D"], case["N"]
    dt = torch.int16 if case["dtype"] == "int16" else torch.int32
    t0 = -(N // 2)
    # activations at the scale that spreads them over the table (2^12 for the int16 range)
    x = (torch.randn((D,), generator=g, device="cuda") * (N / 16.0)).round_().clamp_(t0, t0 + N - 1).to(dt)
    if not case["two_col"]:
        return B.LookupArgs(x, None, None, t0, N, D, x.dtype, False, 0)
    s = torch.arange(t0, t0 + N, dtype=torch.float64) / (N / 16.0)
    tb = (s * torch.sigmoid(s) * (N / 16.0)).round().to(torch.int32).cuda()
    y = tb[x.long() - t0].to(dt)
    return B.LookupArgs(x, y, tb, t0, N, D, x.dtype, True, 0, dtype_y=y.dtype)


def _matrix(case, seed):
    """A committed or opened tensor: weights, updates or a layer's output."""
    g = _gen(seed, 6)
    shape = (case["R"], case["m"])
    if case["dtype"] == "int16":
        return _gauss(g, shape, 0.02)
    if case["dtype"] == "int32":
        return _gauss(g, shape, 4.0, torch.int32, (1 << 30) - 1)
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float64) * 2.0 ** 28).round_().to(torch.int64)


def _point(case, seed):
    g = np.random.default_rng([int(seed), 7])
    n = max(0, (case["R"] - 1).bit_length())
    return [int.from_bytes(g.bytes(40), "little") % P for _ in range(n)]


def prepare(case, seed):
    s = _Bag()
    s.case, s.kind, s.seed = case, case["kind"], int(seed) + 11
    kind = s.kind
    u8 = dict(dtype=torch.uint8, device="cuda")
    if kind in ("product", "layer", "block"):
        s.api = case.get("api", "blocking")
        s.batch = B.GroupBatch(_groups_of(case, seed))
        s.ws = torch.empty(max(256, B.workspace_size(s.batch, async_=s.api != "blocking")), **u8)
        if s.api != "blocking":
            s.stream = torch.cuda.Stream()
            s.proofs = torch.zeros(s.batch.total, dtype=torch.uint8, pin_memory=True)
            s.status = torch.zeros(len(s.batch), dtype=torch.int32, pin_memory=True)
            s.stream.wait_stream(torch.cuda.current_stream())
        if s.api == "graph":
            s.graph = B.ProveGraph(s.batch, s.ws, s.proofs, s.status)
    elif kind == "chain":
        L = _Layer(_gen(seed, 8), case["T"], case["d_in"], case["d_out"], case["r"])
        L.F, L.eta = 12, 3
        L.Y = _mm(L.X, L.W) + _mm(L.H, L.B)
        L.dA, L.dB = _mm(L.X.t(), L.G), _mm(L.H.t(), L.dY)
        L.dX = _mm(L.dY, L.W.t()) + _mm(L.G, L.A.t())
        L.UA = (L.A.to(torch.int64) << L.F) - L.eta * L.dA
        L.UB = (L.B.to(torch.int64) << L.F) - L.eta * L.dB
        s.layer = B.LayerArgs(L)
        s.ws = torch.empty(max(256, B.lora_chain_workspace_size(s.layer)), **u8)
    elif kind == "attention":
        s.batches = _attention(case, seed)
        s.ws = torch.empty(max(256, B.bmm_workspace_size(s.batches)), **u8)
    elif kind == "lookup":
        s.args = [_lookup(case, seed)]
        s.ws = torch.empty(max(256, B.lookup_workspace_size(s.args)), **u8)
    else:
        s.M = _matrix(case, seed)
        R, m = case["R"], case["m"]
        if kind == "commit":
            s.table = B.HyraxTable(m, B.hyrax_windows(s.M.dtype))
            s.out = torch.empty((R, B.HYRAX_POINT_BYTES), **u8)
            s.ws = torch.empty(max(256, B.hyrax_commit_workspace_size(R, m)), **u8)
        else:
            s.x = _point(case, seed)
            n_eq = 1 << len(s.x)
            s.eq = torch.empty((8, n_eq), dtype=torch.int32, device="cuda")
            s.w = torch.empty((8, m), dtype=torch.int32, device="cuda")
            s.canon = torch.empty((m, 8), dtype=torch.int32, device="cuda")
            s.ws = torch.empty(max(256, B.partial_eval_workspace_size(R, m, B.VL_CONTRACT_ROWS, s.M.dtype)), **u8)
    return s


# ------------------------------------------------------------------- run ----
def _bytes(proofs, digests):
    return [np.frombuffer(b"".join(proofs), dtype=np.uint8), np.frombuffer(b"".join(digests), dtype=np.uint8)]


def run(s):
    kind = s.kind
    if kind in ("product", "layer", "block"):
        if s.api == "blocking":
            return _bytes(*B.sumcheck_matmul_prove(s.batch, s.seed, workspace=s.ws))
        if s.api == "async":
            B.sumcheck_matmul_prove_async(s.batch, s.seed, s.proofs, s.status, s.ws, stream=s.stream)
        else:
            s.graph.launch(s.seed, stream=s.stream)
        return [s.proofs, s.status]
    if kind == "chain":
        proof, digest = B.lora_chain_prove(s.layer, s.seed, workspace=s.ws)
        return _bytes([proof], [digest])
    if kind == "attention":
        return _bytes(*B.bmm_prove(s.batches, s.seed, workspace=s.ws))
    if kind == "lookup":
        return _bytes(*B.lookup_prove(s.args, s.seed, workspace=s.ws))
    if kind == "commit":
        return B.hyrax_commit(s.M, s.table, out=s.out, workspace=s.ws)
    # the opening message w = sum_i eq(x, i) M[i][.], canonical
    B.eq_table(s.x, B.fr_vec(s.eq))
    B.mle_partial_eval(s.M, B.VL_CONTRACT_ROWS, B.fr_vec(s.eq), B.fr_vec(s.w), s.ws)
    B.fr_export(B.fr_vec(s.w), s.case["m"], s.canon)
    return s.canon


# ------------------------------------------------------------------ work ----
FR_MUL = 128      # 32-bit multiply-adds of one Montgomery product in Fr
FQ_MUL = 288      # and in Fq
SIZE = {"int16": 2, "int32": 4, "int64": 8}
MACS = {"int16": 8, "int32": 16, "int64": 16}   # digit multiply-adds per contracted entry


def _log2(n):
    return max(0, (int(n) - 1).bit_length())


def _product_work(d0, d1, d2, dtype, out=True):
    """(bytes, multiply-adds) of one product: A and B once, C once per group."""
    e = d0 * d1 + d1 * d2
    b, m = e * SIZE[dtype], e * MACS[dtype]
    if out:
        b, m = b + 8 * d0 * d2, m + 16 * d0 * d2
    n1 = _log2(d1)
    return b + 32 * (3 * n1 + 3), m + 5 * FR_MUL * (1 << n1)


def _layer_work(T, i, o, r, part):
    dims = {"fwd": [(T, i, o, 1), (T, i, r, 1), (T, r, o, 1)],
            "bwd": [(T, o, r, 1), (T, o, i, 1), (T, r, i, 0)],
            "upd": [(i, T, r, 1), (r, T, o, 1)]}
    use = dims["fwd"] + dims["bwd"] + dims["upd"] if part == "all" else dims[part]
    w = [_product_work(a, b, c, "int16", bool(k)) for a, b, c, k in use]
    return sum(x[0] for x in w), sum(x[1] for x in w)


def work(case):
    """Bytes: each input read once, each output written once.  flops: two per
    32-bit multiply-add of the exact arithmetic."""
    k = case["kind"]
    if k == "product":
        b, m = _product_work(case["D0"], case["D1"], case["D2"], case["dtype"])
    elif k == "layer":
        b, m = _layer_work(case["T"], case["d_in"], case["d_out"], case["r"], case["part"])
    elif k == "chain":
        b, m = _layer_work(case["T"], case["d_in"], case["d_out"], case["r"], "all")
    elif k == "block":
        T, h, f, r = case["T"], case["hidden"], case["ffn"], case["r"]
        w = [_layer_work(T, i, o, r, "all") for i, o in [(h, h)] * 4 + [(h, f)] * 2 + [(f, h)]]
        b, m = sum(x[0] for x in w), sum(x[1] for x in w)
    elif k == "attention":
        T, H, d = case["T"], case["H"], case["dh"]
        w = [_product_work(T, d, T, "int16")] * 2 + [_product_work(T, T, d, "int16")] * 4
        b, m = H * sum(x[0] for x in w), H * sum(x[1] for x in w)
    elif k == "lookup":
        D, N = 1 << _log2(max(case["D"], case["N"])), case["N"]
        cols = 2 if case["two_col"] else 1
        b = case["D"] * SIZE[case["dtype"]] * cols + (4 * N if cols == 2 else 0)
        # two folds and three products per entry over all rounds, an inverse per table row
        m = FR_MUL * (5 * D + 16 * N)
    elif k == "commit":
        e = case["R"] * case["m"]
        digits = {"int16": 1.12, "int32": 2.0}[case["dtype"]]
        b = e * SIZE[case["dtype"]] + 96 * (case["R"] + case["m"])
        m = e * digits * 10 * FQ_MUL
    else:
        e = case["R"] * case["m"]
        b = e * SIZE[case["dtype"]] + 32 * case["m"]
        m = e * MACS[case["dtype"]] + FR_MUL * (2 * case["R"] + 2 * case["m"])
    return {"bytes": float(b), "flops": 2.0 * m}


# ----------------------------------------------------------------- exact ----
def exact(case, seed):
    """The opening message in plain integers.  Proofs and commitments are
    bytes that either agree or do not, and have no value here."""
    if case["kind"] != "open":
        return None
    M = _matrix(case, seed).cpu().numpy()
    eq = [1]
    for x in _point(case, seed):
        eq = [v for e in eq for v in (e * (1 - x) % P, e * x % P)]
    limbs = np.array([[(e >> (16 * k)) & 0xffff for e in eq[:case["R"]]] for k in range(16)], dtype=np.float64)
    # 16-bit limbs times 16-bit pieces of the entries: every sum is an integer below 2^53
    w = [0] * case["m"]
    hi, shift = M.astype(np.int64), 0
    for piece in range(SIZE[case["dtype"]] // 2):
        last = piece == SIZE[case["dtype"]] // 2 - 1
        low = hi if last else hi & 0xffff
        sums = (limbs @ low.astype(np.float64)).astype(np.int64)
        for j in range(case["m"]):
            w[j] += sum(int(sums[k, j]) << (16 * k) for k in range(16)) << shift
        hi, shift = hi >> 16, shift + 16
    raw = b"".join((v % P).to_bytes(32, "little") for v in w)
    return torch.from_numpy(np.frombuffer(raw, dtype=np.int32).reshape(case["m"], 8).copy())
