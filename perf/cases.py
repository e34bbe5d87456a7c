"""Timed cases of the self-attention library, through its Python binding.

A case is one call as a program makes it: inputs and weights on the GPU, a context (or the fixed-workspace
entry point), one forward pass into the caller's output.  Inputs follow the repository's recipe: X ~ N(0, 1),
W ~ N(0, 1 / d_model), drawn from the seed.  `listed` holds the repository's five workloads and the other kinds
of call the entry points take (the q = k = v scheme, float storage, head sizes off the matrix-core path, ragged
sizes, a short prompt on the fixed workspace); `draw` gives more of the same ranges.
"""
import math

import torch

from paper_2012_01114_amd import attnring as ar

FULL, SYM, CAUSAL = ar.ATTN_SCHEME_FULL, ar.ATTN_SCHEME_SYMMETRIC, ar.ATTN_SCHEME_CAUSAL
ENTRIES = ("forward", "static", "packed")


def _case(entry, dtype, scheme, batch, rows, parts, d_model, heads, d_k, lengths=False, skip_rows=False, fuse_q=False,
          project=True):
    """`rows` vectors per ring partition and `parts` partitions: n = rows * parts.  `lengths`: items of different
    lengths (key lengths, or the packed layout's own); `project` False: the q = k = v scheme on X itself."""
    return {"entry": entry, "dtype": dtype, "scheme": scheme, "batch": batch, "n": rows * parts, "p": parts,
            "d_model": d_model, "heads": heads, "d_k": d_k, "lengths": lengths, "skip_rows": skip_rows, "fuse_q": fuse_q,
            "project": project}


def listed():
    return [
        # the smallest call: 16 vectors in float, one head; launches and latency are all of it
        dict(_case("forward", "f32", FULL, 1, 4, 4, 64, 1, 64), name="tiny_f32"),
        # a short prompt of one user, masked, on the fixed workspace (no context, no allocation): 200 rows, ragged
        dict(_case("static", "bf16", CAUSAL, 1, 8, 25, 768, 12, 64), name="prompt_static"),
        # bidirectional encoder layer
        dict(_case("forward", "bf16", FULL, 8, 8, 64, 768, 12, 64), name="encoder"),
        # decoder layer, masked
        dict(_case("forward", "bf16", CAUSAL, 8, 8, 128, 768, 12, 64), name="causal"),
        # one long masked sequence with wide heads: the largest call
        dict(_case("forward", "bf16", CAUSAL, 1, 32, 256, 4096, 32, 128), name="long"),
        # padded batch of different lengths, every query row produced
        dict(_case("forward", "bf16", CAUSAL, 32, 8, 256, 1024, 16, 64, lengths=True), name="padded"),
        # the same batch stored back to back
        dict(_case("packed", "bf16", CAUSAL, 32, 8, 256, 1024, 16, 64, lengths=True), name="packed"),
        # encoder layer with one set of vectors in all three roles
        dict(_case("forward", "bf16", SYM, 8, 8, 64, 768, 12, 64), name="encoder_reuse"),
        # encoder layer in float storage, as used where 16 bits are not enough
        dict(_case("forward", "f32", FULL, 8, 8, 64, 768, 12, 64), name="encoder_f32"),
        # q = k = v in float
        dict(_case("forward", "f32", SYM, 2, 8, 64, 768, 12, 64), name="reuse_f32"),
        # 16-bit storage with a head size between the matrix-core ones, masked
        dict(_case("forward", "bf16", CAUSAL, 4, 8, 75, 640, 8, 80), name="head80"),
        # ragged in every size: last row tile nearly empty, d_model not in whole 64-deep slices
        dict(_case("forward", "bf16", FULL, 3, 4, 275, 1000, 8, 128), name="ragged_d128"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more call of the kinds above.  Matrix-core calls up to 6e11 operations and 8192 rows, calls on float
    arithmetic up to 2.1e10 (the listed encoder layer) and 2048 rows."""
    while True:
        kind = rng.choices(["matrix", "reuse", "float"], [0.6, 0.12, 0.28])[0]
        rows = rng.choice([4, 7, 8, 8, 8, 13, 16, 32])
        heads = rng.choice([1, 2, 3, 4, 8, 8, 12, 16, 32])
        batch = _log_int(rng, 1, 32)
        if kind == "float":
            dtype = rng.choice(["f32", "f32", "bf16"])
            d_k = rng.choice([32, 64, 64, 128] if dtype == "f32" else [20, 32, 48, 80, 96, 160, 256])
            n = _log_int(rng, 16, 2048)
            scheme = rng.choice([FULL, CAUSAL, CAUSAL, SYM])
            d_model = heads * d_k if rng.random() < 0.6 else _log_int(rng, 16, 1024)
            c = _case("forward", dtype, scheme, batch, rows, max(1, n // rows), d_model, heads, d_k)
            if scheme == SYM:
                c["project"] = not (d_model == heads * d_k and rng.random() < 0.3)
            if scheme == SYM and batch * heads * c["n"] ** 2 * 4 > 1 << 30:  # score matrices bounded by 1 GiB
                continue
            most, least = 2.1e10, 1e5
        else:
            d_k = rng.choice([64, 64, 128])
            n = _log_int(rng, 64, 8192 if kind == "matrix" else 2048)
            d_model = heads * d_k if rng.random() < 0.6 else 64 * _log_int(rng, 1, 64)
            if rng.random() < 0.2:
                d_model = max(8, d_model - 8 * rng.randrange(1, 8))
            c = _case("forward", "bf16", SYM if kind == "reuse" else rng.choice([FULL, CAUSAL]), batch, rows,
                      max(1, n // rows), d_model, heads, d_k)
            if kind == "matrix":
                scratch = 3 * batch * -(-c["n"] // 256) * 256 * heads * d_k * 2 + (130 << 10)
                if d_model % 64 == 0 and heads * d_k % 128 == 0 and scratch <= ar.ATTN_STATIC_SCRATCH_MIB << 20 and rng.random() < 0.3:
                    c["entry"] = "static"
                elif rng.random() < 0.1:
                    c["entry"] = "packed"
                c["fuse_q"] = c["entry"] == "forward" and rng.random() < 0.08
            most, least = 6e11, 1e7
        if c["scheme"] != SYM:
            c["lengths"] = c["entry"] == "packed" or rng.random() < 0.25
            c["skip_rows"] = c["lengths"] and c["entry"] != "packed" and rng.random() < 0.5
        elif c["dtype"] == "bf16" and c["d_k"] in (64, 128):  # partial row states bounded by 1 GiB
            tiles = -(-c["n"] // 128)
            if batch * heads * tiles * tiles * 128 * (d_k + 2) * 4 > 1 << 30:
                continue
        if batch * heads * c["n"] * c["d_k"] > 1 << 27 or batch * c["n"] * c["d_model"] > 1 << 27:
            continue
        if least <= work(c)["flops"] <= most:
            return c


def _shortest(case):
    """Lengths are uniform in _shortest .. n (64 .. 2048 for the padded workload)."""
    return max(1, case["n"] // 32)


def _inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    B, n, D, hd = case["batch"], case["n"], case["d_model"], case["heads"] * case["d_k"]
    lens = None
    if case["lengths"]:
        lo = _shortest(case)
        lens = torch.randint(lo, n + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
        lens[1::2] = lo + n - lens[0:B - 1:2]  # in pairs that add up to the same: the number of rows is the case's
        if B % 2:
            lens[B - 1] = (lo + n) // 2
    W = [(torch.randn(D, hd, generator=g, device="cuda") * D ** -0.5).to(dtype) if case["project"] else None for _ in range(3)]
    if case["scheme"] == SYM:
        W[1] = W[2] = None
    if case["entry"] == "packed":
        X = torch.randn(int(lens.sum()), D, generator=g, device="cuda").to(dtype)
    else:
        X = torch.randn(B, n, D, generator=g, device="cuda").to(dtype)
    return X, W, lens


class _State:
    """What a program holds between calls."""

    def __init__(self, case, seed):
        self.case, self.ctx = case, None
        self.X, self.W, self.lens = _inputs(case, seed)
        hd = case["heads"] * case["d_k"]
        self.out = torch.empty(*self.X.shape[:-1], hd, dtype=self.X.dtype, device="cuda")
        self.shape = (case["batch"], case["n"], case["d_model"], case["heads"], case["d_k"], case["p"],
                      ar.ATTN_F32 if case["dtype"] == "f32" else ar.ATTN_BF16)
        self.flags = (ar.ATTN_FLAG_SKIP_PADDED_ROWS if case["skip_rows"] else 0) | \
                     (ar.ATTN_FLAG_FUSE_Q_PROJECTION if case["fuse_q"] else 0)
        if case["entry"] != "static":
            self.ctx = ar.attn_init(*self.shape, 0.0, self.flags)
        if case["entry"] == "forward":
            ar.attn_set_key_lengths(self.ctx, self.lens)
        elif case["entry"] == "packed":
            self.first_rows = torch.zeros(case["batch"] + 1, dtype=torch.int32, device="cuda")
            self.first_rows[1:] = self.lens.cumsum(0)

    def __del__(self):
        if self.ctx is not None:
            torch.cuda.synchronize()
            ar.attn_destroy(self.ctx)


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    Wq, Wk, Wv = state.W
    scheme = state.case["scheme"]
    if state.case["entry"] == "static":
        ar.attn_forward_static(*state.shape, state.X, Wq, Wk, Wv, scheme, state.out, lens_dev=state.lens, scale=0.0,
                               flags=state.flags)
    elif state.case["entry"] == "packed":
        ar.attn_forward_packed(state.ctx, state.first_rows, state.X, Wq, Wk, Wv, scheme, state.out)
    else:
        ar.attn_forward(state.ctx, state.X, Wq, Wk, Wv, scheme, state.out)
    return state.out


def work(case):
    """Inputs read once, outputs written once; operations of the needed rows and pairs (their expectation where the
    lengths are drawn)."""
    B, n, D, H, d = case["batch"], case["n"], case["d_model"], case["heads"], case["d_k"]
    hd, size = H * d, 4 if case["dtype"] == "f32" else 2
    lo, hi = (_shortest(case), n) if case["lengths"] else (n, n)
    count = hi - lo + 1
    L = (lo + hi) / 2
    L2 = sum(x * x for x in range(lo, hi + 1)) / count
    short = case["skip_rows"] or case["entry"] == "packed"  # rows past the length are no queries either
    q_rows = L if short else n
    if case["scheme"] == SYM:
        project = (1 if case["project"] else 0) * n
        pairs2 = n * (n + 1) / 2 + n * n
    else:
        project = q_rows + 2 * L
        if case["scheme"] == FULL:
            pairs2 = 2 * (L2 if short else n * L)
        else:
            pairs2 = 2 * ((L2 + L) / 2 + (0 if short else n * L - L2))
    matrices = (0 if not case["project"] else 1) if case["scheme"] == SYM else 3
    stored = L if case["entry"] == "packed" else n
    return {"bytes": size * (B * q_rows * D + matrices * D * hd + B * stored * hd),
            "flops": B * (2.0 * project * D * hd + 2.0 * d * H * pairs2)}


def tolerance(case):
    # float: measured against `exact` 2e-7 .. 8e-7; 16 bits: 1.6e-3 .. 1.9e-3, the rounding of the output, of which
    # another implementation's outputs differ by about the same again
    return {"rel": 4e-6} if case["dtype"] == "f32" else {"rel": 8e-3}


def exact(case, seed):
    X, W, lens = _inputs(case, seed)
    B, n, H, d = case["batch"], case["n"], case["heads"], case["d_k"]
    scale = 1.0 / math.sqrt(d)
    W = [None if w is None else w.double() for w in W]
    out = torch.zeros(*X.shape[:-1], H * d, dtype=torch.float64, device="cuda")
    first = 0
    for b in range(B):
        L = n if lens is None else int(lens[b])
        if case["entry"] == "packed":
            x, o = X[first:first + L].double(), out[first:first + L]
            first += L
        else:
            x, o = X[b].double(), out[b]
        q = x @ W[0] if W[0] is not None else x
        k, v = (q, q) if case["scheme"] == SYM else (x @ W[1], x @ W[2])
        rows = L if case["skip_rows"] else x.shape[0]
        j = torch.arange(L, device="cuda")
        for h in range(H):
            c = slice(h * d, (h + 1) * d)
            for r0 in range(0, rows, 4096):
                r1 = min(rows, r0 + 4096)
                s = (q[r0:r1, c] @ k[:L, c].T) * scale
                if case["scheme"] == CAUSAL:
                    s.masked_fill_(j[None, :] > torch.arange(r0, r1, device="cuda")[:, None], -math.inf)
                o[r0:r1, c] = torch.softmax(s, -1) @ v[:L, c]
    return out
