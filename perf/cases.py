"""What the layer is measured on: the calls a user's program makes, over the sizes and options it makes them with.

Four kinds of call, each through the public entry points and on buffers the program keeps:
  train    one training step of the layer: race_attn_fwd, then race_attn_bwd_saved on the workspace it left behind
           (with the temperature's cotangent where the temperature is trained);
  forward  an inference pass over a whole sequence (an encoder layer, scoring);
  prefill  a prompt: the forward pass and the decoding state behind it (race_attn_fwd, race_attn_state_init);
  decode   one token per sequence on the carried state (race_attn_step), W already in the workspace.
A case's values: kind, B, H, N (decode: tokens of context behind the state), d, L, P, beta (0 = the hard hash,
temperature +infinity), causal, dtype, chunk (0 = the library's choice), rows ("raw": N(0,1) rows of Q and K;
"unit": rows of length one; "option": raw rows that the layer itself normalises), dbeta (the temperature is trained).
"""
import math

import torch

import paper_2510_04008_amd as ra

_SLICE = 1 << 18      # tokens generated at a time (bounds the fp32 temporary)


def _case(name, kind, B, H, N, d, L, P, beta, causal, dtype, rows="raw", chunk=0, dbeta=False):
    return {"name": name, "kind": kind, "B": B, "H": H, "N": N, "d": d, "L": L, "P": P, "beta": beta, "causal": causal,
            "dtype": dtype, "rows": rows, "chunk": chunk, "dbeta": dbeta}


def listed():
    return [
        # one sequence being generated: the smallest call there is, once per token and layer
        _case("decode-1x4", "decode", 1, 4, 4096, 128, 8, 6, 8.0, True, "bf16"),
        # a serving batch: every sequence's state is read and written once per token
        _case("decode-32x8", "decode", 32, 8, 4096, 128, 8, 6, 8.0, True, "bf16"),
        # the tiny fp32 encoder layer of the benchmark's first configuration
        _case("train-f32-encoder-1k", "train", 1, 1, 1024, 64, 4, 4, 8.0, False, "f32"),
        # an fp32 causal layer with a trained temperature, ragged length
        _case("train-f32-causal-2k", "train", 2, 4, 2003, 64, 4, 4, 4.0, True, "f32", rows="unit", dbeta=True),
        # a bf16 layer of a width without a matrix-core instantiation (d = 32)
        _case("train-bf16-narrow-1k", "train", 2, 8, 1024, 32, 4, 4, 4.0, False, "bf16"),
        # short sequences, a few of them, ragged: a small training batch
        _case("train-short-1k", "train", 4, 4, 1000, 128, 8, 6, 8.0, True, "bf16", rows="unit"),
        # a smaller hash than any compiled shape, unit rows inside the layer, trained temperature, odd length
        _case("train-unit-10k", "train", 2, 8, 10007, 64, 6, 5, 4.0, True, "bf16", rows="option", dbeta=True),
        # the benchmark's causal 64K configuration, with its chunk of 1024 tokens
        _case("train-64k", "train", 1, 4, 65536, 128, 8, 6, 8.0, True, "bf16", rows="unit", chunk=1024),
        # the benchmark's encoder configuration
        _case("train-encoder-16k", "train", 8, 8, 16384, 64, 16, 4, 4.0, False, "bf16"),
        # a prompt of odd length: outputs and the state decoding goes on from
        _case("prefill-30k", "prefill", 1, 4, 30011, 128, 8, 6, 8.0, True, "bf16"),
        # the paper's scaling grid, (P, L) = (4, 4), at 2^20 tokens
        _case("train-grid44-1m", "train", 1, 4, 1048576, 128, 4, 4, 8.0, True, "bf16"),
        # long context, the headline shape at 2^22 tokens
        _case("train-4m", "train", 1, 4, 4194304, 128, 8, 6, 8.0, True, "bf16"),
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the ranges above: sizes over their logarithm, odd ones among them."""
    what = rng.choice(["decode", "f32", "f32", "narrow", "bf16", "bf16", "bf16", "bf16"])
    H = rng.choice([1, 2, 3, 4, 6, 8])
    causal = rng.random() < 0.6
    if what == "decode":
        B = _log_uniform(rng, 1, 32)
        dtype = rng.choice(["bf16", "bf16", "f32"])
        d, L, P = rng.choice([(128, 8, 6), (128, 8, 6), (64, 4, 4), (64, 16, 4), (128, 4, 4), (96, 5, 5)])
        return _unnamed("decode", B, H, _log_uniform(rng, 256, 4096), d, L, P, rng.choice([2.0, 4.0, 8.0]), True, dtype)
    if what == "f32":
        # the fp32 path: small layers, up to a few thousand tokens
        B = rng.choice([1, 1, 2, 4])
        d, L, P = rng.choice([32, 64, 64, 128]), rng.randint(1, 8), rng.randint(2, 6)
        N = _log_uniform(rng, 100, 4096)
        kind = rng.choice(["train", "train", "forward"])
        return _unnamed(kind, B, H, N, d, L, P, rng.choice([2.0, 4.0, 8.0]), causal, "f32", rows="unit", dbeta=kind == "train" and rng.random() < 0.5)
    if what == "narrow":
        B = rng.choice([1, 2, 4])
        d, L, P = rng.choice([16, 32, 48, 96]), rng.randint(1, 8), rng.randint(2, 5)
        return _unnamed("train", B, H, _log_uniform(rng, 100, 4096), d, L, P, rng.choice([2.0, 4.0, 8.0]), causal, "bf16", rows="unit")
    # the bf16 matrix-core path: 200 to a million tokens; the short ones in batches
    N = _log_uniform(rng, 200, 1 << 20)
    B = rng.choice([1, 2, 4, 8])
    while B > 1 and B * H * N > 1 << 22:
        B //= 2
    d, L, P = rng.choice([(128, 8, 6), (128, 8, 6), (64, 16, 4), (128, 4, 4), (128, 3, 3), (128, 2, 2), (64, rng.randint(1, 8), rng.randint(2, 6)),
                          (128, rng.randint(1, 16), rng.randint(2, 4))])
    kind = rng.choice(["train", "train", "train", "forward", "prefill"])
    rows = rng.choice(["raw", "unit", "unit", "option"])
    beta = rng.choice([2.0, 4.0, 8.0])
    if kind == "forward" and rng.random() < 0.3:
        beta = 0.0
    chunk = rng.choice([0, 0, 0, 1024])
    return _unnamed(kind, B, H, N, d, L, P, beta, causal or kind == "prefill", "bf16", rows=rows, chunk=chunk,
                    dbeta=kind == "train" and rows != "raw" and beta < 8.0 and rng.random() < 0.3)


def _unnamed(*args, **kw):
    c = _case("", *args, **kw)
    del c["name"]
    return c


def _elem(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _gaussian(shape, dtype, gen, unit):
    """N(0,1) rows of the storage type (unit: scaled to length one first)."""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    for n0 in range(0, shape[2], _SLICE):
        n1 = min(shape[2], n0 + _SLICE)
        x = torch.randn((shape[0], shape[1], n1 - n0, shape[3]), generator=gen, dtype=torch.float32, device="cuda")
        if unit:
            x /= x.norm(dim=-1, keepdim=True)
        out[:, :, n0:n1] = x
    return out


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 7919 + 17)
    dtype = _elem(c)
    shape = (c["B"], c["H"], c["N"], c["d"])
    unit = c["rows"] == "unit"
    desc = ra.make_desc(c["B"], c["H"], c["N"], c["d"], c["L"], c["P"], c["beta"] if c["beta"] > 0 else float("inf"), c["causal"],
                        ra.RACE_F32 if c["dtype"] == "f32" else ra.RACE_BF16, c["chunk"], c["rows"] == "option")
    # the layer's projection is fixed once and for all, one seed per head, like a weight
    s = {"kind": c["kind"], "desc": desc, "seeds": [1 + 1000003 * h for h in range(c["H"])], "want_dbeta": c["dbeta"]}
    buf = lambda *size, t=dtype: torch.empty(size, dtype=t, device="cuda")                     # noqa: E731
    s["K"], s["V"] = _gaussian(shape, dtype, gen, unit), _gaussian(shape, dtype, gen, False)
    if c["kind"] == "decode":
        # a context of N tokens behind every sequence, then the next token's rows; W is in the step's workspace
        s["state"] = ra.race_attn_state_init(desc, s["K"], s["V"], s["seeds"])
        del s["K"], s["V"]
        row = (c["B"], c["H"], 1, c["d"])
        for n in "qkv":
            s[n] = _gaussian(row, dtype, gen, unit and n != "v").reshape(c["B"], c["H"], c["d"])
        s["o"], s["den"] = buf(c["B"], c["H"], c["d"]), buf(c["B"], c["H"], t=torch.float32)
        s["ws"] = buf(ra.race_attn_step_workspace_bytes(desc), t=torch.uint8)
        ra.race_attn_step(desc, s["q"], s["k"], s["v"], s["seeds"], s["state"], s["o"], s["den"], s["ws"])
        return s
    s["Q"] = _gaussian(shape, dtype, gen, unit)
    s["O"], s["den"] = buf(*shape), buf(*shape[:3], t=torch.float32)
    s["ws"] = buf(ra.race_attn_workspace_bytes(desc), t=torch.uint8)
    if c["kind"] == "train":
        s["dO"] = _gaussian(shape, dtype, gen, False)
        s["dQ"], s["dK"], s["dV"] = buf(*shape), buf(*shape), buf(*shape)
        s["dbeta"] = buf(c["B"], c["H"], t=torch.float32) if c["dbeta"] else None
    if c["kind"] == "prefill":
        s["state"] = buf(c["B"], c["H"], c["L"], 1 << c["P"], c["d"] + 1, t=torch.float32)
    return s


def run(state):
    s = state
    if s["kind"] == "decode":
        ra.race_attn_step(s["desc"], s["q"], s["k"], s["v"], None, s["state"], s["o"], s["den"], s["ws"])
        return s["o"], s["den"], s["state"]
    ra.race_attn_fwd(s["desc"], s["Q"], s["K"], s["V"], s["seeds"], s["O"], s["den"], s["ws"])
    if s["kind"] == "train":
        ra.race_attn_bwd_saved(s["desc"], s["Q"], s["K"], s["V"], s["O"], s["den"], s["dO"], s["seeds"], s["ws"],
                               s["dQ"], s["dK"], s["dV"], s["dbeta"])
        outs = (s["O"], s["den"], s["dQ"], s["dK"], s["dV"])
        return outs + (s["dbeta"],) if s["want_dbeta"] else outs
    if s["kind"] == "prefill":
        ra.race_attn_state_init(s["desc"], s["K"], s["V"], s["seeds"], s["state"], s["ws"])
        return s["O"], s["den"], s["state"]
    return s["O"], s["den"]


def work(case):
    """Algorithms 1 and 2 as written: projections of Q and K (2 d L P flop a row), one update and one read-out of the
    (L R) x (d + 1) statistics per token; backward: two more projections' worth and four more passes over the
    statistics.  Bytes: every input read once, every output written once."""
    c = case
    rows, es = c["B"] * c["H"], 4 if c["dtype"] == "f32" else 2
    LR, LP, d = c["L"] << c["P"], c["L"] * c["P"], c["d"]
    proj, upd, state = 4 * d * LP, 2 * LR * (d + 1), LR * (d + 1) * 4
    if c["kind"] == "decode":
        return {"bytes": rows * (2 * state + 4 * d * es + 4) + c["H"] * LP * d * 4, "flops": rows * (proj + 2 * upd)}
    n = rows * c["N"]
    if c["kind"] == "train":
        return {"bytes": n * (8 * d * es + 4), "flops": n * (3 * proj + 6 * upd)}
    return {"bytes": n * (4 * d * es + 4) + (rows * state if c["kind"] == "prefill" else 0), "flops": n * (proj + 2 * upd)}


def tolerance(case):
    # bf16: a few roundings of 2^-9 behind one another; single entries among the first rows of a causal sequence, whose
    # gradients are differences of terms scaled by 1 / Den, keep less (kernels of fp32 arithmetic on the same bf16 inputs
    # are 0.5 of the root mean square away from the matrix-core ones there).  fp32: sums of some thousand terms; the
    # gradients pass through differences (dphi minus its mean over the corners, cotangents of saturated bits)
    return {"rel": 1e-2, "max": 0.8} if case["dtype"] == "bf16" else {"rel": 2e-5}
