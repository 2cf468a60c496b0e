"""Measured workloads of the attention library, over the range its users call it with.

Each case is one call (or one forward + backward step) through a public entry point of
``paper_2606_07713_amd``.  ``listed()`` names the fixed cases, ``draw()`` gives further ones of
the same ranges, ``prepare()`` makes the inputs on the GPU from a seed, ``run()`` makes the call,
``exact()`` is the same computation in fp64 by plain torch, and ``work()`` counts the bytes and
operations the mathematics needs.
"""
import math

import torch

import paper_2606_07713_amd as moa

BF16, F32 = "bf16", "f32"
_TORCH = {BF16: torch.bfloat16, F32: torch.float32}
_CODE = {BF16: moa.MOA_BF16, F32: moa.MOA_F32}
_BYTES = {BF16: 2, F32: 4}


def _case(op, B, H, Nq, Nk, d, dtype=BF16, causal=False, sigma=1.0, out=None, layout="bhnd", dm=0,
          name=None):
    c = {"op": op, "B": B, "H": H, "Nq": Nq, "Nk": Nk, "d": d, "dtype": dtype, "causal": causal,
         "sigma": sigma, "out": out or dtype, "layout": layout, "dm": dm}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: one fp32 head of 128 tokens through the C entry point with every
        # buffer kept by the caller.  Launch and latency.
        _case("fwd_raw", 1, 1, 128, 128, 64, dtype=F32, name="f32_head_128"),
        # fp32 inference or a reference run of an ordinary model: 16 heads, 1K tokens, causal.
        _case("fwd", 1, 16, 1024, 1024, 64, dtype=F32, causal=True, name="f32_causal_1k"),
        # Encoder layer of a small model: four sequences of 1K tokens, no mask.
        _case("fwd", 4, 8, 1024, 1024, 64, name="encoder_1k_d64"),
        # Prompt processing of a decoder layer, 4K tokens.
        _case("fwd", 2, 16, 4096, 4096, 128, causal=True, name="causal_4k"),
        # Long-context prompt, the largest single call: wide logits (Q, K of spread 3).
        _case("fwd", 1, 32, 16384, 16384, 128, causal=True, sigma=3.0, name="causal_16k"),
        # Encoder batch in the usual packed [B][N][3][H][d] projection output, O into [B][N][H][d],
        # a token count that divides by no tile.
        _case("fwd", 8, 12, 777, 777, 64, layout="packed", name="packed_ragged_777"),
        # Chunked prefill: a few hundred new tokens against a long cache, ragged on both sides.
        _case("fwd", 1, 32, 200, 20011, 128, causal=True, name="chunk_200_of_20k"),
        # Decode step of a large serving batch.
        _case("decode", 64, 32, 1, 8192, 128, name="decode_b64_8k"),
        # Decode step of a single conversation, through the entry point for serving loops.
        _case("decode_raw", 1, 32, 1, 4097, 128, name="decode_b1_4k"),
        # Training step of a decoder's attention: forward with LSE, then gradients in fp32.
        _case("train", 2, 16, 4096, 4096, 128, causal=True, out=F32, name="train_causal_4k"),
        # Training step of an encoder's attention on a ragged length, gradients in bf16.
        _case("train", 4, 8, 1000, 1000, 64, out=BF16, name="train_ragged_1000"),
        # Self-attention from the token sequence: input projections and causal attention.
        _case("proj", 1, 32, 4096, 4096, 128, causal=True, dm=4096, name="proj_4k"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _seq(rng, lo, hi):
    """A length of lo..hi, spread over its logarithm; every third one a multiple of 128."""
    n = _log_int(rng, lo, hi)
    return max(128, n // 128 * 128) if rng.random() < 1 / 3 else n


def draw(rng):
    op = rng.choice(["fwd", "fwd", "fwd", "f32", "chunk", "decode", "decode", "train", "train", "proj"])
    d = rng.choice([64, 128])
    causal = rng.random() < 0.5
    if op == "fwd":
        B, H, n = rng.randint(1, 8), rng.randint(4, 32), _seq(rng, 128, 16384)
        # no more pairs than the largest listed case
        while B * H * n * n * (1 if causal else 2) > 32 * 16384 ** 2:
            n = n * 2 // 3
        return _case("fwd", B, H, n, n, d, causal=causal, sigma=rng.choice([1.0, 1.0, 3.0]),
                     layout=rng.choice(["bhnd", "bhnd", "packed"]))
    if op == "f32":
        B, H, n = rng.randint(1, 4), rng.randint(1, 16), _seq(rng, 100, 2048)
        return _case("fwd", B, H, n, n, d, dtype=F32, causal=causal)
    if op == "chunk":
        nq = _log_int(rng, 17, 1024)
        return _case("fwd", rng.randint(1, 2), rng.randint(4, 32), nq, _log_int(rng, 4096, 32768), d,
                     causal=True)
    if op == "decode":
        B, H, nk = _log_int(rng, 1, 64), rng.randint(8, 32), _log_int(rng, 512, 16384)
        if B * H * nk > 64 * 32 * 8192:
            nk = 64 * 32 * 8192 // (B * H)
        return _case("decode" if B > 1 else "decode_raw", B, H, 1, nk, d)
    if op == "train":
        B, H, n = rng.randint(1, 4), rng.randint(4, 16), _seq(rng, 256, 8192)
        while B * H * n * n * (1 if causal else 2) > 32 * 8192 ** 2:
            n = n * 2 // 3
        return _case("train", B, H, n, n, d, causal=causal, out=rng.choice([F32, BF16]))
    B, H, n = rng.randint(1, 4), rng.randint(8, 32), _seq(rng, 512, 4096)
    dm = 64 * rng.randint(8, 64)
    while B * n > 8192:
        n //= 2
    return _case("proj", B, H, n, n, d, causal=causal, dm=dm)


def _inputs(c, seed):
    """The input tensors of a case, on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = _TORCH[c["dtype"]]
    B, H, Nq, Nk, d = c["B"], c["H"], c["Nq"], c["Nk"], c["d"]

    def normal(shape, std=1.0):
        t = torch.empty(shape, dtype=dt, device="cuda")
        return t.normal_(0.0, std, generator=g)

    if c["op"] == "proj":
        x = normal((B, Nq, c["dm"]))
        return {"x": x, "w": [normal((H * d, c["dm"]), c["dm"] ** -0.5) for _ in range(3)]}
    if c["layout"] == "packed":
        qkv = normal((B, Nq, 3, H, d))
        if c["sigma"] != 1.0:
            qkv[:, :, :2] *= c["sigma"]
        q, k, v = (qkv[:, :, i].transpose(1, 2) for i in range(3))
        return {"q": q, "k": k, "v": v}
    s = {"q": normal((B, H, Nq, d), c["sigma"]), "k": normal((B, H, Nk, d), c["sigma"]),
         "v": normal((B, H, Nk, d))}
    if c["op"] == "train":
        s["do"] = normal((B, H, Nq, d))
    return s


def prepare(case, seed):
    c = case
    s = _inputs(c, seed)
    s["case"] = c
    B, H, Nq, Nk, d = c["B"], c["H"], c["Nq"], c["Nk"], c["d"]
    if c["op"] in ("fwd_raw", "decode_raw"):
        # The caller of the C entry point keeps its output buffer and fixed arguments.
        o = torch.empty((B, H, Nq, d), dtype=_TORCH[c["out"]], device="cuda")
        s["o"] = o
        ptrs = (s["q"].data_ptr(), s["k"].data_ptr(), s["v"].data_ptr(), o.data_ptr(), None)
        s["args"] = ptrs + (B, H, Nq, Nk, d, d, 1.0 / math.sqrt(d), int(c["causal"]),
                            _CODE[c["dtype"]], _CODE[c["out"]])
    elif c["layout"] == "packed":
        s["out"] = torch.empty((B, Nq, H, d), dtype=_TORCH[c["out"]], device="cuda").transpose(1, 2)
    elif c["op"] in ("fwd", "decode"):
        # A program that calls one layer shape again and again keeps the workspace.
        n = moa.moa_attn_workspace_bytes(B, H, Nq, Nk, d, d) if c["dtype"] == BF16 else 0
        s["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda") if n else None
    return s


def run(state):
    c = state["case"]
    op = c["op"]
    if op in ("fwd_raw", "decode_raw"):
        stream = torch.cuda.current_stream().cuda_stream
        if op == "fwd_raw":
            st = moa.moa_attn_fwd(*state["args"], None, 0, 0, stream)
        else:
            st = moa.moa_attn_fwd_noalloc(*state["args"], 0, stream)
        if st != moa.MOA_OK:
            raise moa.MoaAttnError(st)
        return state["o"]
    if op == "proj":
        return moa.attn_fwd_proj(state["x"], *state["w"], c["H"], causal=c["causal"])
    q, k, v = state["q"], state["k"], state["v"]
    if op == "train":
        o, lse = moa.attn_fwd(q, k, v, causal=c["causal"], return_lse=True)
        dq, dk, dv = moa.attn_bwd(q, k, v, o, lse, state["do"], causal=c["causal"],
                                  grad_dtype=_TORCH[c["out"]])
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    return moa.attn_fwd(q, k, v, causal=c["causal"], out=state.get("out"), workspace=state.get("ws"))


def _pairs(c):
    """Visible (query, key) pairs of one head."""
    nq, nk = c["Nq"], c["Nk"]
    return nq * nk - (nq * (nq - 1) // 2 if c["causal"] else 0)


def work(case):
    c = case
    B, H, Nq, Nk, d = c["B"], c["H"], c["Nq"], c["Nk"], c["d"]
    bh, es, os_ = B * H, _BYTES[c["dtype"]], _BYTES[c["out"]]
    fwd = 4 * d * bh * _pairs(c)
    if c["op"] == "proj":
        return {"bytes": 2 * (B * Nq * c["dm"] + 3 * H * d * c["dm"]) + bh * Nq * d * os_,
                "flops": fwd + 2 * B * Nq * c["dm"] * 3 * H * d}
    if c["op"] == "train":
        # forward: read q, k, v, write o, lse; backward: read do, write dq, dk, dv
        return {"bytes": bh * ((2 * Nq + 2 * Nk) * d * es + Nq * d * es + 4 * Nq
                               + (Nq + 2 * Nk) * d * os_),
                "flops": fwd + 10 * d * bh * _pairs(c)}
    return {"bytes": bh * ((Nq + 2 * Nk) * d * es + Nq * d * os_), "flops": fwd}


def tolerance(case):
    """About four times the distance from ``exact`` seen over the ranges of ``draw``.  Under the
    causal mask the first rows (few visible keys) hold values far above the result's root mean
    square, and "max" is what the rounding of their neighbours' terms leaves."""
    c = case
    if c["dtype"] == F32:
        return {"rel": 8e-7, "max": 1.3e-5}          # seen: 1.8e-7, 3.2e-6
    if c["op"] in ("decode", "decode_raw"):
        return {"rel": 7e-3, "max": 1.6e-2}          # fp32 weights, bf16 O; seen: 1.7e-3, 3.9e-3
    if c["op"] == "train":                           # P and dS in bf16; seen: 2.9e-3, 0.16 / 2.4e-2
        return {"rel": 1.2e-2, "max": 0.65 if c["causal"] else 0.1}
    return {"rel": 9e-3, "max": 0.2 if c["causal"] else 5e-2}   # seen: 2.3e-3, 5.7e-2 / 1.2e-2


def _attention64(q, k, v, causal, do=None):
    """O, LSE (and dQ, dK, dV) of one head in fp64; q, k, v are [N, d]."""
    q, k, v = q.double(), k.double(), v.double()
    scale = float(torch.tensor(1.0 / math.sqrt(q.shape[1]), dtype=torch.float32))
    s = (q @ k.t().contiguous()) * scale
    if causal:
        nq, nk = s.shape
        hide = torch.ones((nq, nk), dtype=torch.bool, device=s.device).triu_(nk - nq + 1)
        s.masked_fill_(hide, -math.inf)
        del hide
    lse = torch.logsumexp(s, dim=1)
    p = s.sub_(lse[:, None]).exp_()
    o = p @ v
    if do is None:
        return o, lse
    do = do.double()
    dv = p.t().contiguous() @ do
    ds = do @ v.t().contiguous()
    ds.sub_((do * o).sum(1)[:, None]).mul_(p)
    del p
    dq = (ds @ k) * scale
    dk = (ds.t().contiguous() @ q) * scale
    return o, lse, dq, dk, dv


def exact(case, seed):
    c = case
    s = _inputs(c, seed)
    B, H, d = c["B"], c["H"], c["d"]
    if c["op"] == "proj":
        # Q, K, V are held as bf16 between the projections and the attention.
        x = s["x"].double().view(-1, c["dm"])
        q, k, v = ((x @ w.double().t().contiguous()).to(torch.bfloat16)
                   .view(B, c["Nq"], H, d).transpose(1, 2) for w in s["w"])
    else:
        q, k, v = s["q"], s["k"], s["v"]
    do = s.get("do")
    heads = [[_attention64(q[b, h], k[b, h], v[b, h], c["causal"], None if do is None else do[b, h])
              for h in range(H)] for b in range(B)]
    outs = [torch.stack([torch.stack([head[i] for head in row]) for row in heads])
            for i in range(2 if do is None else 5)]
    if do is None:
        return outs[0]
    return dict(zip(("o", "lse", "dq", "dk", "dv"), outs))
