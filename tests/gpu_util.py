"""Helpers for the GPU tests: run the HIP path through the C ABI on seeded
inputs, run the oracle on the same host bytes, compare."""
import sys

import numpy as np

import oracle
import synth

# Max-abs tolerances relative to std(V) (= the generator's sigma_v), per input storage type.
TOL = {"f32": 1e-5, "bf16": 2e-2}


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def gen(B, H, Nq, Nk, d, dtype, seed, sigma_qk=1.0, sigma_v=1.0):
    q = synth.normal(seed * 3 + 0, (B, H, Nq, d), sigma_qk, dtype)
    k = synth.normal(seed * 3 + 1, (B, H, Nk, d), sigma_qk, dtype)
    v = synth.normal(seed * 3 + 2, (B, H, Nk, d), sigma_v, dtype)
    return q, k, v


def run_gpu(q, k, v, causal=False, scale=None, out_dtype=None, num_splits=0, return_lse=False):
    """O (float64 numpy) from the HIP library; inputs are numpy (f32 or bf16 bits)."""
    import torch
    import paper_2606_07713_amd as moa
    tq, tk, tv = (synth.to_torch(a, "cuda") for a in (q, k, v))
    odt = None if out_dtype is None else {"f32": torch.float32, "bf16": torch.bfloat16}[out_dtype]
    r = moa.attn_fwd(tq, tk, tv, scale=scale, causal=causal, out_dtype=odt,
                     num_splits=num_splits, return_lse=return_lse)
    torch.cuda.synchronize()
    if return_lse:
        o, lse = r
        return o.float().cpu().double().numpy(), lse.cpu().double().numpy()
    return r.float().cpu().double().numpy()


def oracle_full(q, k, v, causal=False, scale=None, with_lse=False):
    return oracle.attention(q, k, v, scale=scale, causal=causal, with_lse=with_lse)


def sample_rows(B, H, Nq, n, seed=0, tile=128):
    """Flat rows (b*H + h)*Nq + i: tile edges of the first/last heads plus random rows."""
    rng = np.random.default_rng(seed)
    total = B * H * Nq
    n = min(n, total)
    edges = {min(i, Nq - 1) for i in (0, 1, Nq - 1, tile - 1, tile, Nq // 2)}
    rows = set()
    for bh in {0, B * H - 1, (B * H) // 2}:
        for i in edges:
            rows.add(bh * Nq + i)
    while len(rows) < n:
        rows.add(int(rng.integers(0, total)))
    return np.array(sorted(rows), dtype=np.int64)


def max_err(a, b):
    return float(np.max(np.abs(np.asarray(a, np.float64) - np.asarray(b, np.float64))))


def bf16_weight_model(q, k, v, causal, starts, tile=128):
    """O of one head (fp64 tensor) with the weights rounded to bf16 against a reference per key
    range: weights 2^(s c - m) with m = 32 + the largest visible score (log2 units) of the first 64
    keys of the range, at most 8 below the reference before.  q, k, v: fp64 [N, d] tensors;
    starts(n_kt) lists the first 64-key tiles of the ranges of a query tile (`tile` rows) that sees
    n_kt tiles."""
    import math

    import torch
    Nq, Nk, off = q.shape[0], k.shape[0], k.shape[0] - q.shape[0]
    out = torch.empty_like(q)
    for q0 in range(0, Nq, tile):
        rows = torch.arange(q0, min(Nq, q0 + tile), device=q.device)
        n_kt = -(-(min(Nk, q0 + tile + off) if causal else Nk) // 64)
        keys = torch.arange(min(Nk, 64 * n_kt), device=q.device)
        s = (q[rows] @ k[keys].t().contiguous()) * (math.log2(math.e) / math.sqrt(q.shape[1]))
        if causal:
            s.masked_fill_(keys[None, :] > rows[:, None] + off, -math.inf)
        first = [t for t in starts(n_kt) if t < n_kt] + [n_kt]
        m = torch.empty_like(s)
        ref = None
        for a, b in zip(first, first[1:]):
            new = s[:, 64 * a:64 * a + 64].amax(1) + 32
            ref = new if ref is None else torch.maximum(new, ref - 8)
            m[:, 64 * a:64 * b] = ref[:, None]
        p = torch.exp2(s - m).to(torch.bfloat16).double()
        w = p * torch.exp2(m - m.amax(1, keepdim=True))
        out[rows] = (w @ v[keys]) / w.sum(1, keepdim=True)
    return out
