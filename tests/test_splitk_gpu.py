"""Split-K prefill (keys split across workgroups, partial states merged by the
combine pass) against the fp64 oracle, element by element.

The library splits bf16 prefill automatically when the grid is too small to
fill the GPU and the key range is long; explicit ``num_splits`` forces any
split count, including shares that are empty for some (or all) rows of a
causal query tile.  Tolerances as everywhere: 2e-2 (bf16 inputs), 1e-5 (fp32).
"""
import zlib

import numpy as np
import pytest

import paper_2606_07713_amd as moa
from gpu_util import TOL, gen, max_err, oracle_full, run_gpu, say

pytestmark = pytest.mark.gpu


def _seed(*parts):
    return zlib.crc32(repr(parts).encode()) % 100003


def _lse_tol(ref_lse):
    # bf16 weights (relative error <= 2^-8) plus fp32 rounding.
    return 4e-3 + 1e-5 * np.abs(ref_lse).max()


AUTO_SHAPES = [
    # B, H, Nq, Nk, d: small grids with long key ranges -> automatic split
    (1, 2, 100, 5000, 64),
    (1, 1, 300, 3000, 128),
    (2, 2, 64, 4100, 128),
]


@pytest.mark.parametrize("shape", AUTO_SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
def test_automatic_split_matches_oracle(shape, causal):
    B, H, Nq, Nk, d = shape
    splits = moa.moa_attn_num_splits(B, H, Nq, Nk, d, d, 0)
    assert splits > 1, "shape meant to exercise the split path"
    say(f"split-K auto {shape} causal={causal} splits={splits}")
    q, k, v = gen(B, H, Nq, Nk, d, "bf16", seed=_seed("auto", shape, causal))
    o, lse = run_gpu(q, k, v, causal=causal, out_dtype="f32", return_lse=True)
    ref, ref_lse = oracle_full(q, k, v, causal=causal, with_lse=True)
    err = max_err(o, ref)
    say(f"  max err {err:.3e}")
    assert err <= TOL["bf16"]
    assert max_err(lse, ref_lse) <= _lse_tol(ref_lse)


FORCED = [
    # B, H, Nq, Nk, d, splits
    (1, 2, 130, 700, 128, 7),     # causal: the last share of the first tile is empty
    (2, 1, 33, 1000, 64, 3),
    (1, 1, 200, 200, 64, 16),     # more splits than key tiles: most shares empty
    (1, 3, 257, 513, 128, 2),
]


@pytest.mark.parametrize("case", FORCED, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
@pytest.mark.parametrize("out_dtype", ["bf16", "f32"])
def test_forced_splits_match_oracle(case, causal, out_dtype):
    B, H, Nq, Nk, d, splits = case
    say(f"split-K forced {case} causal={causal} out={out_dtype}")
    q, k, v = gen(B, H, Nq, Nk, d, "bf16", seed=_seed("forced", case, causal))
    o, lse = run_gpu(q, k, v, causal=causal, out_dtype=out_dtype, num_splits=splits,
                     return_lse=True)
    ref, ref_lse = oracle_full(q, k, v, causal=causal, with_lse=True)
    err = max_err(o, ref)
    say(f"  max err {err:.3e}")
    assert err <= TOL["bf16"]
    assert max_err(lse, ref_lse) <= _lse_tol(ref_lse)


def test_split_counts_agree():
    # Every split count computes the same attention (within the bf16 tolerance of
    # the oracle), and one split is the single-pass kernel.
    B, H, Nq, Nk, d = 1, 2, 150, 2500, 128
    q, k, v = gen(B, H, Nq, Nk, d, "bf16", seed=_seed("agree"))
    ref = oracle_full(q, k, v, causal=True)
    for s in (1, 2, 5, 40):
        o = run_gpu(q, k, v, causal=True, out_dtype="f32", num_splits=s)
        err = max_err(o, ref)
        say(f"  splits={s}: max err {err:.3e}")
        assert err <= TOL["bf16"]


def test_split_on_strided_layout():
    # [B, N, H, d] inputs and output (views, no copies) through the split path.
    import torch
    import synth
    B, H, Nq, Nk, d = 1, 4, 96, 3000, 64
    q, k, v = gen(B, H, Nq, Nk, d, "bf16", seed=_seed("strided"))
    tq, tk, tv = (synth.to_torch(a, "cuda").transpose(1, 2).contiguous().transpose(1, 2)
                  for a in (q, k, v))
    out = torch.empty((B, Nq, H, d), dtype=torch.float32, device="cuda").transpose(1, 2)
    assert moa.moa_attn_num_splits(B, H, Nq, Nk, d, d, 0) > 1
    moa.attn_fwd(tq, tk, tv, out=out, out_dtype=torch.float32)
    torch.cuda.synchronize()
    err = max_err(out.cpu().double().numpy(), oracle_full(q, k, v))
    say(f"  max err {err:.3e}")
    assert err <= TOL["bf16"]


def test_fp32_prefill_ignores_split_request():
    B, H, Nq, Nk, d = 1, 1, 70, 300, 64
    q, k, v = gen(B, H, Nq, Nk, d, "f32", seed=_seed("f32"))
    o = run_gpu(q, k, v, causal=True, num_splits=4)
    assert max_err(o, oracle_full(q, k, v, causal=True)) <= TOL["f32"]


# The combine pass takes splits four (up to 4 of them) or eight at a time, and decode runs four or
# eight waves per chunk: edges of both, tolerance as everywhere.
@pytest.mark.parametrize("splits", [2, 4, 5, 8, 9, 17])
@pytest.mark.parametrize("nk_per_split", [31, 512, 513])
def test_decode_chunk_and_combine_edges(splits, nk_per_split):
    B, H, d = 1, 3, 128
    Nk = splits * nk_per_split - 1
    q, k, v = gen(B, H, 1, Nk, d, "bf16", seed=_seed("edges", splits, nk_per_split))
    o, lse = run_gpu(q, k, v, out_dtype="f32", num_splits=splits, return_lse=True)
    ref, ref_lse = oracle_full(q, k, v, with_lse=True)
    assert max_err(o, ref) <= TOL["bf16"]
    assert max_err(lse, ref_lse) <= _lse_tol(ref_lse)


def test_combine_keeps_infinities():
    # An infinite value reaches the output as itself: the spare slots of the combine's last
    # group of splits contribute nothing rather than 0 * inf.
    import torch
    q, k, v = (torch.randn((1, 2, n, 64), device="cuda").bfloat16() for n in (1, 3000, 3000))
    v[:, :, 2990, 5] = float("inf")
    o = moa.attn_fwd(q, k, v, num_splits=5)
    assert torch.isposinf(o[..., 5]).all()
    assert torch.isfinite(o[..., :5]).all() and torch.isfinite(o[..., 6:]).all()


WIDE = [
    # B, H, Nq, Nk, d: 256-query split items (two to a narrow one); ragged rows and keys
    (2, 30, 130, 4100, 128),
    (1, 32, 200, 8200, 128),
    (1, 16, 257, 8200, 64),     # narrow items: too few keys for wide ones at d = 64
    (1, 60, 130, 8200, 64),
]


@pytest.mark.parametrize("case", WIDE, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
def test_wide_splits_and_smaller_workspaces(case, causal):
    # The automatic choice, then the same call with workspaces too small for it: fewer splits,
    # in the end one pass, each against the oracle on sampled rows.
    import torch
    import oracle
    import synth
    from gpu_util import sample_rows
    B, H, Nq, Nk, d = case
    q, k, v = gen(B, H, Nq, Nk, d, "bf16", seed=_seed("wide", case, causal))
    rows = sample_rows(B, H, Nq, 200, seed=3)
    ref, ref_lse = oracle.attention_rows(q, k, v, rows, causal=causal, with_lse=True)
    tq, tk, tv = (synth.to_torch(a, "cuda") for a in (q, k, v))
    full = moa.moa_attn_workspace_bytes(B, H, Nq, Nk, d, d)
    splits = moa.moa_attn_num_splits(B, H, Nq, Nk, d, d)
    assert splits >= 4 and full >= B * H * Nq * splits * (d + 2) * 4
    for size in (full, full - 256, full // 2, 256):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        o, lse = moa.attn_fwd(tq, tk, tv, causal=causal, out_dtype=torch.float32, return_lse=True,
                              workspace=ws)
        err = max_err(o.cpu().double().numpy().reshape(-1, d)[rows], ref)
        say(f"wide {case} causal={causal} workspace {size}: max err {err:.3e}")
        assert err <= TOL["bf16"]
        assert max_err(lse.cpu().double().numpy().reshape(-1)[rows], ref_lse) <= _lse_tol(ref_lse)
    # Asked for explicitly, the automatic split count is the automatic choice.
    a = moa.attn_fwd(tq, tk, tv, causal=causal)
    assert torch.equal(a, moa.attn_fwd(tq, tk, tv, causal=causal, num_splits=splits))


def _narrow_starts(splits, renew=False):
    """First tiles of the references of 128-query split items: two streams per share, each (with
    `renew`) taking a second reference half way."""
    def starts(n_kt):
        out, share = [], -(-n_kt // splits)
        for lo in range(0, n_kt, share):
            n = min(n_kt, lo + share) - lo
            first = (n + 1) // 2
            for a, m in ((lo, first), (lo + first, n - first)):
                out += [a] * (m > 0) + [a + (m + 1) // 2] * (renew and m > 1)
        return out
    return starts


def _check_rounding(H, Nq, Nk, d, causal, starts, tile):
    """O of a call against the model of its weights' rounding: a small part of the rounding itself
    (about 1.5e-3; fp32 scores near a tie may round the other way, about 1 in 2^12 with exponents
    of magnitude 2^5, sqrt(2^-12) of the error, and 3e-4 leaves a factor of three)."""
    import torch
    from gpu_util import bf16_weight_model
    g = torch.Generator(device="cuda").manual_seed(H)
    q, k, v = (torch.randn((1, H, n, d), device="cuda", generator=g).bfloat16() for n in (Nq, Nk, Nk))
    o = moa.attn_fwd(q, k, v, causal=causal, out_dtype=torch.float32)
    for h in (0, H - 1):
        want = bf16_weight_model(*(t[0, h].double() for t in (q, k, v)), causal, starts, tile)
        diff = float((o[0, h].double() - want).norm() / want.norm())
        say(f"  {(H, Nq, Nk, d, causal)} head {h}: {diff:.2e} from the model")
        assert diff <= 3e-4


@pytest.mark.parametrize("case", [(11, 2048, 128), (8, 3000, 128), (6, 3000, 64), (6, 4096, 64)],
                         ids=lambda s: "x".join(map(str, s)))
def test_causal_square_grids_keep_short_items(case):
    # Under the mask the items of a square grid differ in length: two splits of 128-query items,
    # dealt in snake order, not two of 256-query items or none.
    H, n, d = case
    _check_rounding(H, n, n, d, True, _narrow_starts(2), 128)


def _wide_starts(splits):
    """First tiles of the references of 256-query split items: one stream per share, two each."""
    def starts(n_kt):
        out, share = [], -(-n_kt // splits)
        for lo in range(0, n_kt, share):
            n = min(n_kt, lo + share) - lo
            out += [lo] + [lo + (n + 1) // 2] * (n > 1)
        return out
    return starts


@pytest.mark.parametrize("case", [(41, 18, 15038, 128, True, 6), (40, 36, 7362, 64, True, 6),
                                  (11, 2048, 2048, 64, False, 1), (6, 3000, 3000, 128, False, 1)],
                         ids=lambda s: "x".join(str(int(x)) for x in s))
def test_fewer_splits_take_second_references(case):
    # Fewer splits than 128-query items rounded up to the target would have (one pass among them):
    # every key stream takes a second reference half way.
    H, Nq, Nk, d, causal, splits = case
    _check_rounding(H, Nq, Nk, d, causal, _narrow_starts(splits, renew=True), 128)


@pytest.mark.parametrize("case", [(60, 130, 4100, 128, False, 4), (34, 206, 20568, 64, True, 7),
                                  (60, 300, 4500, 128, True, 2)],
                         ids=lambda s: "x".join(str(int(x)) for x in s))
def test_wide_splits_take_second_references(case):
    # 256-query items hold one stream where two 128-query items hold two: the same.
    H, Nq, Nk, d, causal, splits = case
    assert moa.moa_attn_num_splits(1, H, Nq, Nk, d, d) == splits
    _check_rounding(H, Nq, Nk, d, causal, _wide_starts(splits), 256)
