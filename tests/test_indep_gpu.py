"""The independent-workgroup bf16 prefill (grids of uneven rounds) against the fp64 oracle on
sampled rows; the launch rule sends the shapes here to it on a 256-unit GPU, except where a test
names another layout or both sides of a line.  Tolerances as everywhere: 2e-2 for O, 4e-3 (bf16 weights) plus fp32 rounding for LSE."""
import zlib

import numpy as np
import pytest

import oracle
import synth
from gpu_util import TOL, bf16_weight_model, gen, max_err, run_gpu, sample_rows, say

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, H, Nq, Nk: rows and keys on both sides of a wave (32), a tile (64), an item (128)
    (1, 300, 2, 3), (2, 150, 33, 65), (1, 290, 128, 128), (4, 50, 200, 200), (3, 80, 255, 320),
    (2, 65, 257, 511),
]


def _check(q, k, v, o, lse, causal, scale=None):
    B, H, Nq, d = o.shape
    rows = sample_rows(B, H, Nq, 300, seed=5)
    ref, ref_lse = oracle.attention_rows(q, k, v, rows, scale=scale, causal=causal, with_lse=True)
    err = max_err(o.reshape(-1, d)[rows], ref)
    say(f"  max err {err:.3e}")
    assert err <= TOL["bf16"]
    assert max_err(lse.reshape(-1)[rows], ref_lse) <= 4e-3 + 1e-5 * np.abs(ref_lse).max()
    assert np.isfinite(o).all() and np.isfinite(lse).all()


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
@pytest.mark.parametrize("out_dtype", ["bf16", "f32"])
def test_independent_workgroups_match_oracle(shape, d, causal, out_dtype):
    B, H, Nq, Nk = shape
    q, k, v = gen(B, H, Nq, Nk, d, "bf16", seed=zlib.crc32(repr((shape, d, causal)).encode()) % 9973)
    o, lse = run_gpu(q, k, v, causal=causal, out_dtype=out_dtype, return_lse=True)
    _check(q, k, v, o, lse, causal)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("scale", [-0.3, 4.0, 0.0])
def test_independent_workgroups_scales(d, scale):
    # A negative scale, wide logits (the reference is raised over and over) and uniform weights.
    q, k, v = gen(2, 100, 150, 300, d, "bf16", seed=31)
    o, lse = run_gpu(q, k, v, causal=True, scale=scale, out_dtype="f32", return_lse=True)
    _check(q, k, v, o, lse, True, scale)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
def test_independent_workgroups_packed_layout(d, causal):
    # [B][N][3][H][d] projections in, O in [B][N][H][d]: bit-identical to the contiguous call.
    import torch
    import paper_2606_07713_amd as moa
    B, N, H = 6, 230, 30
    qkv = torch.randn((B, N, 3, H, d), device="cuda").bfloat16()
    q, k, v = (qkv[:, :, i].transpose(1, 2) for i in range(3))
    out = torch.empty((B, N, H, d), dtype=torch.bfloat16, device="cuda").transpose(1, 2)
    moa.attn_fwd(q, k, v, causal=causal, out=out)
    ref = moa.attn_fwd(*(t.contiguous() for t in (q, k, v)), causal=causal)
    assert torch.equal(out, ref)


def test_more_items_than_resident_workgroups():
    # Several items per workgroup, the last layer of items partly empty; twice as many 128-query
    # rounds as 256-query ones, so the ping-pong layout (test_rounds_of_resident_workgroups has the
    # independent workgroups).
    q, k, v = gen(1, 700, 200, 190, 64, "bf16", seed=77)
    o, lse = run_gpu(q, k, v, out_dtype="f32", return_lse=True)
    _check(q, k, v, o, lse, False)
    q, k, v = gen(1, 700, 190, 200, 128, "bf16", seed=78)
    o, lse = run_gpu(q, k, v, causal=True, out_dtype="f32", return_lse=True)
    _check(q, k, v, o, lse, True)


@pytest.mark.parametrize("shape", [(203, 183, 183, 64, False), (123, 267, 267, 128, False), (160, 150, 400, 64, False),
                                   (123, 364, 364, 128, True), (120, 400, 450, 64, True)],
                         ids=lambda s: "x".join(str(int(x)) for x in s))
def test_second_reference_on_key_split_grids(shape):
    # Fewer 256-query items than compute units: a row's weights are rounded against two
    # references, as the key split would take them (one reference per row was up to 7.6% further
    # from fp64).  The kernel agrees with a model of that rounding to a small part of the rounding
    # itself (about 1.5e-3): fp32 scores near a tie may round the other way, about 1 in 2^12 with
    # exponents of magnitude 2^5, sqrt(2^-12) of the error, and 3e-4 leaves a factor of three.
    import torch
    import paper_2606_07713_amd as moa
    H, Nq, Nk, d, causal = shape
    g = torch.Generator(device="cuda").manual_seed(H)
    q, k, v = (torch.randn((1, H, n, d), device="cuda", generator=g).bfloat16() for n in (Nq, Nk, Nk))
    o = moa.attn_fwd(q, k, v, causal=causal, out_dtype=torch.float32)
    for h in (0, H // 2, H - 1):
        want = bf16_weight_model(*(t[0, h].double() for t in (q, k, v)), causal, lambda n: (0, (n + 1) // 2))
        diff = float((o[0, h].double() - want).norm() / want.norm())
        say(f"  head {h}: {diff:.2e} from the two-reference model")
        assert diff <= 3e-4


@pytest.mark.parametrize("shape", [(1, 700, 100, 200, 128, True), (1, 700, 120, 333, 128, False), (1, 700, 300, 300, 64, True)],
                         ids=lambda s: "x".join(str(int(x)) for x in s))
def test_rounds_of_resident_workgroups(shape):
    # More 128-query items than workgroups the GPU holds at a time, the last round partly filled.
    B, H, Nq, Nk, d, causal = shape
    q, k, v = gen(B, H, Nq, Nk, d, "bf16", seed=H + Nk)
    o, lse = run_gpu(q, k, v, causal=causal, out_dtype="f32", return_lse=True)
    _check(q, k, v, o, lse, causal)


# Routes on both sides of the launch rule's lines (256 compute units): K and V beyond 256 MB, few
# queries to many keys, no gain in rounds, few more items than units under the mask.
@pytest.mark.parametrize("shape", [(1, 877, 158, 1300, 64, False), (1, 766, 260, 1500, 64, False),
                                   (1, 313, 181, 870, 128, False), (1, 393, 328, 700, 128, False),
                                   (1, 738, 229, 358, 128, True), (1, 256, 200, 200, 128, True),
                                   (1, 835, 500, 1300, 64, False), (1, 86, 300, 320, 128, True),
                                   (1, 102, 330, 330, 64, True), (1, 103, 330, 330, 64, True),
                                   (1, 96, 400, 400, 128, True), (1, 97, 400, 400, 128, True),
                                   (1, 70, 500, 512, 64, True), (1, 80, 700, 700, 128, False),
                                   (1, 125, 500, 61, 128, False), (1, 125, 500, 65, 128, False),
                                   (1, 93, 707, 707, 128, True), (1, 110, 580, 580, 128, True),
                                   (1, 177, 700, 700, 128, True)],
                         ids=lambda s: "x".join(str(int(x)) for x in s))
def test_lines_of_the_launch_rule(shape):
    B, H, Nq, Nk, d, causal = shape
    q, k, v = gen(B, H, Nq, Nk, d, "bf16", seed=H + Nk)
    o, lse = run_gpu(q, k, v, causal=causal, out_dtype="f32", return_lse=True)
    _check(q, k, v, o, lse, causal)
