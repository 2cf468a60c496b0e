"""fp32 prefill on the matrix cores: shapes at the edges of its 16-row tiles, 16-key blocks and
key streams, against the oracle (O within 1e-5 of unit-variance V, LSE within 1e-5 relative: the
bounds of every fp32 path)."""
import numpy as np
import pytest

from gpu_util import TOL, gen, max_err, oracle_full, run_gpu

pytestmark = pytest.mark.gpu

# More than 64 16-row tiles reach the kernel at any length; from 768 keys on and up to 256 tiles
# (512 causal at d = 128) it takes eight key streams, otherwise four.
SHAPES = [
    # B, H, Nq, Nk, d, causal
    (5, 13, 2, 1, 64, False),        # one key: three of four streams empty
    (5, 13, 16, 16, 64, True),       # one tile, one block
    (5, 13, 17, 33, 64, True),       # one row and one key past a tile
    (3, 30, 15, 31, 128, True),      # one short of a tile
    (3, 30, 31, 65, 128, False),
    (9, 30, 40, 40, 64, True),       # more heads than compute units: runs of one tile rank
    (1, 7, 333, 334, 128, True),     # runs of many tile ranks, the last one partial
    (1, 2, 1000, 1003, 64, False),   # eight streams
    (1, 1, 1100, 1100, 64, True),
    (1, 5, 250, 769, 128, True),     # eight streams on 80 tiles, Nq < Nk
    (1, 6, 1000, 1000, 128, True),   # eight streams on 378 tiles
    (1, 6, 1000, 1000, 128, False),  # four streams on the same grid
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(str(int(x)) for x in s))
def test_f32_matrix_core_prefill(shape):
    B, H, Nq, Nk, d, causal = shape
    q, k, v = gen(B, H, Nq, Nk, d, "f32", seed=sum(shape))
    o, lse = run_gpu(q, k, v, causal=causal, return_lse=True)
    ref, ref_lse = oracle_full(q, k, v, causal=causal, with_lse=True)
    assert max_err(o, ref) <= TOL["f32"]
    assert max_err(lse, ref_lse) <= 1e-5 * max(1.0, np.abs(ref_lse).max())


# Lengths that end inside a 16-key block (in every lane group of it), four and eight key streams.
@pytest.mark.parametrize("shape", [(1, 16, 300, 300, 64), (1, 4, 1000, 1000, 64), (1, 6, 1000, 995, 128), (2, 32, 70, 33, 128)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("value", [np.inf, -np.inf])
def test_f32_infinity_in_the_last_value(shape, value):
    # Keys past Nk have no weight: an infinite element of the last V row reaches its own column of
    # every row that sees the key, as itself, and nothing else.
    B, H, Nq, Nk, d = shape
    q, k, v = gen(B, H, Nq, Nk, d, "f32", seed=sum(shape))
    v[:, :, -1, 3] = value
    o = run_gpu(q, k, v)
    assert (o[..., 3] == value).all()
    assert np.isfinite(np.delete(o, 3, axis=-1)).all()


# d = 128, 65 to 128 tiles of 16 rows: 8 lanes per row up to 224 keys, the matrix cores beyond.
@pytest.mark.parametrize("shape", [(1, 5, 211, 211), (2, 4, 200, 224), (1, 8, 250, 225), (3, 4, 97, 160)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
def test_f32_eight_lanes_per_row(shape, causal):
    B, H, Nq, Nk = shape
    if causal and Nq > Nk:
        pytest.skip("causal requires Nq <= Nk")
    q, k, v = gen(B, H, Nq, Nk, 128, "f32", seed=sum(shape))
    o, lse = run_gpu(q, k, v, causal=causal, return_lse=True)
    ref, ref_lse = oracle_full(q, k, v, causal=causal, with_lse=True)
    assert max_err(o, ref) <= TOL["f32"]
    assert max_err(lse, ref_lse) <= 1e-5 * max(1.0, np.abs(ref_lse).max())
