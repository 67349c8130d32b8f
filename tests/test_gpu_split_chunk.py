"""The batch kernel of the product scores up to 128 dimensions (bf16 parts) at the edges of its tiles and slices, and where a table
holds infinities or numbers above the largest bfloat16, which it hands to the fp32 kernel.  Bars and inputs as in the parity tests."""

import numpy as np
import pytest

from tests.test_gpu_nonfinite import DOT, DST, LOGISTIC, MARGIN, _expected, _one_batch
from tests.test_gpu_parity import BOTH, COMPLEX, DISTMULT, SOFTMAX, SOFTMAX_POS, SRC, _case, _check_every_batch
from tests.parity_util import STATE_RTOL, kappa_for

pytestmark = pytest.mark.gpu

# Dimensions on both sides of every class of column blocks (32, 64, 96, 100, 128), of slices of 32 and of the row alignments 16, 8 and 4;
# negatives on both sides of tiles of 32 and 64 and beyond what LDS holds of their ids; rows on both sides of 16, 32 and 64.
_EDGES = [
    # up to 32 dimensions: the consumers share two blocks of columns by halves; every loss at every alignment
    _case("dot_d1_n10000_rows16", DOT, SOFTMAX, DST, 900, 0, 1, 1, 0, 0, 32, 16, 10_000, 0, 70, 0.5),
    _case("dot_d4_n1300_rows50", DOT, MARGIN, DST, 900, 0, 4, 1, 0, 0, 100, 50, 1_300, 0, 140, 0.5),
    _case("dot_d17_n300_rows48", DOT, SOFTMAX_POS, DST, 900, 0, 17, 1, 0, 0, 96, 48, 300, 0, 200, 0.4),
    _case("complex_d18_n300_rows40", COMPLEX, LOGISTIC, BOTH, 900, 3, 18, 1, 0, 0, 80, 40, 300, 0, 170, 0.4),
    _case("complex_d26_n200_rows64", COMPLEX, SOFTMAX, SRC, 900, 3, 26, 2, 1, 0, 128, 64, 200, 0, 270, 0.4),
    _case("dot_d29_n180_rows20", DOT, MARGIN, BOTH, 900, 0, 29, 1, 0, 0, 60, 20, 180, 0, 130, 0.4),
    _case("distmult_d30_n200_rows33", DISTMULT, MARGIN, DST, 900, 3, 30, 1, 0, 0, 99, 33, 200, 0, 210, 0.4),
    _case("dot_d31_n193_rows17", DOT, LOGISTIC, DST, 900, 0, 31, 1, 0, 0, 68, 17, 193, 0, 140, 0.4),
    _case("distmult_d32_n257_rows32", DISTMULT, SOFTMAX, BOTH, 900, 3, 32, 1, 0, 0, 96, 32, 257, 9, 200, 0.4),
    _case("dot_d32_n160_rows64", DOT, LOGISTIC, SRC, 900, 0, 32, 1, 0, 0, 128, 64, 160, 0, 270, 0.4),
    # the other classes
    _case("complex_d34_n129_rows33", COMPLEX, MARGIN, SRC, 900, 3, 34, 2, 1, 0, 99, 33, 129, 0, 210, 0.4),
    _case("dot_d64_n193_rows64", DOT, SOFTMAX_POS, DST, 900, 0, 64, 1, 0, 0, 128, 64, 193, 0, 300, 0.3),
    _case("distmult_d65_n96_rows65", DISTMULT, LOGISTIC, BOTH, 900, 3, 65, 1, 0, 0, 130, 65, 96, 5, 270, 0.3),
    _case("complex_d96_n66_rows1", COMPLEX, SOFTMAX, BOTH, 900, 3, 96, 1, 0, 0, 12, 1, 66, 0, 30, 0.3),
    _case("dot_d97_n257_rows50", DOT, SOFTMAX, SRC, 900, 0, 97, 2, 0, 1, 100, 50, 257, 0, 230, 0.3),
    _case("complex_d98_n100_rows49", COMPLEX, LOGISTIC, DST, 900, 3, 98, 1, 0, 0, 98, 49, 100, 0, 220, 0.3),
    _case("dot_d99_n1030_rows20", DOT, SOFTMAX, DST, 900, 0, 99, 1, 0, 0, 40, 20, 1030, 100, 90, 0.3),
    _case("distmult_d100_n95_rows47", DISTMULT, MARGIN, DST, 900, 3, 100, 1, 0, 0, 94, 47, 95, 0, 220, 0.3),
    _case("dot_d101_n160_rows31", DOT, SOFTMAX_POS, BOTH, 900, 0, 101, 1, 0, 0, 93, 31, 160, 0, 200, 0.25),
    _case("complex_d126_n70_rows63", COMPLEX, SOFTMAX, SRC, 900, 3, 126, 1, 0, 0, 126, 63, 70, 0, 260, 0.25),
    _case("distmult_d128_n1100_rows48", DISTMULT, LOGISTIC, DST, 900, 3, 128, 1, 0, 0, 96, 48, 1100, 0, 200, 0.25),
    # few negatives: tiles that are empty or nearly so
    _case("dot_d128_n20_rows50", DOT, SOFTMAX, DST, 900, 0, 128, 1, 0, 0, 150, 50, 20, 0, 310, 0.25),
    _case("distmult_d100_n33_rows40", DISTMULT, SOFTMAX, BOTH, 2_000, 3, 100, 1, 0, 0, 80, 40, 33, 0, 170, 0.3),
    # more than 4096 gradient rows a batch
    _case("distmult_d100_n100_many", DISTMULT, SOFTMAX, BOTH, 2_000, 3, 100, 1, 0, 0, 1_600, 40, 100, 0, 1_700, 0.3),
    _case("dot_d20_n513_many", DOT, LOGISTIC, DST, 2_000, 0, 20, 1, 0, 0, 2_100, 50, 513, 0, 2_200, 0.3),
]


@pytest.mark.parametrize("c", _EDGES, ids=[c["name"] for c in _EDGES])
def test_at_the_edges_of_its_tiles(c):
    _check_every_batch(c, on_parts=True)


@pytest.mark.parametrize("c", _EDGES, ids=[c["name"] for c in _EDGES])
def test_the_same_through_the_fp32_kernel(monkeypatch, c):
    """What serves atomic mode, small chunks and chunks with numbers that are not finite, at the same sizes."""
    monkeypatch.setenv("LEGEND_NO_FAST_CHUNK", "1")
    _check_every_batch(c, on_parts=False)


@pytest.mark.parametrize("loss", [LOGISTIC, MARGIN], ids=["logistic", "margin"])
@pytest.mark.parametrize("where", ["negative", "source", "huge_negative"])
@pytest.mark.parametrize("d,C,N", [(20, 20, 250), (31, 50, 200), (99, 64, 129), (128, 33, 200)])
def test_infinite_rows(loss, where, d, C, N):
    """One component that is infinite, or finite above the largest bfloat16, in a row of negatives or in a composed row: a gradient
    sum is infinite, or not a number, exactly where the sum in 64 bits of the same numbers is beyond fp32, or not a number."""
    rng = np.random.default_rng(d)
    V = 700
    node = (0.1 * np.abs(rng.standard_normal((V, d))) + 0.01).astype(np.float32)       # positive: no inf - inf in the scores
    edges = np.stack([rng.integers(0, 200, 2 * C), np.zeros(2 * C, np.int64), rng.integers(200, 400, 2 * C)], 1).astype(np.int32)
    kw = dict(C=C, N=N, seed=6)
    _, neg = _one_batch(node, None, edges, score=DOT, loss=loss, corrupt=DST, **kw)
    if where == "source":
        row = next(int(v) for v in edges[:, 0] if v not in set(neg.reshape(-1).tolist()))
    else:
        row = next(int(v) for v in neg[0] if v >= 400)
    node[row, d // 3] = 3.4e38 if where == "huge_negative" else np.inf
    state, _ = _one_batch(node, None, edges, score=DOT, loss=loss, corrupt=DST, on_parts=True, **kw)
    g = _expected(node, edges, loss=loss, **kw)
    with np.errstate(all="ignore"):
        want = (g.astype(np.float32) * g.astype(np.float32))
    assert not np.isfinite(want).all()
    np.testing.assert_array_equal(np.isnan(state), np.isnan(want))
    np.testing.assert_array_equal(np.isinf(state), np.isinf(want))
    # off by at most KAPPA times the sum of the terms' magnitudes: weights of at most 1 (logistic) or N (margin) times the largest
    # finite component, for each occurrence of the row
    weight = 1.0 if loss == LOGISTIC else float(N)
    finite = node[np.isfinite(node) & (node < 1e30)].max()
    occurrences = np.bincount(np.concatenate([edges[:, 0], edges[:, 2], neg.reshape(-1)]), minlength=V)
    off = kappa_for(d) * 2.0 * weight * finite * (occurrences * max(1, C if loss == MARGIN else 1))[:, None]
    fine = np.isfinite(want)
    with np.errstate(all="ignore"):
        allowed = 2.0 * np.abs(g) * off + off ** 2
    assert (np.abs(state[fine].astype(np.float64) - want[fine]) <= STATE_RTOL * want[fine] + allowed[fine]).all()


def _launches(loss, d, N, B, **kw):
    from paper_2505_09258_amd import binding as L
    V = 3_000
    rng = np.random.default_rng(d)
    edges = np.stack([rng.integers(0, V, B), np.zeros(B, np.int64), rng.integers(0, V, B)], 1).astype(np.int32)
    ctx = L.legend_init_partitions(L.make_config(num_nodes=V, dim=d, batch_size=B, chunk_size=50, num_negs=N, score=DOT, loss=loss,
                                                 seed=1, **kw), np.full((V, d), 0.01, np.float32), None)
    try:
        L.legend_swap_partition(ctx, -1, 0)
        L.legend_profile_enable(ctx, 0xffffffff)
        L.legend_train_bucket(ctx, 0, 0, edges)
        return {k: v["launches"] for k, v in L.legend_profile_read(ctx).items()}
    finally:
        L.legend_destroy(ctx)


# 500 edges and 10 chunks of up to 300 negatives are at most 4096 gradient rows, 2 500 edges are more
@pytest.mark.parametrize("d,N,B,split", [(32, 78, 500, False), (36, 70, 500, True), (128, 19, 500, False), (128, 20, 500, True),
                                         (32, 156, 500, False), (32, 157, 500, True), (100, 64, 500, True),
                                         (100, 99, 2_500, False), (100, 100, 2_500, True), (50, 199, 2_500, False),
                                         (128, 124, 2_500, False), (128, 125, 2_500, True), (101, 158, 2_500, False)])
@pytest.mark.parametrize("loss", [SOFTMAX, LOGISTIC, MARGIN], ids=["softmax", "logistic", "margin"])
def test_which_kernel_runs(loss, d, N, B, split):
    """Few negatives of few dimensions are for the fp32 kernel, fewer in small batches, whatever the loss; a launch over flagged
    workgroups follows the kernel on bf16 parts only."""
    launches = _launches(loss, d, N, B)
    assert launches["chunk"] == 1 and launches["chunk_redo"] == (1 if split else 0)
