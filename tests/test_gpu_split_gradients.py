"""Gradients of the batch kernel on bf16 parts (product scores up to 128 dimensions) against 64 bits: sums over many negatives."""

import numpy as np
import pytest

from oracle.bucket import OracleConfig, Tables, batch_gradients

pytestmark = pytest.mark.gpu

DOT = 0
SOFTMAX, LOGISTIC, SOFTMAX_POS, MARGIN = 0, 1, 2, 3


def _source_rows(node, edges, *, C, N, loss, **kw):
    """One batch of the bucket between the two halves of the nodes, destinations corrupted: magnitudes of the gradients of the source
    rows (root of the state, zero before) from the library, and the oracle's gradients."""
    from paper_2505_09258_amd import binding as L
    V, d = node.shape
    args = dict(num_nodes=V, num_relations=0, dim=d, num_partitions=2, batch_size=edges.shape[0], chunk_size=C, num_negs=N,
                score=DOT, loss=loss, seed=3, **kw)
    ctx = L.legend_init_partitions(L.make_config(**args), node, None)
    try:
        for p in range(2):
            L.legend_swap_partition(ctx, -1, p)
        L.legend_profile_enable(ctx, 0xffffffff)
        L.legend_train_bucket(ctx, 0, 1, edges)
        launches = {k: v["launches"] for k, v in L.legend_profile_read(ctx).items()}
        state = L.legend_read_embeddings(ctx, L.TABLE_NODE_STATE, None, V, d)
    finally:
        L.legend_destroy(ctx)
    assert launches["chunk_redo"] == 1                     # the launch behind the kernel on bf16 parts
    rows, grads = batch_gradients(Tables(OracleConfig(**args), node, None), 0, 1, edges, 0, 0)[1][0]
    return np.sqrt(state[rows].astype(np.float64)), grads


@pytest.mark.parametrize("d,N", [(20, 4_000), (100, 4_000), (101, 16_000), (114, 4_000), (128, 1_000), (128, 16_000)])
@pytest.mark.parametrize("loss", [LOGISTIC, MARGIN], ids=["logistic", "margin"])
def test_sums_of_one_sign(d, N, loss):
    """Positive components, weights all near one half, or one, and destinations of zero: a source row's sum grows evenly over N / 32
    additions, each off by at most half an ulp of the sum so far (at most 2^-24 of it): 2^-24 sqrt(N / 32 / 3 / 3) of the result in
    the root mean square.  Twice that is the bar, and four roundings (exponential, sum, division, root of the state) of a weight near
    one half, which all weights may share."""
    rng = np.random.default_rng(d)
    V, B = 4_000, 100
    node = np.abs(0.05 * rng.standard_normal((V, d))).astype(np.float32)
    node[V // 2:V // 2 + 50] = 0
    edges = np.stack([rng.permutation(V // 2)[:B], np.zeros(B, np.int64), rng.integers(0, 50, B)], 1).astype(np.int32)
    got, want = _source_rows(node, edges, C=50, N=N, loss=loss, **(dict(neg_weight=1.0) if loss == LOGISTIC else dict(margin=2.0)))
    assert (want > 0).all()
    roundings = 2.0 * (N / 288) ** 0.5 + (4.0 if loss == LOGISTIC else 0.0)
    error = np.linalg.norm(got - want) / np.linalg.norm(want)
    assert error <= roundings * 2.0 ** -24, error * 2.0 ** 24


@pytest.mark.parametrize("d,N,std", [(20, 700, 2.5), (64, 600, 1.3), (100, 1_000, 1.05), (128, 1_000, 0.95)])
@pytest.mark.parametrize("loss", [SOFTMAX, SOFTMAX_POS], ids=["softmax", "softmax_pos"])
def test_copies_of_a_dominating_negative(d, N, std, loss):
    """Every source row stands several times among the negatives, with a score that lies 50 to 150 above the rest: some waves raise their
    references for a row of their tile above 110, others keep theirs, and the sums of either belong together."""
    rng = np.random.default_rng(d)
    V, B, C = 600, 300, 50
    node = (std * rng.standard_normal((V, d))).astype(np.float32)
    node[V // 2:] = node[:V // 2]
    edges = np.stack([rng.permutation(V // 2)[:B], np.zeros(B, np.int64), rng.integers(0, V // 2, B)], 1).astype(np.int32)
    got, want = _source_rows(node, edges, C=C, N=N, loss=loss)
    # weights that do not add up to 1 to fp32's precision are off by 2^-24 times a score (256 or so at most), and as much for their sum
    bound = 2.0 ** -24 * 512 * np.abs(node).max()
    assert np.abs(got - np.abs(want)).max() <= bound, np.abs(got - np.abs(want)).max() / bound


@pytest.mark.parametrize("d,N,std", [(32, 600, 1.6), (64, 600, 1.2), (96, 1_000, 1.0), (100, 1_000, 1.0), (104, 1_000, 0.95), (128, 1_000, 0.85)])
@pytest.mark.parametrize("loss", [SOFTMAX, SOFTMAX_POS], ids=["softmax", "softmax_pos"])
def test_weight_of_a_dominating_negative(d, N, std, loss):
    """Every source row stands among the destinations too: as a negative its score is near 100, where the others, the softmax reference
    among them, are in the tens.  Its weight is 1, and the gradient the row less the destination's."""
    rng = np.random.default_rng(d)
    V, B, C = 2_000, 400, 50
    node = (std * rng.standard_normal((V, d))).astype(np.float32)
    node[V // 2:] = node[:V // 2]
    edges = np.stack([rng.permutation(V // 2)[:B], np.zeros(B, np.int64), rng.integers(0, V // 2, B)], 1).astype(np.int32)
    got, want = _source_rows(node, edges, C=C, N=N, loss=loss)
    source = node[np.sort(edges[:, 0])].astype(np.float64)
    destination = node[edges[np.argsort(edges[:, 0]), 2]]
    alone = np.abs(want - (source - destination)).max(axis=1) < 1e-8        # the weight is 1 to 64 bits, as good as
    assert alone.sum() > 50
    # the weight: the row's sum in two exponentials squared and a few additions, the logarithm of it in 64 bits and rounded to 48, one
    # exponential: some eight roundings, of the source row; one each of the difference and of the root of the state
    allowed = 2.0 ** -24 * (8.0 * np.abs(source[alone]) + 2.0 * np.abs(want[alone])) + 1e-8
    share = np.abs(got[alone] - np.abs(want[alone])) / allowed
    assert share.max() <= 1.0, share.max()
