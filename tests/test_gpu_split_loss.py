"""Losses of the batch kernel on bf16 parts (product scores up to 128 dimensions) at the ends of what its sums hold."""

import numpy as np
import pytest

from oracle import negatives
from oracle.bucket import OracleConfig, Tables, batch_gradients
from tests.parity_util import kappa_for

pytestmark = pytest.mark.gpu

DOT = 0
SOFTMAX, LOGISTIC, SOFTMAX_POS, MARGIN = 0, 1, 2, 3


def _batch(node, edges, *, C, N, loss, seed=3, **kw):
    """One batch of the bucket between the two halves of the nodes, destinations corrupted: the library's loss, the oracle's loss, and
    the states (squares of the gradients)."""
    from paper_2505_09258_amd import binding as L
    V, d = node.shape
    args = dict(num_nodes=V, num_relations=0, dim=d, num_partitions=2, batch_size=edges.shape[0], chunk_size=C, num_negs=N,
                score=DOT, loss=loss, seed=seed, **kw)
    ctx = L.legend_init_partitions(L.make_config(**args), node, None)
    try:
        for p in range(2):
            L.legend_swap_partition(ctx, -1, p)
        L.legend_profile_enable(ctx, 0xffffffff)
        got = L.legend_train_bucket(ctx, 0, 1, edges)["loss_sum"]
        launches = {k: v["launches"] for k, v in L.legend_profile_read(ctx).items()}
        state = L.legend_read_embeddings(ctx, L.TABLE_NODE_STATE, None, V, d)
    finally:
        L.legend_destroy(ctx)
    assert launches["chunk_redo"] == 1                     # the launch behind the kernel on bf16 parts
    cfg = OracleConfig(**args)
    want, _, _ = batch_gradients(Tables(cfg, node, None), 0, 1, edges, 0, 0)
    return got, want, state


@pytest.mark.parametrize("d,N", [(33, 200), (100, 70), (128, 130), (40, 600)])
@pytest.mark.parametrize("loss", [SOFTMAX, SOFTMAX_POS])
def test_scores_far_below_any_finite_mask(d, N, loss):
    """All scores finite, between -1e34 and -1e32, in tiles with columns past the negatives: none of those may count."""
    rng = np.random.default_rng(d)
    V, B, C = 1_000, 64, 32
    node = (1e16 * (1.0 + rng.random((V, d)))).astype(np.float32)
    node[V // 2:] *= -1
    edges = np.stack([rng.integers(0, V // 2, B), np.zeros(B, np.int64), rng.integers(0, V // 2, B)], 1).astype(np.int32)
    got, want, state = _batch(node, edges, C=C, N=N, loss=loss)
    # scores 1e30 and more apart: the loss is a sum of differences of scores, each off by a few roundings of its own size, 4e32 d at
    # most (a weight is 0, 1 or a power of the rounding of its score: not asked for)
    assert abs(got - want) <= 1e-5 * abs(want) + B * kappa_for(d, "loss") * 4e32 * d
    assert np.isfinite(state).all()


@pytest.mark.parametrize("d,N", [(33, 200), (64, 50), (100, 333), (128, 130)])
@pytest.mark.parametrize("f", [12.0, 30.0, 75.0])
def test_dominating_positive_score(d, N, f):
    """Scores of zero and positive scores of f: the loss of a row is log(1 + N exp(-f)), far below the rounding of f."""
    V, B, C = 4_000, 100, 50
    node = np.zeros((V, d), np.float32)
    edges = np.stack([np.arange(B) % 50, np.zeros(B, np.int64), np.arange(B) % 50], 1).astype(np.int32)
    cfg = OracleConfig(num_nodes=V, num_relations=0, dim=d, num_partitions=2, batch_size=B, chunk_size=C, num_negs=N, score=DOT, seed=3)
    free = np.setdiff1d(np.arange(V // 2), negatives.batch_negatives(cfg, 0, 0, 1, 0, edges, edges))[:50]
    edges[:, 2] = free[edges[:, 2]]                  # uniform negatives do not depend on the edges
    node[:50, 3], node[V // 2 + free, 3] = 2.0, f / 2.0
    got, _, _ = _batch(node, edges, C=C, N=N, loss=SOFTMAX_POS)
    want = B * np.log1p(N * np.exp(-f))              # (a log-sum-exp less f cancels in 64 bits too)
    # x = log N - f is taken in double and rounded once (2^-24 of x, at most f, is the relative change of exp(x)); exp, log1p: some ulp
    assert abs(got - want) <= (f + 16) * 2.0 ** -24 * want


@pytest.mark.parametrize("d,N", [(33, 200), (100, 1000), (128, 333), (64, 61)])
def test_loss_of_equal_scores(d, N):
    """Scores of zero: every row's loss is log N, rounded to fp32 (2^-24; the logarithm is taken in double)."""
    B = 100
    edges = np.stack([np.arange(B), np.zeros(B, np.int64), np.arange(B)], 1).astype(np.int32)
    got, _, state = _batch(np.zeros((2_000, d), np.float32), edges, C=50, N=N, loss=SOFTMAX)
    assert abs(got - B * np.log(N)) <= 2.0 ** -24 * B * np.log(N)
    assert not state.any()


@pytest.mark.parametrize("d", [50, 100, 101, 112, 128])
def test_loss_over_many_scores_has_no_bias(d):
    """Positive scores of zero and no margin: the loss is the sum of the scores above zero, 400 000 of them.  Roundings of either sign
    average out (3 x 2^-24 of a score's root mean square each: 1e-9 of the sum); a mean of an eighth of 2^-24 of a score stays whole
    (9e-9 of the sum), and half of that is the bar."""
    rng = np.random.default_rng(d)
    V, B, N = 4_000, 800, 1_000
    node = (0.3 * rng.standard_normal((V, d))).astype(np.float32)
    node[V // 2:V // 2 + 100] = 0
    edges = np.stack([rng.integers(0, V // 2, B), np.zeros(B, np.int64), rng.integers(0, 100, B)], 1).astype(np.int32)
    errors = []
    for seed in range(4):
        got, want, _ = _batch(node, edges, C=50, N=N, loss=MARGIN, margin=0.0, seed=seed)
        errors.append((got - want) / want)
    assert abs(np.mean(errors)) <= 4.5e-9, errors
