"""Infinities and NaN in the tables: what they make of a gradient is what IEEE arithmetic on the sums of the model says, whatever
instructions the sums are made with, and it costs no more than finite numbers by more than a small factor."""

import numpy as np
import pytest

from oracle import negatives
from oracle.bucket import OracleConfig

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore:overflow encountered")]

DOT, TRANSE = 0, 3
LOGISTIC, SOFTMAX_POS, MARGIN, DST = 1, 2, 3, 0


def _one_batch(node, rel, edges, *, C, N, seed, **kw):
    """The states after one batch of all edges (zero before: squares of the gradients) and the negatives per chunk."""
    from paper_2505_09258_amd import binding as L
    V, d = node.shape
    B = edges.shape[0]
    cfg = L.make_config(num_nodes=V, dim=d, num_relations=0 if rel is None else rel.shape[0], batch_size=B, chunk_size=C,
                        num_negs=N, seed=seed, **kw)
    ctx = L.legend_init_partitions(cfg, node, rel)
    try:
        L.legend_swap_partition(ctx, -1, 0)
        L.legend_train_bucket(ctx, 0, 0, edges)
        state = L.legend_read_embeddings(ctx, L.TABLE_NODE_STATE, None, V, d)
    finally:
        L.legend_destroy(ctx)
    ocfg = OracleConfig(num_nodes=V, num_relations=0 if rel is None else rel.shape[0], dim=d, num_partitions=1, batch_size=B,
                        chunk_size=C, num_negs=N, score=kw["score"], corrupt=DST, seed=seed)
    return state, negatives.batch_negatives(ocfg, 0, 0, 0, 0, edges, edges)[0]


@pytest.mark.parametrize("d,C,N", [(36, 32, 70), (33, 20, 64), (128, 64, 130)])
def test_translational_nan_positive_score_gives_nan_weights(d, C, N):
    """The NaN stands in a row that is only a positive's replaced endpoint: every component of the sums is in range, the weights of
    one row of the chunk are not."""
    rng = np.random.default_rng(d)
    V = 900
    node = (0.3 * rng.standard_normal((V, d))).astype(np.float32)
    rel = (0.3 * rng.standard_normal((2, d))).astype(np.float32)
    edges = np.stack([rng.integers(0, 300, C), rng.integers(0, 2, C), rng.integers(0, 300, C)], 1).astype(np.int32)
    kw = dict(C=C, N=N, seed=4, score=TRANSE, loss=SOFTMAX_POS, corrupt=DST)
    _, neg = _one_batch(node, rel, edges, **kw)
    victim = next(v for v in range(300, V) if v not in set(neg[0].tolist()))
    edges[5, 2] = victim                       # uniform negatives do not depend on the edges
    node[victim, d // 2] = np.nan
    state, neg = _one_batch(node, rel, edges, **kw)
    assert victim not in set(neg[0].tolist())
    assert np.isnan(state[neg[0]]).all()       # each negative's gradient has the NaN weight of edge 5 in it
    assert not np.isinf(state).any()
    rest = np.setdiff1d(np.concatenate([edges[:, 0], edges[:, 2]]), np.concatenate([neg[0], [edges[5, 0], victim]]))
    assert rest.size and np.isfinite(state[rest]).all() and state[rest].any()
