"""Infinities and NaN in the tables: what they make of a gradient is what IEEE arithmetic on the sums of the model says, whatever
instructions the sums are made with, and it costs no more than finite numbers by more than a small factor."""

import numpy as np
import pytest

from oracle import negatives
from oracle.bucket import OracleConfig, Tables, batch_gradients
from tests.parity_util import STATE_RTOL, kappa_for

pytestmark = pytest.mark.gpu

DOT, TRANSE = 0, 3
LOGISTIC, SOFTMAX_POS, MARGIN, DST = 1, 2, 3, 0


def _one_batch(node, rel, edges, *, C, N, seed, on_parts=None, **kw):
    """The states after one batch of all edges (zero before: squares of the gradients) and the negatives per chunk.  on_parts: whether
    the batch has to have run on the kernel on bf16 parts, where that matters."""
    from paper_2505_09258_amd import binding as L
    V, d = node.shape
    B = edges.shape[0]
    cfg = L.make_config(num_nodes=V, dim=d, num_relations=0 if rel is None else rel.shape[0], batch_size=B, chunk_size=C,
                        num_negs=N, seed=seed, **kw)
    ctx = L.legend_init_partitions(cfg, node, rel)
    try:
        L.legend_swap_partition(ctx, -1, 0)
        if on_parts is not None:
            L.legend_profile_enable(ctx, 0xffffffff)
        L.legend_train_bucket(ctx, 0, 0, edges)
        if on_parts is not None:                   # the launch over flagged workgroups follows that kernel only
            assert L.legend_profile_read(ctx)["chunk_redo"]["launches"] == (1 if on_parts else 0)
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


def _expected(node, edges, *, C, N, seed, loss):
    cfg = OracleConfig(num_nodes=node.shape[0], num_relations=0, dim=node.shape[1], num_partitions=1, batch_size=edges.shape[0],
                       chunk_size=C, num_negs=N, score=DOT, loss=loss, corrupt=DST, seed=seed)
    with np.errstate(all="ignore"):
        _, grads, _ = batch_gradients(Tables(cfg, node, None), 0, 0, edges, 0, 0)
    g = np.zeros(node.shape)
    g[grads[0][0]] = grads[0][1]
    return g


@pytest.mark.parametrize("loss", [LOGISTIC, MARGIN], ids=["logistic", "margin"])
@pytest.mark.parametrize("where", ["negative", "source", "huge_negative"])
@pytest.mark.parametrize("d,C,N", [(130, 20, 70), (131, 113, 129), (256, 33, 200)])
def test_wide_path_infinite_rows(loss, where, d, C, N):
    """One component that is infinite, or finite above the largest bfloat16, in a row of negatives or in a composed row: its score
    is +inf (or huge), the weights stay finite, and a gradient sum is infinite exactly where the sum in 64 bits of the same
    numbers is beyond fp32."""
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
    state, _ = _one_batch(node, None, edges, score=DOT, loss=loss, corrupt=DST, **kw)
    g = _expected(node, edges, loss=loss, **kw)
    with np.errstate(all="ignore"):
        want = (g.astype(np.float32) * g.astype(np.float32))
    assert not np.isfinite(want).all()
    np.testing.assert_array_equal(np.isnan(state), np.isnan(want))
    np.testing.assert_array_equal(np.isinf(state), np.isinf(want))
    # a gradient is off by at most KAPPA times the sum of its terms' magnitudes: the positive's and the negatives' at most
    # a weight of 1 (logistic) or N (margin) times the largest finite component, for each occurrence of the row
    weight = 1.0 if loss == LOGISTIC else float(N)
    finite = node[np.isfinite(node) & (node < 1e30)].max()
    occurrences = np.bincount(np.concatenate([edges[:, 0], edges[:, 2], neg.reshape(-1)]), minlength=V)
    off = kappa_for(d) * 2.0 * weight * finite * (occurrences * max(1, C if loss == MARGIN else 1))[:, None]
    fine = np.isfinite(want)
    with np.errstate(all="ignore"):
        allowed = 2.0 * np.abs(g) * off + off ** 2
    assert (np.abs(state[fine].astype(np.float64) - want[fine]) <= STATE_RTOL * want[fine] + allowed[fine]).all()


def _train_ms(node, **kw):
    from paper_2505_09258_amd import binding as L
    V, d = node.shape
    rng = np.random.default_rng(1)
    edges = np.stack([rng.integers(0, V, 20_000), np.zeros(20_000, np.int64), rng.integers(0, V, 20_000)], 1).astype(np.int32)
    cfg = L.make_config(num_nodes=V, dim=d, batch_size=5_000, chunk_size=100, num_negs=1_000, score=DOT, corrupt=DST, seed=1, **kw)
    ctx = L.legend_init_partitions(cfg, node, None)
    try:
        L.legend_swap_partition(ctx, -1, 0)
        L.legend_train_bucket(ctx, 0, 0, edges)
        return min(L.legend_train_bucket(ctx, 0, 0, edges, epoch=k)["ms"] for k in range(3))
    finally:
        L.legend_destroy(ctx)


@pytest.mark.parametrize("share", [1.0, 0.01])
def test_wide_path_time_on_a_diverged_table(share):
    """A batch over a table in which every row, or one row in a hundred, is NaN takes about as long as over a finite one."""
    rng = np.random.default_rng(2)
    node = (0.1 * rng.standard_normal((4_000, 256))).astype(np.float32)
    finite = _train_ms(node, loss=LOGISTIC)
    node[rng.random(4_000) < share] = np.nan
    nan = _train_ms(node, loss=LOGISTIC)
    assert nan < 4 * finite


@pytest.mark.parametrize("share", [1.0, 0.01])
def test_rank_time_on_a_diverged_table(share):
    """The same for ranks."""
    from paper_2505_09258_amd import binding as L
    rng = np.random.default_rng(3)
    V, d, m = 6_000, 256, 3_000
    src, dst = rng.integers(0, V, m), rng.integers(0, V, m)
    node = (0.1 * rng.standard_normal((V, d))).astype(np.float32)
    ms = []
    for nan in (False, True):
        if nan:
            node[rng.random(V) < share] = np.nan
        cfg = L.make_config(num_nodes=V, dim=d, batch_size=1_000, chunk_size=50, num_negs=50, score=DOT, seed=1)
        ctx = L.legend_init_partitions(cfg, node, None)
        try:
            L.legend_swap_partition(ctx, -1, 0)
            L.legend_rank_edges(ctx, src, None, dst, DST, None)
            out = [L.legend_rank_edges(ctx, src, None, dst, DST, None) for _ in range(3)]
        finally:
            L.legend_destroy(ctx)
        ms.append(min(x[2]["ms"] for x in out))
    lost = np.isnan(node[src, 0]) | np.isnan(node[dst, 0])
    assert not out[0][0][lost].any() and not out[0][1][lost].any()
    assert ms[1] < 4 * ms[0]
