"""Gradient rows marked as streaming or not (LEGEND_STREAM_ROWS=1 and 0; by default a matter of size): the same bits from
every kernel that writes or reads them, and the same as by default."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DOT, DISTMULT, COMPLEX, TRANSE = 0, 1, 2, 3


def _tables(monkeypatch, knob, score, d, B, C, N, fp32=False):
    from paper_2505_09258_amd import binding as L
    monkeypatch.setenv("LEGEND_NO_FAST_CHUNK", "1" if fp32 else "0")
    if knob is None:
        monkeypatch.delenv("LEGEND_STREAM_ROWS", raising=False)
    else:
        monkeypatch.setenv("LEGEND_STREAM_ROWS", knob)
    V, nrel, m = 2_000, 3, 2 * B + 7
    rng = np.random.default_rng(d)
    node = (0.2 * rng.standard_normal((V, d))).astype(np.float32)
    rel = (0.2 * rng.standard_normal((nrel, d))).astype(np.float32)
    edges = np.stack([V * rng.random(m) ** 3, rng.integers(0, nrel, m), V * rng.random(m)], 1).astype(np.int32)   # rows with many gradient rows too
    cfg = L.make_config(num_nodes=V, dim=d, num_relations=nrel, score=score, corrupt=L.CORRUPT_BOTH, batch_size=B, chunk_size=C,
                        num_negs=N, seed=9)
    ctx = L.legend_init_partitions(cfg, node, rel if score else None)
    try:
        L.legend_swap_partition(ctx, -1, 0)
        loss = L.legend_train_bucket(ctx, 0, 0, edges)["loss_sum"]
        return [np.float64(loss)] + [L.legend_read_embeddings(ctx, t, None, V if t < 2 else nrel, d) for t in range(4)]
    finally:
        L.legend_destroy(ctx)


# kernel on bf16 parts (which marks none of its stores; rows of 16, 8 and 4 bytes' alignment), translational, wide path; a small batch
@pytest.mark.parametrize("score,d,B,C,N", [(DOT, 100, 500, 50, 200), (COMPLEX, 64, 500, 50, 200), (DOT, 128, 300, 50, 300),
                                           (DISTMULT, 50, 600, 60, 100), (DOT, 33, 600, 60, 100), (TRANSE, 60, 600, 60, 100),
                                           (TRANSE, 31, 600, 60, 100), (DISTMULT, 150, 300, 60, 200), (DOT, 256, 300, 60, 200),
                                           (DISTMULT, 32, 200, 50, 30)])
def test_same_bits(monkeypatch, score, d, B, C, N):
    always, never, chosen = (_tables(monkeypatch, k, score, d, B, C, N) for k in ("1", "0", None))
    for x, y, z in zip(always, never, chosen):
        assert np.array_equal(x, y) and np.array_equal(x, z)


# fp32 kernel, rows of 16 (with the dimension folded in and without), 8 and 4 bytes' alignment
@pytest.mark.parametrize("score,d,B,C,N", [(DOT, 100, 500, 50, 200), (DOT, 128, 300, 50, 300), (COMPLEX, 64, 500, 50, 200),
                                           (DISTMULT, 50, 600, 60, 100), (DOT, 33, 600, 60, 100)])
def test_same_bits_from_the_fp32_kernel(monkeypatch, score, d, B, C, N):
    always, never, chosen = (_tables(monkeypatch, k, score, d, B, C, N, fp32=True) for k in ("1", "0", None))
    for x, y, z in zip(always, never, chosen):
        assert np.array_equal(x, y) and np.array_equal(x, z)
