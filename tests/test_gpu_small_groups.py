"""Small batches, whose index sides are made in groups of 32 on two sets of buffers, against the same calls with every
batch's index side made on its own (LEGEND_SERIAL_SORT=1): same sums in the same order, so the same bits."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _run(monkeypatch, serial, calls, m, update_mode=0, no_small_update=False, d=20, N=33):
    from paper_2505_09258_amd import binding as L
    V, B = 900, 60
    rng = np.random.default_rng(3)
    node = (0.3 * rng.standard_normal((V, d))).astype(np.float32)
    rel = (0.3 * rng.standard_normal((4, d))).astype(np.float32)
    edges = np.stack([(V // 2 * rng.random(m) ** 3), rng.integers(0, 4, m), V // 2 * rng.random(m)], 1).astype(np.int32)
    monkeypatch.setenv("LEGEND_SERIAL_SORT", "1" if serial else "0")
    monkeypatch.setenv("LEGEND_NO_SMALL_UPDATE", "1" if no_small_update else "0")
    cfg = L.make_config(num_nodes=V, dim=d, num_partitions=2, num_relations=4, score=L.SCORE_DISTMULT, corrupt=L.CORRUPT_BOTH,
                        batch_size=B, chunk_size=20, num_negs=N, num_degree_negs=5, seed=2, update_mode=update_mode)
    ctx = L.legend_init_partitions(cfg, node, rel)
    try:
        for p in range(2):
            L.legend_swap_partition(ctx, -1, p)
        out = []
        for k, (lo, hi) in enumerate(calls):
            st = L.legend_train_bucket_range(ctx, 0, 1, edges, epoch=k, batch_begin=lo, batch_end=hi)
            out.append(st["loss_sum"])
        out.append(L.legend_unique_rows_read(ctx))
        return out, [L.legend_read_embeddings(ctx, t, None, V if t < 2 else 4, d) for t in range(4)]
    finally:
        L.legend_destroy(ctx)


# whole buckets of 1, 31, 32, 33, 64, 65 and 97 batches with a ragged last one, and ranges that begin and end inside
@pytest.mark.parametrize("m,calls", [(59, [(0, 1)]), (31 * 60 - 1, [(0, 31)]), (32 * 60, [(0, 32)] * 2), (33 * 60 - 59, [(0, 33)] * 2),
                                     (64 * 60, [(0, 64)]), (65 * 60 - 7, [(0, 65)] * 2), (97 * 60 - 30, [(0, 97)] * 3),
                                     (80 * 60 - 11, [(3, 40), (40, 41), (10, 80)])])
def test_groups_give_the_bits_of_single_batches(monkeypatch, m, calls):
    a, ta = _run(monkeypatch, False, calls, m)
    b, tb = _run(monkeypatch, True, calls, m)
    assert a == b
    for x, y in zip(ta, tb):
        assert (x == y).all()


@pytest.mark.parametrize("m,calls", [(59, [(0, 1)]), (33 * 60 - 59, [(0, 33)] * 2), (80 * 60 - 11, [(3, 40), (40, 41), (10, 80)])])
@pytest.mark.parametrize("d,N", [(36, 70), (100, 33)])
def test_groups_on_the_kernel_on_bf16_parts(monkeypatch, m, calls, d, N):
    """Its two launches a batch (more than 32 dimensions, 2500 negatives x dimensions and more) read their ids from a slab."""
    a, ta = _run(monkeypatch, False, calls, m, d=d, N=N)
    b, tb = _run(monkeypatch, True, calls, m, d=d, N=N)
    assert a == b
    for x, y in zip(ta, tb):
        assert (x == y).all()


@pytest.mark.parametrize("m,calls", [(33 * 60 - 59, [(0, 33)] * 2), (80 * 60 - 11, [(3, 40), (10, 80)])])
def test_groups_with_the_general_update_kernels(monkeypatch, m, calls):
    """The update kernels of larger batches read their lists from a slab: the same bits again."""
    a, ta = _run(monkeypatch, False, calls, m, no_small_update=True)
    b, tb = _run(monkeypatch, True, calls, m)
    assert a == b
    for x, y in zip(ta, tb):
        assert (x == y).all()


@pytest.mark.parametrize("m,calls", [(59, [(0, 1)]), (65 * 60 - 7, [(0, 65)])])
def test_groups_in_atomic_mode(monkeypatch, m, calls):
    """The atomic update reads its rows from a slab.  Sums in arrival order: the first batch of a run to a few roundings
    of a gradient (Adagrad's first step is lr times its sign), rows touched and their number exactly."""
    a, ta = _run(monkeypatch, False, calls, m, update_mode=1)
    b, tb = _run(monkeypatch, True, calls, m, update_mode=1)
    assert a[-1] == b[-1]                                      # unique rows of every batch, batches
    for x, y in zip(a[:-1], b[:-1]):
        assert abs(x - y) <= 1e-5 * abs(y)
    for t in (1, 3):                                           # states: zero exactly where nothing was touched
        assert ((ta[t] != 0) == (tb[t] != 0)).all()
    if calls == [(0, 1)]:
        scale = np.sqrt(tb[1].max())                           # the largest gradient element
        # at most 60 + 3 * 33 terms meet in an element, each off by half a unit of the running sum
        assert np.abs(np.sqrt(ta[1]) - np.sqrt(tb[1])).max() <= 160 * 2.0 ** -24 * scale
