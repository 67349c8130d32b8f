"""Large table reads (pinned ring, several threads) against the table that went in, bit for bit."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# 32 MB is the smallest read that takes the ring of 1 MB blocks
@pytest.mark.parametrize("V,d,n,capacity", [(65_535, 128, 1, 1), (65_536, 128, 1, 1), (65_537, 128, 1, 1), (180_001, 64, 3, 3),
                                            (400_003, 50, 5, 3)])
def test_whole_table_read_returns_the_table(V, d, n, capacity):
    from paper_2505_09258_amd import binding as L
    node = np.random.default_rng(V).standard_normal((V, d)).astype(np.float32)
    cfg = L.make_config(num_nodes=V, dim=d, num_partitions=n, buffer_capacity=capacity, batch_size=100, chunk_size=10,
                        num_negs=10, seed=1)
    ctx = L.legend_init_partitions(cfg, node, None)
    try:
        for p in range(capacity):
            L.legend_swap_partition(ctx, -1, p)                # the others are read from the host tier
        for m in (V, V - 1):
            assert (L.legend_read_embeddings(ctx, L.TABLE_NODE_EMB, None, m, d) == node[:m]).all()
        assert not L.legend_read_embeddings(ctx, L.TABLE_NODE_STATE, None, V, d).any()
    finally:
        L.legend_destroy(ctx)


def test_whole_table_read_into_page_locked_memory():
    """Goes as one copy and not through the ring; the same bytes."""
    import ctypes
    import torch
    from paper_2505_09258_amd import binding as L
    V, d = 90_001, 100
    node = np.random.default_rng(1).standard_normal((V, d)).astype(np.float32)
    cfg = L.make_config(num_nodes=V, dim=d, num_partitions=2, batch_size=100, chunk_size=10, num_negs=10, seed=1)
    ctx = L.legend_init_partitions(cfg, node, None)
    try:
        L.legend_swap_partition(ctx, -1, 0)                    # the second half comes from the host tier
        out = torch.zeros((V, d), dtype=torch.float32, pin_memory=True)
        L._check(L._lib.legend_read_embeddings(ctx, L.TABLE_NODE_EMB, None, V, ctypes.c_void_p(out.data_ptr())))
        assert (out.numpy() == node).all()
    finally:
        L.legend_destroy(ctx)
