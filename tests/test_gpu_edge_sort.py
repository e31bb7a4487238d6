"""The sort that makes the CSC out of the edges, at the sizes where its kernels change: short and long inputs, whole and ragged tiles, digits of
every width; and edges that name no vertex, wherever they stand."""
import numpy as np
import pytest
import torch

from paper_2311_14898_amd import binding as B

pytestmark = pytest.mark.gpu
SHORT, TILE = 128 * 2048, 8192     # stored edges of the short inputs; of a tile of the long ones


@pytest.fixture(scope="module")
def ctx():
    c = B.ht_ctx_create(0)
    yield c
    B.ht_ctx_destroy(c)


@pytest.mark.parametrize("V,stored", [(1, 1), (2, 3), (3, 2_000), (300, 2048 * 3 + 1), (300, SHORT - 1), (300, SHORT), (300, SHORT + 1), (1_000, TILE * 41 - 1),
                                      (1_000, TILE * 41), (1_000, TILE * 41 + 1), (70_001, 8 * TILE * 9), (1_500_000, 2_600_003)])
@pytest.mark.parametrize("loops", [True, False])
def test_csc(ctx, V, stored, loops):
    E = stored - V if loops else stored
    rng = np.random.default_rng(V + stored)
    src, dst = (rng.integers(0, V, E) ** 2 // V).astype(np.int32), rng.integers(0, V, E).astype(np.int32)   # (many duplicates among the low ids)
    g = B.ht_partition(ctx, V, torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), 2, add_self_loops=loops)
    try:
        indptr, col, _, _ = B.ht_graph_export_csc(g)
    finally:
        B.ht_graph_destroy(g)
    v, u = dst.astype(np.int64), src.astype(np.int64)
    if loops:
        v, u = np.concatenate([v, np.arange(V)]), np.concatenate([u, np.arange(V)])
    order = np.lexsort((u, v))
    assert np.array_equal(col, u[order])
    assert np.array_equal(indptr, np.concatenate([[0], np.cumsum(np.bincount(v, minlength=V))]))


@pytest.mark.parametrize("E", [5_000, SHORT + 5])
@pytest.mark.parametrize("where", [0, -1])
@pytest.mark.parametrize("bad", [-1, 777])
def test_edges_that_name_no_vertex(ctx, E, where, bad):
    for side in range(2):
        ids = [torch.zeros(E, dtype=torch.int32) for _ in range(2)]
        ids[side][where] = bad
        with pytest.raises(RuntimeError, match="outside"):
            B.ht_partition(ctx, 777, ids[0].cuda(), ids[1].cuda(), 1)
