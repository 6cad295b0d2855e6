"""Candidate images at the edges of the counting and ranking kernels: image
counts around the 64-image blocks, point counts around the 512-point units and
the slices, and rows where many images share the count that top_k cuts through
(few enough to rank by counting, and more than that).  Against the oracle,
with each counting method and the automatic choice."""
import numpy as np
import pytest

from tests.test_gpu_covis import _check, sfm  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, npts", [(2, 31), (63, 511), (64, 512), (65, 513), (129, 4097),
                                     (200, 40001)])
def test_block_and_unit_edges(sfm, n, npts):
    rng = np.random.default_rng(n)
    lists = [np.sort(rng.choice(npts, size=min(npts, int(rng.integers(1, 900))), replace=False))
             .astype(np.int32) for _ in range(n)]
    lists[0] = np.array([0, npts - 1], np.int32)
    lists[-1] = np.array([0, npts - 1], np.int32)
    m = sfm.Matcher()
    for method in (1, 2, 0):
        sfm.sfm_set_covis_method(m.ctx, method)
        _check(sfm, m, lists, npts, 0, 7)
    m.close()


@pytest.mark.parametrize("shared, rest, k", [(300, 0, 9), (300, 40, 50), (700, 30, 20),
                                             (1100, 3, 1105)])
def test_shared_counts_at_the_cut(sfm, shared, rest, k):
    """`shared` images see the same 40 points, `rest` images some of them."""
    rng = np.random.default_rng(shared)
    every = np.arange(40, dtype=np.int32)
    lists = [every] * shared + [np.sort(rng.choice(40, size=int(s), replace=False)).astype(np.int32)
                                for s in rng.integers(1, 40, rest)]
    lists = [lists[i] for i in rng.permutation(len(lists))]
    m = sfm.Matcher()
    for method in (1, 2):
        sfm.sfm_set_covis_method(m.ctx, method)
        _check(sfm, m, lists, 40, 8, k)
    m.close()
