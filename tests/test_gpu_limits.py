"""Calls at their workspace budget: what fitted a budget once still does, and
gives the same results as with room to spare."""
import math

import numpy as np
import pytest

from tests.fixtures import random_pair, translation_F

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sfm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_06235_amd as sfm
    sfm.lib()
    return sfm


def aligned(sections, to=256):
    return sum(-(-s // to) * to for s in sections)


def four_grids_bytes(pairs, boxes, n):
    """Workspace of the grid search with a table and cursors for each of its four
    grids, a block of sixteen queries and four item lists (what calls were sized
    for first); boxes are (x0, y0, x1, y1) of the targets."""
    cells = 0
    for _, b, d in pairs:
        x0, y0, x1, y1 = boxes[b]
        for sx in (0.0, d):
            for sy in (0.0, d):
                side = [math.floor((hi - s) / (2 * d)) - math.floor((lo - s) / (2 * d)) + 1
                        for lo, hi, s in ((x0, x1, sx), (y0, y1, sy))]
                cells += side[0] * side[1] + 1
    P, na = len(pairs), sum(n[a] for a, _, _ in pairs)
    return aligned([168 * P, 96 * P, 72 * P, 8 * sum(-(-n[a] // 16) for a, _, _ in pairs), 8 * P,
                    4 * cells, 4 * cells, 16 * sum(n[b] for _, b, _ in pairs), 16 * na, 32 * P])


@pytest.mark.parametrize("size,d,n", [((40000, 0.75), 0.5, 5), ((0.5, 30000), 1.0, 3),
                                      ((0.25, 0.25), 2.0, 40), ((1024, 768), 4.0, 300)])
def test_grid_of_thin_boxes_fits(sfm, size, d, n):
    """Boxes one cell thin, a single cell, and an image."""
    from oracle.grid import grid_match
    from tests.test_gpu_grid import _check
    rng = np.random.default_rng(n)
    _, desc, _, _, _ = random_pair(n, 0, seed=n)
    xy = (rng.uniform(0, 1, (n, 2)) * size + 0.25).astype(np.float32)
    xy[:2] = [[0.25, 0.25], [0.25 + size[0], 0.25 + size[1]]]
    images = [(xy, desc // 16)]
    box = tuple(float(v) for v in (*xy.min(axis=0), *xy.max(axis=0)))
    pairs = [(0, 0, d)] * 3
    Fs = [translation_F((1.0, 0.0, 0.0)), translation_F((0.0, 1.0, 0.0)),
          translation_F((size[0] / 2, size[1] / 3, 1.0))]
    m = sfm.Matcher(workspace_budget_bytes=four_grids_bytes(pairs, [box], [n])).register(images)
    out = m.match(pairs, Fs, form="grid", emit_all=True)
    _check(out, images, pairs, Fs, grid_match(images, pairs, Fs))
    m.close()


def _lists(n, npts, most, seed):
    rng = np.random.default_rng(seed)
    return [np.sort(rng.choice(npts, size=int(rng.integers(1, most + 1)), replace=False))
            .astype(np.int32) for _ in range(n)]


def product_bytes(n, npts):
    """Workspace of the bit-matrix product with bitset rows of the points' words."""
    words, side = -(-npts // 32), max(n, npts) + 1
    return aligned([4, 4 * ((side + 8191) // 8192 + 1), 4 * (n + 1), 4 * n * -(-n // 32),
                    4 * n * words, 4 * n * n])


@pytest.mark.parametrize("n, npts", [(2, 1), (65, 33), (129, 523), (200, 70), (300, 4000)])
def test_product_without_padded_rows(sfm, n, npts):
    """The product on a budget that holds the points' words and one count matrix."""
    from tests.test_gpu_covis import _check
    m = sfm.Matcher(workspace_budget_bytes=product_bytes(n, npts))
    for method in (2, 0):
        sfm.sfm_set_covis_method(m.ctx, method)
        _check(sfm, m, _lists(n, npts, min(npts, 200), n), npts, 0, 9)
    m.close()


def test_product_that_does_not_fit_leaves_it_to_the_histogram(sfm):
    """3,200 images of 600 points, for which the product is the faster: a budget
    for its bitsets and counts that has no room for the pairs' bits (1.3 MB)."""
    from tests.test_gpu_covis import _check
    n, npts = 3200, 600
    m = sfm.Matcher(workspace_budget_bytes=4 * n * (32 + n) + (1 << 20))
    _check(sfm, m, _lists(n, npts, 30, 5), npts, 2, 9)
    m.close()


def test_registration_keeps_no_order_of_large_images(sfm):
    """The spatial order (13 bytes a feature and padding) is for images of at most
    65,536 features; larger ones keep the two words per feature that matching
    reads.  Matching at either side of the size equals the exhaustive form on an
    unbounded band."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(1)

    def image(n):
        xy = torch.rand(n, 2, device="cuda", generator=gen) * 1000
        return xy, torch.randint(0, 128, (n, 128), dtype=torch.uint8, device="cuda", generator=gen)

    large = [image(400_000) for _ in range(4)]
    torch.cuda.synchronize()
    m = sfm.Matcher().register([image(40)])   # (kernels are loaded)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    m.register(large)
    took = free - torch.cuda.mem_get_info()[0]
    assert 8 * 1_600_000 <= took < 8 * 1_600_000 + (6 << 20), took
    edge = [image(65536), image(65537), image(40)]
    m.register(edge)
    F = random_pair(1, 1, seed=1)[4]
    pairs = [(2, 0, np.inf), (2, 1, np.inf)]
    for kw in (dict(), dict(accept_single=True, ratio_num=100)):
        a = m.match(pairs, [F] * 2, emit_all=True, **kw)
        b = m.match(pairs, None, form="bruteforce", emit_all=True, **kw)
        for name in ("offset", "n_comparisons", "all_match", "all_d1", "all_d2", "all_count"):
            assert torch.equal(getattr(a, name), getattr(b, name)), name
    m.close()
