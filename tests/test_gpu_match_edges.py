"""The binned match kernel where its buffers, steps and groups end.

A fill of the buffer holds 256 (or 128) targets; a tile's 16-target steps start
at its range's 4-target group, moved back where they would overrun the fill,
or on multiples of 16 when the range takes several fills.  Sizes lie around
those numbers, bands range from empty to everything, and the outputs are
integers: they equal the oracle's.  (A wide recheck margin keeps every pair in
the binned form.)"""
import numpy as np
import pytest

import scenes
from tests.fixtures import random_pair
from tests.gpu_util import compare_all, compare_rows

pytestmark = pytest.mark.gpu

TARGETS = [1, 15, 16, 17, 127, 129, 255, 256, 257, 271, 300, 1030, 2100]
QUERIES = [0, 1, 16, 17, 63, 65, 128, 129, 300]


@pytest.fixture(scope="module")
def sfm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_06235_amd as sfm
    sfm.lib()
    return sfm


@pytest.mark.parametrize("tiles", [4, 8])
@pytest.mark.parametrize("emit_all", [False, True])
def test_sizes_around_fills(sfm, oracle_lib, tiles, emit_all):
    images = []
    for k, n in enumerate(QUERIES + TARGETS):
        xy, desc, _, _, _ = random_pair(n, 0, seed=200 + k)
        images.append((xy, desc // 8))
    F = scenes.make_two_view_2k().F
    nq = len(QUERIES)
    pairs = [(q, nq + t, d) for q in range(nq) for t in range(len(TARGETS))
             for d in ((0.5, 12.0, 90.0, np.inf) if t % 2 else (3.0, 40.0, 250.0))]
    if tiles == 8:
        pairs = 3 * pairs   # fewer groups would be cut into fours
    m = sfm.Matcher().register(images)
    sfm.sfm_set_tuning(m.ctx, tiles, 8)
    assert tiles == 4 or sum(-(-images[a][0].shape[0] // 128) for a, _, _ in pairs) > 1024
    want = oracle_lib.match(images, pairs, [F] * len(pairs))
    out = m.match(pairs, [F] * len(pairs), emit_all=emit_all, recheck_margin_px=6e-3)
    compare_all(out, want, len(pairs))
    m.close()


@pytest.mark.parametrize("n_pairs", [3, 130])
@pytest.mark.parametrize("largest", [27000, 54000])
def test_sides_around_the_sort_in_lds(sfm, oracle_lib, n_pairs, largest):
    """Sides that sort through 64 KB of LDS, through 128 KB and not in LDS, in
    batches of few and of many pairs."""
    images = []
    for k, n in enumerate([largest, 25000, 40]):
        xy, desc, _, _, _ = random_pair(n, 0, seed=300 + k)
        images.append((xy, desc))
    F = scenes.make_two_view_2k().F
    pairs = ([(2, 0, 2.0), (1, 2, 3.0), (2, 1, 0.5)] + [(2, 2, 4.0)] * n_pairs)[:n_pairs]
    pairs[-1] = (0, 2, 3.0)
    m = sfm.Matcher().register(images)
    out = m.match(pairs, [F] * n_pairs, emit_all=True, recheck_margin_px=6e-3)
    compare_all(out, oracle_lib.match(images, pairs, [F] * n_pairs), n_pairs)
    m.close()


@pytest.mark.parametrize("reps", [15, 62])
def test_many_small_pairs(sfm, oracle_lib, reps):
    """15: 720 pairs in one fused emission of narrow workgroups.  62: 2,976, whose
    4,464 groups are more than take a workgroup each, so resident ones draw them
    from the shares' counters."""
    images = []
    for k, n in enumerate([300, 65, 17, 1, 16, 129, 257, 300]):
        xy, desc, _, _, _ = random_pair(n, 0, seed=400 + k)
        images.append((xy, desc // 8))
    F = scenes.make_two_view_2k().F
    pairs = [(q, t, d) for q in range(4) for t in range(4, 8) for d in (0.5, 20.0, np.inf)]
    groups = reps * sum(-(-images[a][0].shape[0] // 128) for a, _, _ in pairs)
    assert (groups > 4096) == (reps == 62)
    want = oracle_lib.match(images, pairs, [F] * len(pairs))
    m = sfm.Matcher().register(images)
    out = m.match(pairs * reps, [F] * (len(pairs) * reps), recheck_margin_px=6e-3)
    for p in range(len(pairs) * reps):
        compare_rows(*out.pair(p), want.pair(p % len(pairs)), what=f"pair {p}: ")
    got = out.n_comparisons[:len(pairs) * reps].cpu().numpy().reshape(reps, -1)
    assert np.array_equal(got, np.tile(want.n_comparisons[:len(pairs)], (reps, 1)))
    m.close()
