"""Guided matching of few pairs runs without preparation (the direct form), of
many or large pairs through the binned one; which of the two depends on the
call's sizes, bands and epipoles alone and must not show.  The same pairs, alone
(direct) and behind a large pair (binned), give every output bit for bit, the
borderline counts among them; and at the sizes where the direct form's boxes,
lists and lanes end, every query equals the oracle's."""
import numpy as np
import pytest

import scenes
from tests.fixtures import random_pair, translation_F
from tests.gpu_util import compare_all

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sfm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_06235_amd as sfm
    sfm.lib()
    return sfm


def _image(n, seed, coarse=False):
    xy, desc, _, _, _ = random_pair(n, 0, seed=seed)
    return xy, desc // 16 if coarse else desc


EPIPOLES = {"side": None, "inside": (512.3, 384.2, 1.0), "edge": (1023.0, 100.0, 1.0),
            "far": (1.0, 0.2, 0.0)}


@pytest.mark.parametrize("epipole", list(EPIPOLES))
def test_direct_equals_binned(sfm, epipole):
    """Alone and behind a pair too large to be matched directly."""
    e = EPIPOLES[epipole]
    F = scenes.make_two_view_2k().F if e is None else translation_F(e)
    images = [_image(n, 60 + k, coarse=k == 2) for k, n in enumerate([900, 2500, 1300, 33, 30000])]
    pairs = [(0, 1, 4.0), (1, 0, 1.5), (1, 2, 7.0), (2, 2, 3.0), (3, 1, 4.0), (1, 3, 60.0),
             (0, 2, 0.0)]
    big = (4, 4, 8.0)
    m = sfm.Matcher().register(images)
    for kw in (dict(), dict(recheck_margin_px=0.0), dict(accept_single=True, ratio_num=99)):
        alone = m.match(pairs, [F] * len(pairs), emit_all=True, **kw)
        both = m.match(pairs + [big], [F] * len(pairs) + [scenes.make_two_view_2k().F],
                       emit_all=True, **kw)
        slots = sfm.sfm_last_stats(m.ctx)["slots"]
        n = sum(images[a][0].shape[0] for a, _, _ in pairs)
        rows = int(alone.offset[len(pairs)])
        for name in ("offset", "n_comparisons", "n_borderline"):
            k = len(pairs) + (name == "offset")
            assert np.array_equal(getattr(alone, name)[:k].cpu(), getattr(both, name)[:k].cpu()), name
        for name in ("query", "match", "d1", "d2"):
            assert np.array_equal(getattr(alone, name)[:rows].cpu(),
                                  getattr(both, name)[:rows].cpu()), name
        for name in ("all_match", "all_d1", "all_d2", "all_count"):
            assert np.array_equal(getattr(alone, name)[:n].cpu(), getattr(both, name)[:n].cpu()), name
        assert slots > 0
    m.close()


@pytest.mark.parametrize("nb", [1, 15, 16, 17, 255, 256, 257, 1024, 1025, 4097])
def test_sizes_around_boxes(sfm, oracle_lib, nb):
    images = [_image(n, 70 + n, coarse=True) for n in (0, 1, 3, 63, 130)] + [_image(nb, nb, True)]
    F = scenes.make_two_view_2k().F
    pairs = [(k, 5, d) for k in range(5) for d in (0.0, 3.0, np.inf)] + [(5, 4, 5.0), (5, 0, 5.0)]
    m = sfm.Matcher().register(images)
    for form in ("batched", "plain", "noalloc"):
        out = m.match(pairs, [F] * len(pairs), form=form, emit_all=True)
        compare_all(out, oracle_lib.match(images, pairs, [F] * len(pairs)), len(pairs))
    m.close()


def test_crowded_boxes_and_lists(sfm, oracle_lib):
    """Many features at the same place or on one line: lanes that keep more
    members than they hold, boxes of no extent, and a band that crosses them all."""
    rng = np.random.default_rng(9)
    xa, da, xb, db, _ = random_pair(200, 3000, seed=8)
    db[1500:1700] = db[10]
    xb[:900] = [400.0, 300.0]
    xb[900:2000, 1] = 300.0
    xa[:80, 1] = 300.0 + rng.uniform(-6, 6, 80).astype(np.float32)
    da[:20] = db[10]
    images = [(xa, da), (xb, db)]
    F = translation_F((1.0, 0.0, 0.0))
    pairs = [(0, 1, 4.0), (0, 1, 0.25), (0, 1, 500.0), (1, 0, 4.0)]
    m = sfm.Matcher().register(images)
    out = m.match(pairs, [F] * 4, emit_all=True)
    compare_all(out, oracle_lib.match(images, pairs, [F] * 4), 4)
    m.close()
