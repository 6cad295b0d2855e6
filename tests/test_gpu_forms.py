"""Which form a guided call takes, the direct or the binned one, shows in the
slots it evaluates: sixteen for every box the direct form opens, 256 for every
step of the binned one.  A recheck margin above half the windows' slack always
takes the binned form, so the same call with one has the slots to compare with
(alike, not equal: the items of a bin or a cell are in no fixed order)."""
import numpy as np
import pytest

from tests.fixtures import random_pair

pytestmark = pytest.mark.gpu

BINNED_MARGIN = 6e-3   # above half of the bin windows' slack of 1e-2 px


@pytest.fixture(scope="module")
def sfm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_06235_amd as sfm
    sfm.lib()
    return sfm


def slots_of(sfm, m, pairs, Fs, **kw):
    out = m.match(pairs, Fs, **kw)
    return out, sfm.sfm_last_stats(m.ctx)["slots"]


def goes_direct(sfm, m, pairs, Fs):
    binned = slots_of(sfm, m, pairs, Fs, recheck_margin_px=BINNED_MARGIN)[1]
    own = slots_of(sfm, m, pairs, Fs)[1]
    return own % 256 != 0 or abs(own - binned) > 0.02 * binned


def test_more_pairs_than_a_launch_has_rows(sfm):
    """70,000 pairs of small images: more than 65,535, which the second and
    third dimension of a launch end at.  Every pair equals the same pair in a
    call of its own few."""
    images, F = [], None
    for k, n in enumerate((50, 41, 16, 1, 0, 33)):
        xy, desc, _, _, F = random_pair(n, 0, seed=500 + k)
        images.append((xy, desc // 16))
    few = [(a, b, 4.0 + a) for a in range(6) for b in range(6)]
    many = [few[k % len(few)] for k in range(70_000)]
    m = sfm.Matcher().register(images)
    assert goes_direct(sfm, m, many, [F] * len(many))
    one = m.match(few, [F] * len(few))
    all_ = m.match(many, [F] * len(many))
    at = np.arange(len(many)) % len(few)
    for name in ("n_comparisons", "n_borderline"):
        a, b = getattr(one, name).cpu().numpy(), getattr(all_, name).cpu().numpy()
        assert np.array_equal(a[at], b), name
    off1, off = one.offset.cpu().numpy(), all_.offset.cpu().numpy()
    assert np.array_equal(np.diff(off), np.diff(off1)[at]) and off1[-1] > 0
    rows = np.concatenate([np.arange(off1[k], off1[k + 1]) for k in at])
    for name in ("query", "match", "d1", "d2"):
        a, b = getattr(one, name).cpu().numpy(), getattr(all_, name).cpu().numpy()
        assert np.array_equal(a[rows], b[:off[-1]]), name
    m.close()


def test_bytes_a_pair_takes(sfm):
    """The workspace of a pair of empty images: descriptor 96, F 72, order 4,
    geometry 184, counters 32, cost 8, 16 padding targets of 16 bytes, two bin
    starts.  (A call at its budget, or at the scratch of the form that does not
    allocate, is refused for a byte more.)"""
    m = sfm.Matcher().register([random_pair(0, 0, seed=1)[:2]])
    few, many = (sfm.sfm_workspace_size(m.ctx, [(0, 0, 4.0)] * n) for n in (4096, 8192))
    assert many - few == 4096 * (96 + 72 + 4 + 184 + 32 + 8 + 16 * 16 + 8)
    m.close()


def test_autotuner_times_its_settings(sfm):
    """The trials of a batch that a call would match directly, or in groups of
    four where the setting says eight, still run as their setting says (the last
    one: eight tiles, sixteen features per bin)."""
    images, F = [], None
    for k, n in enumerate((1500, 16000, 16000)):
        xy, desc, _, _, F = random_pair(n, 0, seed=600 + k)
        images.append((xy, desc))
    m = sfm.Matcher().register(images)
    small, large = [(0, 0, 4.0)], [(1, 2, 2.5)]
    binned = dict(recheck_margin_px=BINNED_MARGIN)

    def tuned(pairs):
        sfm.sfm_autotune(m.ctx, pairs, [F], repeats=1)
        slots = sfm.sfm_last_stats(m.ctx)["slots"]
        sfm.sfm_set_tuning(m.ctx, 8, 16)   # (the winner is any of the six)
        return slots

    assert goes_direct(sfm, m, small, [F])
    got = tuned(small)
    want = slots_of(sfm, m, small, [F], **binned)[1]
    assert got % 256 == 0 and abs(got - want) < 0.05 * want
    # Groups of eight stream more than one buffer here, and round ranges to
    # sixteen instead of four positions.  A call keeps them where the larger table
    # of groups of four does not fit its workspace.
    got = tuned(large)
    fours = slots_of(sfm, m, large, [F], **binned)[1]
    tight = sfm.Matcher(workspace_budget_bytes=sfm.sfm_workspace_size(m.ctx, large)).register(images)
    sfm.sfm_set_tuning(tight.ctx, 8, 16)
    eights = slots_of(sfm, tight, large, [F], **binned)[1]
    assert eights > 1.01 * fours and abs(got - eights) < 0.005 * eights, (fours, eights, got)
    m.close()
    tight.close()


def _strip(n, along, width, seed):
    """Keypoints in a strip of a 1,024 x 768 image, along its middle or a diagonal."""
    rng = np.random.default_rng(seed)
    _, desc, _, _, _ = random_pair(n, 0, seed=seed)
    u, v = rng.uniform(0, 768, n), rng.uniform(-width / 2, width / 2, n)
    xy = {"x": np.stack([u * 4 / 3, 384 + v], 1), "y": np.stack([512 + v, u], 1),
          "diagonal": np.stack([u * 4 / 3 + v, u], 1),
          "antidiagonal": np.stack([1023 - u * 4 / 3 + v, u], 1)}[along]
    xy = np.clip(xy, 0, [1023, 767])
    xy[:4] = [[0, 0], [1023, 0], [0, 767], [1023, 767]]
    return xy.astype(np.float32), desc


LINES = {"x": (1.0, 0.0, 0.0), "y": (0.0, 1.0, 0.0), "diagonal": (4.0, 3.0, 0.0),
         "antidiagonal": (4.0, -3.0, 0.0)}


@pytest.mark.parametrize("along", list(LINES))
def test_crowded_keypoints_are_binned(sfm, along):
    """10,000 features in a strip of 60 px: lines along it have ten times the
    candidates of an even spread's, where the direct form takes twice the binned
    one's time, lines across it no more than an even spread's."""
    from tests.fixtures import translation_F
    across = {"x": "y", "y": "x", "diagonal": "antidiagonal", "antidiagonal": "diagonal"}[along]
    m = sfm.Matcher().register([_strip(10000, along, 60.0, s) for s in (1, 2)])
    pairs = [(0, 1, 4.0)]
    assert not goes_direct(sfm, m, pairs, [translation_F(LINES[along])])
    assert goes_direct(sfm, m, pairs, [translation_F(LINES[across])])
    m.close()


@pytest.mark.parametrize("n, band, direct", [(300, 4.0, True), (8000, 2.0, True), (6000, 8.0, True),
                                             (16000, 2.0, False), (16000, 8.0, False)])
def test_form_of_a_pair(sfm, n, band, direct):
    """A pair of evenly spread features, well to either side of where the two
    forms take as long."""
    images = [random_pair(n, 0, seed=700 + k)[:2] for k in range(2)]
    F = random_pair(1, 1, seed=1)[4]
    m = sfm.Matcher().register(images)
    assert goes_direct(sfm, m, [(0, 1, band)], [F]) == direct
    m.close()


@pytest.mark.parametrize("ext, direct", [(3e4, True), (4e4, False), (6e7, False)])
def test_vast_images_are_binned(sfm, ext, direct):
    """Where the FP32 distance errs by more than the bin windows' slack, the two
    forms would take different slots: boxes of more than 32,768 px are binned."""
    from tests.fixtures import translation_F
    rng = np.random.default_rng(197)
    n = 900
    along = np.array([1.0, 0.3]) / np.hypot(1.0, 0.3)
    xa = rng.uniform(0, ext, (n, 2)).astype(np.float32)
    xb = xa.astype(np.float64) + rng.uniform(-0.3, 0.3, (n, 1)) * ext * along \
        + rng.uniform(-6, 6, (n, 1)) * [-along[1], along[0]]
    xb = np.clip(xb, 0, ext)
    images = [(xa, random_pair(n, 0, seed=11)[1]),
              (xb.astype(np.float32), random_pair(n, 0, seed=12)[1])]
    m = sfm.Matcher().register(images)
    assert goes_direct(sfm, m, [(0, 1, 4.0)], [translation_F((1.0, 0.3, 0.0))]) == direct
    m.close()


EPIPOLES = {"inside": (300.0, 200.0, 1.0), "at infinity": (1.0, 0.3, 0.0), "vertical": (0.0, 1.0, 0.0),
            "just outside": (-40.0, 380.0, 1.0), "far": (5e7, 1e3, 1.0)}


@pytest.mark.parametrize("form", ["direct", "binned"])
@pytest.mark.parametrize("epipole", list(EPIPOLES))
def test_epipoles_in_both_forms(sfm, oracle_lib, epipole, form):
    from tests.fixtures import translation_F
    from tests.gpu_util import compare_all
    xa, da, xb, db, _ = random_pair(1200, 2500, seed=44)
    images = [(xa, da), (xb, db)]
    F = translation_F(EPIPOLES[epipole])
    pairs = [(0, 1, 4.0), (0, 1, 12.0), (1, 0, 2.5)]
    m = sfm.Matcher().register(images)
    assert goes_direct(sfm, m, pairs, [F] * 3)
    kw = dict(recheck_margin_px=BINNED_MARGIN) if form == "binned" else dict()
    out = m.match(pairs, [F] * 3, emit_all=True, **kw)
    compare_all(out, oracle_lib.match(images, pairs, [F] * 3), 3)
    m.close()


@pytest.mark.parametrize("form", ["direct", "binned"])
@pytest.mark.parametrize("na,nb", [(0, 50), (50, 0), (1, 1), (31, 2), (33, 700), (97, 1), (2100, 3000)])
def test_ragged_and_empty_in_both_forms(sfm, oracle_lib, na, nb, form):
    from tests.gpu_util import compare_all
    xa, da, xb, db, F = random_pair(na, nb, seed=na * 7 + nb)
    images = [(xa, da), (xb, db)]
    m = sfm.Matcher().register(images)
    kw = dict(recheck_margin_px=BINNED_MARGIN) if form == "binned" else dict()
    for band in (4.0, 30.0):
        pairs, Fs = [(0, 1, band), (1, 0, band)], [F, F.T]
        if na * nb > 5000 and band < 10.0:
            assert goes_direct(sfm, m, pairs, Fs)
        compare_all(m.match(pairs, Fs, emit_all=True, **kw),
                    oracle_lib.match(images, pairs, Fs), 2)
    m.close()


@pytest.mark.parametrize("nb", [1, 15, 16, 17, 255, 256, 257, 1024, 1025, 4097, 9000])
def test_direct_sizes_around_boxes(sfm, oracle_lib, nb):
    """One box, one outer box, sixteen of them, and one feature to either side."""
    from tests.gpu_util import compare_all
    images = [(xy, desc // 16) for xy, desc in
              (random_pair(n, 0, seed=800 + n)[:2] for n in (1, 3, 63, 130, nb))]
    F = random_pair(1, 1, seed=1)[4]
    pairs = [(k, 4, d) for k in range(4) for d in (0.0, 3.0)] + [(4, 3, 5.0)]
    m = sfm.Matcher().register(images)
    if nb >= 1024:   # (smaller, some opened boxes may happen to be whole steps)
        assert goes_direct(sfm, m, pairs, [F] * len(pairs))
    out = m.match(pairs, [F] * len(pairs), emit_all=True)
    compare_all(out, oracle_lib.match(images, pairs, [F] * len(pairs)), len(pairs))
    m.close()


def test_direct_lists_that_overflow(sfm, oracle_lib):
    """Features exactly on one line and on one point, finer than the strips that
    the choice of the form goes by: lanes with more members than they hold, in
    calls that go direct."""
    from tests.fixtures import translation_F
    from tests.gpu_util import compare_all
    rng = np.random.default_rng(9)
    xa, da, xb, db, _ = random_pair(200, 3000, seed=8)
    db[1500:1700] = db[10]
    xb[:400] = [400.0, 300.0]
    xb[400:900, 1] = 300.0
    xa[:80, 1] = 300.0 + rng.uniform(-0.4, 0.4, 80).astype(np.float32)
    da[:20] = db[10]
    images = [(xa, da), (xb, db)]
    F = translation_F((1.0, 0.0, 0.0))
    m = sfm.Matcher().register(images)
    for pairs in ([(0, 1, 0.25)], [(0, 1, 0.5), (1, 0, 0.25)]):
        assert goes_direct(sfm, m, pairs, [F] * len(pairs))
        out = m.match(pairs, [F] * len(pairs), emit_all=True)
        assert int(out.all_count.max()) >= 900
        compare_all(out, oracle_lib.match(images, pairs, [F] * len(pairs)), len(pairs))
    m.close()


def test_replay_of_a_direct_layout(sfm):
    """A layout that goes direct, captured and replayed with other matrices in
    between, its outputs overwritten before every call and eager work after it."""
    import torch
    images = [random_pair(n, 0, seed=900 + n)[:2] for n in (1500, 1700)]
    F0 = random_pair(1, 1, seed=1)[4]
    turns = [np.array([[1, 0, dx], [0, 1, dy], [0, 0, 1.0]]).T @ F0 for dx, dy in
             ((0, 0), (3, -2), (0, 0), (-7, 5), (11, 4))]
    pairs = [(0, 1, 4.0), (1, 0, 3.0)]
    m = sfm.Matcher().register(images)
    st, opt = torch.cuda.current_stream(), sfm.options(emit_all=True)
    names = ("offset", "n_comparisons", "n_borderline", "all_match", "all_d1", "all_d2", "all_count")
    out, want = m.buffers(pairs, emit_all=True), []

    def call(F):
        for k in names + ("query", "match", "d1", "d2"):
            getattr(out, k).fill_(-7)
        sfm.sfm_guided_match(m.ctx, sfm.PairBatch(pairs, [F, F.T]), None, out, opt, st)
        y = (torch.ones(1 << 16, device="cuda") * 2.0).sum()
        sfm.sfm_sync(m.ctx, st)
        assert y.item() == 2.0 * (1 << 16)
        n = int(out.offset[2])
        return [getattr(out, k).cpu().numpy().copy() for k in names] + \
            [getattr(out, k)[:n].cpu().numpy().copy() for k in ("query", "match", "d1", "d2")]

    for F in turns:
        assert goes_direct(sfm, m, pairs, [F, F.T])
        want.append(call(F))
    assert any(not np.array_equal(a, b) for a, b in zip(want[0], want[1]))
    sfm.sfm_set_graph_replay(m.ctx, True)
    for rep in range(3):
        for F, w in zip(turns, want):
            assert all(np.array_equal(a, b) for a, b in zip(call(F), w)), rep
    sfm.sfm_set_graph_replay(m.ctx, False)
    m.close()
