"""The grid search's walk along a line, against the oracle bit for bit, where
cells and samples are decided as written instead of from one multiplication:
keypoints on multiples of d / 2, lines along a boundary between cells
(horizontal, vertical, diagonal), samples exactly between two cells (blocks then
step by two), lines in every direction from an epipole inside the image, lists
that overflow their LDS, and cell parameters from 0.75 to 900 px."""
import numpy as np
import pytest

from tests.fixtures import random_pair, translation_F
from tests.test_gpu_grid import _check, sfm  # noqa: F401

pytestmark = pytest.mark.gpu


def _match(sfm, images, pairs, Fs):
    from oracle.grid import grid_match
    m = sfm.Matcher().register(images)
    out = m.match(pairs, Fs, form="grid", emit_all=True)
    _check(out, images, pairs, Fs, grid_match(images, pairs, Fs))
    m.close()


@pytest.mark.parametrize("origin", [0.0, 2.0, 1.0])
@pytest.mark.parametrize("e", [(1.0, 0.0, 0.0), (0.0, 1.0, 0.0), (1.0, 1.0, 0.0),
                               (514.0, 386.0, 1.0)])
def test_lattice_keypoints(sfm, e, origin):
    rng = np.random.default_rng(int(origin) + 10)
    xa, da, xb, db, _ = random_pair(90, 1500, seed=3)
    xa = (rng.integers(0, 200, xa.shape) * 2.0 + origin).astype(np.float32)
    xb = (rng.integers(0, 200, xb.shape) * 2.0 + origin).astype(np.float32)
    xb[:2] = [[origin, origin], [origin + 1020.0, origin + 764.0]]   # the box: whole multiples of 4
    F = translation_F(e)
    _match(sfm, [(xa, da), (xb, db)], [(0, 1, 4.0), (0, 1, 2.0), (1, 0, 8.0)], [F] * 3)


@pytest.mark.parametrize("d", [0.75, 3.3, 40.0, 900.0])
def test_cell_parameters(sfm, d):
    n = 900 if d < 500 else 600
    xa, da, xb, db, F = random_pair(70, n, seed=int(10 * d))
    _match(sfm, [(xa, da), (xb, db)], [(0, 1, d)], [F])


def test_dense_cells(sfm):
    """700 features within a few cells of every line: one chunk's list is longer
    than its LDS, next to queries whose lists are short."""
    rng = np.random.default_rng(4)
    xa, da, xb, db, _ = random_pair(64, 1400, seed=5)
    xa[:, 1] = np.where(np.arange(64) % 3 == 0, 300.0, 20.0 + xa[:, 1] / 4)
    xb[:700, 0] = 500.0 + rng.uniform(0, 9, 700)
    xb[:700, 1] = 300.0 + rng.uniform(-3, 3, 700)
    _match(sfm, [(xa, da), (xb, db)], [(0, 1, 4.0), (0, 1, 16.0)],
           [translation_F((1.0, 0.0, 0.0))] * 2)
