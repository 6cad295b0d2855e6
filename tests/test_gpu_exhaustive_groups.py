"""Exhaustive matching keeps a slice's smallest distances by groups of four
consecutive targets and looks into a query's best group afterwards.  Planted
rows put the runner-up, or a copy of the best row, at every distance from the
best one that matters to that: in the same group, in the next one, in another
step, buffer or slice, and in a last group that is not full.  Against the
oracle, bit-exact, with and without per-query outputs."""
import numpy as np
import pytest

from tests.fixtures import random_pair
from tests.test_gpu_exhaustive import run, sfm  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("emit_all", [False, True])
@pytest.mark.parametrize("nb", [2, 4, 5, 63, 1026, 2051])
def test_runner_up_by_group(sfm, oracle_lib, nb, emit_all):
    rng = np.random.default_rng(nb)
    na = 130
    xa, da, xb, db, _ = random_pair(na, nb, seed=40 + nb)
    for i in range(na):
        j = int(rng.integers(0, nb))
        k = (j + int(rng.choice([1, 2, 3, 4, 16, 128, 1024]))) % nb
        if k == j:
            continue
        # db[k] at a distance from the query that passes (or just fails) the
        # ratio test against db[j] taken alone.
        row = db[j].astype(np.int16)
        step = int(rng.integers(0, 4))
        db[k] = np.clip(row + step * rng.integers(-3, 4, 128), 0, 127).astype(np.uint8)
        da[i] = np.clip(db[j].astype(np.int16) + rng.integers(-1, 2, 128), 0, 127).astype(np.uint8)
    n, _ = run(sfm, oracle_lib, [(xa, da), (xb, db)], [(0, 1), (1, 0), (1, 1)], emit_all=emit_all)
    assert n == na + 2 * nb
