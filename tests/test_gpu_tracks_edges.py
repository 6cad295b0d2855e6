"""Triangulation's track list and lane split, and the union's hook, at their
edges.

Sixteen lanes take a track's members and 32,768 groups of lanes the list of
tracks; each workgroup of 1024 nodes claims its stretch of the list.  The sizes
lie around those numbers, and every node may be a root or none.  The reference
is the oracle's least squares; normal equations in float64 differ from it by a
small multiple of eps times the squared condition of A, and by the sums over m
members (2 m rows): 64 m eps cond^2, relative to the point's size."""
import numpy as np
import pytest

from oracle import tracks as tr

pytestmark = pytest.mark.gpu

N_IMAGES = 40


@pytest.fixture(scope="module")
def m():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_06235_amd as sfm
    return sfm.Matcher()


def cameras():
    out = []
    for k in range(N_IMAGES):
        a = 2 * np.pi * k / N_IMAGES
        z = -np.array([np.cos(a), np.sin(a), 0.1])
        z /= np.linalg.norm(z)
        x = np.cross([0, 0, 1.0], z)
        x /= np.linalg.norm(x)
        R = np.stack([x, np.cross(z, x), z])
        out.append(np.hstack([R, (-R @ (-8 * z))[:, None]]))
    return np.stack(out)


def case(sizes, mixed, rng):
    """Labels of tracks of the given sizes (runs, or scattered over all nodes),
    each with noisy observations of one point by distinct cameras."""
    n = int(np.sum(sizes))
    track = np.repeat(np.arange(len(sizes)), sizes)
    image = np.concatenate([rng.permutation(N_IMAGES)[:s] for s in sizes]).astype(np.int32)
    if mixed:
        p = rng.permutation(n)
        track, image = track[p], image[p]
    label = np.full(len(sizes), n)
    np.minimum.at(label, track, np.arange(n))
    P = cameras()
    pts = rng.uniform(-1, 1, (len(sizes), 3))
    h = np.einsum("nij,nj->ni", P[image], np.hstack([pts[track], np.ones((n, 1))]))
    xy = (h[:, :2] / h[:, 2:] + rng.normal(0, 1e-3, (n, 2))).astype(np.float32)
    return label[track].astype(np.int32), image, xy, P


@pytest.mark.parametrize("sizes,mixed", [
    ([1], False), ([2], False), ([1] * 1030, False), ([2] * 513, False), ([40], True),
    ([1, 2, 15, 16, 17, 31, 32, 33, 40], False),
    ([1, 2, 15, 16, 17, 31, 32, 33, 40] * 7, True),
    ([2] * 33_000, True)])
def test_triangulation_sizes(m, sizes, mixed):
    import torch
    import paper_1512_06235_amd as sfm
    label, image, xy, P = case(sizes, mixed, np.random.default_rng(len(sizes)))
    n = label.shape[0]
    X = torch.empty((n, 3), dtype=torch.float64, device="cuda")
    n_obs = torch.empty(n, dtype=torch.int32, device="cuda")
    sfm.sfm_triangulate(m.ctx, torch.as_tensor(label).cuda(), torch.as_tensor(image).cuda(),
                        torch.as_tensor(xy).cuda(), torch.as_tensor(P).cuda(), X, n_obs)
    sfm.sfm_sync(m.ctx)
    X = X.cpu().numpy()
    want, want_n = tr.triangulate(label, image, xy, P)
    assert np.array_equal(n_obs.cpu().numpy(), want_n)
    roots = label == np.arange(n)
    assert np.array_equal(np.isnan(X[roots]), np.isnan(want[roots]))
    for r in np.flatnonzero(want_n >= 2)[:2000]:
        i = np.flatnonzero(label == r)
        p, o = P[image[i]], xy[i].astype(np.float64)
        A = np.concatenate([o[:, :1] * p[:, 2] - p[:, 0], o[:, 1:] * p[:, 2] - p[:, 1]])
        tol = 64 * len(i) * np.finfo(float).eps * np.linalg.cond(A[:, :3]) ** 2
        assert np.linalg.norm(X[r] - want[r]) <= tol * max(1.0, np.linalg.norm(want[r])), r
    big = np.flatnonzero(want_n >= 2)
    assert np.allclose(X[big], want[big], rtol=0, atol=1e-6)


@pytest.mark.parametrize("kind", ["star_low", "star_high", "path", "loops"])
def test_union_shapes(m, kind):
    """Graphs whose hook pass makes one flat tree, one deep one, or nothing."""
    import torch
    import paper_1512_06235_amd as sfm
    n = 5000
    i = np.arange(1, n)
    edges = {"star_low": np.stack([np.zeros_like(i), i], 1),
             "star_high": np.stack([i - 1, np.full_like(i, n - 1)], 1),
             "path": np.stack([i, i - 1], 1),
             "loops": np.stack([i, i], 1)}[kind].astype(np.int32)
    label = torch.empty(n, dtype=torch.int32, device="cuda")
    sfm.sfm_tracks(m.ctx, n, torch.as_tensor(edges).cuda(), label)
    sfm.sfm_sync(m.ctx)
    assert np.array_equal(label.cpu().numpy(), tr.tracks(n, edges))


@pytest.mark.parametrize("n_edges", [1, 2, 255, 256, 257, 1023, 1024, 1025])
def test_few_edges_and_many(m, n_edges):
    """Up to 1,024 edges go to the unions alone, more through hooks first: the
    same labels, whatever the graph and the order of its edges."""
    import torch
    import paper_1512_06235_amd as sfm
    rng = np.random.default_rng(n_edges)
    n = n_edges + 1
    i = np.arange(n_edges)
    relabel = rng.permutation(n)
    chain = np.stack([i, i + 1], 1)
    graphs = {"chain": chain, "chain reversed": chain[::-1], "chain flipped": chain[:, ::-1],
              "edges shuffled": rng.permutation(chain), "nodes shuffled": relabel[chain],
              "star": np.stack([i, np.full(n_edges, n_edges)], 1),
              "chains of nine": np.stack([i, np.where(i % 9 == 8, i, i + 1)], 1),
              "random": rng.integers(0, n, (n_edges, 2))}
    label = torch.empty(n, dtype=torch.int32, device="cuda")
    for what, edges in graphs.items():
        edges = np.ascontiguousarray(edges, np.int32)
        sfm.sfm_tracks(m.ctx, n, torch.as_tensor(edges).cuda(), label)
        sfm.sfm_sync(m.ctx)
        assert np.array_equal(label.cpu().numpy(), tr.tracks(n, edges)), what
    for bad in (-1, n):   # the other edges are still used, the bad one is reported
        edges = np.ascontiguousarray(chain, np.int32)
        edges[n_edges // 2, 1] = bad
        with pytest.raises(sfm.SfmError):
            sfm.sfm_tracks(m.ctx, n, torch.as_tensor(edges).cuda(), label)
            sfm.sfm_sync(m.ctx)
        rest = np.delete(edges, n_edges // 2, 0)
        assert np.array_equal(label.cpu().numpy(), tr.tracks(n, rest))
