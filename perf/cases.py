"""The timed work of this framework: what a structure-from-motion program has it do.

Every case builds a seeded synthetic scene on the GPU (cameras that look at a
cloud of points, keypoints with half a pixel of noise, uint8 descriptors with
view noise, distractor features), registers the images once, and times the
calls a program makes on them:

  guided      sfm_guided_match: one pair, a ragged batch, wide bands, per-query
              outputs, and pairs whose epipole lies inside the image
  exhaustive  sfm_bruteforce_match on the same kind of pairs
  coarse      sfm_preemptive_match: staged matching of many pairs
  grid        sfm_grid_match: the grid search in place of the exact band
  candidates  sfm_candidate_images: which pairs to match, from covisibility
  tracks      sfm_tracks and sfm_triangulate on a match graph
  serve       a burst of requests through the serving loop, rows on the host

Image sizes, pairs and bands follow from the case alone, so its work is known;
points, keypoints and descriptors come from the seed.
"""
import math
import random

import numpy as np
import torch

import paper_1512_06235_amd as sfm

DEVICE = "cuda:0"
IMG_W, IMG_H, FOCAL = 1024.0, 768.0, 1000.0
GOLDEN = 0.6180339887498949


def listed():
    return [
        # The smallest call: one pair of 2,000-feature images, as an
        # incremental reconstruction matches its next image.
        guided("pair_2k", images=2, pairs=1, n_lo=2000, n_hi=2000),
        # One pair of large images, on its own.
        guided("pair_16k", images=2, pairs=1, n_lo=16000, n_hi=16000),
        # Forward motion (a vehicle, a walk through a street): the epipole is
        # inside the image, so lines run through it in every direction.
        guided("pair_forward_7k", images=2, pairs=1, n_lo=7001, n_hi=7001, layout="forward"),
        # The ordinary call: all pairs of a 60-camera arc in one batch.
        guided("arc_500_pairs", images=60, pairs=500, n_lo=2000, n_hi=20000),
        # The largest images and widest bands: a launch of the serving loop
        # under load, bands as the pairs' geometry was estimated.
        guided("rings_200_wide", images=64, pairs=200, n_lo=8000, n_hi=40000,
               band_lo=2.0, band_hi=8.0),
        # Small ragged images with every query's nearest two and counts.
        guided("ragged_37_all", images=15, pairs=37, n_lo=301, n_hi=6007,
               band_lo=1.5, band_hi=6.0, emit_all=True),
        # No geometry known yet: every feature against every feature.
        dict(name="exhaustive_16k", kind="exhaustive", layout="arc", images=2, pairs=1,
             n_lo=16000, n_hi=16000),
        # Coarse matching of a whole collection: all pairs of 60 images.
        dict(name="coarse_1770_pairs", kind="coarse", layout="arc", images=60, pairs=1770,
             n_lo=2000, n_hi=20000),
        # The grid search, the approximate alternative to the exact band.
        dict(name="grid_60_pairs", kind="grid", layout="arc", images=24, pairs=60, n_lo=2000,
             n_hi=20000, band_lo=4.0, band_hi=4.0),
        # Which pairs to match: a collection of 1,000 images.
        dict(name="candidates_1000", kind="candidates", images=1000, points=200000, n_lo=4800,
             n_hi=24000, top_k=100),
        # Tracks and points from the matches of the 500-pair batch.
        dict(name="tracks_60_images", kind="tracks", layout="arc", images=60, pairs=500,
             n_lo=2000, n_hi=20000),
        # Requests that arrive together at the serving loop.
        dict(name="serve_burst_8", kind="serve", layout="arc", images=12, pairs=8, n_lo=4000,
             n_hi=25000, band_lo=4.0, band_hi=4.0),
    ]


def guided(name, images, pairs, n_lo, n_hi, layout="arc", band_lo=4.0, band_hi=4.0,
           emit_all=False):
    c = dict(kind="guided", layout=layout, images=images, pairs=pairs, n_lo=n_lo, n_hi=n_hi,
             band_lo=band_lo, band_hi=band_hi, emit_all=emit_all)
    if name:
        c["name"] = name
    return c


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["guided", "guided", "guided", "guided", "exhaustive", "coarse", "grid",
                       "candidates", "tracks", "serve"])
    if kind == "candidates":
        images = _log_int(rng, 40, 1000)
        points = _log_int(rng, 20000, 400000)
        lo = _log_int(rng, 500, 4800)
        return dict(kind=kind, images=images, points=points, n_lo=lo,
                    n_hi=_log_int(rng, lo, 5 * lo), top_k=rng.randrange(10, 120))
    if kind in ("guided", "exhaustive") and rng.random() < 0.45:
        n = _log_int(rng, 300, 20000)
        m = _log_int(rng, max(300, n // 3), min(20000, 3 * n))
        images, pairs, n_lo, n_hi = 2, 1, min(n, m), max(n, m)
    else:
        n_lo = _log_int(rng, 300, 8000)
        n_hi = _log_int(rng, n_lo, min(40000 if kind in ("guided", "tracks") else 20000, 10 * n_lo))
        images = rng.randrange(4, 60)
        most = {"guided": 400, "exhaustive": 24, "coarse": 1770, "grid": 60, "tracks": 500,
                "serve": 12}[kind]
        mean = 0.5 * (n_lo + n_hi)
        if kind in ("guided", "coarse"):
            most = max(8, min(most, int((500 if kind == "guided" else 1770) * (8000 / mean) ** 2)))
        elif kind == "grid":
            most = max(8, min(most, int(60 * 8000 / mean)))
        pairs = max(2, min(_log_int(rng, 2, most), images * (images - 1)))
    c = dict(kind=kind, layout="arc", images=images, pairs=pairs, n_lo=n_lo, n_hi=n_hi)
    if kind in ("guided", "grid", "serve"):
        c["band_lo"] = round(rng.uniform(2.0, 6.0) if kind == "grid" else rng.uniform(1.0, 5.0), 2)
        c["band_hi"] = round(c["band_lo"] + rng.uniform(0.0, 3.0), 2)
    if kind == "guided":
        c["emit_all"] = rng.random() < 0.25
        if pairs == 1 and n_hi <= 10000 and rng.random() < 0.35:
            c["layout"] = "forward"
    return c


# --- what follows from the case alone ---------------------------------------------------------

def _sizes(case):
    """Features per image: n_lo .. n_hi spread over the logarithm, odd ones among them."""
    lo, hi, n = case["n_lo"], case["n_hi"], case["images"]
    if n == 2:
        return [lo, hi]
    return [int(round(lo * (hi / lo) ** ((0.5 + k * GOLDEN) % 1.0))) for k in range(n)]


def _pairs(case):
    """Ordered pairs of images and their bands: neighbours along the arc first."""
    n, want = case["images"], case["pairs"]
    rng = random.Random(1000 * n + want)
    if case["kind"] == "coarse":
        every = [(a, b) for a in range(n) for b in range(a + 1, n)]
    else:
        reach = max(2, math.ceil(n / 6))
        every = [(a, b) for a in range(n) for b in range(n) if a != b and abs(a - b) <= reach]
        if len(every) < want:
            every = [(a, b) for a in range(n) for b in range(n) if a != b]
    chosen = every if len(every) <= want else sorted(rng.sample(every, want))
    if n == 2 and want == 1:
        chosen = [(0, 1)]
    lo, hi = case.get("band_lo", 4.0), case.get("band_hi", 4.0)
    return [(a, b, lo + (hi - lo) * ((k * GOLDEN) % 1.0)) for k, (a, b) in enumerate(chosen)]


def work(case):
    n = _sizes(case)
    if case["kind"] == "candidates":
        true = sum(n)   # observations
        images, words = case["images"], math.ceil(case["points"] / 32)
        # The lists are read and the ranked candidates written; one AND and
        # one popcount per word of every pair of images' point sets.
        return {"bytes": 4.0 * true + 8.0 * images * case["top_k"],
                "flops": images * images / 2 * words * 2.0}
    pairs = _pairs(case)
    used = sorted({i for a, b, _ in pairs for i in (a, b)})
    if case["kind"] == "tracks":
        nodes, edges = sum(n), sum(int(0.35 * min(n[a], n[b])) for a, b, _ in pairs)
        return {"bytes": 8.0 * edges + (4 + 4 + 8 + 4 + 24 + 4) * nodes,
                "flops": 60.0 * nodes}
    queries = sum(n[a] for a, _, _ in pairs)
    if case["kind"] == "coarse":
        whole = lambda x: x < 1000  # noqa: E731
        rows = lambda x: x if whole(x) else 2 * math.ceil(x / 10)  # noqa: E731
        cols = lambda x: x if whole(x) else math.ceil(x / 5)  # noqa: E731
        compared = sum(float(rows(n[a])) * cols(n[b]) for a, b, _ in pairs)
        queries = sum(rows(n[a]) for a, _, _ in pairs)
        read = 132.0 * sum(cols(n[i]) for i in used)
    elif case["kind"] == "exhaustive":
        compared = sum(float(n[a]) * n[b] for a, b, _ in pairs)
        read = 132.0 * sum(n[i] for i in used)
    else:
        # The share of b within d of a line as long as the image is wide.
        compared = sum(float(n[a]) * n[b] * min(1.0, 2.0 * d / IMG_H) for a, b, d in pairs)
        read = 140.0 * sum(n[i] for i in used)
    out = 16.0 * queries if case.get("emit_all") else 0.0
    out += 16.0 * 0.35 * queries   # about a third of the queries are accepted
    return {"bytes": read + out + 24.0 * len(pairs), "flops": 256.0 * compared}


# --- scenes -----------------------------------------------------------------------------------

def _camera(center, target=(0.0, 0.0, 0.0)):
    c = np.asarray(center, dtype=np.float64)
    fwd = np.asarray(target, dtype=np.float64) - c
    fwd /= np.linalg.norm(fwd)
    right = np.cross(fwd, (0.0, 1.0, 0.0))
    right /= np.linalg.norm(right)
    R = np.stack([right, np.cross(fwd, right), fwd])
    return R, -R @ c


def _cameras(case):
    n = case["images"]
    if case.get("layout") == "forward":
        # Towards the scene, half a unit sideways.
        return [_camera((0.0, 0.0, 22.0)), _camera((0.5, 0.2, 18.5), (0.4, 0.15, 0.0))]
    if case["kind"] == "candidates":
        rings = max(1, n // 100)
        out = []
        for k in range(n):
            el = math.radians(-30.0 + 60.0 * ((k % rings) + 0.5) / rings)
            az, r = 2.0 * math.pi * k / n, 18.0 + 8.0 * (k % rings) / rings
            out.append(_camera((r * math.cos(el) * math.sin(az), r * math.sin(el),
                                r * math.cos(el) * math.cos(az))))
        return out
    span = min(180.0, max(15.0, 3.05 * (n - 1)))
    out = []
    for k in range(n):
        az = math.radians(-span / 2 + span * k / (n - 1))
        out.append(_camera((20.0 * math.sin(az), 0.0, 20.0 * math.cos(az))))
    return out


K_MAT = np.array([[FOCAL, 0.0, IMG_W / 2], [0.0, FOCAL, IMG_H / 2], [0.0, 0.0, 1.0]])


def _fundamental(cam_a, cam_b):
    """F with x_b^T F x_a = 0."""
    (Ra, ta), (Rb, tb) = cam_a, cam_b
    R = Rb @ Ra.T
    t = tb - R @ ta
    tx = np.array([[0.0, -t[2], t[1]], [t[2], 0.0, -t[0]], [-t[1], t[0], 0.0]])
    Ki = np.linalg.inv(K_MAT)
    return Ki.T @ tx @ R @ Ki


class _Scene:
    """Points in decreasing order of preference, and each image's view of them."""

    def __init__(self, case, seed, points):
        self.gen = torch.Generator(device=DEVICE).manual_seed(seed)
        self.cams = _cameras(case)
        self.two_view = case["images"] == 2
        f64 = dict(dtype=torch.float64, device=DEVICE, generator=self.gen)
        self.X = torch.rand(points, 3, **f64) * 10.0 - 5.0
        self.normal = torch.randn(points, 3, **f64)
        self.normal /= self.normal.norm(dim=1, keepdim=True)

    def visible(self, k):
        """(ids, pixel coordinates) of the points image k sees, preferred ones first."""
        R, t = (torch.as_tensor(v, dtype=torch.float64, device=DEVICE) for v in self.cams[k])
        Xc = (self.X[:, None, :] * R).sum(dim=2) + t
        xy = FOCAL * Xc[:, :2] / Xc[:, 2:] + torch.tensor([IMG_W / 2, IMG_H / 2],
                                                          dtype=torch.float64, device=DEVICE)
        xy = xy + 0.5 * torch.randn(xy.shape, dtype=torch.float64, device=DEVICE,
                                    generator=self.gen)
        ok = (Xc[:, 2] > 0) & (xy[:, 0] >= 0) & (xy[:, 0] < IMG_W) & (xy[:, 1] >= 0) \
            & (xy[:, 1] < IMG_H)
        if not self.two_view:   # within 75 degrees of the point's normal
            to = torch.as_tensor(-R.T @ t, device=DEVICE) - self.X
            ok &= (to * self.normal).sum(dim=1) >= math.cos(math.radians(75.0)) * to.norm(dim=1)
        ids = ok.nonzero().reshape(-1)
        return ids, xy[ids]

    def base(self, n):
        v = torch.randn(n, 128, device=DEVICE, generator=self.gen).mul_(30.0).abs_().round_()
        return v.clamp_(0, 127).to(torch.int16)

    def view(self, base):
        noise = torch.randint(-6, 7, base.shape, dtype=torch.int16, device=DEVICE,
                              generator=self.gen)
        return (base + noise).clamp_(0, 127).to(torch.uint8)

    def keypoints(self, k, n, true_frac, shuffle=True):
        """(point id or -1, float32 coordinates) of image k's n features; without
        `shuffle` they come preferred ones first, true and distractor features mixed."""
        ids, xy = self.visible(k)
        n_true = min(int(round(true_frac * n)), ids.shape[0])
        away = torch.rand(n - n_true, 2, dtype=torch.float64, device=DEVICE, generator=self.gen)
        away *= torch.tensor([IMG_W, IMG_H], dtype=torch.float64, device=DEVICE)
        gt = torch.cat([ids[:n_true], torch.full((n - n_true,), -1, device=DEVICE)])
        pts = torch.cat([xy[:n_true], away]).to(torch.float32)
        pts[:, 0].clamp_(max=1023.9375)
        pts[:, 1].clamp_(max=767.9375)
        rank = torch.rand(n, device=DEVICE, generator=self.gen)
        if not shuffle:
            rank[:n_true] = rank[:n_true].sort().values
        order = rank.sort(stable=True).indices
        return gt[order], pts[order].contiguous()

    def images(self, case, shuffle=True):
        frac = 0.4 if self.two_view else 0.6
        base = self.base(self.X.shape[0])
        out = []
        for k, n in enumerate(_sizes(case)):
            gt, xy = self.keypoints(k, n, frac, shuffle)
            b = base[gt.clamp(min=0)]
            away = (gt < 0).nonzero().reshape(-1)
            b[away] = self.base(away.shape[0])
            out.append((xy, self.view(b).contiguous()))
        return out


def _scene(case, seed):
    # Two views share a small cloud, so that most of its points are in both.
    points = max(200, int(0.4 * case["n_hi"])) if case["images"] == 2 else 200000
    return _Scene(case, seed, points)


def _buffers(capacity, pairs, emit_all=False):
    out = sfm.MatchBuffers(capacity, pairs, DEVICE, emit_all)
    for t in (out.query, out.match, out.d1, out.d2):
        t.fill_(-1)   # rows past the last match are never written
    return out


# --- one pass ---------------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind}
    if kind == "candidates":
        return _prepare_candidates(case, seed, st)
    if kind == "tracks":
        return _prepare_tracks(case, seed, st)
    scene = _scene(case, seed)
    m = sfm.Matcher(device=0).register(scene.images(case, shuffle=kind != "coarse"))
    pairs = _pairs(case)
    F = [_fundamental(scene.cams[a], scene.cams[b]) for a, b, _ in pairs]
    batch = sfm.PairBatch(pairs, F)
    queries = sum(m.n_features(a) for a, _, _ in pairs)
    emit_all = bool(case.get("emit_all"))
    st.update(m=m, batch=batch, opt=sfm.options(emit_all=emit_all))
    if kind == "serve":
        st["capacity"] = max(m.n_features(k) for k in range(case["images"]))
        # Where the program gathers the rows of its requests: query, match, d1, d2.
        st["rows"] = np.full((len(pairs), 4, st["capacity"]), -1, dtype=np.int32)
        st["counts"] = np.zeros((len(pairs), 2), dtype=np.int64)
        sfm.sfm_server_start(m.ctx, max_batch_pairs=256, max_inflight=2)
    else:
        st["out"] = _buffers(queries, len(pairs), emit_all)
    return st


def _prepare_candidates(case, seed, st):
    scene = _Scene(case, seed, case["points"])
    renumber = torch.randperm(case["points"], device=DEVICE, generator=scene.gen)
    lists = []
    for k, n in enumerate(_sizes(case)):
        ids, _ = scene.visible(k)
        lists.append(renumber[ids[:n]].sort().values.to(torch.int32))
    off = np.zeros(case["images"] + 1, dtype=np.int32)
    off[1:] = np.cumsum([v.shape[0] for v in lists])
    st.update(m=sfm.Matcher(device=0), off=torch.from_numpy(off).to(DEVICE),
              pts=torch.cat(lists), points=case["points"], top_k=case["top_k"],
              out=sfm.CandidateBuffers(case["images"], case["top_k"], DEVICE))
    return st


def _prepare_tracks(case, seed, st):
    scene = _scene(case, seed)
    first, image, xy, node_of = 0, [], [], []
    for k, n in enumerate(_sizes(case)):
        gt, pts = scene.keypoints(k, n, 0.6)
        at = torch.full((scene.X.shape[0],), -1, dtype=torch.int64, device=DEVICE)
        true = (gt >= 0).nonzero().reshape(-1)
        at[gt[true]] = first + true
        node_of.append(at)
        image.append(torch.full((n,), k, dtype=torch.int32, device=DEVICE))
        xy.append(pts)
        first += n
    edges = []
    for a, b, _ in _pairs(case):
        both = ((node_of[a] >= 0) & (node_of[b] >= 0)).nonzero().reshape(-1)
        found = torch.rand(both.shape[0], device=DEVICE, generator=scene.gen) < 0.95
        both = both[found]
        u, v = node_of[a][both], node_of[b][both]
        order = u.sort().indices   # matches come in ascending query order
        edges.append(torch.stack([u[order], v[order]], dim=1))
    P = np.stack([K_MAT @ np.concatenate([R, t[:, None]], axis=1) for R, t in scene.cams])
    # Points are stored per track root only; the other rows keep what they hold.
    st.update(m=sfm.Matcher(device=0), edges=torch.cat(edges).to(torch.int32).contiguous(),
              image=torch.cat(image), xy=torch.cat(xy).contiguous(),
              P=torch.from_numpy(P).to(DEVICE),
              label=torch.empty(first, dtype=torch.int32, device=DEVICE),
              X=torch.full((first, 3), math.nan, dtype=torch.float64, device=DEVICE),
              n_obs=torch.empty(first, dtype=torch.int32, device=DEVICE))
    return st


def run(st):
    kind, m = st["kind"], st["m"]
    if kind == "candidates":
        out = st["out"]
        sfm.sfm_candidate_images(m.ctx, st["off"], st["pts"], st["points"], 8, st["top_k"], out)
        return {"cand": out.cand, "n_shared": out.n_shared, "n_cand": out.n_cand,
                "pairs": out.pairs, "n_pairs": out.n_pairs}
    if kind == "tracks":
        sfm.sfm_tracks(m.ctx, st["label"].shape[0], st["edges"], st["label"])
        sfm.sfm_triangulate(m.ctx, st["label"], st["image"], st["xy"], st["P"], st["X"],
                            st["n_obs"])
        return {"label": st["label"], "X": st["X"], "n_obs": st["n_obs"]}
    if kind == "serve":
        tickets = sfm.sfm_server_submit_batch(m.ctx, st["batch"])
        for k, t in enumerate(tickets):
            r = sfm.sfm_server_poll(m.ctx, int(t), st["capacity"])
            n = r["query"].shape[0]
            for row, key in zip(st["rows"][k], ("query", "match", "d1", "d2")):
                row[:n] = r[key]
            st["counts"][k] = n, r["n_comparisons"]
        return {"rows": st["rows"], "counts": st["counts"]}
    out = st["out"]
    if kind == "coarse":
        stages = sfm.sfm_preemptive_match(m.ctx, st["batch"], out, st["opt"])
        return {"query": out.query, "match": out.match, "d1": out.d1, "d2": out.d2,
                "offset": out.offset, "n_comparisons": out.n_comparisons, "stages": stages}
    call = {"guided": sfm.sfm_guided_match, "exhaustive": sfm.sfm_bruteforce_match,
            "grid": sfm.sfm_grid_match}[kind]
    call(m.ctx, st["batch"], None, out, st["opt"])
    got = {"query": out.query, "match": out.match, "d1": out.d1, "d2": out.d2,
           "offset": out.offset, "n_comparisons": out.n_comparisons,
           "n_borderline": out.n_borderline}
    if out.emit_all:
        got.update(all_match=out.all_match, all_d1=out.all_d1, all_d2=out.all_d2,
                   all_count=out.all_count)
    return got


def exact(case, seed):
    """Every output but the triangulated points is a whole number, equal or wrong."""
    if case["kind"] != "tracks":
        return None
    st = _prepare_tracks(case, seed, {})
    n = st["label"].shape[0]
    u, v = st["edges"].to(torch.int64).unbind(dim=1)
    label = torch.arange(n, device=DEVICE)
    while True:
        low = torch.minimum(label[u], label[v])
        new = label.scatter_reduce(0, u, low, "amin").scatter_reduce(0, v, low, "amin")
        new = new.scatter_reduce(0, label, new, "amin")
        new = new[new]
        if torch.equal(new, label):
            break
        label = new
    P = st["P"][st["image"].to(torch.int64)]
    x = st["xy"].to(torch.float64)
    A = x[:, :, None] * P[:, 2:3, :] - P[:, :2, :]                    # (n, 2, 4)
    G = (A[:, :, :3, None] * A[:, :, None, :]).sum(dim=1)             # (n, 3, 4)
    label, G = label.cpu(), G.cpu()
    M = torch.zeros(n, 3, 4, dtype=torch.float64).index_add_(0, label, G)
    count = torch.zeros(n, dtype=torch.int64).index_add_(0, label, torch.ones(n, dtype=torch.int64))
    X = torch.full((n, 3), math.nan, dtype=torch.float64)
    root = (count >= 2).nonzero().reshape(-1)
    X[root] = torch.linalg.solve(M[root, :, :3], -M[root, :, 3])
    return {"label": None, "X": X, "n_obs": None}
