"""The work that programs have this framework do, as cases to time and compare.

Every case goes through the package's public binding.  Inputs are planar
straight-line graphs (PSLGs) on the unit square, drawn from a seed: a mixture
of uniform points, Gaussian clusters and a jittered ellipse with short
segments between neighbouring points (contour-like data), uniform points with
long segments, or nested closed polygons.  Sizes run from the hundred points
of a batched instance to the million-point graph of the benchmark; bounds are
B^2 in {2, 2.56, 4} and the 20-degree angle bound.

Kinds of work:
  call     PSLG in host memory in, refined mesh in host memory out;
  refine   a resident initial CDT is copied and refined on the device, by
           cavity insertion (cavity), with Chew's lenses, an angle bound and
           an edge-length bound (criteria), or by Flip-Flop insertion (flipflop);
  cdt      the initial CDT built on the device from a PSLG in host memory;
  batch    many independent PSLGs refined in one call;
  serve    a burst of jobs of mixed sizes through the server;
  quality  the bad-triangle count and area of a resident mesh.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2007_00324_amd import gdp2d

CORNERS = np.array([[0.0, 0.0], [1.0, 0.0], [1.0, 1.0], [0.0, 1.0]])
SIDES = np.array([[0, 1], [1, 2], [2, 3], [3, 0]], dtype=np.int32)
CLEAR = 1e-6  # least distance between a segment and the points not on it
BOUNDS_SQ = (2.0, 2.56, 4.0)
THETA20_SQ = 1.0 / (4.0 * math.sin(math.radians(20.0)) ** 2)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _inside(rng, draw, n):
    """n points of draw(k) that keep CLEAR from the square's sides."""
    pts = draw(n)
    while True:
        bad = np.any((pts < CLEAR) | (pts > 1.0 - CLEAR), axis=1)
        if not bad.any():
            return pts
        pts[bad] = draw(int(bad.sum()))


def _mixed_points(rng, n):
    n3 = n // 3
    centres = rng.random((64, 2))
    uni = _inside(rng, lambda k: rng.random((k, 2)), n - 2 * n3)
    clu = _inside(rng, lambda k: centres[rng.integers(0, 64, k)] + rng.normal(0.0, 0.01, (k, 2)), n3)
    t = rng.random(n3) * (2.0 * math.pi)
    ell = np.stack([0.5 + 0.45 * np.cos(t), 0.5 + 0.3 * np.sin(t)], axis=1) + rng.normal(0.0, 1e-4, (n3, 2))
    return np.concatenate([uni, clu, ell])


def _near(a, b, q):
    """Squared distances of the points q[:, k] from the segments a[:], b[:]."""
    d = b - a
    w = q - a[:, None, :]
    t = np.clip((w * d[:, None, :]).sum(2) / (d * d).sum(1)[:, None], 0.0, 1.0)
    r = w - t[:, :, None] * d[:, None, :]
    return (r * r).sum(2)


def _short_segments(rng, pts, m):
    """About m segments between neighbouring points: the points are split into
    boxes of 8 to 16 by alternating medians, and at most one segment is drawn
    per box, so no two meet.  One that passes within CLEAR of another point
    of its box is left out."""
    n = pts.shape[0]
    levels = max(0, int(math.floor(math.log2(max(1.0, n / 8.0)))))
    leaves = 1 << levels
    size = -(-n // leaves)
    idx = np.concatenate([np.arange(n), np.full(leaves * size - n, -1)]).reshape(1, -1)
    ext = np.concatenate([pts, np.full((1, 2), np.inf)])  # entry -1: padding
    for lv in range(levels):
        half = idx.shape[1] // 2
        order = np.argpartition(ext[idx, lv & 1], half - 1, axis=1)
        idx = np.take_along_axis(idx, order, axis=1).reshape(-1, half)
    full = idx[(idx >= 0).all(axis=1)]
    if full.shape[1] < 2 or full.shape[0] == 0:
        return np.zeros((0, 2), np.int64)
    box = full[rng.permutation(full.shape[0])[:m]]
    k = box.shape[0]
    i = rng.integers(0, box.shape[1], k)
    j = (i + rng.integers(1, box.shape[1], k)) % box.shape[1]
    rows = np.arange(k)
    a, b = box[rows, i], box[rows, j]
    d2 = _near(pts[a], pts[b], pts[box])
    d2[rows, i] = np.inf
    d2[rows, j] = np.inf
    ok = d2.min(axis=1) > CLEAR * CLEAR
    return np.stack([a, b], axis=1)[ok]


def _long_segments(rng, pts, m):
    """m segments between random points, without crossings or shared ends."""
    out, used = [], set()
    A = np.zeros((m, 2))
    D = np.zeros((m, 2))
    for _ in range(400 * m):
        if len(out) == m:
            break
        i, j = (int(v) for v in rng.integers(0, pts.shape[0], 2))
        if i == j or i in used or j in used:
            continue
        a, d = pts[i], pts[j] - pts[i]
        k = len(out)
        if k:
            # proper crossing of (a, a + d) with the accepted (A, A + D)
            w = A[:k] - a
            s1 = d[0] * w[:, 1] - d[1] * w[:, 0]
            s2 = s1 + d[0] * D[:k, 1] - d[1] * D[:k, 0]
            u = -(D[:k, 0] * w[:, 1] - D[:k, 1] * w[:, 0])
            v = u + D[:k, 0] * d[1] - D[:k, 1] * d[0]
            if np.any((s1 * s2 <= 0) & (u * v <= 0)):
                continue
        d2 = _near(a[None], (a + d)[None], pts[None])[0]
        d2[[i, j]] = np.inf
        if d2.min() <= CLEAR * CLEAR:
            continue
        A[k], D[k] = a, d
        out.append((i, j))
        used.update((i, j))
    return np.asarray(out, np.int64).reshape(-1, 2)


def _pslg(pts, segs):
    xy = np.ascontiguousarray(np.concatenate([CORNERS, pts]))
    seg = np.ascontiguousarray(np.concatenate([SIDES, segs.astype(np.int32) + 4]).astype(np.int32))
    return xy, seg


def _mixed(rng, n):
    pts = _mixed_points(rng, n)
    return _pslg(pts, _short_segments(rng, pts, max(1, round(0.05 * n))))


def _uniform(rng, n, long_segments=False):
    pts = _inside(rng, lambda k: rng.random((k, 2)), n)
    m = max(1, round(0.05 * n))
    return _pslg(pts, _long_segments(rng, pts, m) if long_segments else _short_segments(rng, pts, m))


def _circles(rng, n_circles, per, n_free):
    """Nested regular polygons about the centre, and uniform free points that
    keep clear of them."""
    lo, hi, gap = 0.01, 0.49, 1e-4
    r = lo + np.sort(rng.random(n_circles)) * (hi - lo - (n_circles - 1) * gap) + gap * np.arange(n_circles)
    j = np.arange(per)
    ang = rng.random(n_circles)[:, None] * (2.0 * math.pi) + j[None] * (2.0 * math.pi / per)
    poly = np.stack([0.5 + r[:, None] * np.cos(ang), 0.5 + r[:, None] * np.sin(ang)], axis=2).reshape(-1, 2)
    base = (np.arange(n_circles) * per)[:, None]
    segs = np.stack([base + j, base + (j + 1) % per], axis=2).reshape(-1, 2)
    sag = r * (1.0 - math.cos(math.pi / per))

    def draw(k):
        q = rng.random((k, 2))
        while True:
            rho = np.hypot(q[:, 0] - 0.5, q[:, 1] - 0.5)
            c = np.clip(np.searchsorted(r, rho - 2 * CLEAR), 0, n_circles - 1)
            bad = (rho > r[c] - sag[c] - 2 * CLEAR) & (rho < r[c] + 2 * CLEAR)
            if not bad.any():
                return q
            q[bad] = rng.random((int(bad.sum()), 2))

    return _pslg(np.concatenate([poly, _inside(rng, draw, n_free)]), segs)


def _sizes(count, lo, hi):
    """count sizes spread evenly over the logarithm of [lo, hi], hi among them."""
    k = np.arange(1, count + 1) / count
    return [int(lo * (hi / lo) ** v) for v in k]


def _grid_mesh(rng, g):
    """A jittered g x g point grid with every cell cut along one diagonal, as
    mesh arrays (no subsegments): elongated where the jitter is large."""
    step = 1.0 / (g - 1)
    ii, jj = np.meshgrid(np.arange(g), np.arange(g), indexing="ij")
    xy = np.stack([ii, jj], axis=2).reshape(-1, 2) * step
    xy = xy + rng.uniform(-0.3, 0.3, xy.shape) * step
    c = g - 1
    i, j = (v.reshape(-1) for v in np.meshgrid(np.arange(c), np.arange(c), indexing="ij"))
    v00, v10, v11, v01 = i * g + j, (i + 1) * g + j, (i + 1) * g + j + 1, i * g + j + 1
    cell = i * c + j
    lower, upper = 2 * cell, 2 * cell + 1
    tv = np.empty((2 * c * c, 3), np.int32)
    tn = np.empty((2 * c * c, 3), np.int32)
    tv[0::2] = np.stack([v00, v10, v11], axis=1)
    tv[1::2] = np.stack([v00, v11, v01], axis=1)
    tn[0::2] = np.stack([np.where(j > 0, lower - 1, -1), np.where(i + 1 < c, lower + 2 * c + 1, -1), upper], axis=1)
    tn[1::2] = np.stack([lower, np.where(j + 1 < c, lower + 2, -1), np.where(i > 0, upper - 2 * c - 1, -1)], axis=1)
    return xy, tv, tn


def _case_pslg(case, seed):
    rng = np.random.default_rng(seed)
    data = case["data"]
    if data == "circles":
        return _circles(rng, case["circles"], case["per"], case["free"])
    if data == "uniform":
        return _uniform(rng, case["n"], long_segments=True)
    return _mixed(rng, case["n"])


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # a small interactive request: 1,000 uniform points, 50 long segments
        {"name": "call_1k", "kind": "call", "data": "uniform", "n": 1000, "bsq": 2.0},
        # a small resident mesh refined again and again (latency of a round)
        {"name": "refine_5k", "kind": "cavity", "data": "mixed", "n": 5003, "bsq": 2.56},
        # an ordinary mesh, the middle of the serving range
        {"name": "refine_50k", "kind": "cavity", "data": "mixed", "n": 50021, "bsq": 2.0},
        # the benchmark's workload
        {"name": "refine_1m", "kind": "cavity", "data": "mixed", "n": 1000000, "bsq": 2.0},
        # boundary-dominated input: nested contours, large cocircular cavities
        {"name": "refine_circles", "kind": "cavity", "data": "circles", "circles": 512, "per": 1000, "free": 100000,
         "bsq": 2.0},
        # a finite-element mesh: lenses, 20-degree angle bound and a maximal edge length
        {"name": "criteria_200k", "kind": "criteria", "data": "mixed", "n": 200003, "bsq": THETA20_SQ, "len": 1.0},
        # the paper's own insertion, Flip-Flop
        {"name": "flipflop_30k", "kind": "flipflop", "data": "mixed", "n": 30011, "bsq": 2.0},
        # initial CDT on the device: a serving job's size, and the benchmark's
        {"name": "cdt_60k", "kind": "cdt", "data": "mixed", "n": 60013, "bsq": 2.0},
        {"name": "cdt_1m", "kind": "cdt", "data": "mixed", "n": 1000000, "bsq": 2.0},
        # many small meshes in one call
        {"name": "batch_128", "kind": "batch", "count": 128, "lo": 100, "hi": 50000},
        # a burst of jobs of mixed sizes through the server
        {"name": "serve_16", "kind": "serve", "count": 16, "lo": 1000, "hi": 200000},
        # checking a million-vertex mesh
        {"name": "quality_1m", "kind": "quality", "grid": 1000, "bsq": 2.0},
    ]


def draw(rng):
    def size(lo, hi):
        return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))

    kind = rng.choice(["call", "cavity", "cavity", "cavity", "circles", "criteria", "flipflop", "cdt", "cdt", "batch",
                       "serve", "quality"])
    bsq = rng.choice(BOUNDS_SQ)
    if kind == "call":
        n = size(100, 3000)
        return {"kind": "call", "data": "uniform" if n < 1500 else "mixed", "n": n, "bsq": bsq}
    if kind == "circles":
        c, per = rng.randint(16, 300), rng.randint(300, 1000)
        return {"kind": "cavity", "data": "circles", "circles": c, "per": per, "free": size(100, 100000), "bsq": bsq}
    if kind == "batch":
        return {"kind": "batch", "count": rng.randint(16, 128), "lo": 100, "hi": size(5000, 50000)}
    if kind == "serve":
        return {"kind": "serve", "count": rng.randint(4, 16), "lo": 1000, "hi": size(20000, 200000)}
    if kind == "quality":
        return {"kind": "quality", "grid": rng.randint(100, 1000), "bsq": bsq}
    if kind == "criteria":
        return {"kind": "criteria", "data": "mixed", "n": size(1000, 200000), "bsq": rng.choice([2.0, THETA20_SQ]),
                "len": round(rng.uniform(0.8, 2.0), 3)}
    top = {"cavity": 1000000, "flipflop": 30000, "cdt": 1000000}[kind]
    return {"kind": kind, "data": "mixed", "n": size(1000, top), "bsq": bsq}


def _params(case):
    if case["kind"] == "criteria":
        # the edge-length bound is case["len"] mean point spacings
        return gdp2d.make_params(encroach_mode=1, max_edge_len_sq=case["len"] ** 2 / case["n"])
    if case["kind"] == "flipflop":
        return gdp2d.make_params(priority_mode=2, insert_mode=1)
    return gdp2d.make_params()


def prepare(case, seed):
    ctx = gdp2d.Context(0)
    kind = case["kind"]
    s = {"kind": kind, "ctx": ctx, "bsq": case.get("bsq")}
    if kind in ("call", "cdt"):
        s["xy"], s["seg"] = _case_pslg(case, seed)
    elif kind in ("cavity", "criteria", "flipflop"):
        xy, seg = _case_pslg(case, seed)
        s["init"] = gdp2d.gdp_mesh_create_device(ctx, xy, seg)
        s["work"] = s["init"].clone()
        s["params"] = _params(case)
    elif kind in ("batch", "serve"):
        rng = np.random.default_rng(seed)
        sizes = rng.permutation(_sizes(case["count"], case["lo"], case["hi"]))
        make = _uniform if kind == "batch" else _mixed
        s["inputs"] = [make(rng, int(n)) for n in sizes]
        s["bounds"] = [float(b) for b in rng.choice(BOUNDS_SQ, case["count"])]
        if kind == "serve":
            s["server"] = gdp2d.Server(ctx, 12 << 30, 64, line1=(16, 100000))
    if kind == "call":
        V, S = _room(case)
        i32 = np.int32
        s["out"] = {"xy": np.zeros((V, 2)), "vkind": np.zeros(V, i32), "tv": np.zeros((2 * V, 3), i32),
                    "tn": np.zeros((2 * V, 3), i32), "ts": np.zeros((2 * V, 3), i32), "sv": np.zeros((S, 2), i32),
                    "sparent": np.zeros(S, i32), "spend": np.zeros(S, np.uint8)}
    elif kind != "quality":
        s["out"] = _buffers(case)
    else:
        rng = np.random.default_rng(seed)
        xy, tv, tn = _grid_mesh(rng, case["grid"])
        arrays = {"xy": xy, "vkind": np.zeros(len(xy), np.int32), "tv": tv, "tn": tn, "ts": np.full_like(tn, -1),
                  "sv": np.zeros((0, 2), np.int32), "sparent": np.zeros(0, np.int32), "spend": np.zeros(0, np.uint8)}
        s["mesh"] = gdp2d.gdp_mesh_upload(ctx, arrays, len(xy), 0)
    return s


def _room(case):
    """Vertices and subsegments that a case's results are given room for: above
    what its inputs refine to, and the same for every input of the case."""
    kind = case["kind"]
    if kind == "call":
        return 12 * case["n"] + 1000, 4 * case["n"] + 1000
    if kind in ("batch", "serve"):
        n = sum(_sizes(case["count"], case["lo"], case["hi"]))
        return 5 * n + 1000, n + 1000
    if case["data"] == "circles":
        n = case["circles"] * case["per"] + case["free"]
        return 8 * n + 1000, 6 * n + 1000
    n = case["n"]
    if kind == "cdt":
        return n + 4, n // 10 + 100
    return (8 if kind == "criteria" else 5) * n + 1000, n + 1000


def _buffers(case):
    """A program's own buffers for the results (they are copied there, so that
    the library's meshes can be freed or refined again)."""
    V, S = _room(case)
    T = 2 * V
    i32 = {"dtype": torch.int32, "device": "cuda"}
    out = {"xy": torch.zeros((V, 2), dtype=torch.float64, device="cuda"), "tri": torch.zeros((T, 4), **i32),
           "sub_v": torch.zeros((S, 2), **i32), "sub_parent": torch.zeros(S, **i32)}
    if case["kind"] not in ("batch", "serve"):
        out.update(vkind=torch.zeros(V, **i32), sub_pending=torch.zeros(S, **i32))
        if case["kind"] != "flipflop":
            out.update(nbr=torch.zeros((T, 4), **i32), sub_on_edge=torch.zeros((T, 4), **i32))
    return out


def _keep(s, mesh, order_tri=False):
    views = mesh.device_views()
    if order_tri:
        # the triangles in the order of their first directed edge: the slots
        # that flips leave them in are not part of the result
        t = views["tri"]
        views["tri"] = t[torch.argsort(t[:, 0].long() << 32 | t[:, 1].long())]
    for k, b in s["out"].items():
        b[:views[k].shape[0]] = views[k]
    info = mesh.info()
    return dict(s["out"], counts=[info["n_vertices"], info["n_triangles"], info["n_subsegments"]])


def _keep_all(s, meshes):
    views = [m.device_views() for m in meshes]
    for k, b in s["out"].items():
        parts = [v[k] for v in views]
        torch.cat(parts, out=b[:sum(p.shape[0] for p in parts)])
    info = [m.info() for m in meshes]
    counts = np.array([[i["n_vertices"], i["n_triangles"], i["n_subsegments"]] for i in info])
    return dict(s["out"], counts=counts)


def run(s):
    kind, ctx = s["kind"], s["ctx"]
    if kind == "call":
        a = gdp2d.gdp_refine(ctx, s["xy"], s["seg"], s["bsq"]).arrays()
        for k, b in s["out"].items():
            b[:a[k].shape[0]] = a[k]
        return dict(s["out"], counts=[len(a["xy"]), len(a["tv"]), len(a["sv"])])
    if kind in ("cavity", "criteria", "flipflop"):
        s["work"].assign_from(s["init"])
        gdp2d.gdp_mesh_refine(ctx, s["work"], s["bsq"], s["params"])
        return _keep(s, s["work"], order_tri=kind == "flipflop")
    if kind == "cdt":
        return _keep(s, gdp2d.gdp_mesh_create_device(ctx, s["xy"], s["seg"]))
    if kind == "batch":
        meshes, status, _ = gdp2d.gdp_refine_batch(ctx, s["inputs"], s["bounds"])
        return dict(_keep_all(s, meshes), status=np.asarray(status))
    if kind == "serve":
        srv = s["server"]
        jobs = [srv.submit(xy, seg, b) for (xy, seg), b in zip(s["inputs"], s["bounds"])]
        return _keep_all(s, [srv.wait(j)[0] for j in jobs])
    n, area = s["mesh"].quality(s["bsq"])
    return {"n_bad": n, "bad_area": area}


# Refined vertices per input vertex, about (B^2 = 2 on the mixed input; the
# other bounds give fewer, an edge-length bound of one spacing more).
GROWTH = {2.0: 2.3, 2.56: 1.9, 4.0: 1.5}


def work(case):
    """Each input read and each output written once: a vertex 20 bytes, and
    two triangle records of 48 per vertex; one circle test (about 30
    operations) per edge of the result."""
    kind = case["kind"]
    if kind == "quality":
        n = case["grid"] ** 2
        return {"bytes": 48.0 * n, "flops": 2 * 40.0 * n}
    if kind in ("batch", "serve"):
        n_in = float(sum(_sizes(case["count"], case["lo"], case["hi"])))
        growth = 1.9
    else:
        n_in = case["circles"] * case["per"] + case["free"] if case.get("data") == "circles" else case["n"]
        growth = 1.0 if kind == "cdt" else GROWTH.get(case["bsq"], 2.2)
        if kind == "criteria":
            growth = max(growth, 1.0 + 2.0 / case["len"] ** 2)
    read = 16.0 if kind in ("call", "cdt", "batch", "serve") else 116.0
    return {"bytes": n_in * (read + 116.0 * growth), "flops": 90.0 * n_in * growth}


def exact(case, seed):
    """The vertices of an initial CDT are its input; the quality of the grid
    mesh follows from its arrays.  A refined mesh has no value apart from the
    refinement's own rules."""
    if case["kind"] == "cdt":
        return dict.fromkeys(("tri", "sub_v", "sub_parent", "vkind", "sub_pending", "nbr", "sub_on_edge", "counts"),
                             None) | {"xy": _case_pslg(case, seed)[0]}
    if case["kind"] == "quality":
        xy, tv, _ = _grid_mesh(np.random.default_rng(seed), case["grid"])
        a, b, c = xy[tv[:, 0]], xy[tv[:, 1]], xy[tv[:, 2]]
        ab, ac, bc = b - a, c - a, c - b
        d = ab[:, 0] * ac[:, 1] - ab[:, 1] * ac[:, 0]
        sides = np.stack([(v * v).sum(1) for v in (ab, ac, bc)])
        # circumradius^2 = (product of the squared sides) / (4 d^2)
        bad = (d <= 0) | (sides.prod(axis=0) > case["bsq"] * sides.min(axis=0) * 4.0 * d * d)
        return {"n_bad": None, "bad_area": math.fsum((0.5 * d[bad]).tolist())}
    return None
