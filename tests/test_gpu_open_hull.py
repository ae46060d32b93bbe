"""A mesh whose hull has no subsegments (uploaded as arrays): its hull edges
are boundary edges of a cavity like any other.  A convex polygon of n
rounded-cocircular vertices, triangulated from one of them, has its centre
inside every circumcircle, so an insertion there has a cavity of all n - 2
triangles, bounded by the n hull edges, and gives the star of the new point;
n walks the cavity size across the growth lists' steps of four, the lane
groups' and the engine's limits and the cooperative path.  A square beside it
takes the first round (one insertion a round, the largest triangle first),
which always runs on the grid kernels; the polygon's is the second."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2007_00324_amd import gdp2d
    return gdp2d.Context(0)


def _polygon(n, centre, r):
    a = 0.3 + 2 * np.pi * np.arange(n) / n
    xy = np.asarray(centre) + r * np.stack([np.cos(a), np.sin(a)], axis=1)
    i = np.arange(1, n - 1, dtype=np.int32)
    t = np.arange(n - 2, dtype=np.int32)
    tn = np.stack([t - 1, np.full_like(t, -1), np.where(t + 1 < n - 2, t + 1, -1)], axis=1).astype(np.int32)
    return xy, np.stack([np.zeros_like(i), i, i + 1], axis=1), tn


def _mesh(n):
    """The square (vertices 0 to 3, triangles 0 and 1; its halves larger, its
    quarters smaller than the polygon's largest triangle), then the polygon."""
    xy, tv, tn = _polygon(n, (0.5, 0.5), 0.4)
    d1, d2 = xy[tv[:, 1]] - xy[0], xy[tv[:, 2]] - xy[0]
    area = 0.5 * np.max(d1[:, 0] * d2[:, 1] - d1[:, 1] * d2[:, 0])
    sq, stv, stn = _polygon(4, (3.0, 0.5), np.sqrt(1.4 * area))
    tn = np.vstack([stn, np.where(tn >= 0, tn + 2, -1)]).astype(np.int32)
    none = np.zeros(0, np.int32)
    return {"xy": np.vstack([sq, xy]), "vkind": np.zeros(n + 4, np.int32), "tv": np.vstack([stv, tv + 4]), "tn": tn,
            "ts": np.full_like(tn, -1), "sv": none.reshape(0, 2), "sparent": none, "spend": none.astype(np.uint8)}


def _is_star(tv, tn, p, first, n):
    at = {}
    for t, tri in enumerate(tv):
        if p in tri:
            k = int(np.argmax(tri == p))
            at[int(tri[(k + 1) % 3]) - first] = (t, k, int(tri[(k + 2) % 3]) - first)
    assert sorted(at) == list(range(n)) and all(at[i][2] == (i + 1) % n for i in range(n))
    for i in range(n):
        t, k, _ = at[i]  # the edges from the new point, to it, and the hull's
        assert tn[t, k] == at[(i - 1) % n][0] and tn[t, (k + 2) % 3] == at[(i + 1) % n][0] and tn[t, (k + 1) % 3] == -1


@pytest.mark.parametrize("engine", [False, True], ids=["grid", "engine"])
@pytest.mark.parametrize("n", [3, 4, 5, 6, 7, 8, 9, 10, 11, 18, 40, 41, 42, 43, 50, 51, 52, 66, 67, 68, 131])
def test_hull_edges_bound_cavities(ctx, n, engine):
    from paper_2007_00324_amd import gdp2d
    print(f"[hull] {n} engine={engine}", flush=True)
    m = gdp2d.gdp_mesh_upload(ctx, _mesh(n), n + 4, 0)
    prm = gdp2d.make_params(cand_cap_K=1, max_rounds=2, tail_engine_max=(1 << 30) if engine else -1,
                            profile_kernels=1)
    gdp2d.gdp_mesh_refine(ctx, m, 0.3, prm, allow_noterm=True)
    assert any(k["name"] == "k_engine" and k["launches"] for k in m.kernel_profile()) == engine
    a = m.arrays()
    assert m.info()["rounds"] == 2 and len(a["xy"]) == n + 6 and len(a["tv"]) == n + 4
    assert np.allclose(a["xy"][n + 4:], [[3.0, 0.5], [0.5, 0.5]], rtol=0, atol=1e-12)
    _is_star(np.asarray(a["tv"]), np.asarray(a["tn"]), n + 4, 0, 4)
    _is_star(np.asarray(a["tv"]), np.asarray(a["tn"]), n + 5, 4, n)
