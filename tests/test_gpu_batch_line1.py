"""Initial CDTs of a batch built by one workgroup each, at the sizes where such
a build changes (a lane per point and 1,024 threads; a sample of 4,096 points;
every second, third point from 4,097, 8,193 on) and over the layouts that
decide how it goes (cocircular lattices, points in one cell or on one line,
long segments), next to invalid members: every mesh equals the one its input
gives on its own with the host builder.  The points lie in the middle of the
square, outside the sides' lenses, and the bound passes every triangle, so the
initial CDTs come back as they were built (the segments' input is refined)."""
import numpy as np
import pytest

import workloads
from tests.parity_util import diff_arrays
from tests.test_gpu_cdt_rounds import _points

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2007_00324_amd import gdp2d
    return gdp2d.Context(0)


def _invalid():
    sq = workloads.bare_square()
    cross = np.vstack([sq.xy, [[0.25, 0.25], [0.75, 0.75], [0.25, 0.75], [0.75, 0.25]]])
    return [(cross, np.vstack([sq.seg, [[4, 5], [6, 7]]]).astype(np.int32)),
            (np.vstack([sq.xy, [[0.5, 0.5], [0.5, 0.5]]]), sq.seg),                       # duplicate point
            (sq.xy, np.delete(sq.seg, 1, axis=0)),                                        # hull edge without a segment
            (np.vstack([sq.xy, [[0.5, 0.5], [0.25, 0.25], [0.75, 0.75]]]),
             np.vstack([sq.seg, [[5, 6]]]).astype(np.int32))]                             # a vertex on a segment


@pytest.mark.parametrize("kind", ["uniform", "lattice", "one_cell", "line", "segments"])
def test_workgroup_builds_equal_host(ctx, kind):
    from paper_2007_00324_amd import gdp2d
    inputs = []
    for n in [0, 1, 2, 61, 1019, 1020, 1021, 2045, 4091, 4092, 4093, 8189, 12285, 13000]:
        xy = np.vstack([workloads.generators.CORNERS, 0.375 + _points(kind, n).reshape(-1, 2) / 4])
        seg = workloads.generators.BOUNDARY.astype(np.int32)
        if kind == "segments" and n >= 2:
            p = workloads.random_small(9, n, max(1, n // 20))
            xy, seg = p.xy, p.seg
        inputs.append((xy, seg))
    bad = _invalid()
    print(f"[line1] {kind}", flush=True)
    prm = gdp2d.make_params(encroach_mode=1)
    bsq = 2.0 if kind == "segments" else 1e30
    # (a batch of many vertices is built on the device: the inputs eight times)
    many = bad + inputs * 8
    assert sum(len(xy) for xy, _ in many) >= 400000
    meshes, st, _ = gdp2d.gdp_refine_batch(ctx, many, [bsq] * len(many), prm)
    st = list(st)
    # (a refined mesh that outgrows its room is made again on its own, on the host)
    assert kind == "segments" or all(m.info()["cdt_point_rounds"] > 0 for m in meshes[len(bad):])
    assert st[len(bad):] == st[len(bad):len(bad) + len(inputs)] * 8
    assert all(s == -2 for s in st[:len(bad)]) and not any(meshes[:len(bad)])
    for (xy, seg), g, s in zip(inputs, meshes[len(bad):], st[len(bad):]):
        m = gdp2d.gdp_mesh_create(ctx, xy, seg)
        assert s == gdp2d.gdp_mesh_refine(ctx, m, bsq, prm, allow_noterm=True)
        assert kind == "segments" or m.info()["rounds"] == 0
        assert not diff_arrays(m.arrays(), g.arrays()), (kind, len(xy))
    for q, g in enumerate(meshes[len(bad) + len(inputs):]):
        assert not diff_arrays(meshes[len(bad) + q % len(inputs)].arrays(), g.arrays()), (kind, q)
