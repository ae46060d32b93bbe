"""Points that coincide above the sizes up to which the device CDT builder
takes every point into its first step (4,096 points; every second one from
4,097 on, every third from 8,193 on): as many copies as put two of them into
that sample, pairs that do not, and one place for most of the points, by the
builder for one mesh and by the workgroup builds of a batch.  Each is
GDP_E_INPUT, and the device's memory is as it was: a valid input afterwards,
and one among them in the batch, gives the host builder's mesh."""
import numpy as np
import pytest

import workloads
from tests.parity_util import diff_arrays

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2007_00324_amd import gdp2d
    return gdp2d.Context(0)


def _input(n, copies, places):
    """The square and n inner points, of which `places` have `copies` copies."""
    rng = np.random.default_rng(n + copies)
    pts = 0.375 + rng.uniform(size=(n, 2)) / 4
    for k in range(places):
        pts[k * copies:(k + 1) * copies] = pts[k * copies]
    xy = np.vstack([workloads.generators.CORNERS, pts[rng.permutation(n)]])
    return xy, workloads.generators.BOUNDARY.astype(np.int32)


CASES = [(n, copies, places) for n in (4092, 4093, 8189, 20000)
         for copies, places in ((2, 1), (2, 400), (3, 1), (3, 400), (7, 100), (n, 1))]


@pytest.mark.parametrize("n,copies,places", CASES)
def test_builder_rejects_repeated_points(ctx, n, copies, places):
    from paper_2007_00324_amd import gdp2d
    xy, seg = _input(n, copies, places)
    print(f"[repeated] {n} x{copies} at {places}", flush=True)
    with pytest.raises(gdp2d.GdpError) as e:
        gdp2d.gdp_mesh_create_device(ctx, xy, seg)
    assert e.value.code == -2, e.value
    xy, seg = _input(n, 1, 0)
    dev = gdp2d.gdp_mesh_create_device(ctx, xy, seg).arrays()
    assert not diff_arrays(gdp2d.gdp_mesh_create(ctx, xy, seg).arrays(), dev)


def test_batch_rejects_repeated_points(ctx):
    from paper_2007_00324_amd import gdp2d
    bad = [_input(*c) for c in CASES] * 2
    good = [_input(n, 1, 0) for n in (4092, 4093, 8189, 20000)]
    inputs = bad[:30] + good + bad[30:]
    assert sum(len(xy) for xy, _ in inputs) >= 400000  # (built by workgroups from here on)
    print(f"[repeated] batch of {len(inputs)}", flush=True)
    prm = gdp2d.make_params(encroach_mode=1)
    meshes, st, _ = gdp2d.gdp_refine_batch(ctx, inputs, [1e30] * len(inputs), prm)
    assert [int(s) for s in st] == [-2] * 30 + [0] * len(good) + [-2] * (len(bad) - 30)
    for (xy, seg), m in zip(good, meshes[30:]):
        assert not diff_arrays(gdp2d.gdp_mesh_create(ctx, xy, seg).arrays(), m.arrays())
