"""Meshes whose arrays outgrow their first allocation: a mesh of each origin
(host builder, device builder, clone) refined under an edge-length
bound to several times the room it starts with, against the oracle, then once
more as a clone of the refined mesh (nothing left to do)."""
import numpy as np
import pytest

import workloads
from tests.parity_util import diff_arrays, oracle_run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2007_00324_amd import gdp2d
    return gdp2d.Context(0)


@pytest.mark.parametrize("insert_mode", [0, 1], ids=["cavity", "flipflop"])
@pytest.mark.parametrize("origin", ["host", "device", "clone"])
def test_growth_out_of_the_first_allocation(ctx, origin, insert_mode):
    from paper_2007_00324_amd import gdp2d
    p = workloads.random_small(31, 300, 20)
    kw = dict(max_edge_len_sq=0.00025, insert_mode=insert_mode, priority_mode=2 if insert_mode else 0)
    print(f"[growth] {origin} {kw}", flush=True)
    om, rc = oracle_run(p, **kw)
    assert om.arrays()["xy"].shape[0] > 3 * p.xy.shape[0] + 1024
    make = gdp2d.gdp_mesh_create_device if origin == "device" else gdp2d.gdp_mesh_create
    m = make(ctx, p.xy, p.seg)
    if origin == "clone":
        m = m.clone()
    prm = gdp2d.make_params(**kw)
    gdp2d.gdp_mesh_refine(ctx, m, p.ratio_bound_sq, prm)
    c = m.clone()
    gdp2d.gdp_mesh_refine(ctx, c, p.ratio_bound_sq, prm)
    a, b, d = om.arrays(), m.arrays(), c.arrays()
    keys = [k for k in a if isinstance(a[k], np.ndarray)]
    if insert_mode:
        from tests.test_oracle_ff import canon
        assert all(np.array_equal(canon(om)[k], canon(m)[k]) for k in canon(om))
    else:
        assert not diff_arrays(a, b), diff_arrays(a, b)
    assert all(np.array_equal(b[k], d[k]) for k in keys if k in b), "the clone"
