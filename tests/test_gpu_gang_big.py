"""Large cavities of many meshes in shared rounds: the workgroups share out the
queues of 256 meshes at a time, so the meshes with such cavities (polygons of
rounded-cocircular points around their center) are put first, last, alone, in
neighbouring places and past the 256th mesh, among meshes that have none."""
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


@pytest.mark.parametrize("count,places", [(1, [0]), (2, [1]), (7, [0, 6]), (40, [3, 4, 5]), (300, [0, 254, 255, 256, 299])])
def test_queues_shared_out(ctx, count, places):
    from paper_2007_00324_amd import gdp2d
    small = workloads.random_small(5, 40, 2)
    ps = [workloads.scaled_config2(2, 150 + 40 * places.index(q), 4, seed=q, r_lo=0.2, r_hi=0.45) if q in places else small
          for q in range(count)]
    print(f"[gang] {count} meshes, large cavities in {places}", flush=True)
    meshes, st, _ = gdp2d.gdp_refine_batch(ctx, [(p.xy, p.seg) for p in ps], [p.ratio_bound_sq for p in ps],
                                           gdp2d.make_params(batch_engine_max_v=1))
    assert all(s == 0 for s in st)
    ref = {}
    for q, (p, g) in enumerate(zip(ps, meshes)):
        if id(p) not in ref:
            m = gdp2d.gdp_mesh_create(ctx, p.xy, p.seg)
            gdp2d.gdp_mesh_refine(ctx, m, p.ratio_bound_sq, gdp2d.make_params())
            ref[id(p)] = m.arrays()
        assert not diff_arrays(ref[id(p)], g.arrays()), q
        if q in places:
            assert max(k["n_big_cavities"] for k in g.round_stats()) > 0
