"""The quality kernels at the numbers of workgroups where their sum changes (one
partial, remainders of eight, the most there are), against the oracle: the
count equal, the area within the rounding of a sum of all triangles."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2007_00324_amd import gdp2d
    return gdp2d.Context(0)


@pytest.mark.parametrize("n", [10, 127, 130, 900, 1000, 1030, 1150, 2100, 65000, 66000])
def test_quality_sizes(ctx, n):
    import oracle
    from paper_2007_00324_amd import gdp2d
    p = workloads.random_small(40, n, 1)
    print(f"[quality] {n}", flush=True)
    om = oracle.build_cdt(p.xy, p.seg)
    gm = gdp2d.gdp_mesh_create(ctx, p.xy, p.seg)
    for bsq, l2 in ((0.3, 0.0), (2.0, 0.0), (2.0, 1e-4)):
        n_o, a_o = om.quality(bsq, l2)
        n_g, a_g = gm.quality(bsq, l2)
        assert n_o == n_g
        assert abs(a_o - a_g) <= 1e-10 * max(a_o, 1e-300)
