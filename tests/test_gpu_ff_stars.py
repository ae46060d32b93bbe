"""Flip-Flop removals of points with large links, against the oracle: 16 link
vertices go to a group of lanes, 64 to a wave, more to one thread.  The nested
polygons below have circumcenters near their common center, whose stars have
that many triangles (all of 14 to 68 and some up to 108 between them, closed
and on the hull, of circumcenters and of midpoints)."""
import numpy as np
import pytest

import workloads
from tests.parity_util import COMMON_STATS, gpu_run, oracle_run
from tests.test_oracle_ff import canon

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2007_00324_amd import gdp2d
    return gdp2d.Context(0)


@pytest.mark.parametrize("polygons,n,n_free,seed", [(1, 65, 1, 105), (1, 67, 1, 131), (2, 40, 6, 40), (2, 130, 6, 130),
                                                    (3, 67, 0, 107), (3, 71, 0, 111), (3, 70, 0, 118)])
def test_large_links(ctx, polygons, n, n_free, seed):
    r_lo = {1: 0.3, 2: 0.2, 3: 0.1}[polygons]
    p = workloads.scaled_config2(polygons, n, n_free, seed=seed, r_lo=r_lo, r_hi=0.45)
    print(f"[stars] {p.name} seed={seed}", flush=True)
    om, orc_rc = oracle_run(p, priority_mode=2, insert_mode=1)
    gm, gpu_rc = gpu_run(ctx, p, priority_mode=2, insert_mode=1)
    assert orc_rc == gpu_rc
    a, b = canon(om), canon(gm)
    bad = [k for k in a if not np.array_equal(a[k], b[k])]
    assert not bad, bad
    gs = gm.round_stats()
    assert len(gs) == len(om.stats)
    for r, (s, g) in enumerate(zip(om.stats, gs)):
        d = [f for f in COMMON_STATS + ["n_ff_points", "n_ff_iters"] if s[f] != g[f]]
        assert not d, (r, d)
