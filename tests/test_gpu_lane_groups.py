"""Cavities and fans at the limits of the lane groups that grow and insert
them: a regular polygon of n rounded-cocircular vertices has circumcenters
whose cavities are all its n - 2 triangles, so n walks the cavity size across
the group's lanes (8), the growth list (39, 48), the sort (64) and the staged
fan (72); and the batched form's two paths (single-workgroup engine, shared
rounds) at mesh sizes where their inner branches change."""
import numpy as np
import pytest

import workloads
from tests.parity_util import diff_arrays, diff_stats, gpu_run, oracle_run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2007_00324_amd import gdp2d
    return gdp2d.Context(0)


@pytest.mark.parametrize("engine", [False, True], ids=["grid", "engine"])
@pytest.mark.parametrize("n", [4, 9, 10, 11, 18, 40, 41, 42, 50, 51, 65, 66, 67, 71, 72, 73, 75, 130])
def test_cavity_sizes(ctx, n, engine):
    p = workloads.scaled_config2(1, n, 0, seed=n, r_lo=0.40, r_hi=0.45)
    print(f"[groups] {p.name} engine={engine}", flush=True)
    om, orc_rc = oracle_run(p, cand_cap_K=4)
    gm, gpu_rc = gpu_run(ctx, p, cand_cap_K=4, tail_engine_max=(1 << 30) if engine else -1)
    assert orc_rc == gpu_rc
    assert not diff_arrays(om.arrays(), gm.arrays())
    assert not diff_stats(om.stats, gm.round_stats())


@pytest.mark.parametrize("sizes", [[20000], [30000] + [100] * 60, [3, 7, 4000, 4001, 8200]])
@pytest.mark.parametrize("split", [1, 0, 1 << 30], ids=["shared", "auto", "engine"])
def test_batch_paths_equal_the_plain_path(ctx, sizes, split):
    from paper_2007_00324_amd import gdp2d
    ps = [workloads.random_small(17 + i, n, max(1, n // 50), 2.0, pairing="knn" if n > 20 else "uniform")
          for i, n in enumerate(sizes)]
    print(f"[groups] batch of {len(ps)} split={split}", flush=True)
    prm = gdp2d.make_params(batch_engine_max_v=split)
    meshes, st, _ = gdp2d.gdp_refine_batch(ctx, [(p.xy, p.seg) for p in ps], [p.ratio_bound_sq for p in ps], prm)
    assert all(s == 0 for s in st), st
    for p, g in zip(ps, meshes):
        alone, rc = gpu_run(ctx, p)
        assert rc == 0
        assert not diff_arrays(alone.arrays(), g.arrays()), p.name
        assert not diff_stats(alone.round_stats()[:64], g.round_stats()), p.name
