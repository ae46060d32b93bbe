"""The removal kernels of the Flip-Flop insertion (gdp_ff.hip), their own text
run lane by lane on the host (tests/fflanes), in rounds from the
oracle's point sets: after every pass each triangle is counter-clockwise and
the neighbours are mutual, and the round ends in the oracle's mesh.  The nested
polygons have circumcenters with links beyond a group's 16 vertices and a
wave's 64."""
import pytest

import workloads
from tests import ffemu, fflanes
from tests.test_ff_steps_host import CASES, FF, _Arr
from tests.test_oracle_ff import canon, same


def _stars(polygons, n, n_free, seed):
    return workloads.scaled_config2(polygons, n, n_free, seed=seed, r_lo={1: 0.3, 2: 0.2, 3: 0.1}[polygons], r_hi=0.45)


# case, rounds, point classes (link of up to 16, 64, more vertices) that have to come up
LANE_CASES = {
    "near_edge": (CASES["near_edge"], 200, [0]),
    "rand_300": (CASES["rand_300"], 12, [0]),
    "knn_2000": (CASES["knn_2000"], 3, [0]),
    "c0": (CASES["c0"], 5, [0]),
    "circles": (CASES["circles"], 4, [0]),
    "star_65": (lambda: _stars(1, 65, 1, 105), 200, [0, 1]),
    "star_40": (lambda: _stars(2, 40, 6, 40), 8, [0, 1]),
    "star_67": (lambda: _stars(3, 67, 0, 107), 4, [0, 1]),
    "star_130": (lambda: _stars(2, 130, 6, 130), 4, [0, 1]),
    "star_71": (lambda: _stars(3, 71, 0, 111), 3, [0, 1, 2]),
}


@pytest.mark.parametrize("encroach_mode", [0, 1])
@pytest.mark.parametrize("case", list(LANE_CASES))
def test_removal_kernels_match_oracle(orc, case, encroach_mode):
    make, rounds, classes = LANE_CASES[case]
    p = make()
    m = orc.build_cdt(p.xy, p.seg)
    lib = orc.load()
    before = fflanes.links()
    removed = 0
    for r in range(rounds):
        nxt = m.clone()
        rc = orc.refine(nxt, p.ratio_bound_sq, max_rounds=m.rounds + 1, raise_on_error=False,
                        encroach_mode=encroach_mode, **FF)
        assert rc in (0, -5), rc
        if not nxt.stats:
            break
        S = ffemu.last_points(lib)
        res, cnt = fflanes.round_from_points(m.arrays(), p.xy.shape[0], S, enc_mode=encroach_mode, order_seed=r)
        assert cnt["err"] == 0, (r, cnt)
        assert same(canon(nxt), canon(_Arr(res))), f"round {r}"
        removed += cnt["removals"]
        m = nxt
        if rc == 0:
            break
    assert removed > 0
    if encroach_mode == 0:
        assert all(fflanes.links()[c] > before[c] for c in classes), (before, fflanes.links())
