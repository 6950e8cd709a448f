"""Collision pairs on the lane groups are dealt over lanes and rounds of
eight pairs, and the rounds over the dynamics and cost waves: pair counts at
both ends of a round, horizons of one, two and more steps, link-link and
link-obstacle pairs, against the oracle (FP64, costs 1e-9 relative) and,
with thresholds that every pair meets, against the exact count
w_collision n T (FP32: 32 u32 of the largest cost, a sum of up to 18 steps
in two shares)."""
import numpy as np
import pytest

from paper_2609_02020_amd import binding as B
from gpu_util import device_update

pytestmark = pytest.mark.gpu


def with_pairs(case, n, T, d_th):
    every = [[a, b] for a in range(7) for b in range(a + 2, 9)]   # segments 7 and 8: the two obstacles
    assert len(case["cost"]["obstacles"]) >= 2
    pairs = [every[(5 * i) % len(every)] for i in range(n)]
    return dict(case, cost=dict(case["cost"], K=33, T=T, pairs=pairs, d_th=d_th[:n]),
                U_nom=np.tile(np.asarray(case["U_nom"])[:1], (T, 1)))


def costs(case, precision):
    solver = B.Solver(case["robot"], case["cost"], precision)
    out = device_update(solver, case, case["seed"], 3, precision)
    solver.close()
    assert out["status"] == B.OK
    return out["costs"].astype(np.float64)


@pytest.mark.parametrize("n,T", [(1, 18), (8, 2), (9, 1), (16, 18), (17, 3), (25, 18), (32, 2)])
def test_pair_rounds(ora, workloads, n, T):
    base = workloads["collision_k4096"][3]
    case = with_pairs(base, n, T, [0.1 + 0.02 * i for i in range(32)])
    st, _, S_ref, _ = ora.update(case["robot"], case["cost"], case["target"], case["q0"], case["qd0"],
                                 case["U_nom"], case["seed"], 3)
    assert st == B.OK
    S = costs(case, B.FP64)
    assert (np.abs(S - S_ref) / np.abs(S_ref)).max() <= 1e-9
    for precision, tol in ((B.FP64, 1e-9), (B.FP32, 32 * 2.0 ** -24)):
        all_hit = costs(with_pairs(base, n, T, [100.0] * 32), precision)
        no_hit = costs(with_pairs(base, n, T, [0.0] * 32), precision)
        extra = case["cost"]["w_collision"] * n * T
        assert np.abs(all_hit - no_hit - extra).max() <= tol * np.abs(all_hit).max()
