"""The eight-lane update in FP64 (the default for FP64 rollouts of the
articulated-body route): ragged and smallest sizes, both ends of the
horizon, the sampling and wrench variants and the collision term against
the oracle (costs 1e-9 relative, U_new by the stage check), and against the
one-lane launch; the noise through the caller's buffer, the solver's own
buffer and regenerated (no buffer) gives the same bits."""
import numpy as np
import pytest

from paper_2609_02020_amd import binding as B
from gpu_util import device_update, torch_dev

pytestmark = pytest.mark.gpu

CONST = dict(ext_mode=B.EXT_CONST, F_ext=[5.0, -3.0, 8.0, 0.4, -0.2, 0.3])


def resized(case, K, T, **extra):
    return dict(case, cost=dict(case["cost"], K=K, T=T, **extra), U_nom=np.tile(np.asarray(case["U_nom"])[:1], (T, 1)))


@pytest.mark.parametrize("which,i,K,T,extra", [
    ("wall_k4096", 2, 1, 1, {}),
    ("wall_k4096", 2, 15, 18, {}),
    ("wall_k4096", 2, 17, 2, {"noise_rho": 0.8}),
    ("single_k256", 3, 1000, 18, CONST),
    ("wall_k4096", 6, 513, 33, {"dt": 0.006, "force_mode": 1}),
    ("wall_k4096", 2, 33, 256, {"dt": 0.001}),
    ("collision_k4096", 3, 100, 18, {}),
])
def test_group64_matches_oracle(ora, workloads, which, i, K, T, extra):
    case = resized(workloads[which][i], K, T, **extra)
    solver = B.Solver(case["robot"], case["cost"], B.FP64)
    out = device_update(solver, case, case["seed"], 3, B.FP64)
    solver.set_launch(1)
    lane = device_update(solver, case, case["seed"], 3, B.FP64)
    solver.close()
    st, U_ref, S_ref, E_ref = ora.update(case["robot"], case["cost"], case["target"], case["q0"], case["qd0"],
                                         case["U_nom"], case["seed"], 3)
    assert st == out["status"] == B.OK
    assert np.abs(out["noise"] - E_ref).max() <= 1e-12 * max(1.0, np.abs(E_ref).max())
    for S in (S_ref, lane["costs"]):
        assert (np.abs(out["costs"] - S) / np.abs(S)).max() <= 1e-9
    _, U_stage, _ = ora.weights_update(out["costs"], out["noise"], case["U_nom"], case["cost"]["lambda"])
    assert np.abs(out["U_new"] - U_stage).max() <= 1e-9
    assert np.array_equal(out["U_shift"][:-1], out["U_new"][1:])


@pytest.mark.parametrize("K,T", [(16, 18), (1000, 18), (700, 110)])
def test_group64_noise_source_does_not_matter(workloads, K, T):
    torch, dev = torch_dev()
    case = resized(workloads["wall_k4096"][2], K, T, dt=0.002)
    f64 = dict(dtype=torch.float64, device=dev)

    def io(noise):
        return {"q": torch.tensor(case["q0"], **f64), "qd": torch.tensor(case["qd0"], **f64),
                "target": torch.tensor(B.target_vector(case["target"]), **f64),
                "U_nominal": torch.tensor(case["U_nom"], **f64), "U_new": torch.empty((T, 7), **f64),
                "costs": torch.empty(K, **f64), "noise": torch.empty(T * 7 * K, **f64) if noise else None,
                "seed": 5, "tick": 2}
    solver = B.Solver(case["robot"], case["cost"], B.FP64)
    a, b, c = io(True), io(False), io(False)
    solver.update_async(a)
    solver.update_async(b)
    B.update_noalloc(case["robot"], case["cost"], c, B.FP64)
    torch.cuda.synchronize()
    for x in (b, c):
        assert torch.equal(a["U_new"], x["U_new"]) and torch.equal(a["costs"], x["costs"])
    solver.close()


@pytest.mark.parametrize("K", [40960, 40961, 49152, 49153])
def test_group64_launch_rule(workloads, K):
    """Both sides of the sizes at which the default launch changes: costs
    1e-9 relative against the one-lane launch."""
    case = resized(workloads["wall_k4096"][2], K, 1)
    solver = B.Solver(case["robot"], case["cost"], B.FP64)
    out = device_update(solver, case, case["seed"], 3, B.FP64)
    solver.set_launch(1)
    lane = device_update(solver, case, case["seed"], 3, B.FP64)
    solver.close()
    assert (np.abs(out["costs"] - lane["costs"]) / np.abs(lane["costs"])).max() <= 1e-9
    assert np.abs(out["U_new"] - lane["U_new"]).max() <= 1e-9
