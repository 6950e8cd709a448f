"""Which kernel an FP64 call takes when no launch shape was chosen, and that
a chosen shape is kept: the two shapes' costs agree to 1e-9 but not bit for
bit, so equal bits name the kernel that ran.  Sizes at the lines of the rule
(rounds of 8192 samples on lane groups, of 49152 or 65536 on one lane per
sample) for updates, updates that return their noise, rollouts alone, with
and without the force estimate and collision pairs; a few samples against
the oracle."""
import numpy as np
import pytest

from paper_2609_02020_amd import binding as B
from gpu_util import torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,which,i,T,K,shape", [
    ("update", "wall_k4096", 2, 18, 45056, 8),
    ("update", "wall_k4096", 2, 11, 49152, 8),
    ("update", "single_k256", 0, 18, 49152, 8),
    ("update", "collision_k4096", 3, 4, 49152, 8),
    ("update", "wall_k4096", 2, 1, 16384, 8),
    ("update", "wall_k4096", 2, 1, 16385, 1),
    ("update", "wall_k4096", 2, 6, 65536, 1),
    ("update", "wall_k4096", 2, 6, 65537, 8),
    ("update", "wall_k4096", 2, 8, 49152, 1),
    ("update", "wall_k4096", 2, 8, 49153, 8),
    ("update", "wall_k4096", 2, 10, 40960, 8),
    ("update", "wall_k4096", 2, 10, 40961, 1),
    ("update", "single_k256", 0, 4, 40961, 1),
    ("update", "single_k256", 0, 7, 49152, 8),
    ("noise", "wall_k4096", 2, 6, 40961, 1),
    ("noise", "wall_k4096", 2, 7, 49152, 8),
    ("rollout", "wall_k4096", 2, 18, 40960, 8),
    ("rollout", "wall_k4096", 2, 18, 65536, 1),
    ("rollout", "wall_k4096", 2, 18, 65537, 8),
    ("rollout", "collision_k4096", 3, 4, 65536, 8),
])
def test_fp64_launch_rule(ora, workloads, kind, which, i, T, K, shape):
    torch, dev = torch_dev()
    case = workloads[which][i]
    cost = dict(case["cost"], K=K, T=T)
    f64 = dict(dtype=torch.float64, device=dev)
    U = torch.tensor(case["U_nom"], **f64)[:1].expand(T, 7).contiguous()

    def run(chosen):
        io = {"q": torch.tensor(case["q0"], **f64), "qd": torch.tensor(case["qd0"], **f64),
              "target": torch.tensor(B.target_vector(case["target"]), **f64), "U_nominal": U,
              "U_new": torch.empty((T, 7), **f64), "costs": torch.empty(K, **f64),
              "noise": None if kind == "update" else torch.empty(T * 7 * K, **f64), "seed": 5, "tick": 2}
        solver = B.Solver(case["robot"], cost, B.FP64)
        if chosen:
            solver.set_launch(chosen)
        (solver.rollout_async if kind == "rollout" else solver.update_async)(io)
        torch.cuda.synchronize()
        solver.close()
        return io
    default, groups, lanes = run(0), run(8), run(1)
    same, other = (groups, lanes) if shape == 8 else (lanes, groups)
    assert torch.equal(default["costs"], same["costs"]) and not torch.equal(default["costs"], other["costs"])
    assert ((groups["costs"] - lanes["costs"]).abs() / lanes["costs"].abs()).max() <= 1e-9
    if kind != "rollout":
        assert torch.equal(default["U_new"], same["U_new"])
    for k in (0, K // 2, K - 1):
        S = ora.rollout(case["robot"], cost, case["target"], case["q0"], case["qd0"], U.cpu().numpy(), 5, 2, k)[0]
        assert abs(float(default["costs"][k]) / S - 1.0) <= 1e-9
