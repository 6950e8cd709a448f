"""Nominal selection with sequences whose cost leaves the range of the
rollout precision (1e300 N m in FP64, 1e30 in FP32): reported as +inf, never
taken over a finite one, always replaced by one, and kept when the candidate
is no better; over both lane-group parities of a batch too (FP32)."""
import numpy as np
import pytest

from paper_2609_02020_amd import binding as B
from gpu_util import torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,huge", [(B.FP32, 1e30), (B.FP64, 1e300)])
@pytest.mark.parametrize("which,i,T", [("wall_k4096", 2, 18), ("single_k256", 0, 2), ("collision_k4096", 3, 5)])
def test_sequences_without_a_finite_cost(workloads, which, i, T, precision, huge):
    torch, dev = torch_dev()
    f64 = dict(dtype=torch.float64, device=dev)
    case = workloads[which][i]
    solver = B.Solver(case["robot"], dict(case["cost"], K=64, T=T), precision)
    U0 = np.tile(np.asarray(case["U_nom"])[:1], (T, 1))
    bad = np.full_like(U0, huge)
    for nominal, cand, expect, finite in ((U0, bad, U0, (True, False)), (bad, U0, U0, (False, True)),
                                          (bad, 2 * bad, bad, (False, False))):
        io = {"q": torch.tensor(case["q0"], **f64), "qd": torch.tensor(case["qd0"], **f64),
              "target": torch.tensor(B.target_vector(case["target"]), **f64),
              "U_nominal": torch.tensor(nominal, **f64), "seed": 0, "tick": 0}
        costs = torch.zeros(2, **f64)
        solver.select_nominal_async(io, torch.tensor(cand, **f64), costs)
        torch.cuda.synchronize()
        assert np.array_equal(io["U_nominal"].cpu().numpy(), expect)
        assert [c < float("inf") for c in costs.tolist()] == list(finite)
        assert not torch.isnan(costs).any()
    solver.close()


def test_batch_sequences_without_a_finite_cost(workloads):
    torch, dev = torch_dev()
    f64 = dict(dtype=torch.float64, device=dev)
    cases = [workloads["wall_k4096"][2], workloads["single_k256"][0], workloads["collision_k4096"][3]]
    batch = B.Batch([(c["robot"], dict(c["cost"], K=64, T=6)) for c in cases])
    U0 = np.concatenate([np.tile(np.asarray(c["U_nom"])[:1], (6, 1)) for c in cases])
    bad = np.full_like(U0, 1e30)
    for nominal, cand in ((U0, bad), (bad, U0)):
        io = {"q": torch.tensor(np.array([c["q0"] for c in cases]), **f64),
              "qd": torch.tensor(np.array([c["qd0"] for c in cases]), **f64),
              "target": torch.tensor(np.array([B.target_vector(c["target"]) for c in cases]), **f64),
              "U_nominal": torch.tensor(nominal, **f64), "U_new": torch.zeros(U0.shape, **f64),
              "seed": torch.zeros(3, dtype=torch.int64, device=dev)}
        costs = torch.zeros((3, 2), **f64)
        batch.select_nominal_async(io, torch.tensor(cand, **f64), costs)
        torch.cuda.synchronize()
        assert np.array_equal(io["U_nominal"].cpu().numpy(), U0)
        assert (torch.isinf(costs).sum(1) == 1).all() and not torch.isnan(costs).any()
    batch.close()
