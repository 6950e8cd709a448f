"""The solver's own noise buffer belongs to a rollout and the weights that
follow it: a fused update, a host update or the autotuner run on the same
handle in between, none of which asks for the noise, leaves it alone, so the
weights give the same U_new bit for bit."""
import pytest

from paper_2609_02020_amd import binding as B
from gpu_util import torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("between", ["update", "iterated", "host", "autotune"])
@pytest.mark.parametrize("precision", [B.FP32, B.FP64])
@pytest.mark.parametrize("K,T", [(33, 2), (1000, 18)])
def test_updates_leave_a_rollouts_noise(workloads, K, T, precision, between):
    torch, dev = torch_dev()
    case = workloads["wall_k4096"][2]
    cost = dict(case["cost"], K=K, T=T)
    f64 = dict(dtype=torch.float64, device=dev)
    rdt = torch.float64 if precision == B.FP64 else torch.float32
    U = torch.tensor(case["U_nom"], **f64)[:1].expand(T, 7).contiguous()

    def io(seed):
        return {"q": torch.tensor(case["q0"], **f64), "qd": torch.tensor(case["qd0"], **f64),
                "target": torch.tensor(B.target_vector(case["target"]), **f64), "U_nominal": U,
                "U_new": torch.full((T, 7), float("nan"), **f64), "costs": torch.empty(K, dtype=rdt, device=dev),
                "seed": seed, "tick": 2}
    solver = B.Solver(case["robot"], cost, precision)
    a, other = io(5), io(6)
    solver.rollout_async(a)
    solver.weights_async(a)
    torch.cuda.synchronize()
    want = a["U_new"].clone()
    a["U_new"].fill_(float("nan"))
    solver.rollout_async(a)
    torch.cuda.synchronize()
    if between == "update":
        solver.update_async(other)
    elif between == "iterated":
        solver.set_cost(dict(cost, iterations=3))
        solver.update_async(other)
        solver.set_cost(cost)
    elif between == "host":
        solver.update(case["q0"], case["qd0"], case["target"], U.cpu().numpy(), 6, 2)
    else:
        solver.autotune(other, budget_ms=3)
    solver.weights_async(a)
    torch.cuda.synchronize()
    assert torch.equal(a["U_new"], want)
    solver.close()
