"""The eight-lane FP64 plant over the problems of a batch (eight to a wave)
against the oracle: partial and several waves, each external-wrench model,
torques past the limits, one and several substeps.  Tolerances as for the
single plant: rounding of FP64 dynamics over at most ten substeps."""
import numpy as np
import pytest

from paper_2609_02020_amd import binding as B
from gpu_util import torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,substeps", [(1, 10), (7, 1), (8, 10), (9, 3), (17, 10)])
def test_batch_plant_matches_oracle(ora, workloads, n, substeps):
    torch, dev = torch_dev()
    f64 = dict(dtype=torch.float64, device=dev)
    rng = np.random.default_rng(50 + n)
    cases = []
    for i in range(n):
        c = (workloads["wall_k4096"] + workloads["single_k256"])[i]
        cost = dict(c["cost"], K=64, T=2 + i % 3)
        if i % 3 == 1:
            cost.update(ext_mode=B.EXT_CONST, F_ext=[5.0, -3.0, 8.0, 0.4, -0.2, 0.3])
        cases.append(dict(c, cost=cost))
    batch = B.Batch([(c["robot"], c["cost"]) for c in cases])
    q = np.array([c["q0"] for c in cases]) + rng.uniform(-0.1, 0.1, (n, 7))
    qd = rng.uniform(-0.5, 0.5, (n, 7))
    U = rng.uniform(-100.0, 100.0, (batch.u_total // 7, 7))   # the distal joints' limits are 12 N m
    io = {"q": torch.tensor(q, **f64), "qd": torch.tensor(qd, **f64), "U_nominal": torch.tensor(U, **f64),
          "U_new": torch.tensor(U, **f64), "target": torch.zeros((n, 13), **f64),
          "seed": torch.zeros(n, dtype=torch.int64, device=dev)}
    batch.plant_step_async(io, 1e-3 * substeps, substeps)
    torch.cuda.synchronize()
    for p, c in enumerate(cases):
        qr, qdr = ora.plant_step(c["robot"], c["cost"], q[p], qd[p], U[batch.u_off[p] // 7], 1e-3 * substeps, substeps)
        assert np.abs(io["q"][p].cpu().numpy() - qr).max() < 1e-10, p
        assert np.abs(io["qd"][p].cpu().numpy() - qdr).max() < 1e-8, p
    batch.close()
