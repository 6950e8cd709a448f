"""Inference on four rows per workgroup (up to 1024 rows) against sixteen:
a row's result does not depend on how many rows share its workgroup, so the
leading rows of a 1040-row batch come out bit for bit in every smaller one
(partial and full workgroups of both sizes, the line at 1024 rows)."""
import numpy as np
import pytest

from paper_2609_02020_amd import binding as B, inputs
from gpu_util import torch_dev

pytestmark = pytest.mark.gpu


def test_rows_do_not_depend_on_the_workgroup_size(workloads):
    torch, dev = torch_dev()
    n = 1040
    net = B.Mlp(workloads["wall_k4096"][0]["robot"], n)
    net.set_params(inputs.draw_mlp_params(7).astype(np.float32))
    rng = np.random.default_rng(8)
    x = torch.tensor(rng.uniform(-1, 1, (n, 21)), dtype=torch.float32, device=dev)
    f64 = dict(dtype=torch.float64, device=dev)
    q, qd = (torch.tensor(rng.uniform(-2, 2, (n, 7)), **f64) for _ in range(2))
    tg = torch.tensor(rng.uniform(-1, 1, (n, 13)), **f64)
    y, U = torch.empty((n, 126), device=dev), torch.empty((n, 140), **f64)
    net.forward_async(x, y)
    net.propose_async(q, qd, tg, U, u_stride=140)
    for B_ in (1, 3, 4, 5, 15, 17, 63, 1021, 1024, 1025):
        ys = torch.full((B_, 126), float("nan"), device=dev)
        Us = torch.full((B_, 140), float("nan"), **f64)
        net.forward_async(x[:B_], ys)
        net.propose_async(q[:B_], qd[:B_], tg[:B_], Us, u_stride=140)
        torch.cuda.synchronize()
        assert torch.equal(ys, y[:B_]) and torch.equal(Us[:, :126], U[:B_, :126]), B_
        assert torch.isnan(Us[:, 126:]).all()
    net.close()
