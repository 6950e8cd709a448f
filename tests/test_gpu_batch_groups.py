"""mppi_batch_set_launch(b, 2, groups) with fewer workgroups than tiles: each
wave takes tiles of its own, so that 2 groups tiles are in flight as with one
wave per workgroup; only a workgroup per tile puts its two waves on one.
The latter's costs differ from the former's in their last bits for some
problems (tells), which names the launch that ran."""
import numpy as np
import pytest

from paper_2609_02020_amd import binding as B
from gpu_util import torch_dev
from test_gpu_batch_split import make_io, problems

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,T,tells", [
    ([64, 65, 1000], 18, True),
    ([4096, 4096, 4096, 4096], 10, True),
    ([500, 70], 40, False),
])
def test_fewer_workgroups_than_tiles(workloads, sizes, T, tells):
    torch, dev = torch_dev()
    cases = problems(workloads, sizes, T, dt=0.004)
    tiles = sum((K + 63) // 64 for K in sizes)
    batch = B.Batch([(c["robot"], c["cost"]) for c in cases])

    def run(w, groups):
        io = make_io(batch, cases, torch, dev)
        batch.set_launch(w, groups)
        for _ in range(2):   # the second finds the queue and counters reset
            batch.update_async(io, tick=4)
        torch.cuda.synchronize()
        assert (io["status"] == B.OK).all()
        return io
    single, whole = run(1, tiles), run(2, tiles)
    assert not (tells and torch.equal(single["costs"], whole["costs"]))
    for groups in (1, tiles // 2, tiles - 1):
        io = run(2, groups)
        assert torch.equal(io["costs"], single["costs"]) and torch.equal(io["U_new"], single["U_new"])
    io = run(2, tiles + 1)
    assert torch.equal(io["costs"], whole["costs"]) and torch.equal(io["U_new"], whole["U_new"])
    assert (np.abs((single["costs"] / whole["costs"]).double().cpu().numpy() - 1.0)).max() <= 1e-6
    batch.close()
