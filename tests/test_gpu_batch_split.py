"""Batches of at most 256 tiles run two waves per tile: at the line (256 and
257 tiles), for partial tiles, the collision term, FP64 weights and several
iterations, and replayed from a graph between eager updates, they equal the
one-wave-per-tile launch (the same arithmetic; the compiler contracts a few
multiply-adds differently, 1e-6 relative as for the single-problem launches)
and leave the queue and counters ready for the next launch."""
import numpy as np
import pytest

from paper_2609_02020_amd import binding as B
from gpu_util import torch_dev

pytestmark = pytest.mark.gpu


def problems(workloads, sizes, T, **extra):
    out = []
    for i, K in enumerate(sizes):
        c = workloads["wall_k4096"][(2, 6)[i % 2]] if i % 3 else workloads["single_k256"][0]
        out.append(dict(c, cost=dict(c["cost"], K=K, T=T, **extra), U_nom=np.tile(np.asarray(c["U_nom"])[:1], (T, 1))))
    return out


def make_io(batch, cases, torch, dev):
    f64 = dict(dtype=torch.float64, device=dev)
    U = np.concatenate([c["U_nom"] for c in cases])
    return {"q": torch.tensor(np.array([c["q0"] for c in cases]), **f64),
            "qd": torch.tensor(np.array([c["qd0"] for c in cases]), **f64),
            "target": torch.tensor(np.array([B.target_vector(c["target"]) for c in cases]), **f64),
            "U_nominal": torch.tensor(U, **f64), "U_new": torch.empty(U.shape, **f64),
            "costs": torch.empty(batch.k_total, dtype=torch.float32, device=dev),
            "status": torch.full((len(cases),), -1, dtype=torch.int32, device=dev),
            "seed": torch.arange(5, 5 + len(cases), dtype=torch.int64, device=dev)}


@pytest.mark.parametrize("sizes,T,coll,extra", [
    ([1], 1, False, {}),
    ([63, 64, 65, 129], 18, False, {"lambda": 0.01}),
    ([100, 1000, 300], 64, True, {"dt": 0.002}),
    ([100, 65], 27, True, {"dt": 0.002}),
    ([100, 65], 28, False, {"dt": 0.002, "noise_rho": 0.5}),
    ([4096, 4096, 4096, 4096], 10, False, {"lambda": 100.0}),
    ([4096, 4096, 4096, 4097], 10, False, {"lambda": 100.0}),
    ([500, 70], 12, False, {"iterations": 3, "noise_rho": 0.5, "lambda": 100.0}),
])
def test_two_waves_per_tile_match_one(workloads, sizes, T, coll, extra):
    torch, dev = torch_dev()
    cases = problems(workloads, sizes, T, **extra)
    if coll:
        c = workloads["collision_k4096"][3]
        cases[1] = dict(c, cost=dict(c["cost"], K=sizes[1], T=T, **extra), U_nom=np.tile(np.asarray(c["U_nom"])[:1], (T, 1)))
    batch = B.Batch([(c["robot"], c["cost"]) for c in cases])
    io, ref = make_io(batch, cases, torch, dev), make_io(batch, cases, torch, dev)
    batch.update_async(io, tick=4)
    first = {k: io[k].clone() for k in ("costs", "U_new", "status")}
    batch.update_async(io, tick=4)   # the queue and counters were reset
    torch.cuda.synchronize()
    assert all(torch.equal(first[k], io[k]) for k in first)
    batch.set_launch(1, 300)
    batch.update_async(ref, tick=4)
    torch.cuda.synchronize()
    S, R = io["costs"].double().cpu().numpy(), ref["costs"].double().cpu().numpy()
    assert (np.abs(S - R) / np.abs(R)).max() <= 1e-6
    assert np.abs(io["U_new"].cpu().numpy() - ref["U_new"].cpu().numpy()).max() <= 1e-4
    assert (io["status"] == B.OK).all()
    batch.set_launch(2, 7)   # fewer workgroups than tiles, from a graph between eager updates
    g = make_io(batch, cases, torch, dev)
    batch.graph_capture(g)
    batch.set_tick(4)
    for r in range(3):
        batch.graph_launch(torch.cuda.current_stream())
        batch.update_async(ref, tick=4 + r)
        torch.cuda.synchronize()
        assert torch.equal(g["U_new"], ref["U_new"]) and torch.equal(g["costs"], ref["costs"])
    batch.close()
