"""What an entry of the autotune cache is replayed for: not for other kernels
(an entry without the present key's kernel tag), nor for a batch on the other
side of the 256 tiles up to which two waves take a tile together, and within
that side two waves per tile stay two waves per tile at another tile count."""
import json

import pytest

from paper_2609_02020_amd import binding as B
from gpu_util import torch_dev
from test_gpu_batch_split import make_io, problems

pytestmark = pytest.mark.gpu


@pytest.fixture
def cache(tmp_path):
    path = tmp_path / "tune.json"
    B.set_autotune_cache(path)
    yield path
    B.set_autotune_cache(None)


@pytest.mark.parametrize("precision", [B.FP32, B.FP64])
def test_entries_of_other_kernels_are_timed_again(workloads, cache, precision):
    torch, dev = torch_dev()
    case = workloads["wall_k4096"][2]
    f64 = dict(dtype=torch.float64, device=dev)
    io = {"q": torch.tensor(case["q0"], **f64), "qd": torch.tensor(case["qd0"], **f64),
          "target": torch.tensor(B.target_vector(case["target"]), **f64),
          "U_nominal": torch.tensor(case["U_nom"], **f64), "U_new": torch.zeros((18, 7), **f64), "seed": 5, "tick": 3}
    solver = B.Solver(case["robot"], dict(case["cost"], K=1000), precision)
    best, _ = solver.autotune(io, budget_ms=6)
    (key, entry), = json.load(open(cache)).items()
    old = key[:key.index("|it1") + 4]   # the key of the first kernels
    cache.write_text('{\n"%s": {"waves_per_group": 1, "groups": 0, "ms": %f}\n}\n' % (old, entry["ms"]))
    again, times = solver.autotune(io, budget_ms=6)
    assert all(t > 0 for t in times) and times[(8, 2, 1).index(again)] == min(times)
    solver.close()


def tune(workloads, torch, dev, tiles):
    cases = problems(workloads, [64 * tiles], 18)
    batch = B.Batch([(c["robot"], c["cost"]) for c in cases])
    w, g, times = batch.autotune(make_io(batch, cases, torch, dev), reps=2)
    batch.close()
    return w, g, times


def test_batches_on_either_side_of_256_tiles(workloads, cache):
    torch, dev = torch_dev()
    for tiles in (240, 400):   # one power of two of sample-steps at T = 18
        assert all(t > 0 for t in tune(workloads, torch, dev, tiles)[2])
    w, g, times = tune(workloads, torch, dev, 250)
    assert times == [-1.0] * 16 and (w != 2 or g >= 250)


def test_two_waves_per_tile_at_another_tile_count(workloads, cache):
    torch, dev = torch_dev()
    tune(workloads, torch, dev, 120)
    entries = json.load(open(cache))
    (key, entry), = entries.items()
    if entry["waves_per_group"] == 2:   # a workgroup per tile at any of these counts
        assert entry["groups"] >= 256
    w, g, times = tune(workloads, torch, dev, 220)
    assert times == [-1.0] * 16 and (w, g) == (entry["waves_per_group"], entry["groups"])
