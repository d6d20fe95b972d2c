"""The launch choices of the autotune cache file: one stored for other kernels (an older
signature) is not taken, one that this library stored is."""
import pytest
import torch

import workloads as W
from gpu_helpers import dev
from paper_2606_01478_amd import binding as B

pytestmark = pytest.mark.gpu


def test_choices_of_older_kernels_are_dropped(gpu_lib, tmp_path, monkeypatch):
    path = tmp_path / "cache.txt"
    monkeypatch.setenv("CFSIM_AUTOTUNE_CACHE", str(path))
    w = W.id_swarm(seed=51, n_worlds=3, n_drones=40, steps=8)
    sim = B.Sim.from_workload(w)
    sim.autotune(dev(w.x0), dev(w.cmds), 8, budget_ms=5)
    torch.cuda.synchronize()
    key, wq, tile, chunk, split, ms = path.read_text().split()
    assert key.startswith("v")
    version = int(key[1:].split("|")[0])
    other = {"0": "1", "1": "0"}[wq]
    line = f"{other} 256 0 1 0.001\n"
    path.write_text(f"{key} {line}")
    taken = B.Sim.from_workload(w).launch_config()
    assert (taken["workqueue"], taken["tile"]) == (int(other), 256)
    for old in range(version):
        path.write_text(f"v{old}|{key.split('|', 1)[1]} {line}")
        assert B.Sim.from_workload(w).launch_config()["tile"] == 64
    assert version >= 4   # 3: the kernels before four lanes a drone
