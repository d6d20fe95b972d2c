"""Single-step kernels and both layouts of the per-lane worlds' records (a row per field,
quads of fields where worlds hold three drones or more): states bit for bit those of the
work-queue kernel, gradients against the FP64 oracle."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads as W
from gpu_helpers import dev
from test_gpu_lane_lds import _workload
from test_gpu_parity import _check_against_oracle, _rollout_grads, _sim

pytestmark = pytest.mark.gpu


def _shared(w, per_world):
    """The drones of w in worlds of per_world (which keep the first worlds' parameters)."""
    M = w.n_worlds // per_world
    return dataclasses.replace(
        w, n_worlds=M, drones_per_world=np.full(M, per_world, np.int32), model_per_world=w.model_per_world[:M],
        params={k: np.ascontiguousarray(v[:M]) for k, v in w.params.items()})


def _drones(control, D, T):
    if control == "identified":
        return W.id_rollout_grad(seed=11, n_worlds=D, steps=T)
    if control == "rotor":
        return W.fp_rotor_open_loop(seed=12, n_worlds=D, steps=T)
    return _workload(control, D, T)


@pytest.mark.parametrize("control", ["rotor", "attitude", "torque", "position", "identified"])
@pytest.mark.parametrize("per_world", [1, 2, 3, 31])
def test_steps_equal_the_work_queue(gpu_lib, control, per_world):
    D = per_world * (16 * torch.cuda.get_device_properties(0).multi_processor_count // per_world + 70)
    w = _shared(_drones(control, D, 2), per_world)
    u = dev(w.cmds[0])
    x, y = dev(w.x0), dev(w.x0)
    lane, queue = _sim(w), _sim(w)
    queue.set_launch_config(workqueue=1, tile=64)
    for k in (1, 1, 7, 1):
        lane.step_k(x, u, k)
        queue.step_k(y, u, k)
        torch.cuda.synchronize()
        assert torch.equal(x, y), k


@pytest.mark.parametrize("control", ["torque", "position"])
def test_gradients_of_shared_worlds(gpu_lib, control):
    w = _shared(_workload(control, 66, 12), 3)
    _check_against_oracle(w, _rollout_grads(w, 5))
