"""Inputs at the edge of the number range, where a kernel must not use what the model
does not: non-finite commands that the controller's limits absorb."""
import pytest
import torch

import workloads as W
from gpu_helpers import dev
from paper_2606_01478_amd import binding as B
from test_gpu_parity import _sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("K", [1, 5])
def test_absorbed_thrust_commands_flag_no_world(gpu_lib, value, K):
    """The allocation clamps a non-finite thrust command: the states stay finite, and no
    world is flagged whichever kernel the batch's size selects."""
    w = W.gradient_goal(seed=91, n_worlds=37, steps=1)
    u = dev(w.cmds[0])
    u[3, 11] = value
    u[0, 23] = float("nan")          # not absorbed: an attitude command
    flags, states = [], []
    for wq in (0, 1):
        sim = _sim(w, flags=B.F_NONFINITE_CHECK)
        sim.set_launch_config(workqueue=wq, tile=64)
        x, f = dev(w.x0), torch.zeros(37, dtype=torch.int32, device="cuda")
        sim.step_k(x, u, K, nonfinite=f)
        torch.cuda.synchronize()
        flags.append(f)
        states.append(x)
    few, queue = states
    assert torch.isfinite(few[:, 11]).all()
    assert torch.equal(few.nan_to_num(7.0), queue.nan_to_num(7.0))
    assert torch.equal(flags[0], flags[1])
    assert flags[0].nonzero().flatten().tolist() == [23]

