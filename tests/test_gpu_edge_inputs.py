"""Inputs at the edge of the number range, where a kernel must not use what the model
does not: non-finite commands that the controller's limits absorb, and the thrust row of
worlds without thrust dynamics."""
import dataclasses

import pytest
import torch

import workloads as W
from gpu_helpers import dev
from paper_2606_01478_amd import binding as B
from test_gpu_parity import _rollout_grads, _sim

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


@pytest.mark.parametrize("value", [float("nan"), float("inf"), 3e38, -3e38])
@pytest.mark.parametrize("layout", ["few", "queue", "many"])
def test_thrust_row_is_not_read_without_thrust_dynamics(gpu_lib, value, layout):
    """c_tau = 0: the commanded thrust acts directly and the row receives it; what the row
    held before changes nothing, forward or backward."""
    n = 128 * torch.cuda.get_device_properties(0).multi_processor_count + 70 if layout == "many" else 40
    w = W.id_rollout_grad(seed=92, n_worlds=n, steps=6)
    P = {k: v.copy() for k, v in w.params.items()}
    P["c_tau"][:] = 0
    w = dataclasses.replace(w, params=P, gain=None, gain_index=None)
    x0 = w.x0.copy()
    x0[12, 1::3] = value
    odd = dataclasses.replace(w, x0=x0)
    held = []
    for v in (w, odd):
        sim = _sim(v)
        if layout == "queue":
            sim.set_launch_config(workqueue=1, tile=64)
        for k in (1, 3):
            x = dev(v.x0)
            sim.step_k(x, dev(v.cmds[0]), k)
            held.append(x)
    a, b = _rollout_grads(w, 4), _rollout_grads(odd, 4)
    torch.cuda.synchronize()
    assert torch.equal(held[0], held[2]) and torch.equal(held[1], held[3])
    for k in ("loss", "x", "g_cmds", "g_x0"):
        assert torch.isfinite(a[k]).all() and torch.equal(a[k], b[k]), k
    assert (a["g_x0"][12] == 0).all()
