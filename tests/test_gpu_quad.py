"""One drone on four lanes (small batches): held states bit for bit those of the
one-lane work-queue kernel, rollouts and gradients against the FP64 oracle, at batch
sizes around a wave's 16 drones and checkpoint intervals around the horizon."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from gpu_helpers import assert_states_close, dev
from paper_2606_01478_amd import binding as B
from test_gpu_mlp import _grads
from test_gpu_parity import _check_against_oracle, _rollout_grads, _sim

pytestmark = pytest.mark.gpu


def _workload(model, D, T=24):
    if model == "id":
        return W.id_rollout_grad(seed=81 + D, n_worlds=D, steps=T)
    if model == "pid":
        w = W.gradient_goal(seed=82 + D, n_worlds=D, steps=T)
    else:
        w = W.fp_rotor_open_loop(seed=83 + D, n_worlds=D, steps=T)
        w = dataclasses.replace(w, dloss=np.ones(D, np.float32))
    return w


@pytest.mark.parametrize("model", ["rotor", "pid", "id"])
@pytest.mark.parametrize("D", [1, 15, 16, 67])
def test_held_states_equal_one_lane_per_drone(gpu_lib, model, D):
    w = _workload(model, D)
    u = dev(w.cmds[0])
    x, y = dev(w.x0), dev(w.x0)
    quad, lane = _sim(w), _sim(w)
    lane.set_launch_config(workqueue=1, tile=64)
    for k in (1, 19, 40):
        quad.step_k(x, u, k)
        lane.step_k(y, u, k)
        torch.cuda.synchronize()
        assert torch.equal(x, y), k
    held = dataclasses.replace(w, cmds=np.ascontiguousarray(w.cmds[0]), steps=60)
    assert_states_close(x, O.simulate_held(held), held)


@pytest.mark.parametrize("model", ["rotor", "pid", "id"])
@pytest.mark.parametrize("D,K", [(1, 1), (17, 5), (67, 24), (16, 50)])
def test_rollout_gradients(gpu_lib, model, D, K):
    w = _workload(model, D)
    _check_against_oracle(w, _rollout_grads(w, K))


def test_feedback_through_the_attitude_controller(gpu_lib):
    w = _workload("pid", 21, 40)
    rng = np.random.Generator(np.random.Philox(7))
    gain = rng.normal(0.0, 0.01, size=(2, 4, 13)).astype(np.float32)
    w = dataclasses.replace(w, gain=gain, gain_index=(np.arange(21) % 2).astype(np.int32))
    _check_against_oracle(w, _rollout_grads(w, 8))


def test_nonfinite_world_is_flagged(gpu_lib):
    w = _workload("id", 37)
    sim = _sim(w, flags=B.F_NONFINITE_CHECK)
    x = dev(w.x0)
    x[7, 20] = float("inf")
    flag = torch.zeros(37, dtype=torch.int32, device="cuda")
    sim.step_k(x, dev(w.cmds[0]), 3, nonfinite=flag)
    torch.cuda.synchronize()
    assert flag[20] == 1 and int(flag.sum()) == 1


@pytest.mark.parametrize("hidden,T", [(5, 30), (13, 30), (16, 3), (31, 12)])
def test_two_policies_of_odd_width(gpu_lib, hidden, T):
    """Padded units, two policies in one batch, and (T = 3) a horizon so short that
    records take less scratch than each drone's own sum of the weight gradient."""
    w = W.id_rollout_grad_mlp(seed=90 + hidden, n_worlds=21, steps=T, hidden=hidden, out_scale=0.05)
    rng = np.random.Generator(np.random.Philox(hidden))
    w = dataclasses.replace(w, gain=W.mlp_policy_params(rng, 2, hidden, 0.05),
                            gain_index=(np.arange(21) % 2).astype(np.int32))
    _check_against_oracle(w, _grads(_sim(w), w, 7))
