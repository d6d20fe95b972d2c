"""Adjoint of a world per lane whose coefficients and controller gains are held in LDS
(one wave a workgroup): batches around a wave's 64 drones against the FP64 oracle, and a
batch above the four-lane range against the same worlds on four lanes."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from gpu_helpers import assert_grad_close
from test_gpu_parity import _check_against_oracle, _rollout_grads

pytestmark = pytest.mark.gpu


def _workload(control, D, T):
    w = W.gradient_goal(seed=60 + D, n_worlds=D, steps=T)
    if control == "attitude":
        return w
    rng = np.random.Generator(np.random.Philox(D))
    mg = (9.81 * w.params["mass"].reshape(-1)).astype(np.float32)
    u = np.zeros_like(w.cmds)
    if control == "torque":
        u[:, 0] = mg * rng.uniform(0.9, 1.1, size=(T, D))
        u[:, 1:] = rng.normal(0.0, 1e-5, size=(T, 3, D))
    else:
        u[:, 0:3] = w.x0[None, 0:3] + rng.normal(0.0, 0.05, size=(T, 3, D))
    code = {"torque": W.CTRL_TORQUE, "position": W.CTRL_POSITION}[control]
    return dataclasses.replace(w, control=code, x0=np.ascontiguousarray(w.x0[:17]), cmds=u)


@pytest.mark.parametrize("control", ["torque", "position"])
@pytest.mark.parametrize("D,K", [(1, 1), (63, 4), (64, 20), (130, 7)])
def test_gradients_around_a_wave(gpu_lib, control, D, K):
    w = _workload(control, D, 12)
    _check_against_oracle(w, _rollout_grads(w, K))


@pytest.mark.parametrize("control", ["torque", "position"])
def test_gradients_with_feedback(gpu_lib, control):
    D = 65
    w = _workload(control, D, 12)
    gain = np.random.Generator(np.random.Philox(5)).normal(0.0, 1.0, size=(2, 4, 13))
    gain *= 1e-3 if control == "position" else np.array([1e-3, 1e-6, 1e-6, 1e-6])[None, :, None]
    w = dataclasses.replace(w, gain=gain.astype(np.float32), gain_index=(np.arange(D) % 2).astype(np.int32))
    _check_against_oracle(w, _rollout_grads(w, 5))


def test_attitude_batch_above_the_four_lane_range(gpu_lib):
    import torch

    D = 128 * torch.cuda.get_device_properties(0).multi_processor_count + 70
    w = _workload("attitude", D, 6)
    s = slice(D - 65, D)
    tail = W.subset(w, list(range(D - 65, D)))
    full, few = _rollout_grads(w, 4), _rollout_grads(tail, 4)
    assert torch.equal(full["x"][:, s], few["x"])
    for k in ("g_cmds", "g_x0"):
        assert_grad_close(full[k][..., s], few[k].double().cpu(), k)
