"""Rollouts and adjoints of batches above the four-lane range, on the kernels that larger
batches get (a drone per lane, or tiles of one world), in the forms whose small batches run
four lanes a drone: the last drones of the batch against the FP64 oracle."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_mlp import _grads
from test_gpu_one_step import _shared
from test_gpu_parity import _check_against_oracle, _rollout_grads, _sim

pytestmark = pytest.mark.gpu

PER_WORLD = {"lanes": 1, "tiles": 65}   # tiles: two of 64 lanes a world, one of them of a single drone


def _above_the_range(layout):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return (128 * cus // PER_WORLD[layout] + 7) * PER_WORLD[layout]


def _tail(w, got, n):
    """The last n worlds of w and their part of got (g_gain: of the whole batch)."""
    worlds = list(range(w.n_worlds - n, w.n_worlds))
    s = slice(int(w.world_offsets()[-1 - n]), None)
    part = dict(loss=got["loss"][s], loss_world=got["loss_world"][-n:], x=got["x"][:, s], g_gain=got["g_gain"],
                g_cmds=got["g_cmds"][..., s], g_x0=got["g_x0"][:, s])
    return W.subset(w, worlds), part


def _only_tail_counts(w, n):
    """The loss of the last n worlds alone, so that gain gradients are theirs."""
    dloss = np.zeros(w.n_drones_total, np.float32)
    dloss[int(w.world_offsets()[-1 - n]):] = 1.0
    return dataclasses.replace(w, dloss=dloss)


@pytest.mark.parametrize("layout", ["lanes", "tiles"])
@pytest.mark.parametrize("K", [1, 4])
def test_rotor_interface(gpu_lib, layout, K):
    w = _shared(W.fp_rotor_open_loop(seed=101, n_worlds=_above_the_range(layout), steps=6), PER_WORLD[layout])
    n = 65 // PER_WORLD[layout] + 1
    w = _only_tail_counts(w, n)
    _check_against_oracle(*_tail(w, _rollout_grads(w, K), n))


@pytest.mark.parametrize("layout", ["lanes", "tiles"])
def test_attitude_interface_with_feedback(gpu_lib, layout):
    w = _shared(W.gradient_goal(seed=102, n_worlds=_above_the_range(layout), steps=6), PER_WORLD[layout])
    gain = np.random.Generator(np.random.Philox(102)).normal(0.0, 0.01, size=(1, 4, 13)).astype(np.float32)
    n = 65 // PER_WORLD[layout] + 1
    w = _only_tail_counts(dataclasses.replace(w, gain=gain), n)
    _check_against_oracle(*_tail(w, _rollout_grads(w, 4), n))


@pytest.mark.parametrize("layout", ["lanes", "tiles"])
@pytest.mark.parametrize("form", ["linear", "reward", "squash", "policy 8", "policy 16", "policy 31"])
def test_identified(gpu_lib, layout, form):
    D, T = _above_the_range(layout), 6
    rng = np.random.Generator(np.random.Philox(103))
    if form == "squash":
        w = W.bptt_tracking(n_envs=D, steps=T)
        # (beside the reference: within rounding of it the reward's gradient has no direction)
        x0 = w.x0.copy()
        x0[:3] += rng.normal(0.0, 0.05, size=(3, D)).astype(np.float32)
        w = dataclasses.replace(w, x0=x0, gain=rng.normal(0.0, 0.5, size=(1, 4, 13)).astype(np.float32))
    elif form.startswith("policy"):
        hidden = int(form.split()[1])
        w = W.id_rollout_grad_mlp(seed=104, n_worlds=D, steps=T, hidden=hidden, out_scale=0.05)
    else:
        w = W.id_rollout_grad(seed=105, n_worlds=D, steps=T)
        if form == "reward":
            w = dataclasses.replace(w, reward=W.BPTT_REWARD)
    w = _shared(w, PER_WORLD[layout])
    n = 65 // PER_WORLD[layout] + 1
    w = _only_tail_counts(w, n)
    _check_against_oracle(*_tail(w, _grads(_sim(w), w, 4), n))
