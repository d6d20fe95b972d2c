"""The structured RK4 steps (position, velocity, rotor, thrust and attitude rows in
the closed form that RK4 gives them) against the FP64 oracle where they can go
wrong: stage offsets and angles beyond the short series, no thrust dynamics, no
renormalisation, steps long against the rotor lag."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from gpu_helpers import assert_states_close, dev
from test_gpu_parity import _check_against_oracle, _rollout_grads, _sim

pytestmark = pytest.mark.gpu


def _variant(w, kind):
    P = {k: v.copy() for k, v in w.params.items()}
    x0 = w.x0.copy()
    idm = w.model_per_world[0] == W.MODEL_ID
    if kind == "fast":          # stage offsets beyond 1/16 rad, large body rates
        x0[9:12] += np.float32(60.0) if idm else np.float32(8.0)
    elif kind == "wound":       # angles beyond 2^15 rad (one step: their spacing is 1/256 rad)
        x0[3:6] += np.float32(40000.0)
        w = dataclasses.replace(w, steps=1, cmds=w.cmds[:1] if w.cmds.ndim == 3 else w.cmds)
    elif kind == "direct":      # no thrust dynamics
        P["c_tau"][::2] = 0
    elif kind == "long":        # step of 20 ms: z = c h = 0.67
        w = dataclasses.replace(w, dt=float(np.float32(0.02)), steps=min(w.steps, 25),
                                cmds=w.cmds[:25] if w.cmds.ndim == 3 else w.cmds)
    elif kind == "free":        # quaternion not renormalised
        w = dataclasses.replace(w, renorm_q=0)
    return dataclasses.replace(w, params=P, x0=x0)


@pytest.mark.parametrize("kind", ["fast", "wound", "direct", "long"])
def test_identified(gpu_lib, kind):
    w = _variant(W.id_swarm(seed=71, n_worlds=5, n_drones=29, steps=60), kind)
    x = dev(w.x0)
    _sim(w).step_k(x, dev(w.cmds), w.steps)
    torch.cuda.synchronize()
    assert_states_close(x, O.simulate_held(w), w)
    if kind != "wound":
        w = _variant(W.id_rollout_grad(seed=72, n_worlds=67, steps=40), kind)
        _check_against_oracle(w, _rollout_grads(w, 8))


@pytest.mark.parametrize("kind", ["fast", "long", "free"])
@pytest.mark.parametrize("ctrl", ["rotor", "pid"])
def test_first_principles(gpu_lib, kind, ctrl):
    if ctrl == "rotor":
        w = _variant(W.fp_rotor_open_loop(seed=73, n_worlds=67, steps=40), kind)
        w = dataclasses.replace(w, dloss=np.ones(w.n_drones_total, np.float32))
    else:
        w = _variant(W.gradient_goal(seed=74, n_worlds=67, steps=25), kind)
    _check_against_oracle(w, _rollout_grads(w, 8))
    held = dataclasses.replace(w, cmds=np.ascontiguousarray(w.cmds[0]))
    x = dev(held.x0)
    _sim(held).step_k(x, dev(held.cmds), held.steps)
    torch.cuda.synchronize()
    assert_states_close(x, O.simulate_held(held), held)
