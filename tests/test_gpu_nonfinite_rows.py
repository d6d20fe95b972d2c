"""Drones with a non-finite input among others, four lanes a drone and one: what the input
does not reach stays finite and the same, whichever kernel the batch's size selects. Each
batch is run as it is and as the first drones of one above the four-lane range."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_mlp import _grads
from test_gpu_parity import _rollout_grads, _sim

pytestmark = pytest.mark.gpu

FEW, BAD = 40, 17   # drones of the small batch, the one with the input


def _pair(w, plant):
    """Results of the first FEW drones alone and within the whole batch."""
    x0, cmds = w.x0.copy(), w.cmds.copy()
    plant(x0, cmds)
    w = dataclasses.replace(w, x0=x0, cmds=cmds)
    run = (lambda v: _grads(_sim(v), v, 2)) if w.policy_hidden else (lambda v: _rollout_grads(v, 2))
    few, many = run(W.subset(w, list(range(FEW)))), run(w)
    return [(k, few[k][..., :FEW], many[k][..., :FEW]) for k in ("loss", "x", "g_cmds", "g_x0")]


def _check(results):
    for k, few, many in results:
        few, many = few.double().cpu(), many.double().cpu()
        assert torch.equal(torch.isfinite(few), torch.isfinite(many)), k
        few, many = few.nan_to_num(0.0, 0.0, 0.0), many.nan_to_num(0.0, 0.0, 0.0)
        per_drone = [v.reshape(-1, FEW).norm(dim=0) for v in (few - many, many)]
        assert (per_drone[0] <= 1e-3 * per_drone[1].clamp_min(1e-12)).all(), k


def _large():
    return 128 * torch.cuda.get_device_properties(0).multi_processor_count + 70


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("where", ["angle", "rate", "command"])
def test_yaw_does_not_reach_the_height(gpu_lib, where, value):
    """The identified model's vertical acceleration does not depend on the yaw angle."""
    w = dataclasses.replace(W.id_rollout_grad(seed=121, n_worlds=_large(), steps=3), gain=None, gain_index=None)

    def plant(x0, cmds):
        if where == "command":
            cmds[:, 2, BAD] = value
        else:
            x0[5 if where == "angle" else 11, BAD] = value

    results = _pair(w, plant)
    _check(results)
    x = dict((k, v) for k, v, _ in results)["x"]
    assert torch.isfinite(x[2, BAD]) and torch.isfinite(x[8, BAD])


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("row", [0, 1, 2, 3])
def test_commands_that_saturate_the_attitude_controller(gpu_lib, row, value):
    """The torque of an infinite angle or rate command saturates at the rotors' limits."""
    w = W.gradient_goal(seed=122, n_worlds=_large(), steps=3)

    def plant(x0, cmds):
        cmds[1, row, BAD] = value

    _check(_pair(w, plant))


@pytest.mark.parametrize("k", [1, 4])
def test_held_commands_that_saturate(gpu_lib, k):
    """The same on held steps, bit for bit the one-lane kernel's."""
    from gpu_helpers import dev

    w = W.gradient_goal(seed=123, n_worlds=FEW, steps=1)
    u = dev(w.cmds[0])
    for d, (row, value) in enumerate([(2, "inf"), (2, "-inf"), (0, "inf"), (1, "-inf"), (3, "inf"), (2, "nan")]):
        u[row, 3 * d] = float(value)
    out = []
    for wq in (0, 1):
        sim, x = _sim(w), dev(w.x0)
        sim.set_launch_config(workqueue=wq, tile=64)
        sim.step_k(x, u, k)
        torch.cuda.synchronize()
        out.append(x)
    assert torch.equal(torch.isfinite(out[0]), torch.isfinite(out[1]))
    assert torch.equal(out[0].nan_to_num(0.0, 0.0, 0.0), out[1].nan_to_num(0.0, 0.0, 0.0))
    # the yaw torque's sign is the command's: one pair of rotors speeds up, the other slows down
    turn = (out[0][13] - out[0][14])[[0, 3]]
    assert turn[0] * turn[1] < 0


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("row", [3, 5, 11])
def test_thrust_row_gradient_without_thrust_dynamics(gpu_lib, row, value):
    """c_tau = 0: the start's thrust row has no influence, so its gradient is zero whatever
    the drone's other gradients are."""
    w = W.id_rollout_grad(seed=124, n_worlds=_large(), steps=3)
    P = {k: v.copy() for k, v in w.params.items()}
    P["c_tau"][:] = 0
    w = dataclasses.replace(w, params=P, gain=None, gain_index=None)

    def plant(x0, cmds):
        x0[row, BAD] = value

    results = _pair(w, plant)
    _check(results)
    for k, few, many in results:
        if k == "g_x0":
            assert (few[12] == 0).all() and (many[12] == 0).all()


@pytest.mark.parametrize("hidden", [1, 8, 9, 13, 31])
@pytest.mark.parametrize("row", [0, 12])
@pytest.mark.parametrize("steps", [1, 3])
def test_policies_saturate_where_their_input_is_infinite(gpu_lib, hidden, row, steps):
    """tanh of an infinite activation is one, so the commands stay finite; widths that a
    quad's lanes pad with units of zero weights among them. (For one step: the compensated
    sums make an infinite position, or the velocity under an infinite thrust, NaN.)"""
    w = W.id_rollout_grad_mlp(seed=125, n_worlds=_large(), steps=steps, hidden=hidden, out_scale=0.05)

    def plant(x0, cmds):
        x0[row, BAD] = np.inf

    results = _pair(w, plant)
    _check(results)
    x = dict((k, v) for k, v, _ in results)["x"]
    assert steps > 1 or torch.isfinite(x[3:6, BAD]).all()
