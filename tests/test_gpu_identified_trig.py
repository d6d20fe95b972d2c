"""The identified model's sines and cosines step by step, without a tolerance: a drone
whose velocity is exactly zero after its first step (it starts with minus that step's
increment) has the second step's increment alone as its velocity after two, which must
be, bit for bit, what a run started at its second state gives."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads as W
from gpu_helpers import dev
from paper_2606_01478_amd import binding as B
from test_gpu_mppi import _make
from test_gpu_parity import _sim

pytestmark = pytest.mark.gpu

ROWS = slice(3, 13)   # angles, velocity, rates, thrust (positions integrate other velocities)


def _cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


def _two_steps(w, advance):
    """advance(x, t, n): n steps of x from step t. Returns the states after two steps and
    after the second alone, identified drones' columns."""
    world = np.repeat(np.arange(w.n_worlds), w.drones_per_world)
    idm = torch.as_tensor(w.model_per_world[world] == W.MODEL_ID, device="cuda")
    rng = np.random.Generator(np.random.Philox(w.n_drones_total))
    x0 = dev(w.x0)
    kick = dev(rng.uniform(-1.0, 1.0, size=(6, w.n_drones_total)))
    x0[3:6] += torch.where(idm, 0.5 * kick[:3], 0.0)     # angles and rates of all sizes
    x0[9:12] += torch.where(idm, 2.0 * kick[3:], 0.0)
    x0[6:9] = torch.where(idm, 0.0, x0[6:9])
    x1 = advance(x0, 0, 1)
    back = x0.clone()
    back[6:9] = torch.where(idm, -x1[6:9], x0[6:9])
    two = advance(back, 0, 2)
    x1[6:9] = torch.where(idm, 0.0, x1[6:9])
    one = advance(x1, 1, 1)
    torch.cuda.synchronize()
    return two[ROWS][:, idm], one[ROWS][:, idm]


def _workload(layout, integ):
    if layout == "four lanes":
        w = W.id_swarm(seed=61, n_worlds=5, n_drones=17, steps=2)
    elif layout == "lanes":
        n = 128 * _cus() + 70
        w = W.id_rollout_grad(seed=62, n_worlds=n, steps=2)
    elif layout == "tiles":
        w = W.id_swarm(seed=63, n_worlds=2 * _cus() + 3, n_drones=65, steps=2)
    else:
        w = W.uneven_mixed(seed=64, n_worlds=24, steps=2, n_max=90)
    if w.cmds.ndim == 2:
        w = dataclasses.replace(w, cmds=np.ascontiguousarray(np.stack([w.cmds, 0.9 * w.cmds])))
    return dataclasses.replace(w, integrator=integ)


@pytest.mark.parametrize("integ", [W.INTEG_RK4, W.INTEG_EULER])
@pytest.mark.parametrize("layout", ["four lanes", "lanes", "tiles", "mixed"])
def test_rollouts_evaluate_the_start_angles_at_every_step(gpu_lib, layout, integ):
    w = _workload(layout, integ)
    sim, cmds = _sim(w), dev(w.cmds)

    def advance(x, t, n):
        out = torch.empty_like(x)
        sim.rollout(x, cmds[t:t + n].contiguous(), n, None, 50, x_T=out)
        return out

    two, one = _two_steps(w, advance)
    assert torch.equal(two, one), int((two != one).sum())


def test_sampled_rollouts_evaluate_the_start_angles_at_every_step(gpu_lib):
    """Cost of one noise-free sample, |v|^2 after one command of two substeps."""
    over = dict(C=1, N=1, H=1, model=W.MODEL_ID, n_elite=1, sigma=[0.0] * 4, r_u=[0.0] * 4, q_p=0.0, q_v=1.0,
                w_obs=0.0)
    w, _, mean0, sim, pair = _make(substeps=2, **over)
    single = B.Mppi(sim, dict(_make(substeps=1, **over)[1]))
    rng = np.random.Generator(np.random.Philox(65))
    state = torch.empty(sim.S, 1, device="cuda")

    def cost(m, x, mean):
        j = torch.empty((1, 1), device="cuda")
        m.step(x.reshape(-1).contiguous(), mean.clone(), 0, 0, cost=j)
        torch.cuda.synchronize()
        return float(j)

    different = 0
    for _ in range(64):
        x = w.x0.copy()
        x[3:6, 0] += rng.uniform(-0.5, 0.5, 3).astype(np.float32)
        x[9:12, 0] += rng.uniform(-2.0, 2.0, 3).astype(np.float32)
        x[6:9] = 0
        mean = mean0.copy()
        mean[0, 0, :3] = rng.uniform(-0.3, 0.3, 3)
        u = dev(np.ascontiguousarray(mean[0, 0].reshape(1, 4, 1)))
        x0 = dev(x)
        sim.rollout(x0, u, 1, None, 50, x_T=state)
        back = x0.clone()
        back[6:9] = -state[6:9]
        rest = state.clone()
        rest[6:9] = 0
        different += cost(pair, back, dev(mean)) != cost(single, rest, dev(mean))
    assert different == 0

