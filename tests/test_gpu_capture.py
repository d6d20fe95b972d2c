"""Calls recorded into a graph after one earlier call of the kind on the handle, whatever
lane mapping each takes: they allocate nothing, and every replay equals the direct call."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads as W
from gpu_helpers import dev
from test_gpu_mlp import _obj
from test_gpu_parity import _sim

pytestmark = pytest.mark.gpu


def _captured(call):
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            call()
    torch.cuda.current_stream().wait_stream(s)
    return g


@pytest.mark.parametrize("first,then", [(4, 4), (4, 1)])
def test_steps_after_a_call_of_another_length(gpu_lib, first, then):
    """100 worlds of 50 drones: few enough for four lanes a drone over several steps, too
    many for a single one, which goes in tiles."""
    w = W.id_swarm(seed=31, n_worlds=100, n_drones=50, steps=4)
    u, x, y = dev(w.cmds), dev(w.x0), dev(w.x0)
    sim, ref = _sim(w), _sim(w)
    sim.step_k(x.clone(), u, first)
    torch.cuda.synchronize()
    g = _captured(lambda: sim.step_k(x, u, then))
    for _ in range(3):
        g.replay()
        ref.step_k(y, u, then)
        torch.cuda.synchronize()
        assert torch.equal(x, y)


@pytest.mark.parametrize("steps", [12, 3])
def test_noalloc_backward_of_a_policy(gpu_lib, steps):
    """Two worlds of 40 identified drones with a policy each: over 3 steps the backward goes
    in tiles, though the forward takes four lanes a drone."""
    w = W.id_swarm(seed=32, n_worlds=2, n_drones=40, steps=steps)
    rng = np.random.Generator(np.random.Philox(9))
    w = dataclasses.replace(w, cmds=np.ascontiguousarray(np.tile(w.cmds, (steps, 1, 1))),
                            gain=W.mlp_policy_params(rng, 2, 8, 0.05), gain_index=np.arange(2, dtype=np.int32),
                            policy_hidden=8, ref_amp=1.0, ref_period=4.0, w_u=1e-3)
    sim = _sim(w)
    x0, cmds, obj = dev(w.x0), dev(w.cmds), _obj(w)
    ckpt = sim.ckpt_buffer(steps, 2)
    sim.rollout(x0, cmds, steps, obj, 2, ckpt=ckpt)
    torch.cuda.synchronize()
    got = dict(g_cmds=torch.empty_like(cmds), g_x0=torch.empty_like(x0), g_gain=torch.empty_like(dev(w.gain)))
    g = _captured(lambda: sim.rollout_backward_noalloc(x0, cmds, steps, obj, 2, ckpt, **got))
    ref = {k: torch.empty_like(v) for k, v in got.items()}
    for _ in range(3):
        for v in got.values():
            v.fill_(7.0)
        g.replay()
        torch.cuda.synchronize()
        sim.rollout_backward(x0, cmds, steps, obj, 2, ckpt, **ref)
        torch.cuda.synchronize()
        for k in got:
            assert torch.isfinite(ref[k]).all() and torch.equal(got[k], ref[k]), k
