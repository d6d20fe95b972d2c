"""The backward of a policy from a checkpoint buffer that was overwritten since its forward:
NaN in every requested output, the policy's gradient among them, and the sticky status."""
import pytest
import torch

import workloads as W
from gpu_helpers import dev
from paper_2606_01478_amd import binding as B
from test_gpu_mlp import _mlp, _obj
from test_gpu_parity import _sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["own sums", "records", "tiles"])
def test_every_output_is_nan(gpu_lib, kind):
    if kind == "tiles":
        w = _mlp(W.uneven_mixed_adjoint(seed=111, n_worlds=12, n_subset=8, steps=12, n_max=90), 8, 111)
    else:
        w = W.id_rollout_grad_mlp(seed=112, n_worlds=40, steps=12, hidden=8 if kind == "own sums" else 31)
    sim, T, K = _sim(w), w.steps, 5
    x0, cmds, obj = dev(w.x0), dev(w.cmds), _obj(w)
    ckpt = sim.ckpt_buffer(T, K)
    g = [torch.zeros_like(cmds), torch.zeros_like(x0), torch.zeros_like(dev(w.gain))]
    sim.rollout(x0, cmds, T, obj, K, ckpt=ckpt)
    sim.rollout_backward(x0, cmds, T, obj, K, ckpt, g_cmds=g[0], g_x0=g[1], g_gain=g[2])
    torch.cuda.synchronize()
    assert all(torch.isfinite(v).all() for v in g) and sim.last_error() == B.CF_OK
    ckpt[-4:] += 1.0
    sim.rollout_backward(x0, cmds, T, obj, K, ckpt, g_cmds=g[0], g_x0=g[1], g_gain=g[2])
    torch.cuda.synchronize()
    for v in g:
        assert torch.isnan(v).all()
    assert sim.last_error() == B.CF_ESTATE
