"""The allocation-free backward of a policy refuses what its contract says, whichever
layout of the weight-gradient sums the batch's kernels use."""
import ctypes
import dataclasses

import pytest
import torch

import workloads as W
from gpu_helpers import dev
from paper_2606_01478_amd import binding as B
from test_gpu_mlp import _grads, _obj
from test_gpu_parity import _sim

pytestmark = pytest.mark.gpu


def test_refused_by_the_records_that_the_contract_counts(gpu_lib):
    """(17 + 4 H) T D floats of records, H = 8: 5000 drones over 60 steps fit in the 64 MiB,
    over 80 they do not."""
    w = W.id_rollout_grad_mlp(seed=41, n_worlds=5000, steps=80, hidden=8, out_scale=0.05)
    sim, x0 = _sim(w), dev(w.x0)
    T, K = w.steps, 4
    cmds, obj = dev(w.cmds), _obj(w)
    ckpt = sim.ckpt_buffer(T, K)
    sim.rollout(x0, cmds, T, obj, K, ckpt=ckpt)
    g = torch.full_like(cmds, 7.0)
    gg = torch.full_like(dev(w.gain), 7.0)
    st = sim._lib.cf_rollout_backward_noalloc(sim._h, x0.data_ptr(), cmds.data_ptr(), T, ctypes.byref(obj), K,
                                              ckpt.data_ptr(), None, g.data_ptr(), None, gg.data_ptr())
    torch.cuda.synchronize()
    assert st == B.CF_EINVAL
    assert (g == 7.0).all() and (gg == 7.0).all()
    w = dataclasses.replace(w, steps=60, cmds=w.cmds[:60].copy())
    ref, got = _grads(sim, w, K), _grads(sim, w, K, noalloc=True)
    for k in ("g_cmds", "g_x0", "g_gain"):
        assert torch.equal(ref[k], got[k]), k
