"""Gradients of many gains and policies, each summed over its own drones: gains that
outnumber a workgroup's components, several chunks of drones, gains that no drone has."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from test_gpu_mlp import _grads
from test_gpu_parity import _check_against_oracle, _rollout_grads, _sim

pytestmark = pytest.mark.gpu


def _with_gains(w, G, index):
    rng = np.random.Generator(np.random.Philox(G))
    return dataclasses.replace(w, gain=rng.normal(0.0, 0.01, size=(G, 4, 13)).astype(np.float32),
                               gain_index=np.asarray(index, np.int32))


@pytest.mark.parametrize("G", [16, 17, 67])
def test_against_the_oracle(gpu_lib, G):
    w = W.id_rollout_grad(seed=71, n_worlds=90, steps=8)
    w = _with_gains(w, G, np.arange(90) * 7 % G)
    _check_against_oracle(w, _rollout_grads(w, 5))


@pytest.mark.parametrize("n", [16384, 16385, 40000])
@pytest.mark.parametrize("G", [16, 17, 300])
def test_each_gain_sums_its_own_drones(gpu_lib, n, G):
    """One shared gain and a loss of gain k's drones alone give the gradient of gain k."""
    w = W.id_rollout_grad(seed=72, n_worlds=n, steps=2)
    index = np.random.Generator(np.random.Philox(n)).integers(0, G - 1, size=n)   # none has the last
    many = dataclasses.replace(w, gain=np.repeat(w.gain, G, axis=0), gain_index=index.astype(np.int32))
    g = _rollout_grads(many, 2)["g_gain"]
    assert (g[G - 1] == 0).all()
    for k in (0, G // 2, G - 2):
        one = dataclasses.replace(w, dloss=(index == k).astype(np.float32))
        ref = _rollout_grads(one, 2)["g_gain"][0]
        # sums of at most 40000 / 15 terms in binary32, in another order: 16 serial additions
        # a thread and trees of 10 levels round by less than 2^-19 of the terms' magnitudes,
        # which exceed the sum's by less than a factor of 100 (commands of 2 % noise)
        assert ((g[k] - ref).abs().max() <= 2e-4 * ref.abs().max()).item(), k


def test_policies_against_the_oracle(gpu_lib):
    """20 policies of width 8: 220 components, each drone's own sums (12 steps)."""
    w = W.id_rollout_grad_mlp(seed=73, n_worlds=50, steps=12, hidden=8, out_scale=0.05)
    rng = np.random.Generator(np.random.Philox(73))
    w = dataclasses.replace(w, gain=W.mlp_policy_params(rng, 20, 8, 0.05),
                            gain_index=(np.arange(50) * 3 % 20).astype(np.int32))
    _check_against_oracle(w, _grads(_sim(w), w, 5))
