"""Elite selection and weighted mean of the sampled-rollout controller at the edges of
its parts: wave-sized and odd elite counts, the sampled threshold (all samples, a
sample of them) and its fallback, plans shorter and longer than one block of steps."""
import numpy as np
import pytest

from test_gpu_mppi import _check_step, _jittered_mean, _make, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,n_e", [(1, 1), (65, 64), (2047, 65), (2049, 129), (6000, 2048), (6000, 2049), (9001, 90)])
@pytest.mark.parametrize("H", [1, 33])
def test_elites_and_mean(gpu_lib, N, n_e, H):
    w, P, mean0, sim, mp = _make(C=2, N=N, H=H, n_elite=n_e)
    mean = _jittered_mean(mean0, 3)
    got = _run(w, P, mp, mean, 1, 2)
    rng = np.random.default_rng(5)
    some = (rng.integers(0, 2, 64), rng.integers(0, N, 64))
    _check_step(w, P, mean, 1, 2, got, sample=some)
