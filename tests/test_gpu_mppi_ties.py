"""Elites among costs that hardly differ: spreads of a few units in the last place, ties
beyond the candidate list, infinite costs, with the sampled threshold taken to the last
bit and the index."""
import numpy as np
import pytest

from oracle import mppi as OM
from test_gpu_mppi import _jittered_mean, _make, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,n_e", [(4100, 41), (20000, 200), (20000, 2048), (50001, 1)])
@pytest.mark.parametrize("scale", [1e-2, 1e-3, 1e-4, 1e-5, 0.0])
def test_elites_of_close_costs(gpu_lib, N, n_e, scale):
    sigma = [s * scale for s in (0.15, 0.15, 0.3, 0.05)]
    w, P, mean0, sim, mp = _make(C=2, N=N, H=5, n_elite=n_e, sigma=sigma)
    got = _run(w, P, mp, _jittered_mean(mean0, 6), 0, 3)
    assert np.array_equal(got["el"], OM.select_elites(got["cost"].astype(np.float64), n_e))
    if scale == 0.0:
        assert np.array_equal(got["el"][0], np.arange(n_e))


def test_elites_of_infinite_costs(gpu_lib):
    """Commands that overflow the cost: every sample's is infinite, the elites are the first."""
    w, P, mean0, sim, mp = _make(C=1, N=9000, H=3, n_elite=90, q_p=3e38)
    got = _run(w, P, mp, mean0[:1], 0, 1)
    assert np.isinf(got["cost"]).all()
    assert np.array_equal(got["el"][0], np.arange(90))
