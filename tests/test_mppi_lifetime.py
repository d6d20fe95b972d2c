"""A controller set and its simulation closed or collected in either order: each library
object is destroyed once, the set before the handle it was made on (recorded calls of a
stand-in library; no GPU needed)."""
import gc
from ctypes import c_void_p

import pytest

from paper_2606_01478_amd import binding as B


class _Library:
    def __init__(self):
        self.calls = []

    def cf_mppi_create(self, h, d, out):
        out._obj.value = 0x20
        return B.CF_OK

    def cf_mppi_destroy(self, m):
        self.calls.append(("set", m.value))
        return B.CF_OK

    def cf_mppi_step(self, m, *a):
        self.calls.append(("step", m.value))
        return B.CF_OK if m.value else B.CF_EINVAL

    def cf_destroy(self, h):
        self.calls.append(("sim", h.value))
        return B.CF_OK


def _pair():
    lib = _Library()
    sim = B.Sim.__new__(B.Sim)
    sim._lib, sim._h, sim._sets, sim.S = lib, c_void_p(0x10), [], 13
    P = dict(n_controllers=1, n_samples=8, horizon=4, n_elite=2, sigma=[0.1] * 4, beta=0.5, u_lo=[-1.0] * 4,
             u_hi=[1.0] * 4, u_ref=[0.0] * 4, r_u=[0.1] * 4, goal=[0.0] * 3, q_p=1.0, q_v=0.1, w_obs=1.0, seed=3)
    P["lambda"] = 1.0
    return lib, sim, B.Mppi(sim, P)


@pytest.mark.parametrize("order", ["sim first", "set first", "dropped", "cycle"])
def test_destroyed_once_and_in_order(order):
    lib, sim, mp = _pair()
    if order == "sim first":
        sim.close()
        with pytest.raises(Exception):
            mp.step(None, None, 0, 0)
        lib.calls = [c for c in lib.calls if c[0] != "step"]
        mp.close()
    elif order == "set first":
        mp.close()
        mp.close()
        sim.close()
    elif order == "cycle":
        sim._other, mp._other = mp, sim   # only the cyclic collector frees them
    sim.close() if order.endswith("first") else None
    del sim, mp
    gc.collect()
    assert lib.calls == [("set", 0x20), ("sim", 0x10)]
