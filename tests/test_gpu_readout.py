"""hs_sample_moments into arrays of the caller's: one block, separate arrays, some of them, below
and above the staging memory's size, on a sim with and without it; all give the same bytes."""
import ctypes as C

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _read(sim, mode, want):
    nc = sim.num_cells(0)
    out = dict(n=np.full(nc, -1.0), u=np.full((nc, 3), -1.0), T=np.full(nc, -1.0), q=np.full((nc, 3), -1.0))
    ptr = [out[k].ctypes.data_as(C.POINTER(C.c_double)) if k in want else None for k in ("n", "u", "T", "q")]
    ns = C.c_int64()
    assert sim.L.hs_sample_moments(sim.h, 0, mode, *ptr, C.byref(ns)) == 0
    return out, ns.value


@pytest.mark.parametrize("nx,static", [(40, False), (40, True), (420, False)])
def test_sample_moments_any_arrays(gas, nx, static):
    from paper_2506_23917_amd.hs import Sim
    case = W.cylinder_2d(nx=nx, ny=nx // 4 * 3, ppc=4, n_steady=0)
    sim = Sim(gas, case, precision="fp32", static_scratch=static, device="cuda:0")
    sim.step(3)
    for mode in (0, 1):
        full = sim.sample_moments(0, mode)
        assert full["n_samples"] == 3 and full["n"].max() > 0 and full["q"].any()
        for want in ("nuTq", "u", "nT", "q", ""):
            part, ns = _read(sim, mode, want)
            assert ns == 3
            for k in "nuTq":
                if k in want:
                    assert np.array_equal(part[k], full[k])
                else:
                    assert np.all(part[k] == -1.0)
