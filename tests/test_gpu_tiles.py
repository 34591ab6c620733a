"""The tile walk of the gather, scalar and collision kernels: every tile is visited once at the
tile counts where the XCD chunk size changes (single tiles, the doublings, full chunks)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


# about 13/256 tiles a cell: 1, 7, 63-65, 127-129 and 16384 tiles
@pytest.mark.parametrize("ncells", [2, 130, 1240, 1260, 1280, 2520, 2540, 322700])
def test_every_tile_once(gas, ncells):
    from oracle.oracle import Oracle
    from paper_2506_23917_amd.hs import Sim
    case = W.sod_1d(ncells=ncells, ppc_left=16, n_steady=0)
    sim = Sim(gas, case, precision="fp64", device="cuda:0")
    ora = Oracle(gas, case)
    ora.init_particles()
    sim.step(1)
    ora.step(1)
    g, o = sim.export_state(0), ora.get_state(0)
    assert np.array_equal(g["id"], o["id"]) and np.array_equal(g["cell"], o["cell"])
    # velocities: the bound of the other parity tests (rounding of the cell sums)
    scale = np.abs(o["v"]).max()
    assert np.abs(g["vel"] - o["v"]).max() <= 1e-12 * scale
    assert g["acc"][:, 0].sum() == len(g["id"])
