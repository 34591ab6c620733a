"""The tile walk where tiles are dealt out in parts (four up to 512 tiles, two up to 2048, one above, in
batches of up to 3072 tiles of capacity): the walk goes over tiles times parts, in chunks that double at
128, 256, .. 4096 of these.  And the tile kernel's NTC beyond the candidates that a claim word numbers."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncells,tiles", [(610, 31), (630, 32), (648, 33), (5020, 255), (5040, 256), (5060, 257),
                                          (10062, 511), (10082, 512), (10102, 513), (20144, 1023), (20164, 1024),
                                          (20184, 1025), (40310, 2047), (40328, 2048), (40348, 2049), (49230, 2500)])
def test_every_part_once(gas, ncells, tiles):
    from oracle.oracle import Oracle
    from paper_2506_23917_amd.hs import Sim
    case = W.sod_1d(ncells=ncells, ppc_left=16, n_steady=0)
    assert (case["capacity"] + 4 * ncells) // 256 + 1 <= 3072
    sim = Sim(gas, case, precision="fp64", device="cuda:0")
    ora = Oracle(gas, case)
    ora.init_particles()
    sim.step(1)
    ora.step(1)
    g, o = sim.export_state(0), ora.get_state(0)
    assert -(-(len(g["id"]) + 4 * ncells) // 256) == tiles
    assert np.array_equal(g["id"], o["id"]) and np.array_equal(g["cell"], o["cell"])
    # velocities: the bound of the other parity tests (rounding of the cell sums)
    assert np.abs(g["vel"] - o["v"]).max() <= 1e-12 * np.abs(o["v"]).max()
    assert np.array_equal(g["acc"][:, 0], np.bincount(g["cell"], minlength=ncells))


# one cell (no parts of it) with more candidates than a claim word's 16 bits: they are numbered anew
# from the lowest one still held, once and more often
@pytest.mark.parametrize("ppc,rate", [(192, 240.0), (192, 400.0), (60, 2500.0)])
def test_ntc_window_renumbered(gas, ppc, rate):
    from oracle.oracle import Oracle
    from paper_2506_23917_amd.hs import Sim
    case = W.relax_0d(ncells=1, ppc=ppc)
    case["dt_over_tau"] = np.full(1, 0.9)                # all DSMC
    v, cell, ids = W.relax_0d_state(case, ppc=ppc)
    ora = Oracle(gas, case, trace=True)
    ora.set_state(0, None, v, cell, ids, len(ids), 0)
    sigc = ora.get_cells(0)["sigc_max"] * rate           # more candidates, each less often accepted
    ora.set_cells(0, sigc_max=sigc)
    sim = Sim(gas, case, precision="fp64", trace=True, no_particles=True, device="cuda:0")
    sim.import_state(0, dict(pos=np.zeros((len(ids), 3)), vel=v, cell=cell, id=ids, next_id=len(ids), step=0,
                             sigc_max=sigc))
    sim.step(1)
    ora.step(1)
    tg, to = sim.trace(0), ora.trace(0)
    assert to["ncol"].max() > 0x10000
    for f in ("n", "ncol", "nacc", "acc_hash"):
        assert np.array_equal(tg[f], to[f]), f
    g, o = sim.export_state(0), ora.get_state(0)
    assert np.abs(g["vel"] - o["v"]).max() <= 1e-12 * np.abs(o["v"]).max()
