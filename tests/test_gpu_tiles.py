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


# queue lengths around a wave's 64 draws, single draws, whole tiles; the last particle of every
# cell is fast, so the heat flux and with it the number of attempts (up to the cap) is large
@pytest.mark.parametrize("ncells,ppc", [(1, 3), (1, 33), (1, 64), (1, 65), (1, 192), (2, 100), (60, 3), (21, 8)])
def test_shakhov_draw_queue(gas, ncells, ppc):
    from oracle.oracle import Oracle
    from paper_2506_23917_amd.hs import Sim
    case = W.relax_0d(ncells=ncells, ppc=ppc)
    case["dt_over_tau"] = 10.0 ** np.linspace(2, -0.5, ncells)
    v, cell, ids = W.relax_0d_state(case, ppc=ppc)
    v[ppc - 1::ppc] *= 30.0
    ora = Oracle(gas, case, trace=True)
    ora.set_state(0, None, v, cell, ids, len(ids), 0)
    cells = ora.get_cells(0)
    sim = Sim(gas, case, precision="fp64", trace=True, no_particles=True, device="cuda:0")
    sim.import_state(0, dict(pos=np.zeros((len(ids), 3)), vel=v, cell=cell, id=ids, next_id=len(ids), step=0,
                             sigc_max=cells["sigc_max"]))
    attempts = 0
    for _ in range(4):
        sim.step(1)
        ora.step(1)
        tg, to = sim.trace(0), ora.trace(0)
        for f in ("n", "ncol", "nacc", "nrelax", "ar_attempts", "ar_cap", "acc_hash"):
            assert np.array_equal(tg[f], to[f]), f
        attempts += int((to["ar_attempts"] - to["nrelax"]).sum())
    assert attempts > 0
    g, o = sim.export_state(0), ora.get_state(0)
    assert np.abs(g["vel"] - o["v"]).max() <= 1e-12 * np.abs(o["v"]).max()
    assert sim.counters(0) == ora.counters(0)


# cells of one to many source blocks of 64 and their edges, still particles (one run a cell) to
# flights over several cells (many short runs)
@pytest.mark.parametrize("ncells,ppc", [(700, 1), (300, 5), (9, 63), (9, 64), (9, 65), (40, 170)])
@pytest.mark.parametrize("speed", [0.0, 300.0, 4000.0])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_stable_order_by_runs(gas, ncells, ppc, speed, precision):
    from paper_2506_23917_amd.hs import Sim
    rng = np.random.default_rng(ncells * ppc)
    case = W.sod_1d(ncells=ncells, ppc_left=2)
    case.update(h=(1.0, 1.0, 1.0), regions=[], F_N=1.0, dt_G=1e-3, capacity=ncells * ppc + 64)
    m = ncells * ppc
    cell = np.sort(rng.integers(0, ncells, m).astype(np.int32))
    pos = np.zeros((m, 3))
    pos[:, 0] = rng.random(m)
    vel = np.zeros((m, 3))
    vel[:, 0] = speed * rng.standard_normal(m)
    ids = rng.permutation(m).astype(np.int64)
    sim = Sim(gas, case, precision=precision, no_particles=True, device="cuda:0")
    sim.import_state(0, dict(pos=pos, vel=vel, cell=cell, id=ids, next_id=m, step=0,
                             sigc_max=np.full(ncells, 1e-16)))
    for _ in range(2):
        before = sim.export_state(0)
        sim.step(1)
        after = sim.export_state(0)
        # the cells the particles went to, then the stable order of the particles before the step
        where = dict(zip(after["id"], after["cell"]))
        new = np.array([where[i] for i in before["id"]])
        assert np.array_equal(after["id"], before["id"][np.argsort(new, kind="stable")])


# sims made one after the other and alive together (each picks its side stream), and one replaying
# a graph, whose dense cells run beside the tiles
@pytest.mark.parametrize("n", [1, 6])
def test_sims_side_by_side(gas, n):
    from paper_2506_23917_amd.hs import Sim
    case = W.sod_1d(ncells=40, ppc_left=600, n_steady=0)
    sims = [Sim(gas, case, precision="fp64", device="cuda:0", graph=k == 5) for k in range(n + 1)]
    for s in sims:
        s.step(4)
    first = sims[0].export_state(0)
    for s in sims[1:]:
        st = s.export_state(0)
        assert np.array_equal(st["id"], first["id"]) and np.array_equal(st["vel"], first["vel"])
        assert np.array_equal(st["acc"], first["acc"])


# the block kernel's stable order and draw queue on sorted cells of every class: tubes (no two runs
# of a block in a cell) and a stream that reflects at a cylinder (such runs)
@pytest.mark.parametrize("ppc", [300, 520, 1100, 2500, 4500])
def test_dense_cells_sorted(gas, ppc):
    from oracle.oracle import Oracle
    from paper_2506_23917_amd.hs import Sim
    cases = [W.sod_1d(seed=5, ncells=6, ppc_left=ppc, n_steady=0)]
    body = W.cylinder_2d(nx=16, ny=12, ppc=ppc, seed=6, n_steady=0)
    body.update(regions=[((1.5, 2.0, 0.0, 2.1, 4.0, 1.0), body["inflow"])], bc=("outflow",) * 6, capacity=16 * ppc)
    cases.append(body)
    sim = Sim(gas, cases, precision="fp64", device="cuda:0")
    ora = Oracle(gas, cases)
    ora.init_particles()
    for _ in range(2):
        sim.step(1)
        ora.step(1)
    for k in range(2):
        g, o = sim.export_state(k), ora.get_state(k)
        assert np.array_equal(g["id"], o["id"]) and np.array_equal(g["cell"], o["cell"])
        assert np.abs(g["vel"] - o["v"]).max() <= 1e-12 * np.abs(o["v"]).max()
        assert sim.counters(k) == ora.counters(k)
    assert sim.counters(1)["wall_hits"] > 0


# cell counts around the scan's block size (4096) and the last one scanned without block sums
@pytest.mark.parametrize("ncells", [1, 3, 4094, 4096, 4098, 32766, 32768, 32770])
@pytest.mark.parametrize("ncases", [1, 3])
def test_scan_sizes(gas, ncells, ncases):
    from oracle.oracle import Oracle
    from paper_2506_23917_amd.hs import Sim
    cases = [W.sod_1d(seed=3 + k, ncells=max(ncells, 1) if k == 0 else 2 + 4 * k, ppc_left=8, n_steady=0)
             for k in range(ncases)]
    sim = Sim(gas, cases, precision="fp64", device="cuda:0")
    ora = Oracle(gas, cases)
    ora.init_particles()
    sim.step(2)
    ora.step(2)
    for k in range(ncases):
        g, o = sim.export_state(k), ora.get_state(k)
        assert np.array_equal(g["id"], o["id"]) and np.array_equal(g["cell"], o["cell"])
        assert np.array_equal(g["acc"][:, 0], np.asarray(ora.get_cells(k)["acc"])[:, 0])


# inflow faces counted in the scan or apart, and lanes per face from 8 to 64 (a few to hundreds of
# new particles a face and step)
@pytest.mark.parametrize("ny,ppc", [(6, 4), (6, 60), (12, 900), (4095, 2), (4096, 2), (4097, 2), (9000, 2)])
def test_injection_sizes(gas, ny, ppc):
    from oracle.oracle import Oracle
    from paper_2506_23917_amd.hs import Sim
    st = dict(n=W.N_INF, u=(W.U_INF, 0.0, 0.0), T=W.T_INF)
    case = W.cylinder_2d(nx=16, ny=12, ppc=8)
    case.update(nx=2, ny=ny, h=(0.1, 0.1, 1.0), bc=("inflow",) + ("outflow",) * 5, body="none", n_surf=0, regions=[],
                F_N=W.N_INF * 0.01 / ppc, dt_G=0.09 / W.U_INF, inflow=st, capacity=3 * ny * ppc + 64)
    sim = Sim(gas, case, precision="fp64", device="cuda:0")
    ora = Oracle(gas, case)
    ora.init_particles()
    sim.step(2)
    ora.step(2)
    g, o = sim.export_state(0), ora.get_state(0)
    assert len(g["id"]) > ny * ppc // 2 and np.array_equal(g["id"], o["id"]) and np.array_equal(g["cell"], o["cell"])
    assert np.abs(g["vel"] - o["v"]).max() <= 1e-12 * np.abs(o["v"]).max()
    assert sim.counters(0) == ora.counters(0)


# the NTC's candidate window: fewer candidates than lanes, about as many, and thousands on a few
# particles (long chains of candidates sharing a particle), alone and in tiles of several cells
@pytest.mark.parametrize("ncells,ppc,rate", [(1, 2, 1.0), (1, 2, 2000.0), (1, 60, 0.5), (1, 192, 1.0), (5, 40, 30.0),
                                             (30, 4, 300.0), (2, 100, 100.0)])
def test_ntc_window(gas, ncells, ppc, rate):
    from oracle.oracle import Oracle
    from paper_2506_23917_amd.hs import Sim
    case = W.relax_0d(ncells=ncells, ppc=ppc)
    case["dt_over_tau"] = np.full(ncells, 0.9)           # all DSMC
    v, cell, ids = W.relax_0d_state(case, ppc=ppc)
    ora = Oracle(gas, case, trace=True)
    ora.set_state(0, None, v, cell, ids, len(ids), 0)
    sigc = ora.get_cells(0)["sigc_max"] * rate           # more candidates, each less often accepted
    ora.set_cells(0, sigc_max=sigc)
    sim = Sim(gas, case, precision="fp64", trace=True, no_particles=True, device="cuda:0")
    sim.import_state(0, dict(pos=np.zeros((len(ids), 3)), vel=v, cell=cell, id=ids, next_id=len(ids), step=0,
                             sigc_max=sigc))
    for _ in range(2):
        sim.step(1)
        ora.step(1)
        tg, to = sim.trace(0), ora.trace(0)
        for f in ("n", "ncol", "nacc", "acc_hash"):
            assert np.array_equal(tg[f], to[f]), f
    g, o = sim.export_state(0), ora.get_state(0)
    assert np.abs(g["vel"] - o["v"]).max() <= 1e-12 * np.abs(o["v"]).max()


# the block kernel's candidate window: few candidates, thousands, and more than one claim word counts
@pytest.mark.parametrize("ppc,rate", [(200, 0.01), (200, 30.0), (700, 20.0), (5000, 3.0), (460, 700.0)])
def test_ntc_window_dense(gas, ppc, rate):
    from oracle.oracle import Oracle
    from paper_2506_23917_amd.hs import Sim
    case = W.relax_0d(ncells=2, ppc=ppc)
    case["dt_over_tau"] = np.array([0.9, 0.3])           # all DSMC
    v, cell, ids = W.relax_0d_state(case, ppc=ppc)
    ora = Oracle(gas, case, trace=True)
    ora.set_state(0, None, v, cell, ids, len(ids), 0)
    sigc = ora.get_cells(0)["sigc_max"] * rate
    ora.set_cells(0, sigc_max=sigc)
    sim = Sim(gas, case, precision="fp64", trace=True, no_particles=True, device="cuda:0")
    sim.import_state(0, dict(pos=np.zeros((len(ids), 3)), vel=v, cell=cell, id=ids, next_id=len(ids), step=0,
                             sigc_max=sigc))
    sim.step(1)
    ora.step(1)
    tg, to = sim.trace(0), ora.trace(0)
    for f in ("n", "ncol", "nacc", "acc_hash"):
        assert np.array_equal(tg[f], to[f]), f
    if rate > 500:
        assert to["ncol"].max() > 65536
    g, o = sim.export_state(0), ora.get_state(0)
    assert np.abs(g["vel"] - o["v"]).max() <= 1e-12 * np.abs(o["v"]).max()


# many tiles a block of the scalars kernel: batches of one case and over the edges of cases, of few
# and many cells a tile, with empty, dense and heat-carrying cells between
@pytest.mark.parametrize("blocks", [8, 24])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_scalar_batches(gas, blocks, precision):
    from paper_2506_23917_amd.hs import Sim
    cases = [W.sod_1d(seed=5 + k, ncells=nc, ppc_left=ppc, n_steady=0)
             for k, (nc, ppc) in enumerate([(40, 8), (6, 160), (90, 24), (4, 300), (200, 2), (2, 8)])]
    cases[2]["adapt_dt"] = True
    ref = Sim(gas, cases, precision=precision, trace=True, device="cuda:0")
    sim = Sim(gas, cases, precision=precision, trace=True, device="cuda:0")
    sim.set_grid("scalars", blocks)
    for s in (ref, sim):
        s.step(4)
    for k in range(len(cases)):
        a, b = ref.export_state(k), sim.export_state(k)
        for f in ("id", "cell", "pos", "vel", "acc"):
            assert np.array_equal(a[f], b[f]), (k, f)
        assert ref.trace(k).tobytes() == sim.trace(k).tobytes()
        assert ref.counters(k) == sim.counters(k) and ref.step_dt(k) == sim.step_dt(k)


# tiles dealt out in four and two parts (up to 512 and 2048 tiles) and whole: the same bits for a case
# in batches of each size, with few and many cells a tile, empty, dense and heat-carrying cells
@pytest.mark.parametrize("filler", [1500, 9000])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_tile_parts(gas, filler, precision):
    from paper_2506_23917_amd.hs import Sim
    cases = [W.sod_1d(seed=5 + k, ncells=nc, ppc_left=ppc, n_steady=1)
             for k, (nc, ppc) in enumerate([(40, 8), (6, 160), (90, 24), (4, 300), (200, 2), (2, 8)])]
    cases[2]["adapt_dt"] = True
    ref = Sim(gas, cases + [W.sod_1d(seed=99, ncells=filler)], precision=precision, trace=True, device="cuda:0")
    sim = Sim(gas, cases, precision=precision, trace=True, device="cuda:0")
    for s in (ref, sim):
        s.step(4)
    for k in range(len(cases)):
        a, b = ref.export_state(k), sim.export_state(k)
        for f in ("id", "cell", "pos", "vel", "acc"):
            assert np.array_equal(a[f], b[f]), (k, f)
        assert ref.trace(k).tobytes() == sim.trace(k).tobytes()
        assert ref.counters(k) == sim.counters(k) and ref.step_dt(k) == sim.step_dt(k)
