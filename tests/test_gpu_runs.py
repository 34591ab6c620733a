"""Particles that come to their cells from all over the domain: the sorted order of a cell is found from
its runs of sources where these are few, and by counting or sorting where they are many (flights over
many cells).  Both keep the stable order, and many runs cost no multiple of few."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _flights(nx, ny, per, width, body=False, seed=3):
    """One step's flights: each particle to a point up to width / 2 cells away (periodically), or anywhere
    (width 0), in an open box of unit cells, around a cylinder if `body`."""
    rng = np.random.default_rng(seed)
    m = nx * ny * per
    x = rng.random((m, 2)) * (nx, ny)
    t = rng.random((m, 2)) * (nx, ny) if width == 0 else np.mod(x + width * (rng.random((m, 2)) - 0.5), (nx, ny))
    case = W.cylinder_2d(nx=4 * ny // 3, ny=ny, ppc=8)
    case.update(nx=nx, h=(1.0, 1.0, 1.0), bc=("outflow",) * 6, regions=[], F_N=1.0, dt_G=1e-3, n_surf=0)
    if body:
        case.update(body_c=(0.5 * nx, 0.5 * ny, 0.0), body_r=0.2 * ny)
        out = np.all([((p - (0.5 * nx, 0.5 * ny)) ** 2).sum(1) > (0.201 * ny) ** 2 for p in (x, t)], axis=0)
        x, t = x[out], t[out]
    else:
        case.update(body="none")
    m = len(x)
    case["capacity"] = m + 64
    ij = np.minimum(x.astype(int), (nx - 1, ny - 1))
    cell = (ij[:, 0] + nx * ij[:, 1]).astype(np.int32)
    order = np.argsort(cell, kind="stable")
    pos, vel = np.zeros((m, 3)), np.zeros((m, 3))
    pos[:, :2] = np.clip(x - ij, 0.0, 1.0 - 1e-7)
    vel[:, :2] = (t - x) / 1e-3
    return case, dict(pos=pos[order], vel=vel[order], cell=cell[order], id=rng.permutation(m).astype(np.int64), next_id=m,
                      step=0, sigc_max=np.full(nx * ny, 1e-16))


def _sim(gas, case, state, precision):
    from paper_2506_23917_amd.hs import Sim
    sim = Sim(gas, case, precision=precision, no_particles=True, device="cuda:0")
    sim.import_state(0, state)
    return sim


# runs from one or two a cell to one a particle; tile cells (about 2.5 particles a run and both sides of it),
# block cells of each size the sort pads to, and those about a body, with runs that share a source block
@pytest.mark.parametrize("per", [4, 30, 90, 180, 300, 500, 1000, 2000, 3800])
@pytest.mark.parametrize("width,body", [(1.0, False), (5.0, False), (0, False), (3.0, True), (0, True)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_order_at_any_number_of_runs(gas, per, width, body, precision):
    case, state = _flights(12, 9, per, width, body)
    sim = _sim(gas, case, state, precision)
    sim.step(1)
    after = sim.export_state(0)
    new = np.full(len(state["id"]), -1)
    new[after["id"]] = after["cell"]
    new = new[state["id"]]                       # the cell each particle went to (-1: it left)
    kept = new >= 0
    assert kept.mean() > 0.9
    assert np.array_equal(after["id"], state["id"][kept][np.argsort(new[kept], kind="stable")])


# Kernel times with flights to anywhere against flights within a cell.  The bound lies between what the
# ways for many runs take (2.7 and 3 times as long) and what the placing of runs takes (19 and 5.4).
@pytest.mark.parametrize("group,nx,ny,per,precision,bound", [("dense", 20, 15, 3850, "fp32", 6.0),
                                                             ("gather", 64, 48, 160, "fp64", 4.2)])
def test_many_runs_cost_no_multiple(gas, group, nx, ny, per, precision, bound):
    took = []
    for width in (1.0, 0):
        case, state = _flights(nx, ny, per, width)
        ms = []
        for _ in range(5):
            sim = _sim(gas, case, state, precision)
            sim.set_timing([group])
            sim.step(1)
            ms.append(sim.kernel_timing(group)[0])
            sim.close()
        took.append(float(np.median(ms)))
    print(group, took)
    assert took[1] < bound * took[0]
