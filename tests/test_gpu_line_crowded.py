"""Crowded states of the fused 1D step: runs of cells that do not fit a workgroup's LDS go through the
separate phases.  Bitwise the window-scan variant's states (single problems) and the plain steps
(batches), from calls that start crowded, become crowded or stop being so, and no slower than the
separate launches by more than their word checks."""
import time

import numpy as np
import pytest

from paper_1908_01682_amd import inputs as I
from tests.gpu_util import HAVE_GPU, banner, needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

if HAVE_GPU:
    import torch
    from paper_1908_01682_amd import tfsph as T


def _wave(n, per=2.0, kick=0.0, seed=3, **shares):
    """n + n particles, per to a cell; shares gas / dust of a phase in the tenth of the box from 0.3
    on, cell_gas / cell_dust particles in one cell, masses: per-particle ones."""
    rng = np.random.default_rng(seed)
    prob = I.dusty_wave(n_side=n, cells_per_axis=max(5, int(n / per)), h_over_dx=2.0 * per / 2.0)
    p = prob.params
    D = p.hi[0] / p.n_cells[0]
    for name, ph in (("gas", prob.gas), ("dust", prob.dust)):
        k = int(shares.get(name, 0.0) * n)
        ph.x[:k, 0] = 0.3 + 0.1 * rng.random(k)
        k = shares.get("cell_" + name, 0)
        ph.x[:k, 0] = (p.n_cells[0] // 2 + 0.05 + 0.9 * rng.random(k)) * D
        ph.v = ph.v + kick * rng.standard_normal(ph.v.shape)
        if shares.get("masses"):
            ph.m = ph.m * rng.uniform(0.9, 1.1, n)
    prob.params = p.replace(cfl=0.25, dt=p.dt if kick else 1e-3 * p.dt)
    return prob


CASES = {
    "both_tenth": lambda: _wave(20000, gas=0.9, dust=0.9),
    "both_tenth_moving": lambda: _wave(5000, gas=0.9, dust=0.9, kick=0.3),
    "spreading": lambda: _wave(3000, gas=0.6, kick=8.0),
    "dust_tenth": lambda: _wave(20000, dust=0.9, masses=True),
    "dust_cell": lambda: _wave(9000, cell_dust=3000),
    "gas_cell": lambda: _wave(9000, cell_gas=700, masses=True),
    "hundred_a_cell": lambda: _wave(5000, per=100.0),
    "thirty_a_cell": lambda: _wave(50000, per=30.0, kick=0.1),
    "many_tiles": lambda: _wave(90000, gas=0.5, dust=0.5, kick=0.1),
    "only_dust": lambda: _without_gas(_wave(9000, cell_dust=3000)),
}


def _without_gas(prob):
    g = prob.gas
    prob.gas = I.Phase(g.x[:0], g.v[:0], g.m[:0], g.id[:0], None)
    return prob


def _bits(phases):
    return [(tag + k, np.ascontiguousarray(v).tobytes()) for tag, ph in zip("gd", phases)
            for k, v in ph.items() if v is not None and not (tag == "d" and k == "rho")]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", sorted(CASES))
def test_crowded_steps_equal_separate_launches_bitwise(name, precision):
    prob = CASES[name]()
    banner(f"line crowded {name} n=({prob.gas.n},{prob.dust.n}) precision {precision}")
    got = []
    for variant in (T.TFSPH_VARIANT_AUTO, T.TFSPH_VARIANT_GLOBAL):
        sim = T.Simulation(prob, precision=precision)
        T.tfsph_set_kernel_variant(sim.ctx, variant)
        sim.step(3)
        sim.step_graph(7, 3)
        sim.step_graph(6, 3)
        sim.density(1)
        sim.step(1)
        torch.cuda.synchronize()
        got.append((_bits((sim.gas.numpy(), sim.dust.numpy())), sim.flags(), sim.signal_speed()))
        sim.close()
    assert got[0] == got[1]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("cells_per_block", [0, 7, 256])
def test_batch_with_crowded_instances_equals_plain_steps_bitwise(cells_per_block, precision):
    probs = [_wave(12), _wave(4000, gas=0.9, dust=0.9, kick=0.2), _wave(2000, kick=0.3), _wave(3000, cell_dust=1500),
             _wave(900, gas=0.6, kick=8.0)]
    banner(f"line crowded batch cells per block {cells_per_block} precision {precision}")
    bs = T.BatchedSimulation(probs, precision=precision, form=T.TFSPH_BATCH_FLAT, cells_per_block=cells_per_block)
    bs.step(3)
    bs.step_graph(4)
    bs.step_graph(4)
    torch.cuda.synchronize()
    for i, p in enumerate(probs):
        sim = T.Simulation(p, precision=precision)
        T.tfsph_set_kernel_variant(sim.ctx, T.TFSPH_VARIANT_GLOBAL)
        sim.step(11)
        torch.cuda.synchronize()
        for ph, have in zip((sim.gas.numpy(), sim.dust.numpy()), bs.instance(i)):
            for k in ("cell", "id", "off", "vel"):
                assert np.array_equal(ph[k], have[k]), (i, k)
        sim.close()
    bs.close()


def _best(step, n=10):
    step(2)
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(4):
        t = time.perf_counter()
        step(n)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


# one workgroup per run took 3.4, 13, 2.2 and 2.7 times the separate launches here; the limit
# leaves 3 short launches and the spread of two timings
SLOW = {
    "both_tenth": lambda: _wave(100000, gas=0.9, dust=0.9),
    "dust_cell": lambda: _wave(100000, cell_dust=5000),
    "gas_cell": lambda: _wave(100000, cell_gas=1000),
    "hundred_a_cell": lambda: _wave(100000, per=100.0),
}


@pytest.mark.parametrize("name", sorted(SLOW))
def test_crowded_step_takes_the_time_of_separate_launches(name):
    prob = SLOW[name]()
    banner(f"line crowded time {name}")
    t = []
    for variant in (T.TFSPH_VARIANT_AUTO, T.TFSPH_VARIANT_GLOBAL):
        sim = T.Simulation(prob, precision=0)
        T.tfsph_set_kernel_variant(sim.ctx, variant)
        t.append(_best(sim.step))
        sim.close()
    assert t[0] < 1.5 * t[1], t


@pytest.mark.parametrize("name", ["crowded", "one_dense"])
def test_crowded_batch_takes_the_time_of_separate_launches(name):
    """The separate launches run where the workspace has no room for the records (16 bytes a particle)."""
    probs = ([_wave(5000, gas=0.9, dust=0.9) for _ in range(64)] if name == "crowded" else
             [_wave(5000) for _ in range(63)] + [_wave(5000, per=100.0)])
    banner(f"line crowded batch time {name}")
    bs = T.BatchedSimulation(probs, precision=0, form=T.TFSPH_BATCH_FLAT)
    fused = _best(bs.step)
    T.tfsph_batch_destroy(bs.handle)
    bs.handle = T.tfsph_batch_init(bs.desc, bs.state, T.BatchTuning(0, T.TFSPH_BATCH_FLAT, 0), bs._ws,
                                   bs.ws_bytes - 12 * (bs.gas.n + bs.dust.n))
    separate = _best(bs.step)
    bs.close()
    assert fused < 1.5 * separate, (fused, separate)
