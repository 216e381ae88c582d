"""The fused 1D step (records scattered into cell ranges, then one kernel per run of cells) against the
separate launches of the window-scan variant: bitwise the same state, flags and signal speed, on runs
that fit LDS and runs that work in the global workspace, windows of one and two cells, few cells
(every run's halo wraps onto itself), crowded and empty cells, every force loop, single and double
precision, and a workspace without room for the records."""
import numpy as np
import pytest

from paper_1908_01682_amd import inputs as I
from tests.gpu_util import HAVE_GPU, banner, needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

if HAVE_GPU:
    import torch
    from paper_1908_01682_amd import tfsph as T


def _kick(prob, scale, seed=3, clump=0.0, drop_dust=0.0):
    """Velocities that carry particles over faces; a share of the gas pulled into a tenth of the box;
    part of the dust left out (cells of one phase)."""
    rng = np.random.default_rng(seed)
    p = prob.params
    for ph in (prob.gas, prob.dust):
        ph.v = ph.v + scale * rng.standard_normal(ph.v.shape)
    k = int(clump * prob.gas.n)
    L = p.hi[0] - p.lo[0]
    prob.gas.x[:k, 0] = p.lo[0] + 0.1 * L * rng.random(k)
    if drop_dust:
        d = prob.dust
        keep = np.sort(rng.permutation(d.n)[:d.n - int(drop_dust * d.n)])
        prob.dust = I.Phase(d.x[keep], d.v[keep], d.m[keep], np.arange(keep.size, dtype=np.int32), None)
    prob.params = p.replace(cfl=0.25)
    return prob


def _masses(prob, seed=5):
    prob.gas.m = prob.gas.m * np.random.default_rng(seed).uniform(0.9, 1.1, prob.gas.n)
    return prob


CASES = {
    "wave": lambda: _kick(I.dusty_wave(n_side=5001, cells_per_axis=2500), 0.3),
    "wave_many_runs": lambda: _kick(I.dusty_wave(n_side=150000, cells_per_axis=75000), 0.3),
    "wave_mass": lambda: _masses(_kick(I.dusty_wave(n_side=4000, cells_per_axis=2000), 0.3)),
    "shock": lambda: _kick(I.dusty_shock(n=6007), 0.1),
    "window_one": lambda: _kick(I.dusty_wave(n_side=4096, cells_per_axis=1024), 0.3),
    "viscous": lambda: _viscous(_kick(I.dusty_wave(n_side=3000, cells_per_axis=1500), 0.3)),
    "clump": lambda: _kick(I.dusty_wave(n_side=4000, cells_per_axis=2000), 0.3, clump=0.95),
    "clump_shock": lambda: _kick(I.dusty_shock(n=3000), 0.1, clump=0.9, drop_dust=0.7),
    "five_cells": lambda: _kick(I.dusty_wave(n_side=2100, h_over_dx=420.0, cells_per_axis=5), 0.3),
    "no_dust_left": lambda: _kick(I.dusty_wave(n_side=2500, cells_per_axis=1250), 0.3, drop_dust=1.0),
}


def _viscous(prob):
    prob.params = prob.params.replace(av_alpha=1.0, av_beta=2.0)
    return prob


def _bits(sim):
    out = []
    for tag, ph in (("g", sim.gas.numpy()), ("d", sim.dust.numpy())):
        for k, v in ph.items():
            if v is not None and not (tag == "d" and k == "rho"):
                out.append((tag + k, np.ascontiguousarray(v).tobytes()))
    return out


def _run(prob, precision, variant, cpb):
    sim = T.Simulation(prob, precision=precision)
    T.tfsph_set_kernel_variant(sim.ctx, variant)
    if cpb:
        T.tfsph_set_cells_per_block(sim.ctx, cpb)
    sim.step(3)
    sim.step(1)
    sim.step_graph(5, 2)
    sim.density(0)
    sim.step(2)
    torch.cuda.synchronize()
    out = (_bits(sim), sim.flags(), sim.signal_speed())
    sim.close()
    return out


# the default run length covers the large grid
RUNS = [(name, cpb) for name in sorted(CASES) for cpb in ((0,) if name == "wave_many_runs" else (0, 7, 256))]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name,cpb", RUNS)
def test_fused_step_equals_separate_launches_bitwise(name, precision, cpb):
    prob = CASES[name]()
    banner(f"line {name} n=({prob.gas.n},{prob.dust.n}) precision {precision} cells per block {cpb}")
    assert _run(prob, precision, T.TFSPH_VARIANT_AUTO, cpb) == _run(prob, precision, T.TFSPH_VARIANT_GLOBAL, cpb)


def test_workspace_without_the_records_is_accepted():
    """The records are the last part of the size asked for: 8 or 16 bytes a particle less is the
    layout of the separate launches, which then run."""
    prob = CASES["wave"]()
    got = []
    for short in (0, 20000):
        st = T.DeviceState(prob, precision=0)
        need = T.tfsph_workspace_size(st.params, st.gas.n, st.dust.n)
        ws = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
        ws = ws[(-ws.data_ptr()) % 256:]
        banner(f"line workspace {need - short}")
        ctx = T.tfsph_init(st.params, st.state, ws, need - short)
        T.tfsph_step(ctx, st.state, 3)
        torch.cuda.synchronize()
        got.append(_bits(st))
        T.tfsph_destroy(ctx)
    assert got[0] == got[1]


@pytest.mark.parametrize("viscous", [False, True])
def test_flattened_batch_equals_separate_launches_bitwise(viscous):
    probs = []
    for i, n in enumerate([12, 900, 2600, 5003]):
        p = _kick(I.dusty_wave(n_side=n, cells_per_axis=n // 2, eps=0.5 + i), 0.05, seed=i,
                  clump=0.8 if i == 2 else 0.0)
        probs.append(_viscous(p) if viscous and i % 2 else p)
    banner(f"line batch viscous {viscous}")
    bs = T.BatchedSimulation(probs, precision=0, form=T.TFSPH_BATCH_FLAT)
    bs.step(4)
    bs.step_graph(2)
    torch.cuda.synchronize()
    for i, p in enumerate(probs):
        sim = T.Simulation(p, precision=0)
        T.tfsph_set_kernel_variant(sim.ctx, T.TFSPH_VARIANT_GLOBAL)
        sim.step(6)
        torch.cuda.synchronize()
        for ph, have in zip((sim.gas.numpy(), sim.dust.numpy()), bs.instance(i)):
            for k in ("cell", "id", "off", "vel"):
                assert np.array_equal(ph[k], have[k]), (i, k)
        sim.close()
    bs.close()
