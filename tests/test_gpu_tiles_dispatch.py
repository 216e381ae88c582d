"""The matrix-core support test where it is really taken: cases that assert the dispatch conditions of the
kernels they aim at (a window of one cell, cells below four smoothing lengths, 38 (FP64: 25) to 55
candidates per pair of rows on average; the FP32 density pass also more waves than one round of the scan holds),
with cells up to the width that widens the inclusion radius most, rows longer than a group of 16
cells, populations on either side of the lines and a grid with a crowded cell.  Bitwise the window
scans, and sparse grids in their time."""
import time

import numpy as np
import pytest

from paper_1908_01682_amd import inputs as I
from tests.gpu_util import HAVE_GPU, banner, needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

if HAVE_GPU:
    import torch
    from paper_1908_01682_amd import tfsph as T

H = 0.05
SCAN_WAVES = 7 * 4 * 256


def _problem(cells, n_gas, n_dust, width, seed, clump=0, rough=False):
    """Random particles in cells of `width` smoothing lengths, `clump` of either phase in one cell; with
    rough a third of the particles lie close to the support's radius from another one."""
    rng = np.random.default_rng(seed)
    hi = np.array(cells) * width * H

    def phase(n):
        x = rng.uniform(0.0, 1.0, (n, 3)) * hi
        x[:clump] = (np.array(cells) // 2 + rng.uniform(0.0, 1.0, (clump, 3))) * width * H
        if rough:
            k = n // 3
            d = rng.standard_normal((k, 3))
            d *= (2.0 * H * (1.0 + rng.uniform(-3e-3, 3e-3, k)) / np.linalg.norm(d, axis=1))[:, None]
            x[-k:] = np.mod(x[:k] + d, hi)
        return I.Phase(x=x, v=0.1 * rng.standard_normal((n, 3)), m=rng.uniform(0.5, 1.5, n) / n,
                       id=rng.permutation(n).astype(np.int32))

    p = I.Params(dim=3, n_cells=tuple(cells), lo=(0.0,) * 3, hi=tuple(hi), h=H, c_s=1.0, t_stop=0.05, dt=0.002)
    return I.Problem("tiles", p, phase(n_gas), phase(n_dust), 1)


CASES = {
    "wide_cells": dict(cells=(9, 7, 6), n_gas=3400, n_dust=3400, width=3.99, rough=True),
    "wide_long_rows": dict(cells=(41, 5, 4), n_gas=7400, n_dust=5200, width=3.99, rough=True),
    "mid_long_rows": dict(cells=(37, 4, 5), n_gas=6700, n_dust=6000, width=3.0, rough=True),
    "at_the_line": dict(cells=(6, 5, 5), n_gas=1375, n_dust=1300, width=2.0),
    "crowded_cell": dict(cells=(10, 9, 8), n_gas=5200, n_dust=4700, width=2.0, clump=600),
}


def _dispatches(prob, *ns, pairs=38):
    p = prob.params
    D = p.cell_width()
    cells = int(np.prod(p.n_cells))
    return 6 * max(ns) <= 55 * cells and 6 * min(ns) >= pairs * cells and all(2.0 * p.h <= d * (1 + 1e-12) <= 4.0 * p.h for d in D)


def _bits(sim, scheme):
    return [(tag + k, np.ascontiguousarray(v).tobytes()) for tag, ph in zip("gd", (sim.gas.numpy(), sim.dust.numpy()))
            for k, v in ph.items() if v is not None and (tag == "g" or k != "rho" or scheme >= 2)]


def _compare(prob, precision, scheme, steps):
    got = []
    for variant in (T.TFSPH_VARIANT_AUTO, T.TFSPH_VARIANT_GLOBAL):
        sim = T.Simulation(prob, precision=precision)
        T.tfsph_set_kernel_variant(sim.ctx, variant)
        sim.step(steps)
        torch.cuda.synchronize()
        got.append((_bits(sim, scheme), sim.flags()))
        sim.close()
    assert got[0] == got[1]


@pytest.mark.parametrize("scheme", [0, 1, 2, 3])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", sorted(CASES))
def test_cases_that_take_tiles_equal_window_scans_bitwise(name, precision, scheme):
    prob = _problem(seed=len(name), **CASES[name])
    assert _dispatches(prob, prob.gas.n, prob.dust.n)
    prob.params = prob.params.replace(scheme=scheme)
    banner(f"tiles dispatch {name} precision {precision} scheme {scheme}")
    _compare(prob, precision, scheme, 2)


@pytest.mark.parametrize("name,cells,n,width", [
    ("just_above", (40, 37, 36), SCAN_WAVES * 64 + 1, 2.0),      # one wave more than the scan holds
    ("wide", (43, 36, 35), 470000, 3.99),
    ("long_rows", (211, 17, 16), 480001, 3.0),
    ("line_between_phases", (36, 37, 38), 463962, 2.0),          # gas at the 55-candidate line, dust above
])
@pytest.mark.parametrize("scheme", [0, 2])
def test_large_fp32_density_equals_window_scan_bitwise(name, cells, n, width, scheme):
    prob = _problem(cells, n, n + 20 if name == "line_between_phases" else 1000, width, 11, rough=width > 2.0)
    assert _dispatches(prob, n) and (n + 63) // 64 > SCAN_WAVES
    assert name != "line_between_phases" or not _dispatches(prob, prob.dust.n)
    prob.params = prob.params.replace(scheme=scheme)
    banner(f"tiles dispatch large {name} scheme {scheme}")
    _compare(prob, 0, scheme, 1)


@pytest.mark.parametrize("n,dust", [(458752, False), (2 ** 19, True)])
def test_fp32_density_passes_that_scan(n, dust):
    """One round of the scan, and a phase whose density records no masks, keep the scan: the same bits (the
    drag sums of the pair schemes take tiles either way)."""
    prob = _problem((41, 37, 36), 1000 if dust else n, n if dust else 1000, 2.0, 12)
    assert dust or (n + 63) // 64 <= SCAN_WAVES
    prob.params = prob.params.replace(scheme=2)
    banner(f"tiles dispatch scan n {n} dust {dust}")
    _compare(prob, 0, 2, 1)


@pytest.mark.parametrize("precision", [0, 1])
def test_grids_below_the_line_equal_window_scans_bitwise(precision):
    """A phase at the line, and one particle short of it."""
    pairs = (38, 25)[precision]
    for n in (pairs * 150 // 6, pairs * 150 // 6 - 1):
        prob = _problem((6, 5, 5), n + 60, n, 2.0, 13)
        assert _dispatches(prob, n + 60, n, pairs=pairs) == (n == pairs * 25)
        prob.params = prob.params.replace(scheme=2)
        banner(f"tiles dispatch line {n} precision {precision}")
        _compare(prob, precision, 2, 2)


def _best(step, n=8):
    step(2)
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(4):
        t = time.perf_counter()
        step(n)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("cells", [64, 128])
def test_sparse_grids_take_the_time_of_window_scans(cells, precision):
    """64^3 + 64^3 particles, 1 or 1/8 a cell: the drag sums on tiles took 1.4 to 2.2 times the scans' step."""
    prob = I.dusty_box(n_side=64, cells_per_axis=cells)
    prob.params = prob.params.replace(scheme=2, t_stop=0.05, h=0.5 / cells, dt=1e-5)
    banner(f"tiles dispatch sparse {cells} precision {precision}")
    t = []
    for variant in (T.TFSPH_VARIANT_AUTO, T.TFSPH_VARIANT_GLOBAL):
        sim = T.Simulation(prob, precision=precision)
        T.tfsph_set_kernel_variant(sim.ctx, variant)
        t.append(_best(sim.step))
        sim.close()
    assert t[0] < 1.2 * t[1], t


def test_small_fp32_density_passes_cost_no_more_than_scans():
    """64^3 + 64^3 particles, one round of the scan: 100 steps in, the two density passes take about 1.02 times the
    mask-free scans; on tiles they took 1.18 times."""
    prob = I.dusty_box(n_side=64, cells_per_axis=32)
    prob.params = prob.params.replace(scheme=2, t_stop=0.05)
    banner("tiles dispatch density time")
    ms = []
    for variant in (T.TFSPH_VARIANT_AUTO, T.TFSPH_VARIANT_GLOBAL):
        sim = T.Simulation(prob, precision=0)
        T.tfsph_set_kernel_variant(sim.ctx, variant)
        sim.step(100)
        T.tfsph_profile(sim.ctx, True)
        sim.step(30)
        torch.cuda.synchronize()
        T.tfsph_profile(sim.ctx, False)
        ms.append(T.tfsph_profile_read(sim.ctx, T.TFSPH_KERNEL_DENSITY)[0] / 30)
        sim.close()
    assert ms[0] < 1.1 * ms[1], ms
