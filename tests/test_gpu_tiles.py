"""The matrix-core support test of the 3D pair kernels against the window scans (the scan variant):
bitwise the same states for every scheme, on grids and populations at its edges: three cells along an
axis (every wave's window wraps), rows of cells shorter and longer than a half wave, empty cells and
wide runs of cells, crowded cells (pairs of rows beyond 64 candidates, runs beyond the tile limit,
averages on either side of the dispatch line), cells from one support radius to four smoothing
lengths wide, and particles on cell faces."""
import numpy as np
import pytest

from paper_1908_01682_amd import inputs as I
from tests.gpu_util import HAVE_GPU, banner, needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

if HAVE_GPU:
    import torch
    from paper_1908_01682_amd import tfsph as T


def _problem(cells, n_gas, n_dust, width, seed, clump=0.0, faces=False):
    """Random particles in a box of cells of `width` smoothing lengths; a share `clump` of each phase
    in one cell, with `faces` a tenth of the coordinates exactly on cell faces."""
    rng = np.random.default_rng(seed)
    h = 0.05
    hi = tuple(c * width * h for c in cells)

    def phase(n):
        x = rng.uniform(0.0, 1.0, (n, 3)) * hi
        k = int(clump * n)
        x[:k] = (np.array(cells) // 2 + rng.uniform(0.0, 1.0, (k, 3))) * width * h
        if faces:
            on = rng.random((n, 3)) < 0.1
            x = np.where(on, np.round(x / (width * h)) * width * h, x)
            x = np.where(x >= hi, 0.0, x)
        return I.Phase(x=x, v=0.1 * rng.standard_normal((n, 3)), m=rng.uniform(0.5, 1.5, n) / max(n, 1),
                       id=rng.permutation(n).astype(np.int32))

    p = I.Params(dim=3, n_cells=tuple(cells), lo=(0.0,) * 3, hi=hi, h=h, c_s=1.0, t_stop=0.05, dt=0.002)
    return I.Problem("tiles", p, phase(n_gas), phase(n_dust), 1)


CASES = {
    "three_cells": dict(cells=(3, 3, 3), n_gas=211, n_dust=190, width=2.0, seed=1),
    "short_rows": dict(cells=(5, 4, 7), n_gas=1000, n_dust=1003, width=2.0, seed=2),
    "sparse": dict(cells=(40, 6, 5), n_gas=700, n_dust=65, width=2.0, seed=3),
    "long_rows": dict(cells=(31, 5, 3), n_gas=4097, n_dust=3000, width=2.3, seed=4),
    "clumped": dict(cells=(8, 8, 8), n_gas=4000, n_dust=3000, width=2.0, seed=5, clump=0.25),
    "clumped_tiny": dict(cells=(3, 3, 4), n_gas=900, n_dust=700, width=2.0, seed=6, clump=0.9),
    "wide_cells": dict(cells=(4, 5, 3), n_gas=1500, n_dust=1500, width=4.0, seed=7),
    "on_faces": dict(cells=(9, 7, 6), n_gas=3000, n_dust=2999, width=2.0, seed=8, faces=True),
    "full_pairs": dict(cells=(6, 5, 5), n_gas=1420, n_dust=1430, width=2.0, seed=10),
    "one_gas": dict(cells=(6, 6, 6), n_gas=1, n_dust=63, width=2.0, seed=9),
}


@pytest.mark.parametrize("scheme", [0, 1, 2, 3])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", sorted(CASES))
def test_tile_test_equals_window_scans_bitwise(name, precision, scheme):
    prob = _problem(**CASES[name])
    prob.params = prob.params.replace(scheme=scheme)
    banner(f"tiles {name} precision {precision} scheme {scheme}")
    got = []
    for variant in (T.TFSPH_VARIANT_AUTO, T.TFSPH_VARIANT_GLOBAL):
        sim = T.Simulation(prob, precision=precision)
        T.tfsph_set_kernel_variant(sim.ctx, variant)
        sim.step(2)
        torch.cuda.synchronize()
        out = []
        for tag, ph in zip("gd", (sim.gas.numpy(), sim.dust.numpy())):
            for k, v in ph.items():
                if v is not None and (tag == "g" or k != "rho" or scheme >= 2):
                    out.append((tag + k, np.ascontiguousarray(v).tobytes()))
        got.append((out, sim.flags()))
        sim.close()
    assert got[0] == got[1]
