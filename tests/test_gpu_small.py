"""The one-workgroup step of small 1D and 2D problems (working set in LDS) against the multi-launch
step of the window-scan variant: bitwise the same state, flags and signal speed, at the edges of its
thread and LDS ranges; and batches that mix instances in LDS with instances in global memory."""
import numpy as np
import pytest

from paper_1908_01682_amd import inputs as I
from tests.gpu_util import HAVE_GPU, banner, needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

if HAVE_GPU:
    import torch
    from paper_1908_01682_amd import tfsph as T


def _bits(phases):
    out = []
    for tag, ph in zip("gd", phases):
        for k, v in ph.items():
            if v is not None and not (tag == "d" and k == "rho"):
                out.append((tag + k, np.ascontiguousarray(v).tobytes()))
    return out


def _jitter(prob, seed=7, scale=0.2):
    """Velocities that carry particles over cell faces, and a dust phase of another size."""
    rng = np.random.default_rng(seed)
    for ph in (prob.gas, prob.dust):
        ph.v = ph.v + scale * rng.standard_normal(ph.v.shape)
    d = prob.dust
    keep = np.sort(rng.permutation(d.n)[:max(1, d.n * 3 // 4)])
    prob.dust = I.Phase(d.x[keep], d.v[keep], d.m[keep], np.arange(keep.size, dtype=np.int32), None)
    prob.params = prob.params.replace(cfl=0.25)
    return prob


CASES = {
    "wave1d_10": lambda: I.dusty_wave(n_side=10, cells_per_axis=5),
    "wave1d_64": lambda: I.dusty_wave(n_side=64, cells_per_axis=32),
    "wave1d_65": lambda: I.dusty_wave(n_side=65, cells_per_axis=32),
    "wave1d_513": lambda: I.dusty_wave(n_side=513, cells_per_axis=256),
    "wave1d_1024": lambda: I.dusty_wave(n_side=1024, cells_per_axis=512),
    "wave1d_1025": lambda: I.dusty_wave(n_side=1025, cells_per_axis=512),
    "wave1d_1500": lambda: I.dusty_wave(n_side=1500, cells_per_axis=750),
    "wave1d_wide": lambda: I.paper_dustywave(n=300),
    "shock1d_90": lambda: I.dusty_shock(n=90),
    "shock1d_700": lambda: I.dusty_shock(n=700),
    "wave2d_10": lambda: I.wave_2d(n_side=10),
    "wave2d_25": lambda: I.wave_2d(n_side=25),
    "wave2d_32": lambda: I.wave_2d(n_side=32),
}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", sorted(CASES))
def test_small_step_equals_multi_launch_bitwise(name, precision):
    prob = _jitter(CASES[name]())
    banner(f"small {name} n=({prob.gas.n},{prob.dust.n}) precision {precision}")
    got = []
    for variant in (T.TFSPH_VARIANT_AUTO, T.TFSPH_VARIANT_GLOBAL):
        sim = T.Simulation(prob, precision=precision)
        T.tfsph_set_kernel_variant(sim.ctx, variant)
        sim.step(3)
        sim.step(1)
        sim.step_graph(5, 2)
        torch.cuda.synchronize()
        got.append((_bits((sim.gas.numpy(), sim.dust.numpy())), sim.flags(), sim.signal_speed()))
        sim.close()
    assert got[0] == got[1]


@pytest.mark.parametrize("side", ["gas", "dust", "both"])
def test_small_step_with_an_empty_phase_and_a_bad_cell(side):
    prob = I.dusty_wave(n_side=100, cells_per_axis=50)
    none = I.Phase(np.zeros((0, 1)), np.zeros((0, 1)), np.zeros(0), np.zeros(0, dtype=np.int32), None)
    if side == "gas":
        prob.gas = none
    if side == "dust":
        prob.dust = none
    got = []
    for variant in (T.TFSPH_VARIANT_AUTO, T.TFSPH_VARIANT_GLOBAL):
        banner(f"small without {side}, variant {variant}")
        sim = T.Simulation(prob, precision=0)
        T.tfsph_set_kernel_variant(sim.ctx, variant)
        for ph in (sim.gas, sim.dust):
            if ph.n and side == "both":
                ph.cell[3] = 4711               # out of range: flagged, taken as cell 0
        sim.step(2)
        torch.cuda.synchronize()
        flags, cells = sim.flags()
        assert bool(flags & T.TFSPH_FLAG_BAD_CELL) == (side == "both")
        got.append((_bits((sim.gas.numpy(), sim.dust.numpy())), flags, cells))
        sim.close()
    assert got[0] == got[1]


@pytest.mark.parametrize("dim", [1, 2])
def test_batch_mixing_lds_and_global_instances_equals_plain_bitwise(dim):
    sizes = [10, 130, 800, 1400, 2600] if dim == 1 else [11, 20, 33, 60]
    probs = []
    for i, n in enumerate(sizes):
        p = I.dusty_wave(n_side=n, cells_per_axis=n // 2, eps=0.5 + i) if dim == 1 else I.wave_2d(n_side=n)
        probs.append(_jitter(p, seed=i, scale=0.05))
    banner(f"mixed batch dim {dim}")
    bs = T.BatchedSimulation(probs, precision=0, block=1024)
    bs.step(4)
    bs.step_graph(2)
    torch.cuda.synchronize()
    for i, p in enumerate(probs):
        sim = T.Simulation(p, precision=0)
        T.tfsph_set_kernel_variant(sim.ctx, T.TFSPH_VARIANT_GLOBAL)
        sim.step(6)
        torch.cuda.synchronize()
        want = dict(_bits((sim.gas.numpy(), sim.dust.numpy())))
        have = dict(_bits(bs.instance(i)))
        for k in ("gcell", "gid", "goff", "gvel", "grho", "dcell", "did", "doff", "dvel"):
            assert have[k] == want[k], (i, k)
        sim.close()
    bs.close()
