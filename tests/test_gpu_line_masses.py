"""Per-particle gas and dust masses in the fused 1D step (isothermal, inviscid: the force loop with masses,
the dust mass array and the four-word records): runs in LDS and crowded runs in the global workspace,
cells of one phase, single problems and flattened batches, bitwise the separate launches'.  Viscous and
adiabatic problems take those themselves."""
import numpy as np
import pytest

from paper_1908_01682_amd import inputs as I
from tests.gpu_util import HAVE_GPU, banner, needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

if HAVE_GPU:
    import torch
    from paper_1908_01682_amd import tfsph as T


def _problem(n, seed, crowd=0.0, keep_dust=1.0, gas_masses=True, dust_masses=True, kick=0.2):
    rng = np.random.default_rng(seed)
    prob = I.dusty_wave(n_side=n, cells_per_axis=n // 2)
    k = int(crowd * n)
    prob.gas.x[:k, 0] = 0.4 + 40.0 / n * rng.random(k)           # about k / 20 in each of 20 cells
    d = prob.dust
    d.x[:k, 0] = 0.4 + 40.0 / n * rng.random(k)
    kept = np.sort(rng.permutation(n)[:int(keep_dust * n)])
    prob.dust = I.Phase(d.x[kept], d.v[kept], d.m[kept], np.arange(kept.size, dtype=np.int32), None)
    for ph, own in ((prob.gas, gas_masses), (prob.dust, dust_masses)):
        ph.v = ph.v + kick * rng.standard_normal(ph.v.shape)
        if own:
            ph.m = ph.m * rng.uniform(0.8, 1.2, ph.n)
    prob.params = prob.params.replace(cfl=0.25)
    return prob


CASES = {
    "even": dict(n=6001),
    "many_runs": dict(n=80000),
    "crowded": dict(n=9000, crowd=0.9),          # over 256 gas particles a cell: the global workspace
    "some_dust": dict(n=5000, keep_dust=0.3),
    "no_dust": dict(n=4000, keep_dust=0.0),
    "gas_only_masses": dict(n=5000, crowd=0.5, dust_masses=False),
    "dust_only_masses": dict(n=5000, crowd=0.5, gas_masses=False),
}


def _bits(phases):
    return {tag + k: np.ascontiguousarray(v).tobytes() for tag, ph in zip("gd", phases) for k, v in ph.items()
            if v is not None and not (tag == "d" and k == "rho")}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", sorted(CASES))
def test_fused_step_with_masses_equals_separate_launches_bitwise(name, precision):
    prob = _problem(seed=4, **CASES[name])
    banner(f"line masses {name} precision {precision}")
    got = []
    for variant in (T.TFSPH_VARIANT_AUTO, T.TFSPH_VARIANT_GLOBAL):
        sim = T.Simulation(prob, precision=precision)
        T.tfsph_set_kernel_variant(sim.ctx, variant)
        sim.step(4)
        sim.step_graph(4, 2)
        torch.cuda.synchronize()
        got.append((_bits((sim.gas.numpy(), sim.dust.numpy())), sim.flags(), sim.signal_speed()))
        sim.close()
    assert got[0] == got[1]


@pytest.mark.parametrize("precision", [0, 1])
def test_flattened_batch_with_masses_equals_plain_steps_bitwise(precision):
    even = [_problem(n, i, gas_masses=False, dust_masses=False) for i, n in enumerate([900, 2601, 5003])]
    even.append(_problem(4000, 7, crowd=0.9, keep_dust=0.5, gas_masses=False, dust_masses=False))
    rng = np.random.default_rng(9)
    banner(f"line masses batch precision {precision}")
    bs = T.BatchedSimulation(even, precision=precision, form=T.TFSPH_BATCH_FLAT)
    T.tfsph_batch_destroy(bs.handle)
    for p in even:
        p.gas.m = p.gas.m * rng.uniform(0.8, 1.2, p.gas.n)
        p.dust.m = p.dust.m * rng.uniform(0.8, 1.2, p.dust.n)
    for ph, parts in ((bs.gas, [p.gas.m for p in even]), (bs.dust, [p.dust.m for p in even])):
        ph.mass = torch.as_tensor(np.concatenate(parts)).to(ph.vel[0].dtype).cuda()
    bs.state = T.StateC(bs.gas.cstruct(), bs.dust.cstruct())
    bs.handle = T.tfsph_batch_init(bs.desc, bs.state, T.BatchTuning(0, T.TFSPH_BATCH_FLAT, 0), bs._ws, bs.ws_bytes)
    bs.step(4)
    bs.step_graph(3)
    torch.cuda.synchronize()
    for i, p in enumerate(even):
        sim = T.Simulation(p, precision=precision)
        T.tfsph_set_kernel_variant(sim.ctx, T.TFSPH_VARIANT_GLOBAL)
        sim.step(7)
        torch.cuda.synchronize()
        want, have = _bits((sim.gas.numpy(), sim.dust.numpy())), _bits(bs.instance(i))
        for k in ("gcell", "gid", "goff", "gvel", "gmass", "grho", "dcell", "did", "doff", "dvel", "dmass"):
            assert have[k] == want[k], (i, k)
        sim.close()
    bs.close()
