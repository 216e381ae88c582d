"""The pressure and viscosity terms of a pair at the ends of their range: particles at the same place
(r = 0 between two particles) against the FP64 oracle in every force loop, and problems scaled by powers of
two, where every operation is exact and the state must scale with them bit for bit."""
import numpy as np
import pytest

from paper_1908_01682_amd import inputs as I
from tests.gpu_util import HAVE_GPU, banner, compare_states, needs_gpu, oracle_phase

pytestmark = [pytest.mark.gpu, needs_gpu]

if HAVE_GPU:
    import torch
    from paper_1908_01682_amd import tfsph as T

TOL = {0: 1e-5, 1: 1e-11}        # per step, as for the other comparisons with the oracle


def _coincident(prob, masses=False, **params):
    """Every seventh gas particle, and its right neighbour at every fourteenth, on top of the one before."""
    rng = np.random.default_rng(2)
    x = prob.gas.x
    m = x[1::7].shape[0]
    x[1::7] = x[0::7][:m]
    m = x[2::14].shape[0]
    x[2::14] = x[0::14][:m]
    prob.gas.v = prob.gas.v + 0.1 * rng.standard_normal(prob.gas.v.shape)
    if masses:
        prob.gas.m = prob.gas.m * rng.uniform(0.9, 1.1, prob.gas.n)
    prob.params = prob.params.replace(**params)
    return prob


COINCIDENT = {
    "wave1d": lambda: _coincident(I.dusty_wave(n_side=400, cells_per_axis=200)),
    "wave1d_runs": lambda: _coincident(I.dusty_wave(n_side=4200, cells_per_axis=2100), masses=True),
    "wave2d": lambda: _coincident(I.wave_2d(n_side=40)),
    "wave2d_mass": lambda: _coincident(I.wave_2d(n_side=40), masses=True),
    "box3d": lambda: _coincident(I.dusty_box(n_side=16, cells_per_axis=8, regions_per_axis=2)),
    "box3d_mass": lambda: _coincident(I.dusty_box(n_side=16, cells_per_axis=8, regions_per_axis=2), masses=True),
    "box3d_viscous": lambda: _coincident(I.dusty_box(n_side=16, cells_per_axis=8, regions_per_axis=2),
                                         av_alpha=1.0, av_beta=2.0),
    "shock": lambda: _coincident(I.dusty_shock(n=1000)),
    "shock_small": lambda: _coincident(I.dusty_shock(n=200)),
}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", sorted(COINCIDENT))
def test_particles_at_the_same_place_match_the_oracle(orc, name, precision):
    prob = COINCIDENT[name]()
    p = prob.params
    banner(f"coincident {name} precision {precision}")
    sim = T.Simulation(prob, precision=precision)
    og, od = oracle_phase(orc, sim.gas.numpy(), p.dim), oracle_phase(orc, sim.dust.numpy(), p.dim)
    orc.step(p, og, od, 1)
    sim.step(1)
    torch.cuda.synchronize()
    err = compare_states(p, sim.gas.numpy(), sim.dust.numpy(), og, od, p.c_s)
    flags, _ = sim.flags()
    sim.close()
    assert all(v <= TOL[precision] for v in err.values()), err
    assert not (flags & T.TFSPH_FLAG_NONFINITE)


def _scaled(prob, k):
    """Lengths, times and masses times 2^k: in 1D velocities, densities and energies stay."""
    s = 2.0 ** k
    p = prob.params
    for ph in (prob.gas, prob.dust):
        ph.x = ph.x * s
        ph.m = ph.m * s
    prob.params = p.replace(lo=(p.lo[0] * s,) + tuple(p.lo[1:]), hi=(p.hi[0] * s,) + tuple(p.hi[1:]), h=p.h * s,
                            dt=p.dt * s, t_stop=p.t_stop * s)
    return prob


def _viscous(n):
    prob = I.dusty_wave(n_side=n, cells_per_axis=n // 2, amp=0.2)
    prob.params = prob.params.replace(av_alpha=1.0, av_beta=2.0)
    return prob


# FP32: (2h)^2 near the largest float, so that r^2 + 0.01 h^2 of the outer pairs exceeds the largest
# reciprocal of a normal one; FP64: r^2 down to 2^-935
SCALED = [("shock", lambda: I.dusty_shock(n=90), 0, 68), ("shock_runs", lambda: I.dusty_shock(n=3000), 0, 73),
          ("viscous", lambda: _viscous(90), 0, 68), ("shock", lambda: I.dusty_shock(n=90), 1, -460),
          ("wave", lambda: I.dusty_wave(n_side=90, cells_per_axis=45, amp=0.1), 1, -460),
          ("wave_runs", lambda: I.dusty_wave(n_side=3000, cells_per_axis=1500, amp=0.1), 1, -450),
          ("shock", lambda: I.dusty_shock(n=90), 1, 400)]


@pytest.mark.parametrize("name,make,precision,k", SCALED, ids=[f"{n}_f{32 + 32 * p}_2^{k}" for n, _, p, k in SCALED])
def test_state_scales_with_powers_of_two(name, make, precision, k):
    banner(f"scaled {name} precision {precision} 2^{k}")
    got = []
    for prob, s in ((make(), 1.0), (_scaled(make(), k), 2.0 ** k)):
        sim = T.Simulation(prob, precision=precision)
        sim.step(4)
        torch.cuda.synchronize()
        out = {}
        for tag, ph in zip("gd", (sim.gas.numpy(), sim.dust.numpy())):
            for f in ("cell", "id", "vel", "rho", "energy"):
                if ph[f] is not None and not (tag == "d" and f == "rho"):
                    out[tag + f] = ph[f]
            out[tag + "off"] = ph["off"].astype(np.float64) / s
        got.append(out)
        sim.close()
    for f in got[0]:
        assert np.array_equal(got[0][f], got[1][f]), f
