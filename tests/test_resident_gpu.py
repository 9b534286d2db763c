"""Runs of small clusters kept inside one workgroup, against the FP64 oracle: the
smallest sizes, both parities (an even cluster meets its opposite atoms from both
ends), each width of lanes per atom and both sides of its limits, every bath.

Tolerances: forces and energies 1e-10 relative (summation order); a trajectory of
24 steps amplifies rounding by less than 1e3 from ~1e-14 A, so positions agree to
1e-10 A and velocities to 1e-11 A/fs.  Cutting a run into calls changes no bit.
"""
import os

import numpy as np
import pytest

import oracle
from paper_1210_3559_amd import inputs, scmd

pytestmark = pytest.mark.gpu

NT = min(16, os.cpu_count() or 1)
BATHS = {"nve": None, "ber": dict(T_start=900.0, T_end=500.0, ramp_steps=15, tau=60.0),
         "lan": dict(kind="langevin", T_start=900.0, T_end=600.0, ramp_steps=10, gamma=10.0, seed=41)}


def _cluster(n, seed):
    rng = np.random.default_rng(seed)
    p = inputs.jitter(inputs.fcc_exact(n), 0.05, rng) if n else np.zeros((0, 3))
    return p, inputs.maxwell_boltzmann(p, 900.0, rng)


def _check(sizes, kinds, parts, params=None):
    cl = [_cluster(n, 300 + k) for k, n in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)])
    ths = [BATHS[kinds[k % len(kinds)]] for k in range(len(sizes))]
    runs = []
    for cut in parts:
        with scmd.Simulation(off, np.concatenate([c[0] for c in cl]), np.concatenate([c[1] for c in cl]), dt=1.0,
                             thermostats=ths, params=params) as sim:
            for m in cut:
                sim.step(m)
            runs.append((sim.positions(), sim.velocities(), sim.forces(), sim.density(),
                         [sim.energy(k) for k in range(len(sizes))]))
    for other in runs[1:]:
        for a, b in zip(runs[0][:4], other[:4]):
            np.testing.assert_array_equal(a, b)
    r, v, f, rho, e = runs[0]
    for k, n in enumerate(sizes):
        if n == 0:
            assert e[k] == (0.0, 0.0, 0.0)
            continue
        s = slice(off[k], off[k + 1])
        steps = sum(parts[0])
        r_ref, v_ref, _, log = oracle.vv_run(cl[k][0], cl[k][1], steps, dt=1.0, thermostat=ths[k], params=params,
                                             nthreads=NT)
        assert np.abs(r[s] - r_ref).max() < 1e-10
        assert np.abs(v[s] - v_ref).max() < 1e-11
        f_ref, rho_ref, _ = oracle.forces(r[s], params=params, nthreads=NT)
        assert np.linalg.norm(f[s] - f_ref) <= 1e-10 * max(np.linalg.norm(f_ref), 1e-300)
        np.testing.assert_allclose(rho[s], rho_ref, rtol=1e-10, atol=0)
        assert e[k][0] == pytest.approx(log[-1, 0], rel=1e-10, abs=1e-300)


@pytest.mark.parametrize("bath", sorted(BATHS))
@pytest.mark.parametrize("n", [1, 2, 3, 4, 13, 48, 49, 96, 97, 147, 152])
def test_resident_run_follows_the_oracle(n, bath):
    print(f"[resident] n={n} bath={bath}", flush=True)
    _check([n], [bath], ([24], [1, 7, 16]))


@pytest.mark.parametrize("params", [None, dict(n=12, m=6), dict(n=10, m=7)])
def test_resident_batch_of_uneven_clusters(params):
    print(f"[resident] batch params={params}", flush=True)
    _check([190, 1, 0, 64, 189, 2, 3, 147, 55, 13, 5, 100, 31, 32, 33, 128], ["nve", "lan", "ber"], ([24], [3, 21]),
           params)


def test_resident_compute_and_profiled_sweeps_agree():
    # the same trajectory with the sweeps launched one by one (profiling on)
    p, v = _cluster(147, 7)
    out = []
    for profiled in (False, True):
        with scmd.Simulation([0, 147], p, v, dt=1.0) as sim:
            scmd.scmd_set_profiling(sim.ctx, profiled)
            sim.compute()
            f = sim.forces()
            sim.step(40)
            out.append((f, sim.positions(), sim.energy()))
    assert np.linalg.norm(out[0][0] - out[1][0]) <= 1e-10 * np.linalg.norm(out[1][0])
    assert np.abs(out[0][1] - out[1][1]).max() < 1e-10
    np.testing.assert_allclose(out[0][2], out[1][2], rtol=1e-10)
