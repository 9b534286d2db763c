"""Symmetric sweeps with four wavefronts per item and the drift folded into the
density sweep: tile and group edges, every bath, against the FP64 oracle.

A trajectory of a few tens of steps amplifies rounding differences by less
than 1e3 from ~1e-14 A, so positions agree to 1e-10 A and velocities to
1e-11 A/fs; splitting a run into calls changes no bit.
"""
import os

import numpy as np
import pytest

import oracle
from paper_1210_3559_amd import inputs, scmd

pytestmark = pytest.mark.gpu

NT = min(16, os.cpu_count() or 1)
# one atom, one tile, one past a tile, one past a group of two and of four tiles, several items
SIZES = [1, 64, 65, 0, 129, 257, 700]


def _baths(kinds):
    th = {"nve": None, "ber": dict(T_start=900.0, T_end=500.0, ramp_steps=15, tau=60.0),
          "lan": dict(kind="langevin", T_start=900.0, T_end=600.0, ramp_steps=10, gamma=10.0, seed=41)}
    return [th[kinds[k % len(kinds)]] for k in range(len(SIZES))]


@pytest.mark.parametrize("kinds", [("nve",), ("ber",), ("lan",), ("nve", "lan", "ber")])
@pytest.mark.parametrize("ipt", [2, 4])
def test_folded_drift_follows_the_oracle(ipt, kinds):
    pos, vel = [], []
    for k, n in enumerate(SIZES):
        rng = np.random.default_rng(100 + k)
        p = inputs.jitter(inputs.fcc_exact(n), 0.05, rng) if n else np.zeros((0, 3))
        pos.append(p)
        vel.append(inputs.maxwell_boltzmann(p, 900.0, rng))
    off = np.concatenate([[0], np.cumsum(SIZES)])
    ths = _baths(kinds)
    runs = []
    for parts in ([21], [1, 2, 18]):
        print(f"[split-sym] ipt={ipt} baths={kinds} parts={parts}", flush=True)
        with scmd.Simulation(off, np.concatenate(pos), np.concatenate(vel), dt=1.0, thermostats=ths,
                             tuning=dict(pairs=2, ipt=ipt, target_items=3)) as sim:
            for n in parts:
                sim.step(n)
            runs.append((sim.positions(), sim.velocities(), [sim.energy(k)[0] for k in range(len(SIZES))]))
    np.testing.assert_array_equal(runs[0][0], runs[1][0])
    np.testing.assert_array_equal(runs[0][1], runs[1][1])
    r, v, e = runs[0]
    for k, n in enumerate(SIZES):
        if n == 0:
            continue
        r_ref, v_ref, _, log = oracle.vv_run(pos[k], vel[k], 21, dt=1.0, thermostat=ths[k], nthreads=NT)
        assert np.abs(r[off[k]:off[k + 1]] - r_ref).max() < 1e-10
        assert np.abs(v[off[k]:off[k + 1]] - v_ref).max() < 1e-11
        assert e[k] == pytest.approx(log[-1, 0], rel=1e-10, abs=1e-300)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [3072, 3073, 4096])
def test_default_plan_around_the_row_limits(n, precision):
    # a single cluster leaves the row sweeps for the symmetric ones above 3072
    # atoms in double, above 4096 in mixed precision
    rng = np.random.default_rng(n)
    p = inputs.jitter(inputs.fcc_exact(n), 0.05, rng)
    print(f"[split-sym] default plan n={n} {precision}", flush=True)
    with scmd.Simulation([0, n], p, None, precision=precision) as sim:
        sim.compute()
        f, rho, e = sim.forces(), sim.density(), sim.energy()[0]
    f_ref, rho_ref, site = oracle.forces(p, nthreads=NT)
    tol = 1e-10 if precision == "fp64" else 1e-5
    assert np.linalg.norm(f - f_ref) <= tol * np.linalg.norm(f_ref)
    np.testing.assert_allclose(rho, rho_ref, rtol=tol, atol=0)
    assert e == pytest.approx(site.sum(), rel=tol)
