"""Resident runs in every form the kernel is built in: both precisions, general
exponents, each width of lanes per atom, single evaluations and runs, against the
FP64 oracle.

Tolerances.  FP64: as in the other trajectory tests (summation order; 24 steps
amplify 1e-14 A by less than 1e3).  Mixed: a pair term is a few roundings of 2^-24
off, 2.4e-7 relative, and the sums are double, so densities and energies agree to
1e-6.  In a force some 12 near pairs of up to 10 eV/A cancel: at most 3e-5 eV/A,
within 1e-5 of the norm; over 24 fs that moves a nickel atom by 1.4e-6 A and
changes its velocity by 1.2e-7 A/fs, and the trajectory amplifies little in that
time: 5e-6 A and 5e-7 A/fs.
"""
import os

import numpy as np
import pytest

import oracle
from paper_1210_3559_amd import inputs, scmd

pytestmark = pytest.mark.gpu

NT = min(16, os.cpu_count() or 1)


def _cluster(n, seed):
    rng = np.random.default_rng(seed)
    p = inputs.jitter(inputs.fcc_exact(n), 0.05, rng)
    return p, inputs.maxwell_boltzmann(p, 900.0, rng)


@pytest.mark.parametrize("sizes", [[13], [96], [97], [147], [152], [150] * 15 + [13], [176, 3] * 8])
def test_an_evaluation_between_calls_changes_no_bit(sizes):
    cl = [_cluster(n, 40 + k) for k, n in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)])
    pos, vel = np.concatenate([c[0] for c in cl]), np.concatenate([c[1] for c in cl])
    print(f"[resident] evaluation between calls, {len(sizes)} clusters, largest {max(sizes)}", flush=True)
    out = []
    for compute in (False, True):
        with scmd.Simulation(off, pos, vel, dt=1.0) as sim:
            if compute:
                sim.compute()
            sim.step(7)
            if compute:
                before = (sim.forces(), sim.density())
                sim.compute()
                for a, b in zip(before, (sim.forces(), sim.density())):
                    np.testing.assert_array_equal(a, b)
            sim.step(9)
            out.append((sim.positions(), sim.velocities(), sim.forces()))
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)


# c puts the fcc lattice constant at 3.52 A, so the lattice cut is near equilibrium
PARAMS = {"9_6": None, "12_6": dict(n=12, m=6, c=144.41), "10_7": dict(n=10, m=7, c=45.778)}
LAN = dict(kind="langevin", T_start=900.0, T_end=600.0, ramp_steps=10, gamma=10.0, seed=41)


@pytest.mark.parametrize("exponents", sorted(PARAMS))
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,copies,bath", [(13, 1, None), (48, 1, LAN), (49, 1, None), (96, 1, LAN), (97, 1, None),
                                           (152, 1, LAN), (190, 44, None)])
def test_every_form_follows_the_oracle(n, copies, bath, precision, exponents):
    # larger clusters are resident in batches that fill the chip
    params = PARAMS[exponents]
    if n > 96 and params:
        copies = 72
    p, v = _cluster(n, 70)
    print(f"[resident] n={n} x {copies} {precision} {exponents}", flush=True)
    with scmd.Simulation(np.arange(copies + 1) * n, np.tile(p, (copies, 1)), np.tile(v, (copies, 1)), dt=1.0,
                         precision=precision, params=params, thermostats=[bath] * copies) as sim:
        sim.compute()
        f0, rho0, e0 = sim.forces(), sim.density(), sim.energy()[0]
        sim.step(24)
        r, w, f, e = sim.positions(), sim.velocities(), sim.forces(), sim.energy()[0]
    for a in (f0, rho0, r, w, f):
        np.testing.assert_array_equal(a[:n], a[-n:])
    fp64 = precision == "fp64"
    f_ref, rho_ref, site = oracle.forces(p, params=params, nthreads=NT)
    assert np.linalg.norm(f0[:n] - f_ref) <= (1e-10 if fp64 else 1e-5) * np.linalg.norm(f_ref)
    np.testing.assert_allclose(rho0[:n], rho_ref, rtol=1e-10 if fp64 else 1e-6, atol=0)
    assert e0 == pytest.approx(copies * site.sum(), rel=1e-10 if fp64 else 1e-6)
    r_ref, v_ref, _, log = oracle.vv_run(p, v, 24, dt=1.0, thermostat=bath, params=params, nthreads=NT)
    assert np.abs(r[:n] - r_ref).max() < (1e-10 if fp64 else 5e-6)
    assert np.abs(w[:n] - v_ref).max() < (1e-11 if fp64 else 5e-7)
    f_ref, _, _ = oracle.forces(r[:n], params=params, nthreads=NT)
    assert np.linalg.norm(f[:n] - f_ref) <= (1e-10 if fp64 else 1e-5) * np.linalg.norm(f_ref)
    assert e == pytest.approx(copies * log[-1, 0], rel=1e-10 if fp64 else 1e-6)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [13, 55, 96])
def test_resident_evaluations_agree_with_the_row_sweeps(n, precision):
    # profiling switches the resident kernel off
    p, _ = _cluster(n, 80)
    out = []
    for profiled in (False, True):
        with scmd.Simulation([0, n], p, precision=precision) as sim:
            scmd.scmd_set_profiling(sim.ctx, profiled)
            sim.compute()
            out.append((sim.forces(), sim.density(), sim.energy()[0]))
    tol = 1e-10 if precision == "fp64" else 1e-5
    assert np.linalg.norm(out[0][0] - out[1][0]) <= tol * np.linalg.norm(out[1][0])
    np.testing.assert_allclose(out[0][1], out[1][1], rtol=tol)
    assert out[0][2] == pytest.approx(out[1][2], rel=tol)
