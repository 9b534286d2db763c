"""Density sums whose pairs share a reciprocal (row and symmetric sweeps), where
the product of their r^2 leaves the range of a double: a pair of coincident atoms
spoils its own two densities only, and atoms flung out of the cluster leave the
others' as they are, against sums in numpy.

The sums differ in order from numpy's and one term in them by a few 2^-53: 1e-12
relative is a hundred times that over 700 terms.
"""
import numpy as np
import pytest

from paper_1210_3559_amd import inputs, scmd

pytestmark = pytest.mark.gpu

A = 3.52
PLANS = [dict(pairs=2, ipt=2), dict(pairs=2, ipt=4), dict(pairs=2, ipt=8), dict(pairs=3), dict(pairs=3, waves_j=16)]


def _density(p, rows):
    out = np.empty(len(rows))
    for k, i in enumerate(rows):
        r2 = ((np.delete(p, i, 0) - p[i]) ** 2).sum(1)
        out[k] = ((A * A / r2) ** 3).sum()
    return out


@pytest.mark.parametrize("plan", PLANS, ids=str)
@pytest.mark.parametrize("pair", [(5, 40), (5, 200), (130, 699)])
def test_a_coincident_pair_spoils_only_its_own_densities(plan, pair):
    n = 700
    p = inputs.jitter(inputs.fcc_exact(n), 0.05, np.random.default_rng(11))
    p[pair[1]] = p[pair[0]]
    print(f"[shared] coincident {pair} {plan}", flush=True)
    with scmd.Simulation([0, n], p, tuning=plan) as sim:
        with pytest.raises(scmd.ScmdError) as e:
            sim.compute()
        assert e.value.status == scmd.SCMD_ENONFINITE
        rho = sim.density()
    assert not np.isfinite(rho[list(pair)]).any()
    others = np.setdiff1d(np.arange(n), pair)
    np.testing.assert_allclose(rho[others], _density(p, others), rtol=1e-12)


@pytest.mark.parametrize("speed", [1e38, 1e60])
@pytest.mark.parametrize("plan", PLANS, ids=str)
def test_atoms_flung_out_leave_the_others_as_they_are(plan, speed):
    n, far = 700, [0, 63, 64, 300, 301, 302, 699]
    rng = np.random.default_rng(12)
    p = inputs.jitter(inputs.fcc_exact(n), 0.05, rng)
    v = np.zeros((n, 3))
    d = rng.standard_normal((len(far), 3))
    v[far] = speed * d / np.linalg.norm(d, axis=1)[:, None]
    print(f"[shared] flung out at {speed} {plan}", flush=True)
    with scmd.Simulation([0, n], p, v, dt=1.0, tuning=plan) as sim:
        sim.step(1)
        q, rho, e = sim.positions(), sim.density(), sim.energy()
    assert np.isfinite(e).all() and np.abs(q[far]).max() > 0.3 * speed
    near = np.setdiff1d(np.arange(n), far)
    np.testing.assert_allclose(rho[near], _density(q[near], np.arange(len(near))), rtol=1e-12)
    assert (np.abs(rho[far]) < 1e-200).all()
