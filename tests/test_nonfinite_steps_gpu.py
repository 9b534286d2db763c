"""Symmetric, one-sided and cell-list runs report an energy that becomes non-finite
on any step of a call, also when the thermostat has brought it back by the call's
last step.  Two atoms 5e-16 A apart repel with 1e157 eV/A: every energy of the
evaluation is finite, the first step throws them out at about 1e153 A/fs, where the
kinetic energy overflows while v^2 and r^2 do not, and a thermostat that rescales
fully (tau = dt) stops them."""
import numpy as np
import pytest

from paper_1210_3559_amd import inputs, scmd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,kw", [(300, dict(tuning=dict(pairs=2, ipt=2))), (300, dict(tuning=dict(pairs=2, ipt=4))),
                                  (300, dict(tuning=dict(pairs=2, ipt=8))), (300, dict(rc=8.8)),
                                  (300, dict(tuning=dict(ipt=1, waves_i=1, waves_j=8, pairs=1)))], ids=str)
def test_an_overflow_on_an_inner_step_is_reported(n, kw):
    p = inputs.jitter(inputs.fcc_exact(n), 0.05, np.random.default_rng(3))
    p -= p[0]
    p[1] = (5e-16, 0.0, 0.0)
    th = dict(T_start=900.0, T_end=900.0, ramp_steps=0, tau=1.0)
    print(f"[nonfinite] n={n} {kw}", flush=True)
    with scmd.Simulation([0, n], p, dt=1.0, thermostats=[th], **kw) as sim:
        sim.compute()
        assert np.isfinite(sim.energy()).all()
        with pytest.raises(scmd.ScmdError) as e:
            sim.step(4)
        assert e.value.status == scmd.SCMD_ENONFINITE
        assert np.isfinite(sim.positions()).all() and np.isfinite(sim.velocities()).all()
