"""Resident runs in every form the kernel is built in: both precisions, general
exponents, each width of lanes per atom, single evaluations and runs, against the
FP64 oracle.

Tolerances.  FP64: as in the other trajectory tests.  Mixed: pair terms in single
precision (2^-24 each, a few per pair) summed in double give 1e-5 of the force
norm; over 24 fs that moves an atom by (1e-5 F / m) t^2 / 2 < 1e-6 A for the
forces of a few eV/A met here.
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
