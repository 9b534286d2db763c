"""Cell-list builds on both sides of the largest grid whose cell starts every
scattering workgroup scans for itself, against the FP64 oracle.

Forces agree with the oracle at the run's own final positions, where only the
order of an atom's few dozen pair sums differs (relative 1e-10 of the largest
force); the two skins' trajectories amplify 1e-14 A by less than 1e3 in these
few steps.
"""
import os

import numpy as np
import pytest

import oracle
from paper_1210_3559_amd import inputs, scmd

pytestmark = pytest.mark.gpu

NT = min(16, os.cpu_count() or 1)
RC = 8.8
SCAN_LIMIT = 12288  # cells


def _capacity(p, edge):
    return int(np.prod(np.floor((p.max(0) - p.min(0)) / edge).astype(int) + 5)) if len(p) else 125


# one cluster; the last grid below the limit (two workgroups) and the first one
# above it; a large cluster and an empty one among the small
@pytest.mark.parametrize("sizes", [[1], [1024], [1025], [13] * 98, [13] * 99, [13] * 60 + [2243, 0] + [13] * 34,
                                   [13] * 60 + [2243, 0] + [13] * 38])
def test_builds_around_the_scan_limit(sizes):
    pos, vel = [], []
    for k, n in enumerate(sizes):
        rng = np.random.default_rng(500 + k)
        p = inputs.jitter(inputs.fcc_exact(n), 0.05, rng) if n else np.zeros((0, 3))
        pos.append(p)
        vel.append(inputs.maxwell_boltzmann(p, 900.0, rng) if n > 1 else np.zeros((n, 3)))
    off = np.concatenate([[0], np.cumsum(sizes)])
    cells = sum(_capacity(p, RC) for p in pos)
    print(f"[cell-scan] {len(sizes)} clusters, {off[-1]} atoms, {cells} cells", flush=True)
    if sizes == [13] * 98:
        assert cells <= SCAN_LIMIT
    if sizes == [13] * 99:
        assert cells > SCAN_LIMIT
    runs = []
    for skin in (0.0, 0.4):
        with scmd.Simulation(off, np.concatenate(pos), np.concatenate(vel), dt=2.0, rc=RC) as sim:
            sim.set_cell_skin(skin)
            sim.step(12)
            runs.append((sim.positions(), sim.forces(), sim.density()))
            if skin == 0.0:
                assert sim.cell_rebuilds() == 13  # every force evaluation
    assert np.abs(runs[0][0] - runs[1][0]).max() < 1e-10
    for r, f, rho in runs:
        for k in {0, len(sizes) // 2, min(60, len(sizes) - 1), len(sizes) - 1}:
            a, b = off[k], off[k + 1]
            if a == b:
                continue
            f_ref, rho_ref, _ = oracle.forces(r[a:b], params=dict(rc=RC), nthreads=NT)
            assert np.abs(f[a:b] - f_ref).max() <= 1e-10 * max(np.abs(f_ref).max(), 1.0)
            np.testing.assert_allclose(rho[a:b], rho_ref, rtol=1e-10, atol=0)
