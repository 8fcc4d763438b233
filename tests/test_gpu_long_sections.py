"""Observables of capillary sections around the number of columns (511) that the
device decides in one pass: every column counts once, whichever pass holds it.

The states are built so that what happens lies in the last columns: bumps of
different heights, a closed column, the front, and a patch of solute that makes
the walls grow there.  Radii, Delta e and the closure step are integer counts on
the oracle's masks and must be equal; the front may differ by the FP32 rounding
of the stored densities."""

import numpy as np
import pytest

import parity as PT
from paper_1309_6726_amd import inputs
from test_gpu_parity import lbm  # noqa: F401

pytestmark = pytest.mark.gpu

LENGTHS = (510, 511, 512, 513, 1021, 1022, 1023, 1024, 1533, 1534)
INTEGER = ("r_min", "r_ave", "r_h", "delta_e", "closure_step", "n_solid", "n_events")
W = 9


def _problem(L, closed):
    """Section of L columns whose walls have bumps in the first and last ones;
    closed: its last column is solid from the start."""
    nx, ny = L + 40, W + 6
    x_in, x_out, y0 = 20, 20 + L, 3
    solid = np.zeros((ny, nx), dtype=np.uint8)
    solid[:y0, x_in:x_out] = solid[y0 + W:, x_in:x_out] = 1
    solid[y0, x_in] = 1
    solid[y0:y0 + 2, x_out - 7] = solid[y0 + W - 3:y0 + W, x_out - 4] = 1
    solid[y0:y0 + (W if closed else 1), x_out - 1] = 1
    wet = np.zeros((ny, nx), dtype=bool)
    wet[:, :x_out - (5 if closed else 1)] = True
    rho1 = np.where(solid, 0.0, np.where(wet, 1.0, 0.05))
    rho2 = np.where(solid, 0.0, np.where(wet, 0.05, 1.0))
    conc = np.zeros((ny, nx))
    conc[:, x_out - 9:x_out - 5] = 1.0
    conc[solid != 0] = 0.0
    # a wall node beside the patch gains k_r phi C = 0.095 in the first step
    p = inputs.Params(nx=nx, ny=ny, tau_g=0.65, k_r=0.1, threshold=0.05, G_ads1=-0.33, G_ads2=0.33,
                      x_in=x_in, x_out=x_out, y0=y0, W=W)
    return inputs.Problem(p, solid, rho1, rho2, conc)


def _same(got, want, where):
    for k in INTEGER:
        assert got[k] == want[k], (where, k, got[k], want[k])
    assert abs(got["front_z"] - want["front_z"]) <= PT.Z_TOL, (where, got["front_z"], want["front_z"])


@pytest.mark.parametrize("scheme", ["moments", "populations"])
def test_every_column_counts_once(lbm, oracle_mod, scheme):  # noqa: F811
    probs = [_problem(L, closed) for L in LENGTHS for closed in (False, True)]
    sims = [lbm.Sim.from_problem(p, scheme=scheme) for p in probs]
    batch = lbm.Batch(probs, scheme=scheme, nslots=1)
    orcs = [oracle_mod.Oracle.from_problem(p) for p in probs]
    for n in (0, 1, 2, 3, 20):
        PT.say(f"[long sections] {scheme} step {n}")
        batch.step(n - batch.observe(0)["step"])
        batch.record_fronts(0)
        fronts = batch.fronts()[:, 0]
        for i, (s, o) in enumerate(zip(sims, orcs)):
            s.step(n - s.observe()["step"])
            o.step(n - o.steps)
            where = (probs[i].params.x_out - probs[i].params.x_in, i % 2, n)
            want, got = o.observe(), s.observe()
            _same(got, want, where)
            assert batch.observe(i) == got, where
            assert fronts[i] == got["front_z"], where
    assert all(len(s.events()) > 0 for s in sims)


def test_straight_slit_has_its_width(lbm):  # noqa: F811
    for L in LENGTHS:
        PT.say(f"[long sections] straight slit of {L}")
        ob = lbm.Sim.from_problem(inputs.capillary_problem(L + 40, 20, 12, x_in=20, x_out=20 + L)).observe()
        assert ob["r_min"] == ob["r_ave"] == ob["r_h"] == 12.0, L
