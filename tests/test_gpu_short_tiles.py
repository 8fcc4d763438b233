"""Short tiles of the moment step (one wavefront per row) against tall ones
(one wavefront per tile), bit for bit, where strips, segments and the lattice
itself are ragged."""

import numpy as np
import pytest

import parity as PT
from paper_1309_6726_amd import inputs
from test_gpu_parity import VARIANTS, _random_state, lbm  # noqa: F401

pytestmark = pytest.mark.gpu


def _state(lbm, p, f, solid, g, m, tile):  # noqa: F811
    z = np.zeros(solid.shape)
    one = np.where(solid, 0.0, 1.0)
    sim = lbm.Sim(p, solid, one, one, z if p.tau_g > 0 else None, tile=tile)
    sim.load_state(f, solid, g, m)
    sim.step(40)
    blob, ev = sim.save(), sorted(PT.event_set(sim.events()))
    sim.close()
    n_ev = int(np.frombuffer(blob[32:40], dtype=np.int64)[0])
    return blob[:len(blob) - n_ev * lbm.EVENT_DTYPE.itemsize], ev


@pytest.mark.parametrize("kind", ["plain", "all", "solute", "flow"])
@pytest.mark.parametrize("nx,ny", [(3, 3), (8, 5), (60, 7), (61, 13), (121, 4), (300, 19)])
def test_short_tiles_bitwise(lbm, nx, ny, kind):  # noqa: F811
    PT.say(f"[short tiles] {nx}x{ny} {kind}")
    solid, f, g, m = _random_state(nx, ny, seed=nx + 7 * ny)
    kw = dict(VARIANTS["all"], hold_x=min(5, nx)) if kind == "all" else {}
    if kind == "all":
        g[0] = 0.0  # D2Q4: no rest link
    p = inputs.Params(nx=nx, ny=ny, tau=1.0, G=1.6, G_ads1=-0.33, G_ads2=0.33,
                      tau_g=0.0 if kind == "flow" else 0.65,
                      k_r=0.02 if kind in ("plain", "all") else 0.0, threshold=0.6,
                      accel_x=2e-5, accel_y=-1e-5, **kw)
    ref, ev = _state(lbm, p, f, solid, g, m, (64, 16))
    for sy in (1, 2, 3, 4, 8, 11, 12):
        got, gev = _state(lbm, p, f, solid, g, m, (64, sy))
        assert gev == ev, sy
        assert got == ref, sy
    assert kind in ("solute", "flow") or nx * ny < 100 or len(ev) > 0
