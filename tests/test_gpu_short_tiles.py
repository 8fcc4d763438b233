"""Short tiles of the moment step (one wavefront per row) against tall ones
(one wavefront per tile), bit for bit, where strips, segments and the lattice
itself are ragged."""

import numpy as np
import pytest

import parity as PT
from paper_1309_6726_amd import inputs
from test_gpu_parity import VARIANTS, _random_state, lbm  # noqa: F401

pytestmark = pytest.mark.gpu


def _state(lbm, p, f, solid, g, m, tile, scheme="auto"):  # noqa: F811
    z = np.zeros(solid.shape)
    one = np.where(solid, 0.0, 1.0)
    sim = lbm.Sim(p, solid, one, one, z if p.tau_g > 0 else None, tile=tile, scheme=scheme)
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


@pytest.mark.parametrize("kind", ["plain", "all", "flow"])
@pytest.mark.parametrize("nx,ny", [(3, 3), (62, 13), (63, 16), (125, 29)])
def test_population_tiles_bitwise(lbm, nx, ny, kind):  # noqa: F811
    """Population tiles of every height class: 14 rows share a workgroup."""
    PT.say(f"[population tiles] {nx}x{ny} {kind}")
    solid, f, g, m = _random_state(nx, ny, seed=nx + 7 * ny)
    kw = dict(VARIANTS["all"], hold_x=min(5, nx)) if kind == "all" else {}
    if kind == "all":
        g[0] = 0.0
    p = inputs.Params(nx=nx, ny=ny, tau=1.0, G=1.6, G_ads1=-0.33, G_ads2=0.33,
                      tau_g=0.0 if kind == "flow" else 0.65,
                      k_r=0.0 if kind == "flow" else 0.02, threshold=0.6, **kw)
    ref, ev = _state(lbm, p, f, solid, g, m, (64, 1), "populations")
    for sy in (2, 6, 13, 14, 15, 28, 30):
        got, gev = _state(lbm, p, f, solid, g, m, (128, sy), "populations")
        assert gev == ev, sy
        assert got == ref, sy


def test_default_shapes_match_a_set_one(lbm):  # noqa: F811
    """The launch shapes chosen from the lattice, with the first
    (population-in) step among them."""
    for nx, ny, W, scheme in ((256, 32, 20, "moments"), (1024, 64, 48, "moments"),
                              (300, 41, 29, "populations")):
        PT.say(f"[default shapes] {nx}x{ny} {scheme}")
        prob = inputs.capillary_problem(nx, ny, W, seed=3, k_r=0.02, threshold=0.3, D=0.05)
        a = lbm.Sim.from_problem(prob, scheme=scheme)
        b = lbm.Sim.from_problem(prob, scheme=scheme, tile=(64, 16))
        a.step(60)
        b.step(60)
        fa, fb = a.fields(), b.fields()
        assert all(np.array_equal(fa[k], fb[k]) for k in fa)
        assert PT.event_set(a.events()) == PT.event_set(b.events())
