"""Every tile height that an autotuner times, heights between and beyond them, and
both load hints, on lattices whose strips, segments and last tiles are ragged: the
state and the growth events are those of the lowest tiles, bit for bit.  A tile
taller than one workgroup's rows is shared by several."""

import numpy as np
import pytest

import parity as PT
from paper_1309_6726_amd import inputs
from test_gpu_parity import VARIANTS, _random_state, lbm  # noqa: F401

pytestmark = pytest.mark.gpu

SIZES = [(3, 3), (61, 13), (63, 17), (125, 29), (300, 40)]
HEIGHTS = (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 20, 24, 25, 28, 30, 32, 40, 64, 128, 4096)


def _run(lbm, p, state, tile, nt, scheme):  # noqa: F811
    solid, f, g, m = state
    one = np.where(solid, 0.0, 1.0)
    sim = lbm.Sim(p, solid, one, one, 0.0 * one if p.tau_g > 0 else None, tile=tile, scheme=scheme)
    sim.set_load_hint(nt)
    sim.load_state(f, solid, g, m)
    sim.step(20)
    blob, ev = sim.save(), sorted(PT.event_set(sim.events()))
    sim.close()
    n_ev = int(np.frombuffer(blob[32:40], dtype=np.int64)[0])
    return blob[:len(blob) - n_ev * lbm.EVENT_DTYPE.itemsize], ev


def _all_heights(lbm, nx, ny, kind, scheme):  # noqa: F811
    PT.say(f"[tuned shapes] {scheme} {nx}x{ny} {kind}")
    solid, f, g, m = _random_state(nx, ny, seed=nx + 7 * ny)
    kw = dict(VARIANTS["all"], hold_x=min(5, nx)) if kind == "all" else {}
    if kind == "all":
        g[0] = 0.0  # D2Q4: no rest link
    p = inputs.Params(nx=nx, ny=ny, tau=1.0, G=1.6, G_ads1=-0.33, G_ads2=0.33,
                      tau_g=0.0 if kind == "flow" else 0.65, k_r=0.0 if kind == "flow" else 0.02,
                      threshold=0.6, accel_x=2e-5, accel_y=-1e-5, **kw)
    want = _run(lbm, p, (solid, f, g, m), (64, 1), 0, scheme)
    for sy in HEIGHTS:
        for nt in (0, 1):
            got = _run(lbm, p, (solid, f, g, m), (64, sy), nt, scheme)
            assert got[1] == want[1] and got[0] == want[0], (sy, nt)


@pytest.mark.parametrize("kind", ["plain", "all", "flow"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_population_heights_bitwise(lbm, nx, ny, kind):  # noqa: F811
    _all_heights(lbm, nx, ny, kind, "populations")


@pytest.mark.parametrize("kind", ["plain", "all", "flow"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_moment_heights_bitwise(lbm, nx, ny, kind):  # noqa: F811
    _all_heights(lbm, nx, ny, kind, "moments")


def _large(nx, ny, k_r):
    """A lattice that gives a marching wavefront to every SIMD up to some height,
    with growth in its first steps."""
    rng = np.random.default_rng(nx)
    solid = (rng.uniform(size=(ny, nx)) < 0.2).astype(np.uint8)
    rho = np.where(solid, 0.0, rng.uniform(0.2, 1.0, size=(ny, nx)))
    p = inputs.Params(nx=nx, ny=ny, tau_g=0.65 if k_r else 0.0, k_r=k_r, threshold=0.02)
    return inputs.Problem(p, solid, rho, rho[::-1, ::-1] * (solid == 0) + (solid == 0), rho if k_r else None)


# up to 74 and up to 70 rows marching, more shared; the second beyond the size
# for which nine rows and more are shared
@pytest.mark.parametrize("nx,ny,k_r", [(901, 1203, 0.02), (1741, 1163, 0.0)])
def test_large_moment_heights_bitwise(lbm, nx, ny, k_r):  # noqa: F811
    prob = _large(nx, ny, k_r)
    want = None
    for sy, nt in ((4, 0), (1, 1), (2, 1), (5, 0), (6, 1), (8, 1), (9, 0), (10, 1), (12, 0), (12, 1), (14, 0),
                   (16, 1), (24, 0), (40, 1), (70, 0), (200, 0)):
        PT.say(f"[tuned shapes] moments {nx}x{ny} height {sy} hint {nt}")
        sim = lbm.Sim.from_problem(prob, scheme="moments", tile=(64, sy))
        sim.set_load_hint(nt)
        sim.step(5)
        got, ev = sim.fields(), sorted(PT.event_set(sim.events()))
        sim.close()
        want = want or (got, ev)
        assert ev == want[1] and all(np.array_equal(got[k], want[0][k]) for k in got), (sy, nt)
    assert len(want[1]) > 0 or not k_r
