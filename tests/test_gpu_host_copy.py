"""Fields read into ordinary host memory, which go through pinned slots (one
thread below 16 MB, four from there on), against the same fields read into pinned
memory, which the GPU writes directly: equal to the byte, nothing beyond the end."""

import numpy as np
import pytest

import parity as PT
from paper_1309_6726_amd import inputs
from test_gpu_parity import lbm  # noqa: F401

pytestmark = pytest.mark.gpu

GUARD = 4096  # doubles after the end

# (nx, ny, field bits), 8 nx ny bytes a field: less than one slot (and small
# enough that the first copy makes no slots), one slot of 512 KB exactly and a
# row more, an odd number of slots, the last size of one
# thread and the first of four, a last chunk of one row, a ragged many
CASES = [(32, 8, 0x10), (256, 256, 0x01), (256, 257, 0x02), (301, 211, 0x4d), (1023, 1025, 0x02),
         (1023, 1025, 0x03), (1024, 1024, 0x03), (1024, 1025, 0x08 | 0x10), (700, 501, 0x7f)]


@pytest.fixture(scope="module")
def sims(lbm):  # noqa: F811
    """The lattices as single simulations and as one batch, a few steps on."""
    def problem(nx, ny, seed):
        rng = np.random.default_rng(seed)
        solid = (rng.uniform(size=(ny, nx)) < 0.1).astype(np.uint8)
        p = inputs.Params(nx=nx, ny=ny, tau=1.0, G=1.6, G_ads1=-0.33, G_ads2=0.33, tau_g=0.65,
                          k_r=0.01, threshold=0.6)
        rho = np.where(solid, 0.0, rng.uniform(0.2, 1.0, size=(ny, nx)))
        return inputs.Problem(p, solid, rho, rho[::-1, ::-1] * (solid == 0) + (solid == 0), rho, name="",
                              steps=3)
    ps = [problem(nx, ny, k) for k, (nx, ny, _) in enumerate(CASES)]
    singles = [lbm.Sim.from_problem(p) for p in ps]
    for s in singles:
        s.step(3)
    batch = lbm.Batch(ps)
    batch.step(3)
    yield singles, batch
    for s in singles:
        s.close()
    batch.close()


@pytest.mark.parametrize("k", range(len(CASES)))
@pytest.mark.parametrize("kind", ["single", "batch"])
def test_fields_to_pageable_memory(lbm, sims, kind, k):  # noqa: F811
    import torch
    nx, ny, mask = CASES[k]
    PT.say(f"[host copy] {kind} {nx}x{ny} fields {mask:#x}")
    n = nx * ny * bin(mask).count("1")

    def read(ptr):
        if kind == "single":
            lbm.check(lbm.lib().lbm_fields(sims[0][k].h, mask, ptr))
        else:
            lbm.check(lbm.lib().lbm_batch_fields(sims[1].h, k, mask, ptr))
    pinned = torch.full((n + GUARD,), -7.5, dtype=torch.float64, pin_memory=True)
    read(pinned.data_ptr())
    want = pinned.numpy()
    for shift in (0, 1):  # an unaligned destination too
        raw = np.full(8 * (n + GUARD) + shift, 0xA5, dtype=np.uint8)
        read(raw.ctypes.data + shift)
        assert (raw[:shift] == 0xA5).all() and (raw[shift + 8 * n:] == 0xA5).all()
        assert raw[shift:shift + 8 * n].tobytes() == want[:n].tobytes()
    assert (want[n:] == -7.5).all() and len(np.unique(want[:n])) > 1
