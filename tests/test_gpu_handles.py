"""Handles beside other work on the GPU: destroying one neither waits for another
stream nor disturbs a stream capture, and the pinned memory that calls share is
each call's own while it lasts."""

import threading

import numpy as np
import pytest

import parity as PT
from paper_1309_6726_amd import inputs
from test_gpu_parity import lbm  # noqa: F401

pytestmark = pytest.mark.gpu


def _lattice(nx, ny, seed):
    rng = np.random.default_rng(seed)
    solid = (rng.uniform(size=(ny, nx)) < 0.1).astype(np.uint8)
    p = inputs.Params(nx=nx, ny=ny, tau_g=0.65, k_r=0.01, threshold=5.0)
    rho = np.where(solid, 0.0, rng.uniform(0.2, 1.0, size=(ny, nx)))
    return inputs.Problem(p, solid, rho, rho[::-1, ::-1] * (solid == 0) + (solid == 0), rho)


def _surrogate():
    from paper_1309_6726_amd import surrogate
    net = surrogate.Surrogate(max_batch=64, max_data=64)
    net.set_params(inputs.mlp_init_params(1))
    x = inputs.surrogate_inputs(inputs.sweep_params(0, 64)).astype(np.float32)
    net.gradients(x, np.ones((64, 65), dtype=np.float32))
    net.predict(x)
    return net


def _used(lbm, kind):  # noqa: F811
    """A handle that has read fields (small: one thread; large: four) or answered."""
    if kind == "surrogate":
        return _surrogate()
    prob = _lattice(1024, 600, 1) if kind == "large" else _lattice(256, 200, 2)
    h = lbm.Batch([prob]) if kind == "batch" else lbm.Sim.from_problem(prob)
    h.step(2)
    for _ in range(2):
        if kind == "batch":
            h.fields(0)
        else:
            h.fields()
    return h


KINDS = ["small", "large", "batch", "surrogate"]


@pytest.mark.parametrize("kind", KINDS)
def test_destroy_beside_a_busy_stream(lbm, kind):  # noqa: F811
    import torch
    PT.say(f"[handles] destroy {kind} beside a busy stream")
    h = _used(lbm, kind)
    s = torch.cuda.Stream()
    other = lbm.Sim.from_problem(_lattice(1024, 1024, 3), stream=s)
    torch.cuda.synchronize()
    other.step(8000)  # 0.2 s
    end = torch.cuda.Event()
    end.record(s)
    h.close()
    assert not end.query()
    torch.cuda.synchronize()


@pytest.mark.parametrize("mode", ["global", "thread_local"])
@pytest.mark.parametrize("kind", KINDS)
def test_destroy_during_a_capture(lbm, kind, mode):  # noqa: F811
    import torch
    PT.say(f"[handles] destroy {kind} during a capture ({mode})")
    h = _used(lbm, kind)
    x = torch.zeros(64, device="cuda:0")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode=mode):
        x += 1.0
        lbm_handle, ws = h.h, h.workspace  # the workspace stays
        del lbm_handle
        h.close()
        x += 1.0
    for _ in range(3):
        g.replay()
    torch.cuda.synchronize()
    assert (x == 6.0).all() and ws is not None


def test_calls_of_several_threads(lbm):  # noqa: F811
    """Twelve threads, more than blocks are kept, each with handles and a stream
    of its own: fields and answers equal those of the same calls made alone."""
    import torch
    from paper_1309_6726_amd import surrogate
    n = 12
    probs = [_lattice(200 + 9 * i, 150, 10 + i) if i % 4 else _lattice(1024, 520 + i, 10 + i) for i in range(n)]
    streams = [torch.cuda.Stream() for _ in range(n)]
    sims = [lbm.Sim.from_problem(p, stream=s) for p, s in zip(probs, streams)]
    nets = [surrogate.Surrogate(max_batch=64, max_data=64, stream=s) for s in streams]
    xs = [inputs.surrogate_inputs(inputs.sweep_params(i, 300)).astype(np.float32) for i in range(n)]
    want = []
    for i in range(n):
        sims[i].step(3)
        nets[i].set_params(inputs.mlp_init_params(i))
        want.append((sims[i].fields(), nets[i].predict(xs[i]), nets[i].params()))
    bad = []

    def work(i):
        try:
            for _ in range(6):
                f, y, p = sims[i].fields(), nets[i].predict(xs[i]), nets[i].params()
                same = all(np.array_equal(f[k], want[i][0][k]) for k in f)
                if not (same and np.array_equal(y, want[i][1]) and np.array_equal(p, want[i][2])):
                    bad.append(i)
        except Exception as e:  # noqa: BLE001
            bad.append((i, repr(e)))

    PT.say("[handles] twelve threads")
    threads = [threading.Thread(target=work, args=(i,)) for i in range(n)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad
    for h in sims + nets:
        h.close()
