"""Predictions whose answers lie over their queries in memory equal those of
separate arrays, for every place of the queries within the answers: on the device
(allocating nothing, also captured and replayed) and on the host."""

import numpy as np
import pytest

import parity as PT
from paper_1309_6726_amd import inputs
from test_gpu_parity import lbm  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def net():
    from paper_1309_6726_amd import surrogate
    s = surrogate.Surrogate(max_batch=4096, max_data=1)
    s.set_params(inputs.mlp_init_params(5))
    yield s
    s.close()


def _queries(n):
    return inputs.surrogate_inputs(inputs.sweep_params(3, n)).astype(np.float32)


def _places(n):
    """First value of the queries, counted from the first of the answers."""
    return [p for p in (-2 * n, -1, 0, 1, 160, 31 * n, 60 * n - 1, 60 * n, 60 * n + 1, 64 * n) if p <= 64 * n]


# 32 rows: one workgroup; 1024: the most on the device
@pytest.mark.parametrize("n", [1, 32, 33, 64, 97, 1000, 1024])
def test_device_answers_over_queries(lbm, net, n):  # noqa: F811
    import torch
    x = _queries(n)
    want = net.predict(x)
    for place in _places(n):
        PT.say(f"[surrogate overlap] device, {n} rows at {place}")
        lead = 5 * n  # before and after the answers
        buf = torch.full((lead + 65 * n + lead,), -3.0, device="cuda:0")
        q = buf[lead + place:lead + place + 5 * n].view(n, 5)
        y = buf[lead:lead + 65 * n].view(n, 65)
        q.copy_(torch.from_numpy(x))
        net.predict_noalloc(q, y)
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), want), place
        q.fill_(-3.0)
        y.fill_(-3.0)
        assert (buf == -3.0).all()  # nothing else was written


def test_captured_answers_over_queries(lbm, net):  # noqa: F811
    import torch
    n = 300
    x = _queries(n)
    want = net.predict(x)
    buf = torch.zeros(65 * n, device="cuda:0")
    xd = torch.from_numpy(x).to("cuda:0")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        buf[:5 * n] = xd.view(-1)
        net.predict_noalloc(buf[:5 * n].view(n, 5), buf.view(n, 65), stream=torch.cuda.current_stream())
    for k in range(3):
        PT.say(f"[surrogate overlap] replay {k}")
        buf.fill_(float(k))
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(buf.view(n, 65).cpu().numpy(), want)


@pytest.mark.parametrize("n", [33, 1024, 1025, 2500])
def test_host_answers_over_queries(lbm, net, n):  # noqa: F811
    x = _queries(n)
    want = net.predict(x)
    for place in _places(n):
        PT.say(f"[surrogate overlap] host, {n} rows at {place}")
        lead = 5 * n
        buf = np.full(lead + 65 * n + lead, -3.0, dtype=np.float32)
        q = buf[lead + place:lead + place + 5 * n]
        q[:] = x.ravel()
        lbm.check(lbm.lib().surr_predict(net.h, q.ctypes.data, n, buf[lead:].ctypes.data))
        assert np.array_equal(buf[lead:lead + 65 * n].reshape(n, 65), want), place
        q[:] = buf[lead:lead + 65 * n] = -3.0
        assert (buf == -3.0).all()  # nothing else was written
