"""The surrogate's fused passes at the edges of their tiles: 32 samples per
workgroup, 16 samples per contraction step, 1024 samples per launch that reads
host memory."""

import numpy as np
import pytest

import parity as PT
from oracle import mlp_oracle as M
from paper_1309_6726_amd import inputs
from test_gpu_surrogate import GRAD_BOUND, _data, _rel, surr  # noqa: F401

pytestmark = pytest.mark.gpu


# The forward bound (1% relative L2) is the one of test_forward_matches_fp64_oracle:
# BF16 operands (2^-9 each) through four layers.
@pytest.mark.parametrize("n", [1, 31, 32, 33, 255, 1024, 1025, 2100])
def test_predict_rows(surr, n):  # noqa: F811
    PT.say(f"[surrogate rows] predict {n}")
    net = surr.Surrogate(max_batch=32, max_data=1)
    p = inputs.mlp_init_params(3).astype(np.float32)
    net.set_params(p)
    x, _ = _data(n, 21)
    y = net.predict(x)
    yo, _ = M.forward(p.astype(np.float64), x, net.lo, net.hi)
    assert _rel(y, yo) <= 1e-2
    # a row's answer does not depend on the rows beside it
    for k in {0, n // 2, n - 1}:
        assert np.array_equal(net.predict(x[k:k + 1])[0], y[k])


# 1100 rows: samples copied to the device instead of read from host memory
@pytest.mark.parametrize("n", [1, 16, 17, 32, 33, 95, 256, 1100])
def test_gradient_rows(surr, n):  # noqa: F811
    PT.say(f"[surrogate rows] gradients {n}")
    net = surr.Surrogate(max_batch=max(n, 40), max_data=1)
    p = inputs.mlp_init_params(8).astype(np.float32)
    net.set_params(p)
    w = np.linspace(0.5, 2.0, 65).astype(np.float32)
    net.set_loss_weights(w)
    x, t = _data(n, 5)
    p64, w64 = p.astype(np.float64), w.astype(np.float64)
    lo_, go = M.loss_and_grad(p64, x, t, net.lo, net.hi, w64)
    E = M.grad_error_scale(p64, x, t, net.lo, net.hi, w64)
    for _ in range(2):  # the loss starts from zero each time
        loss, g = net.gradients(x, t)
        assert abs(loss - lo_) <= 1e-2 * lo_
        assert (np.abs(g - go) <= GRAD_BOUND * E).all()


def test_ragged_epoch_matches_oracle_adam(surr):  # noqa: F811
    """An epoch of 150 samples in minibatches of 64 (the last of 22) equals
    the oracle's Adam on the gradients the GPU reports for each minibatch, and
    its loss is their mean."""
    PT.say("[surrogate rows] epoch 150/64")
    x, t = _data(150, 9)
    p = inputs.mlp_init_params(4).astype(np.float32)
    perm = np.argsort(inputs.uniform53(3, np.arange(150, dtype=np.uint64))).astype(np.int32)
    net = surr.Surrogate(max_batch=64, max_data=150)
    net.set_params(p)
    net.set_data(x, t)
    loss = net.train_epoch(perm, 64, 1e-3)
    ref = surr.Surrogate(max_batch=64, max_data=150)
    po, m, v, losses = p.astype(np.float64), np.zeros(p.size), np.zeros(p.size), []
    for s, off in enumerate(range(0, 150, 64), 1):
        ref.set_params(po.astype(np.float32))
        at = perm[off:off + 64]
        ls, g = ref.gradients(x[at], t[at])
        losses.append(ls)
        po, m, v = M.adam_step(po, m, v, g.astype(np.float64), s, 1e-3)
    # Adam moves an entry by at most about lr a step; where a BF16 copy of a
    # weight rounds differently in the two runs (FP32 against FP64 Adam, 2^-24
    # apart), later gradients differ by 2^-8 of their products, which moves
    # the few entries whose gradient nearly cancels by up to a step's lr
    d = np.abs(net.params() - po)
    assert d.max() <= 2e-3 and np.mean(d <= 1e-6 + 1e-5 * np.abs(po).max()) >= 0.99
    assert abs(loss - np.mean(losses)) <= 1e-4 * loss
