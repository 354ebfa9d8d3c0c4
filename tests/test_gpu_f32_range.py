"""The fp32 products far from 1: tiny operands and tiny results keep their 24 bits, through every kind of product."""
import numpy as np
import pytest
import torch

from oracle import dw_oracle as O
from paper_2409_09242_amd import binding as B
from paper_2409_09242_amd import workloads as W
from parity import RTOL_GRAD, RTOL_HV, close_layers, oracle_config

pytestmark = pytest.mark.gpu

SMALL = ((260, 68, 132, 10), 65, 2)          # every forward product in the small-model kernel
TILES = ((260, 516, 260, 10), 193, 13)       # hidden products in at least 256 tiles of 64 x 64


def _problem(dims, batch, k, seed, **kw):
    w = W.scaled(W.C2, k=k, dims=dims, batch=batch, input_dist="normal", seed=seed, **kw)
    x, y = W.minibatch_pool(w, 1)
    return w, W.init_theta(dims, seed).astype(np.float32), x[0].astype(np.float32), y[0]


def _step(w, theta0, x, y):
    h = B.Handle(B.config_from_workload(w), theta0)
    h.worker_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
    return h


@pytest.mark.parametrize("dims,batch,k", [SMALL, TILES])
def test_tiny_inputs_under_huge_weights_give_the_same_bits(dims, batch, k):
    """Inputs times 2^-104 and first-layer weights times 2^104 leave every product of the two as it is, so the activations
    are the same bits and the first layer's gradient is 2^-104 times the same bits.  (|x| >= 2^-10, |W| < 1: no operand
    leaves the normal numbers or reaches 2^104.)"""
    print("tiny inputs", dims, batch, k, flush=True)
    w, theta0, x, y = _problem(dims, batch, k, 82, optimizer=B.DW_OPT_SGD)
    x = np.where(np.abs(x) < 2.0 ** -10, np.float32(2.0 ** -10), x)
    n1 = dims[0] * dims[1]
    h0 = _step(w, theta0, x, y)
    t1 = theta0.copy()
    t1[:n1] *= np.float32(2.0 ** 104)
    h1 = _step(w, t1, x * np.float32(2.0 ** -104), y)
    for i in range(k):
        np.testing.assert_array_equal(h1.get_state(B.DW_S_ACT + 1, i), h0.get_state(B.DW_S_ACT + 1, i))
        g0, g1 = h0.get_state(B.DW_S_G, i), h1.get_state(B.DW_S_G, i)
        np.testing.assert_array_equal(g1[:n1], g0[:n1] * np.float32(2.0 ** -104))
        np.testing.assert_array_equal(g1[n1:], g0[n1:])


@pytest.mark.parametrize("dims,batch,k", [SMALL, TILES])
def test_tiny_gradients_follow_the_oracle(dims, batch, k):
    """Output weights times 2^-112: the gradients of the layers below are of 2^-115 and less, and as close to the oracle
    as at any other size (both are scaled up by 2^112 for the comparison)."""
    print("tiny gradients", dims, batch, k, flush=True)
    w, theta0, x, y = _problem(dims, batch, k, 83)
    offs, _ = O.layer_offsets(dims)
    last = slice(offs[-1][0], offs[-1][1])
    theta0[last] *= np.float32(2.0 ** -112)
    h = _step(w, theta0, x, y)
    tr = O.OracleTrainer(oracle_config(w), theta0.astype(np.float64))
    tr.worker_step(x, y)
    up = 2.0 ** 112
    below = slice(0, offs[-1][0])
    for i in range(k):
        g, ref = h.get_state(B.DW_S_G, i).astype(np.float64), tr.traces[i].g.copy()
        g[below] *= up; ref[below] *= up
        close_layers(g, ref, dims, RTOL_GRAD, "g[%d]" % i)
        close_layers(h.get_state(B.DW_S_HZ, i), tr.traces[i].hz, dims, RTOL_HV, "hz[%d]" % i)


@pytest.mark.parametrize("dims", [(260, 68, 132, 10), (260, 516, 260, 10)])
def test_a_single_product_is_rounded_once(dims):
    """One sample: gW_l = d_l a_{l-1}^T is one product an entry, and HzW_1 = Rd_1 x^T too (the input has no derivative).
    d_l and Rd_l are the bias gradients then, so every entry is known to the bit."""
    w, theta0, x, y = _problem(dims, 1, 2, 84)
    h = _step(w, theta0, x, y)
    offs, _ = O.layer_offsets(dims)
    for i in range(2):
        g, hz = h.get_state(B.DW_S_G, i), h.get_state(B.DW_S_HZ, i)
        for l, (wo, bo) in enumerate(offs, start=1):
            a = x[i, 0] if l == 1 else h.get_state(B.DW_S_ACT + l - 1, i).reshape(-1)
            np.testing.assert_array_equal(g[wo:bo], np.outer(g[bo:bo + dims[l]], a).reshape(-1))
            if l == 1:
                np.testing.assert_array_equal(hz[wo:bo], np.outer(hz[bo:bo + dims[l]], a).reshape(-1))


@pytest.mark.parametrize("classes", [2, 3, 4])
def test_the_data_gradient_through_few_classes_is_as_close_as_fp32_sums(classes):
    """One sample: d_1 = d_L W_2 is a sum of `classes` products, d_L and d_1 are the bias gradients.  A chain of K fp32
    multiply-adds is off by at most 2^-24 at each of its K steps; in the 2-norm the library is no further off than
    such a chain computed here."""
    dims = (260, 2052, classes)
    w, theta0, x, y = _problem(dims, 1, 3, 85)
    h = _step(w, theta0, x, y)
    (_, b1), (w2, b2) = O.layer_offsets(dims)[0]
    W2 = theta0[w2:b2].reshape(classes, dims[1])
    for i in range(3):
        g, on = h.get_state(B.DW_S_G, i), h.get_state(B.DW_S_ACT + 1, i).reshape(-1) > 0
        p = g[b2:b2 + classes, None].astype(np.float64) * W2
        want = np.where(on, p.sum(0), 0.0)
        err = np.abs(g[b1:b1 + dims[1]] - want)
        assert np.all(err <= 1.001 * classes * 2.0 ** -24 * np.abs(p).sum(0)), (err / np.abs(p).sum(0)).max()
        chain = np.zeros(dims[1], dtype=np.float32)
        for q in p:
            chain = (chain + q).astype(np.float32)
        assert np.linalg.norm(err) <= 1.02 * np.linalg.norm(np.where(on, chain, 0.0) - want)     # (2 %: 1000 roundings)
