"""The fp32 products in bf16 pieces: infinities and NaN, huge and tiny operands, and one network per edge of the tiles."""
import numpy as np
import pytest
import torch

from oracle import dw_oracle as O
from paper_2409_09242_amd import binding as B
from paper_2409_09242_amd import workloads as W
from parity import RTOL_GRAD, RTOL_HV, TIE_BAND, bound_ties, check_hidden, close_layers, gpu_hidden, oracle_config, slopes_of

pytestmark = pytest.mark.gpu


def _step(dims, batch, k, theta0, x, y):
    w = W.scaled(W.C2, k=k, dims=dims, batch=batch, input_dist="normal")
    h = B.Handle(B.config_from_workload(w), theta0.astype(np.float32))
    loss = torch.zeros(k, device="cuda")
    h.worker_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), loss=loss)
    return w, h, loss


def _inputs(dims, batch, k, seed):
    w = W.scaled(W.C2, k=k, dims=dims, batch=batch, input_dist="normal", seed=seed)
    x, y = W.minibatch_pool(w, 1)
    return W.init_theta(dims, seed), x[0], y[0]


@pytest.mark.parametrize("dims,batch,k", [
    ((260, 68, 132, 10), 65, 2),         # gradients one row, four columns past a 64 x 64 tile, the data gradient in two slices; forward
                                         # products in the small-model kernel, 4 past a step of 32 k
    ((132, 192, 64, 3), 31, 3),          # minibatch shorter than a tile of 32 k
    ((1280, 256, 128, 16), 128, 2),      # whole tiles, the first forward product in slices
    ((2048, 512, 10), 128, 4),           # the longest contraction of the small-model kernel
    ((132, 1028, 1036, 7), 193, 4),      # every hidden product in 64 x 64 tiles (272 of them): ragged rows, columns and last k-tile, with
                                         # and without the input's derivative
])
def test_tile_and_chain_edges_follow_the_oracle(dims, batch, k):
    print("pieces", dims, batch, k, flush=True)
    theta0, x, y = _inputs(dims, batch, k, 77)
    w, h, loss = _step(dims, batch, k, theta0, x, y)
    tr = O.OracleTrainer(oracle_config(w), theta0.astype(np.float64))
    hidden = gpu_hidden(h, w)                                  # (a unit within rounding of its kink may be on either side)
    tr.worker_step(x, y, tie_band=TIE_BAND, tie_choice=slopes_of(hidden))
    check_hidden(hidden, {i: tr.traces[i] for i in range(k)}, False, "pieces")
    bound_ties(False)
    for i in range(k):
        close_layers(h.get_state(B.DW_S_G, i), tr.traces[i].g, dims, RTOL_GRAD, "g[%d]" % i)
        close_layers(h.get_state(B.DW_S_HZ, i), tr.traces[i].hz, dims, RTOL_HV, "hz[%d]" % i)


@pytest.mark.parametrize("scale", [2.0 ** -60, 2.0 ** 40])
def test_scaled_weights_scale_the_products_exactly(scale):
    """Powers of two commute with the splitting: scaling the first layer's weights and bias by one and its inputs by none
    scales its activations bit for bit (no piece over- or underflows at 2^-60 or 2^40)."""
    dims, batch, k = (260, 96, 68, 10), 64, 1
    theta0, x, y = _inputs(dims, batch, k, 78)
    n1 = dims[0] * dims[1] + dims[1]
    _, h0, _ = _step(dims, batch, k, theta0, x, y)
    t1 = theta0.copy(); t1[:n1] *= np.float32(scale)
    _, h1, _ = _step(dims, batch, k, t1, x, y)
    np.testing.assert_array_equal(h1.get_state(B.DW_S_ACT + 1, 0), h0.get_state(B.DW_S_ACT + 1, 0) * np.float32(scale))


@pytest.mark.parametrize("dims,batch", [((256, 96, 68, 10), 64), ((256, 96, 32, 10), 130)])
def test_infinities_stay_infinite_and_nans_stay_nans(dims, batch):
    """The small-model kernel (the tiles: test_gpu_f32_redo.py).  One input entry is inf: the units of the first layer are +-inf there, by the sign of their weight, and the
    activation is inf or 0, as any fp32 sum gives it; a NaN input makes the sample's pre-activations NaN, which the
    ReLU's comparison turns into 0.  Other samples of the block are computed again on another instruction, so both are
    sums of the same K products in some order: within 2 K 2^-24 sum |x w| of each other."""
    k = 1
    theta0, x, y = _inputs(dims, batch, k, 79)
    _, h0, _ = _step(dims, batch, k, theta0, x, y)
    a0 = h0.get_state(B.DW_S_ACT + 1, 0)
    xb = x.copy()
    xb[0, 5, 17] = np.inf; xb[0, 40, 3] = -np.inf; xb[0, 41, 200] = np.nan; xb[0, 42, 9] = np.finfo(np.float32).max
    _, h1, _ = _step(dims, batch, k, theta0, xb, y)
    a1 = h1.get_state(B.DW_S_ACT + 1, 0)
    W1 = theta0[:dims[0] * dims[1]].reshape(dims[1], dims[0])
    np.testing.assert_array_equal(a1[5], np.where(W1[:, 17] > 0, np.inf, 0))
    np.testing.assert_array_equal(a1[40], np.where(W1[:, 3] < 0, np.inf, 0))
    np.testing.assert_array_equal(a1[41], 0)
    want = np.maximum(W1[:, 9].astype(np.float64) * np.finfo(np.float32).max, 0)      # the other terms are 1e38 times smaller
    np.testing.assert_allclose(a1[42], want, rtol=1e-6)
    rest = [i for i in range(batch) if i not in (5, 40, 41, 42)]
    bound = 2 * dims[0] * 2.0 ** -24 * (np.abs(x[0][rest]) @ np.abs(W1).T + 1)
    assert np.all(np.abs(a1[rest] - a0[rest]) <= bound)


@pytest.mark.parametrize("opt", [B.DW_OPT_SGD, B.DW_OPT_MOMENTUM])
@pytest.mark.parametrize("dims,batch,k", [
    ((260, 68, 132, 10), 65, 2),         # every forward product in the small-model kernel, contraction past a step of 32 k; data
                                         # gradient in two slices
    ((64, 36, 4), 5, 1),                 # contractions of at most two steps
    ((132, 1028, 260, 7), 256, 4),       # tiles of 64 x 64, whole and ragged
])
def test_first_order_steps_compute_the_plain_products_alone(opt, dims, batch, k):
    print("first order", opt, dims, batch, k, flush=True)
    theta0, x, y = _inputs(dims, batch, k, 80)
    w = W.scaled(W.C2, k=k, dims=dims, batch=batch, input_dist="normal", optimizer=opt, seed=80)
    h = B.Handle(B.config_from_workload(w), theta0)
    tr = O.OracleTrainer(oracle_config(w), theta0.astype(np.float64))
    loss = torch.zeros(k, device="cuda")
    h.worker_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), loss=loss)
    np.testing.assert_allclose(loss.cpu().numpy(), tr.worker_step(x, y), rtol=1e-5)
    for i in range(k):
        close_layers(h.get_state(B.DW_S_G, i), tr.traces[i].g, dims, RTOL_GRAD, "g[%d]" % i)
        # the step is lr * g with g held to 1e-4; read back as a difference of two stored parameters it carries an ulp of
        # theta, up to 2^-24 * 0.5 = 3e-8, against lr * rms(g) of 2e-5 and more in every layer
        close_layers(h.get_state(B.DW_S_THETA, i) - theta0, tr.theta[i] - theta0, dims, 2e-3, "update[%d]" % i)


def test_a_first_order_step_with_the_callers_z_leaves_its_hessian_vector_product_readable():
    dims, batch, k = (132, 192, 64, 3), 31, 2
    theta0, x, y = _inputs(dims, batch, k, 81)
    z = torch.from_numpy(np.random.default_rng(81).integers(0, 2 ** 32, size=(k, 2 * ((len(theta0) + 63) // 64)),
                                                            dtype=np.uint32).view(np.int32)).cuda()
    hz = []
    for opt in (B.DW_OPT_ADAHESSIAN, B.DW_OPT_MOMENTUM):
        w = W.scaled(W.C2, k=k, dims=dims, batch=batch, input_dist="normal", optimizer=opt, seed=81)
        h = B.Handle(B.config_from_workload(w), theta0.astype(np.float32))
        h.worker_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), zbits=z)
        hz.append([h.get_state(B.DW_S_HZ, i) for i in range(k)])
    np.testing.assert_array_equal(hz[0], hz[1])                       # the same products of the same kernels
