"""The small models' product kernels where their steps end: one to five k-steps for a wave, data gradients of one step, of an uneven number
and in slices, weight gradients of all layers in one launch over one to five tiles of samples, and weight gradients beyond the
range of the pieces."""
import numpy as np
import pytest
import torch

import test_gpu_cnn as N
import test_gpu_f32_pieces as P
from oracle import dw_cnn as OC
from oracle import dw_oracle as O
from paper_2409_09242_amd import binding as B
from paper_2409_09242_amd import workloads as W
from parity import RTOL_GRAD, close_layers, oracle_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,batch,k", [
    ((36, 32, 4), 1, 1),                 # one sample, contractions of 36 and of 4
    ((516, 260, 68, 5), 31, 1),          # 17 steps of 32 k over eight waves; data gradient of three steps for two ... eight waves
    ((768, 100, 772, 9), 64, 2),         # three steps a wave and 25 of eight waves, the last of four k; two tiles of samples
    ((1028, 36, 1036, 3), 65, 1),        # four and five steps a wave
    ((128, 64, 1300, 10), 96, 1),        # data gradient through 1300 outputs in slices; three tiles of samples
    ((3072, 256, 16), 160, 4),           # twelve steps a wave; five tiles of samples
])
def test_steps_and_tiles_follow_the_oracle(dims, batch, k):
    P.test_tile_and_chain_edges_follow_the_oracle(dims, batch, k)


@pytest.mark.parametrize("dims,batch,k", [
    ((32, 2048, 64, 5), 64, 4), ((32, 2052, 64, 5), 64, 4),        # data gradient: 512 blocks of 32 x 32, then 520 in 64 x 64 tiles
    ((32, 3072, 256, 5), 64, 4), ((32, 3076, 256, 5), 64, 4),      # 768 blocks, then 776 in slices of the tiles
    ((32, 256, 896, 5), 64, 4), ((32, 256, 900, 5), 64, 4),        # few blocks: up to 896 columns, then slices
    ((16, 2048, 1024, 5), 64, 4), ((16, 2048, 1028, 5), 64, 4),    # later layer's forward product: 256 blocks, then 264 in slices
    ((1156, 2048, 5), 64, 4), ((1156, 508, 5), 64, 4),             # first layer's: 128 tiles of 64 x 64, then 32
])
def test_products_on_either_side_of_the_rules_lines(dims, batch, k):
    P.test_tile_and_chain_edges_follow_the_oracle(dims, batch, k)


def test_data_gradient_to_the_pooled_map_in_slices(monkeypatch):
    """A long contraction over few columns of the pooled map."""
    name = "few columns, long contraction"
    monkeypatch.setitem(N.SPECS, name, (OC.CnnSpec(img=(12, 10, 1), conv=(8,), fc=(1028, 7)), 5, 2))
    N.test_cnn_step_matches_the_oracle(name, 0)


@pytest.mark.parametrize("dims,batch,k", [((32, 2052, 64, 5), 64, 4), ((32, 3072, 256, 5), 64, 4), ((32, 2052, 644, 5), 64, 4),
                                          ((16, 2048, 1028, 5), 64, 4), ((1156, 2048, 5), 64, 4)])
def test_first_order_steps_on_either_side_of_the_rules_lines(dims, batch, k):
    theta0, x, y = P._inputs(dims, batch, k, 80)
    w = W.scaled(W.C2, k=k, dims=dims, batch=batch, input_dist="normal", optimizer=B.DW_OPT_SGD, seed=80)
    h = B.Handle(B.config_from_workload(w), theta0)
    tr = O.OracleTrainer(oracle_config(w), theta0.astype(np.float64))
    h.worker_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
    tr.worker_step(x, y)
    for i in range(k):
        close_layers(h.get_state(B.DW_S_G, i), tr.traces[i].g, dims, RTOL_GRAD, "g[%d]" % i)


@pytest.mark.parametrize("dims,batch,k", [((516, 260, 68, 5), 31, 1), ((768, 100, 772, 9), 64, 2), ((128, 64, 1300, 10), 160, 1)])
def test_first_order_steps(dims, batch, k):
    P.test_first_order_steps_compute_the_plain_products_alone(B.DW_OPT_MOMENTUM, dims, batch, k)


def test_activations_beyond_the_pieces_range():
    """Activations of 2^100 give results of 2^80 and more in the second layer's weight gradient: its tiles are computed again from whole
    floats and are those of the same network with the factor taken out, times the factor."""
    dims, batch, k = (68, 100, 132, 6), 70, 1
    theta0, x, y = P._inputs(dims, batch, k, 83)
    h0 = P._step(dims, batch, k, theta0, x, y)[1]
    # the first layer's activations 2^100 times as large, the second's weights 2^-100: everything behind stays as it is
    f = np.float32(2.0 ** 100)
    n1 = dims[0] * dims[1] + dims[1]
    t = theta0.copy()
    t[:n1] *= f
    t[n1:n1 + dims[1] * dims[2]] /= f
    h1 = P._step(dims, batch, k, t, x, y)[1]
    g0, g1 = (h.get_state(B.DW_S_G, 0).astype(np.float64) for h in (h0, h1))
    w2 = slice(n1, n1 + dims[1] * dims[2])
    assert np.abs(g1[w2]).max() > 2.0 ** 80                    # (of the pieces' 2^48-fold results: past the largest float)
    # two fp32 gradients of the same network, each held to RTOL_GRAD of the exact one
    assert np.all(np.abs(g1[w2] / f - g0[w2]) <= 2 * RTOL_GRAD * np.maximum(np.abs(g0[w2]), np.sqrt(np.mean(g0[w2] ** 2))))
