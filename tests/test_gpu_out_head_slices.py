"""The fp32 output layer whose contraction is cut over the grid: few samples, 2048 inputs and more."""
import numpy as np
import pytest
import torch

from oracle import dw_oracle as O
from paper_2409_09242_amd import binding as B
from paper_2409_09242_amd import workloads as W
from parity import RTOL_GRAD, RTOL_HV, close_layers, oracle_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,batch,k,opt", [
    ((2048, 10), 17, 2, 0),              # the shortest that is cut, in whole groups of 64; a ragged block of samples; no hidden layer
    ((2044, 10), 17, 2, 0),              # four short of it
    ((32, 2052, 16), 93, 3, 0),          # four past a whole group
    ((32, 2052, 3), 5, 3, 1),
    ((16388, 7), 40, 1, 0),              # 32 slices of 576 where 29 cover the contraction: the last three are empty
    ((2056, 10), 4096, 1, 0),            # 256 blocks of samples: the most that are cut
    ((2056, 10), 4097, 1, 0),            # and one more
])
def test_output_layers_around_the_cut_follow_the_oracle(dims, batch, k, opt):
    print("output layer in slices", dims, batch, k, opt, flush=True)
    w = W.scaled(W.C2, k=k, dims=dims, batch=batch, input_dist="normal", optimizer=opt, seed=90)
    theta0 = W.init_theta(dims, 90).astype(np.float32)
    x, y = W.minibatch_pool(w, 1)
    h = B.Handle(B.config_from_workload(w), theta0)
    loss = torch.zeros(k, device="cuda")
    active = None if k < 3 else np.array([1, 0, 1], dtype=np.uint8)
    h.worker_step(torch.from_numpy(x[0]).cuda(), torch.from_numpy(y[0]).cuda(), loss=loss, active=active)
    tr = O.OracleTrainer(oracle_config(w), theta0.astype(np.float64))
    ref = tr.worker_step(x[0], y[0], active=active)
    for i in range(k):
        if active is not None and not active[i]:
            np.testing.assert_array_equal(h.get_state(B.DW_S_THETA, i), theta0)
            continue
        np.testing.assert_allclose(loss[i].item(), ref[i], rtol=1e-5)
        close_layers(h.get_state(B.DW_S_G, i), tr.traces[i].g, dims, RTOL_GRAD, "slices g[%d]" % i)
        if opt == 0:
            close_layers(h.get_state(B.DW_S_HZ, i), tr.traces[i].hz, dims, RTOL_HV, "slices hz[%d]" % i)
