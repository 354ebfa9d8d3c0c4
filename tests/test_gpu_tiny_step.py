"""The one-kernel step of small models where its tiles, its four samples a wave and its groups of parameters end: minibatches around
16 and 64 samples, widths that are no multiple of 16, one class and sixteen, models around 4096 parameters (a group of four per
thread, then four), no hidden layer and many."""
import numpy as np
import pytest
import torch

import test_gpu_network as N
from paper_2409_09242_amd import binding as B
from paper_2409_09242_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,batch,k", [
    ((4, 4, 2), 1, 1), ((8, 20, 3), 15, 2), ((12, 16, 16), 17, 3), ((36, 48, 9), 64, 2), ((20, 32, 5), 65, 2),
    ((32, 108, 4), 9, 2),                  # P = 4000
    ((32, 112, 4), 33, 2),                 # P = 4148
    ((64, 72, 40, 10), 20, 2),             # P = 8010
    ((28, 1), 6, 2), ((52, 16), 31, 2),    # no hidden layer: one class (its gradient is zero) and sixteen
    ((16, 12, 20, 8, 28, 12, 7), 18, 2),
])
def test_gradient_and_hvp_of_small_models(dims, batch, k):
    print("tiny", dims, batch, k, flush=True)
    N.test_gradient_and_hvp_match_the_oracle(dims, batch, k)


@pytest.mark.parametrize("dims,batch,k,avg_block,hpow", [
    ((4, 4, 2), 1, 1, 4, 1.0), ((32, 112, 4), 17, 2, 16, 1.0), ((64, 64, 40, 10), 18, 2, 8, 1.0), ((64, 10), 40, 2, 64, 1.0),
])
def test_update_of_small_models(dims, batch, k, avg_block, hpow):
    print("tiny update", dims, batch, k, avg_block, flush=True)
    N.test_small_models_take_the_whole_step_in_one_kernel(dims, batch, k, avg_block, hpow)


@pytest.mark.parametrize("dims,batch,k,one_kernel", [
    ((32, 64, 10), 68, 2, True), ((32, 64, 10), 69, 2, False), ((80, 14), 243, 1, True), ((80, 14), 244, 1, False),
    ((64, 96, 16), 12, 2, True), ((64, 96, 16), 13, 2, False), ((512, 16, 100, 15), 1, 2, False), ((124, 124, 7), 4, 2, False),
])
def test_models_past_the_size_of_the_one_kernel_step_take_the_launches_of_a_layer_each(dims, batch, k, one_kernel):
    """The largest minibatches that the one kernel takes and the next ones, and models that would fit in LDS but are more exact in
    pieces."""
    print("tiny size", dims, batch, k, one_kernel, flush=True)
    h = B.Handle(B.make_config(dims=dims, k=k, batch=batch), np.zeros(B.param_count(B.make_config(dims=dims, k=k, batch=batch)), dtype=np.float32))
    h.profile(True)
    h.worker_step(torch.zeros((k, batch, dims[0]), device="cuda"), torch.zeros((k, batch), dtype=torch.int32, device="cuda"))
    prof = h.profile_read()
    assert (prof["step"][0], prof["update"][0]) == ((1, 0) if one_kernel else (0, 1))
    N.test_gradient_and_hvp_match_the_oracle(dims, batch, k)


def test_a_logit_that_is_infinite_or_no_number():
    """A bias of +inf makes its worker's loss infinite or no number, as softmax in fp32 does, and leaves the other worker's step alone."""
    dims, batch = (8, 12, 5), 6
    cfg = B.make_config(dims=dims, k=2, batch=batch)
    P = B.param_count(cfg)
    theta0 = W.rng_for(94, 23).standard_normal(P).astype(np.float32)
    x = torch.randn((2, batch, dims[0]), generator=torch.Generator().manual_seed(94)).cuda()
    y = torch.zeros((2, batch), dtype=torch.int32, device="cuda")
    out = []
    for bad in (False, True):
        h = B.Handle(cfg, theta0)
        if bad:
            t = theta0.copy(); t[P - 3] = np.inf
            h.set_state(B.DW_S_THETA, 0, t)
        loss = torch.zeros(2, device="cuda")
        h.worker_step(x, y, loss=loss)
        out.append((loss.cpu().numpy(), h.get_state(B.DW_S_THETA, 1)))
    assert np.isfinite(out[0][0]).all() and not np.isfinite(out[1][0][0]) and out[1][0][1] == out[0][0][1]
    np.testing.assert_array_equal(out[0][1], out[1][1])
