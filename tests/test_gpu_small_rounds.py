"""The round of a small model around the sizes where it runs in one block, up to 4096 parameters and three workers; the sum of a large
model's distances around the number of partial sums that are loaded together."""
import numpy as np
import pytest
import torch

from oracle import dw_oracle as O
from paper_2409_09242_amd import binding as B
from paper_2409_09242_amd import workloads as W
from parity import RTOL_UPDATE, close, oracle_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [B.DW_DYNAMIC, B.DW_DYNAMIC | B.DW_SEQUENTIAL])
@pytest.mark.parametrize("P", [4, 4032, 4096, 4100])
@pytest.mark.parametrize("k", [1, 3, 4])
def test_rounds_around_one_block_follow_the_oracle(P, k, mode):
    print("small round", P, k, mode, flush=True)
    rng = W.rng_for(91, 23)
    theta0 = rng.uniform(-0.01, 0.01, size=P).astype(np.float32)
    w = W.scaled(W.C5, k=k, n_params=P, seed=91)
    h = B.Handle(B.config_from_workload(w), theta0)
    tr = O.OracleTrainer(oracle_config(w, dims=None), theta0.astype(np.float64))
    for step in range(3):
        g, hz = (rng.normal(0, 0.1, size=(k, P)).astype(np.float32) for _ in range(2))
        part = None if k < 3 else np.array([1, step == 1, 1, 1][:k], dtype=np.uint8)
        h.update_only(torch.from_numpy(g).cuda(), torch.from_numpy(hz).cuda())
        tr.update_only(g, hz)
        assert h.elastic_sync(mode, tau=1, participate=part)
        tr.elastic_sync(O.MODE_DYNAMIC, tau=1, participate=part, **({"sequential": True} if mode & B.DW_SEQUENTIAL else {}))
        for i in range(k):
            close(h.get_state(B.DW_S_THETA, i), tr.theta[i], RTOL_UPDATE, "small round theta[%d]" % i)
        close(h.get_state(B.DW_S_CENTRE), tr.centre, RTOL_UPDATE, "small round centre")


@pytest.mark.parametrize("k", [1, 4])
def test_the_bf16_weights_follow_the_round(k):
    """After a step and a round the bf16 copy the next step reads is that of the pulled parameters: a second handle given those
    parameters has the same activations."""
    dims, batch = (24, 40, 7), 8
    cfg = B.make_config(dims=dims, k=k, batch=batch, bf16=True)
    theta0 = (W.rng_for(92, 23).random(B.param_count(cfg), dtype=np.float32) - 0.5)
    x = torch.randn((k, batch, dims[0]), generator=torch.Generator().manual_seed(92)).to(torch.bfloat16).cuda()
    y = torch.zeros((k, batch), dtype=torch.int32, device="cuda")
    a, b = B.Handle(cfg, theta0), B.Handle(cfg, theta0)
    a.worker_step(x, y)
    assert a.elastic_sync(B.DW_FIXED, tau=1)
    for i in range(k):
        b.set_state(B.DW_S_THETA, i, a.get_state(B.DW_S_THETA, i))
    a.worker_step(x, y); b.worker_step(x, y)
    for i in range(k):
        np.testing.assert_array_equal(a.get_state(B.DW_S_ACT + 1, i), b.get_state(B.DW_S_ACT + 1, i))


@pytest.mark.parametrize("P", [66 << 10, (1 << 20) + 4, 1 << 23, (1 << 23) + 4])
def test_the_distance_of_many_partial_sums(P):
    """72, 1032, 8192 (one load of each thread's eight) and 8200 partial sums of 1024 parameters each: u is the logarithm of the
    distance, which fp32 squares of the stored parameters give to 2^-23."""
    rng = W.rng_for(93, 23)
    theta0 = rng.uniform(-0.01, 0.01, size=P).astype(np.float32)
    cfg = B.make_config(dims=None, n_params=P, k=2, optimizer=B.DW_OPT_SGD, lr=0.1)
    h = B.Handle(cfg, theta0)
    g = torch.randn((2, P), generator=torch.Generator(device="cuda").manual_seed(93), device="cuda")
    h.update_only(g, None)
    theta = [h.get_state(B.DW_S_THETA, i).astype(np.float64) for i in range(2)]
    assert h.elastic_sync(B.DW_FIXED, tau=1)
    for i in range(2):
        want = np.log(np.linalg.norm(theta[i] - theta0.astype(np.float64)))
        assert abs(h.get_state(B.DW_S_SCORE, i)[0] - want) < 1e-6
