"""The streaming update and the pull at the edges of their blocks and stretches, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import dw_oracle as O
from paper_2409_09242_amd import binding as B
from paper_2409_09242_amd import workloads as W
from parity import RTOL_UPDATE, close, oracle_config

pytestmark = pytest.mark.gpu

STRETCH = 1 << 20            # parameters of one worker that are walked before the next worker's turn


@pytest.mark.parametrize("P,k,avg_block,opt", [
    (8192, 3, 256, 0), (8196, 3, 4, 0),                      # a whole group of eight blocks; four parameters more
    (65536, 2, 1, 0), (65540, 2, 1, 0),                      # weights inside the pull; in a launch of their own
    (STRETCH, 3, 2, 0), (STRETCH + 4, 3, 1, 0), (2 * STRETCH + 8192, 2, 32, 0), (STRETCH + 1028, 3, 1, 1),
    (STRETCH - 4, 3, 1, 2), (STRETCH + 4, 6, 1, 0),          # six workers: the pull's second batch is not full
])
def test_update_and_round_at_the_edges_of_the_walk(P, k, avg_block, opt):
    print("update stretches", P, k, avg_block, opt, flush=True)
    rng = W.rng_for(50 + k, 29)
    theta0 = rng.uniform(-0.01, 0.01, size=P).astype(np.float32)
    w = W.scaled(W.C5, k=k, n_params=P, avg_block=avg_block, optimizer=opt)
    h = B.Handle(B.config_from_workload(w), theta0)
    tr = O.OracleTrainer(oracle_config(w, dims=None), theta0.astype(np.float64))
    frozen = [i != 1 for i in range(k)]
    for step, (active, part, mode) in enumerate(((None, frozen, 0), (frozen, None, B.DW_SEQUENTIAL))):
        g = (rng.standard_normal((k, P)) * 0.1).astype(np.float32)
        hz = (rng.standard_normal((k, P)) * 0.1).astype(np.float32)
        h.update_only(torch.from_numpy(g).cuda(), torch.from_numpy(hz).cuda(), active=active)
        tr.update_only(g, hz, active=active)
        for i in range(k):
            close(h.get_state(B.DW_S_THETA, i), tr.theta[i], RTOL_UPDATE, "step %d theta[%d]" % (step, i))
            if opt == 0:
                close(h.get_state(B.DW_S_V, i), tr.v[i], RTOL_UPDATE, "step %d v[%d]" % (step, i))
        assert h.elastic_sync(B.DW_DYNAMIC | mode, tau=1, participate=part)
        if mode:
            tr.elastic_sync(O.MODE_DYNAMIC, tau=1, participate=part, sequential=True)
        else:
            tr.elastic_sync(O.MODE_DYNAMIC, tau=1, participate=part)
        for i in range(k):
            assert abs(h.get_state(B.DW_S_SCORE, i)[0] - tr.last_u[i]) < 1e-5, (step, i)
            close(h.get_state(B.DW_S_THETA, i), tr.theta[i], RTOL_UPDATE, "round %d theta[%d]" % (step, i))
        close(h.get_state(B.DW_S_CENTRE), tr.centre, RTOL_UPDATE, "round %d centre" % step)
