"""bf16 output layer and softmax head in one kernel: widths that are not whole steps of the contraction's four waves,
minibatches that are not whole blocks of 16 samples, the class counts' ends, and the network without a hidden layer,
whose output layer is a product of its own."""
import numpy as np
import pytest
import torch

from paper_2409_09242_amd import binding as B
from paper_2409_09242_amd import workloads as W

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _f64_of_bf16(bits):
    return (bits.astype(np.uint32) << 16).view(np.float32).astype(np.float64)


def _head64(S, RS, y):
    p = np.exp(S - S.max(1, keepdims=True))
    p /= p.sum(1, keepdims=True)
    n = len(y)
    d = p.copy()
    d[np.arange(n), y] -= 1.0
    diff = RS[:, :, None] - RS[:, None, :]
    rd = p * np.einsum("bj,bij->bi", p, diff)
    spread = np.einsum("bj,bij->bi", p, np.abs(diff))
    return p, d / n, rd / n, spread, -np.log(p[np.arange(n), y]).mean()


@pytest.mark.parametrize("dims,batch", [
    ((8, 8, 2), 1),              # one load of 8: one lane group of the first wave, the others have nothing
    ((8, 136, 10), 15),          # waves of 64, 64, 8 and 0
    ((8, 776, 16), 17),          # a second block with one sample; every class lane
    ((8, 1024, 10), 33),         # whole steps: the instance without the check at the end
    ((8, 1032, 3), 16),          # eight past them
    ((8, 2056, 10), 48),
    ((40, 10), 17),              # no hidden layer
])
def test_output_layer_and_head_against_64_bits(dims, batch):
    """Inputs of -1, 0, 1 make the first layer's R-activations small integers, exact in bf16; its activations are read
    back.  What is left is the output layer: fp32 sums of K + 1 terms (2 (K + 8) 2^-24 of the terms' sum of magnitudes,
    the matrix unit may truncate), the head in fp32, and the rounding of d and Rd to bf16 (2^-9) before their column
    sums, which are the bias gradient and its R-companion."""
    print("out_head_bf16", dims, batch, flush=True)
    k, K, C = 2, dims[-2], dims[-1]
    w = W.scaled(W.C2, k=k, dims=dims, batch=batch, bf16=True, seed=31)
    theta0 = W.init_theta(dims, 31).astype(np.float32)
    h = B.Handle(B.config_from_workload(w), theta0)
    rng = np.random.default_rng(K + batch)
    x = rng.integers(-1, 2, size=(k, batch, dims[0])).astype(np.float32)
    y = rng.integers(0, C, size=(k, batch)).astype(np.int32)
    loss = torch.zeros(k, device="cuda")
    h.worker_step(torch.from_numpy(x).cuda().to(torch.bfloat16).view(torch.int16), torch.from_numpy(y).cuda(), loss=loss)
    woff = len(theta0) - C * K - C
    Wl = _f64_of_bf16(torch.from_numpy(theta0[woff:woff + C * K]).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16))
    Wl, bl = Wl.reshape(C, K), theta0[woff + C * K:].astype(np.float64)
    for i in range(k):
        words = h.get_state(B.DW_S_ZBITS, i)
        z = np.unpackbits(words.view(np.uint8), bitorder="little")[:len(theta0)].astype(np.float64) * 2 - 1
        V, c = z[woff:woff + C * K].reshape(C, K), z[woff + C * K:]
        if len(dims) == 3:
            A = _f64_of_bf16(h.get_state(B.DW_S_ACT + 1, i))
            n1 = dims[0] * K
            RA = (A > 0) * (x[i].astype(np.float64) @ z[:n1].reshape(K, dims[0]).T + z[n1:n1 + K])
        else:
            A, RA = x[i].astype(np.float64), np.zeros((batch, K))
        S, RS = A @ Wl.T + bl, RA @ Wl.T + A @ V.T + c
        E = (2 * (K + 8) * U * (np.abs(A) @ np.abs(Wl).T + np.abs(bl))).max(1, keepdims=True)
        ER = (4 * (K + 8) * U * (np.abs(RA) @ np.abs(Wl).T + np.abs(A) @ np.abs(V).T + 1)).max(1, keepdims=True)
        p, d, rd, spread, mean_loss = _head64(S, RS, y[i])
        ed = np.abs(d) * (2 * E + 40 * U)
        erd = p / batch * (2 * ER + (6 * E + 80 * U) * spread)
        round_off = 2.0 ** -9 + batch * U
        got = h.get_state(B.DW_S_G, i)[woff + C * K:].astype(np.float64)
        rgot = h.get_state(B.DW_S_HZ, i)[woff + C * K:].astype(np.float64)
        assert np.all(np.abs(got - d.sum(0)) <= (1.01 * ed + round_off * np.abs(d)).sum(0) + 1e-30)
        assert np.all(np.abs(rgot - rd.sum(0)) <= (1.01 * erd + round_off * np.abs(rd)).sum(0) + 1e-30)
        assert abs(float(loss[i]) - mean_loss) <= (2 * E).mean() + (40 + batch) * U * (1 + mean_loss)
