"""Tiles of the fp32 products whose results are not finite in bf16 pieces and are computed again on the fp32 instruction: the
products of every direction through the 64 x 64 tiles, their slices, the fused update and the convolutions' views."""
import numpy as np
import pytest
import torch

from oracle import dw_cnn as OC
from oracle import dw_oracle as O
from paper_2409_09242_amd import binding as B
from paper_2409_09242_amd import workloads as W
from parity import RTOL_GRAD, RTOL_HV, close, per_layer
from test_gpu_cnn import _inputs as cnn_inputs
from test_gpu_conv_slabs import second_convolution_on_slabs

pytestmark = pytest.mark.gpu

TILES = ((132, 1028, 1036, 7), 193, 4)       # hidden products of 272 tiles of 64 x 64, no size a multiple of a tile
SLICES = ((260, 68, 132, 10), 65, 2)         # few tiles: forward and data gradient in the small-model kernel


def _inputs(dims, batch, k, seed, **kw):
    w = W.scaled(W.C2, k=k, dims=dims, batch=batch, input_dist="normal", seed=seed, **kw)
    x, y = W.minibatch_pool(w, 1)
    return w, W.init_theta(dims, seed).astype(np.float32), x[0].astype(np.float32), y[0]


def _dual_network(theta, z, x, y, dims, patterns):
    """Gradient and Hessian-vector product in 64 bits, infinities and NaN as fp32 kernels treat them: a unit is on where its
    pre-activation compares greater than 0 (a NaN does not).  `patterns`: which hidden units the library had on; it may differ
    from the 64-bit signs within 1e-5 of the layer's rms only."""
    offs, P = O.layer_offsets(dims)
    Ws = [(theta[w:b].reshape(n, -1).astype(np.float64), z[w:b].reshape(n, -1)) for (w, b), n in zip(offs, dims[1:])]
    bs = [(theta[b:b + n].astype(np.float64), z[b:b + n]) for (w, b), n in zip(offs, dims[1:])]
    L, n = len(dims) - 1, x.shape[0]
    a, ra, on = [x.astype(np.float64)], [np.zeros(x.shape)], []
    g, hz = np.zeros(P), np.zeros(P)
    with np.errstate(all="ignore"):
        for l in range(L):
            (Wl, Vl), (bl, cl) = Ws[l], bs[l]
            s = a[l] @ Wl.T + bl
            rs = a[l] @ Vl.T + cl + (ra[l] @ Wl.T if l else 0.0)
            if l < L - 1:
                finite = np.isfinite(s)
                rms = np.sqrt(np.mean(s[finite & (np.abs(s) < 1e20)] ** 2))
                differ = patterns[l] != (s > 0)
                assert not np.any(differ & ~(np.abs(s) <= 1e-5 * rms)), l
                on.append(patterns[l])
                a.append(np.where(on[l], s, 0.0)); ra.append(np.where(on[l], rs, 0.0))
        e = np.exp(s - s.max(1, keepdims=True))
        p = e / e.sum(1, keepdims=True)
        d = (p - np.eye(dims[-1])[y]) / n
        rd = p * (rs - (p * rs).sum(1, keepdims=True)) / n
        for l in range(L - 1, -1, -1):
            w, b = offs[l]
            g[w:b] = (d.T @ a[l]).reshape(-1)
            hz[w:b] = (rd.T @ a[l] + (d.T @ ra[l] if l else 0.0)).reshape(-1)
            g[b:b + dims[l + 1]], hz[b:b + dims[l + 1]] = d.sum(0), rd.sum(0)
            if l:
                (Wl, Vl) = Ws[l]
                d, rd = np.where(on[l - 1], d @ Wl, 0.0), np.where(on[l - 1], rd @ Wl + d @ Vl, 0.0)
    return g, hz


def _compare(h, theta0, x, y, dims, batch, k, what):
    P = len(theta0)
    for i in range(k):
        on = [h.get_state(B.DW_S_ACT + l, i).reshape(batch, -1) > 0 for l in range(1, len(dims) - 1)]
        bits = h.get_state(B.DW_S_ZBITS, i)
        z = np.where((bits[np.arange(P) >> 5] >> (np.arange(P) & 31)) & 1, 1.0, -1.0)
        g, hz = _dual_network(theta0, z, x[i], y[i], dims, on)
        for name, got, ref, rtol in (("g", h.get_state(B.DW_S_G, i), g, RTOL_GRAD), ("hz", h.get_state(B.DW_S_HZ, i), hz, RTOL_HV)):
            np.testing.assert_array_equal(np.isnan(got), np.isnan(ref), err_msg="%s %s[%d]" % (what, name, i))
            ok = np.isfinite(ref)
            for layer, sl in per_layer(dims):
                close(got[sl][ok[sl]], ref[sl][ok[sl]], rtol, "%s %s[%d]/%s" % (what, name, i, layer))


@pytest.mark.parametrize("probes", [1, 2])
@pytest.mark.parametrize("dims,batch,k", [TILES, SLICES])
def test_infinite_and_huge_inputs_reach_what_fp32_sums_give(dims, batch, k, probes):
    """Samples of the second worker with an inf, a -inf, a NaN and an entry of 2^100.  The forward tiles that hold them are
    computed again; the units of an inf sample are inf or 0, the layer above has inf - inf and is off, so nothing comes back
    but 0 x inf: NaN in those columns of the weight gradients, everything else as without them.  The other workers share no
    tile with it."""
    print("redo inputs", dims, batch, k, probes, flush=True)
    w, theta0, x, y = _inputs(dims, batch, k, 86)
    x[1, 5, 17] = np.inf; x[1, 64, 3] = -np.inf; x[1, 20, 9] = np.nan; x[1, 33, 30] = 2.0 ** 100
    h = B.Handle(B.config_from_workload(w, n_samples=probes), theta0)
    h.worker_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
    _compare(h, theta0, x, y, dims, batch, k, "redo inputs")


@pytest.mark.parametrize("dims,batch,k", [TILES, SLICES])
def test_huge_gradients_follow_the_64_bit_network(dims, batch, k):
    """Output weights times 2^95: the softmax is one-hot, the gradients below are of 2^85, more than the pieces' range holds, and
    every data and weight gradient under the output layer is computed again."""
    print("redo gradients", dims, batch, k, flush=True)
    w, theta0, x, y = _inputs(dims, batch, k, 87)
    offs, _ = O.layer_offsets(dims)
    theta0[offs[-1][0]:offs[-1][1]] *= np.float32(2.0 ** 95)
    h = B.Handle(B.config_from_workload(w), theta0)
    h.worker_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
    _compare(h, theta0, x, y, dims, batch, k, "redo gradients")


def test_a_fused_weight_gradient_with_an_infinity_updates_as_the_unfused_one():
    """The first moment after one step is (1 - beta1) g: the fused tiles and the tiles that store g agree on where it is
    NaN and elsewhere to rounding.  The tiles differ in size, so an entry may be in pieces on one side and on the fp32
    instruction on the other: each is within 64 * 2^-24 of the sum of its 64 products' sizes, which is about five times
    the layer's rms (64 against sqrt(64), and 0.64 for the mean size of a product of normal numbers): 2 * 64 * 2^-24 * 5."""
    dims, batch, k = (1024, 1024, 1024, 10), 64, 8
    w, theta0, x, y = _inputs(dims, batch, k, 88)
    x[2, 11, 700] = np.inf; x[5, 63, 1023] = np.nan
    m = {}
    for fuse in (0, 1):
        h = B.Handle(B.config_from_workload(w, fuse_update=fuse), theta0)
        h.worker_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
        m[fuse] = [h.get_state(B.DW_S_M, i) for i in range(k)]
    offs, _ = O.layer_offsets(dims)
    for i in range(k):
        nan = np.isnan(m[0][i])
        assert nan.any() == (i in (2, 5))
        np.testing.assert_array_equal(np.isnan(m[1][i]), nan)
        if i == 2:                                                    # the first layer: that input's column and no other
            np.testing.assert_array_equal(nan[:offs[0][1]].reshape(1024, 1024).nonzero()[1], 700)
        for w0, b0 in offs:
            a, b, ok = m[1][i][w0:b0], m[0][i][w0:b0], ~nan[w0:b0]
            close(a[ok], b[ok], 2 * 64 * 2.0 ** -24 * 5, "redo fused m[%d]/W" % i)


def _smooth_cnn(spec, batch, k, seed):
    """Parameters and inputs far from every ReLU kink (closest pooling choice 2.7e-6): non-negative inputs, kernels of one
    sign per output channel."""
    offs, P = spec.offsets()
    rng = W.rng_for(seed, 3)
    theta = np.zeros(P)
    for n, (w, b, shape) in enumerate(offs):
        fan = int(np.prod(shape[1:]))
        u = rng.uniform(-1, 1, size=b - w) / np.sqrt(fan)
        if n < 2:
            u = np.abs(u)
        if n == 1:
            u = u.reshape(shape[0], -1); u[::3] *= -1; u = u.reshape(-1)
        theta[w:b] = u
        theta[b:b + shape[0]] = np.abs(rng.uniform(-1, 1, size=shape[0])) / np.sqrt(fan) * (1 if n != 1 else 0.1)
    theta = theta.astype(np.float32).astype(np.float64)
    x = rng.uniform(0, 1, size=(k, batch) + spec.img).astype(np.float32)
    return theta, x, rng.integers(0, spec.fc[-1], size=(k, batch)).astype(np.int32)


# The second convolution's forward product and data gradient on slabs of the map, its weight gradient in tiles
CNNS = {
    "paper_shape": (OC.CnnSpec(img=(28, 28, 1), conv=(32, 64), fc=(128, 10)), 16, 2),
    "many_rows": (OC.CnnSpec(img=(14, 12, 1), conv=(36, 36), fc=(24, 7)), 128, 7),
}
# maps too wide for slabs: all products in tiles on views of the map, 128 x 32, 64 x 64 and (from 512 blocks of rows on) 128 x 64
VIEWS = {
    "few_channels": (OC.CnnSpec(img=(30, 30, 1), conv=(8, 8), fc=(12, 5)), 3, 2),
    "wide": (OC.CnnSpec(img=(8, 78, 1), conv=(36, 36), fc=(16, 7)), 5, 2),
    "wide_many_rows": (OC.CnnSpec(img=(8, 78, 1), conv=(36, 36), fc=(16, 7)), 40, 6),
}


@pytest.mark.parametrize("name,where", [(n, w) for n in CNNS for w in ("forward", "backward")] +
                         [(n, w) for n in VIEWS for w in ("in range", "forward", "backward")])
def test_convolutions_beyond_the_pieces_range(name, where):
    """The second convolution's forward product (first kernels and biases times 2^84, the first linear layer's weights 2^-84) and
    its data and weight gradients (output weights times 2^95) are computed again; against the 64-bit oracle.  On maps too wide for
    slabs also with operands that need no second pass."""
    spec, batch, k = {**CNNS, **VIEWS}[name]
    print("redo cnn", name, where, flush=True)
    assert second_convolution_on_slabs(spec, batch, k) == (name in CNNS)
    theta0, x, y = cnn_inputs(spec, batch, k, 100) if name == "paper_shape" else _smooth_cnn(spec, batch, k, 100)
    theta0 = theta0.copy()
    offs, _ = spec.offsets()
    if where == "forward":
        for (w, b, shape), s in zip(offs, (2.0 ** 84, 1.0, 2.0 ** -84)):
            theta0[w:b] *= s
        for (_, b, shape) in offs[:2]:
            theta0[b:b + shape[0]] *= 2.0 ** 84
    elif where == "backward":
        w, b, _ = offs[-1]
        theta0[w:b] *= 2.0 ** 95
    idx, P_lib = B.conv_param_index(spec.img, spec.conv, spec.fc)
    cfg = B.make_config(dims=(spec.flat,) + spec.fc, k=k, batch=batch, img=spec.img, conv=spec.conv, seed=77, lr=0.01,
                        optimizer=B.DW_OPT_SGD)
    th_lib = np.zeros(P_lib, dtype=np.float32); th_lib[idx] = theta0
    h = B.Handle(cfg, th_lib)
    h.worker_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
    for i in (0, k - 1):
        with np.errstate(divide="ignore"):                           # (the loss of a one-hot softmax)
            g = OC.grad_and_hvp(theta0, x[i], y[i], spec)[1]
        got = h.get_state(B.DW_S_G, i)[idx].astype(np.float64)
        for n, (w, b, shape) in enumerate(offs):
            for part, sl in (("W", slice(w, b)), ("b", slice(b, b + shape[0]))):
                up = 2.0 ** -np.round(np.log2(np.abs(g[sl]).max()))     # (the comparison has a floor of 1e-30)
                close(got[sl] * up, g[sl] * up, RTOL_GRAD, "redo cnn g[%d]/%s%d" % (i, part, n))
