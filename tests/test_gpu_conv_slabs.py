"""The convolution kernels on slabs of the map where they can go wrong: channel counts around a k-step and a slab, outputs around a
tile and a group, maps of a few positions and of several blocks, the widest slab of each direction and maps past it (which read patches
as operand views instead), more units than blocks, and an input that leaves the range of the pieces."""
import numpy as np
import pytest
import torch

import test_gpu_cnn as N
from oracle import dw_cnn as OC
from paper_2409_09242_amd import binding as B

pytestmark = pytest.mark.gpu

SPECS = {
    "few channels, few positions": (OC.CnnSpec(img=(8, 10, 1), conv=(4, 4), fc=(8, 3)), 3, 2),
    "a k-step and four channels": (OC.CnnSpec(img=(12, 14, 1), conv=(20, 36), fc=(12, 5)), 2, 2),
    "a slab and four channels, three tiles of outputs": (OC.CnnSpec(img=(10, 10, 2), conv=(36, 68), fc=(8, 4)), 2, 1),
    "narrow and tall": (OC.CnnSpec(img=(40, 6, 1), conv=(8, 16), fc=(8, 4)), 2, 2),
    "two blocks an image forward, three back": (OC.CnnSpec(img=(18, 20, 1), conv=(40, 40), fc=(8, 4)), 1, 2),
    "widest slab forward (384 positions)": (OC.CnnSpec(img=(14, 34, 1), conv=(8, 8), fc=(8, 4)), 1, 1),
    "widest slab back (384 positions)": (OC.CnnSpec(img=(12, 32, 1), conv=(8, 12), fc=(8, 4)), 1, 1),
    "more units than blocks": (OC.CnnSpec(img=(8, 8, 1), conv=(4, 8), fc=(8, 3)), 70, 4),
}
# maps whose slab would be too wide, in one of the directions at least
VIEWS = {
    "390 positions back": (OC.CnnSpec(img=(26, 30, 1), conv=(16, 40), fc=(8, 4)), 2, 1),
    "420 positions back": (OC.CnnSpec(img=(10, 42, 1), conv=(8, 8), fc=(8, 4)), 1, 1),
    "390 positions forward": (OC.CnnSpec(img=(16, 32, 1), conv=(8, 8), fc=(8, 4)), 1, 1),
    "past the widest slab in both directions": (OC.CnnSpec(img=(12, 64, 1), conv=(8, 8), fc=(8, 4)), 1, 1),
}


def second_convolution_on_slabs(spec, batch, k):
    """By the launches: its weights' pieces and the product on slabs are two, the product on a view of the map is one.  (One for the
    first convolution of one-channel images, two with patches; one for the pooling and for every hidden linear layer.)"""
    cfg = B.make_config(dims=(spec.flat,) + spec.fc, k=k, batch=batch, img=spec.img, conv=spec.conv)
    h = B.Handle(cfg, np.zeros(B.param_count(cfg), dtype=np.float32), N.DEV)
    h.profile(True)
    h.worker_step(torch.zeros((k, batch) + spec.img, device=N.DEV), torch.zeros((k, batch), dtype=torch.int32, device=N.DEV))
    others = (1 if spec.img[2] == 1 else 2) + 1 + len(spec.fc) - 1
    n = h.profile_read()["gemm_fwd"][0] - others
    assert n in (1, 2)
    return n == 2


@pytest.mark.parametrize("name", list(SPECS) + list(VIEWS))
def test_convolutions_on_slabs_follow_the_oracle(name, monkeypatch):
    spec = {**SPECS, **VIEWS}[name]
    assert second_convolution_on_slabs(*spec) == (name in SPECS)
    monkeypatch.setitem(N.SPECS, name, spec)
    N.test_cnn_step_matches_the_oracle(name, 0)


def test_a_map_beyond_the_pieces_range():
    """One pixel of worker 1 is 1e30, so that results of the second convolution around it are past 2^80: their tiles are computed again
    from whole floats and the loss is the oracle's; the other worker's step is the same to the bit."""
    spec, batch, k = SPECS["a k-step and four channels"]
    theta0, x, y = N._inputs(spec, batch, k, 100)
    idx, P = B.conv_param_index(spec.img, spec.conv, spec.fc)
    th = np.zeros(P, dtype=np.float32); th[idx] = theta0
    out = []
    for bad in (False, True):
        cfg = B.make_config(dims=(spec.flat,) + spec.fc, k=k, batch=batch, img=spec.img, conv=spec.conv, seed=77, lr=0.01, eps=1e-4)
        h = B.Handle(cfg, th, N.DEV)
        xb = x.copy()
        if bad:
            xb[1, 0, 5, 5, 0] = 1e30
        loss = torch.zeros(k, device=N.DEV)
        h.worker_step(torch.from_numpy(xb).to(N.DEV), torch.from_numpy(y).to(N.DEV), loss=loss)
        out.append((loss.cpu().numpy(), h.get_state(B.DW_S_THETA, 0)))
        ref = OC.grad_and_hvp(theta0, xb[1], y[1], spec)[0]
        assert abs(out[-1][0][1] - ref) <= 1e-5 * abs(ref)
    assert out[1][0][1] != out[0][0][1] and out[1][0][0] == out[0][0][0]
    np.testing.assert_array_equal(out[0][1], out[1][1])
