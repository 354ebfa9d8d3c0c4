"""The mean loss of the output-layer kernels: a sum over the minibatch that adds no more than its own rounding."""
import numpy as np
import pytest
import torch

from paper_2409_09242_amd import binding as B

pytestmark = pytest.mark.gpu


def _loss(dims, batch, bf16):
    cfg = B.make_config(dims=dims, k=2, batch=batch, bf16=bf16)
    h = B.Handle(cfg, np.zeros(B.param_count(cfg), dtype=np.float32))
    loss = torch.zeros(2, device="cuda")
    x = torch.zeros((2, batch, dims[0]), dtype=torch.bfloat16 if bf16 else torch.float32, device="cuda")
    h.worker_step(x, torch.zeros((2, batch), dtype=torch.int32, device="cuda"), loss=loss)
    return loss.cpu().numpy()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("batch", [15, 25, 203, 589])
def test_equal_losses_have_themselves_as_their_mean(batch, bf16):
    """A network of zeros gives every sample the same loss.  Added up in 64 bits, each sixteen rounded once, their mean is off
    by one last bit at most (half for the partial sums' rounding, half for the result's); in fp32 these minibatches of seven
    classes are two to four off."""
    dims = (264, 72, 136, 7)
    print("equal losses", batch, bf16, flush=True)
    one = _loss(dims, 1, bf16)
    many = _loss(dims, batch, bf16)
    assert np.all(one == one[0]) and abs(one[0] - np.log(7.0)) < 1e-6
    assert np.all(np.abs(many - one) <= np.spacing(one)), (many, one)
