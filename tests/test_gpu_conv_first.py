"""The first convolution straight from images of one channel where it can go wrong: channels around a group of 32, columns around a
block, rows cut into strips and not, a single output row, two channels (which go through patches instead) and many blocks to add up."""
import pytest

import test_gpu_cnn as N
from oracle import dw_cnn as OC

pytestmark = pytest.mark.gpu

SPECS = {
    "one pooled entry a channel": (OC.CnnSpec(img=(4, 4, 1), conv=(4,), fc=(4, 3)), 2, 2),
    "a group of channels and four": (OC.CnnSpec(img=(8, 10, 1), conv=(36,), fc=(8, 4)), 3, 2),
    "columns past a block": (OC.CnnSpec(img=(6, 14, 1), conv=(8,), fc=(8, 3)), 3, 1),
    "strips with a remainder": (OC.CnnSpec(img=(24, 6, 1), conv=(32, 8), fc=(8, 4)), 2, 1),
    "whole columns, many blocks": (OC.CnnSpec(img=(4, 6, 1), conv=(4,), fc=(8, 3)), 200, 2),
    "two channels": (OC.CnnSpec(img=(10, 10, 2), conv=(16,), fc=(8, 4)), 4, 2),
}


@pytest.mark.parametrize("name", list(SPECS))
def test_first_convolution_follows_the_oracle(name, monkeypatch):
    monkeypatch.setitem(N.SPECS, name, SPECS[name])
    N.test_cnn_step_matches_the_oracle(name, 0)
