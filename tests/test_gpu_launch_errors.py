"""A launch that the device refuses (more threads than a grid holds) is
reported by its own call and not again by the next one."""

import pytest
import torch

import test_gpu_kernels as G
from paper_2509_12207_amd import capi

pytestmark = pytest.mark.gpu


# rows of one float, 16 and 64 threads a row
@pytest.mark.parametrize("op,rows", [("rowsum", 1 << 28), ("softmax", 1 << 27)])
def test_refused_launch_is_reported_once(op, rows):
    x, out = torch.zeros(rows, device=G.DEV), torch.zeros(rows, device=G.DEV)
    with pytest.raises(capi.UgError) as e:
        G.launch({"op": op, "shape": (rows, 1), "in": (0,), "out": (1,)}, [x, out])
    assert e.value.status == capi.EDEVICE
    a, b, y = torch.ones(4, 4, device=G.DEV), torch.ones(4, device=G.DEV), torch.zeros(4, 4, device=G.DEV)
    G.launch({"op": "bias_relu", "shape": (4, 4, 0), "in": (0, 1), "out": (2,)}, [a, b, y])
    assert (y == 2).all()
