"""Feedback memory's vector path at the edges of its rules: outputs around the
1 / 2 / 4 / 8 accumulator sets, layers around the four requested ahead, element
counts that are multiples of 4 and of 8, bases 8 and 16 bytes aligned, and calls
of several chunks per thread with a last one that is partly idle.  Same bounds as
the oracle test."""
import pytest
import torch

from tests.gpu_helpers import banner
from tests.test_gpu_feedback_memory import _check

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("xdt,mdt", [(torch.bfloat16, torch.bfloat16), (torch.bfloat16, torch.float32),
                                     (torch.float32, torch.bfloat16), (torch.float32, torch.float32)])
@pytest.mark.parametrize("n_out,layers,B,d,off", [(1, 1, 1, 4, 0), (3, 4, 3, 12, 0), (4, 5, 7, 264, 4), (5, 3, 1, 1028, 0),
                                                  (8, 9, 2, 8, 8), (2, 3, 1, 2100004, 0), (1, 2, 1, 4210696, 0)])
def test_chunks(xdt, mdt, n_out, layers, B, d, off):
    banner(f"feedback memory chunks x={xdt} m={mdt} n_out={n_out} layers={layers} B={B} d={d} off={off}")
    g = torch.Generator(device=DEV).manual_seed(77 + n_out + layers + d)
    buf = (torch.randn(layers * B * d + off, generator=g, device=DEV) * 2).to(xdt)
    w = torch.randn((n_out, layers), generator=g, device=DEV) * 3
    _check(buf[off:].view(layers, B, d), w, mdt)
