"""Token and block verification on probability rows at every 4-byte offset: the
kernels read 16 bytes at a time from any of them, and a row's last one to three
entries apart.  V takes every remainder, below one group of four, around a piece
of 2048 and across pieces; the bases of p and q are shifted by 0..3 entries.
Results equal the CPU oracles' bit for bit."""
import numpy as np
import pytest
import torch

from oracle import block_verify as BV
from oracle import token_verify as TV
from paper_2504_06419_amd import spire
from paper_2504_06419_amd import workloads as W
from tests.gpu_helpers import banner

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _shifted(t: torch.Tensor, by: int) -> torch.Tensor:
    flat = torch.full((t.numel() + 8,), float("nan"), dtype=t.dtype, device=DEV)
    view = flat[by:by + t.numel()].view(t.shape)
    view.copy_(t)
    return view


@pytest.mark.parametrize("V", [2, 3, 5, 2046, 2047, 2050, 2051, 4099, 131071])
@pytest.mark.parametrize("pby,qby", [(0, 0), (1, 3), (2, 0), (3, 2)])
def test_rows_at_any_offset(V, pby, qby):
    B, k = (24, 4) if V < 100000 else (3, 2)
    banner(f"rows at any offset: B={B} k={k} V={V} p + {pby}, q + {qby}")
    t = W.make_token_inputs(W.TokenSpec(B=B, k=k, V=V, sigma=3.0, eps=0.7), 900 + V + pby, device=DEV)
    p, q = _shifted(t.p, pby), _shifted(t.q, qby)
    assert p.data_ptr() % 16 == 4 * pby and q.data_ptr() % 16 == 4 * qby
    host = [x.cpu().numpy() for x in (t.p, t.q, t.draft, t.u_accept, t.u_sample)]
    for fn, oracle in ((spire.token_verify, TV.verify_tokens), (spire.block_verify, BV.verify_block)):
        n, tok = fn(p, q, t.draft, t.u_accept, t.u_sample)
        torch.cuda.synchronize()
        rn, rtok = oracle(*host)
        assert np.array_equal(n.cpu().numpy(), rn) and np.array_equal(tok.cpu().numpy(), rtok)
