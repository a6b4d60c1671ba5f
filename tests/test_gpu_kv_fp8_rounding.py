"""fp8 rounding of the cache writes' vector path, which converts with the
hardware instruction: every bf16 value, and in fp32 every tie between neighbouring
e4m3fn codes with the floats on either side of it, at scales that divide exactly
and that do not.  The element path (rows off a 4-element boundary) rounds with
integer arithmetic: both must store the same bytes, and the ties equal the CPU
oracle.  Ring slots near the largest positions check the 32-bit slot arithmetic."""
import numpy as np
import pytest
import torch

from oracle import kv_update as KU
from paper_2504_06419_amd import spire
from tests.gpu_helpers import banner
from tests.test_gpu_kv_update import _on_device

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _stored(x, scale, offset):
    """x [B, 1, 1, 128] appended at position 0; the stored K bytes [B, 128]."""
    B = x.shape[0]
    k = torch.zeros((B, 1, 4, 128), dtype=torch.uint8, device=DEV).view(torch.float8_e4m3fn)
    v = torch.zeros((B, 1, 4, 128), dtype=torch.uint8, device=DEV).view(torch.float8_e4m3fn)
    s = torch.tensor([scale], dtype=torch.float32, device=DEV)
    n = _on_device(x, offset)
    pos = torch.zeros((B,), dtype=torch.int32, device=DEV)
    spire.kv_append(spire.kv_view(k, v, k_scale=s, v_scale=s), n, n, pos)
    torch.cuda.synchronize()
    assert torch.equal(k.view(torch.uint8), v.view(torch.uint8))
    return k.view(torch.uint8)[:, 0, 0].cpu().numpy()


def _ties():
    codes = np.array([KU.e4m3fn_value(c) for c in range(0x7F)], dtype=np.float32)
    mid = ((codes[1:].astype(np.float64) + codes[:-1]) / 2).astype(np.float32)
    x = np.concatenate([codes, mid, np.float32([464.0, 479.9, 480.0, 1e38, np.inf, 2.0 ** -149, 2.0 ** -127, np.nan])])
    x = np.concatenate([x, np.nextafter(x, np.float32(0)), np.nextafter(x, np.float32(np.inf))])
    x = np.concatenate([x, -x])
    return torch.from_numpy(np.resize(x, ((len(x) + 127) // 128) * 128)).view(-1, 1, 1, 128)


@pytest.mark.parametrize("scale", [1.0, 0.0078125, 0.37, 3.0e-3, 1.7e38, 1.0e-38])
def test_vector_path_rounds_as_the_element_path(scale):
    banner(f"fp8 rounding, scale {scale}")
    every = torch.arange(65536, dtype=torch.int32).to(torch.int16).view(torch.bfloat16).view(-1, 1, 1, 128)
    ties = _ties()
    for x in (every, ties, (ties.double() * scale).float()):
        assert np.array_equal(_stored(x, scale, 0), _stored(x, scale, 1))
    if scale == 1.0:
        got = _stored(ties, scale, 0).reshape(-1)
        assert np.array_equal(got, KU.to_storage(ties.numpy().reshape(-1), "fp8", scale).reshape(-1))


@pytest.mark.parametrize("S,Wn", [(4, 37), (0, 1), (3, 4096)])
def test_slots_of_large_positions(S, Wn):
    """Positions up to 2^31 - 2 with offsets at both ends of int32."""
    banner(f"ring slots of large positions S={S} W={Wn}")
    lens = [1, S + 1, S + Wn + 1, 2 ** 31 - 1, 2 ** 31 - 2, 10 ** 9 + 7]
    offs = [0, -1, 2 ** 31 - 1, -(2 ** 31), 5, -123456789]
    B, D = len(lens), 128
    bufs = [torch.zeros((B, 1, max(n, 1), D), dtype=torch.bfloat16, device=DEV) for n in (S, S, Wn, Wn)]
    sink, ring = spire.kv_view(bufs[0], bufs[1], capacity=S), spire.kv_view(bufs[2], bufs[3], capacity=Wn)
    new = (1 + torch.arange(B, device=DEV, dtype=torch.float32)).view(B, 1, 1).expand(B, 1, D).contiguous()
    spill = [torch.zeros((1, B, 1, D), dtype=torch.bfloat16, device=DEV) for _ in range(2)]
    m = torch.tensor(lens, dtype=torch.int32, device=DEV)
    o = torch.tensor(offs, dtype=torch.int32, device=DEV)
    spire.draft_append(sink, ring, new, new, m, o, S, Wn, spill[0][0], spill[1][0])
    torch.cuda.synchronize()
    for b in range(B):
        where, slot = KU.draft_slot(lens[b] - 1, S, Wn, offs[b])
        for i, view in enumerate((bufs[0], bufs[2])):
            want = torch.zeros_like(view[b, 0])
            if (where == "sink") == (i == 0):
                want[slot] = b + 1
            assert torch.equal(view[b, 0], want)
    n = torch.full((B,), -1, dtype=torch.int32, device=DEV)   # nothing accepted: the write is undone
    spire.draft_rollback(sink, ring, spill[0], spill[1], m - 1, n, o, S, Wn)
    torch.cuda.synchronize()
    assert all(float(t.abs().max()) == 0 for t in bufs)
