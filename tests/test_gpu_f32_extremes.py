"""Finite extremes on the calls of the fp32 matrix path (head_dim 64, and fp32
K/V): scores of 1e10, scores on both sides of 2^20 (where the path turns from its
fast to its careful form), values of 1e37, both, and a few such values among
ordinary ones or behind weights that only denormal numbers hold, in segments of one worker and of many, next to ordinary sequences.

Scores: query and key entries are small integers times a power of two, so every
score is exact in fp32 in any order of summation and two different scores differ
by far more than fp32 resolves; the softmax is then flat over the ties of the
maximum, and the outputs are fp32 sums as in the path's other tests.  A log-sum-exp
of 1e10 carries the roundings of the scale, of log2(e) and ln(2) and of three
products and a sum: at most eight of 2^-24 each.
Values: integers times 2^123 (4e37 at most); an output is a convex mix of them, so
the path's absolute tolerance for N(0, 1) values scales by 2^123."""
import numpy as np
import pytest
import torch

from paper_2504_06419_amd import workloads as W
from tests.gpu_helpers import banner, oracle_draft, oracle_verify, run_draft, run_verify

pytestmark = pytest.mark.gpu
DEV = "cuda"
TOL32 = 1e-5
KINDS = [("f32", 64), ("f32", 128), ("bf16", 64), ("fp8", 64)]
BIG_V = 2.0 ** 123


def _cases(scores, values):
    """fp8 values do not exceed 448: scores only."""
    return [(kv, D, what) for kv, D in KINDS for what in scores + (values if kv != "fp8" else [])]


def _grid(t, seed, scale):
    """Integers in [-4, 4] times `scale` in place of the data (NaN storage that no
    sequence exposes stays)."""
    g = torch.Generator().manual_seed(seed)
    x = torch.randint(-4, 5, t.shape, generator=g).to(t.device).float() * scale
    old = t.float()
    return torch.where(old.isnan(), old, x).to(t.dtype)


def _check(out, lse, ref, vscale):
    g, gl = out.double().cpu().numpy(), lse.double().cpu().numpy()
    ro, rl = ref
    assert np.isfinite(ro).all() and np.isfinite(g).all(), f"{(~np.isfinite(g)).sum()} outputs not finite"
    assert np.array_equal(np.isneginf(gl), np.isneginf(rl)) and np.isfinite(rl).any()
    live = np.isfinite(rl)
    eo = float(np.max(np.abs(g - ro))) / vscale
    el = float(np.max(np.abs(gl[live] - rl[live]) / np.maximum(1.0, np.abs(rl[live]) * (2.0 ** -21 / TOL32))))
    print(f"  max|out-oracle|/{vscale:.0e}={eo:.3e} scaled max|lse-oracle|={el:.3e} max|lse|={np.abs(rl[live]).max():.2e}",
          flush=True)
    assert eo <= TOL32 and el <= TOL32


def _extreme_scores(q, k, k_scale, seed, even=2.0 ** 15):
    """Even sequences of `q` [B, ...] score about 1e10, odd ones about 1."""
    kk = _grid(k, seed, 1.0 if k_scale is not None else 2.0 ** 15)
    if k_scale is not None:
        k_scale.fill_(2.0 ** 15)
    qq = _grid(q, seed + 1, 1.0)
    f = torch.full((q.shape[0],) + (1,) * (q.dim() - 1), 2.0 ** -17, device=q.device)
    f[::2] = even
    return (qq.float() * f).to(q.dtype), kk


# one worker a segment, one segment over many workers, several segments a worker
@pytest.mark.parametrize("kv,D,what", _cases(["scores", "edge"], ["values", "both", "few", "faint"]))
@pytest.mark.parametrize("B,Hkv,lo,hi,ps", [(3, 2, 40, 300, 0), (1, 2, 9000, 9000, 16), (300, 8, 1, 60, 16)])
def test_verify(kv, D, B, Hkv, lo, hi, ps, what):
    banner(f"extremes verify {kv} D={D} B={B} ctx=[{lo},{hi}] ps={ps}: {what}")
    spec = W.VerifySpec(B=B, Hq=4 * Hkv, Hkv=Hkv, D=D, k=2, ctx_lo=lo, ctx_hi=hi, kv_dtype=kv,
                        q_dtype="f32" if kv == "f32" else "bf16", page_size=ps)
    inp = W.make_verify_inputs(spec, 4000 + B + D, device=DEV)
    if what in ("scores", "both", "edge"):     # edge: rows' maxima around 2^20 in base 2
        inp.q, inp.k_cache = _extreme_scores(inp.q, inp.k_cache, inp.k_scale, 11 + B,
                                             1.0 if what == "edge" else 2.0 ** 15)
    elif what == "values":
        inp.q[::2] = 0.0                        # every weight equal: the sum of the values overflows
    vscale = 1.0
    if what in ("values", "both"):
        inp.v_cache, vscale = _grid(inp.v_cache, 17 + B, BIG_V), BIG_V
    elif what == "few":
        row = inp.v_cache[int(inp.block_table[0, 0]) if ps else 0]   # the first keys of sequence 0
        row[:, 3:6] = _grid(row[:, 3:6], 19, BIG_V)
        vscale = BIG_V
    elif what == "faint":   # the same values behind weights of e^-90, which make up about 1e-2 / the row sum
        blk = int(inp.block_table[0, 0]) if ps else 0
        inp.q[..., 0] = 64.0
        inp.k_cache[..., 0] = torch.where(inp.k_cache[..., 0].isnan(), inp.k_cache[..., 0], 0.0)
        inp.k_cache[blk, :, 3:6, 0] = -90.0 * D ** 0.5 / 64.0
        inp.v_cache[blk, :, 3:6] = _grid(inp.v_cache[blk, :, 3:6], 19, BIG_V)
    ids = list(range(B)) if B < 10 else [0, 1, 2, 150, 151, 298, 299]
    out, lse = run_verify(inp)
    _check(out[ids], lse[ids], oracle_verify(inp, ids), vscale)


# whole segments with four, two and one wave each; the partition; more than 16 rows
@pytest.mark.parametrize("kv,D,what", _cases(["scores"], ["values", "both"]))
@pytest.mark.parametrize("B,g,kernel", [(9, 4, 0), (280, 4, 0), (600, 4, 0), (9, 4, 2), (9, 24, 0)])
def test_draft(kv, D, B, g, kernel, what):
    banner(f"extremes draft {kv} D={D} B={B} g={g} kernel={kernel}: {what}")
    spec = W.DraftSpec(B=B, Hq=g, Hkv=1, D=D, S=4, W=124 if B < 100 else 52, steps=1, ctx_lo=20, ctx_hi=400,
                       kv_dtype=kv, q_dtype="f32" if kv == "f32" else "bf16")
    inp = W.make_draft_inputs(spec, 4100 + B + D, device=DEV)
    W.write_step_token(inp, 0)
    if what != "values":
        inp.q[0], inp.ring_k = _extreme_scores(inp.q[0], inp.ring_k, inp.k_scale, 23 + B)
        inp.sink_k = _grid(inp.sink_k, 29, 1.0 if kv == "fp8" else 2.0 ** 15)
    else:
        inp.q[0][::2] = 0.0
    vscale = 1.0
    if what != "scores":
        inp.ring_v, vscale = _grid(inp.ring_v, 31, BIG_V), BIG_V
        inp.sink_v = _grid(inp.sink_v, 37, BIG_V)
    _check(*run_draft(inp, 0, kernel=kernel), oracle_draft(inp, 0), vscale)
