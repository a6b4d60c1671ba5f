"""GPU parity of the fp32 matrix path (head_dim 64, and fp32 K/V at 64 and 128)
at the edges of its tiles and units: row counts around 16-row blocks and units
of two or three blocks, keys around 16/32-key tiles, ragged contiguous
capacities, paged caches, filling and wrapped rings, short and empty sequences,
workers covering many segments and segments covering many workers, and
non-finite values under the causal mask.  Compared with the fp64 oracle at the
fp32 tolerance for every cache dtype: probabilities stay fp32 here (products
with the exactly converted values, sums of at most a few thousand fp32 terms of
magnitude <= max|v|: below 1e-5 in absolute terms for N(0, 1) data)."""
import numpy as np
import pytest
import torch

from paper_2504_06419_amd import spire
from paper_2504_06419_amd import workloads as W
from tests.gpu_helpers import banner, draft_views, lse_err, max_err, oracle_draft, oracle_verify, run_draft, run_verify

pytestmark = pytest.mark.gpu
DEV = "cuda"
TOL32 = 1e-5


def _spec(kv, D, k, g, **kw):
    return W.VerifySpec(Hq=2 * g, Hkv=2, D=D, k=k, kv_dtype=kv, q_dtype="f32" if kv == "f32" else "bf16", **kw)


def _check(out, lse, ref):
    eo, el = max_err(out, ref[0]), lse_err(lse, ref[1])
    print(f"  max|out-oracle|={eo:.3e} max|lse-oracle|={el:.3e}", flush=True)
    assert eo <= TOL32 and el <= TOL32


# rows per KV head: 1, 16, 17, 20, 33, 48, 49, 72, 128
@pytest.mark.parametrize("kv,D", [("f32", 64), ("f32", 128), ("bf16", 64), ("fp8", 64)])
@pytest.mark.parametrize("k,g", [(0, 1), (1, 8), (0, 17), (4, 4), (2, 11), (5, 8), (6, 7), (8, 8), (15, 8)])
@pytest.mark.parametrize("ps", [0, 48])
def test_verify_rows_and_units(kv, D, k, g, ps):
    banner(f"fp32 path verify {kv} D={D} k={k} g={g} ps={ps}")
    spec = _spec(kv, D, k, g, B=5, ctx_lo=1, ctx_hi=300, page_size=ps, spare_pages=2 if ps else 0)
    inp = W.make_verify_inputs(spec, 600 + 13 * k + g + ps, device=DEV)
    _check(*run_verify(inp), oracle_verify(inp))


@pytest.mark.parametrize("kv,D", [("f32", 64), ("f32", 128), ("bf16", 64), ("fp8", 64)])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 32, 33, 49, 1000])
def test_verify_tile_edges(kv, D, n):
    """Every sequence holds n keys (fewer than k + 1 for n < 4: rows without
    visible keys), capacity exactly n; plus one empty sequence."""
    banner(f"fp32 path tile edges {kv} D={D} n={n}")
    inp = W.make_verify_inputs(_spec(kv, D, 3, 4, B=3, ctx_lo=max(n - 4, 0), ctx_hi=max(n - 4, 0)), 700 + n, device=DEV)
    inp.kv_lens = torch.tensor([min(n, inp.capacity), 0, min(n, inp.capacity)], dtype=torch.int32, device=DEV)
    _check(*run_verify(inp), oracle_verify(inp))


@pytest.mark.parametrize("kv,D", [("f32", 128), ("bf16", 64), ("fp8", 64)])
@pytest.mark.parametrize("B,lo,hi", [(1, 9000, 9000), (300, 1, 60)])
def test_verify_split_and_many_segments(kv, D, B, lo, hi):
    """One long segment over many workers; more segments than workers."""
    banner(f"fp32 path {kv} D={D} B={B} ctx=[{lo},{hi}]")
    spec = W.VerifySpec(B=B, Hq=32, Hkv=8, D=D, k=4, ctx_lo=lo, ctx_hi=hi, kv_dtype=kv,
                        q_dtype="f32" if kv == "f32" else "bf16", page_size=16)
    inp = W.make_verify_inputs(spec, 800 + B, device=DEV)
    out, lse = run_verify(inp)
    ids = list(range(B)) if B < 10 else [0, 1, 7, 150, 298, 299]
    _check(out[ids], lse[ids], oracle_verify(inp, ids))
    again, lse2 = run_verify(inp)
    assert torch.equal(out, again) and torch.equal(lse, lse2)


@pytest.mark.parametrize("kv,D", [("f32", 64), ("f32", 128), ("bf16", 64), ("fp8", 64)])
@pytest.mark.parametrize("S,Wn,lo,hi,g", [(4, 64, 1, 200, 4), (0, 40, 1, 100, 1), (4, 0, 1, 10, 8), (8, 500, 300, 900, 24)])
def test_draft(kv, D, S, Wn, lo, hi, g):
    banner(f"fp32 path draft {kv} D={D} S={S} W={Wn} g={g}")
    spec = W.DraftSpec(B=7, Hq=2 * g, Hkv=2, D=D, S=S, W=Wn, steps=2, ctx_lo=lo, ctx_hi=hi, kv_dtype=kv,
                       q_dtype="f32" if kv == "f32" else "bf16")
    inp = W.make_draft_inputs(spec, 900 + S + Wn, device=DEV)
    for step in range(spec.steps):
        W.write_step_token(inp, step)
        _check(*run_draft(inp, step), oracle_draft(inp, step))


def test_bf16_queries_on_f32_cache():
    banner("fp32 path: bf16 queries, fp32 K/V")
    spec = W.VerifySpec(B=4, Hq=8, Hkv=2, D=128, k=4, ctx_lo=10, ctx_hi=500, kv_dtype="f32", q_dtype="bf16")
    inp = W.make_verify_inputs(spec, 31, device=DEV)
    _check(*run_verify(inp), oracle_verify(inp))


@pytest.mark.parametrize("kv,D", [("f32", 128), ("bf16", 64), ("fp8", 64)])
@pytest.mark.parametrize("lo,hi", [(200, 700), (9000, 9000)])
def test_nonfinite_values_under_the_mask(kv, D, lo, hi):
    """Values of keys only later rows see: NaN (and inf) reach exactly the rows
    that see them, in segments of one worker and of many (whose merge is left
    to the recomputation); the other segments keep their bits."""
    banner(f"fp32 path: non-finite values at keys n-1, n-2: {kv} D={D} ctx=[{lo},{hi}]")
    k = 3
    spec = W.VerifySpec(B=3, Hq=8, Hkv=2, D=D, k=k, ctx_lo=lo, ctx_hi=hi, kv_dtype=kv,
                        q_dtype="f32" if kv == "f32" else "bf16")
    inp = W.make_verify_inputs(spec, 41, device=DEV)
    clean, _ = run_verify(inp)
    n = inp.kv_lens.tolist()
    v = inp.v_cache.view(torch.uint8) if kv == "fp8" else inp.v_cache
    nan = 0x7F if kv == "fp8" else float("nan")
    v[0, 1, n[0] - 1, 5] = nan
    v[2, 0, n[2] - 2, 7] = nan
    if kv != "fp8":
        v[2, 0, n[2] - 1, 60] = float("inf")
        v[2, 1, 10, 3] = -float("inf")                # every row sees it
    out, lse = run_verify(inp)
    ref_o, ref_l = oracle_verify(inp)
    g = out.double().cpu().numpy()
    assert np.array_equal(np.isnan(g), np.isnan(ref_o)) and np.array_equal(np.isposinf(g), np.isposinf(ref_o))
    assert np.array_equal(np.isneginf(g), np.isneginf(ref_o))
    fin = np.isfinite(ref_o)
    assert np.isfinite(g[:2, :k - 1]).all() and np.isfinite(g[2, :k - 1, :4]).all() and not fin.all()
    assert np.max(np.abs(g[fin] - ref_o[fin])) <= TOL32
    assert lse_err(lse, ref_l) <= TOL32
    assert torch.equal(out[1], clean[1]) and torch.equal(out[0, :, :4], clean[0, :, :4])


def test_nonfinite_keys_and_draft_values():
    banner("fp32 path: NaN key, -inf scores, NaN ring value")
    inp = W.make_verify_inputs(_spec("bf16", 64, 2, 4, B=3, ctx_lo=300, ctx_hi=300), 51, device=DEV)
    inp.k_cache[1, 0, 5, 7] = float("nan")
    inp.q[2, ..., 0] = -inp.q[2, ..., 0].abs().clamp(min=0.5)
    inp.k_cache[2, :, :, 0] = float("inf")             # every score of sequence 2 is -inf: empty rows
    out, lse = run_verify(inp)
    ref_o, ref_l = oracle_verify(inp)
    g, gl = out.double().cpu().numpy(), lse.double().cpu().numpy()
    assert np.array_equal(np.isnan(g), np.isnan(ref_o)) and np.array_equal(np.isneginf(gl), np.isneginf(ref_l))
    assert (g[2] == 0).all() and np.isnan(gl[1, :, :4]).all()
    spec = W.DraftSpec(B=3, Hq=8, Hkv=2, D=64, S=4, W=64, steps=1, ctx_lo=100, ctx_hi=100)
    d = W.make_draft_inputs(spec, 52, device=DEV)
    W.write_step_token(d, 0)
    d.ring_v[1, 0, 9, 4] = float("nan")
    sink, ring = draft_views(d)
    out, lse = spire.draft_sparse_attn(d.q[0].contiguous(), sink, ring, d.seq_lens(0), d.ring_offset, 4, 64,
                                       d.sm_scale, 2)
    torch.cuda.synchronize()
    ref_o, ref_l = oracle_draft(d, 0)
    g = out.double().cpu().numpy()
    assert np.array_equal(np.isnan(g), np.isnan(ref_o)) and np.isnan(ref_o).any()


# the merge's forms with the check in the same launch: a workgroup per worker, per
# segment without and with groups of threads; one and two units per KV head
@pytest.mark.parametrize("kv,D,k,g,B,Hkv", [("bf16", 64, 3, 4, 200, 8), ("f32", 64, 3, 4, 200, 8), ("bf16", 64, 4, 4, 64, 8),
                                            ("fp8", 64, 4, 4, 64, 8), ("f32", 64, 8, 8, 3, 2), ("f32", 128, 8, 8, 3, 2),
                                            ("bf16", 64, 15, 8, 3, 2), ("f32", 64, 8, 8, 60, 8), ("f32", 64, 8, 8, 40, 16)])
def test_nonfinite_values_under_the_mask_in_every_merge(kv, D, k, g, B, Hkv):
    """Every third sequence holds a NaN (not fp8: and an infinity) at keys that only
    later rows see; every row against the oracle, and the other sequences' bits as
    without them."""
    banner(f"fp32 path: non-finite tails {kv} D={D} k={k} g={g} B={B} Hkv={Hkv}")
    spec = W.VerifySpec(B=B, Hq=Hkv * g, Hkv=Hkv, D=D, k=k, ctx_lo=40, ctx_hi=6000 if B < 10 else 900, kv_dtype=kv,
                        q_dtype="f32" if kv == "f32" else "bf16")
    inp = W.make_verify_inputs(spec, 61 + B + k, device=DEV)
    clean, _ = run_verify(inp)
    n = inp.kv_lens.tolist()
    v = inp.v_cache.view(torch.uint8) if kv == "fp8" else inp.v_cache
    for b in range(0, B, 3):
        h = (b // 3) % Hkv
        v[b, h, n[b] - 1 - (b // 3) % k, (7 * b) % D] = 0x7F if kv == "fp8" else float("nan")
        if kv != "fp8":
            v[b, (h + 1) % Hkv, n[b] - 1, (5 * b + 1) % D] = float("inf")
    out, lse = run_verify(inp)
    ref_o, ref_l = oracle_verify(inp)
    got = out.double().cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(ref_o)) and np.array_equal(np.isposinf(got), np.isposinf(ref_o))
    fin = np.isfinite(ref_o)
    assert np.array_equal(np.isfinite(got), fin) and not fin.all() and np.isnan(ref_o).any()
    eo = float(np.max(np.abs(got[fin] - ref_o[fin])))
    print(f"  {B * Hkv} segments, {int((~fin).sum())} non-finite outputs, max|out-oracle|={eo:.3e}", flush=True)
    assert eo <= TOL32 and lse_err(lse, ref_l) <= TOL32
    rest = [b for b in range(B) if b % 3]
    assert torch.equal(out[rest], clean[rest])


@pytest.mark.parametrize("kv,D", [("f32", 64), ("f32", 128), ("bf16", 64), ("fp8", 64)])
@pytest.mark.parametrize("n,scale", [(60, 2.0 ** 6), (60, 2.0 ** 10), (3000, 2.0 ** 10)])
def test_scores_of_hundreds_and_thousands(kv, D, n, scale):
    """Scores far apart: the reference maximum of every tile has to be that tile's
    own (one that is off by more than the exponent's range empties the row).
    Queries and keys are integers, the keys times a power of two: every score is
    exact, and a log-sum-exp of a few thousand carries at most eight roundings of
    2^-24 each."""
    banner(f"fp32 path: scores of {scale:.0f} x integers, {kv} D={D} n={n}")
    inp = W.make_verify_inputs(_spec(kv, D, 1, 4, B=12, ctx_lo=n, ctx_hi=n), 71 + n, device=DEV, poison=None)
    g = torch.Generator().manual_seed(n)
    ints = lambda t: torch.randint(-4, 5, t.shape, generator=g).to(DEV).float()
    inp.q = ints(inp.q).to(inp.q.dtype)
    inp.k_cache = (ints(inp.k_cache) * (1.0 if kv == "fp8" else scale)).to(inp.k_cache.dtype)
    if kv == "fp8":
        inp.k_scale.fill_(scale)
    out, lse = run_verify(inp)
    ref_o, ref_l = oracle_verify(inp)
    eo, el = max_err(out, ref_o), lse_err(lse, ref_l)
    print(f"  max|out-oracle|={eo:.3e} max|lse-oracle|={el:.3e} max|lse|={np.abs(ref_l).max():.0f}", flush=True)
    assert eo <= TOL32 and el <= TOL32 + np.abs(ref_l).max() * 2.0 ** -21


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,Hkv,g,W_,lo,hi", [(96, 8, 2, 248, 249, 529), (5, 1, 8, 1884, 83, 341), (12, 2, 4, 60, 100, 200)])
def test_no_further_from_64_bits_than_the_vector_kernel(D, B, Hkv, g, W_, lo, hi):
    """fp32 K/V: the matrix kernels' sums round no more than those of the vector
    kernel, in the 2-norm over all outputs of the same inputs."""
    banner(f"fp32 path: error against 64 bits D={D} B={B} W={W_}")
    spec = W.DraftSpec(B=B, Hq=g * Hkv, Hkv=Hkv, D=D, S=4, W=W_, steps=1, ctx_lo=lo, ctx_hi=hi, kv_dtype="f32", q_dtype="f32")
    inp = W.make_draft_inputs(spec, 81 + B, device=DEV)
    W.write_step_token(inp, 0)
    ref = oracle_draft(inp, 0)[0]
    err = [float(np.linalg.norm(run_draft(inp, 0, kernel=kernel)[0].double().cpu().numpy() - ref) / np.linalg.norm(ref))
           for kernel in (0, 1)]
    print(f"  matrix {err[0]:.2e} vector {err[1]:.2e}", flush=True)
    assert err[0] <= err[1]


def _reorder(t, order):
    """The same [blk, head, tok, d] values in another storage order: tokens before
    heads, rows with 16 more elements behind them, or blocks innermost of the three."""
    if order == "tokens":
        return t.transpose(1, 2).contiguous().transpose(1, 2)
    if order == "padded":
        wide = torch.empty(t.shape[:3] + (t.shape[3] + 16,), dtype=t.dtype, device=t.device)
        wide[..., : t.shape[3]].copy_(t)
        return wide[..., : t.shape[3]]
    return t.permute(1, 2, 0, 3).contiguous().permute(2, 0, 1, 3)


@pytest.mark.parametrize("order", ["tokens", "padded", "blocks"])
@pytest.mark.parametrize("kv,D", [("f32", 64), ("f32", 128), ("bf16", 64), ("fp8", 64)])
def test_storage_orders(kv, D, order):
    """Strides other than [blk, head, tok, d]: verify on contiguous and paged caches
    and drafts, whole and on the partition, equal what the usual order gives, bit for
    bit."""
    banner(f"fp32 path: storage order {order} {kv} D={D}")

    def store(t):
        return _reorder(t.view(torch.uint8), order).view(t.dtype) if kv == "fp8" else _reorder(t, order)

    for ps in (0, 16):
        inp = W.make_verify_inputs(_spec(kv, D, 3, 4, B=5, ctx_lo=1, ctx_hi=400, page_size=ps), 91 + ps, device=DEV)
        want = run_verify(inp)
        inp.k_cache, inp.v_cache = store(inp.k_cache), store(inp.v_cache)
        got = run_verify(inp)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    spec = W.DraftSpec(B=7, Hq=8, Hkv=2, D=D, S=4, W=100, steps=1, ctx_lo=1, ctx_hi=300, kv_dtype=kv,
                       q_dtype="f32" if kv == "f32" else "bf16")
    for kernel in (0, 2):
        d = W.make_draft_inputs(spec, 95, device=DEV)
        W.write_step_token(d, 0)
        want = run_draft(d, 0, kernel=kernel)
        d.sink_k, d.sink_v, d.ring_k, d.ring_v = store(d.sink_k), store(d.sink_v), store(d.ring_k), store(d.ring_v)
        got = run_draft(d, 0, kernel=kernel)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
