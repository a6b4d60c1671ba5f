"""GPU parity of draft steps with short segments: one workgroup per segment for
few segments (every wave merges), two waves or one wave per segment beyond one
segment per CU, one wave in several rounds beyond one per wave.  Compared with
the CPU oracle and with the stream-K path (kernel choice 2), at the edges of the
tile split: fewer tiles than waves, ragged tails, rings that wrap, empty and
negative lengths, non-finite keys and values, and segment counts that leave the
last workgroup partly idle."""
import pytest
import torch

from paper_2504_06419_amd import spire
from paper_2504_06419_amd import workloads as W
from tests.gpu_helpers import banner
from tests.test_gpu_draft_coop import _check, _run

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _cus() -> int:
    return torch.cuda.get_device_properties(0).multi_processor_count


def _inputs(B, Hkv, kv_dtype, g, S, Wn, lo, hi, seed, D=128):
    spec = W.DraftSpec(B=B, Hq=g * Hkv, Hkv=Hkv, D=D, S=S, W=Wn, steps=1, ctx_lo=lo, ctx_hi=hi, kv_dtype=kv_dtype,
                       q_dtype="f32" if kv_dtype == "f32" else "bf16")
    inp = W.make_draft_inputs(spec, seed, device=DEV)
    W.write_step_token(inp, 0)
    return inp


def _tol(inp):
    """Each probability rounds to bf16 (relative 2^-9; fp16, 2^-11, with fp8 K/V)
    before the product with the values, while their sum is fp32: an output is off
    by at most 2^-9 sum p |v| / sum p <= 2^-9 max |v|, and fp32 rounding."""
    def top(t, scale):
        x = torch.nan_to_num(t.float(), 0.0, 0.0, 0.0).abs()
        return float((x if scale is None else x * scale.view(1, -1, 1, 1)).max()) if x.numel() else 0.0
    v = max(top(inp.sink_v, inp.v_scale), top(inp.ring_v, inp.v_scale))
    return (2.0 ** -9 if inp.v_scale is None else 2.0 ** -11) * v + 1e-5


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("g", [1, 4, 16, 17, 32])
@pytest.mark.parametrize("B,Hkv,S,Wn,lo,hi", [(1, 1, 4, 476, 2000, 2000), (13, 8, 4, 37, 1, 90),
                                              (7, 2, 0, 33, 1, 60), (5, 3, 8, 0, 1, 12), (3, 8, 4, 252, 100, 900)])
def test_few_segments(kv_dtype, g, B, Hkv, S, Wn, lo, hi):
    banner(f"few short segments {kv_dtype} g={g} B={B} Hkv={Hkv} S={S} W={Wn} ctx=[{lo},{hi}]")
    inp = _inputs(B, Hkv, kv_dtype, g, S, Wn, lo, hi, 5100 + g + B + S + Wn)
    _check(inp, inp.seq_lens(0), _tol(inp))


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("g", [4, 24])
@pytest.mark.parametrize("extra", [1, 257, 513, 771, 1027])
def test_more_segments_than_cus(kv_dtype, g, extra):
    """cus + extra segments: two waves each, one wave each, and several rounds."""
    B = _cus() + extra
    banner(f"short segments, more than CUs: {B} x 1, {kv_dtype} g={g}")
    inp = _inputs(B, 1, kv_dtype, g, 4, 60, 1, 300, 5200 + extra + g)
    _check(inp, inp.seq_lens(0), _tol(inp))


@pytest.mark.parametrize("B", [9, 600])
def test_degenerate_lengths_and_nonfinite(B):
    banner(f"short segments B={B}: degenerate lengths, NaN / inf keys and values")
    inp = _inputs(B, 2, "bf16", 4, 4, 96, 200, 400, 5300 + B)
    lens = inp.seq_lens(0).clone()
    lens[3], lens[4], lens[5], lens[6], lens[7] = 4, 0, -7, 5, 10 ** 6
    inp.ring_v[0, 0, 5] = float("nan")
    inp.ring_k[1, 1, 90] = float("nan")
    inp.sink_v[2, 1, 0] = float("inf")
    inp.q[0][3, :4] = -1.0                       # KV head 0 of sequence 3: every score -inf
    inp.sink_k[3, 0] = float("inf")
    out, lse = _check(inp, lens, _tol(inp))
    assert torch.isnan(out[0, :4]).all() and torch.isnan(out[1, 4:]).all()
    assert (out[3, :4] == 0).all() and torch.isneginf(lse[3, :4]).all()
    assert (out[4:6] == 0).all() and torch.isneginf(lse[4:6]).all()


@pytest.mark.parametrize("B,Hkv,Wn,whole", [(8, 1, 480, True), (8, 1, 512, False), (320, 1, 376, True),
                                            (320, 1, 400, False), (600, 1, 248, True), (600, 1, 260, False),
                                            (1100, 1, 124, True), (1100, 1, 132, False)])
def test_rule_edges(B, Hkv, Wn, whole):
    """Both sides of the size limits: whole segments take one launch, the
    partition two."""
    if _cus() != 256:
        pytest.skip("the limits are per CU of a 256-CU device")
    banner(f"short segments: rule edge {B} segments, W={Wn}")
    inp = _inputs(B, Hkv, "bf16", 4, 4, Wn, 10, 2000, 5400 + B + Wn)
    sink = spire.kv_view(inp.sink_k, inp.sink_v)
    ring = spire.kv_view(inp.ring_k, inp.ring_v)
    rec = spire.LaunchRecorder(4)
    s = inp.spec
    out, _ = spire.draft_sparse_attn(inp.q[0].contiguous(), sink, ring, inp.seq_lens(0), inp.ring_offset, s.S, s.W,
                                     inp.sm_scale, s.Hkv, opts=rec.opts(0))
    assert [nm for nm, _ in rec.collect()] == (["draft_partial"] if whole else ["draft_partial", "combine"])
    ref, _ = spire.draft_sparse_attn(inp.q[0].contiguous(), sink, ring, inp.seq_lens(0), inp.ring_offset, s.S, s.W,
                                     inp.sm_scale, s.Hkv, kernel=2)
    assert float((out - ref).abs().max()) <= 2 * _tol(inp)


F32 = [("f32", 64), ("f32", 128), ("bf16", 64), ("fp8", 64)]
TOL32 = 1e-5   # fp32 throughout: as the fp32 path's other tests


@pytest.mark.parametrize("kv_dtype,D", F32)
@pytest.mark.parametrize("g", [1, 4, 16])
@pytest.mark.parametrize("B,Hkv,S,Wn,lo,hi", [(1, 1, 4, 100, 2000, 2000), (13, 8, 4, 37, 1, 90), (7, 2, 0, 33, 1, 60),
                                              (5, 3, 8, 0, 1, 12), (300, 1, 4, 60, 1, 300), (777, 1, 4, 28, 1, 90),
                                              (1283, 1, 4, 12, 1, 40)])
def test_fp32_path(kv_dtype, D, g, B, Hkv, S, Wn, lo, hi):
    banner(f"short segments, fp32 path {kv_dtype} D={D} g={g} B={B} Hkv={Hkv} S={S} W={Wn} ctx=[{lo},{hi}]")
    inp = _inputs(B, Hkv, kv_dtype, g, S, Wn, lo, hi, 5500 + g + B + S + Wn, D=D)
    _check(inp, inp.seq_lens(0), TOL32)


@pytest.mark.parametrize("kv_dtype,D", [("f32", 128), ("bf16", 64)])
@pytest.mark.parametrize("B", [9, 280, 600])
def test_fp32_path_degenerate_lengths_and_nonfinite(kv_dtype, D, B):
    """As above on the fp32 path: one, two and four waves per segment; an
    infinite value is visible to every row, which it makes infinite or NaN."""
    banner(f"short segments, fp32 path {kv_dtype} D={D} B={B}: degenerate lengths, NaN / inf keys and values")
    inp = _inputs(B, 1, kv_dtype, 4, 4, 52, 200, 400, 5600 + B, D=D)
    lens = inp.seq_lens(0).clone()
    lens[3], lens[4], lens[5], lens[6], lens[7] = 4, 0, -7, 5, 10 ** 6
    inp.ring_v[0, 0, 5] = float("nan")
    inp.ring_k[1, 0, 50] = float("nan")
    inp.sink_v[2, 0, 0] = float("inf")
    inp.q[0][3, :4] = -1.0                       # sequence 3: every score -inf
    inp.sink_k[3, 0] = float("inf")
    out, lse = _check(inp, lens, TOL32)
    assert torch.isnan(out[0]).all() and torch.isnan(out[1]).all()
    assert torch.isinf(out[2]).all()
    assert (out[3:6] == 0).all() and torch.isneginf(lse[3:6]).all()


# one workgroup a segment (one and two row blocks), two waves a segment
@pytest.mark.parametrize("B,g", [(9, 4), (9, 24), (280, 4)])
def test_merge_does_not_overflow(B, g):
    """128 equal weights on values of 2^121: the values of one wave sum to at most
    2^127, those of the segment to 2^128.  The partition's partials are means."""
    banner(f"short segments: merge of large values B={B} g={g}")
    inp = _inputs(B, 1, "bf16", g, 4, 124, 500, 500, 5700 + B)
    inp.q[0].zero_()
    inp.ring_v.fill_(2.0 ** 121)
    inp.sink_v.fill_(2.0 ** 121)
    rec = spire.LaunchRecorder(4)
    for kernel, names in ((0, ["draft_partial"]), (2, ["draft_partial", "combine"])):
        out, _ = _run(inp, inp.seq_lens(0), kernel, rec)
        assert [nm for nm, _ in rec.collect()] == names
        print(f"  kernel {kernel}: least {float(out.min()):.6e} largest {float(out.max()):.6e}", flush=True)
        assert float((out / 2.0 ** 121 - 1).abs().max()) <= TOL32
