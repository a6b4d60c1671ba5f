"""GPU parity of the merge of split segments where it can go wrong: segments
over hundreds of workers (groups of threads share the partials), row counts off
the row chunks, fewer positions than workers (most have no work), a quarter as
many segments as workers on either side of the line between the grouped and the
ungrouped form, and NaN and empty partials among many."""
import numpy as np
import pytest
import torch

from paper_2504_06419_amd import workloads as W
from tests.gpu_helpers import TOL, banner, lse_err, max_err, oracle_verify, run_verify

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("B,Hkv,k,g,lo,hi", [(1, 1, 4, 4, 20000, 20000), (1, 1, 0, 1, 70000, 70000),
                                            (3, 2, 6, 3, 500, 9000), (2, 1, 15, 8, 3000, 3000),
                                            (1, 3, 2, 5, 1, 40), (32, 8, 4, 4, 100, 900), (33, 8, 4, 4, 100, 900)])
def test_merge_of_many_partials(kv, B, Hkv, k, g, lo, hi):
    banner(f"combine {kv} B={B} Hkv={Hkv} k={k} g={g} ctx=[{lo},{hi}]")
    spec = W.VerifySpec(B=B, Hq=Hkv * g, Hkv=Hkv, D=128, k=k, ctx_lo=lo, ctx_hi=hi, kv_dtype=kv, page_size=16)
    inp = W.make_verify_inputs(spec, 60 + B + k, device=DEV)
    out, lse = run_verify(inp)
    ids = list(range(min(B, 4)))
    ref_o, ref_l = oracle_verify(inp, ids)
    eo, el = max_err(out[ids], ref_o), lse_err(lse[ids], ref_l)
    print(f"  max|out-oracle|={eo:.3e} max|lse-oracle|={el:.3e}", flush=True)
    assert eo <= TOL[kv] and el <= TOL[kv]


def test_nan_and_empty_partials_among_many():
    banner("combine: a NaN key in one of many partials; all but one partial empty")
    spec = W.VerifySpec(B=2, Hq=8, Hkv=2, D=128, k=1, ctx_lo=16000, ctx_hi=16000)
    inp = W.make_verify_inputs(spec, 77, device=DEV)
    inp.q[..., 0] = -inp.q[..., 0].abs().clamp(min=0.5)
    inp.k_cache[0, 0, 9000, 3] = float("nan")
    inp.k_cache[1, :, 40:, 0] = float("inf")          # every later score is -inf
    out, lse = run_verify(inp)
    ref_o, ref_l = oracle_verify(inp)
    g, gl = out.double().cpu().numpy(), lse.double().cpu().numpy()
    assert np.array_equal(np.isnan(g), np.isnan(ref_o)) and np.array_equal(np.isnan(gl), np.isnan(ref_l))
    assert np.isnan(ref_l[0, :, :4]).all() and np.isfinite(ref_l[1]).all()
    fin = np.isfinite(ref_o)
    assert np.max(np.abs(g[fin] - ref_o[fin])) <= TOL["bf16"]
