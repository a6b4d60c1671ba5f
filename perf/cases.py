"""The work this library is measured on, through its public entry points.

Every case is one call (or one round of calls) that a serving program makes per
speculation round on resident caches: target verification, draft attention,
token and block verification, the cache writes, the feedback memory, and a
whole small round.  listed() names fixed cases, draw() gives others of the same
ranges; prepare() makes the seeded inputs and what such a program keeps
(caches, views, workspace, outputs), run() is one pass.

Ranges: batch 1..512; contexts 64..65536 (log-uniform within a batch); k 0..8;
1..32 KV heads, 1..8 query heads per KV head; head_dim 64 and 128; f32, bf16 and
fp8 caches; contiguous and paged; windows 128..4096; vocabularies 1000..131072.
"""
import math

import torch

from paper_2504_06419_amd import spire
from paper_2504_06419_amd import workloads as W

DEV = "cuda"
ES = {"f32": 4, "bf16": 2, "fp8": 1}
DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def _verify(name, B, Hq, Hkv, D, k, lo, hi, kv, page, out):
    return dict(name=name, kind="verify", B=B, Hq=Hq, Hkv=Hkv, D=D, k=k, lo=lo, hi=hi, kv=kv, page=page, out=out)


def _draft(name, B, Hq, Hkv, D, S, W, lo, hi, kv, out):
    return dict(name=name, kind="draft", B=B, Hq=Hq, Hkv=Hkv, D=D, S=S, W=W, lo=lo, hi=hi, kv=kv, out=out)


def listed():
    return [
        # the target's verify pass of a large mixed batch: the library's headline workload
        _verify("verify_bf16_paged_B256_k4", 256, 32, 8, 128, 4, 512, 65536, "bf16", 16, "f32"),
        # the same pass of a larger model on an fp8 cache with long drafts (72 rows per KV head)
        _verify("verify_fp8_paged_B512_k8", 512, 64, 8, 128, 8, 2048, 65536, "fp8", 16, "f32"),
        # a small model's heads (64 wide) at an ordinary batch
        _verify("verify_bf16_d64_paged_B64_k4", 64, 32, 8, 64, 4, 512, 8192, "bf16", 16, "bf16"),
        # the smallest call: a full-precision check run of a tiny model
        _verify("verify_f32_d64_B4_k4", 4, 8, 2, 64, 4, 512, 512, "f32", 0, "f32"),
        # one draft step of an ordinary batch
        _draft("draft_bf16_B64_W2048", 64, 32, 8, 128, 4, 2048, 32768, 32768, "bf16", "f32"),
        # one draft step of the fp8 round: rings at every stage of filling
        _draft("draft_fp8_B512_W4096", 512, 64, 8, 128, 4, 4096, 2048, 65536, "fp8", "f32"),
        # one draft step of a few requests, ragged, short window
        _draft("draft_bf16_B13_W500", 13, 32, 8, 128, 4, 500, 100, 8000, "bf16", "bf16"),
        # token verification after the target's pass, a large vocabulary
        dict(name="token_verify_B256_k4_V128256", kind="token", B=256, k=4, V=128256),
        # block verification, a vocabulary whose rows are not 16-byte aligned
        dict(name="block_verify_B64_k4_V50257", kind="block", B=64, k=4, V=50257),
        # every cache write of one fp8 round: 8 draft writes, the target append, the rollback
        dict(name="kv_update_fp8_B512_k8", kind="kv", B=512, Hkv=8, D=128, k=8, S=4, W=1024, lo=2048, hi=65536,
             kv="fp8", page=16),
        # the draft's memory vectors of one step
        dict(name="feedback_bf16_B512_d8192", kind="fm", B=512, d=8192, layers=3, n_out=2, x="bf16", m="bf16"),
        # a whole speculation round of a few requests: launches and host work count
        dict(name="round_bf16_B16_k4", kind="round", B=16, Hq=32, Hkv=8, D=128, k=4, S=4, W=512, lo=512, hi=8192,
             kv="bf16", page=16, V=32000),
    ]


# ---- drawing -----------------------------------------------------------------------
def _log(rng, lo, hi):
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _heads(rng):
    """(Hkv, queries per KV head): grouped heads, and as many KV heads as query heads."""
    g = rng.choice([1, 2, 4, 4, 8])
    return rng.choice([1, 2, 4, 8, 8] if g > 1 else [2, 8, 16, 32]), g


def _shape(rng):
    """(cache dtype, head_dim, most cache bytes): 64-wide heads and f32 caches belong to smaller models."""
    kv = rng.choice(["bf16", "bf16", "bf16", "fp8", "fp8", "f32"])
    D = rng.choice([128, 128, 64])
    return kv, D, 2.5e8 if kv == "f32" or D == 64 else 1.2e10


def _draw_verify(rng):
    kv, D, most = _shape(rng)
    Hkv, g = _heads(rng)
    k = rng.choice([0, 1, 2, 3, 4, 4, 5, 7, 8])
    if most < 1e9:
        most /= ((k + 1) * g + 15) // 16
    hi = _log(rng, 64, 65536)
    lo = max(16, _log(rng, max(1, hi // 128), hi))
    per = 2 * Hkv * D * ES[kv] * (_mean(lo, hi) + k + 1)
    B = _log(rng, 1, 512)
    while B > 1 and B * per > most:
        B = (B + 1) // 2
    while per > most and hi > 64:
        lo, hi = max(16, lo // 2), max(64, hi // 2)
        per = 2 * Hkv * D * ES[kv] * (_mean(lo, hi) + k + 1)
    return dict(kind="verify", B=B, Hq=Hkv * g, Hkv=Hkv, D=D, k=k, lo=min(lo, hi), hi=hi, kv=kv,
                page=rng.choice([0, 16, 16, 32, 64, 256]) if B * hi * Hkv * D * ES[kv] < 8e9 else 16,
                out=rng.choice(["f32", "bf16"]))


def _draw_draft(rng):
    kv, D, most = _shape(rng)
    Hkv, g = _heads(rng)
    S, Wn = rng.choice([0, 1, 4, 4, 8]), _log(rng, 128, 4096)
    B = _log(rng, 1, 512)
    while B > 1 and 2 * B * Hkv * (S + Wn) * D * ES[kv] > most:
        B = (B + 1) // 2
    hi = _log(rng, 256, 65536)
    return dict(kind="draft", B=B, Hq=Hkv * g, Hkv=Hkv, D=D, S=S, W=Wn, lo=_log(rng, 64, hi), hi=hi, kv=kv,
                out=rng.choice(["f32", "bf16"]))


def draw(rng):
    kind = rng.choice(["verify"] * 5 + ["draft"] * 4 + ["token", "token", "block", "block", "kv", "kv", "fm", "round"])
    if kind == "verify":
        return _draw_verify(rng)
    if kind == "draft":
        return _draw_draft(rng)
    if kind in ("token", "block"):
        B, k, V = _log(rng, 1, 512), rng.randint(1, 8), _log(rng, 1000, 131072)
        while 4 * B * (2 * k + 1) * V > 3e9:
            B = (B + 1) // 2
        return dict(kind=kind, B=B, k=k, V=V)
    if kind == "kv":
        return dict(kind="kv", B=_log(rng, 1, 512), Hkv=rng.choice([1, 2, 8]), D=rng.choice([64, 128, 128]),
                    k=rng.randint(1, 8), S=4, W=_log(rng, 128, 1024), lo=64, hi=_log(rng, 256, 65536),
                    kv=rng.choice(["bf16", "fp8", "f32"]), page=rng.choice([16, 64]))
    if kind == "fm":
        return dict(kind="fm", B=_log(rng, 1, 512), d=rng.choice([512, 1000, 2048, 4096, 8192]),
                    layers=rng.randint(2, 9), n_out=rng.randint(1, 4), x=rng.choice(["bf16", "f32"]),
                    m=rng.choice(["bf16", "f32"]))
    kv = rng.choice(["bf16", "fp8"])
    return dict(kind="round", B=_log(rng, 1, 64), Hq=32, Hkv=8, D=128, k=rng.randint(2, 6), S=4,
                W=_log(rng, 128, 1024), lo=256, hi=_log(rng, 512, 8192), kv=kv, page=16, V=rng.choice([8000, 32000, 50257]))


# ---- inputs ------------------------------------------------------------------------
def _vspec(c):
    return W.VerifySpec(B=c["B"], Hq=c["Hq"], Hkv=c["Hkv"], D=c["D"], k=c["k"], ctx_lo=c["lo"], ctx_hi=c["hi"],
                        kv_dtype=c["kv"], q_dtype="f32" if c["kv"] == "f32" else "bf16", page_size=c["page"])


def _dspec(c, steps=1):
    return W.DraftSpec(B=c["B"], Hq=c["Hq"], Hkv=c["Hkv"], D=c["D"], S=c["S"], W=c["W"], steps=steps,
                       ctx_lo=c["lo"], ctx_hi=c["hi"], kv_dtype=c["kv"], q_dtype="f32" if c["kv"] == "f32" else "bf16")


def _verify_state(c, seed, out):
    i = W.make_verify_inputs(_vspec(c), seed, device=DEV, poison=None)
    B, Hq, D, k = c["B"], c["Hq"], c["D"], c["k"]
    return dict(i=i, kv=spire.kv_view(i.k_cache, i.v_cache, i.block_table, i.page_size, i.k_scale, i.v_scale),
                out=torch.empty((B, k + 1, Hq, D), dtype=DT[out], device=DEV),
                lse=torch.empty((B, k + 1, Hq), dtype=torch.float32, device=DEV),
                ws=spire.workspace(spire.verify_workspace_size(B, Hq, c["Hkv"], D, k)))


def _run_verify(c, s):
    i = s["i"]
    return spire.verify_attn(i.q, s["kv"], i.kv_lens, c["Hkv"], c["k"], i.sm_scale, out=s["out"], lse=s["lse"], ws=s["ws"])


def _draft_state(c, seed, steps, out):
    i = W.make_draft_inputs(_dspec(c, steps), seed, device=DEV, poison=None)
    B, Hq, D = c["B"], c["Hq"], c["D"]
    return dict(i=i, sink=spire.kv_view(i.sink_k, i.sink_v, k_scale=i.k_scale, v_scale=i.v_scale),
                ring=spire.kv_view(i.ring_k, i.ring_v, k_scale=i.k_scale, v_scale=i.v_scale),
                q=[i.q[t].contiguous() for t in range(steps)], lens=[i.seq_lens(t) for t in range(steps)],
                out=[torch.empty((B, Hq, D), dtype=DT[out], device=DEV) for _ in range(steps)],
                lse=[torch.empty((B, Hq), dtype=torch.float32, device=DEV) for _ in range(steps)],
                ws=spire.workspace(spire.draft_workspace_size(B, Hq, c["Hkv"], D)))


def _run_draft(c, s, t):
    i = s["i"]
    return spire.draft_sparse_attn(s["q"][t], s["sink"], s["ring"], s["lens"][t], i.ring_offset, c["S"], c["W"],
                                   i.sm_scale, c["Hkv"], out=s["out"][t], lse=s["lse"][t], ws=s["ws"])


def _token_state(c, seed):
    size = spire.block_verify_workspace_size if c["kind"] == "block" else spire.token_verify_workspace_size
    return dict(t=W.make_token_inputs(W.TokenSpec(B=c["B"], k=c["k"], V=c["V"]), seed, device=DEV),
                n=torch.empty((c["B"],), dtype=torch.int32, device=DEV),
                tok=torch.empty((c["B"], c["k"] + 1), dtype=torch.int32, device=DEV),
                tws=spire.workspace(size(c["B"], c["k"], c["V"])))


def _run_token(c, s):
    t, fn = s["t"], spire.block_verify if c["kind"] == "block" else spire.token_verify
    return fn(t.p, t.q, t.draft, t.u_accept, t.u_sample, n_accepted=s["n"], tokens=s["tok"], ws=s["tws"])


def prepare(c, seed):
    kind = c["kind"]
    if kind == "verify":
        s = _verify_state(c, seed, c["out"])
    elif kind == "draft":
        s = _draft_state(c, seed, 1, c["out"])
        W.write_step_token(s["i"], 0)
    elif kind in ("token", "block"):
        s = _token_state(c, seed)
    elif kind == "kv":
        i = W.make_kvupdate_inputs(W.KvUpdateSpec(B=c["B"], Hkv=c["Hkv"], D=c["D"], k=c["k"], S=c["S"], W=c["W"],
                                                  ctx_lo=c["lo"], ctx_hi=c["hi"], kv_dtype=c["kv"],
                                                  page_size=c["page"]), seed, device=DEV)
        # a page pool of one size for every seed: the pages that the contexts' ends map, and spare ones
        pool = (c["B"] * (c["k"] // c["page"] + 2),) + tuple(i.k_cache.shape[1:])
        kc, vc = (torch.zeros(pool, dtype=i.k_cache.dtype, device=DEV) for _ in range(2))
        _bytes(kc)[: i.k_cache.shape[0]].copy_(_bytes(i.k_cache))
        _bytes(vc)[: i.v_cache.shape[0]].copy_(_bytes(i.v_cache))
        s = dict(i=i, kc=kc, vc=vc, kv=spire.kv_view(kc, vc, i.block_table, c["page"], i.k_scale, i.v_scale),
                 sink=spire.kv_view(i.sink_k, i.sink_v, k_scale=i.k_scale, v_scale=i.v_scale),
                 ring=spire.kv_view(i.ring_k, i.ring_v, k_scale=i.k_scale, v_scale=i.v_scale),
                 lens=[i.base_lens + t + 1 for t in range(c["k"])],
                 spill_k=torch.zeros((c["k"],) + tuple(i.draft_k.shape[1:]), dtype=i.ring_k.dtype, device=DEV),
                 spill_v=torch.zeros((c["k"],) + tuple(i.draft_k.shape[1:]), dtype=i.ring_k.dtype, device=DEV))
    elif kind == "fm":
        i = W.make_feedback_inputs(W.FeedbackSpec(B=c["B"], d=c["d"], layers=c["layers"], n_out=c["n_out"],
                                                  x_dtype=c["x"], m_dtype=c["m"]), seed, device=DEV)
        s = dict(i=i, out=torch.empty((c["n_out"], c["B"], c["d"]), dtype=DT[c["m"]], device=DEV))
    else:  # round: the draft's and the target's caches of the same requests, and the tokens' distributions
        s = dict(v=_verify_state(c, seed, "bf16"), d=_draft_state(c, seed, c["k"], "bf16"))
        s.update(_token_state(c, seed))
        B, k = c["B"], c["k"]
        # the draft and target caches hold the same contexts (both drawn first, from the same seed)
        dt = s["d"]["i"].ring_k.dtype
        s["new_k"] = torch.randn((B, k + 1, c["Hkv"], c["D"]), device=DEV, generator=_gen(seed + 1)).to(torch.bfloat16)
        s["new_v"] = torch.randn((B, k + 1, c["Hkv"], c["D"]), device=DEV, generator=_gen(seed + 2)).to(torch.bfloat16)
        s["dk"] = [s["new_k"][:, t].contiguous() for t in range(k)]
        s["dv"] = [s["new_v"][:, t].contiguous() for t in range(k)]
        s["base"] = s["v"]["i"].kv_lens - (k + 1)
        s["spill_k"] = torch.zeros((k, B, c["Hkv"], c["D"]), dtype=dt, device=DEV)
        s["spill_v"] = torch.zeros((k, B, c["Hkv"], c["D"]), dtype=dt, device=DEV)
    s["c"] = c
    return s


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


# ---- one pass -----------------------------------------------------------------------
def _bytes(t):
    """fp8 storage as its bytes."""
    return t.view(torch.uint8) if t.dtype == torch.float8_e4m3fn else t


def run(s):
    c = s["c"]
    kind = c["kind"]
    if kind == "verify":
        return _run_verify(c, s)
    if kind == "draft":
        return _run_draft(c, s, 0)
    if kind in ("token", "block"):
        return _run_token(c, s)
    i = s.get("i")
    if kind == "fm":
        return spire.feedback_memory(i.x, i.w, out=s["out"])
    if kind == "kv":
        for t in range(c["k"]):
            spire.draft_append(s["sink"], s["ring"], i.draft_k[t], i.draft_v[t], s["lens"][t], i.ring_offset,
                               c["S"], c["W"], s["spill_k"][t], s["spill_v"][t])
        spire.kv_append(s["kv"], i.new_k, i.new_v, i.base_lens)
        spire.draft_rollback(s["sink"], s["ring"], s["spill_k"], s["spill_v"], i.base_lens, i.n_accepted,
                             i.ring_offset, c["S"], c["W"])
        return [_bytes(t) for t in (s["kc"], s["vc"], i.sink_k, i.sink_v, i.ring_k, i.ring_v, s["spill_k"], s["spill_v"])]
    v, d = s["v"], s["d"]
    for t in range(c["k"]):
        spire.draft_append(d["sink"], d["ring"], s["dk"][t], s["dv"][t], d["lens"][t], d["i"].ring_offset,
                           c["S"], c["W"], s["spill_k"][t], s["spill_v"][t])
        _run_draft(c, d, t)
    spire.kv_append(v["kv"], s["new_k"], s["new_v"], s["base"])
    _run_verify(c, v)
    n, tok = _run_token(c, s)
    spire.draft_rollback(d["sink"], d["ring"], s["spill_k"], s["spill_v"], s["base"], n, d["i"].ring_offset, c["S"], c["W"])
    return dict(drafts=d["out"], draft_lse=d["lse"], out=v["out"], lse=v["lse"], n=n, tokens=tok,
                ring_k=_bytes(d["i"].ring_k), ring_v=_bytes(d["i"].ring_v))


# ---- what a pass cannot do without ----------------------------------------------------
def _mean(lo, hi):
    return lo if lo == hi else (hi - lo) / math.log(hi / lo)


def _attn_work(c, keys, k, out):
    """Visible K and V once, queries, outputs and their log-sum-exps."""
    rows = c["B"] * c["Hq"] * (k + 1)
    qs, os = (4 if c["kv"] == "f32" else 2), (4 if out == "f32" else 2)
    b = 2 * c["B"] * keys * c["Hkv"] * c["D"] * ES[c["kv"]] + rows * (c["D"] * (qs + os) + 4) + 4 * c["B"]
    if c.get("page", 0) and c["kind"] != "draft":
        b += 4 * c["B"] * keys / c["page"]
    return b, 4.0 * rows * keys * c["D"]


def _window(c):
    """Mean visible keys of a draft step over log-uniform contexts."""
    n, lo, hi = c["S"] + c["W"], c["lo"], c["hi"]
    if lo == hi or hi <= n or lo >= n:
        return min(n, _mean(lo, hi))
    return ((n - lo) + n * math.log(hi / n)) / math.log(hi / lo)


def _kv_bytes(c, src):
    row, es = c["B"] * c["Hkv"] * c["D"] * 2, ES[c["kv"]]
    # draft writes: the new row in, the old row read, spilled and overwritten; the append; rejected rows back
    return c["k"] * row * (src + 3 * es) + (c["k"] + 1) * row * (src + es) + 0.3 * c["k"] * row * 2 * es


def work(c):
    kind = c["kind"]
    if kind == "verify":
        b, f = _attn_work(c, _mean(c["lo"], c["hi"]) + c["k"] + 1, c["k"], c["out"])
    elif kind == "draft":
        b, f = _attn_work(c, _window(c), 0, c["out"])
    elif kind == "token":  # one row of p and of q per sequence
        b, f = 8.0 * c["B"] * c["V"] + 16 * c["B"] * (c["k"] + 1), 2.0 * c["B"] * c["V"]
    elif kind == "block":  # every row
        b, f = 4.0 * c["B"] * (2 * c["k"] + 1) * c["V"], 4.0 * c["B"] * c["k"] * c["V"]
    elif kind == "kv":
        b, f = _kv_bytes(c, 4), 0
    elif kind == "fm":
        n = c["B"] * c["d"]
        b = n * (c["layers"] * (4 if c["x"] == "f32" else 2) + c["n_out"] * (4 if c["m"] == "f32" else 2))
        f = 2.0 * n * c["layers"] * c["n_out"]
    else:
        bv, fv = _attn_work(c, _mean(c["lo"], c["hi"]) + c["k"] + 1, c["k"], "bf16")
        bd, fd = _attn_work(dict(c, kind="draft"), _window(c), 0, "bf16")
        b = bv + c["k"] * bd + 8.0 * c["B"] * c["V"] + _kv_bytes(c, 2)
        f = fv + c["k"] * fd
    return {"bytes": float(b), "flops": float(f)}


def tolerance(c):
    """Attention on bf16 and fp8 caches rounds the probabilities (bf16: 2^-9,
    fp8: 2^-11) and, where asked, the output (2^-9) once; f32 caches keep fp32
    throughout.  Verification, sampling and cache writes are exact."""
    kind = c["kind"]
    if kind in ("token", "block", "kv"):
        return "exact"
    if kind == "fm":
        return {"rel": 1e-5} if c["m"] == "f32" else {"rel": 1e-2}
    if c["kv"] == "f32" and c["out"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 1e-2}


# ---- the same in 64 bits ---------------------------------------------------------------
def _attend(q, K, V, limit, scale):
    """q [Hkv, rows, D], K / V [Hkv, n, D] in fp64; row r sees keys [0, limit[r])."""
    s = torch.matmul(q, K.transpose(1, 2).contiguous()) * scale
    s = s.masked_fill(torch.arange(K.shape[1], device=DEV)[None, None, :] >= limit[None, :, None], -math.inf)
    lse = torch.logsumexp(s, dim=-1)
    return torch.matmul(torch.exp(s - lse[..., None]), V), lse


def _exact_verify(c, i):
    B, Hq, Hkv, D, k = c["B"], c["Hq"], c["Hkv"], c["D"], c["k"]
    g = Hq // Hkv
    out = torch.zeros((B, k + 1, Hq, D), dtype=torch.float64, device=DEV)
    lse = torch.zeros((B, k + 1, Hq), dtype=torch.float64, device=DEV)
    ks, vs = ((i.k_scale.double().view(-1, 1, 1), i.v_scale.double().view(-1, 1, 1)) if i.k_scale is not None else (1.0, 1.0))
    for b, n in enumerate(i.kv_lens.tolist()):
        if c["page"]:
            pages = i.block_table[b, : (n + c["page"] - 1) // c["page"]].long()
            K, V = (_bytes(x)[pages].view(x.dtype).transpose(0, 1).reshape(Hkv, -1, D)[:, :n].double() for x in (i.k_cache, i.v_cache))
        else:
            K, V = i.k_cache[b, :, :n].double(), i.v_cache[b, :, :n].double()
        q = i.q[b].double().view(k + 1, Hkv, g, D).permute(1, 0, 2, 3).reshape(Hkv, (k + 1) * g, D)
        limit = n - k + torch.arange(k + 1, device=DEV).repeat_interleave(g)
        o, l = _attend(q, K * ks, V * vs, limit, i.sm_scale)
        out[b] = o.view(Hkv, k + 1, g, D).permute(1, 0, 2, 3).reshape(k + 1, Hq, D)
        lse[b] = l.view(Hkv, k + 1, g).permute(1, 0, 2).reshape(k + 1, Hq)
    return out, lse


def _exact_draft(c, i, q, m_all):
    B, Hq, Hkv, D, S, Wn = c["B"], c["Hq"], c["Hkv"], c["D"], c["S"], c["W"]
    g = Hq // Hkv
    out = torch.zeros((B, Hq, D), dtype=torch.float64, device=DEV)
    lse = torch.zeros((B, Hq), dtype=torch.float64, device=DEV)
    ks, vs = ((i.k_scale.double().view(-1, 1, 1), i.v_scale.double().view(-1, 1, 1)) if i.k_scale is not None else (1.0, 1.0))
    off = i.ring_offset.tolist()
    for b, m in enumerate(m_all.tolist()):
        slots = (off[b] + torch.arange(max(S, m - Wn), m, device=DEV) - S) % Wn
        K, V = (torch.cat([x[b, :, : min(S, m)].double(), y[b].double()[:, slots]], dim=1)
                for x, y in ((i.sink_k, i.ring_k), (i.sink_v, i.ring_v)))
        limit = torch.full((g,), K.shape[1], device=DEV)
        o, l = _attend(q[b].double().view(Hkv, g, D), K * ks, V * vs, limit, i.sm_scale)
        out[b], lse[b] = o.reshape(Hq, D), l.reshape(Hq)
    return out, lse


def exact(c, seed):
    kind = c["kind"]
    if kind == "verify":
        return _exact_verify(c, prepare(c, seed)["i"])
    if kind == "draft":
        s = prepare(c, seed)
        return _exact_draft(c, s["i"], s["q"][0], s["lens"][0])
    if kind == "fm":
        i = prepare(c, seed)["i"]
        return torch.einsum("il,lbd->ibd", torch.softmax(i.w.double(), dim=-1), i.x.double())
    return None  # tokens and stored bytes, compared whole; a round's attention is its layers', listed above
