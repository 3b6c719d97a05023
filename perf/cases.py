"""What a user of the head-wise attention library has it do, as cases that can be timed and compared.

A case is a dict of plain values; `kind` says which entry points a pass goes through:

  prefill  Session.prefill_group over the KV heads of one layer, chunk after chunk, behind `past` cached rows
  decode   Session.decode_group (or hi_decode_group_ragged over `sequences` of different lengths), one token, `layers` layers
  block    AttentionBlock.forward: Q/K/V projection with rotary embedding, attention, output projection
  window   Session.prefill_group over the streaming heads of a layer (Appendix E), two chunks of a fresh prompt
  proj     hi_qkv_rope and hi_out_proj alone
  rows4    hi_kv_quantize and hi_kv_dequantize, the 4-bit rows of the host link

Sizes are the repository's own: Llama-3-8B attention layers (32 query / 8 KV heads of 128 channels, hidden size 4096),
the contexts, chunks and head groups of its benchmark and tests.  Inputs are N(0, 1) rows in bf16, as everywhere in the
repository; `peaked` scales one key in ten by four, as its extreme-context configuration does.
"""
from __future__ import annotations

import math

import torch

from paper_2502_12574_amd import binding as hb
from paper_2502_12574_amd.attention_block import AttentionBlock
from paper_2502_12574_amd.session import Session

D = 128                          # channels of a head
DEV = "cuda:0"
THETA = 500000.0                 # rotary base of the evaluated model


def _prefill(name, **kw):
    c = dict(name=name, kind="prefill", offload=False, heads=8, group=4, past=0, rows=512, chunk=512, per_call=8,
             fp32=False, prescaled=False, peaked=False)
    c.update(kw)
    return c


def _decode(name, **kw):
    c = dict(name=name, kind="decode", offload=False, layers=1, heads=8, group=4, past=1024, per_call=8, sequences=1,
             fp32=False, prescaled=False, peaked=False)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest configuration of the benchmark: one KV head, 2048 tokens in chunks of 512, cache on the host
        _prefill("tiny_prefill", offload=True, heads=1, rows=2048, chunk=512, per_call=1, fp32=True),
        # a short question (odd length) behind a document of 100 thousand tokens that is already cached in HBM
        _prefill("followup_100k", past=100003, rows=77, chunk=77),
        # the last 8192-token chunk of a 128K prompt, K/V on the host, two heads per call as the plan recommends
        _prefill("prefill_128k", offload=True, past=122880, rows=8192, chunk=8192, per_call=2, prescaled=True),
        # one head of the last chunk of a 1M prompt: the unit that the headline benchmark repeats
        _prefill("prefill_1m_head", heads=1, past=(1 << 20) - 16384, rows=16384, chunk=16384, per_call=1, prescaled=True),
        # one token through 32 layers of attention at a 1K context, cache in HBM: launches and latency
        _decode("decode_stack_1k", layers=32, past=1000),
        # one token of one layer at 1M context, cache in HBM: the benchmark's HBM-roofline leg
        _decode("decode_1m", past=(1 << 20) - 64),
        # one token of one layer at 128K context, cache on the host
        _decode("decode_128k_link", offload=True, past=131072 - 64, per_call=2),
        # a whole attention block: a second turn of 600 tokens behind 3000, and one generated token behind 6000
        dict(name="block_turn", kind="block", past=3001, rows=600, prescaled=True),
        dict(name="block_token", kind="block", past=6003, rows=1, prescaled=True),
        # the streaming half of a layer's heads over a long prompt
        dict(name="streaming_prompt", kind="window", heads=4, group=4, chunk=8192, sink=128, recent=512, prescaled=False),
        # both projections of a full-size chunk
        dict(name="proj_16k", kind="proj", rows=16384, past=(1 << 20) - 16384, model=4096, q_heads=32, kv_heads=8),
        # a staging slice of 4-bit rows, both ways
        dict(name="rows4_slice", kind="rows4", rows=262144),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Sizes over the ranges of the listed cases: odd ones, other group sizes, fp32 output, plain and scaled queries."""
    kind = rng.choice(["prefill", "prefill", "followup", "decode", "decode", "ragged", "block", "window", "proj", "rows4"])
    group = rng.choice([1, 2, 4, 4, 4, 8])
    opt = dict(group=group, fp32=rng.random() < 0.25, prescaled=rng.random() < 0.5, peaked=rng.random() < 0.25)
    heads = 32 // group
    if kind == "prefill":
        offload = rng.random() < 0.5
        chunk = _log(rng, 128, 8192)
        rows = min(int(chunk * rng.uniform(1.0, 3.0)), 12288)
        past = rng.choice([0, _log(rng, 100, 60000)])
        per_call = min(heads, rng.choice([1, 2, 8]))
        # a staging slice (a quarter of one head's rows) holds 64 rows of every head of a group
        per_call = min(per_call, max(1, (past + rows) // 512)) if offload else per_call
        c = _prefill("", offload=offload, heads=heads, past=past, rows=rows, chunk=chunk, per_call=per_call, **opt)
    elif kind == "followup":
        rows = _log(rng, 2, 512)
        c = _prefill("", heads=heads, past=_log(rng, 2000, 120000), rows=rows, chunk=rows, per_call=heads, **opt)
    elif kind == "decode":
        offload = rng.random() < 0.3
        past = _log(rng, 600, (130000 if offload else 1 << 20) * 8 // max(8, heads))
        layers = 1 if past > 65536 else rng.choice([1, 4])
        per_call = min(2, heads) if offload else heads
        c = _decode("", offload=offload, layers=layers, heads=heads, past=past, per_call=per_call, **opt)
    elif kind == "ragged":
        opt["group"], seqs = 4, rng.choice([2, 3, 5, 8])
        c = _decode("", heads=8, past=_log(rng, 100, 60000), sequences=seqs, **opt)
    elif kind == "block":
        rows = rng.choice([1, _log(rng, 2, 3000)])
        c = dict(kind="block", past=_log(rng, 10, 30000), rows=rows, prescaled=rng.random() < 0.5)
    elif kind == "window":
        c = dict(kind="window", heads=rng.choice([2, 4]), group=4, chunk=_log(rng, 300, 8192), sink=rng.choice([0, 4, 64, 128]),
                 recent=_log(rng, 100, 2000), prescaled=opt["prescaled"])
    elif kind == "proj":
        model, q_heads, kv_heads = rng.choice([(4096, 32, 8), (4096, 32, 8), (1024, 8, 2), (8192, 64, 8)])
        c = dict(kind="proj", rows=_log(rng, 2, 12000), past=_log(rng, 1, 1 << 20), model=model, q_heads=q_heads, kv_heads=kv_heads)
    else:
        c = dict(kind="rows4", rows=_log(rng, 100, 500000))
    c.pop("name", None)
    return c


# ---- inputs, from the seed alone (the same tensors for the library and for exact()) -------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _rows(g, *shape, scale=1.0):
    x = torch.randn(*shape, dtype=torch.bfloat16, device=DEV, generator=g)
    return x if scale == 1.0 else (x.float() * scale).to(torch.bfloat16)


def _keys(case, g, *shape):
    k = _rows(g, *shape)
    if case.get("peaked"):
        k[torch.rand(shape[:-1], device=DEV, generator=g) < 0.1] *= 4
    return k


def _q_scale(case):
    return hb.HI_Q_PRESCALE if case["prescaled"] else 1.0


def _lens(case):
    """Cached rows of each sequence of a decode case (past, spread over the batch)."""
    b = case["sequences"]
    return [max(1, case["past"] * (j + 1) // b) for j in range(b)]


def _attn_inputs(case, seed, layer=0):
    """(past K/V [heads][2][past][D], q [heads][group][rows][D], new K/V [heads][2][rows][D]) of one layer."""
    g = _gen(seed * 1009 + layer)
    n = case.get("rows", 1)
    h = case["heads"] * case.get("sequences", 1)
    past = torch.empty(h, 2, case["past"], D, dtype=torch.bfloat16, device=DEV)
    for j in range(h if case["past"] else 0):
        past[j, 0] = _keys(case, g, case["past"], D)
        past[j, 1] = _rows(g, case["past"], D)
    q = _rows(g, h, case["group"], n, D, scale=_q_scale(case))
    new = torch.stack([_keys(case, g, h, n, D), _rows(g, h, n, D)], dim=1)
    return past, q, new


def _block_inputs(case, seed):
    g = _gen(seed)
    w_qkv, w_o = _rows(g, 48 * D, 4096, scale=1 / 64), _rows(g, 4096, 32 * D, scale=1 / 64)
    past = _rows(g, 8, 2, case["past"], D)
    return w_qkv, w_o, past, _rows(g, case["rows"], 4096)


def _window_inputs(case, seed):
    g = _gen(seed)
    n = 2 * case["chunk"]
    return (_rows(g, case["heads"], case["group"], n, D, scale=_q_scale(case)), _rows(g, case["heads"], n, D),
            _rows(g, case["heads"], n, D))


def _proj_inputs(case, seed):
    g = _gen(seed)
    m, hq, hkv, n = case["model"], case["q_heads"], case["kv_heads"], case["rows"]
    scale = 2.0 ** -round(math.log2(m) / 2)
    return (_rows(g, n, m), _rows(g, (hq + 2 * hkv) * D, m, scale=scale), _rows(g, hq, n, D), _rows(g, m, hq * D, scale=scale))


# ---- what a program has in hand ------------------------------------------------------------------------------------

_shared = []


def _session(n_layers, heads, group, context, chunk, **kw):
    """A Session on one set of streams for the whole program, as programs with several contexts have: the runtime maps
    the streams of a process to a few hardware queues, and streams of idle contexts would share them with busy ones."""
    ss = Session(n_layers, heads, group, max(context, 256), chunk, **kw)
    if not _shared:
        _shared.extend((ss.s_compute, ss.s_h2d, ss.s_d2h))
    hb.hi_ctx_destroy(ss.ctx)
    ss.s_compute, ss.s_h2d, ss.s_d2h = _shared
    ss.ctx = hb.hi_ctx_create(ss.problem, ss.plan, ss.mode, ss.kv, ss.staging, ss.workspace, *_shared)
    return ss


class _State:
    """A case's buffers; closes the Session it holds."""

    def __init__(self, case, ss=None, **kw):
        self.case, self.ss = case, ss
        self.__dict__.update(kw)

    def __del__(self):
        if self.ss is not None:
            self.ss.close()


def _fill_past(ss, layer, past):
    """The cached rows of a layer as earlier calls left them."""
    view = ss.cache_view()
    n = past.shape[2]
    for j in range(past.shape[0] if n else 0):
        for w in range(2):
            view[layer, j, w, :n].copy_(past[j, w])


def prepare(case, seed):
    kind = case["kind"]
    if kind == "prefill":
        past, q, new = _attn_inputs(case, seed)
        ss = _session(1, case["heads"], case["group"], case["past"] + case["rows"], case["chunk"],
                     mode=hb.HI_MODE_OFFLOAD if case["offload"] else hb.HI_MODE_RESIDENT, out_fp32=int(case["fp32"]),
                     q_prescaled=case["prescaled"])
        _fill_past(ss, 0, past)
        chunks = []
        for p in range(0, case["rows"], case["chunk"]):
            e = min(p + case["chunk"], case["rows"])
            chunks.append((case["past"] + p, q[:, :, p:e].contiguous(), new[:, 0, p:e].contiguous(), new[:, 1, p:e].contiguous(),
                           torch.empty(case["heads"], case["group"], e - p, D, dtype=ss.out_dtype, device=DEV)))
        return _State(case, ss, chunks=chunks, appended=ss.cache_view()[0, :, :, case["past"]:case["past"] + case["rows"]])
    if kind == "decode":
        heads = case["heads"] * case["sequences"]
        ss = _session(case["layers"], heads, case["group"], case["past"] + 1, 1,
                     mode=hb.HI_MODE_OFFLOAD if case["offload"] else hb.HI_MODE_RESIDENT, out_fp32=int(case["fp32"]),
                     q_prescaled=case["prescaled"])
        layers = []
        for l in range(case["layers"]):
            past, q, new = _attn_inputs(case, seed, l)
            _fill_past(ss, l, past)
            layers.append((q[:, :, 0].contiguous(), new[:, 0, 0].contiguous(), new[:, 1, 0].contiguous()))
        out = torch.empty(case["layers"], heads, case["group"], D, dtype=ss.out_dtype, device=DEV)
        lens = [n for n in _lens(case) for _ in range(case["heads"])]
        view = ss.cache_view()
        appended = [view[:, j:j + case["heads"], :, lens[j]] for j in range(0, heads, case["heads"])] if case["sequences"] > 1 else \
            [view[:, :, :, case["past"]]]
        return _State(case, ss, layers=layers, out=out, lens=lens, appended=appended)
    if kind == "block":
        w_qkv, w_o, past, x = _block_inputs(case, seed)
        ss = _session(1, 8, 4, case["past"] + case["rows"], max(case["rows"], 2), mode=hb.HI_MODE_RESIDENT, out_fp32=0,
                     q_prescaled=case["prescaled"])
        _fill_past(ss, 0, past)
        return _State(case, ss, block=AttentionBlock(ss, 0, w_qkv, w_o, THETA), x=x, y=torch.empty_like(x),
                      appended=ss.cache_view()[0, :, :, case["past"]:case["past"] + case["rows"]])
    if kind == "window":
        q, k, v = _window_inputs(case, seed)
        n, h = case["chunk"], case["heads"]
        ss = _session(1, 2 * h, case["group"], 2 * n, n, mode=hb.HI_MODE_RESIDENT, out_fp32=0, streaming_heads=h,
                     sink_tokens=case["sink"], recent_tokens=case["recent"], q_prescaled=case["prescaled"])
        ss.staging.zero_()
        chunks = [(p, q[:, :, p:p + n].contiguous(), k[:, p:p + n].contiguous(), v[:, p:p + n].contiguous(),
                   torch.empty(h, case["group"], n, D, dtype=ss.out_dtype, device=DEV)) for p in (0, n)]
        return _State(case, ss, chunks=chunks, store=ss.stream_view())
    if kind == "proj":
        x, w_qkv, attn, w_o = _proj_inputs(case, seed)
        n, hq, hkv = case["rows"], case["q_heads"], case["kv_heads"]
        outs = [torch.empty(h, n, D, dtype=torch.bfloat16, device=DEV) for h in (hq, hkv, hkv)]
        return _State(case, x=x, w_qkv=w_qkv, attn=attn, w_o=w_o, outs=outs, y=torch.empty_like(x),
                      ws=torch.empty(hb.hi_proj_workspace_bytes(n), dtype=torch.uint8, device=DEV))
    rows = _rows(_gen(seed), case["rows"], D)
    return _State(case, rows=rows, packed=torch.empty(case["rows"], 80, dtype=torch.uint8, device=DEV), back=torch.empty_like(rows))


# ---- one pass ------------------------------------------------------------------------------------------------------

def _groups(case):
    return [(h, min(case["per_call"], case["heads"] - h)) for h in range(0, case["heads"], case["per_call"])]


def run(st):
    case, ss = st.case, st.ss
    here = torch.cuda.current_stream()
    kind = case["kind"]
    if ss is not None:
        ss.s_compute.wait_stream(here)              # the inputs come from the program's own stream, the outputs go back to it
    if kind == "prefill":
        units = [(c, g) for c in range(len(st.chunks)) for g in _groups(case)]
        for i, (c, (h, nh)) in enumerate(units):
            past, q, k, v, out = st.chunks[c]
            nxt = None
            if case["offload"] and i + 1 < len(units):
                c2, (h2, nh2) = units[i + 1]
                nxt = (0, h2, nh2, st.chunks[c2][0])
            ss.prefill_group(0, h, nh, q[h:h + nh], k[h:h + nh], v[h:h + nh], past, out[h:h + nh], nxt)
        outs = {"out": [c[4] for c in st.chunks], "appended": st.appended}
    elif kind == "decode" and case["sequences"] > 1:
        for l, (q, k, v) in enumerate(st.layers):
            hb.hi_decode_group_ragged(ss.ctx, l, 0, q.shape[0], q, k, v, st.lens, st.out[l])
        outs = {"out": st.out, "appended": st.appended}
    elif kind == "decode":
        units = [(l, g) for l in range(case["layers"]) for g in _groups(case)]
        for i, (l, (h, nh)) in enumerate(units):
            q, k, v = st.layers[l]
            nxt = None
            if case["offload"] and i + 1 < len(units):
                l2, (h2, nh2) = units[i + 1]
                nxt = (l2, h2, nh2, case["past"])
            ss.decode_group(l, h, nh, q[h:h + nh], k[h:h + nh], v[h:h + nh], case["past"], st.out[l, h:h + nh], nxt)
        outs = {"out": st.out, "appended": st.appended}
    elif kind == "block":
        st.block.forward(st.x, case["past"], st.y)
        outs = {"y": st.y, "appended": st.appended}
    elif kind == "window":
        h = case["heads"]
        for past, q, k, v, out in st.chunks:
            ss.prefill_group(0, h, h, q, k, v, past, out)
        outs = {"out": [c[4] for c in st.chunks], "store": st.store}
    elif kind == "proj":
        m, hq, hkv, n = case["model"], case["q_heads"], case["kv_heads"], case["rows"]
        hb.hi_qkv_rope(here, st.x, st.w_qkv, m, hq, hkv, n, case["past"], THETA, 0, *st.outs, st.ws)
        hb.hi_out_proj(here, st.attn, st.w_o, hq, m, n, 0, st.y)
        outs = {"qkv": st.outs, "y": st.y}
    else:
        hb.hi_kv_quantize(here, st.rows, case["rows"], st.packed)
        hb.hi_kv_dequantize(here, st.packed, case["rows"], st.back)
        outs = {"packed": st.packed, "rows": st.back}
    if ss is not None:
        here.wait_stream(ss.s_compute)
    return outs


# ---- what a pass cannot do without ---------------------------------------------------------------------------------

def _visible(case):
    """(row, key) pairs of the windowed attention of one query head over the two chunks, and key rows read."""
    n, total = 2 * case["chunk"], 0
    full = case["sink"] + case["recent"]
    for p in range(min(n, full)):
        total += p + 1
    return total + max(0, n - full) * full


def work(case):
    kind = case["kind"]
    if kind == "prefill":
        n, p, h, g = case["rows"], case["past"], case["heads"], case["group"]
        pairs = n * p + n * (n + 1) // 2
        # each pass over the past is one chunk's: a later chunk has to see the rows of the earlier ones again
        past_rows = sum(p + c for c in range(0, n, case["chunk"]))
        return {"flops": 4.0 * D * g * h * pairs,
                "bytes": 512.0 * h * (past_rows + 2 * n) + h * g * n * D * (2.0 + (4 if case["fp32"] else 2))}
    if kind == "decode":
        rows = case["layers"] * case["heads"] * (sum(_lens(case)) if case["sequences"] > 1 else case["past"])
        heads = case["layers"] * case["heads"] * case["sequences"]
        return {"flops": 4.0 * D * case["group"] * (rows + heads),
                "bytes": 512.0 * (rows + 2 * heads) + heads * case["group"] * D * (2.0 + (4 if case["fp32"] else 2))}
    if kind == "block":
        n, p = case["rows"], case["past"]
        return {"flops": 2.0 * n * 4096 * (48 + 32) * D + 4.0 * D * 32 * (n * p + n * (n + 1) // 2),
                "bytes": 2.0 * 4096 * (48 + 32) * D + 512.0 * 8 * (p + n) + 4.0 * n * 4096}
    if kind == "window":
        h, g, n = case["heads"], case["group"], 2 * case["chunk"]
        return {"flops": 4.0 * D * g * h * _visible(case),
                "bytes": 512.0 * h * (n + min(n, case["sink"] + case["recent"])) + 4.0 * h * g * n * D}
    if kind == "proj":
        m, hq, hkv, n = case["model"], case["q_heads"], case["kv_heads"], case["rows"]
        outs = (hq + 2 * hkv) * D
        return {"flops": 2.0 * n * m * (outs + hq * D), "bytes": 2.0 * (m * (outs + hq * D) + n * (2 * m + outs + hq * D))}
    return {"flops": 0.0, "bytes": case["rows"] * 2.0 * (256 + 80)}


def tolerance(case):
    if case["kind"] == "rows4":
        return "exact"                                   # codes, scales and zeros are fixed bit by bit, so the rows are too
    if case["kind"] == "block":
        return {"rel": 1.2e-2, "max": 0.1}               # q, k, v, the attention output and y are each rounded to bf16
    if case["kind"] == "proj":
        return {"rel": 2e-3, "max": 3e-2}                # one rounding to bf16; fp32 sums in another order move some by one step
    return {"rel": 8e-3, "max": 0.06}                    # softmax weights and outputs in bf16


# ---- the same values in 64 bits, in plain torch --------------------------------------------------------------------

def _attend64(q, k, v, first, prescaled, sink=None, recent=None):
    """q [G][n][D] rows at positions first .., k, v [S][D] rows at positions 0 ..: causal (and windowed) attention."""
    scale = math.log(2.0) if prescaled else 1.0 / math.sqrt(D)
    G, n, _ = q.shape
    out = torch.empty(G, n, D, dtype=torch.float64, device=DEV)
    k, v = k.double(), v.double()
    if recent is not None:
        step = 512
    else:
        step = max(1, min(n, (1 << 29) // max(1, (first + n) * G)))
    for a in range(0, n, step):
        b = min(n, a + step)
        keys = torch.arange(first + b, device=DEV)
        if recent is not None:
            keys = keys[(keys < sink) | (keys > first + a - recent)]
        kk, vv = (k[:first + b], v[:first + b]) if recent is None else (k[keys], v[keys])
        s = (q[:, a:b].reshape(-1, D).double() @ kk.t().contiguous()).view(G, b - a, -1).mul_(scale)
        pos = torch.arange(first + a, first + b, device=DEV)
        if recent is not None:
            seen = (keys[None] <= pos[:, None]) & ((keys[None] < sink) | (pos[:, None] - keys[None] < recent))
            s.masked_fill_(~seen, float("-inf"))
        elif b - a > 1:
            tail = first + a                                  # only the block's own rows can lie ahead of one of them
            s[:, :, tail:].masked_fill_(keys[None, tail:] > pos[:, None], float("-inf"))
        s.sub_(s.amax(-1, keepdim=True)).exp_()
        w = s.sum(-1)
        out[:, a:b] = (s.view(G * (b - a), -1) @ vv).view(G, b - a, D) / w[..., None]
    return out


def _rope64(x, past):
    """x [heads][n][D]: rotate channel i < 64 with channel i + 64 by position * THETA^(-i / 64)."""
    n = x.shape[1]
    pos = torch.arange(past, past + n, dtype=torch.float64, device=DEV)
    ang = pos[:, None] * THETA ** (-torch.arange(64, dtype=torch.float64, device=DEV) / 64)[None]
    c, s = ang.cos(), ang.sin()
    lo, hi = x[..., :64], x[..., 64:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], dim=-1)


def _qkv64(x, w, hq, hkv, past):
    y = (x.double() @ w.double().t().contiguous()).view(x.shape[0], hq + 2 * hkv, D).transpose(0, 1)
    return _rope64(y[:hq], past), _rope64(y[hq:hq + hkv], past), y[hq + hkv:].contiguous()


def exact(case, seed):
    kind = case["kind"]
    if kind == "prefill":
        past, q, new = _attn_inputs(case, seed)
        kv = torch.cat([past, new], dim=2)
        full = torch.stack([_attend64(q[h], kv[h, 0], kv[h, 1], case["past"], case["prescaled"]) for h in range(case["heads"])])
        outs = [full[:, :, p:p + case["chunk"]].contiguous() for p in range(0, case["rows"], case["chunk"])]
        return {"out": outs, "appended": None}
    if kind == "decode":
        out = torch.empty(case["layers"], case["heads"] * case["sequences"], case["group"], D, dtype=torch.float64, device=DEV)
        for l in range(case["layers"]):
            past, q, new = _attn_inputs(case, seed, l)
            for h in range(q.shape[0]):
                n = _lens(case)[h // case["heads"]]
                kv = torch.cat([past[h, :, :n], new[h]], dim=1)
                out[l, h] = _attend64(q[h], kv[0], kv[1], n, case["prescaled"])[:, 0]
        return {"out": out, "appended": None}
    if kind == "block":
        w_qkv, w_o, past, x = _block_inputs(case, seed)
        q, k, v = _qkv64(x, w_qkv, 32, 8, case["past"])
        new = torch.stack([k, v], dim=1)
        kv = torch.cat([past.double(), new], dim=2)
        attn = torch.stack([_attend64(q[4 * h:4 * h + 4], kv[h, 0], kv[h, 1], case["past"], False) for h in range(8)])
        y = attn.view(32, -1, D).transpose(0, 1).reshape(-1, 32 * D) @ w_o.double().t().contiguous()
        return {"y": y, "appended": new}
    if kind == "window":
        q, k, v = _window_inputs(case, seed)
        full = torch.stack([_attend64(q[h], k[h], v[h], 0, case["prescaled"], case["sink"], case["recent"])
                            for h in range(case["heads"])])
        n = case["chunk"]
        return {"out": [full[:, :, p:p + n].contiguous() for p in (0, n)], "store": None}
    if kind == "proj":
        x, w_qkv, attn, w_o = _proj_inputs(case, seed)
        q, k, v = _qkv64(x, w_qkv, case["q_heads"], case["kv_heads"], case["past"])
        y = attn.transpose(0, 1).reshape(case["rows"], -1).double() @ w_o.double().t().contiguous()
        return {"qkv": [q, k, v], "y": y}
    # the codes are defined by single-precision steps; the decoded value is zero + code * scale
    x = _rows(_gen(seed), case["rows"], D).float().view(-1, 4, 32)
    zero = x.amin(-1, keepdim=True)
    scale = ((x.amax(-1, keepdim=True) - zero) * (torch.ones((), device=DEV) / 15.0)).to(torch.bfloat16).float()
    scale = torch.where(scale >= 2.0 ** -120, scale, torch.zeros_like(scale))
    inv = torch.where(scale > 0, 1.0 / scale, torch.zeros_like(scale))
    code = torch.clamp(torch.round((x - zero) * inv), max=15.0)
    return {"packed": None, "rows": (zero.double() + code.double() * scale.double()).view(-1, D)}
