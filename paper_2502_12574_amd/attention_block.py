"""One layer's attention block on top of the library: hidden states -> Q/K/V projection with rotary embedding
(hi_qkv_rope) -> head-wise attention with offloaded / resident / streaming KV heads (hi_prefill_group,
hi_decode_group, Algorithm 1's head loop) -> output projection (hi_out_proj).

Only buffers and call order live here; every step runs in the library.  The projection writes Q, K and V
head-major, which is what the attention calls read, and the attention calls write the head-major block the
output projection reads: nothing is reshuffled in between.
"""
from __future__ import annotations

import torch

from . import binding as hb
from .session import Session


class AttentionBlock:
    """The attention block of layer `layer` of a Session (the Session owns the K/V cache of all layers).

    w_qkv [(Hq + 2 Hkv) * 128][d_model] (rows of W_Q, W_K, W_V) and w_o [d_model][Hq * 128], bf16 on the device.
    Heads are called in groups of plan.heads_per_group, retrieval heads first, then the streaming heads."""

    def __init__(self, ss: Session, layer: int, w_qkv: torch.Tensor, w_o: torch.Tensor, rope_theta: float = 500000.0):
        p = ss.problem
        self.ss, self.layer, self.theta = ss, layer, rope_theta
        self.Hkv, self.G, self.Hq, self.D = p.n_kv_heads, p.gqa_group, p.n_kv_heads * p.gqa_group, w_o.shape[0]
        assert w_qkv.shape == ((self.Hq + 2 * self.Hkv) * 128, self.D) and w_o.shape == (self.D, self.Hq * 128)
        self.w_qkv, self.w_o = w_qkv, w_o
        C, dev = p.chunk, ss.device
        self.q = torch.empty(self.Hq * C * 128, dtype=torch.bfloat16, device=dev)
        # K/V of a call are borrowed by its asynchronous write-back to the host: two sets, used in turn, and a set
        # is written again only after the write-back stream has passed the call that last used it
        self.kv = [(torch.empty(self.Hkv * C * 128, dtype=torch.bfloat16, device=dev),
                    torch.empty(self.Hkv * C * 128, dtype=torch.bfloat16, device=dev)) for _ in range(2)]
        self.kv_done = [None, None]
        self.turn = 0
        self.attn = torch.empty(self.Hq * C * 128, dtype=torch.bfloat16, device=dev)
        self.ws = torch.empty(hb.hi_proj_workspace_bytes(C), dtype=torch.uint8, device=dev)
        n_ret, g = self.Hkv - p.streaming_heads, max(1, ss.plan.heads_per_group)
        self.calls = [(h, min(g, n_ret - h)) for h in range(0, n_ret, g)]
        self.calls += [(h, min(g, self.Hkv - h)) for h in range(n_ret, self.Hkv, g)]

    def forward(self, x: torch.Tensor, past_len: int, y: torch.Tensor, nxt=None):
        """x [n][d_model] bf16 hidden states of the tokens at positions past_len .., n = 1 for a decode step;
        y [n][d_model] bf16 receives the block's output.  nxt: the (layer, first head, heads, past) unit that will
        be called after this block's last one, for the prefetch.  Enqueues on the Session's compute stream.

        A generated token is 4 to 5 launches of about 10 us each, so the calls hand addresses to the library instead of
        slicing views for every head group: head-major q and output are [Hkv][G][n][128], k and v [Hkv][n][128]."""
        ss, n = self.ss, x.shape[0]
        assert ss.out_dtype == torch.bfloat16, "the output projection reads bf16 attention outputs"
        if n > ss.problem.chunk:                 # before anything is enqueued: the projection would write past these buffers
            raise RuntimeError(f"{n} rows in one call: the block's buffers hold the Session's chunk of {ss.problem.chunk}")
        # a launch goes to a stream of the current device: make it the Session's, whatever the caller's is
        with torch.cuda.device(ss.s_compute.device_index):
            k, v = self.kv[self.turn]
            q, k, v, o = self.q.data_ptr(), k.data_ptr(), v.data_ptr(), self.attn.data_ptr()
            s, row = ss.s_compute, n * 256                       # bytes of one head's rows of this call
            offload = ss.mode == hb.HI_MODE_OFFLOAD              # (resident heads are appended on the compute stream itself)
            if offload and self.kv_done[self.turn] is not None:
                s.wait_event(self.kv_done[self.turn])
            # the softmax scale rides on the queries when the Session's attention calls expect it there
            hb.hi_qkv_rope(s, x, self.w_qkv, self.D, self.Hq, self.Hkv, n, past_len, self.theta, 0, q, k, v, self.ws,
                           q_scale=hb.HI_Q_PRESCALE if ss.problem.q_prescaled else 1.0)
            for i, (h0, nh) in enumerate(self.calls):
                hint = nxt
                if i + 1 < len(self.calls):
                    hint = (self.layer, self.calls[i + 1][0], self.calls[i + 1][1], past_len)
                nl, nhead, nheads, npast = hint if hint is not None else (-1, 0, 1, 0)
                at, at_q = h0 * row, h0 * self.G * row
                if n == 1:
                    hb.hi_decode_group(ss.ctx, self.layer, h0, nh, q + at_q, k + at, v + at, past_len, o + at_q, nl,
                                       nhead, nheads, npast)
                else:
                    hb.hi_prefill_group(ss.ctx, self.layer, h0, nh, q + at_q, k + at, v + at, past_len, n, o + at_q, nl,
                                        nhead, nheads, npast)
            hb.hi_out_proj(s, o, self.w_o, self.Hq, self.D, n, 0, y)
            if offload:
                if self.kv_done[self.turn] is None:
                    self.kv_done[self.turn] = torch.cuda.Event()
                self.kv_done[self.turn].record(ss.s_d2h)
        self.turn ^= 1
        return y
