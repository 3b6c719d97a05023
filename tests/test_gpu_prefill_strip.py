"""Chunks that leave their last block of positions part empty: every row against plain torch in 64 bits, and how far rows reach.

Bound: weights and outputs rounded to bf16 and fp32 like in every other form of the kernel - the parity bounds of the suite."""
import math

import pytest
import torch

from paper_2502_12574_amd import binding as hb
from paper_2502_12574_amd.session import Session

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# last rows on either side of a multiple of 16, one to three launches, every group size
@pytest.mark.parametrize("G,H,past,C,flags", [(4, 8, 3000, 77, 0), (4, 8, 3000, 96, 0), (4, 8, 700, 97, hb.HI_FLAG_PREFILL_DEEP),
                                              (4, 8, 3001, 140, 0), (4, 4, 0, 130, hb.HI_FLAG_PREFILL_DEEP), (1, 32, 3000, 300, 0),
                                              (2, 16, 3000, 150, 0), (8, 4, 1000, 77, hb.HI_FLAG_PREFILL_DEEP),
                                              (4, 2, 2000, 193, hb.HI_FLAG_PREFILL_DEEP | hb.HI_FLAG_PREFILL_PAIRED)])
@pytest.mark.parametrize("mode", [hb.HI_MODE_RESIDENT, hb.HI_MODE_OFFLOAD])
def test_rows(G, H, past, C, flags, mode):
    gen = torch.Generator(device=DEV).manual_seed(past + C)
    row = lambda *s: torch.randn(*s, dtype=torch.bfloat16, device=DEV, generator=gen)          # noqa: E731
    kv, q, k, v = row(H, 2, past, 128), row(H, G, C, 128), row(H, C, 128), row(H, C, 128)
    with Session(1, H, G, max(past + C, 256), C, mode=mode, out_fp32=1) as ss:
        hb.hi_ctx_set_flags(ss.ctx, flags)
        ss.cache_view()[0, :, :, :past] = kv.to(ss.cache_view().device)
        out = torch.full((H, G, C, 128), float("nan"), device=DEV)
        torch.cuda.synchronize()
        step = H if mode == hb.HI_MODE_RESIDENT else min(H, max(1, (past + C) // 512))
        for h in range(0, H, step):
            n = min(step, H - h)
            ss.prefill_group(0, h, n, q[h:h + n], k[h:h + n], v[h:h + n], past, out[h:h + n])
        ss.sync()
    keys, vals = torch.cat([kv[:, 0], k], 1).double(), torch.cat([kv[:, 1], v], 1).double()
    hidden = torch.arange(past + C, device=DEV)[None] > torch.arange(past, past + C, device=DEV)[:, None]
    for h in range(H):
        s = (q[h].reshape(-1, 128).double() @ keys[h].t().contiguous()).view(G, C, -1) / math.sqrt(128)
        p = torch.softmax(s.masked_fill(hidden, float("-inf")), -1)
        ref = (p.view(G * C, -1) @ vals[h]).view(G, C, 128)
        assert (out[h] - ref).abs().max() <= 1e-2 and (out[h] - ref).norm() <= 5e-3 * ref.norm(), h


# A query's tiles go on to the end of its block of positions - 64 with four query heads and more, 128 with two, 256 with one - and a
# hidden row there has weight zero, which makes NaN of an infinite value.  Rows of blocks behind it are not read at all: whatever they
# hold, the rows in front of them are the same bits.
@pytest.mark.parametrize("G,H,past,C,flags", [(4, 8, 3000, 77, 0), (4, 8, 100003, 77, 0), (8, 4, 1000, 77, hb.HI_FLAG_PREFILL_DEEP),
                                              (4, 8, 3001, 140, 0), (1, 32, 3000, 300, 0), (2, 16, 3000, 150, 0), (4, 1, 700, 333, 0),
                                              (4, 2, 2000, 193, hb.HI_FLAG_PREFILL_DEEP | hb.HI_FLAG_PREFILL_PAIRED)])
def test_later_blocks_are_not_read(G, H, past, C, flags):
    gen = torch.Generator(device=DEV).manual_seed(C)
    row = lambda *s: torch.randn(*s, dtype=torch.bfloat16, device=DEV, generator=gen)          # noqa: E731
    kv, q, k, v = row(H, 2, past, 128), row(H, G, C, 128), row(H, C, 128), row(H, C, 128)
    block = 256 // min(G, 4)
    with Session(1, H, G, past + C, C, mode=hb.HI_MODE_RESIDENT, out_fp32=1) as ss:
        hb.hi_ctx_set_flags(ss.ctx, flags)
        ss.cache_view()[0, :, :, :past] = kv.to(ss.cache_view().device)

        def pass_over(k, v):
            out = torch.empty(H, G, C, 128, device=DEV)
            torch.cuda.synchronize()
            ss.prefill_group(0, 0, H, q, k, v, past, out)
            ss.sync()
            return out

        good = pass_over(k, v)
        for first in range(block, C, block):
            for x in (float("inf"), float("nan")):
                k2, v2 = k.clone(), v.clone()
                k2[:, first:], v2[:, first:] = x, x
                bad = pass_over(k2, v2)
                same = torch.equal(bad[:, :, :first], good[:, :, :first])
                assert same, (first, x)
                assert not torch.isfinite(bad[:, :, first:]).any(), (first, x)
