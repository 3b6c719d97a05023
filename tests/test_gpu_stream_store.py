"""A chunk's rows on their way into a streaming head's store along with the chunk's attention, or behind it: every row of the store, bit
for bit, and every output against plain torch in 64 bits, chunk after chunk; twice on one context (the counters go back to zero).

Sizes: sink rows that fill their tiles and that do not, a store smaller and larger than a chunk, few strips that read it, half of
them and all, the first chunk (nobody reads), chunks that end inside a tile, two grid rows a head (G = 8), calls that are timed."""
import math

import pytest
import torch

from paper_2502_12574_amd import binding as hb
from paper_2502_12574_amd.session import Session

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("flags", [0, hb.HI_FLAG_TIME_KERNELS])
@pytest.mark.parametrize("G,H,sink,recent,chunks", [(4, 4, 64, 100, (1000, 900, 1100)), (4, 2, 128, 512, (2048, 2100, 2048)),
                                                    (4, 2, 4, 200, (700, 800)), (8, 2, 0, 130, (600, 1027, 900)),
                                                    (1, 4, 64, 1, (300, 290, 1200)), (2, 3, 192, 300, (100, 60, 700, 1500)),
                                                    (4, 2, 64, 700, (500, 800, 900, 3000))])
def test_store_and_outputs(G, H, sink, recent, chunks, flags):
    S = sum(chunks)
    gen = torch.Generator(device=DEV).manual_seed(S + sink)
    row = lambda *s: torch.randn(*s, dtype=torch.bfloat16, device=DEV, generator=gen)          # noqa: E731
    q, k, v = row(H, G, S, 128), row(H, S, 128), row(H, S, 128)
    pos = torch.arange(S, device=DEV)
    seen = (pos[None] <= pos[:, None]) & ((pos[None] < sink) | (pos[:, None] - pos[None] < recent))
    ref = torch.empty(H, G, S, 128, dtype=torch.float64, device=DEV)
    for h in range(H):
        for g in range(G):
            s = (q[h, g].double() @ k[h].double().t().contiguous()) / math.sqrt(128)
            ref[h, g] = torch.softmax(s.masked_fill(~seen, float("-inf")), -1) @ v[h].double()
    with Session(1, 2 * H, G, S, max(chunks), mode=hb.HI_MODE_RESIDENT, out_fp32=1, streaming_heads=H, sink_tokens=sink,
                 recent_tokens=recent) as ss:
        hb.hi_ctx_set_flags(ss.ctx, flags)
        for _ in range(2):
            ss.staging.zero_()
            torch.cuda.synchronize()
            past = 0
            for n in chunks:
                out = torch.full((H, G, n, 128), float("nan"), device=DEV)
                e = past + n
                ss.prefill_group(0, H, H, q[:, :, past:e].contiguous(), k[:, past:e].contiguous(), v[:, past:e].contiguous(), past, out)
                ss.sync()
                assert (out - ref[:, :, past:e]).abs().max() <= 1e-2 and (out - ref[:, :, past:e]).norm() <= 5e-3 * ref[:, :, past:e].norm(), past
                tokens = [j for j in range(e) if j < sink or j >= e - recent]
                at = torch.tensor([j if j < sink else sink + (j - sink) % recent for j in tokens], device=DEV)
                tokens = torch.tensor(tokens, device=DEV)
                store = ss.stream_view().view(H, 2, sink + recent, 128)
                assert torch.equal(store[:, 0, at], k[:, tokens]) and torch.equal(store[:, 1, at], v[:, tokens]), past
                past = e
