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


def _rows(seed, H, G, S):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    return tuple(torch.randn(*s, dtype=torch.bfloat16, device=DEV, generator=gen) for s in ((H, G, S, 128), (H, S, 128), (H, S, 128)))


# a chunk whose rows would ride with a counter (its first strips read the store), one without readers, one that reads everywhere
@pytest.mark.parametrize("sink,recent,past,C", [(128, 200, 2048, 2100), (128, 512, 0, 900), (4, 200, 700, 800)])
def test_captured_chunk(sink, recent, past, C):
    """A captured chunk holds no counters: replayed from a graph, with eager chunks of another context in between, it leaves the same store
    and the same outputs, bit for bit, as the eager call."""
    G, H = 4, 2
    q, k, v = _rows(past + C, H, G, past + C)
    make = lambda: Session(1, 2 * H, G, past + C, max(past, C), mode=hb.HI_MODE_RESIDENT, out_fp32=1, streaming_heads=H,  # noqa: E731
                           sink_tokens=sink, recent_tokens=recent)
    part = lambda a, b: (q[:, :, a:b].contiguous(), k[:, a:b].contiguous(), v[:, a:b].contiguous())                      # noqa: E731
    with make() as ss, make() as other:
        out, out2 = (torch.full((H, G, C, 128), float("nan"), device=DEV) for _ in range(2))
        head, tail = part(0, past), part(past, past + C)
        torch.cuda.synchronize()

        def begin(ctx):
            ctx.staging.zero_()
            torch.cuda.synchronize()
            if past:
                ctx.prefill_group(0, H, H, *head, 0, torch.empty(H, G, past, 128, device=DEV))
            ctx.sync()

        hb.hi_ctx_set_run_ahead(ss.ctx, 0)
        begin(ss)
        ss.prefill_group(0, H, H, *tail, past, out)
        ss.sync()
        want, store = out.clone(), ss.stream_view().clone()
        assert torch.isfinite(want).all()
        begin(ss)
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=ss.s_compute):
            ss.prefill_group(0, H, H, *tail, past, out)
        for _ in range(3):
            begin(ss)
            begin(other)
            out.zero_()
            torch.cuda.synchronize()
            graph.replay()
            other.prefill_group(0, H, H, *tail, past, out2)      # (on its own stream and counters)
            torch.cuda.synchronize()
            assert torch.equal(out, want) and torch.equal(ss.stream_view(), store)
            assert torch.equal(out2, want) and torch.equal(other.stream_view(), store)


def test_contexts_without_counters():
    """More contexts than there are counters: those that got none write the chunk's rows in a launch of their own - the same rows, the
    same outputs, whoever has one."""
    G, H, sink, recent, past, C = 4, 1, 64, 100, 700, 900
    q, k, v = _rows(7, H, G, past + C)
    part = lambda a, b: (q[:, :, a:b].contiguous(), k[:, a:b].contiguous(), v[:, a:b].contiguous())                      # noqa: E731
    one_launch, first = [], None
    open_ = [Session(1, 2, G, past + C, C, mode=hb.HI_MODE_RESIDENT, out_fp32=1, streaming_heads=H, sink_tokens=sink, recent_tokens=recent)
             for _ in range(68)]
    for ss in open_:
        out = torch.full((H, G, C, 128), float("nan"), device=DEV)
        ss.staging.zero_()
        ss.cache_view()[:] = 0
        torch.cuda.synchronize()
        for a, b, o in ((0, past, torch.empty(H, G, past, 128, device=DEV)), (past, past + C, out)):
            ss.prefill_group(0, 1, H, *part(a, b), a, o)
            ss.sync()
        # whether this one has counters: a token over a short resident history takes one launch with them, two without
        ss.decode_group(0, 0, 1, q[:, :, 0].contiguous(), k[:, 0].contiguous(), v[:, 0].contiguous(), 130, torch.empty(1, G, 128, device=DEV))
        ss.sync()
        one_launch.append(ss.stats().n_combine_kernels == 0)
        got = (out, ss.stream_view().clone())
        first = first or got
        assert torch.isfinite(out).all() and torch.equal(got[0], first[0]) and torch.equal(got[1], first[1])
    for ss in open_:
        ss.close()
    assert one_launch == [True] * 64 + [False] * 4
