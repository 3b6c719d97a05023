"""Decode launches that combine their own partials (the workgroup of a head that finishes last does it) against the oracle:
one partition and many, both sides of the limit above which a combine launch follows, several tokens in a row (the
counters go back to zero), heads of different lengths, streaming heads whose store has just filled up, and the same
calls replayed from a graph."""
import numpy as np
import pytest
import torch

from oracle import attention as oa
from paper_2502_12574_amd import binding as hb
from paper_2502_12574_amd import synth
from paper_2502_12574_amd.session import Session

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MAX_ABS, REL_L2 = 1e-2, 5e-3          # the bounds of the parity tests
MAX_PARTS = 16                        # partitions of a head that one workgroup combines


def _check(got, ref, what):
    err, rel = float(np.abs(got - ref).max()), float(np.sqrt(((got - ref) ** 2).sum() / (ref ** 2).sum()))
    assert err <= MAX_ABS and rel <= REL_L2, (what, err, rel)


def _head(seed, h, G, n):
    return ([synth.draw_q(seed, 0, h * G + g, 0, n) for g in range(G)], synth.draw_k(seed, 0, h, 0, n, peaked=True),
            synth.draw_v(seed, 0, h, 0, n))


# heads and lengths such that a head has 1 .. 16 partitions (one launch) and 17 and more (two)
@pytest.mark.parametrize("G,H,past", [(4, 8, 1), (4, 8, 64), (4, 8, 65), (4, 8, 1022), (4, 3, 1100), (4, 17, 5000),
                                      (1, 1, 900), (1, 2, 1023), (8, 1, 2048), (8, 2, 700), (8, 18, 3000), (2, 5, 640)])
def test_tokens_in_a_row(G, H, past):
    seed, nt = 53000, 3
    heads = [_head(seed, h, G, past + nt) for h in range(H)]
    with Session(1, H, G, max(past + nt, 256), 1, mode=hb.HI_MODE_RESIDENT, out_fp32=1) as ss:
        view = ss.cache_view()[:, :, :, :past + nt]
        for h, (_, k, v) in enumerate(heads):
            view[0, h, 0, :past] = k[:past].to(DEV)
            view[0, h, 1, :past] = v[:past].to(DEV)
        out = torch.full((nt, H, G, 128), float("nan"), device=DEV)
        rows = [(torch.stack([torch.stack([q[g][past + t] for g in range(G)]) for q, _, _ in heads]).to(DEV),
                 torch.stack([k[past + t] for _, k, _ in heads]).to(DEV),
                 torch.stack([v[past + t] for _, _, v in heads]).to(DEV)) for t in range(nt)]
        ss.s_compute.wait_stream(torch.cuda.current_stream())
        for t in range(nt):
            ss.decode_group(0, 0, H, *rows[t], past + t, out[t])
        ss.sync()
        # a combine launch follows exactly where a head has more partitions than one workgroup combines
        two = [min(-(-(past + t) // 64), 256 // H) > MAX_PARTS for t in range(nt)]
        assert (ss.stats().n_decode_kernels, ss.stats().n_combine_kernels) == (nt, sum(two))
        for h, (_, k, v) in enumerate(heads):
            assert torch.equal(view[0, h, 0].cpu(), k) and torch.equal(view[0, h, 1].cpu(), v)
    for h, (q, k, v) in enumerate(heads):
        for g in range(G):
            ref = oa.attn_rows(synth.to_f64(q[g][past:]), synth.to_f64(k), synth.to_f64(v), range(past, past + nt))
            _check(out[:, h, g].cpu().double().numpy(), ref, (h, g))


def test_different_lengths_and_replays_from_a_graph():
    """A ragged step and a uniform one, captured once and replayed; eager work and synchronisations in between."""
    seed, G, H, cap = 53100, 4, 6, 2300
    lens = [0, 1, 64, 700, 1999, 2048]
    heads = [_head(seed, h, G, cap) for h in range(H)]
    with Session(1, H, G, cap, 1, mode=hb.HI_MODE_RESIDENT, out_fp32=1) as ss:
        hb.hi_ctx_set_run_ahead(ss.ctx, 0)
        view = ss.cache_view()
        for h, (_, k, v) in enumerate(heads):
            view[0, h, 0], view[0, h, 1] = k.to(DEV), v.to(DEV)
        q = torch.stack([torch.stack([q[g][lens[h]] for g in range(G)]) for h, (q, _, _) in enumerate(heads)]).to(DEV)
        k = torch.stack([k[lens[h]] for h, (_, k, _) in enumerate(heads)]).to(DEV)
        v = torch.stack([v[lens[h]] for h, (_, _, v) in enumerate(heads)]).to(DEV)
        out, uni = torch.zeros(H, G, 128, device=DEV), torch.zeros(H, G, 128, device=DEV)

        def step():
            hb.hi_decode_group_ragged(ss.ctx, 0, 0, H, q, k, v, lens, out)

        torch.cuda.synchronize()
        step()
        ss.sync()
        want = out.clone()
        ref = [oa.attn_rows(synth.to_f64(qs[g][n:n + 1]), synth.to_f64(kk), synth.to_f64(vv), [n])[0]
               for (qs, kk, vv), n in zip(heads, lens) for g in range(G)]
        _check(want.cpu().double().numpy().reshape(-1, 128), np.stack(ref), "eager")
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=ss.s_compute):
            step()
        for _ in range(4):
            out.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
            ss.decode_group(0, 0, H, q, k, v, 2100, uni)
            ss.sync()
            for h in range(H):               # the uniform step replaced row 2100 of every head: no ragged length reaches it
                assert torch.equal(view[0, h, 0, 2100], k[h])


def test_more_contexts_than_counter_slots():
    """Contexts beyond the built-in counters keep the second launch; closed contexts give their counters back."""
    past, G, H = 130, 4, 2
    q, k, v = (torch.randn(s, device=DEV).to(torch.bfloat16) for s in ((H, G, 128), (H, 128), (H, 128)))
    rows = torch.randn(1, H, 2, past, 128, device=DEV).to(torch.bfloat16)
    outs, one_launch = [], []
    for _ in range(2):
        open_ = [Session(1, H, G, 256, 1, mode=hb.HI_MODE_RESIDENT, out_fp32=1) for _ in range(70)]
        for ss in open_:
            ss.cache_view()[:, :, :, :past] = rows
            out = torch.empty(H, G, 128, device=DEV)
            ss.s_compute.wait_stream(torch.cuda.current_stream())
            ss.decode_group(0, 0, H, q, k, v, past, out)
            outs.append(out)
        for ss in open_:
            ss.sync()
        one_launch.append(sum(ss.stats().n_combine_kernels == 0 for ss in open_))
        for ss in open_:
            ss.close()
    assert one_launch == [64, 64]
    for out in outs:                    # three partials, summed in the same order by either way
        assert torch.equal(out, outs[0])


@pytest.mark.parametrize("lens", [[5000, 3, 0, 64, 65, 1290], [70000, 1, 1, 20000], [2000] * 20, [15, 16, 17, 0, 1, 900, 4000, 129]])
def test_partitions_follow_the_lengths(lens):
    """A batch whose lengths are far apart: every head gets partitions in proportion, the shortest ones a single one."""
    G, H, cap, seed = 2, len(lens), max(lens) + 1, 53200
    with Session(1, H, G, cap, 1, mode=hb.HI_MODE_RESIDENT, out_fp32=1) as ss:
        view = ss.cache_view()
        gen = torch.Generator(device=DEV).manual_seed(seed)
        view.copy_(torch.randn(view.shape, device=DEV, generator=gen, dtype=torch.bfloat16))
        q = torch.randn(H, G, 128, device=DEV, generator=gen).to(torch.bfloat16)
        k, v = (torch.randn(H, 128, device=DEV, generator=gen).to(torch.bfloat16) for _ in range(2))
        out = torch.full((H, G, 128), float("nan"), device=DEV)
        ss.s_compute.wait_stream(torch.cuda.current_stream())
        for _ in range(2):
            hb.hi_decode_group_ragged(ss.ctx, 0, 0, H, q, k, v, lens, out)
        ss.sync()
        for h, n in enumerate(lens):
            K, V = synth.to_f64(view[0, h, 0, :n + 1]), synth.to_f64(view[0, h, 1, :n + 1])
            assert np.array_equal(K[n], synth.to_f64(k[h])) and np.array_equal(V[n], synth.to_f64(v[h]))
            ref = oa.attn_rows(synth.to_f64(q[h]), K, V, [n] * G)
            _check(out[h].cpu().double().numpy(), ref, (h, n))


def _integer_rows(H, G, cap, seed):
    """A resident cache of small whole numbers and queries of zeros: every weight is 1 and every sum exact."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rows = torch.randint(-8, 9, (1, H, 2, cap, 128), device=DEV, generator=gen).to(torch.bfloat16)
    return rows, torch.zeros(H, G, 128, dtype=torch.bfloat16, device=DEV)


# 1, 2, 3, 11, 16 partitions of a head (one launch), and 17 (two)
@pytest.mark.parametrize("H,G,past", [(8, 4, 5), (8, 4, 101), (3, 8, 130), (2, 1, 700), (8, 4, 1022), (4, 2, 1030)])
@pytest.mark.parametrize("ragged", [False, True])
def test_quotients_are_rounded_once(H, G, past, ragged):
    """Whole sums over a whole number of rows: the fp32 result is the correctly rounded quotient, by either way."""
    rows, q = _integer_rows(H, G, past + 1, 53300)
    with Session(1, H, G, max(past + 1, 256), 1, mode=hb.HI_MODE_RESIDENT, out_fp32=1) as ss:
        ss.cache_view()[:, :, :, :past] = rows[:, :, :, :past]
        k, v = rows[0, :, 0, past].contiguous(), rows[0, :, 1, past].contiguous()
        out = torch.full((H, G, 128), float("nan"), device=DEV)
        ss.s_compute.wait_stream(torch.cuda.current_stream())
        if ragged:
            hb.hi_decode_group_ragged(ss.ctx, 0, 0, H, q, k, v, [past] * H, out)
        else:
            ss.decode_group(0, 0, H, q, k, v, past, out)
        ss.sync()
        assert ss.stats().n_combine_kernels == (1 if -(-past // 64) > MAX_PARTS else 0)
    # (53 bits are more than 2 * 24 + 2: rounding the double quotient to single is the one correct rounding)
    want = (rows[0, :, 1].double().sum(dim=1) / (past + 1)).float()
    assert torch.equal(out, want[:, None].expand(H, G, 128))


@pytest.mark.parametrize("H,G,past", [(8, 4, 3), (8, 4, 130), (1, 8, 700), (2, 2, 1022), (2, 2, 1030)])
def test_an_infinite_value_stays_infinite(H, G, past):
    """An infinite channel of a visible V row makes that channel infinite and no other, whatever partition holds the row."""
    rows, q = _integer_rows(H, G, past + 1, 53400)
    # the first row of the last 16-row block (the last row itself also stands in for the rows behind the end, with weight 0)
    at = (past - 2) // 16 * 16
    rows[0, :, 1, at, 5] = float("inf")
    rows[0, :, 1, at, 77] = float("-inf")
    with Session(1, H, G, max(past + 1, 256), 1, mode=hb.HI_MODE_RESIDENT, out_fp32=1) as ss:
        ss.cache_view()[:, :, :, :past] = rows[:, :, :, :past]
        k, v = rows[0, :, 0, past].contiguous(), rows[0, :, 1, past].contiguous()
        out = torch.full((H, G, 128), float("nan"), device=DEV)
        ss.s_compute.wait_stream(torch.cuda.current_stream())
        ss.decode_group(0, 0, H, q, k, v, past, out)
        ss.sync()
    want = (rows[0, :, 1].double().sum(dim=1) / (past + 1)).float()
    assert torch.isinf(want).sum() == 2 * H
    assert torch.equal(torch.isinf(out), torch.isinf(want)[:, None].expand(H, G, 128))
    assert (out[:, :, 5] == float("inf")).all() and (out[:, :, 77] == float("-inf")).all() and not torch.isnan(out).any()


def _step_session():
    ss = Session(1, 2, 4, 256, 1, mode=hb.HI_MODE_RESIDENT, out_fp32=1)
    hb.hi_ctx_set_run_ahead(ss.ctx, 0)
    ss.cache_view().zero_()
    q, k, v = (torch.ones(s, dtype=torch.bfloat16, device=DEV) for s in ((2, 4, 128), (2, 128), (2, 128)))
    out = torch.zeros(2, 4, 128, device=DEV)
    ss.s_compute.wait_stream(torch.cuda.current_stream())
    return ss, lambda: ss.decode_group(0, 0, 2, q, k, v, 130, out), out


def test_a_captured_step_holds_no_counters():
    """A graph may be replayed when its context is gone and another one owns the counters: its launches are the two that use
    the caller's buffers only."""
    ss, step, out = _step_session()
    step()
    ss.sync()
    assert ss.stats().n_combine_kernels == 0
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=ss.s_compute):
        step()
    assert ss.stats().n_combine_kernels == 1
    want = out.clone()
    step()
    ss.sync()
    assert ss.stats().n_combine_kernels == 1
    ss.close()
    other, step2, out2 = _step_session()
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        step2()
        torch.cuda.synchronize()
        assert (out - want).abs().max() <= 1e-6 and (out2 - want).abs().max() <= 1e-6
    assert other.stats().n_combine_kernels == 0
    other.close()


@pytest.mark.parametrize("last_unit", ["captured", "failed"])
def test_counters_come_back_whatever_the_last_unit_was(last_unit):
    """More contexts one after the other than there are counter slots; each ends with a captured or a failed unit."""
    for i in range(70):
        ss, step, _ = _step_session()
        step()
        if last_unit == "captured":
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=ss.s_compute):
                step()
        else:
            hb.hi_ctx_set_flags(ss.ctx, hb.HI_FLAG_INJECT_FAILURE)
            with pytest.raises(hb.HiError):
                step()
        ss.close()
    ss, step, _ = _step_session()
    step()
    ss.sync()
    assert ss.stats().n_combine_kernels == 0
    ss.close()


# 1, 2, 3, 11, 16 partitions of a head, every group size, bf16 and fp32 outputs, plain and scaled queries
@pytest.mark.parametrize("H,G,past,fp32,pre", [(8, 4, 5, 1, False), (8, 4, 101, 0, True), (3, 8, 130, 1, True), (2, 1, 700, 1, False),
                                               (8, 4, 1022, 1, True), (16, 2, 1020, 0, False), (4, 4, 1023, 1, False)])
def test_one_launch_and_two_give_the_same_bits(H, G, past, fp32, pre):
    """An eager step combines its partials in the launch, a captured one in a launch of its own."""
    gen = torch.Generator(device=DEV).manual_seed(53500 + past)
    with Session(1, H, G, max(past + 1, 256), 1, mode=hb.HI_MODE_RESIDENT, out_fp32=fp32, q_prescaled=pre) as ss:
        hb.hi_ctx_set_run_ahead(ss.ctx, 0)
        view = ss.cache_view()
        view.copy_(torch.randn(view.shape, device=DEV, generator=gen))
        q = (torch.randn(H, G, 128, device=DEV, generator=gen) * (hb.HI_Q_PRESCALE if pre else 1.0)).to(torch.bfloat16)
        k, v = (torch.randn(H, 128, device=DEV, generator=gen).to(torch.bfloat16) for _ in range(2))
        out = torch.zeros(H, G, 128, dtype=ss.out_dtype, device=DEV)
        torch.cuda.synchronize()
        ss.decode_group(0, 0, H, q, k, v, past, out)
        ss.sync()
        assert ss.stats().n_combine_kernels == 0
        want = out.clone()
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=ss.s_compute):
            ss.decode_group(0, 0, H, q, k, v, past, out)
        assert ss.stats().n_combine_kernels == 1
        for _ in range(3):
            out.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
            assert torch.equal(view[0, :, 0, past], k) and torch.equal(view[0, :, 1, past], v)
