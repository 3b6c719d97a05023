"""prefill_kernel_deep16 where its sweep can go wrong: passes of one tile and more, on either side of the twelve full ones from which
some do not take their maxima, partial tiles at the end of the past and of the chunk, blocks of 16 query rows that the chunk leaves empty (in the
last block of positions, across launches too), and ranges of own tiles whose first tile some rows do not see at all."""
import pytest
import torch

from oracle import attention as oa
from paper_2502_12574_amd import binding as hb
from paper_2502_12574_amd import synth
from paper_2502_12574_amd.session import Session
from test_gpu_parity_small import check, one_unit

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [0, 1, 64, 129, 256, 300, 321, 700, 767, 768, 1100])
@pytest.mark.parametrize("G,C", [(4, 16), (4, 17), (4, 33), (4, 64), (4, 77), (4, 97), (1, 5), (1, 44), (1, 256), (1, 300), (2, 145), (8, 50)])
@pytest.mark.parametrize("mode", [hb.HI_MODE_RESIDENT, hb.HI_MODE_OFFLOAD])
@pytest.mark.parametrize("paired", [False, True])
def test_short_sweeps_and_empty_blocks(G, C, P, mode, paired):
    flags = hb.HI_FLAG_PREFILL_DEEP | (hb.HI_FLAG_PREFILL_PAIRED if paired else 0)
    out, Q, K, V = one_unit(G, P, C, seed=61000 + P + C, mode=mode, flags=flags, peaked=P == 300)
    ref = oa.attn_head(synth.to_f64(Q), synth.to_f64(K), synth.to_f64(V), past_len=P)
    for g in range(G):
        check(out[g:g + 1], ref[g:g + 1], f"G={G} P={P} C={C} head {g}")


# units with a merge launch, which takes the append along: of the 8-wave kernel (few blocks, many; two grid rows a head) and of
# the 4-wave kernel's ranges
MERGED = [(1, 17, 1, 16, 3000, 150), (4, 8, 0, 8, 3001, 77), (8, 9, 2, 7, 1500, 130), (4, 3, 1, 1, 4000, 33), (1, 2, 0, 2, 2500, 1)]
# and without one, where the append is a launch of its own
ALONE = [(4, 8, 0, 8, 64, 1000), (1, 5, 2, 3, 100, 40)]


def _rows_land(G, H, first, nh, past, C, flags=0):
    dev = "cuda:0"
    gen = torch.Generator(device=dev).manual_seed(61500 + past)
    with Session(1, H, G, past + C + 200, C, mode=hb.HI_MODE_RESIDENT, out_fp32=1) as ss:
        hb.hi_ctx_set_flags(ss.ctx, flags)
        view = ss.cache_view()
        view.copy_(torch.randn(view.shape, device=dev, generator=gen).to(torch.bfloat16))
        k, v = (torch.randn(nh, C, 128, device=dev, generator=gen).to(torch.bfloat16) for _ in range(2))
        q = torch.randn(nh, G, C, 128, device=dev, generator=gen).to(torch.bfloat16)
        out = torch.full((nh, G, C, 128), float("nan"), device=dev)
        want = view.clone()
        want[0, first:first + nh, 0, past:past + C], want[0, first:first + nh, 1, past:past + C] = k, v
        ss.s_compute.wait_stream(torch.cuda.current_stream())
        ss.prefill_group(0, first, nh, q, k, v, past, out)
        ss.sync()
        assert torch.equal(view, want)
        rows = want[0, first:first + nh, :, :past + C].cpu()
    for h in range(nh):
        ref = oa.attn_head(synth.to_f64(q[h].cpu()), synth.to_f64(rows[h, 0]), synth.to_f64(rows[h, 1]), past_len=past)
        check(out[h], ref, f"head {h}")


@pytest.mark.parametrize("G,H,first,nh,past,C", MERGED)
def test_rows_land_in_place_along_with_a_merge(G, H, first, nh, past, C):
    _rows_land(G, H, first, nh, past, C)


@pytest.mark.parametrize("G,H,first,nh,past,C", ALONE)
def test_rows_land_in_place_without_a_merge(G, H, first, nh, past, C):
    _rows_land(G, H, first, nh, past, C)


@pytest.mark.parametrize("G,H,first,nh,past,C", MERGED[:2])
def test_rows_land_in_place_where_launches_are_timed(G, H, first, nh, past, C):
    _rows_land(G, H, first, nh, past, C, hb.HI_FLAG_TIME_KERNELS)


# ranges of the 8-wave kernel (2, 3, 5, 16 and more images of a block: below, at and beyond what the merge has in flight), its other
# forms, and the 4-wave kernel's ranges
@pytest.mark.parametrize("G,H,past,C,flags", [(4, 8, 3001, 600, 0), (4, 8, 3001, 77, 0), (4, 8, 20003, 77, 0), (1, 16, 5000, 150, 0),
                                              (4, 1, 4000, 300, hb.HI_FLAG_PREFILL_DEEP), (8, 2, 1500, 130, hb.HI_FLAG_PREFILL_DEEP),
                                              (4, 2, 3001, 300, hb.HI_FLAG_PREFILL_DEEP | hb.HI_FLAG_PREFILL_PAIRED),
                                              (4, 2, 3001, 300, hb.HI_FLAG_PREFILL_DEEP | hb.HI_FLAG_PREFILL_MFMA32),
                                              (4, 2, 3001, 300, hb.HI_FLAG_PREFILL_DEEP | hb.HI_FLAG_PREFILL_WIDE), (4, 1, 4000, 33, 0)])
@pytest.mark.parametrize("mode", [hb.HI_MODE_RESIDENT, hb.HI_MODE_OFFLOAD])
def test_an_infinite_value_stays_infinite(G, H, past, C, flags, mode):
    """An infinite channel of a cached V row makes that channel infinite and no other, whatever range of tiles holds the row."""
    dev = "cuda:0"
    gen = torch.Generator(device=dev).manual_seed(62000 + past + C)
    rows = torch.randint(-8, 9, (H, 2, past + C, 128), device=dev, generator=gen).to(torch.bfloat16)
    q = torch.zeros(H, G, C, 128, dtype=torch.bfloat16, device=dev)
    ats = [0, past // 3, past // 2, past - 70, past - 2]         # (the last row stands in for rows behind the end, with weight 0)
    want = rows[:, 1].double().cumsum(dim=1)[:, past:] / torch.arange(past + 1, past + C + 1, device=dev)[None, :, None]
    with Session(1, H, G, past + C, C, mode=mode, out_fp32=1) as ss:
        hb.hi_ctx_set_flags(ss.ctx, flags)
        view = ss.cache_view()
        k, v = (rows[:, w, past:].contiguous() for w in (0, 1))
        for at in ats:
            cached = rows[:, :, :past].clone()
            cached[:, 1, at, 5], cached[:, 1, at, 77] = float("inf"), float("-inf")
            view[0, :, :, :past] = cached.to(view.device)
            out = torch.full((H, G, C, 128), float("nan"), device=dev)
            torch.cuda.synchronize()
            ss.prefill_group(0, 0, H, q, k, v, past, out)
            ss.sync()
            assert (out[..., 5] == float("inf")).all() and (out[..., 77] == float("-inf")).all(), at
            out[..., 5], out[..., 77] = want[:, None, :, 5].float(), want[:, None, :, 77].float()
            # whole sums in fp32, one quotient: two roundings of numbers up to 8
            assert (out - want[:, None]).abs().max() <= 1e-5, at


@pytest.mark.parametrize("past", [512, 576, 640, 704])
def test_short_sweeps_take_every_maximum(past):
    """A pass of fewer than twelve full cached tiles takes the maximum of each tile: the key that has it weighs exactly 1, wherever
    it is, and the result is good to fp32 - where weights against an older maximum are rounded to bf16, 1.9256 by 0.0037."""
    dev, G, H, C, d = "cuda:0", 4, 192, 64, 121 / 128
    gen = torch.Generator(device=dev).manual_seed(62100 + past)
    tiles = past // 64
    with Session(1, H, G, past + C, C, mode=hb.HI_MODE_RESIDENT, out_fp32=1, q_prescaled=1) as ss:
        hb.hi_ctx_set_flags(ss.ctx, hb.HI_FLAG_PREFILL_DEEP)
        view = ss.cache_view()
        view.copy_(torch.randn(view.shape, device=dev, generator=gen))
        view[0, :, 0] = 0
        view[0, :, 0, :, 0] = -64.0                     # score of all others: weight 2^-64
        view[0, :, 0, :4, 0] = 0.0                      # four rows of one lane in the first tile
        at = 64 * (torch.arange(H, device=dev) % (tiles - 1) + 1)
        heads = torch.arange(H, device=dev)
        view[0, heads, 0, at, 0] = d                    # and one in a later tile, the same lane's
        q = torch.zeros(H, G, C, 128, dtype=torch.bfloat16, device=dev)
        q[..., 0] = 1.0
        k = torch.zeros(H, C, 128, dtype=torch.bfloat16, device=dev)
        k[..., 0] = -64.0
        v = torch.randn(H, C, 128, device=dev, generator=gen).to(torch.bfloat16)
        out = torch.full((H, G, C, 128), float("nan"), device=dev)
        V = view[0, :, 1].double()
        want = (V[:, :4].sum(dim=1) + 2.0 ** d * V[heads, at]) / (4 + 2.0 ** d)
        torch.cuda.synchronize()
        ss.prefill_group(0, 0, H, q, k, v, past, out)
        ss.sync()
        # sums of five fp32 products and one exponential, of values up to 6: some roundings of 2^-24 each
        assert (out - want[:, None, None]).abs().max() <= 1e-5


def test_long_sweeps_over_blocks_in_part_take_the_wide_form():
    """1300 rows of 32 one-query heads behind 60 thousand, five full blocks of 256 positions and a rest, 957 tiles a workgroup: the
    bits of the form that launches of 640 tiles and more run, and not those of the other one."""
    dev, H, past, C = "cuda:0", 32, 60000, 1300
    gen = torch.Generator(device=dev).manual_seed(62200)
    with Session(1, H, 1, past + C, C, mode=hb.HI_MODE_RESIDENT, out_fp32=1, q_prescaled=1) as ss:
        view = ss.cache_view()
        for h in range(H):
            view[0, h] = torch.randn(view.shape[2:], device=dev, generator=gen).to(torch.bfloat16)
        q = (torch.randn(H, 1, C, 128, device=dev, generator=gen) * hb.HI_Q_PRESCALE).to(torch.bfloat16)
        k, v = (torch.randn(H, C, 128, device=dev, generator=gen).to(torch.bfloat16) for _ in range(2))
        outs = []
        for flags in (0, hb.HI_FLAG_PREFILL_WIDE, hb.HI_FLAG_PREFILL_8WAVE):
            hb.hi_ctx_set_flags(ss.ctx, flags)
            outs.append(torch.full((H, 1, C, 128), float("nan"), device=dev))
            torch.cuda.synchronize()
            ss.prefill_group(0, 0, H, q, k, v, past, outs[-1])
            ss.sync()
    assert torch.equal(outs[0], outs[1]) and not torch.equal(outs[0], outs[2]) and torch.isfinite(outs[2]).all()
