"""prefill_kernel (4 wavefronts) where its pipelined sweep can go wrong: sweeps of one visit, two and three (the scores run one visit
ahead, K tiles two), a past that ends inside a tile, on its edge and one row behind it, wavefronts without a position, ranges of tiles
that end before the chunk's own rows or start inside them (short chunks), state carried from launch to launch and slices in two pieces
(offloaded)."""
import pytest
import torch

from oracle import attention as oa
from paper_2502_12574_amd import binding as hb
from paper_2502_12574_amd import synth
from paper_2502_12574_amd.session import Session
from test_gpu_parity_small import check, one_unit

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [0, 1, 63, 64, 65, 128, 191, 700, 3000, 3009])
@pytest.mark.parametrize("G,C,flags", [(4, 1, 0), (4, 33, 0), (8, 50, 0), (1, 100, 0), (4, 64, hb.HI_FLAG_PREFILL_NARROW),
                                       (2, 65, hb.HI_FLAG_PREFILL_NARROW), (1, 300, hb.HI_FLAG_PREFILL_NARROW),
                                       (4, 200, hb.HI_FLAG_PREFILL_NARROW)])
@pytest.mark.parametrize("mode", [hb.HI_MODE_RESIDENT, hb.HI_MODE_OFFLOAD])
def test_pipelined_sweeps(G, C, flags, P, mode):
    out, Q, K, V = one_unit(G, P, C, seed=63000 + P + C, mode=mode, flags=flags, peaked=P == 700)
    ref = oa.attn_head(synth.to_f64(Q), synth.to_f64(K), synth.to_f64(V), past_len=P)
    for g in range(G):
        check(out[g:g + 1], ref[g:g + 1], f"G={G} P={P} C={C} head {g}")


# Cut units of more workgroups than compute units are swept straight, smaller ones a visit ahead: the heads of a call together (more than
# 256 workgroups) and one by one are the same bits, and both are right.  Ranges of odd and even length, past rows that end on
# a tile's edge and inside it, blocks that end inside the chunk's last tile, two grid rows a head.
@pytest.mark.parametrize("H,G,P,C,mode", [(8, 4, 50000, 30, hb.HI_MODE_RESIDENT), (8, 4, 50000, 30, hb.HI_MODE_OFFLOAD),
                                          (2, 4, 13013, 378, hb.HI_MODE_RESIDENT), (4, 8, 30016, 33, hb.HI_MODE_RESIDENT),
                                          (4, 8, 30016, 33, hb.HI_MODE_OFFLOAD), (1, 2, 10532, 1756, hb.HI_MODE_RESIDENT)])
def test_straight_and_pipelined_sweeps_give_the_same_bits(H, G, P, C, mode):
    gen = torch.Generator(device="cuda:0").manual_seed(P + C)
    row = lambda *s: torch.randn(*s, dtype=torch.bfloat16, device="cuda:0", generator=gen)          # noqa: E731
    q, k, v, kv = row(H, G, C, 128), row(H, C, 128), row(H, C, 128), row(H, 2, P, 128)
    with Session(1, H, G, P + C, C, mode=mode, out_fp32=1) as ss:
        view = ss.cache_view()
        view[0, :, :, :P] = kv.to(view.device)
        outs = []
        for nh in (H, 1):
            out = torch.full((H, G, C, 128), float("nan"), device="cuda:0")
            torch.cuda.synchronize()
            for h in range(0, H, nh):
                ss.prefill_group(0, h, nh, q[h:h + nh], k[h:h + nh], v[h:h + nh], P, out[h:h + nh])
            ss.sync()
            outs.append(out)
        assert torch.equal(*outs)
    hidden = torch.arange(P + C, device="cuda:0")[None] > P + torch.arange(C, device="cuda:0")[:, None]
    for h in range(0, H, 7):
        keys = torch.cat([kv[h, 0], k[h]]).double().t().contiguous()
        s = ((q[h].double().view(G * C, 128) @ keys) / 128 ** 0.5).view(G, C, -1)
        p = torch.softmax(s.masked_fill(hidden, float("-inf")), -1)
        ref = (p.view(G * C, -1) @ torch.cat([kv[h, 1], v[h]]).double()).view(G, C, 128)
        assert (outs[0][h] - ref).abs().max() <= 1e-2 and (outs[0][h] - ref).norm() <= 5e-3 * ref.norm(), h
