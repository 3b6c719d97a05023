"""prefill_kernel (4 wavefronts) where its pipelined sweep can go wrong: sweeps of one visit, two and three (the scores run one visit
ahead, K tiles two), a past that ends inside a tile, on its edge and one row behind it, wavefronts without a position, ranges of tiles
that end before the chunk's own rows or start inside them (short chunks), state carried from launch to launch and slices in two pieces
(offloaded)."""
import pytest

from oracle import attention as oa
from paper_2502_12574_amd import binding as hb
from paper_2502_12574_amd import synth
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
