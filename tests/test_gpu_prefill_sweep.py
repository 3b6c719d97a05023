"""prefill_kernel_deep16 where its sweep can go wrong: passes of one tile and more on either side of the four that take their
maxima first, partial tiles at the end of the past and of the chunk, blocks of 16 query rows that the chunk leaves empty (in the
last block of positions, across launches too), and ranges of own tiles whose first tile some rows do not see at all."""
import pytest

from oracle import attention as oa
from paper_2502_12574_amd import binding as hb
from paper_2502_12574_amd import synth
from test_gpu_parity_small import check, one_unit

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [0, 1, 64, 129, 256, 300, 321])
@pytest.mark.parametrize("G,C", [(4, 16), (4, 17), (4, 33), (4, 64), (4, 77), (4, 97), (1, 5), (1, 44), (1, 256), (1, 300), (2, 145), (8, 50)])
@pytest.mark.parametrize("mode", [hb.HI_MODE_RESIDENT, hb.HI_MODE_OFFLOAD])
@pytest.mark.parametrize("paired", [False, True])
def test_short_sweeps_and_empty_blocks(G, C, P, mode, paired):
    flags = hb.HI_FLAG_PREFILL_DEEP | (hb.HI_FLAG_PREFILL_PAIRED if paired else 0)
    out, Q, K, V = one_unit(G, P, C, seed=61000 + P + C, mode=mode, flags=flags, peaked=P == 300)
    ref = oa.attn_head(synth.to_f64(Q), synth.to_f64(K), synth.to_f64(V), past_len=P)
    for g in range(G):
        check(out[g:g + 1], ref[g:g + 1], f"G={G} P={P} C={C} head {g}")
