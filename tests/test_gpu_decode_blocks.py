"""The 16-row blocks of the split-KV decode kernel at the edges of its ring: histories that end inside a block, at its end and one
row behind it, with none to five blocks for a wavefront, one launch and two, every group size, against plain torch in 64 bits.

Bound: weights and outputs are rounded to bf16 (weights) and fp32 (outputs); a weight's rounding is 2^-9 of it at most, so is that
of the weighted mean of values around 1: 2^-9 times the mean of |v| with room for the fp32 sums, and far below the 1e-2 asked here."""
import math

import pytest
import torch

from paper_2502_12574_amd import binding as hb
from paper_2502_12574_amd.session import Session

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ROUND = 128 * 16                      # rows of one block for each wavefront of 8 heads' 32 partitions


@pytest.mark.parametrize("G,H,past", [(4, 8, 1), (4, 8, 15), (4, 8, 16), (4, 8, 17), (1, 32, 63), (2, 16, 65), (8, 4, 1023),
                                      (4, 8, ROUND - 1), (4, 8, ROUND), (4, 8, ROUND + 1), (4, 8, 3 * ROUND + 5), (4, 8, 4 * ROUND),
                                      (4, 8, 4 * ROUND + 1), (8, 8, 5 * ROUND - 15), (1, 1, 5000), (2, 3, 7777)])
def test_history_ends(G, H, past):
    gen = torch.Generator(device=DEV).manual_seed(past * 16 + G)
    row = lambda *s: torch.randn(*s, dtype=torch.bfloat16, device=DEV, generator=gen)          # noqa: E731
    kv, q, k, v = row(H, 2, past, 128), row(H, G, 128), row(H, 128), row(H, 128)
    with Session(1, H, G, max(past + 1, 256), 1, mode=hb.HI_MODE_RESIDENT, out_fp32=1) as ss:
        view = ss.cache_view()
        view[0, :, :, :past] = kv
        out = torch.full((H, G, 128), float("nan"), device=DEV)
        ss.s_compute.wait_stream(torch.cuda.current_stream())
        ss.decode_group(0, 0, H, q, k, v, past, out)
        ss.sync()
        assert torch.equal(view[0, :, 0, past], k) and torch.equal(view[0, :, 1, past], v)
    keys, vals = torch.cat([kv[:, 0], k[:, None]], 1).double().cpu(), torch.cat([kv[:, 1], v[:, None]], 1).double().cpu()
    p = torch.softmax(torch.matmul(q.double().cpu(), keys.transpose(1, 2).contiguous()) / math.sqrt(128), -1)
    ref = torch.matmul(p, vals)
    err = (out.double().cpu() - ref).abs().max()
    assert err <= 1e-2 and (out.double().cpu() - ref).norm() <= 5e-3 * ref.norm(), float(err)
