"""Units of few query rows (the 4-wave prefill kernel): the same bits whether the cached rows come from HBM in one launch or
through the staging ring slice by slice, and whether the heads of a layer are called one by one or together - at 2048 rows
in all, beyond them, and where a staging slice ends inside a range of tiles that one workgroup sweeps."""
import pytest
import torch

from paper_2502_12574_amd import binding as hb
from paper_2502_12574_amd.session import Session

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _run(mode, G, H, nh, past, C, seed, budget, flags=0):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rows = torch.randn(H, 2, past + C, 128, device=DEV, generator=gen).to(torch.bfloat16)
    rows[:, 0][torch.rand(H, past + C, device=DEV, generator=gen) < 0.05] *= 4
    q = torch.randn(H, G, C, 128, device=DEV, generator=gen).to(torch.bfloat16)
    out = torch.full((H, G, C, 128), float("nan"), device=DEV)
    with Session(1, H, G, past + C, C, mode=mode, out_fp32=1, gpu_kv_budget_heads=budget) as ss:
        hb.hi_ctx_set_flags(ss.ctx, flags)
        ss.cache_view()[0, :, :, :past] = rows[:, :, :past].to(ss.cache_view().device)
        torch.cuda.synchronize()
        k, v = rows[:, 0, past:].contiguous(), rows[:, 1, past:].contiguous()
        ss.s_compute.wait_stream(torch.cuda.current_stream())
        for h in range(0, H, nh):
            ss.prefill_group(0, h, nh, q[h:h + nh], k[h:h + nh], v[h:h + nh], past, out[h:h + nh])
        ss.sync()
        slices = -(-past // (ss.plan.slice_tokens // nh // 64 * 64))
    return out, (q, rows), slices


# (G, heads, heads per call, past, chunk, budget in heads): the last is a ring of larger slices
CASES = [(4, 1, 1, 1536, 512, 1), (4, 1, 1, 2048, 512, 1), (4, 1, 1, 2049, 77, 1), (4, 2, 2, 9001, 64, 1), (4, 8, 4, 20000, 30, 1),
         (4, 3, 1, 12345, 300, 1), (1, 2, 1, 3000, 77, 1), (2, 2, 2, 5000, 33, 2), (8, 1, 1, 7777, 100, 1), (8, 2, 2, 4100, 1, 1),
         (4, 1, 1, 30000, 960, 1), (4, 8, 8, 60000, 17, 2)]


@pytest.mark.parametrize("G,H,nh,past,C,budget", CASES)
def test_same_bits_in_both_modes_and_any_grouping(G, H, nh, past, C, budget):
    seed = 61000 + past
    a, (q, rows), _ = _run(hb.HI_MODE_RESIDENT, G, H, nh, past, C, seed, budget)
    b, _, slices = _run(hb.HI_MODE_OFFLOAD, G, H, nh, past, C, seed, budget)
    assert slices > 1 and torch.equal(a, b)
    c, _, _ = _run(hb.HI_MODE_OFFLOAD, G, H, nh, past, C, seed, budget, hb.HI_FLAG_PREFILL_SINGLE_SLICES)
    assert torch.equal(a, c)                # (by default two short slices go into one launch)
    one, _, _ = _run(hb.HI_MODE_RESIDENT, G, H, 1, past, C, seed, budget)
    assert torch.equal(a, one)
    # and the right ones: fp64 on the same rows, the parity tests' bounds
    pos = torch.arange(past, past + C, device=DEV)
    for h in range(H):
        k, v = rows[h, 0].double(), rows[h, 1].double()
        s = (q[h].double().view(G * C, 128) @ k.t().contiguous()).view(G, C, -1) / 128 ** 0.5
        s.masked_fill_(torch.arange(past + C, device=DEV)[None] > pos[:, None], float("-inf"))
        ref = (torch.softmax(s, dim=-1).view(G * C, -1) @ v).view(G, C, 128)
        err, rel = float((a[h] - ref).abs().max()), float((a[h] - ref).norm() / ref.norm())
        assert err <= 1e-2 and rel <= 5e-3, (h, err, rel)
