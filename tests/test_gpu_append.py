"""Rows of HBM-resident heads entering the cache: exactly the chunk's rows, at their places, nothing beside them, from one
row to several workgroups' worth, one head and a group, at odd positions."""
import pytest
import torch

from paper_2502_12574_amd import binding as hb
from paper_2502_12574_amd.session import Session

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("H,first,nh,past,C", [(1, 0, 1, 0, 1), (3, 1, 2, 7, 63), (3, 0, 3, 200, 64), (4, 2, 1, 131, 65), (2, 0, 2, 1, 1000)])
def test_rows_land_in_place(H, first, nh, past, C):
    with Session(1, H, 1, past + C + 300, C, mode=hb.HI_MODE_RESIDENT, out_fp32=1) as ss:
        view = ss.cache_view()
        view.fill_(3.0)
        k, v = (torch.randn(nh, C, 128, device=DEV).to(torch.bfloat16) for _ in range(2))
        q = torch.randn(nh, 1, C, 128, device=DEV).to(torch.bfloat16)
        out = torch.empty(nh, 1, C, 128, device=DEV)
        want = view.clone()
        want[0, first:first + nh, 0, past:past + C], want[0, first:first + nh, 1, past:past + C] = k, v
        ss.s_compute.wait_stream(torch.cuda.current_stream())
        ss.prefill_group(0, first, nh, q, k, v, past, out)
        ss.sync()
        assert torch.equal(view, want)
