"""The rotation that the 128-row projection tile forms for itself: tokens on either side of a wavefront's share (32) and of a tile (128),
contractions of four steps and more, positions up to a million, no rotation at all, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import projection as op
from paper_2502_12574_amd import binding as hb
from paper_2502_12574_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("D,Hq,Hkv", [(256, 2, 1), (640, 1, 1)])
@pytest.mark.parametrize("C,past,theta", [(65, 0, 500000.0), (95, 1048000, 500000.0), (128, 999983, 10000.0), (129, 7, 500000.0),
                                          (161, 131072, 500000.0), (130, 5000, 0.0)])
def test_rotation(D, Hq, Hkv, C, past, theta):
    seed = 9900 + D + C
    X = synth.draw_hidden(seed, 0, past, C, D, device=DEV)
    W = synth.draw_weight(seed, synth.TENSOR_WQKV, 0, (Hq + 2 * Hkv) * 128, D, device=DEV)
    q = torch.full((Hq, C, 128), float("nan"), dtype=torch.bfloat16, device=DEV)
    k, v = (torch.full((Hkv, C, 128), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    ws = torch.empty(hb.hi_proj_workspace_bytes(C), dtype=torch.uint8, device=DEV)
    hb.hi_qkv_rope(torch.cuda.current_stream(), X, W, D, Hq, Hkv, C, past, theta, 0, q, k, v, ws, q_scale=0.5)
    Wf = synth.to_f64(W.cpu())
    Q, K, V = op.qkv_rope(synth.to_f64(X.cpu()), Wf[:Hq * 128], Wf[Hq * 128:(Hq + Hkv) * 128], Wf[(Hq + Hkv) * 128:],
                          np.arange(past, past + C), 128, theta or None)      # (0: no rotation)
    for got, ref, name in ((q, 0.5 * Q, "Q"), (k, K, "K"), (v, V, "V")):
        got = got.double().cpu().numpy()
        rel = float(np.sqrt(((got - ref) ** 2).sum() / (ref ** 2).sum()))
        # one rounding to bf16 (2^-9 at most, 1.7e-3 in the mean square) on fp32 sums
        assert rel <= 2.0e-3 and float((np.abs(got - ref) / (np.abs(ref) + 1.0)).max()) <= 2.0 ** -8 + 1e-5, (name, rel)


# The 256-row tile (fp32 output) reads its rotation from a table, the 128-row tile (bf16) forms its own: the same angles, so that bf16 output
# is the fp32 output rounded, to the bit.  A last bit of the angle shows in one of a million outputs, at long positions.
@pytest.mark.parametrize("past", [131072, 4000000, 100000000])
def test_bf16_output_is_fp32_output_rounded(past):
    D, Hq, Hkv, C = 256, 126, 1, 128
    gen = torch.Generator(device=DEV).manual_seed(past)
    ws = torch.empty(hb.hi_proj_workspace_bytes(C), dtype=torch.uint8, device=DEV)
    for r in range(16):
        x = torch.randn(C, D, device=DEV, generator=gen).to(torch.bfloat16)
        w = (torch.randn((Hq + 2 * Hkv) * 128, D, device=DEV, generator=gen) / 16).to(torch.bfloat16)
        out = []
        for dtype in (torch.bfloat16, torch.float32):
            q, k, v = (torch.empty(h, C, 128, dtype=dtype, device=DEV) for h in (Hq, Hkv, Hkv))
            hb.hi_qkv_rope(torch.cuda.current_stream(), x, w, D, Hq, Hkv, C, past + 1000 * r, 500000.0, int(dtype == torch.float32),
                           q, k, v, ws)
            out.append((q, k, v))
        for a, b in zip(*out):
            assert torch.equal(a, b.to(torch.bfloat16)), r
