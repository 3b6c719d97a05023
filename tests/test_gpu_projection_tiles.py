"""The two tile sizes of the projection kernel and the few-token sizes below them: bf16 output through whichever kernel
the launcher picks, against the fp64 oracle, at the edges of token tiles, contractions of two to many steps and shapes
on both sides of the line between the tiles."""
import numpy as np
import pytest
import torch

from oracle import projection as op
from paper_2502_12574_amd import binding as hb
from paper_2502_12574_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _close(got, ref, what):
    got = got.double().cpu().numpy()
    assert np.isfinite(got).all(), what
    rel = float(np.sqrt(((got - ref) ** 2).sum() / (ref ** 2).sum()))
    # one rounding to bf16 (2^-9 at most, 1.7e-3 in the mean square) on fp32 sums
    assert rel <= 2.0e-3 and float((np.abs(got - ref) / (np.abs(ref) + 1.0)).max()) <= 2.0 ** -8 + 1e-5, (what, rel)


@pytest.mark.parametrize("D,Hq,Hkv,C", [(128, 2, 1, 130), (256, 1, 1, 127), (384, 3, 1, 128), (640, 4, 2, 129),
                                        (1024, 8, 2, 385), (1024, 32, 8, 2700), (1024, 32, 8, 2740), (256, 5, 3, 2),
                                        (384, 2, 2, 33), (512, 4, 1, 64), (128, 3, 2, 65), (1152, 8, 4, 17)])
def test_projections(D, Hq, Hkv, C):
    seed, past, theta = 9700 + D + C, 54321, 500000.0
    X = synth.draw_hidden(seed, 0, past, C, D, device=DEV)
    W = synth.draw_weight(seed, synth.TENSOR_WQKV, 0, (Hq + 2 * Hkv) * 128, D, device=DEV)
    q = torch.full((Hq, C, 128), float("nan"), dtype=torch.bfloat16, device=DEV)
    k, v = (torch.full((Hkv, C, 128), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    ws = torch.empty(hb.hi_proj_workspace_bytes(C), dtype=torch.uint8, device=DEV)
    s = torch.cuda.current_stream()
    hb.hi_qkv_rope(s, X, W, D, Hq, Hkv, C, past, theta, 0, q, k, v, ws, q_scale=0.5)
    Wf = synth.to_f64(W.cpu())
    Qr, Kr, Vr = op.qkv_rope(synth.to_f64(X.cpu()), Wf[:Hq * 128], Wf[Hq * 128:(Hq + Hkv) * 128], Wf[(Hq + Hkv) * 128:],
                             np.arange(past, past + C), 128, theta)
    _close(q, 0.5 * Qr, "Q")
    _close(k, Kr, "K")
    _close(v, Vr, "V")
    A = torch.stack([synth.draw_q(seed, 0, h, 0, C, device=DEV) for h in range(Hq)])
    Wo = synth.draw_weight(seed, synth.TENSOR_WO, 0, D, Hq * 128, device=DEV)
    y = torch.full((C, D), float("nan"), dtype=torch.bfloat16, device=DEV)
    hb.hi_out_proj(s, A, Wo, Hq, D, C, 0, y)
    _close(y, op.out_proj(synth.to_f64(A.cpu()), synth.to_f64(Wo.cpu())), "Y")
