"""The split and pairing the library picks for a prefill unit (prefill_unit_shape): replayed on the host over tile ids,
and on the GPU against the oracle at splits that are no power of two, more than eight workgroups per block, a ragged
last block, an empty past and several staging slices."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from oracle import attention as oa
from paper_2502_12574_amd import binding as hb
from paper_2502_12574_amd import synth
from paper_2502_12574_amd.session import Session

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAX_ABS, REL_L2 = 1e-2, 5e-3        # the bounds of the parity tests: bf16 softmax weights, fp32 sums and output


def test_every_tile_is_counted_exactly_once(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "unit_shape_check")
    subprocess.run([gxx, "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2502_12574_amd", "csrc"),
                    os.path.join(ROOT, "tests", "unit_shape_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and " 0 failures" in r.stdout, r.stdout[-4000:]


# (G, heads, past, chunk, offload, flags)
SHAPES = [(4, 2, 3001, 77, False, 0), (4, 8, 1500, 30, False, 0), (4, 3, 700, 200, True, 0), (1, 2, 1000, 77, False, 0),
          (8, 2, 2049, 65, False, 0), (2, 1, 5000, 1, False, 0), (4, 8, 0, 600, False, 0), (4, 8, 448, 600, False, 0),
          (4, 1, 4000, 300, True, hb.HI_FLAG_PREFILL_DEEP), (4, 1, 4000, 300, False, hb.HI_FLAG_PREFILL_DEEP | hb.HI_FLAG_PREFILL_PAIRED),
          (4, 1, 4000, 300, False, hb.HI_FLAG_PREFILL_DEEP | hb.HI_FLAG_PREFILL_MFMA32),
          (4, 1, 4000, 300, False, hb.HI_FLAG_PREFILL_DEEP | hb.HI_FLAG_PREFILL_WIDE)]


@pytest.mark.gpu
@pytest.mark.parametrize("G,H,past,C,offload,flags", SHAPES)
def test_unit_against_the_oracle(G, H, past, C, offload, flags):
    dev, seed, S = "cuda:0", 52000, past + C
    Q = [torch.stack([synth.draw_q(seed, 0, h * G + g, past, C) for g in range(G)]) for h in range(H)]
    K = [synth.draw_k(seed, 0, h, 0, S, peaked=True) for h in range(H)]
    V = [synth.draw_v(seed, 0, h, 0, S) for h in range(H)]
    with Session(1, H, G, S, C, mode=hb.HI_MODE_OFFLOAD if offload else hb.HI_MODE_RESIDENT, out_fp32=1) as ss:
        hb.hi_ctx_set_flags(ss.ctx, flags)
        view = ss.cache_view()
        for h in range(H):
            view[0, h, 0, :past] = K[h][:past]
            view[0, h, 1, :past] = V[h][:past]
        q = torch.stack(Q).to(dev)
        k = torch.stack([x[past:] for x in K]).to(dev)
        v = torch.stack([x[past:] for x in V]).to(dev)
        out = torch.full((H, G, C, 128), float("nan"), dtype=torch.float32, device=dev)
        ss.s_compute.wait_stream(torch.cuda.current_stream())
        for _ in range(2):                              # the second call finds the first one's states in the workspace
            ss.prefill_group(0, 0, H, q, k, v, past, out)
        ss.sync()
        got = out.cpu().double().numpy()
    for h in range(H):
        k64, v64 = synth.to_f64(K[h]), synth.to_f64(V[h])
        for g in range(G):
            ref = oa.attn_rows(synth.to_f64(Q[h][g]), k64, v64, range(past, S))
            err = float(np.abs(got[h, g] - ref).max())
            rel = float(np.sqrt(((got[h, g] - ref) ** 2).sum() / (ref ** 2).sum()))
            assert err <= MAX_ABS and rel <= REL_L2, (h, g, err, rel)
