"""bf16 prefill at head dimension 64 at the edges of its tiles (64 keys), blocks of rows and ranks, against the oracle."""
import numpy as np
import pytest

from oracle import seka_oracle as orc
from paper_2603_01281_amd import inputs
from tests import helpers as H

pytestmark = pytest.mark.gpu


# every workgroup shape (4 x 64, 2 x 128, 1 x 256, 7 x 32 rows), both forms of the edit, one tile to several turns of the
# ring, and (80 prompts and more) the sizes that stay with the register-staged kernel: plain up to 256 / heads rows, steered at 64 and up to 8
@pytest.mark.parametrize("B,S,Hq,Hkv,M,r", [
    (1, 1, 4, 1, 1, 8), (2, 64, 8, 2, 1, 32), (1, 65, 4, 2, 1, 40), (1, 129, 3, 3, 4, 8), (2, 257, 6, 2, 2, 64), (1, 448, 14, 2, 1, 16),
    (1, 900, 4, 1, 2, 16), (1, 833, 7, 1, 4, 32), (1, 1100, 2, 1, 1, 64), (80, 130, 4, 4, 1, 32), (80, 260, 4, 4, 3, 32),
    (80, 64, 4, 4, 1, 32), (140, 64, 4, 2, 2, 32), (80, 8, 4, 4, 1, 64), (80, 9, 4, 4, 1, 32), (80, 65, 4, 4, 1, 64), (140, 128, 4, 2, 1, 16)])
@pytest.mark.parametrize("scaled", [False, True])
def test_d64(seka, B, S, Hq, Hkv, M, r, scaled):
    import torch
    print(f"d64 B={B} S={S} {Hq}/{Hkv} {M} x {r} scaled={scaled}", flush=True)
    inp = inputs.make_layer("d64", "bf16", B=B, S=S, Hq=Hq, Hkv=Hkv, D=64, M=M, r=r, gain=0.5 if scaled else 1.0,
                            mask_recipe=("cover", 0.3, 0.3, 2 if S > 8 else 1), seed=S + r)
    dev = H.DeviceInputs(inp)
    o = H.oracle_inputs(inp)
    w = torch.softmax(torch.randn(B, Hkv, M, generator=torch.Generator().manual_seed(S)), -1)
    key_scale = [0.75] * Hkv if scaled else None
    O = torch.full_like(dev.Q, float("nan"))
    lse = dev.lse_buffer()
    seka.seka_attention_prefill(dev.Q, dev.K, dev.V, O, dev.U, [0.5 if scaled else 1.0] * Hkv, dev.mask, w=w.cuda(), lse=lse,
                                scale=inp.scale, key_scale=key_scale)
    P = torch.full_like(dev.Q, float("nan"))
    seka.seka_attention_plain(dev.Q, dev.K, dev.V, P, scale=inp.scale)
    torch.cuda.synchronize()
    some = sorted({0, B - 1})
    Uc, w64 = o["U"], w.numpy().astype(np.float64)
    for b in some:
        sl = slice(b, b + 1)
        K = o["K"][sl].copy()
        for h in range(Hkv):
            proj = sum(w64[b, h, m] * Uc[h, m] @ Uc[h, m].T for m in range(M))
            rows = inp.mask[b] != 0
            K[0, rows, h] = (0.75 if scaled else 1.0) * K[0, rows, h] + (0.5 if scaled else 1.0) * K[0, rows, h] @ proj
        ref_O, ref_L = orc.causal_attention(o["Q"][sl], K, o["V"][sl], scale=inp.scale)
        H.assert_close_bf16(H.to_f64(O[sl]), ref_O, f"prompt {b}")
        H.assert_lse_close_bf16(H.to_f64(lse[sl]), ref_L, f"prompt {b} LSE", path="steered", n_keys=S)
        ref_P, _ = orc.causal_attention(o["Q"][sl], o["K"][sl], o["V"][sl], scale=inp.scale)
        H.assert_close_bf16(H.to_f64(P[sl]), ref_P, f"prompt {b} plain")
