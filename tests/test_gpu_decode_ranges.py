"""Generation step where the ranges of a cache matter: a multiple of four of them (ragged batches turn their order), empty
ranges, prompts without tokens, fp32's short ranges, and the eight-wave kernel of a single range."""
import numpy as np
import pytest

from oracle import seka_oracle as orc
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,S,Hq,Hkv,D,lens", [
    ("bf16", 4, 4100, 12, 3, 128, [4100, 1, 0, 513]), ("bf16", 5, 2048, 8, 2, 64, [512, 2048, 0, 1536, 33]),
    ("bf16", 3, 1500, 8, 8, 128, [1500, 750, 749]), ("bf16", 2, 1000, 14, 2, 128, [1000, 129]), ("bf16", 1, 129, 4, 4, 64, None),
    ("f32", 3, 700, 14, 2, 128, [700, 64, 0]), ("f32", 2, 257, 6, 3, 64, [257, 65]), ("f32", 1, 4200, 8, 1, 128, None),
    ("f32", 2, 127, 4, 4, 128, [127, 63])])
def test_ranges(seka, dtype, B, S, Hq, Hkv, D, lens):
    import torch
    print(f"decode ranges {dtype} B={B} S={S} {Hq}/{Hkv} D={D}", flush=True)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(S)
    q, K, V = (torch.randn(shape, generator=g, device="cuda").to(dt) for shape in ((B, Hq, D), (B, S, Hkv, D), (B, S, Hkv, D)))
    ln = np.full(B, S, np.int32) if lens is None else np.asarray(lens, np.int32)
    O = torch.full_like(q, float("nan"))
    lse = torch.full((B, Hq), float("nan"), dtype=torch.float32, device="cuda")
    # stale partial states of other calls must not show: the workspace starts as NaN
    code = seka.SEKA_BF16 if dtype == "bf16" else seka.SEKA_F32
    ws = torch.full((max(16, seka.seka_decode_workspace_bytes(B, S, Hq, Hkv, D, code)),), 0xff, dtype=torch.uint8, device="cuda")
    seka.seka_attention_decode(q, K, V, O, seq_lens=None if lens is None else torch.from_numpy(ln).cuda(), lse=lse, workspace=ws)
    torch.cuda.synchronize()
    live = ln > 0
    ref_O, ref_L = orc.decode_attention(H.to_f64(q)[live], H.to_f64(K)[live], H.to_f64(V)[live], ln[live])
    got_O, got_L = H.to_f64(O), H.to_f64(lse)
    if dtype == "f32":
        H.assert_close_f32(got_O[live], ref_O, "O", tol=1e-5)
        H.assert_close_f32(got_L[live], ref_L, "LSE", tol=1e-5)
    else:
        H.assert_close_bf16(got_O[live], ref_O, "O")
        H.assert_lse_close_bf16(got_L[live], ref_L, "LSE", path="decode")
    assert np.all(got_O[~live] == 0.0) and np.all(np.isneginf(got_L[~live]))
