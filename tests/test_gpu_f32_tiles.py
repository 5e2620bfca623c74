"""fp32 attention at the edges of its tiles: 16-row units, 16-key blocks, the two ways of handing units to waves
(keys of a unit split over four waves / a unit per wave), rank blocks of 16, key scales, partial last units."""
import numpy as np
import pytest

from oracle import seka_oracle as orc
from paper_2603_01281_amd import inputs
from tests import helpers as H

pytestmark = pytest.mark.gpu

# (B, S, Hq, Hkv, D, M, r): the first five take the split form, the last three fill the chip (a unit per wave)
CASES = [(1, 1, 2, 1, 64, 1, 1), (1, 16, 2, 2, 128, 1, 16), (2, 33, 3, 1, 64, 1, 17), (1, 130, 4, 2, 128, 2, 64), (1, 257, 2, 1, 64, 4, 16),
         (40, 17, 6, 2, 128, 1, 9), (32, 47, 7, 1, 64, 3, 40), (12, 97, 10, 2, 128, 1, 33),
         # both sides of a line between the forms: few steps and about 500 units, few steps and over 1024, more steps and over 1024
         (3, 67, 32, 8, 64, 1, 8), (15, 66, 8, 2, 64, 1, 8), (71, 49, 4, 2, 64, 1, 16), (3, 162, 32, 8, 64, 1, 8), (19, 70, 12, 2, 128, 1, 8),
         (17, 129, 12, 3, 128, 1, 8)]


@pytest.mark.parametrize("B,S,Hq,Hkv,D,M,r", CASES)
def test_f32_tile_edges(seka, B, S, Hq, Hkv, D, M, r):
    import torch
    print(f"f32 edges B={B} S={S} Hq={Hq} Hkv={Hkv} D={D} M={M} r={r}", flush=True)
    gain = [(-0.5, 1.25)[h % 2] for h in range(Hkv)]
    kscale = [(1.0, 0.75)[h % 2] for h in range(Hkv)]
    inp = inputs.make_layer("f32edges", "f32", B=B, S=S, Hq=Hq, Hkv=Hkv, D=D, M=M, r=r, gain=gain, mask_recipe=("cover", 0.3, 0.3, 1),
                            seed=S, qkv_mult=0.5)
    dev, o = H.DeviceInputs(inp), H.oracle_inputs(inp)
    w = (np.random.default_rng(S).standard_normal((B, Hkv, M)) if M > 1 else np.ones((B, Hkv, M))).astype(np.float32)
    O, lse = torch.full_like(dev.Q, float("nan")), dev.lse_buffer()
    seka.seka_attention_prefill(dev.Q, dev.K, dev.V, O, dev.U, gain, dev.mask, w=torch.from_numpy(w).cuda(), lse=lse, scale=inp.scale,
                                key_scale=kscale)
    torch.cuda.synchronize()
    ref_O, ref_L = orc.steered_attention(o["Q"], o["K"], o["V"], o["U"], gain, inp.mask, w=w.astype(np.float64), scale=inp.scale,
                                         key_scale=kscale)
    # scores are sums of D fp32 products of values around 0.25 and edited keys at most about 5 times larger: their
    # error is below sqrt(128) * 5 * 2^-24 * 3 / sqrt(64) < 2e-6, and an output moves by at most 2 max|V| (4) of that
    H.assert_close_f32(H.to_f64(O), ref_O, "O", tol=1e-5)
    H.assert_close_f32(H.to_f64(lse), ref_L, "LSE", tol=1e-5)


@pytest.mark.parametrize("B,S,D,r,bad", [(1, 90, 64, 8, "weight"), (1, 90, 128, 20, "basis"), (64, 90, 128, 8, "weight"), (64, 90, 64, 20, "basis")])
def test_f32_edit_touches_highlighted_keys_only(seka, B, S, D, r, bad):
    """A weight or a basis that is not finite reaches the highlighted keys and no other key of their block: rows that see
    none of them have the bits of plain attention."""
    import torch
    print(f"f32 not finite B={B} S={S} D={D} r={r} {bad}", flush=True)
    Hq, Hkv = 4, 2
    inp = inputs.make_layer("f32edges", "f32", B=B, S=S, Hq=Hq, Hkv=Hkv, D=D, M=2, r=r, gain=1.0, mask_recipe=("cover", 0.3, 0.3, 1),
                            seed=S, qkv_mult=0.5)
    dev = H.DeviceInputs(inp)
    first = 37                                                    # inside a 16-key block
    mask = torch.zeros((B, S), dtype=torch.uint8, device="cuda")
    mask[:, first:first + 9] = 1
    w = torch.full((B, Hkv, 2), 0.5, device="cuda")
    if bad == "weight":
        w[:, 0, 1], w[:, 1, 0] = float("nan"), float("inf")
    else:
        dev.U[:, 1, 5, 3] = float("nan")
    P, O = torch.full_like(dev.Q, 7.0), torch.full_like(dev.Q, 7.0)
    seka.seka_attention_plain(dev.Q, dev.K, dev.V, P, scale=inp.scale)
    seka.seka_attention_prefill(dev.Q, dev.K, dev.V, O, dev.U, [1.0] * Hkv, mask, w=w, scale=inp.scale)
    torch.cuda.synchronize()
    assert torch.equal(O[:, :first], P[:, :first])
    assert not torch.isfinite(O[:, first:]).all(-1).any()
