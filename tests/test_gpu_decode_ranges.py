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
    ("f32", 2, 127, 4, 4, 128, [127, 63]),
    # fp32 on the matrix cores: groups of 4 to 16 heads, odd ones, two chunks of ten; steps of 16 keys, turns of 64
    ("f32", 3, 1500, 32, 8, 128, [1500, 64, 1]), ("f32", 2, 1137, 9, 1, 64, [1137, 0]), ("f32", 2, 15, 20, 1, 64, [15, 1]),
    ("f32", 1, 65, 16, 1, 128, None), ("f32", 5, 200, 6, 2, 128, [200, 17, 16, 0, 193]), ("f32", 2, 333, 6, 2, 64, [333, 79]),
    ("f32", 3, 4000, 7, 1, 128, [129, 4000, 3937]), ("f32", 16, 500, 32, 8, 128, None),
    # three and four heads with more than one workgroup per compute unit: on the vector unit, on the matrix cores, ...
    ("f32", 48, 300, 6, 2, 128, None), ("f32", 80, 300, 6, 2, 128, [300, 129] * 40), ("f32", 72, 300, 6, 2, 64, None),
    ("f32", 160, 300, 6, 2, 64, [300, 1] * 80), ("f32", 28, 384, 16, 4, 128, None),
    # bf16 caches of few groups at D = 128: one range up to 700 tokens, then one per compute unit, at least 64 tokens each
    ("bf16", 1, 700, 8, 2, 128, None), ("bf16", 1, 701, 8, 2, 128, None), ("bf16", 2, 1000, 32, 8, 128, [1000, 65]),
    ("bf16", 1, 4133, 6, 1, 128, None), ("bf16", 5, 1030, 14, 2, 128, [1030, 0, 1, 64, 700]), ("bf16", 33, 1100, 8, 8, 128, None),
    # one range of eight waves for 129 to 256 groups
    ("bf16", 17, 1535, 8, 8, 64, None), ("bf16", 17, 1536, 8, 8, 64, None), ("bf16", 8, 2047, 24, 24, 64, [2047, 0, 1, 33, 512, 1024, 257, 700])])
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


def test_small_workspace(seka):
    """A workspace that holds the states of fewer, longer ranges than there would be: another order of sums, the same result."""
    import torch
    B, S, Hq, Hkv, D = 2, 2100, 8, 2, 128
    print("decode small workspace", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    q, K, V = (torch.randn(shape, generator=g, device="cuda").bfloat16() for shape in ((B, Hq, D), (B, S, Hkv, D), (B, S, Hkv, D)))
    most = seka.seka_decode_workspace_bytes(B, S, Hq, Hkv, D, seka.SEKA_BF16)
    least = B * Hq * (S // 512) * (D + 2) * 4                 # ranges of 512 tokens and more
    ref, _ = orc.decode_attention(H.to_f64(q), H.to_f64(K), H.to_f64(V), np.full(B, S, np.int32))
    for nbytes in (most, least):
        O = torch.full_like(q, float("nan"))
        ws = torch.full((nbytes + 4096,), 0xa5, dtype=torch.uint8, device="cuda")
        seka.seka_attention_decode(q, K, V, O, workspace=ws[:nbytes])
        torch.cuda.synchronize()
        assert bool((ws[nbytes:] == 0xa5).all())              # nothing behind it is written
        H.assert_close_bf16(H.to_f64(O), ref, f"O with {nbytes} bytes")
    assert least < most
    with pytest.raises(seka.SekaError):
        seka.seka_attention_decode(q, K, V, O, workspace=ws[:least - 16])


# bf16 in a single range, of less than a turn of the four waves too; in several, also ragged; fp32 on the matrix cores and on the
# vector unit
@pytest.mark.parametrize("dtype,B,S,Hq,Hkv,D,ragged", [
    ("bf16", 770, 97, 32, 8, 128, False), ("bf16", 74, 1000, 32, 8, 128, False), ("bf16", 148, 1001, 8, 8, 64, False), ("bf16", 37, 2000, 32, 8, 128, False),
    ("bf16", 74, 2003, 8, 8, 64, False), ("bf16", 148, 2100, 32, 8, 128, True), ("f32", 37, 1000, 32, 8, 128, False),
    ("f32", 73, 1017, 56, 8, 64, False), ("f32", 37, 1001, 40, 8, 128, False), ("f32", 148, 1050, 40, 8, 128, True)])
def test_larger_than_the_caches(seka, dtype, B, S, Hq, Hkv, D, ragged):
    """More than 300 MB of keys and values (of a ragged batch four times that), which are read without keeping a place for
    them; the first, a middle and the last prompt."""
    import torch
    print(f"decode large {dtype} B={B} S={S} {Hq}/{Hkv} D={D} ragged={ragged}", flush=True)
    assert 2 * B * S * Hkv * D * (2 if dtype == "bf16" else 4) * (0.25 if ragged else 1) > 300e6
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(S)
    q, K, V = (torch.randn(shape, generator=g, device="cuda").to(dt) for shape in ((B, Hq, D), (B, S, Hkv, D), (B, S, Hkv, D)))
    lens = np.full(B, S, np.int32)
    if ragged:
        lens[:] = np.random.default_rng(S).integers(1, S, B)
    O = torch.full_like(q, float("nan"))
    ws = torch.full((seka.seka_decode_workspace_bytes(B, S, Hq, Hkv, D, seka.SEKA_BF16 if dtype == "bf16" else seka.SEKA_F32),), 0xff,
                    dtype=torch.uint8, device="cuda")
    seka.seka_attention_decode(q, K, V, O, seq_lens=torch.from_numpy(lens).cuda() if ragged else None, workspace=ws)
    for b in (0, B // 2, B - 1):
        ref, _ = orc.decode_attention(H.to_f64(q[b:b + 1]), H.to_f64(K[b:b + 1]), H.to_f64(V[b:b + 1]), lens[b:b + 1])
        if dtype == "f32":
            H.assert_close_f32(H.to_f64(O[b:b + 1]), ref, "O", tol=1e-5)
        else:
            H.assert_close_bf16(H.to_f64(O[b:b + 1]), ref, "O")
