"""bf16 attention where the softmax reference has to move: one key far above everything before it, at every position within a
tile, and keys that are not numbers."""
import numpy as np
import pytest

from tests import helpers as H

pytestmark = pytest.mark.gpu


def _reference(Q, K, V):
    q, k, v = (x.double().cpu() for x in (Q, K, V))
    B, S, Hq, D = q.shape
    k, v = (x.repeat_interleave(Hq // k.shape[2], dim=2) for x in (k, v))
    s = (q.permute(0, 2, 1, 3).contiguous() @ k.permute(0, 2, 3, 1).contiguous()) * D ** -0.5
    mask = np.triu(np.ones((S, S), dtype=bool), 1)
    s.masked_fill_(__import__("torch").from_numpy(mask), float("-inf"))
    return (s.softmax(-1) @ v.permute(0, 2, 1, 3).contiguous()).permute(0, 2, 1, 3).numpy()


@pytest.mark.parametrize("D,Hq,Hkv", [(128, 8, 2), (128, 2, 2), (128, 7, 1), (64, 8, 2)])
def test_late_raise(seka, D, Hq, Hkv):
    import torch
    S = 456                                              # seven full tiles and eight keys
    for j in (0, 5, 17, 31, 32, 63, 64, 100, 191, 192, 250, 383, 447, 448, 455):
        print(f"late raise D={D} heads {Hq}/{Hkv} key {j}", flush=True)
        g = torch.Generator(device="cuda")
        g.manual_seed(j)
        Q, K, V = (torch.randn((1, S, h, D), generator=g, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
        K[:, j] = (3.0 * Q[:, S // 2].reshape(1, Hkv, Hq // Hkv, D)[:, :, 0]).bfloat16()     # some rows score it 2^40 above the rest
        O = torch.full_like(Q, float("nan"))
        seka.seka_attention_plain(Q, K, V, O)
        torch.cuda.synchronize()
        H.assert_close_bf16(H.to_f64(O), _reference(Q, K, V), f"late raise at {j}")


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_keys_that_are_not_numbers(seka, D, bad):
    """Rows before such a key are untouched; rows from it on are not numbers (an infinite key scores inf or -inf by the sign of
    the query, and a row of -inf and finite scores is an ordinary one)."""
    import torch
    S, Hq, Hkv, j = 300, 8, 2, 170
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    Q, K, V = (torch.randn((1, S, h, D), generator=g, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    clean = torch.empty_like(Q)
    seka.seka_attention_plain(Q, K, V, clean)
    K[:, j, :, 3] = bad
    O = torch.empty_like(Q)
    seka.seka_attention_plain(Q, K, V, O)
    torch.cuda.synchronize()
    assert torch.equal(O[:, :j], clean[:, :j])
    tail = O[:, j:].float()
    hit = torch.ones_like(tail, dtype=torch.bool) if bad != bad else (Q[:, j:, :, 3:4].float() > 0).expand_as(tail)
    assert torch.isnan(tail[hit]).all()
    assert torch.isfinite(tail[~hit]).all()


@pytest.mark.parametrize("D,r,Hq,Hkv", [(128, 32, 8, 2), (128, 8, 2, 2), (64, 16, 8, 2), (64, 32, 2, 1), (128, 64, 8, 2)])
@pytest.mark.parametrize("j", [0, 17, 31])
def test_first_reference_of_highlighted_keys(seka, D, r, Hq, Hkv, j):
    """A highlighted key of the first block that is all of a row: its probability is a power of two (against a reference without the
    edit it is rounded to bf16, 2^-9 of the sum).  Scores are exact here; the other keys are e^-15 of the sum, exp2 and the
    logarithm of a number near 20 are good to 4e-6."""
    import torch
    S = 200
    for top in (14.0, 14.375, 15.0, 15.5):               # 8 significant bits; the edit doubles the key's score
        print(f"first reference D={D} r={r} heads {Hq}/{Hkv} key {j} score {top}", flush=True)
        Q, K = torch.zeros((1, S, Hq, D), device="cuda"), torch.zeros((1, S, Hkv, D), device="cuda")
        Q[..., 0] = 8.0
        K[:, j, :, 0] = top / 2
        V = torch.randn((1, S, Hkv, D), device="cuda")
        U = torch.zeros((Hkv, 1, D, r), device="cuda")
        U[:, 0, torch.arange(r), torch.arange(r)] = 1.0
        Q, K, V, U = (x.bfloat16() for x in (Q, K, V, U))
        mask = torch.zeros((1, S), dtype=torch.uint8, device="cuda")
        mask[:, j] = 1
        O, lse = torch.empty_like(Q), torch.empty((1, Hq, S), device="cuda")
        seka.seka_attention_prefill(Q, K, V, O, U, [1.0] * Hkv, mask, scale=0.125, lse=lse)
        torch.cuda.synchronize()
        i = np.arange(S)
        ref = np.where(i < j, np.log(i + 1.0), np.log(i + np.exp(top)))
        d = np.abs(lse.double().cpu().numpy() - ref)
        assert d.max() <= 1e-5, f"{d.max():.3g} at row {int(d.max((0, 1)).argmax())}"


@pytest.mark.parametrize("D,r", [(128, 16), (128, 64), (64, 16), (64, 64)])
def test_infinite_key_beside_a_highlighted_one(seka, D, r):
    """A key that is not highlighted gets no correction, not even 0 times what its products with the basis are."""
    import torch
    S, Hq, Hkv, j = 300, 8, 2, 170
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    Q, K, V = (torch.randn((1, S, h, D), generator=g, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    U = torch.zeros((Hkv, 1, D, r), device="cuda")
    U[:, 0, torch.arange(r), torch.arange(r)] = 1.0
    mask = torch.zeros((1, S), dtype=torch.uint8, device="cuda")
    mask[:, j - 1] = 1                                   # one of the same 16 keys
    out = []
    for K3 in (K[:, j, :, 3].clone(), float("inf")):
        K[:, j, :, 3] = K3
        O = torch.empty_like(Q)
        seka.seka_attention_prefill(Q, K, V, O, U.bfloat16(), [0.5] * Hkv, mask)
        torch.cuda.synchronize()
        out.append(O)
    assert torch.equal(out[1][:, :j], out[0][:, :j])
    low = (Q[:, j:, :, 3:4].float() < 0).expand_as(out[1][:, j:])       # scores of -inf: ordinary rows
    assert torch.isfinite(out[1][:, j:].float()[low]).all()
    assert torch.isnan(out[1][:, j:].float()[~low]).all()


@pytest.mark.parametrize("D,r,Hq,Hkv", [(128, 16, 8, 2), (128, 32, 7, 1), (128, 64, 8, 2), (64, 16, 8, 2), (64, 64, 2, 2)])
def test_late_raise_by_a_highlighted_key(seka, D, r, Hq, Hkv):
    """The edit doubles the key that is far above everything before it: scores of both sides of the reference come from the correction
    (rank <= 32) or from the edited tile."""
    import torch
    S = 456
    U = torch.zeros((Hkv, 1, D, r), device="cuda")
    U[:, 0, torch.arange(r), torch.arange(r)] = 1.0
    for j in (17, 32, 63, 64, 100, 191, 250, 383, 447, 448, 455):
        print(f"late raise, highlighted D={D} r={r} heads {Hq}/{Hkv} key {j}", flush=True)
        g = torch.Generator(device="cuda")
        g.manual_seed(100 + j)
        Q, K, V = (torch.randn((1, S, h, D), generator=g, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
        q = Q[:, S // 2].reshape(1, Hkv, Hq // Hkv, D)[:, :, 0].float()
        q[..., r:] = 0                                   # all of it in the basis: the edit doubles it exactly
        K[:, j] = (1.5 * q * (D / r) ** 0.5).bfloat16()
        mask = torch.zeros((1, S), dtype=torch.uint8, device="cuda")
        mask[:, j] = 1
        Ke = K.clone()
        Ke[:, j] *= 2
        O = torch.full_like(Q, float("nan"))
        seka.seka_attention_prefill(Q, K, V, O, U.bfloat16(), [1.0] * Hkv, mask)
        torch.cuda.synchronize()
        H.assert_close_bf16(H.to_f64(O), _reference(Q, Ke, V), f"late raise, highlighted key {j}")


@pytest.mark.parametrize("D,Hq,Hkv,r", [(128, 8, 2, 0), (128, 2, 2, 0), (128, 7, 1, 0), (128, 3, 3, 0), (64, 8, 2, 0), (64, 7, 1, 0),
                                        (128, 8, 2, 16), (128, 8, 2, 64), (64, 8, 2, 16), (64, 2, 1, 64)])
def test_row_sums_of_long_rows(seka, D, Hq, Hkv, r):
    """Keys that all score the same: every probability is the power of two that the reference leaves (kept exactly in bf16), so row i's sum is
    that of i + 1 equal terms, exact in fp32, and its log-sum-exp is the score + log(i + 1).  What is left is the rounding of numbers below
    16, the reference and the logarithm: a few times 2^-21.  Highlighted keys are orthogonal to the basis: the edit changes nothing."""
    import torch
    S, score = 8231, 1.375
    Q, K = torch.zeros((1, S, Hq, D), device="cuda"), torch.zeros((1, S, Hkv, D), device="cuda")
    Q[..., 0] = 8.0
    K[..., 0] = score
    V = torch.ones((1, S, Hkv, D), device="cuda")
    Q, K, V = (x.bfloat16() for x in (Q, K, V))
    O, lse = torch.full_like(Q, float("nan")), torch.empty((1, Hq, S), device="cuda")
    if r:
        U = torch.zeros((Hkv, 1, D, r), device="cuda")
        U[:, 0, torch.arange(1, r + 1) % D, torch.arange(r)] = 1.0
        U[:, 0, 0] = 0.0
        mask = (torch.arange(S, device="cuda")[None] % 3 == 1).to(torch.uint8).contiguous()
        seka.seka_attention_prefill(Q, K, V, O, U.bfloat16(), [1.0] * Hkv, mask, scale=0.125, lse=lse)
    else:
        seka.seka_attention_plain(Q, K, V, O, lse=lse, scale=0.125)
    torch.cuda.synchronize()
    d = np.abs(lse.double().cpu().numpy() - (score + np.log(np.arange(S) + 1.0)))
    assert d.max() <= 5e-6, f"{d.max():.3g} at row {int(d.max((0, 1)).argmax())}"
    assert (O == 1).all()
