"""Which workgroup takes which block of query rows: the rows of a prompt do not depend on it, so a prompt computed in
a batch, in a ragged or packed batch, or alone has the same bits, and one of them is compared with the oracle."""
import numpy as np
import pytest

from oracle import seka_oracle as orc
from paper_2603_01281_amd import inputs
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _layer(B, S, Hq, Hkv, rank, seed):
    return inputs.make_layer("dealing", "bf16", B=B, S=S, Hq=Hq, Hkv=Hkv, D=128, M=1, r=rank, gain=1.0,
                             mask_recipe=("cover", 0.2, 0.2, 2), seed=seed)


def _attend(seka, dev, sl, steered, scale, **ragged):
    import torch
    Q, K, V, mask = (x[sl].contiguous() for x in (dev.Q, dev.K, dev.V, dev.mask))
    O = torch.full_like(Q, float("nan"))
    lse = torch.full((Q.shape[0], Q.shape[2], Q.shape[1]), float("nan"), dtype=torch.float32, device="cuda")
    if ragged:
        st = (dev.U, dev.gain, mask) if steered else ()
        seka.seka_attention_prefill_ragged(Q, K, V, O, ragged["lens"], *st, scale=scale, lse=lse)
    elif steered:
        seka.seka_attention_prefill(Q, K, V, O, dev.U, dev.gain, mask, scale=scale, lse=lse)
    else:
        seka.seka_attention_plain(Q, K, V, O, scale=scale, lse=lse)
    torch.cuda.synchronize()
    return O, lse


# workgroups of 4 x 64, 2 x 128, 1 x 256 and 7 x 32 rows; batches that take single blocks, pairs and several deals
@pytest.mark.parametrize("B,S,Hq,Hkv,rank", [
    (3, 65, 4, 1, 8), (40, 1000, 8, 2, 32), (24, 1217, 16, 4, 64), (33, 700, 8, 4, 32), (20, 897, 6, 2, 128),
    (48, 500, 14, 2, 32), (2, 1537, 14, 2, 64), (70, 1500, 4, 1, 32)])
@pytest.mark.parametrize("steered", [False, True])
def test_batch_equals_prompts(seka, B, S, Hq, Hkv, rank, steered):
    import torch
    print(f"dealing B={B} S={S} {Hq}/{Hkv} rank {rank} steered={steered}", flush=True)
    inp = _layer(B, S, Hq, Hkv, rank, seed=B + S)
    dev = H.DeviceInputs(inp)
    O, lse = _attend(seka, dev, slice(0, B), steered, inp.scale)
    for b in {0, B // 2, B - 1}:
        o1, l1 = _attend(seka, dev, slice(b, b + 1), steered, inp.scale)
        assert torch.equal(O[b:b + 1], o1) and torch.equal(lse[b:b + 1], l1), f"prompt {b}"
    b = B - 1
    o = H.oracle_inputs(inp)
    sl = slice(b, b + 1)
    if steered:
        ref, _ = orc.steered_attention(o["Q"][sl], o["K"][sl], o["V"][sl], o["U"], inp.gain, inp.mask[sl], scale=inp.scale)
    else:
        ref, _ = orc.causal_attention(o["Q"][sl], o["K"][sl], o["V"][sl], scale=inp.scale)
    H.assert_close_bf16(H.to_f64(O[sl]), ref, "prompt in a batch")
    assert torch.isfinite(O.float()).all() and torch.isfinite(lse).all()


# one prompt, a few, as many as a wave has lanes, more than that, and more than workgroups run at a time per head
# chunk (16 chunks of one 256-row head); empty and one-token prompts among them
@pytest.mark.parametrize("B,S,Hq,Hkv", [(1, 1100, 14, 2), (2, 2100, 4, 1), (12, 1024, 8, 2), (64, 300, 4, 1), (66, 200, 4, 1),
                                        (17, 400, 16, 16), (31, 333, 14, 2)])
@pytest.mark.parametrize("steered", [False, True])
def test_ragged_and_packed_equal_prompts(seka, B, S, Hq, Hkv, steered):
    import torch
    print(f"dealing ragged B={B} S={S} {Hq}/{Hkv} steered={steered}", flush=True)
    inp = _layer(B, S, Hq, Hkv, 32, seed=B * S)
    dev = H.DeviceInputs(inp)
    g = np.random.default_rng(B + S)
    lens = np.exp(g.uniform(0, np.log(S), size=B)).astype(np.int32)
    lens[g.integers(B)] = S
    if B > 2:
        lens[1:3] = (0, 1) if lens[1] != S and lens[2] != S else lens[1:3]
    O, lse = _attend(seka, dev, slice(0, B), steered, inp.scale, lens=torch.from_numpy(lens).cuda())
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    pack = lambda x: torch.cat([x[b, :lens[b]] for b in range(B)]).contiguous()
    Qp = pack(dev.Q)
    Op = torch.full_like(Qp, float("nan"))
    st = (dev.U, dev.gain, pack(dev.mask)) if steered else ()
    seka.seka_attention_prefill_packed(Qp, pack(dev.K), pack(dev.V), Op, torch.from_numpy(cu).cuda(), S, *st, scale=inp.scale)
    torch.cuda.synchronize()
    for b in range(B):
        n = int(lens[b])
        if n == 0:
            continue
        one = type("Prompt", (), dict(Q=dev.Q[:, :n], K=dev.K[:, :n], V=dev.V[:, :n], mask=dev.mask[:, :n], U=dev.U, gain=dev.gain))
        o1, l1 = _attend(seka, one, slice(b, b + 1), steered, inp.scale)
        assert torch.equal(O[b:b + 1, :n], o1) and torch.equal(lse[b:b + 1, :, :n], l1), f"ragged prompt {b} of {n} tokens"
        assert torch.equal(Op[cu[b]:cu[b + 1]], o1[0]), f"packed prompt {b} of {n} tokens"


# fp32: single prompts split a row's keys over four waves, the batches here give a row to one wave; up to 5, 9, 21 and 65 steps.
# bf16, D = 64: workgroups of 4 x 64, 2 x 128 and 1 x 256 rows, all on the pipelined kernel
@pytest.mark.parametrize("dtype,B,S,Hq,Hkv,D,r", [
    ("f32", 64, 33, 4, 1, 64, 8), ("f32", 40, 130, 8, 2, 64, 20), ("f32", 30, 143, 6, 2, 128, 8), ("f32", 24, 333, 6, 2, 128, 40),
    ("f32", 6, 1033, 32, 8, 128, 8), ("bf16", 64, 150, 8, 2, 64, 32), ("bf16", 20, 700, 6, 3, 64, 64), ("bf16", 9, 1100, 3, 3, 64, 32)])
@pytest.mark.parametrize("steered", [False, True])
def test_prompts_do_not_depend_on_the_batch(seka, dtype, B, S, Hq, Hkv, D, r, steered):
    import torch
    print(f"dealing {dtype} B={B} S={S} {Hq}/{Hkv} D={D} rank {r} steered={steered}", flush=True)
    inp = inputs.make_layer("dealing", dtype, B=B, S=S, Hq=Hq, Hkv=Hkv, D=D, M=1, r=r, gain=1.0, mask_recipe=("cover", 0.2, 0.2, 2), seed=B + S)
    dev = H.DeviceInputs(inp)
    lens = np.random.default_rng(S).integers(1, S + 1, size=B).astype(np.int32)
    lens[B // 2] = S
    O, lse = _attend(seka, dev, slice(0, B), steered, inp.scale)
    Or, lr = _attend(seka, dev, slice(0, B), steered, inp.scale, lens=torch.from_numpy(lens).cuda())
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    pack = lambda x: torch.cat([x[b, :lens[b]] for b in range(B)]).contiguous()
    Qp = pack(dev.Q)
    Op = torch.full_like(Qp, float("nan"))
    st = (dev.U, dev.gain, pack(dev.mask)) if steered else ()
    seka.seka_attention_prefill_packed(Qp, pack(dev.K), pack(dev.V), Op, torch.from_numpy(cu).cuda(), S, *st, scale=inp.scale)
    torch.cuda.synchronize()
    for b in {0, 1, B // 2, B - 1}:
        o1, l1 = _attend(seka, dev, slice(b, b + 1), steered, inp.scale)
        assert torch.equal(O[b:b + 1], o1) and torch.equal(lse[b:b + 1], l1), f"prompt {b}"
        n = int(lens[b])
        one = type("Prompt", (), dict(Q=dev.Q[:, :n], K=dev.K[:, :n], V=dev.V[:, :n], mask=dev.mask[:, :n], U=dev.U, gain=dev.gain))
        o1, l1 = _attend(seka, one, slice(b, b + 1), steered, inp.scale)
        assert torch.equal(Or[b:b + 1, :n], o1) and torch.equal(lr[b:b + 1, :, :n], l1), f"ragged prompt {b} of {n} tokens"
        assert torch.equal(Op[cu[b]:cu[b + 1]], o1[0]), f"packed prompt {b} of {n} tokens"
