"""The workloads whose speed matters to a user of this library, as data: what is called, on which inputs, how much
work it is and how closely two correct implementations agree.

Every case goes through the public binding the way a serving or evaluation program does: device buffers and
workspaces are allocated once, a pass is the library calls alone.  Shapes are the five benchmark configurations
and the shapes of the tests, with odd lengths among them.  A case is a dict of plain values; `kind` says which
calls one pass makes:

  fused    seka_attention_prefill            SEKA prefill, keys left untouched (scoring, ablations)
  routed   seka_route, then the above        AdaSEKA: expert weights from the prompt's queries, then the prefill
  hook     seka_edit_keys, seka_attention_plain   the paper's hook: edited keys kept (for generation), plain prefill
  packed   seka_route_ragged, seka_attention_prefill_packed   unpadded batch of prompts of different lengths
  decode   seka_attention_decode             one generation step over the cache of edited keys
  project  seka_project_route                query projection with the routing in its epilogue
  learn    seka_learn_projection, seka_head_distance, seka_edit_keys   offline stage of one layer and its first use
"""
import math

import numpy as np
import torch

from paper_2603_01281_amd import binding as seka
from paper_2603_01281_amd import inputs


def listed():
    return [
        # the fp32 path at the size people try the library on: latency and launches
        dict(name="tiny_f32", kind="fused", dtype="f32", B=1, S=256, Hq=4, Hkv=2, D=64, M=1, r=8, gain=0.5, cover=0.125, spans=1),
        # one 4k prompt of a Llama-3-8B-shaped layer: the ordinary single request
        dict(name="seka_4k", kind="fused", dtype="bf16", B=1, S=4096, Hq=32, Hkv=8, D=128, M=1, r=32, gain=1.0, cover=0.10, spans=3),
        # a layer of the batched 8k stack: the headline workload
        dict(name="seka_8k_batch4", kind="fused", dtype="bf16", B=4, S=8192, Hq=32, Hkv=8, D=128, M=1, r=32, gain=1.1, cover=0.13, spans=4),
        # AdaSEKA on a batch of prompts: routing pass and rank-128 edit
        dict(name="adaseka_batch8", kind="routed", dtype="bf16", B=8, S=4096, Hq=32, Hkv=8, D=128, M=4, r=32, gain=1.0, cover=0.10, spans=3),
        # long context, Qwen2.5-7B-shaped heads
        dict(name="seka_32k", kind="fused", dtype="bf16", B=1, S=32768, Hq=28, Hkv=4, D=128, M=1, r=64, gain=1.5, cover=0.07, spans=8),
        # the paper's prompt length (about 4.4k tokens, no multiple of anything), the edited keys kept for generation
        dict(name="hook_4423", kind="hook", dtype="bf16", B=2, S=4423, Hq=32, Hkv=8, D=128, M=2, r=24, gain=0.8, cover=0.12, spans=4),
        # unpadded batch of unequal prompts, routed by their last token (the paper's rule)
        dict(name="packed_ragged", kind="packed", dtype="bf16", B=12, S=4096, Hq=32, Hkv=8, D=128, M=3, r=16, gain=1.0, cover=0.10, spans=3),
        # 64-wide heads
        dict(name="seka_d64", kind="fused", dtype="bf16", B=4, S=4096, Hq=32, Hkv=8, D=64, M=1, r=32, gain=1.0, cover=0.10, spans=3),
        # generation step of a batch at mixed positions of 8k caches
        dict(name="decode_batch16", kind="decode", dtype="bf16", B=16, S=8192, Hq=32, Hkv=8, D=128, ragged=True),
        # generation step of one conversation with a short cache
        dict(name="decode_single", kind="decode", dtype="bf16", B=1, S=1000, Hq=32, Hkv=8, D=128, ragged=False),
        # query projection of a batch of prompts with AdaSEKA's routing
        dict(name="project_batch8", kind="project", dtype="bf16", B=8, S=4096, Hq=32, Hkv=8, D=128, M=4, E=4096),
        # offline stage of one layer: 16k paired key samples
        dict(name="learn_layer", kind="learn", dtype="bf16", n=16384, Hkv=8, D=128, gamma=0.85),
    ]


# ---- drawn cases: the same kinds over their ranges ----------------------------------------------------------------

_HEADS = [(32, 8), (32, 8), (28, 4), (24, 8), (32, 32), (32, 4), (16, 8), (8, 2), (6, 2)]
_MOST_FLOPS = 2.5e12          # per drawn attention or projection; the longest listed prompt takes three times that


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fused", "fused", "fused", "routed", "hook", "packed", "decode", "decode", "project", "learn"])
    if kind == "learn":
        return dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "f32"]), n=_log(rng, 256, 16384), Hkv=rng.choice([2, 4, 8, 8, 12]),
                    D=rng.choice([64, 128, 128]), gamma=0.85)
    Hq, Hkv = rng.choice(_HEADS)
    if kind == "decode":
        S = _log(rng, 128, 32768)
        most = max(1, min(64, (1 << 29) // (S * Hkv * 128)))
        return dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]), B=_log(rng, 1, most), S=S, Hq=Hq, Hkv=Hkv,
                    D=rng.choice([64, 128, 128]), ragged=rng.random() < 0.6)
    if kind == "project":
        c = dict(kind=kind, dtype="bf16", B=_log(rng, 1, 8), S=128 * _log(rng, 1, 32), Hq=Hq, Hkv=Hkv, D=128, M=rng.choice([1, 2, 4, 8]),
                 E=64 * _log(rng, 8, 80))
        return c
    f32 = kind == "fused" and rng.random() < 0.33
    S = _log(rng, 48, 1536) if f32 else _log(rng, 128, 16384)
    if f32:
        Hq, Hkv = rng.choice([(4, 2), (8, 2), (6, 3), (32, 8)])
    D = rng.choice([64, 128]) if f32 or kind == "fused" and rng.random() < 0.3 else 128
    most = max(1, min(16, int(_MOST_FLOPS / (2.0 * D * Hq * S * S)), 65536 // S))
    M = rng.choice([2, 3, 4]) if kind in ("routed", "packed") else rng.choice([1, 1, 1, 2])
    if f32:
        r = rng.choice([3, 8, 12, 16])
    else:
        r = 8 * rng.randint(1, min(16 // M, D // 8))
    return dict(kind=kind, dtype="f32" if f32 else "bf16", B=_log(rng, 1, most), S=S, Hq=Hq, Hkv=Hkv, D=D, M=M, r=r,
                gain=round(rng.uniform(0.25, 1.5), 3), cover=round(rng.uniform(0.03, 0.20), 3), spans=rng.randint(1, 6))


# ---- inputs -------------------------------------------------------------------------------------------------------

def _lengths(case):
    """Prompt lengths of a ragged batch: spread over [S/16, S], the longest one S.  They belong to the case, not to the
    seed, so that every pass of a case is the same amount of work."""
    B, S = case["B"], case["S"]
    g = np.random.Generator(np.random.Philox(key=[B, S]))
    lens = np.maximum(1, np.exp(g.uniform(math.log(max(1, S / 16)), math.log(S), size=B)).astype(np.int64))
    lens[int(g.integers(B))] = S
    return [int(x) for x in lens]


def _spans(n, case, g):
    """0/1 bytes of n tokens: `spans` contiguous highlighted passages of together `cover` of them."""
    m = np.zeros(n, dtype=np.uint8)
    total = max(1, round(case["cover"] * n))
    parts = max(1, min(case["spans"], total, n // 8))
    for s, length in inputs.draw_spans(n, inputs.split_total(total, parts, g), g):
        m[s:s + length] = 1
    return m


class State:
    """Plain attributes: what the calls of one pass take."""


def prepare(case, seed):
    st = State()
    st.kind = case["kind"]
    dev = torch.device("cuda")
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def normal(*shape, mult=1.0):
        x = torch.randn(shape, generator=gen, device=dev, dtype=torch.float32)
        return (x * mult if mult != 1.0 else x).to(dt)

    def scratch(nbytes):
        return torch.empty(max(int(nbytes), 16), dtype=torch.uint8, device=dev)

    Hkv, D = case["Hkv"], case["D"]
    if st.kind == "learn":
        _prepare_learn(st, case, seed, dt, gen, dev)
        return st
    B, S, Hq = case["B"], case["S"], case["Hq"]
    code = seka.SEKA_BF16 if dt == torch.bfloat16 else seka.SEKA_F32
    if st.kind == "decode":
        st.q, st.K, st.V = normal(B, Hq, D), normal(B, S, Hkv, D), normal(B, S, Hkv, D)
        st.O = torch.empty_like(st.q)
        st.lens = torch.tensor(_lengths(case), dtype=torch.int32, device=dev) if case["ragged"] else None
        st.ws = scratch(seka.seka_decode_workspace_bytes(B, S, Hq, Hkv, D, code))
        return st
    if st.kind == "project":
        st.X, st.Wq = normal(B, S, case["E"]), normal(Hq * D, case["E"], mult=case["E"] ** -0.5)
        st.Q = torch.empty((B, S, Hq, D), dtype=dt, device=dev)
        st.Hkv = Hkv
        st.proto = torch.from_numpy(inputs.unit_prototypes(Hkv, case["M"], D, seed)).to(dev)
        st.w = torch.empty((B, Hkv, case["M"]), dtype=torch.float32, device=dev)
        st.ws = scratch(seka.seka_project_route_workspace_bytes(B, S, Hq, Hkv, D, code))
        return st

    M, r = case["M"], case["r"]
    mult = 0.125 if case["dtype"] == "f32" else 1.0       # the fp32 configuration scales its inputs by 1/8
    lens = _lengths(case) if st.kind == "packed" else [S] * B
    rows = (sum(lens),) if st.kind == "packed" else (B, S)
    st.Q, st.K, st.V = (normal(*rows, h, D, mult=mult) for h in (Hq, Hkv, Hkv))
    st.O = torch.empty_like(st.Q)
    U = inputs.orthonormal_bases(Hkv, M, D, r, seed, "f32")
    st.U = torch.from_numpy(U).to(dev).to(dt)
    st.gain = [case["gain"]] * Hkv
    g = np.random.Generator(np.random.Philox(key=[seed, 1]))
    mask = np.concatenate([_spans(n, case, g) for n in lens])
    st.mask = torch.from_numpy(mask).to(dev).reshape(rows)
    st.w = None
    if st.kind in ("routed", "packed"):
        st.proto = torch.from_numpy(inputs.unit_prototypes(Hkv, M, D, seed)).to(dev)
        st.w = torch.empty((B, Hkv, M), dtype=torch.float32, device=dev)
    elif M > 1:                                           # per-prompt expert weights that routing gave earlier
        st.w = torch.softmax(torch.randn((B, Hkv, M), generator=gen, device=dev), dim=-1).contiguous()
    if st.kind == "routed":
        st.S = S
        st.ws = scratch(seka.seka_route_workspace_bytes(B, S, Hq, Hkv, D, code, 0, S))
    if st.kind == "packed":
        st.cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device=dev)
        st.S = max(lens)
        st.ws = scratch(B * Hkv * D * 4)                  # a window of one token is one partial sum per (prompt, head)
    if st.kind == "hook":
        st.K_edited = torch.empty_like(st.K)
    return st


def _prepare_learn(st, case, seed, dt, gen, dev):
    """Paired samples as inputs.paired_key_samples describes them (a 12-dimensional latent code seen through two frames
    with decaying amplitudes, over a noise floor), drawn on the device, and the keys of one prompt to edit."""
    n, Hkv, D, rank = case["n"], case["Hkv"], case["D"], 12
    g = np.random.Generator(np.random.Philox(key=[seed, 2]))
    frames = np.stack([[np.linalg.qr(g.standard_normal((D, rank)))[0] for _ in range(Hkv)] for _ in range(2)])
    frames = torch.from_numpy(frames.astype(np.float32)).to(dev)
    z = torch.randn((Hkv, n, rank), generator=gen, device=dev)
    amp = 2.0 * 0.8 ** torch.arange(rank, device=dev, dtype=torch.float32)
    shift = 0.5 * torch.randn((Hkv, 1, D), generator=gen, device=dev) / math.sqrt(D)
    views = []
    for k in range(2):
        x = torch.bmm(z * amp if k == 0 else z, frames[k].transpose(1, 2).contiguous())
        x = x + 0.05 * torch.randn((Hkv, n, D), generator=gen, device=dev) + (shift if k else 0.0)
        views.append(x.transpose(0, 1).contiguous().to(dt).reshape(1, n, Hkv, D))
    st.ha, st.hb = views
    st.gamma, st.r_pad = case["gamma"], 16
    st.U = torch.empty((Hkv, D, D), dtype=torch.float32, device=dev)
    st.sigma = torch.empty((Hkv, D), dtype=torch.float32, device=dev)
    st.k = torch.empty((Hkv,), dtype=torch.int32, device=dev)
    st.U_packed = torch.empty((Hkv, D, st.r_pad), dtype=dt, device=dev)
    st.U4 = st.U_packed.reshape(Hkv, 1, D, st.r_pad)
    st.dist = torch.empty((Hkv,), dtype=torch.float32, device=dev)
    code = seka.SEKA_BF16 if dt == torch.bfloat16 else seka.SEKA_F32
    st.ws = torch.empty(seka.seka_learn_workspace_bytes(1, n, Hkv, D, code), dtype=torch.uint8, device=dev)
    st.K = torch.randn((1, 1024, Hkv, D), generator=gen, device=dev).to(dt)
    st.K_edited = torch.empty_like(st.K)
    st.mask = torch.ones((1, 1024), dtype=torch.uint8, device=dev)
    st.gain = [1.0] * Hkv


# ---- one pass -----------------------------------------------------------------------------------------------------

def run(st):
    if st.kind == "fused":
        return seka.seka_attention_prefill(st.Q, st.K, st.V, st.O, st.U, st.gain, st.mask, w=st.w)
    if st.kind == "routed":
        seka.seka_route(st.Q, st.proto, 0, st.S, w_out=st.w, workspace=st.ws)
        seka.seka_attention_prefill(st.Q, st.K, st.V, st.O, st.U, st.gain, st.mask, w=st.w)
        return [st.w, st.O]
    if st.kind == "hook":
        seka.seka_edit_keys(st.K, st.K_edited, st.U, st.gain, st.mask, w=st.w)
        seka.seka_attention_plain(st.Q, st.K_edited, st.V, st.O)
        return [st.K_edited, st.O]
    if st.kind == "packed":
        seka.seka_route_ragged(st.Q, st.proto, 1, cu_seqlens=st.cu, max_len=st.S, mode=seka.SEKA_ROUTE_PAPER_EQ6, w_out=st.w,
                               workspace=st.ws)
        seka.seka_attention_prefill_packed(st.Q, st.K, st.V, st.O, st.cu, st.S, st.U, st.gain, st.mask, w=st.w)
        return [st.w, st.O]
    if st.kind == "decode":
        return seka.seka_attention_decode(st.q, st.K, st.V, st.O, seq_lens=st.lens, workspace=st.ws)
    if st.kind == "project":
        seka.seka_project_route(st.X, st.Wq, st.Q, st.Hkv, proto=st.proto, w_out=st.w, workspace=st.ws)
        return [st.Q, st.w]
    # learn: the signs of singular vectors are free and those of the noise floor are any basis of it, so what is
    # returned of them is what they are for: the keys edited with the learned subspace
    seka.seka_learn_projection(st.ha, st.hb, st.gamma, st.U, st.sigma, st.k, U_packed=st.U_packed, workspace=st.ws)
    seka.seka_head_distance(st.ha, st.hb, st.dist, workspace=st.ws)
    seka.seka_edit_keys(st.K, st.K_edited, st.U4, st.gain, st.mask)
    return [st.sigma, st.k, st.dist, st.K_edited]


# ---- work and agreement -------------------------------------------------------------------------------------------

def work(case):
    es = 2 if case["dtype"] == "bf16" else 4
    kind, Hkv, D = case["kind"], case["Hkv"], case["D"]
    if kind == "learn":
        n = case["n"]
        # covariance, and the usual count of a singular value decomposition with one side of vectors
        return {"bytes": 2 * n * Hkv * D * es + Hkv * D * D * 4 + 2 * 1024 * Hkv * D * es,
                "flops": Hkv * (2.0 * n * D * D + 12.0 * D ** 3 + 3.0 * n * D)}
    B, S, Hq = case["B"], case["S"], case["Hq"]
    if kind == "decode":
        tokens = sum(_lengths(case)) if case["ragged"] else B * S
        return {"bytes": 2 * tokens * Hkv * D * es + 2 * B * Hq * D * es, "flops": 4.0 * tokens * Hq * D}
    if kind == "project":
        E, N = case["E"], Hq * D
        return {"bytes": es * (B * S * E + N * E + B * S * N), "flops": 2.0 * B * S * E * N}
    lens = _lengths(case) if kind == "packed" else [S] * B
    tokens = sum(lens)
    nbytes = es * tokens * D * (2 * Hq + 2 * Hkv) + tokens + es * Hkv * case["M"] * D * case["r"]
    if kind == "hook":
        nbytes += es * tokens * D * Hkv                   # the edited keys are an output
    # causal pairs; the edit's own products are under one per cent of them
    return {"bytes": nbytes, "flops": 4.0 * D * Hq * sum(0.5 * n * (n + 1) for n in lens)}


def tolerance(case):
    # Measured against the same path in 64 bits on the listed and on drawn cases (2-norms, and largest errors over
    # the larger of the value and the rms), then taken four times:
    #   bf16 attention   rel 1.8e-3 to 3.5e-3, max 0.007 to 0.056 (late rows average many values of random sign)
    #   bf16 decode, projection, learning   rel 1.6e-3 to 2.4e-3, max 0.004 to 0.008
    #   fp32 attention, decode   rel 0.9e-7 to 2.0e-7;  fp32 learning   rel 6e-7 where the cut falls between well separated values
    if case["dtype"] == "f32":
        return {"rel": 1e-5} if case["kind"] == "learn" else {"rel": 1e-6}
    if case["kind"] in ("decode", "project", "learn"):
        return {"rel": 8e-3, "max": 0.03}
    return {"rel": 1e-2, "max": 0.2}
