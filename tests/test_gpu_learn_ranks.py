"""Offline stage on cross-covariances of exact low rank, around the edges of the factorisation's column blocks (8
columns, pairs of blocks): the pivoted factor stops early and the empty blocks are left out of the iteration."""
import numpy as np
import pytest

from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,n,scale", [(128, 0, 1.0), (128, 1, 1.0), (128, 7, 1e-3), (128, 8, 1.0), (128, 9, 1.0), (128, 16, 30.0),
                                       (128, 17, 1.0), (128, 121, 1.0), (64, 8, 1.0), (64, 33, 1e-3), (64, 57, 1.0)])
def test_low_rank_samples(seka, D, n, scale):
    import torch
    print(f"learn rank D={D} n={n} scale={scale}", flush=True)
    Hkv, gamma = 3, 0.9
    g = np.random.default_rng(100 * D + n)
    ha = (scale * g.standard_normal((max(n, 1), Hkv, D))).astype(np.float32) * (n > 0)      # n tokens: rank n; n = 0: all zero
    hb = g.standard_normal((max(n, 1), Hkv, D)).astype(np.float32)
    U = torch.full((Hkv, D, D), float("nan"), device="cuda")
    sig = torch.full((Hkv, D), float("nan"), device="cuda")
    k = torch.full((Hkv,), -1, dtype=torch.int32, device="cuda")
    seka.seka_learn_projection(torch.from_numpy(ha)[None].cuda(), torch.from_numpy(hb)[None].cuda(), gamma, U, sig, k)
    torch.cuda.synchronize()
    got_U, got_S, got_k = H.to_f64(U), H.to_f64(sig), k.cpu().numpy()
    for h in range(Hkv):
        omega = ha[:, h].astype(np.float64).T @ hb[:, h].astype(np.float64) / max(n, 1)
        s = np.linalg.svd(omega, compute_uv=False)
        # the bounds of the other learning tests: a few fp32 ulp of sigma_1 times sqrt(D)
        assert np.abs(got_S[h] - s).max() <= 2e-5 * s[0] and np.all(np.diff(got_S[h]) <= 0)
        live = got_S[h] > 1e-5 * got_S[h, 0]
        assert live.sum() == n and np.all(got_U[h][:, ~live] == 0.0)
        G = got_U[h][:, live].T @ got_U[h][:, live]
        assert n == 0 or np.abs(G - np.eye(n)).max() <= 1e-4
        assert n == 0 or np.abs(np.linalg.norm(got_U[h][:, live].T @ omega, axis=1) - s[:n]).max() <= 1e-4 * s[0]
        frac = np.cumsum(s) / s.sum() if n else np.ones(D)
        want = int(np.sum(frac < gamma)) + 1
        if np.abs(frac - gamma).min() > 1e-4:
            assert got_k[h] == want


def _learn(seka, ha, hb, gamma, dtype, r_pad=16):
    """U, sigma, k and the packed basis of [n, Hkv, D] samples; every output buffer starts as a value no result has."""
    import torch
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    _, Hkv, D = ha.shape
    U = torch.full((Hkv, D, D), 7.0, device="cuda")
    sig = torch.full((Hkv, D), -7.0, device="cuda")
    k = torch.full((Hkv,), -1, dtype=torch.int32, device="cuda")
    Up = torch.full((Hkv, D, r_pad), 7.0, device="cuda", dtype=dt)
    seka.seka_learn_projection(torch.from_numpy(ha)[None].cuda().to(dt), torch.from_numpy(hb)[None].cuda().to(dt), gamma, U, sig, k,
                               U_packed=Up)
    torch.cuda.synchronize()
    return U, sig, k, Up


# one sample of the middle head: in the neutral view a row of Omega is lost, in the other a column, so every row
@pytest.mark.parametrize("dtype,D,view,value", [("f32", 128, 0, np.nan), ("bf16", 128, 1, np.nan), ("bf16", 64, 0, np.nan),
                                                ("f32", 64, 1, np.inf), ("f32", 128, 0, -np.inf), ("f32", 64, 0, 3e38)])
def test_samples_that_are_not_finite(seka, dtype, D, view, value):
    import torch
    print(f"learn not finite {dtype} D={D} view={view} value={value}", flush=True)
    g = np.random.default_rng(D + view)
    ha, hb = (g.standard_normal((300, 3, D)).astype(np.float32) for _ in range(2))
    clean = _learn(seka, ha, hb, 0.9, dtype)
    (ha, hb)[view][137:139, 1, D // 2] = value                    # two: 3e38 is finite, the sum of its products is not
    (hb, ha)[view][137:139, 1] = np.where(np.arange(D) % 2, 4.0, -4.0)
    U, sig, k, Up = _learn(seka, ha, hb, 0.9, dtype)
    for out in (U, sig, Up):
        assert torch.isnan(out[1].float()).all()
    assert int(k[1]) == D
    for got, want in zip((U, sig, k, Up), clean):                 # the other heads: the same bits as without it
        assert torch.equal(got[[0, 2]], want[[0, 2]]) and torch.isfinite(got[[0, 2]].float()).all()


# squares of Omega's elements, and their reciprocals, beyond fp32 at either end
@pytest.mark.parametrize("dtype,D,n,scale_a,scale_b", [("f32", 128, 300, 1e-10, 1e-10), ("bf16", 128, 300, 1e-10, 1e-10),
                                                       ("f32", 64, 20, 1e-18, 1e-12), ("bf16", 64, 300, 1e-17, 1e-17), ("f32", 128, 9, 1e10, 1e10),
                                                       ("bf16", 128, 300, 1e15, 1e20)])
def test_small_and_large_samples(seka, dtype, D, n, scale_a, scale_b):
    import torch
    print(f"learn scale {dtype} D={D} n={n} {scale_a} {scale_b}", flush=True)
    g = np.random.default_rng(n)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    ha, hb = (torch.from_numpy((s * g.standard_normal((n, 2, D))).astype(np.float32)).to(dt).float().numpy() for s in (scale_a, scale_b))
    U, sig, k, Up = _learn(seka, ha, hb, 0.9, dtype)
    got_U, got_S = H.to_f64(U), H.to_f64(sig)
    assert torch.isfinite(U).all() and torch.isfinite(Up.float()).all()
    for h in range(2):
        omega = ha[:, h].astype(np.float64).T @ hb[:, h].astype(np.float64) / n
        s = np.linalg.svd(omega, compute_uv=False)
        rank = min(n, D)
        assert np.abs(got_S[h] - s).max() <= 2e-5 * s[0] and np.all(np.diff(got_S[h]) <= 0)       # bounds as above
        live = got_S[h] > 1e-5 * got_S[h, 0]
        assert live[:rank // 2].all() and np.all(got_U[h][:, ~live] == 0.0)
        G = got_U[h][:, live].T @ got_U[h][:, live]
        assert np.abs(G - np.eye(int(live.sum()))).max() <= 1e-4
        assert np.abs(np.linalg.norm(got_U[h][:, live].T @ omega, axis=1) - s[live]).max() <= 1e-4 * s[0]
        frac = np.cumsum(s) / s.sum()
        if np.abs(frac - 0.9).min() > 1e-4:
            assert int(k[h]) == int(np.sum(frac < 0.9)) + 1


@pytest.mark.parametrize("D,n", [(128, 1), (128, 9), (128, 60), (64, 5), (64, 33), (64, 64), (128, 300)])
def test_all_of_the_mass(seka, D, n):
    """gamma = 1: values that are exactly zero are not asked for, and what is left out is lost in the sum's rounding."""
    print(f"learn gamma 1 D={D} n={n}", flush=True)
    g = np.random.default_rng(D + n)
    ha, hb = (g.standard_normal((n, 12, D)).astype(np.float32) for _ in range(2))
    U, sig, k, Up = _learn(seka, ha, hb, 1.0, "f32")
    got_S, got_k = H.to_f64(sig), k.cpu().numpy()
    for h in range(12):
        assert 1 <= got_k[h] <= np.count_nonzero(got_S[h]), (h, got_k[h], np.count_nonzero(got_S[h]))
        # a value is absorbed if it is below half an ulp of the sum so far, at most 2^-24 of the total; D of them at most
        assert got_S[h, got_k[h]:].sum() <= D * 2.0 ** -24 * got_S[h].sum()


def _few_valued(kind, n, Hkv, D, g):
    """Samples that take few values, as quantised keys do: what is left of their exactly low-rank Gram matrix, behind the last
    step of the reduction that has something to reduce, shrinks by a factor of 1e-16 and more per step."""
    if kind == "fixed":
        return np.tile((np.arange(D) % 7 - 4).astype(np.float32), (n, Hkv, 1)), np.ones((n, Hkv, D), np.float32)
    if kind == "bits":
        return tuple(g.integers(0, 2, (n, Hkv, D)).astype(np.float32) for _ in range(2))
    if kind == "signs":
        return tuple((2.0 * g.integers(0, 2, (n, Hkv, D)) - 1.0).astype(np.float32) for _ in range(2))
    return tuple(np.round(2.0 * g.standard_normal((n, Hkv, D))).astype(np.float32) for _ in range(2))


# copies: the same tokens 64 times over, which is the same Omega
@pytest.mark.parametrize("copies", [1, 64])
@pytest.mark.parametrize("kind,n,D,dtype", [("fixed", 1, 64, "f32"), ("fixed", 1, 128, "f32")] + [
    (kind, n, D, "bf16" if n == 3 else "f32") for kind in ("bits", "signs", "integers") for n in (1, 2, 3, 4) for D in (64, 128)])
def test_few_valued_samples(seka, kind, n, D, dtype, copies):
    import torch
    print(f"learn few values {kind} n={n} D={D} {dtype} copies={copies}", flush=True)
    Hkv = 32
    ha, hb = _few_valued(kind, n, Hkv, D, np.random.default_rng(1000 * D + n))
    U, sig, k, Up = _learn(seka, np.repeat(ha, copies, axis=0), np.repeat(hb, copies, axis=0), 0.9, dtype)
    got_U, got_S = H.to_f64(U), H.to_f64(sig)
    assert torch.isfinite(U).all() and torch.isfinite(sig).all() and torch.isfinite(Up.float()).all()
    for h in range(Hkv):
        omega = ha[:, h].astype(np.float64).T @ hb[:, h].astype(np.float64) / n
        s = np.linalg.svd(omega, compute_uv=False)
        assert np.abs(got_S[h] - s).max() <= 2e-5 * s[0] and np.all(np.diff(got_S[h]) <= 0)       # bounds as above
        rank = int(np.sum(s > 1e-4 * s[0]))      # integers: the next value is Omega's rounding to fp32
        live = got_S[h] > 1e-5 * got_S[h, 0]
        assert live.sum() == rank and np.all(got_U[h][:, ~live] == 0.0)
        G = got_U[h][:, live].T @ got_U[h][:, live]
        assert rank == 0 or np.abs(G - np.eye(rank)).max() <= 1e-4
        assert rank == 0 or np.abs(np.linalg.norm(got_U[h][:, live].T @ omega, axis=1) - s[:rank]).max() <= 1e-4 * s[0]
        frac = np.cumsum(s) / s.sum() if rank else np.ones(D)
        if np.abs(frac - 0.9).min() > 1e-4:
            assert int(k[h]) == int(np.sum(frac < 0.9)) + 1


# the last number of samples that goes straight to the iteration, and the first that does not
@pytest.mark.parametrize("dtype,D,Hkv,line", [("f32", 128, 2, 31), ("f32", 128, 9, 36), ("f32", 128, 40, 51), ("bf16", 128, 4, 46), ("f32", 64, 8, 18),
                                              ("bf16", 64, 3, 22), ("f32", 64, 40, 34), ("bf16", 64, 32, 32)])
def test_few_samples(seka, dtype, D, Hkv, line):
    import torch
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    for n in (line, line + 1):
        print(f"learn few samples {dtype} D={D} Hkv={Hkv} n={n}", flush=True)
        g = np.random.default_rng(D + n)
        ha, hb = (torch.from_numpy(g.standard_normal((n, Hkv, D)).astype(np.float32)).to(dt).float().numpy() for _ in range(2))
        U, sig, k, _ = _learn(seka, ha, hb, 0.9, dtype)
        got_U, got_S = H.to_f64(U), H.to_f64(sig)
        for h in range(Hkv):
            omega = ha[:, h].astype(np.float64).T @ hb[:, h].astype(np.float64) / n
            s = np.linalg.svd(omega, compute_uv=False)
            assert np.abs(got_S[h] - s).max() <= 2e-5 * s[0] and np.all(np.diff(got_S[h]) <= 0)       # bounds as above
            live = got_S[h] > 1e-5 * got_S[h, 0]
            assert live.sum() == n and np.all(got_U[h][:, ~live] == 0.0)
            G = got_U[h][:, live].T @ got_U[h][:, live]
            # pairs above 2e-7 are rotated, seen through sums of D fp32 products (7 or 8 additions deep: 2^-24 each), and U is
            # rounded to fp32 (2^-24 per column)
            assert np.abs(G - np.eye(n)).max() <= 2e-7 + (8 + 2) * 2.0 ** -24
            assert np.abs(np.linalg.norm(got_U[h][:, live].T @ omega, axis=1) - s[:n]).max() <= 1e-4 * s[0]
            frac = np.cumsum(s) / s.sum()
            if np.abs(frac - 0.9).min() > 1e-4:
                assert int(k[h]) == int(np.sum(frac < 0.9)) + 1
