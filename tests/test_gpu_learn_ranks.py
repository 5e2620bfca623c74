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
