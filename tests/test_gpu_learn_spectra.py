"""Offline stage on prescribed singular values: spread ones take the tridiagonal path and are held to its accuracy, which the
iteration does not reach; equal and nearly equal ones the iteration, which needs no gaps (or either, where the samples'
rounding separates them); around the threshold between them; matrices that are diagonal already."""
import numpy as np
import pytest

from tests import helpers as H

pytestmark = pytest.mark.gpu


def _spectrum(name, D):
    s = 1.0 / (1.0 + np.arange(D))
    if name == "equal":
        s[:] = 0.5
    elif name == "pairs":
        s = np.repeat(s[:D // 2], 2)
    elif name == "cluster":
        s[D // 2:D // 2 + 5] = s[D // 2]
    elif name == "near":                     # squares that differ by 2e-9 .. 2e-2 of themselves: both sides of 1e-7
        for j in range(8):
            s[8 * j + 1] = s[8 * j] * (1.0 - 10.0 ** (-9 + j))
    elif name == "geometric":                # across the limit of a direction (1e-5) and of a value (1e-7)
        s = 10.0 ** (-9.0 * np.arange(D) / D)
    elif name == "two_levels":
        s = np.where(np.arange(D) < D // 3, 1.0, 1e-3)
    return np.sort(s)[::-1]


@pytest.mark.parametrize("rotated", [True, False])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("name", ["spread", "equal", "pairs", "cluster", "near", "geometric", "two_levels"])
def test_prescribed_singular_values(seka, name, D, rotated):
    import torch
    print(f"learn spectrum {name} D={D} rotated={rotated}", flush=True)
    g = np.random.default_rng(D + len(name))
    Hkv = 2
    ha, hb = np.empty((D, Hkv, D), np.float32), np.empty((D, Hkv, D), np.float32)
    want = _spectrum(name, D)
    for h in range(Hkv):                     # Omega = Q1 diag(s) Q2^T; not rotated: diagonal, in an order of its own
        Q1, Q2 = (np.linalg.qr(g.standard_normal((D, D)))[0] if rotated else np.eye(D)[g.permutation(D)] for _ in range(2))
        ha[:, h] = np.sqrt(D) * want[:, None] * Q1.T
        hb[:, h] = np.sqrt(D) * Q2.T
    U = torch.full((Hkv, D, D), float("nan"), device="cuda")
    sig = torch.full((Hkv, D), float("nan"), device="cuda")
    k = torch.full((Hkv,), -1, dtype=torch.int32, device="cuda")
    seka.seka_learn_projection(torch.from_numpy(ha)[None].cuda(), torch.from_numpy(hb)[None].cuda(), 0.9, U, sig, k)
    torch.cuda.synchronize()
    got_U, got_S = H.to_f64(U), H.to_f64(sig)
    for h in range(Hkv):
        omega = ha[:, h].astype(np.float64).T @ hb[:, h].astype(np.float64) / D
        s = np.linalg.svd(omega, compute_uv=False)
        assert np.abs(got_S[h] - s).max() <= 2e-5 * s[0] and np.all(np.diff(got_S[h]) <= 0)      # bounds of the other learning tests
        live = got_S[h] > 1e-5 * got_S[h, 0]
        assert np.all(got_U[h][:, ~live] == 0.0)
        G = got_U[h][:, live].T @ got_U[h][:, live]
        # Spread: relative gaps r of the squares are 1.5e-2 and more, where the vectors in fp64 are orthogonal to D 2^-53 / r < 1e-12;
        # rounding U_out to fp32 moves a dot product by at most 2 x 2^-24 sum |u_i u_j| <= 2^-23.  The iteration stops at 2e-6.
        assert np.abs(G - np.eye(int(live.sum()))).max() <= (2.0 ** -23 + 1e-9 if name in ("spread", "geometric") else 1e-4)
        # columns are left singular vectors: u_i^T Omega has length sigma_i, and different ones are orthogonal.  The iteration
        # stops at |u_i . u_j| = 2e-6, and u_i^T Omega Omega^T u_j is at most sigma_1^2 times what both of u_i and u_j are off
        # their directions: 2 x 2e-6, and rounding of U_out to fp32; 1e-5 covers both
        R = got_U[h][:, live].T @ omega
        assert np.abs(np.linalg.norm(R, axis=1) - s[live]).max() <= 1e-4 * s[0]
        off = R @ R.T - np.diag(np.sum(R * R, axis=1))
        assert np.abs(off).max() <= 1e-5 * s[0] ** 2
        frac = np.cumsum(s) / s.sum()
        if np.abs(frac - 0.9).min() > 1e-4:
            assert int(k[h]) == int(np.sum(frac < 0.9)) + 1
