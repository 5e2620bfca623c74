"""GPU parity of seka_project_route over its four tile sizes: half tiles at the edges, counts of slices of E that end in
every turn of the three-stage ring (1 to 7 and 11) and of the four-stage ring (1 to 7 and 11 to 13); and over the kernel for rows of 2^22 elements and more."""
import pytest

from paper_2603_01281_amd import inputs
from tests.test_gpu_project_route import test_project_route as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (1, 128, 3, 3, 704), (2, 128, 5, 1, 448), (1, 384, 7, 7, 64),                        # 128 x 64
    (1, 128, 3, 3, 128), (1, 128, 3, 3, 192), (1, 128, 3, 3, 256), (1, 128, 3, 3, 320), (1, 128, 3, 3, 384), (1, 128, 3, 3, 768), (1, 128, 3, 3, 832),
    (5, 128, 31, 31, 64), (1, 640, 32, 8, 448), (3, 256, 30, 6, 320), (5, 128, 32, 8, 128),      # 128 x 128
    (1, 2176, 17, 17, 256), (17, 128, 16, 4, 448), (2, 1152, 16, 8, 384),                # 256 x 128
    (1, 4224, 17, 17, 64), (11, 384, 18, 6, 256), (33, 128, 19, 19, 320), (11, 384, 17, 17, 384)])      # 256 x 256
def test_project_route_tiles(seka, shape):
    check(seka, shape)


def test_project_route_long_rows(seka):
    """E = 2^22, the kernel with 64-bit offsets: whole numbers, whose sums over E are exact in fp32, and an odd number of slices."""
    import torch
    S, Hkv, M, D = 128, 1, 4, 128
    for E in (1 << 22, (1 << 22) + 64):
        print(f"project_route long rows E={E}", flush=True)
        g = torch.Generator(device="cuda")
        g.manual_seed(E)
        X, W = (torch.randint(-1, 2, (128, E), generator=g, device="cuda", dtype=torch.int8).bfloat16() for _ in range(2))
        proto = torch.from_numpy(inputs.unit_prototypes(Hkv, M, D, 3)).cuda()
        Q = torch.full((1, S, 1, D), float("nan"), dtype=torch.bfloat16, device="cuda")
        w = seka.seka_project_route(X[None], W, Q, Hkv, proto=proto)
        w2 = seka.seka_route(Q, proto, 0, S)
        Q2 = torch.full_like(Q, float("nan"))
        seka.seka_project_route(X[None], W, Q2, Hkv)
        ref = torch.zeros(128, 128, device="cuda")
        for e in range(0, E, 1 << 20):
            ref += X[:, e:e + (1 << 20)].float() @ W[:, e:e + (1 << 20)].float().T.contiguous()
        torch.cuda.synchronize()
        assert torch.equal(Q[0, :, 0], ref.bfloat16()) and torch.equal(Q2, Q)
        assert float((w - w2).abs().max()) <= 1e-6
