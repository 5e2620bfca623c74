"""GPU parity of seka_project_route over its four tile sizes: half tiles at the edges, counts of slices of E that end in
every turn of the three-stage ring (1 to 7 and 11)."""
import pytest

from tests.test_gpu_project_route import test_project_route as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (1, 128, 3, 3, 704), (2, 128, 5, 1, 448), (1, 384, 7, 7, 64),                        # 128 x 64
    (5, 128, 31, 31, 64), (1, 640, 32, 8, 448), (3, 256, 30, 6, 320), (5, 128, 32, 8, 128),      # 128 x 128
    (1, 2176, 17, 17, 256), (17, 128, 16, 4, 448), (2, 1152, 16, 8, 384),                # 256 x 128
    (1, 4224, 17, 17, 64), (11, 384, 18, 6, 256), (33, 128, 19, 19, 320), (11, 384, 17, 17, 384)])      # 256 x 256
def test_project_route_tiles(seka, shape):
    check(seka, shape)
