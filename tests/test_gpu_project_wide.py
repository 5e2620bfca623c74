"""GPU parity of seka_project_route at middle sizes (256 x 128 tiles): half tiles at the tokens' edge, 1 to 6 slices of E, several
prompts in one tile."""
import pytest

from tests.test_gpu_project_route import test_project_route as check

pytestmark = pytest.mark.gpu


# tokens x features in 128s: 17 x 17 (half a tile of tokens missing), 34 x 8, 16 x 18, 18 x 16 and 45 x 6 (half a tile missing)
@pytest.mark.parametrize("shape", [(1, 2176, 17, 17, 64), (2, 2176, 8, 2, 128), (1, 2048, 18, 6, 192), (6, 384, 16, 4, 256),
                                   (15, 384, 6, 3, 384)])
def test_project_route_wide(seka, shape):
    check(seka, shape)
