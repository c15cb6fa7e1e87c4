"""GPU: the mapping loss at the edges of its 16 x 48 tiles: the two image heights between
which a workgroup takes all three channels or one, last tiles of one row or column, and
tile counts that are not a multiple of the eight XCDs, against the oracle with the
tolerances of test_gpu_mapping_loss."""

import pytest

from tests.test_gpu_mapping_loss import ml  # noqa: F401
from tests.test_gpu_mapping_loss import test_mapping_loss_sizes as _check_size

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hw", [(16, 150), (17, 150), (32, 15), (48, 16), (49, 17), (96, 65), (97, 31), (145, 129)])
def test_mapping_loss_tile_edges(ml, hw):  # noqa: F811
    _check_size(ml, hw)
