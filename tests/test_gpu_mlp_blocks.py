"""A training step where the row blocks per workgroup change back to one (past 8192 rows):
as in test_gpu_mlp_sizes, whose check this is."""
import pytest

from test_gpu_mlp_sizes import test_training_step_at_tile_edges as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [8191, 8192, 8193])
def test_training_step_around_two_blocks(B):
    check(B)
