"""The network on either side of the size at which its bricks change from 2 to 8 rows."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import test_gpu_cnn_bricks as bricks  # noqa: E402


# 24: two-row bricks that overhang in z; 48: the largest of them; 52: eight-row bricks, overhanging
@pytest.mark.parametrize("n", [24, 48, 52])
def test_rows_of_a_brick_match_oracle(n):
    bricks.test_overhanging_bricks_match_oracle(n)
    bricks.test_last_layer_every_voxel(n)
