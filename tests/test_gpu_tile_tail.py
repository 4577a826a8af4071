"""Blocks at the level counts whose last step runs furthest past a column's
end (three slices with no packed remainder, stepped over two at a time; nine
slices), as test_gpu_tile_blocks: bit for bit the gather, up to the sign of
zero."""
import pytest
import torch

from test_gpu_tile_blocks import CODES
from test_gpu_tile_blocks import test_tiles_equal_the_gather as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", list(CODES), ids=["f64", "f32", "bf16"])
@pytest.mark.parametrize("L", [161, 180, 191, 192, 193, 545, 576])
def test_last_steps(L, dtype):
    check(L, dtype)
    torch.cuda.synchronize()
