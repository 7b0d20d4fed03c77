"""The allocation-free update where its kernels find tiles and cells in the layer offsets themselves: layer counts either
side of a round of that search (64 places) and of the most it is used for, layers that start on multiples of the tile, cells of one and of 256
layers, and the first size that takes the maps; bit for bit the plan's results."""
import pytest

from paper_2403_04206_amd import workloads as W
from test_zz_no_alloc import both_ways

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("K,sizes", [
    (4, [300] * 64), (4, [300] * 65), (1, [3] * 2560), (1, [3] * 2561), (2, [3] * 1281), (3, [1] * 700 + [9000] + [2] * 100),
    (8, [4096, 4096, 8192, 1, 4095, 12288, 5]), (15, [256] * 40 + [1] * 256 + [255, 257]), (1, [20000]),
    (4, [655360 - 300, 300]), (4, [655361 - 300, 300])])                 # 2560 and 2561 cells: the last without maps, the first with
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_static_without_maps(K, sizes, dtype):
    w, x, g = W.make_small(900 + K, K, sizes, grad_dtype=dtype, ld_pad=8, device=DEV)
    both_ways(w, x, g, 0.3)
