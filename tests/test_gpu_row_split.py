"""GPU parity of the row-split center+pull kernels: the worker counts where the number of rows per wave group
changes (multiples of 8 and their neighbours, the first and last of the range), an odd number of columns,
layer boundaries inside cells, cached and streaming accesses."""
import pytest
import torch

from paper_2403_04206_amd import workloads as W
from test_gpu_full_configs import run_workload
from test_gpu_parity import run_variant

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SIZES = [1, 3, 2049, 2, 5, 255, 4000, 7, 257]                # P odd: the last lane holds a single column


@pytest.mark.parametrize("K", [16, 23, 24, 25, 31, 39, 47, 48, 55, 63, 71, 72])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ld_pad", [0, 8])
def test_row_split_worker_counts(K, dtype, ld_pad):
    w, x, g = W.make_small(1300 + K, K, SIZES, grad_dtype=dtype, ld_pad=ld_pad, device=DEV)
    assert w.P % 2 == 1
    run_variant(w, x, g, "lgrawa", 0.3)
    run_variant(w, x, g, "mgrawa", 0.3)
    run_variant(w, x, g, "lgrawa", 0.25, fused=True, lr=0.1)


@pytest.mark.parametrize("K,dtype,fused", [(24, "f32", False), (43, "bf16", True), (33, "f32", True)])
def test_row_split_streaming(K, dtype, fused):
    # arrays over 512 MB on line-aligned rows: the streaming instantiations
    P = (560 << 20) // (4 * K) | 1
    w = W.Workload("split_K%d" % K, K, [P // 3, 5, P - P // 3 - 5], grad_dtype=dtype, lam=0.1, lr=0.1, fused_sgd=fused,
                   variants=("lgrawa",), seed=(4, K))
    run_workload(w, "lgrawa", "chunks", 40 + K)
    torch.cuda.empty_cache()
