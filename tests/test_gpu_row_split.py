"""GPU parity of the row-split center+pull kernels: the worker counts where the number of rows per wave group
changes (multiples of 8 and their neighbours, the first and last of the range), an odd number of columns,
layer boundaries inside cells, cached and streaming accesses."""
import pytest
import torch

from paper_2403_04206_amd import grawa, workloads as W
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


@pytest.mark.parametrize("K", [24, 25, 31, 32, 33, 40])
@pytest.mark.parametrize("cells", [800, 801])
def test_either_side_of_few_cells(K, cells):
    # up to 800 cells the plain form serves up to 32 workers; cells with one, two, a few and many layers
    P = cells * 256 - 3
    many = [5] * 100 + [1] * 30
    sizes = [P // 2] + many + [P - P // 2 - sum(many) - 2000, 2000]
    w, x, g = W.make_small(1500 + K, K, sizes, device=DEV)
    run_variant(w, x, g, "lgrawa", 0.3)
    run_variant(w, x, g, "mgrawa", 0.3)
    _, _, gb = W.make_small(1600 + K, K, sizes, grad_dtype="bf16", device=DEV)
    wb = W.Workload("bf16", K, sizes, grad_dtype="bf16", seed=(7, K))
    run_variant(wb, x, gb, "lgrawa", 0.25, fused=True, lr=0.1)


@pytest.mark.parametrize("K,dtype,fused", [(24, "f32", False), (43, "bf16", True), (33, "f32", True)])
def test_row_split_streaming(K, dtype, fused):
    # arrays over 512 MB on line-aligned rows: the streaming instantiations
    P = (560 << 20) // (4 * K) | 1
    w = W.Workload("split_K%d" % K, K, [P // 3, 5, P - P // 3 - 5], grad_dtype=dtype, lam=0.1, lr=0.1, fused_sgd=fused,
                   variants=("lgrawa",), seed=(4, K))
    run_workload(w, "lgrawa", "chunks", 40 + K)
    torch.cuda.empty_cache()


# Rows on the line grid: one cell a block; 8 elements off it: 8 cells a block (6 workers), 4 (10 and 16) and 2 (24 and 25).
@pytest.mark.parametrize("K,pad", [(16, 0), (24, 0), (6, 8), (10, 8), (16, 8), (24, 8), (25, 8)])
def test_row_split_second_launch(K, pad):
    # 2^18 cells are one launch; one column more starts a second.  The caller's weights, so that x is the only large array.
    for P in ((1 << 26) + 1, (1 << 26) + 256 + 1):
        x = torch.empty((K, W.round_up(P, 256) + pad), device=DEV).normal_(0.0, 0.05, generator=torch.Generator(device=DEV).manual_seed(K))
        x0 = x.clone()
        off = [0, P // 2 + 3, P]
        beta = torch.rand((K, 2), device=DEV, generator=torch.Generator(device=DEV).manual_seed(P))
        cen = torch.empty(W.round_up(P, 4), device=DEV)
        with grawa.Plan(K, P, off) as plan:
            plan.center_pull(x[:, :P], beta, 0.25, center_out=cen)
            torch.cuda.synchronize()
        step = 1 << 22
        for a in range(0, P, step):
            b = min(P, a + step)
            xd = x0[:, a:b].double()
            cut = min(max(off[1], a), b)
            c = torch.cat([(beta[:, :1].double() * xd[:, :cut - a]).sum(0), (beta[:, 1:].double() * xd[:, cut - a:]).sum(0)])
            # K products and sums of at most 0.5 in all, each rounded to 24 bits, and the pull
            bound = (K + 3) * 2.0 ** -24 * (xd.abs().max() * (1.0 + beta.double().sum(0).max()))
            assert float((cen[a:b].double() - c).abs().max()) <= float(bound)
            assert float((x[:, a:b].double() - (xd + 0.25 * (c - xd))).abs().max()) <= float(bound)
        assert torch.equal(x[:, P:], x0[:, P:])
        del x, x0, cen
        torch.cuda.empty_cache()
