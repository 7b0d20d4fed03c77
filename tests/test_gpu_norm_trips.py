"""Gradient norms at the lengths where the last trip of the norm pass changes its number of loads (1, 2, 4 or 8 of
256 lanes of 8 bytes, fp32 and bf16), one value to either side, at every alignment of the layer's start."""
import pytest
import torch

from oracle import grawa_oracle as orc
from paper_2403_04206_amd import grawa, workloads as W
from parity_util import TIGHT, assert_table_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("lead", [0, 1, 2, 3])
def test_norms_at_trip_edges(dtype, lead):
    per = 512 if dtype == "f32" else 1024                # values of one load of all lanes
    edges = [n * per + d for n in (1, 2, 3, 4, 5, 7, 8) for d in (-1, 0, 1)]
    sizes = ([lead] if lead else []) + edges + [4096, 4097, 16384, 1]
    w, x, g = W.make_small(3000 + lead, 3, sizes, grad_dtype=dtype, device=DEV)
    with grawa.Plan(w.K, w.P, w.offsets) as plan:
        A = plan.grad_norms(g[:, :w.P])
        torch.cuda.synchronize()
    ref = orc.layer_norms(orc.grad_sumsq(W.to_numpy_grads(g), w.offsets))
    worst = assert_table_close(A.cpu().numpy(), ref, TIGHT, "norms")
    assert worst < 2e-7                                  # squares and sums in fp64, one rounding to the float32 table
