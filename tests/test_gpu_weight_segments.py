"""Weights of the layers inside a cell, by a segment of lanes each up to two rounds of them and by a lane each beyond: either side of that
line for every segment length, with norms of zero (on some workers and on all) and one that is not finite among them; the update with and
without maps, and the communication of a local round, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import grawa_oracle as orc
from paper_2403_04206_amd import grawa, workloads as W
from parity_util import TIGHT, assert_params_close, assert_table_close, operand_scale

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def two_rounds(K):
    G = next(g for g in (1, 2, 4, 8, 16) if g >= K)
    return 4 * (64 // G)


@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 8, 9, 15])
@pytest.mark.parametrize("more", [-1, 0, 1])
def test_layers_inside_a_cell(K, more):
    middle = min(two_rounds(K) + more, 250)
    sizes = [1] * (middle + 1) + [8200 - middle, 3, 2] + [2, 1] * 20 + [300]
    w, x, g = W.make_small(9900 + K, K, sizes, device=DEV)
    P, L = w.P, w.L
    g[0, 3] = 0.0                      # layer 3: worker 0 alone has no gradient; layer 5: nobody
    g[:, 5] = 0.0
    xh, gh = W.to_numpy_params(x), W.to_numpy_grads(g)
    ref = orc.lgrawa_update(xh, gh, w.offsets, 0.3)
    sc = operand_scale(xh[:, :P])
    off = torch.from_numpy(np.asarray(w.offsets, dtype=np.int64)).to(DEV)
    bits = []
    with grawa.Plan(K, P, w.offsets) as plan:
        for maps in (True, False):
            xg, wts = x.clone(), torch.empty((K, L), device=DEV)
            if maps:
                plan.lgrawa_update(xg[:, :P], g[:, :P], 0.3, weights_out=wts)
            else:
                grawa.lgrawa_update_static(xg[:, :P], g[:, :P], off, 0.3, weights_out=wts)
            torch.cuda.synchronize()
            assert_table_close(wts.cpu().numpy(), ref["beta"], TIGHT, "beta")
            assert_params_close(xg.cpu().numpy()[:, :P], ref["x"], w.offsets, TIGHT, "x", sc)
            bits.append((xg, wts))
        assert torch.equal(bits[0][0], bits[1][0]) and torch.equal(bits[0][1], bits[1][1])
        assert plan.nonfinite() == 0
        # one local step: the estimate is the norms, and so are its weights
        est, wts = torch.empty((K, L), device=DEV), torch.empty((K, L), device=DEV)
        xg = x.clone()
        plan.local_step_scored(xg[:, :P], g[:, :P], 0.0, 0.5)
        plan.local_lgrawa_update(xg[:, :P], 0.3, weights_out=wts, est_out=est)
        torch.cuda.synchronize()
        assert_table_close(wts.cpu().numpy(), ref["beta"], TIGHT, "beta of the estimate")
        assert_params_close(xg.cpu().numpy()[:, :P], ref["x"], w.offsets, TIGHT, "x of the estimate", sc)
        assert plan.nonfinite() == 0
        g[K - 1, 4] = float("inf")
        plan.lgrawa_update(xg[:, :P], g[:, :P], 0.3, weights_out=wts)
        assert plan.nonfinite() == grawa.NONFINITE_LAYER_SCORE
        assert K == 1 or float(wts[K - 1, 4]) == 0.0
