"""The scored step in one launch (a block owns a layer of one worker): layer starts and ends at every place of a 16-byte vector,
layers inside one vector, of one trip of a block and of more, and the sizes either side of the rule; three steps with
and without the center against the oracle's running estimate, every element of x in float64."""
import numpy as np
import pytest
import torch

from oracle import grawa_oracle as orc
from paper_2403_04206_amd import grawa, workloads as W
from parity_util import TIGHT, assert_table_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
RAGGED = [1, 1, 2, 1, 3, 4, 5, 6, 7, 9, 2, 1, 63, 1021, 4, 5119, 5122, 33]
CASES = [(2, RAGGED), (5, RAGGED + [7000]),                              # up to 7 tiles of 1024 columns,
         (16, [10 * 1024] + [300] * 40), (3, [1] * 640 + [10 * 1024]),
         (3, RAGGED + [8100, 2]),
         (3, RAGGED + [10239, 2]), (3, RAGGED + [12001, 2]), (2, RAGGED + [20481, 40963]),
         (4, [40000, 9000, 1]), (1, [40 * 1024, 5]), (1, [40 * 1024 + 1, 5]),
         (16, [700] * 160), (16, [700] * 161), (10, [11 * 1024] + [300] * 63), (10, [11 * 1024] + [300] * 64),
         (4, [8000] * 99 + [9 * 1024 + 2]), (4, [8000] * 99 + [10 * 1024 + 2])]  # 10 where there are many columns; beyond, blocks of 1024 columns


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("prox", [False, True])
def test_scored_step_by_layers(case, dtype, prox):
    K, sizes = CASES[case]
    w, x, g = W.make_small(3100 + case, K, sizes, grad_dtype=dtype, ld_pad=8 * (case % 2), device=DEV)
    P, L = w.P, w.L
    cen = torch.empty(W.round_up(P, 4), device=DEV).normal_(0.0, 0.05, generator=torch.Generator(device=DEV).manual_seed(case))
    lr, gamma, mu, tau = 0.05, 0.9, 0.05, 16.0
    x0 = x.clone()
    est, wts = torch.empty((K, L), device=DEV), torch.empty((K, L), device=DEV)
    scores = orc.LocalScores(K, L, gamma)
    ref = x0[:, :P].double()
    size = ref.abs()
    lr64, w64 = float(np.float32(lr)), float(np.float32(mu) / np.float32(tau))
    with grawa.Plan(K, P, w.offsets) as plan:
        for _ in range(3):
            plan.local_step_scored(x[:, :P], g[:, :P], lr, gamma, center=cen if prox else None, mu=mu, tau=tau)
            scores.step(W.to_numpy_grads(g), w.offsets)
            ref = ref - lr64 * g[:, :P].double()
            if prox:
                ref = ref + w64 * (cen[:P].double() - ref)
            size = size + lr * g[:, :P].double().abs() + (cen[:P].double().abs() if prox else 0.0)
        # two or three roundings to 24 bits a step, of values no larger than `size`
        assert float(((x[:, :P].double() - ref).abs() / size.clamp_min(1e-30)).max()) <= 3 * 3 * 2.0 ** -24
        assert torch.equal(x[:, P:], x0[:, P:])
        plan.local_lgrawa_update(x[:, :P], 0.0, weights_out=wts, est_out=est)
        torch.cuda.synchronize()
    assert_table_close(est.cpu().numpy(), scores.g_est, TIGHT, "g_est")
