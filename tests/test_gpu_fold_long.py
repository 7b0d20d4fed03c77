"""Scored steps whose tile sums the next launch folds in, where some layers are longer than a wave adds (512 tiles of 1024 columns): in the
step, in a launch of its own and in the launch of the weights, at either side of what each takes; and rows of more than one group of column blocks (with a center from 4096 blocks on), the last one short.  Calls
and replays give the same bits; the estimates and every element of x against float64."""
import numpy as np
import pytest
import torch

from oracle import grawa_oracle as orc
from paper_2403_04206_amd import grawa, workloads as W
from parity_util import TIGHT, assert_table_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
T = 1024
CASES = {
    "the first is long": (5, [600 * T] + [700] * 50, False),
    "one between is long": (5, [700] * 30 + [600 * T + 3] + [700] * 31, False),
    "1024 sums": (8, [600 * T] + [700] * 127, False),
    "1032 sums": (8, [600 * T] + [700] * 128, False),                          # the estimate in a launch of its own
    "eight workers in the weights": (8, [513 * T + 5, 512 * T, 30, 5 * T, 17 * T], True),
    "nine workers": (9, [513 * T, 40, 17 * T], False),
    "4096 tiles": (2, [5, 4096 * T - 5, 7], False),
    "4097 tiles": (2, [5, 4096 * T + 5, 7], False),
    "two are long": (17, [300] * 30 + [513 * T, 600 * T] + [300] * 28, False),
    "three groups": (2, [500 * T] * 16 + [399 * T + 77, 5, 3000], True),
    "three groups, long layers": (3, [5000 * T, 3000 * T - 1, 400 * T + 77, 5], True),
}


@pytest.mark.parametrize("policy", ["lgrawa", "mgrawa"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_long_layers(name, policy):
    K, sizes, prox = CASES[name]
    w, x, g = W.make_small(5200 + K, K, sizes, grad_dtype="bf16" if K == 8 else "f32", device=DEV)
    P, L, lr, gamma, mu, tau, lam = w.P, w.L, 0.05, 0.9, 0.05, 4.0, 0.3
    grads = [g, g.roll(1, 0).contiguous(), g.flip(0).contiguous()]
    cen = torch.empty(W.round_up(P, 4), device=DEV).normal_(0.0, 0.05, generator=torch.Generator(device=DEV).manual_seed(K))
    outs = [(x.clone(), torch.zeros((K, L), device=DEV), torch.zeros((K, L) if policy == "lgrawa" else (K,), device=DEV)) for _ in range(3)]

    def round_(plan, out):
        xs, est, wts = out
        for gs in grads:
            plan.local_step_scored(xs[:, :P], gs[:, :P], lr, gamma, center=cen if prox else None, mu=mu, tau=tau)
        (plan.local_lgrawa_update if policy == "lgrawa" else plan.local_mgrawa_update)(xs[:, :P], lam, est_out=est, weights_out=wts)

    stream = torch.cuda.Stream()
    with grawa.Plan(K, P, w.offsets) as plan, torch.cuda.stream(stream):
        round_(plan, outs[0])
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            round_(plan, outs[1])
        for _ in range(2):
            outs[1][0].copy_(x)
            graph.replay()
        round_(plan, outs[2])                          # and called again after the replays
        torch.cuda.synchronize()
        assert plan.nonfinite() == 0
    for other in outs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(outs[0], other))

    scores = orc.LocalScores(K, L, gamma)
    ref = x[:, :P].double()
    size = ref.abs()
    w64 = float(np.float32(mu) / np.float32(tau))
    for gs in grads:
        scores.step(W.to_numpy_grads(gs), w.offsets)
        ref = ref - float(np.float32(lr)) * gs[:, :P].double()
        if prox:
            ref = ref + w64 * (cen[:P].double() - ref)
        size = size + lr * gs[:, :P].double().abs() + (cen[:P].double().abs() if prox else 0.0)
    assert_table_close(outs[0][1].cpu().numpy(), scores.g_est, TIGHT, "g_est")
    beta = torch.from_numpy(np.asarray(scores.weights(policy))).to(DEV)
    assert_table_close(outs[0][2].cpu().numpy(), beta.cpu().numpy(), TIGHT, "weights")
    if policy == "lgrawa":
        beta = beta.repeat_interleave(torch.from_numpy(np.diff(w.offsets)).to(DEV), dim=1)
    else:
        beta = beta[:, None]
    ref = ref + lam * ((beta * ref).sum(0, keepdim=True) - ref)
    size = size.max(dim=0, keepdim=True).values
    # each step rounds x two or three times to 24 bits, the average of K workers and the pull K + 3 times, the weights once
    bound = (3 * 3 + K + 4) * 2.0 ** -24
    assert float(((outs[0][0][:, :P].double() - ref).abs() / size.clamp_min(1e-30)).max()) <= bound
    assert torch.equal(outs[0][0][:, P:], x[:, P:])
