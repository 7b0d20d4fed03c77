"""GPU parity of the row-by-row local steps on arrays beyond the caches, on line-aligned rows and on rows that are not,
every element of them:
steps with and without the center and the scores, the Nesterov step; odd row ends, a layer boundary inside a block."""
import numpy as np
import pytest
import torch

from oracle import grawa_oracle as orc
from paper_2403_04206_amd import grawa, workloads as W
from parity_util import TIGHT, assert_params_close, assert_table_close, grads_to_f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
COLS = 1 << 16                                           # columns compared with the oracle at each end and around the boundary


def windows(P, at):
    for a in (0, max(0, at - COLS // 2), P - COLS):
        yield a, min(P, a + COLS)


@pytest.mark.parametrize("pad", [0, 8])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("step", ["sgd", "prox", "scored", "scored prox", "nesterov"])
def test_large_row_steps(step, dtype, pad):
    K = 3
    P = (530 << 20) // (4 * K) // 1024 * 1024 + (1 if pad else 3)
    cut = P // 3
    w = W.Workload("steps", K, [cut, P - cut], grad_dtype=dtype, seed=(6, pad + len(step)))
    x, g = W.make_inputs(w, device=DEV, ld_pad=pad)
    x0 = x.clone()
    cen = 0.05 * torch.randn(W.round_up(P, 4), device=DEV, generator=torch.Generator(device=DEV).manual_seed(3))
    lr, gamma, mu, tau = 0.05, 0.9, 0.05, 16.0
    prox = "prox" in step
    buf = None
    if step == "sgd":
        grawa.local_sgd(x[:, :P], g[:, :P], lr)
    elif step == "prox":
        grawa.local_sgd_prox(x[:, :P], g[:, :P], lr, cen, mu, tau)
    elif step == "nesterov":
        buf = 0.01 * torch.randn(x.shape, device=DEV, generator=torch.Generator(device=DEV).manual_seed(4))
        buf0 = buf.clone()
        grawa.local_nesterov(x[:, :P], g[:, :P], buf[:, :P], lr, 0.9, 5e-4)
    else:
        est = torch.empty((K, 2), device=DEV)
        with grawa.Plan(K, P, w.offsets) as plan:
            plan.local_step_scored(x[:, :P], g[:, :P], lr, gamma, center=cen if prox else None, mu=mu, tau=tau)
            plan.local_lgrawa_update(x[:, :P], 0.0, est_out=est)        # lambda = 0: x keeps the step's result
            torch.cuda.synchronize()
        scores = orc.LocalScores(K, 2, gamma)
        scores.step(W.to_numpy_grads(g), w.offsets)
        assert_table_close(est.cpu().numpy(), scores.g_est, TIGHT, "g_est")
    torch.cuda.synchronize()
    for a, b in windows(P, cut):
        xs = np.ascontiguousarray(x0[:, a:b].cpu().numpy())
        gs = W.to_numpy_grads(g[:, a:b].contiguous())
        gabs = np.abs(grads_to_f64(gs))
        if step == "nesterov":
            bs = buf0[:, a:b].cpu().numpy().astype(np.float64)
            ref, ref_b = orc.nesterov_sgd(xs.astype(np.float64), bs, gs, lr, 0.9, 5e-4, P=b - a)
            sb = np.abs(bs) + gabs + np.abs(xs)
            assert_params_close(buf[:, a:b].cpu().numpy(), ref_b, [0, b - a], TIGHT, "buf", sb.max(axis=0))
            sc = (np.abs(xs) + lr * sb * 2).max(axis=0)
        else:
            ch = cen[a:b].cpu().numpy().astype(np.float64) if prox else None
            kw = dict(prox_center=ch, mu=mu, tau=tau) if prox else {}
            ref = orc.local_sgd(xs, gs, lr, **kw)
            sc = (np.abs(xs) + lr * gabs).max(axis=0)
            if prox:
                sc = np.maximum(sc, np.abs(ch))
        assert_params_close(x[:, a:b].cpu().numpy(), ref, [0, b - a], TIGHT, "x [%d,%d)" % (a, b), sc)
    # everywhere, element by element against the same formulas in float64.  Each result is one to three fused
    # multiply-adds of terms of magnitude at most |x| + lr (|g| + |buf|) (with weight decay and momentum, each below 2 of
    # it), rounded to 24 bits each; the center enters with weight mu / tau.
    chunk = 1 << 24
    for k in range(K):
        for a in range(0, P, chunk):
            b = min(P, a + chunk)
            xs, gs = x0[k, a:b].double(), g[k, a:b].double()
            size = xs.abs() + lr * gs.abs()
            if step == "nesterov":
                m, wd = float(np.float32(0.9)), float(np.float32(5e-4))
                d = gs + wd * xs
                bs = m * buf0[k, a:b].double() + d
                want = xs - float(np.float32(lr)) * (d + m * bs)
                bsize = buf0[k, a:b].double().abs() + gs.abs() + wd * xs.abs()
                assert bool(((buf[k, a:b].double() - bs).abs() <= 3 * 2.0 ** -24 * bsize).all())
                size = xs.abs() + 4 * lr * bsize
            else:
                want = xs - float(np.float32(lr)) * gs
                if prox:
                    w_c = float(np.float32(mu) / np.float32(tau))
                    want = want + w_c * (cen[a:b].double() - want)
                    size = size + w_c * cen[a:b].double().abs()
            assert bool(((x[k, a:b].double() - want).abs() <= 4 * 2.0 ** -24 * size).all())
    if buf is not None:
        assert torch.equal(buf[:, P:], buf0[:, P:])
    assert torch.equal(x[:, P:], x0[:, P:])
    torch.cuda.empty_cache()
