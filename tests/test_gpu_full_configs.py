"""GPU parity at the full benchmark sizes (configurations 1-4), in the launch configuration
the benchmark times (streaming accesses of the pull above 128 MB of parameters, i.e. all four).

The norm and weight tables are compared in full (the CPU reference streams every gradient
element), and so are the pulled parameters and the center: EVERY element of x (K x P) and of the
center (P) is compared with the reference.  For configurations 2-4 the arrays are walked in
chunks of 2 M columns copied from the device one at a time and handed to a pool of host threads,
each of which calls the reference for its chunk (a sub-problem with the chunk's layers and their
weights) and applies the comparison rule, so host memory holds a few chunks, not the arrays.
Two properties that hold for every element at any size are evaluated over the whole arrays on
the device as well: differences between workers contract by exactly (1 - lambda), and the
weighted sum of the pulled workers reproduces the stored center.  The calls of the other rows
(local round, Nesterov, EASGD, LSGD) at these sizes are compared on sampled column windows.
"""
import os
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

from oracle import grawa_oracle as orc
from paper_2403_04206_amd import grawa, workloads as W
from parity_util import TIGHT, assert_params_close, assert_table_close, grads_to_f64, operand_scale

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
WINDOW = 4096


def say(msg):
    print("[case] " + msg, flush=True)


def sample_windows(w, rng, n_random=24):
    P, off = w.P, w.offsets
    starts = {0, max(0, P - WINDOW)}
    for l in rng.choice(w.L, size=min(w.L, 12), replace=False):       # layer boundaries
        starts.add(int(max(0, min(P - WINDOW, off[l] - WINDOW // 2))))
    small = np.argsort(np.diff(off))[:4]                                # the smallest layers
    for l in small:
        starts.add(int(max(0, min(P - WINDOW, off[l] - 100))))
    for t in rng.integers(1, max(2, P // 8192), size=6):               # tile boundaries
        starts.add(int(max(0, min(P - WINDOW, t * 8192 - WINDOW // 2))))
    for s in rng.integers(0, max(1, P - WINDOW), size=n_random):
        starts.add(int(s))
    return sorted(starts)


def window_reference(w, beta, x0, g, i0, i1, lam, fused, lr):
    """Reference for columns [i0, i1): a sub-problem with the window's layers and their weights."""
    off = w.offsets
    xs = np.ascontiguousarray(x0[:, i0:i1].cpu().numpy())
    per_layer = beta.ndim == 2
    if per_layer:
        l0 = int(np.searchsorted(off, i0, side="right") - 1)
        l1 = int(np.searchsorted(off, i1, side="left"))
        sub_off = np.clip(off[l0:l1 + 1], i0, i1) - i0
        b = np.ascontiguousarray(beta[:, l0:l1])
    else:
        sub_off = np.array([0, i1 - i0], dtype=np.int64)
        b = beta
    kw = {}
    gs = None
    if fused:
        gs = W.to_numpy_grads(g[:, i0:i1].contiguous())
        kw = dict(g_sgd=gs, lr=lr)
    rx, rc = orc.center_pull(xs, b, sub_off, lam, **kw)
    return rx, rc, operand_scale(xs, gs, lr)


CHUNK = 1 << 21
POOL = max(1, min(8, (os.cpu_count() or 2) - 1))


def compare_every_element(w, beta, x0, x, g, cen, lam, fused, lr):
    """x0: inputs, x: outputs, g: gradients, cen: stored center (device tensors).  Every column chunk
    is copied to the host, recomputed by the reference and compared; returns the elements compared."""
    P, K, off = w.P, w.K, w.offsets
    per_layer = beta.ndim == 2

    def job(i0, i1, xs, gs, got, cgot):
        if per_layer:
            l0 = int(np.searchsorted(off, i0, side="right") - 1)
            l1 = int(np.searchsorted(off, i1, side="left"))
            sub_off = np.clip(off[l0:l1 + 1], i0, i1) - i0
            b = np.ascontiguousarray(beta[:, l0:l1])
        else:
            sub_off = np.array([0, i1 - i0], dtype=np.int64)
            b = beta
        kw = dict(g_sgd=gs, lr=lr) if fused else {}
        rx, rc = orc.center_pull(xs, b, sub_off, lam, chunk=1 << 19, **kw)
        sc = operand_scale(xs, gs, lr)
        assert_params_close(got, rx, off, TIGHT, "x [%d,%d)" % (i0, i1), sc, col0=i0)
        assert_params_close(cgot, rc, off, TIGHT, "center [%d,%d)" % (i0, i1), sc, col0=i0)
        return got.size + cgot.size

    done = 0
    pending = []
    with ThreadPoolExecutor(max_workers=POOL) as pool:
        for i0 in range(0, P, CHUNK):
            i1 = min(P, i0 + CHUNK)
            xs = np.ascontiguousarray(x0[:, i0:i1].cpu().numpy())
            gs = W.to_numpy_grads(g[:, i0:i1].contiguous()) if fused else None
            got = x[:, i0:i1].cpu().numpy()
            cgot = cen[i0:i1].cpu().numpy()
            pending.append(pool.submit(job, i0, i1, xs, gs, got, cgot))
            while len(pending) >= 2 * POOL:              # bound the chunks held in host memory
                done += pending.pop(0).result()
        for f in pending:
            done += f.result()
    assert done == K * P + P
    return done


def run_full(cfg_index, variant, full_compare):
    run_workload(W.config(cfg_index), variant, full_compare, cfg_index)


def run_workload(w, variant, full_compare, cfg_index):
    P, K = w.P, w.K
    fused = w.fused_sgd
    lr = w.lr if fused else 0.0
    say("%s (%d) %s K=%d L=%d P=%d grads=%s fused_sgd=%s" % (w.name, cfg_index, variant, K, w.L, P, w.grad_dtype, fused))
    x, g = W.make_inputs(w, device=DEV)
    x0 = x.clone()
    per_layer = variant == "lgrawa"
    cen = torch.empty(W.round_up(P, 4), device=DEV)
    wts = torch.empty((K, w.L) if per_layer else (K,), device=DEV)
    with grawa.Plan(K, P, w.offsets) as plan:
        norms = plan.grad_norms(g[:, :P])
        xv = x[:, :P]
        if per_layer and fused:
            plan.lgrawa_update_sgd(xv, g[:, :P], w.lam, g[:, :P], lr, center_out=cen, weights_out=wts)
        elif per_layer:
            plan.lgrawa_update(xv, g[:, :P], w.lam, center_out=cen, weights_out=wts)
        elif fused:
            plan.mgrawa_update_sgd(xv, g[:, :P], w.lam, g[:, :P], lr, center_out=cen, weights_out=wts)
        else:
            plan.mgrawa_update(xv, g[:, :P], w.lam, center_out=cen, weights_out=wts)
        torch.cuda.synchronize()
    say("gpu done; reference norms over %d elements" % (K * P))

    # full tables
    gh = W.to_numpy_grads(g)
    S = orc.grad_sumsq(gh, w.offsets)
    del gh
    A = orc.layer_norms(S)
    assert_table_close(norms.cpu().numpy(), A, TIGHT, "norms")
    beta = orc.weights(A) if per_layer else orc.weights(orc.model_norms(S, "layersum"))
    assert_table_close(wts.cpu().numpy(), beta, TIGHT, "beta")
    if w.tiny_worker is not None and per_layer:
        assert np.all(beta[w.tiny_worker] > 0.95)      # the 1e-6-scale worker dominates every layer

    # properties over every element, on the device
    lam = w.lam
    xs0 = x0[:, :P]
    if fused:
        xs0 = xs0 - lr * g[:, :P].float()
    scale = xs0.abs().max().item()
    for m in range(1, K):
        d = ((x[m, :P] - x[0, :P]) - (1.0 - lam) * (xs0[m] - xs0[0])).abs().max().item()
        assert d <= 4e-6 * scale, "contraction property, worker %d: %g" % (m, d)
    layer_of = torch.repeat_interleave(torch.arange(w.L, device=DEV), torch.from_numpy(np.diff(w.offsets)).to(DEV))
    bt = wts if per_layer else wts[:, None].expand(K, w.L)
    acc = torch.zeros(P, device=DEV, dtype=torch.float64)
    for m in range(K):
        acc += bt[m][layer_of].double() * x[m, :P].double()
    d = (acc - cen[:P].double()).abs().max().item()
    assert d <= 1e-5 * scale, "fixed-point property: %g" % d
    del acc, layer_of, xs0
    say("properties ok; element-wise comparison")

    if full_compare == "chunks":
        n = compare_every_element(w, beta, x0, x, g, cen, lam, fused, lr)
        say("compared %d elements of x and center with the reference" % n)
    elif full_compare:
        xh = W.to_numpy_params(x0)
        gh = W.to_numpy_grads(g)
        got = x.cpu().numpy()
        cgot = cen.cpu().numpy()
        kw = dict(g_sgd=gh, lr=lr) if fused else {}
        for i0, i1, xd, c in orc.update_chunks(xh, beta, w.offsets, lam, chunk=1 << 21, **kw):
            sc = operand_scale(xh[:, i0:i1], gh[:, i0:i1] if fused else None, lr)
            assert_params_close(got[:, i0:i1], xd, w.offsets, TIGHT, "x", sc, col0=i0)
            assert_params_close(cgot[i0:i1], c, w.offsets, TIGHT, "center", sc, col0=i0)
    else:
        rng = np.random.default_rng(cfg_index)
        for i0 in sample_windows(w, rng):
            i1 = min(P, i0 + WINDOW)
            rx, rc, sc = window_reference(w, beta, x0, g, i0, i1, lam, fused, lr)
            assert_params_close(x[:, i0:i1].cpu().numpy(), rx, w.offsets, TIGHT, "x window %d" % i0, sc, col0=i0)
            assert_params_close(cen[i0:i1].cpu().numpy(), rc, w.offsets, TIGHT, "center window %d" % i0, sc, col0=i0)
    # padding columns untouched
    assert torch.equal(x[:, P:], x0[:, P:])


@pytest.mark.parametrize("variant", ["mgrawa", "lgrawa"])
def test_config1_full(variant):
    run_full(1, variant, full_compare=True)
    # the configuration also takes one local SGD step (lr 0.1)
    if variant == "lgrawa":
        w = W.config(1)
        x, g = W.make_inputs(w, device=DEV)
        xh, gh = W.to_numpy_params(x), W.to_numpy_grads(g)
        grawa.local_sgd(x[:, :w.P], g[:, :w.P], w.lr)
        torch.cuda.synchronize()
        got = x.cpu().numpy()
        for i0 in range(0, w.P, 1 << 22):
            i1 = min(w.P, i0 + (1 << 22))
            ref = orc.local_sgd(np.ascontiguousarray(xh[:, i0:i1]), np.ascontiguousarray(gh[:, i0:i1]), w.lr)
            assert_params_close(got[:, i0:i1], ref, w.offsets, TIGHT, "local_sgd",
                                operand_scale(xh[:, i0:i1], gh[:, i0:i1], w.lr), col0=i0)


def test_config2_wrn_lgrawa():
    run_full(2, "lgrawa", full_compare="chunks")


@pytest.mark.parametrize("variant", ["mgrawa", "lgrawa"])
def test_config3_transformer_bf16(variant):
    run_full(3, variant, full_compare="chunks")


def test_config4_resnet50_fused_sgd():
    run_full(4, "lgrawa", full_compare="chunks")


def test_config2_local_round_full_size():
    """Appendix G round at the size of configuration 2: two scored local steps with the proximity
    step, then the LGRAWA communication from the running estimate.  Estimate and weight tables are
    compared in full, parameters on sampled windows."""
    w = W.config(2)
    P, K, L = w.P, w.K, w.L
    lr, lam, gamma, mu, tau = 0.05, w.lam, 0.9, 0.05, 16.0
    say("config 2 local round K=%d L=%d P=%d" % (K, L, P))
    x, g1 = W.make_inputs(w, device=DEV)
    w2 = W.config(2)
    w2.seed = (0, 22)
    _, g2 = W.make_inputs(w2, device=DEV)
    x0 = x.clone()
    cprev = 0.05 * torch.randn(W.round_up(P, 256), device=DEV, generator=torch.Generator(device=DEV).manual_seed(3))
    cen = torch.empty(W.round_up(P, 4), device=DEV)
    wts = torch.empty((K, L), device=DEV)
    est = torch.empty((K, L), device=DEV)
    with grawa.Plan(K, P, w.offsets) as plan:
        plan.local_step_scored(x[:, :P], g1[:, :P], lr, gamma, center=cprev, mu=mu, tau=tau)
        plan.local_step_scored(x[:, :P], g2[:, :P], lr, gamma, center=cprev, mu=mu, tau=tau)
        plan.local_lgrawa_update(x[:, :P], lam, center_out=cen, weights_out=wts, est_out=est)
        torch.cuda.synchronize()
    say("gpu done; reference estimate")
    sc = orc.LocalScores(K, L, gamma)
    sc.step(W.to_numpy_grads(g1), w.offsets)
    sc.step(W.to_numpy_grads(g2), w.offsets)
    assert_table_close(est.cpu().numpy(), sc.g_est, TIGHT, "g_est")
    beta = sc.weights("lgrawa")
    assert_table_close(wts.cpu().numpy(), beta, TIGHT, "beta")
    rng = np.random.default_rng(5)
    off = w.offsets
    for i0 in sample_windows(w, rng, n_random=12):
        i1 = min(P, i0 + WINDOW)
        xs = np.ascontiguousarray(x0[:, i0:i1].cpu().numpy())
        gs = [W.to_numpy_grads(g[:, i0:i1].contiguous()) for g in (g1, g2)]
        cp = cprev[i0:i1].cpu().numpy().astype(np.float64)
        cur = orc.local_sgd(xs, gs[0], lr, prox_center=cp, mu=mu, tau=tau)
        # second step from the float64 state: x - lr g, then the proximity step
        from parity_util import grads_to_f64
        cur = cur - lr * grads_to_f64(gs[1])
        cur = (1.0 - mu / tau) * cur + (mu / tau) * cp
        l0 = int(np.searchsorted(off, i0, side="right") - 1)
        l1 = int(np.searchsorted(off, i1, side="left"))
        layer_of = np.repeat(np.arange(l0, l1), np.diff(np.clip(off[l0:l1 + 1], i0, i1)))
        c = (beta[:, layer_of] * cur).sum(axis=0)
        want = (1.0 - lam) * cur + lam * c
        scale = np.maximum((np.abs(xs.astype(np.float64)) + lr * (np.abs(grads_to_f64(gs[0])) + np.abs(grads_to_f64(gs[1])))).max(axis=0), np.abs(cp))
        assert_params_close(x[:, i0:i1].cpu().numpy(), want, off, TIGHT, "x window %d" % i0, scale, col0=i0)
        assert_params_close(cen[i0:i1].cpu().numpy(), c, off, TIGHT, "center window %d" % i0, scale, col0=i0)
    assert torch.equal(x[:, P:], x0[:, P:])


@pytest.mark.parametrize("cfg_index", [2, 3])
def test_full_size_nesterov_easgd_lsgd(cfg_index):
    # The local optimizer of the experiments (two steps, so the momentum buffer is used) and the two
    # Appendix F phases at the benchmark's sizes, on sampled windows (every step is column-local once
    # the leader / the weights are known).
    w = W.config(cfg_index)
    P, K = w.P, w.K
    say("config %d nesterov/easgd/lsgd K=%d P=%d grads=%s" % (cfg_index, K, P, w.grad_dtype))
    x, g = W.make_inputs(w, device=DEV)
    x0 = x.clone()
    rng = np.random.default_rng(300 + cfg_index)
    wins = sample_windows(w, rng, n_random=10)
    lr, mom, wd, lam, rho = 0.05, 0.9, 5e-4, 0.3, 0.25

    buf = torch.zeros_like(x)
    grawa.local_nesterov(x[:, :P], g[:, :P], buf[:, :P], lr, mom, wd)
    grawa.local_nesterov(x[:, :P], g[:, :P], buf[:, :P], lr, mom, wd)
    torch.cuda.synchronize()
    for i0 in wins:
        i1 = min(P, i0 + WINDOW)
        xs = np.ascontiguousarray(x0[:, i0:i1].cpu().numpy())
        gs = W.to_numpy_grads(g[:, i0:i1].contiguous())
        rx, rb = orc.nesterov_sgd(xs, np.zeros((K, i1 - i0)), gs, lr, mom, wd)
        rx, rb = orc.nesterov_sgd(rx, rb, gs, lr, mom, wd)
        sc = operand_scale(xs, gs, lr * (2 + 3 * mom))
        off = np.array([0, i1 - i0])
        assert_params_close(x[:, i0:i1].cpu().numpy(), rx, off, 2 * TIGHT, "nesterov x [%d,%d)" % (i0, i1), sc)
        sb = (1 + mom) * (np.abs(grads_to_f64(gs)).max(axis=0) + wd * sc)
        assert_params_close(buf[:, i0:i1].cpu().numpy(), rb, off, 2 * TIGHT, "nesterov buf [%d,%d)" % (i0, i1), sb)
    assert torch.equal(x[:, P:], x0[:, P:]) and not buf[:, P:].any()
    del buf

    x.copy_(x0)
    cen = 0.05 * torch.randn(W.round_up(P, 256), device=DEV, generator=torch.Generator(device=DEV).manual_seed(5))
    cen0 = cen.clone()
    losses = torch.rand(K, device=DEV, generator=torch.Generator(device=DEV).manual_seed(6))
    lead = torch.zeros(1, dtype=torch.int32, device=DEV)
    x2 = x0.clone()
    with grawa.Plan(K, P, w.offsets) as plan:
        plan.easgd_update(x[:, :P], lam, rho, cen)
        plan.lsgd_update(x2[:, :P], losses, lam, leader_out=lead)
        torch.cuda.synchronize()
    want_lead = int(np.argmin(losses.cpu().numpy()))
    assert int(lead.item()) == want_lead
    for i0 in wins:
        i1 = min(P, i0 + WINDOW)
        xs = np.ascontiguousarray(x0[:, i0:i1].cpu().numpy())
        off = np.array([0, i1 - i0])
        rx, rc = orc.easgd_update(xs, cen0[i0:i1].cpu().numpy().astype(np.float64), lam, rho)
        sc = np.maximum(operand_scale(xs), np.abs(cen0[i0:i1].cpu().numpy().astype(np.float64)))
        assert_params_close(x[:, i0:i1].cpu().numpy(), rx, off, TIGHT, "easgd x [%d,%d)" % (i0, i1), sc)
        assert_params_close(cen[i0:i1].cpu().numpy(), rc, off, TIGHT, "easgd center [%d,%d)" % (i0, i1), sc)
        rx, _ = orc.lsgd_update(xs, losses.cpu().numpy().astype(np.float64), lam)
        assert_params_close(x2[:, i0:i1].cpu().numpy(), rx, off, TIGHT, "lsgd x [%d,%d)" % (i0, i1), operand_scale(xs))
    assert torch.equal(x2[want_lead], x0[want_lead])          # the leader does not move
    assert torch.equal(x[:, P:], x0[:, P:]) and torch.equal(cen[P:], cen0[P:])


def test_more_than_2_31_columns():
    # 64-bit indexing: a row longer than 2^31 elements, a layer boundary three columns below 2^31, a row
    # length that is not a multiple of 4; fused LGRAWA update with bf16 gradients (x 17 GB, g 8.6 GB).
    free, _ = torch.cuda.mem_get_info()
    if free < 150 * (1 << 30):
        pytest.skip("needs 150 GB of free device memory")
    w = W.Workload("wide_K2", 2, [2 ** 31 - 3, 8200], grad_dtype="bf16", lam=0.3, lr=0.1, fused_sgd=True,
                   variants=("lgrawa",), seed=(2, 1))
    run_workload(w, "lgrawa", False, 99)
    # the row-by-row local steps on the same shape: scored SGD + proximity step, then the communication
    P, K = w.P, w.K
    x, g = W.make_inputs(w, device=DEV)
    x0 = x.clone()
    cen = 0.05 * torch.randn(W.round_up(P, 4), device=DEV, generator=torch.Generator(device=DEV).manual_seed(3))
    est = torch.empty((K, w.L), device=DEV)
    lr, gamma, mu, tau = 0.05, 0.9, 0.05, 16.0
    with grawa.Plan(K, P, w.offsets) as plan:
        plan.local_step_scored(x[:, :P], g[:, :P], lr, gamma, center=cen, mu=mu, tau=tau)
        plan.local_lgrawa_update(x[:, :P], 0.0, est_out=est)       # lambda = 0: x keeps the local step's result
        torch.cuda.synchronize()
    scores = orc.LocalScores(K, w.L, gamma)
    scores.step(W.to_numpy_grads(g), w.offsets)
    assert_table_close(est.cpu().numpy(), scores.g_est, TIGHT, "g_est beyond 2^31")
    for i0 in (0, 2 ** 31 - 2051, 2 ** 31 - 3, P - WINDOW):
        i1 = min(P, i0 + WINDOW)
        xs = np.ascontiguousarray(x0[:, i0:i1].cpu().numpy())
        gs = W.to_numpy_grads(g[:, i0:i1].contiguous())
        ch = cen[i0:i1].cpu().numpy().astype(np.float64)
        ref = orc.local_sgd(xs, gs, lr, prox_center=ch, mu=mu, tau=tau)
        sc = np.maximum(operand_scale(xs, gs, lr), np.abs(ch))
        assert_params_close(x[:, i0:i1].cpu().numpy(), ref, np.array([0, i1 - i0]), TIGHT, "local step [%d,%d)" % (i0, i1), sc)
    assert torch.equal(x[:, P:], x0[:, P:])
