"""Rows off the cache-line grid: each side of the sizes at which a local step changes its form, every element compared with
the same formula in float64 on the device.

Tolerance: a result is two (plain), three (center) or up to four (momentum, decay) fused multiply-adds, each rounded to 24
bits of a value no larger than the sum of the magnitudes that enter: 4 * 2^-24 of it, doubled."""
import pytest
import torch

from paper_2403_04206_amd import grawa, workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 8 * 2.0 ** -24
MB = 1 << 20


def rows(K, P, dtype, gen, scale):
    """A [K, P] view whose rows are 16 bytes apart from the line grid, sentinels behind every row."""
    per16 = 8 if dtype is torch.bfloat16 else 4
    ld = (P + per16 - 1) // per16 * per16
    if ld * (2 if per16 == 8 else 4) % 128 == 0:
        ld += per16
    t = torch.full((K, ld), 777.0, dtype=dtype, device=DEV)
    t[:, :P].normal_(0.0, scale, generator=gen)
    return t


def close(got, ref, size):
    worst = ((got.double() - ref).abs() / size.clamp_min(1e-30)).max().item()
    assert worst <= TOL, "worst scaled error %.3g" % worst


@pytest.mark.parametrize("step,dtype,mb", [
    ("prox", torch.bfloat16, 120), ("prox", torch.bfloat16, 136), ("prox", torch.float32, 72),
    ("scored", torch.float32, 72), ("scored", torch.float32, 322), ("scored", torch.bfloat16, 72),
    ("nesterov", torch.bfloat16, 130), ("nesterov", torch.bfloat16, 200), ("nesterov", torch.float32, 130)])
def test_local_steps_either_side_of_a_line(step, dtype, mb):
    K = 3
    P = mb * MB // 4 // K // 1024 * 1024 + 3                             # the last vector of a row is partly filled
    gen = torch.Generator(device=DEV).manual_seed(mb)
    x, g = rows(K, P, torch.float32, gen, 0.05), rows(K, P, dtype, gen, 1.0)
    xs, gs, x0 = x[:, :P], g[:, :P], x.clone()
    lr, lr64 = 0.1, float(torch.tensor(0.1))
    if step == "prox":
        cen = torch.empty((P + 3) // 4 * 4, device=DEV).normal_(0.0, 0.05, generator=gen)
        grawa.local_sgd_prox(xs, gs, lr, cen[:P], 0.05, 4.0)
        w = float(torch.tensor(0.05) / torch.tensor(4.0))
    elif step == "scored":
        est = torch.empty((K, 2), device=DEV)
        with grawa.Plan(K, P, [0, P // 3, P]) as plan:
            plan.local_step_scored(xs, gs, lr, 0.9)
            plan.local_lgrawa_update(xs, 0.0, est_out=est)               # lambda = 0: x keeps the step's result
            torch.cuda.synchronize()
        norms = torch.stack([gs[:, a:b].double().norm(dim=1) for a, b in ((0, P // 3), (P // 3, P))], 1)
        # after one step the estimate is gamma times the norm; gamma and the result are rounded to 24 bits
        assert float((est.double() / (0.9 * norms) - 1.0).abs().max()) <= 2.0 ** -23
    else:
        buf = rows(K, P, torch.float32, gen, 0.01)
        b0 = buf.clone()
        grawa.local_nesterov(xs, gs, buf[:, :P], lr, 0.9, 5e-4)
        m, wd = float(torch.tensor(0.9)), float(torch.tensor(5e-4))
    for k in range(K):
        x64, g64 = x0[k, :P].double(), g[k, :P].double()
        size = x64.abs() + lr * g64.abs()
        if step == "prox":
            c64 = cen[:P].double()
            v = x64 - lr64 * g64
            close(x[k, :P], v + w * (c64 - v), size + c64.abs())
        elif step == "scored":
            close(x[k, :P], x64 - lr64 * g64, size)
        else:
            b64 = b0[k, :P].double()
            d = g64 + wd * x64
            nb = m * b64 + d
            close(buf[k, :P], nb, b64.abs() + g64.abs() + x64.abs())
            close(x[k, :P], x64 - lr64 * (d + m * nb), size + 2 * lr * (b64.abs() + g64.abs()))
            assert (buf[k, P:] == 777.0).all()
        assert (x[k, P:] == 777.0).all()


# Each number of wave groups (2, 4, 8) with and without the guarded row, the first and last worker count of each, and the
# neighbours of the dispatch's lines (5/6, 9/10, 11/12, 15/16, 23/24, 71/72).
@pytest.mark.parametrize("K", [3, 5, 6, 9, 10, 11, 12, 15, 16, 19, 23, 24, 25, 40, 63, 71, 72])
@pytest.mark.parametrize("kind,mb", [("pull", 130), ("pull", 322), ("easgd", 130), ("easgd", 322), ("f32", 130), ("bf16", 130)])
def test_pull_of_rows_off_the_grid(K, kind, mb):
    # cells of one layer, of 2 to 8 and of 256, a boundary on a cell's edge; the row ends inside a lane, a cell and a block.
    # 130 MB and 322 MB: either side of the line from which the counts of bursts alone take them without the step
    P = (mb * MB) // (4 * K) // 2048 * 2048 + 2048 + 256 * (K % 5) + 1 + K % 3
    sizes = [256, 100, 412] + [32] * 8 + [1] * 256 + [300] * 200
    sizes += [P - sum(sizes) - 130, 120, 10]
    L, gen = len(sizes), torch.Generator(device=DEV).manual_seed(K)
    off = torch.tensor([0] + sizes).cumsum(0)
    x = rows(K, P, torch.float32, gen, 0.05)
    x0, lam = x.clone(), 0.25
    cen = torch.full(((P + 7) // 4 * 4,), 777.0, device=DEV)
    layer = torch.repeat_interleave(torch.arange(L, device=DEV), torch.tensor(sizes, device=DEV))
    lr = 0.0
    with grawa.Plan(K, P, off.numpy()) as plan:
        if kind == "pull":
            beta = torch.rand((K, L), device=DEV, generator=gen)
            plan.center_pull(x[:, :P], beta, lam, center_out=cen[:P])
        elif kind == "easgd":
            cen[:P].normal_(0.0, 0.05, generator=gen)
            c0, beta = cen[:P].double(), torch.full((K, L), 1.0 / K, device=DEV)
            plan.easgd_update(x[:, :P], lam, 0.5, cen[:P])
        else:
            lr = 0.1
            g = rows(K, P, torch.float32 if kind == "f32" else torch.bfloat16, gen, 1.0)
            beta = torch.zeros((K, L), device=DEV)
            plan.lgrawa_update_sgd(x[:, :P], g[:, :P], lam, g[:, :P], lr, center_out=cen[:P], weights_out=beta)
    lr64 = float(torch.tensor(lr))
    size, c = torch.zeros(P, dtype=torch.float64, device=DEV), torch.zeros(P, dtype=torch.float64, device=DEV)
    moved = lambda k: x0[k, :P].double() - lr64 * g[k, :P].double() if lr else x0[k, :P].double()
    for k in range(K):
        v, b = moved(k), beta[k].double()[layer]
        c += b * v
        size = torch.maximum(size, (x0[k, :P].double().abs() + (lr * g[k, :P].double().abs() if lr else 0.0)) * (b * K).clamp_min(1.0))
    if kind == "easgd":
        c = c0 + 0.5 * (c - c0)
        size = torch.maximum(size, c0.abs())
    # the step, K products and sums and the pull, each rounded to 24 bits of a value no larger than K / K of the largest term
    tol = (K + 5) * 2.0 ** -24
    assert float(((cen[:P].double() - c).abs() / size.clamp_min(1e-30)).max()) <= tol
    for k in range(K):
        v = moved(k)
        assert float(((x[k, :P].double() - (v + lam * (c - v))).abs() / size.clamp_min(1e-30)).max()) <= 2 * tol
    assert (x[:, P:] == 777.0).all() and (cen[P:] == 777.0).all()


# A fused pull streams by the size of x and g together (128 MB), with the plain form's cap on cached accesses from 64 MB on
# where rows are off the grid: either side of both lines, for a cap of 2 (17 workers) and of 5 or 4 waves.
@pytest.mark.parametrize("K", [4, 6, 17, 24])
@pytest.mark.parametrize("dtype,mb", [("f32", 60), ("f32", 68), ("bf16", 40), ("bf16", 80), ("bf16", 90)])
@pytest.mark.parametrize("pad", [0, 8])
def test_fused_pull_either_side_of_the_lines(K, dtype, mb, pad):
    P = mb * MB // 4 // K // 1024 * 1024 + 5
    w = W.Workload("fused_K%d" % K, K, [P // 3, 1, 700, P - P // 3 - 701], grad_dtype=dtype, lam=0.25, lr=0.1, seed=(9, K + mb))
    x, g = W.make_inputs(w, device=DEV, ld_pad=pad)
    x0 = x.clone()
    cen = torch.empty(W.round_up(P, 4), device=DEV)
    beta = torch.zeros((K, w.L), device=DEV)
    with grawa.Plan(K, P, w.offsets) as plan:
        plan.lgrawa_update_sgd(x[:, :P], g[:, :P], 0.25, g[:, :P], 0.1, center_out=cen, weights_out=beta)
        torch.cuda.synchronize()
    layer = torch.repeat_interleave(torch.arange(w.L, device=DEV), torch.tensor(w.offsets, device=DEV).diff())
    lr = float(torch.tensor(0.1))
    c, size = torch.zeros(P, dtype=torch.float64, device=DEV), torch.zeros(P, dtype=torch.float64, device=DEV)
    for k in range(K):
        b = beta[k].double()[layer]
        c += b * (x0[k, :P].double() - lr * g[k, :P].double())
        size = torch.maximum(size, (x0[k, :P].double().abs() + lr * g[k, :P].double().abs()) * (b * K).clamp_min(1.0))
    tol = (K + 5) * 2.0 ** -24                           # as in the test above
    assert float(((cen[:P].double() - c).abs() / size.clamp_min(1e-30)).max()) <= tol
    for k in range(K):
        v = x0[k, :P].double() - lr * g[k, :P].double()
        assert float(((x[k, :P].double() - (v + 0.25 * (c - v))).abs() / size.clamp_min(1e-30)).max()) <= 2 * tol
    assert torch.equal(x[:, P:], x0[:, P:])
