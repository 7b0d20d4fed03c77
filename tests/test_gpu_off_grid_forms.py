"""Rows off the cache-line grid: each side of the sizes at which a local step changes its form, every element compared with
the same formula in float64 on the device.

Tolerance: a result is two (plain), three (center) or up to four (momentum, decay) fused multiply-adds, each rounded to 24
bits of a value no larger than the sum of the magnitudes that enter: 4 * 2^-24 of it, doubled."""
import pytest
import torch

from paper_2403_04206_amd import grawa

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
        else:
            b64 = b0[k, :P].double()
            d = g64 + wd * x64
            nb = m * b64 + d
            close(buf[k, :P], nb, b64.abs() + g64.abs() + x64.abs())
            close(x[k, :P], x64 - lr64 * (d + m * nb), size + 2 * lr * (b64.abs() + g64.abs()))
            assert (buf[k, P:] == 777.0).all()
        assert (x[k, P:] == 777.0).all()
