"""GPU parity of the center+pull forms with 16-byte lanes on arrays beyond the last-level cache: rows that do not start on cache-line
boundaries (a plain [K, P] tensor) as the wide form (up to 5 workers, with the fp32 step also 12 and 23) and as row-split bursts
(6, 16 and 24 workers, 23 without the step), and line-aligned rows of one and two workers (the wide form)."""
import pytest
import torch

from paper_2403_04206_amd import grawa, workloads as W
from test_gpu_full_configs import compare_every_element
from oracle import grawa_oracle as orc
from parity_util import TIGHT, assert_table_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("K,pad", [(1, 0), (2, 8), (4, 8), (5, 8), (16, 8)])
def test_16_byte_lanes_with_layers_in_every_cell(K, pad):
    # cells of 2, 8, 9 and 256 layers and one that ends with the row: weights by scalar loads, and by column
    P = (140 << 20) // (4 * K) // 256 * 256 + 129
    sizes = [100, 412] + [32] * 8 + [29] * 8 + [24] + [1] * 256 + [7] * 500 + [300] * 2000
    sizes += [P - sum(sizes) - 130, 120, 10]
    off = torch.tensor([0] + sizes).cumsum(0).tolist()
    L = len(sizes)
    gen = torch.Generator(device=DEV).manual_seed(K)
    x = torch.empty((K, W.round_up(P, 256) + pad), device=DEV).normal_(0.0, 0.05, generator=gen)
    x0 = x.clone()
    beta = torch.rand((K, L), device=DEV, generator=gen)
    cen = torch.empty(W.round_up(P, 4), device=DEV)
    with grawa.Plan(K, P, off) as plan:
        plan.center_pull(x[:, :P], beta, 0.25, center_out=cen)
        torch.cuda.synchronize()
    layer = torch.repeat_interleave(torch.arange(L, device=DEV), torch.tensor(sizes, device=DEV))
    c = torch.zeros(P, dtype=torch.float64, device=DEV)
    for k in range(K):
        c += beta[k].double()[layer] * x0[k, :P].double()
    # K products and sums of magnitude at most max|x| sum(beta), each rounded to 24 bits, and the pull
    bound = (K + 3) * 2.0 ** -24 * float(x0.abs().max()) * (1.0 + K)
    assert float((cen[:P].double() - c).abs().max()) <= bound
    for k in range(K):
        xd = x0[k, :P].double()
        assert float((x[k, :P].double() - (xd + 0.25 * (c - xd))).abs().max()) <= bound
    assert torch.equal(x[:, P:], x0[:, P:])
    torch.cuda.empty_cache()


@pytest.mark.parametrize("K,dtype,fused,tail,pad", [(1, "f32", False, 3, 8), (2, "f32", False, 1, 8), (5, "bf16", True, 3, 8),
                                                    (6, "f32", False, 2, 8), (12, "f32", True, 0, 8), (23, "bf16", False, 2, 8),
                                                    (23, "f32", True, 1, 8), (24, "f32", False, 1, 8), (1, "bf16", True, 1, 0),
                                                    (1, "f32", True, 2, 0), (2, "f32", False, 3, 0), (2, "bf16", True, 1, 0)])
def test_16_byte_lanes(K, dtype, fused, tail, pad):
    P = (530 << 20) // (4 * K) // 1024 * 1024 + 1024 - 300 + tail       # the last block is partly empty, its last lane too
    w = W.Workload("tight_K%d" % K, K, [P // 3, 1, 5, P - P // 3 - 6], grad_dtype=dtype, lam=0.1, lr=0.1, seed=(5, K))
    x, g = W.make_inputs(w, device=DEV, ld_pad=pad)
    assert bool(x.stride(0) % 32) == bool(pad)
    x0, lr = x.clone(), w.lr if fused else 0.0
    cen = torch.empty(W.round_up(P, 4), device=DEV)
    wts = torch.empty((K, w.L), device=DEV)
    with grawa.Plan(K, P, w.offsets) as plan:
        if fused:
            plan.lgrawa_update_sgd(x[:, :P], g[:, :P], w.lam, g[:, :P], lr, center_out=cen, weights_out=wts)
        else:
            plan.lgrawa_update(x[:, :P], g[:, :P], w.lam, center_out=cen, weights_out=wts)
        torch.cuda.synchronize()
    beta = orc.weights(orc.layer_norms(orc.grad_sumsq(W.to_numpy_grads(g), w.offsets)))
    assert_table_close(wts.cpu().numpy(), beta, TIGHT, "beta")
    compare_every_element(w, beta, x0, x, g, cen, w.lam, fused, lr)
    assert torch.equal(x[:, P:], x0[:, P:])
    if fused:
        return
    # the moving center reads the previous one where the fixed center only writes it
    xa, xb = x0.clone(), x0.clone()
    ca, cb = cen.clone(), cen.clone()
    with grawa.Plan(K, P, w.offsets) as plan:
        plan.easgd_update(xa[:, :P], 0.3, 1.0, ca)                      # rho = 1: the plain average
        plan.center_pull(xb[:, :P], torch.full((K,), 1.0 / K, device=DEV), 0.3, center_out=cb)
        torch.cuda.synchronize()
        scale = float(x0[:, :P].abs().max())
        assert float((ca[:P] - cb[:P]).abs().max()) <= TIGHT * scale
        assert float((xa[:, :P] - xb[:, :P]).abs().max()) <= TIGHT * scale
        ch = ca.clone()
        plan.easgd_update(xa[:, :P], 0.0, 0.25, ca)                     # lambda = 0: only the center moves
        torch.cuda.synchronize()
        want = ch[:P].double() + 0.25 * (xa[:, :P].double().mean(0) - ch[:P].double())
        assert float((ca[:P].double() - want).abs().max()) <= TIGHT * scale
    torch.cuda.empty_cache()
