"""The native argument checks of the binding against the Python ones, over tensors that are in order and tensors that are
not: where the native code gives an answer it is the Python checks' answer, and what they refuse it leaves to them."""
import itertools

import pytest
import torch

from paper_2403_04206_amd import grawa


def forms(dev):
    for dtype in (torch.float32, torch.bfloat16, torch.float64, torch.int32):
        base = torch.zeros(400, device=dev).to(dtype)
        yield base[:360].view(6, 60)
        yield base[:360].view(6, 60)[:, :40]
        yield base[4:364].view(6, 60)[1:, 3:44]
        yield base.as_strided((6, 40), (40, 1))
        yield base.as_strided((6, 40), (32, 1))                         # rows overlap
        yield base.as_strided((1, 40), (7, 1))                          # one row: any stride
        yield base.as_strided((40, 6), (1, 40)).t()
        yield base.as_strided((40, 6), (1, 40))
        yield base[:240].view(3, 80)[:, ::2]
        yield base[:120].view(2, 60)
        yield base[:40]
        yield base[:360].view(2, 3, 60)
        yield base.as_strided((6, 40), (72, 1))                         # ends with the storage
        yield torch.nn.Parameter(base[:360].view(6, 60)) if dtype.is_floating_point else base[:360].view(6, 60)
    yield torch.zeros((6, 0), device=dev)


def python_answer(t, K, P, grads, monkeypatch):
    monkeypatch.setattr(grawa, "_native_rows", lambda *a: None)
    try:
        return grawa._grads(t, K, P) if grads else grawa._params(t, K, P) + (grawa.F32,)
    except (TypeError, ValueError):
        return None
    finally:
        monkeypatch.undo()


def compare(dev, monkeypatch):
    rows, seen = grawa._native_rows, set()
    for t, K, P, grads in itertools.product(forms(dev), (1, 2, 6, 7), (1, 40, 41, 60, 61), (False, True)):
        got, want = rows(t, K, P, grads), python_answer(t, K, P, grads, monkeypatch)
        assert got == want or (got is None and dev == "cpu"), (t.shape, t.stride(), t.dtype, K, P, grads, got, want)
        seen.add(got is not None)
    for t in (None, 3, "x", [[1.0]]):
        assert rows(t, 1, 1, False) is None
    with pytest.raises(TypeError):
        rows(1)
    return seen


def test_host_tensors_are_left_to_the_python_checks(monkeypatch):
    if grawa._native_rows.__module__ == grawa.__name__:
        pytest.skip("the native checks are not built here")
    assert compare("cpu", monkeypatch) == {False}


@pytest.mark.gpu
def test_native_checks_agree(monkeypatch):
    assert grawa._native_rows.__module__ != grawa.__name__, "the native checks are not built"
    assert compare("cuda:0", monkeypatch) == {False, True}


@pytest.mark.gpu
def test_tensors_of_transforms_are_left_alone():
    rows, seen = grawa._native_rows, []
    t = torch.zeros((3, 6, 40), device="cuda:0")
    torch.func.vmap(lambda v: (seen.append(rows(v, 6, 40, False)), v)[1])(t)
    torch.func.grad(lambda v: (seen.append(rows(v, 6, 40, False)), v.sum())[1])(t[0])
    assert all(s is None or len(s) == 3 for s in seen) and seen[0] is None
