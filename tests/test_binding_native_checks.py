"""The native argument checks of the binding against the Python ones, over tensors that are in order and tensors that are
not: where the native code gives an answer it is the Python checks' answer, and what they refuse it leaves to them."""
import importlib.util
import itertools
import os
import sys
import types

import pytest
import torch

from paper_2403_04206_amd import buildlib, grawa


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


@pytest.mark.parametrize("built_for", [None, "torch 1.0 abc, cpython-310", buildlib.rows_built_for() + "0"])
def test_module_of_another_torch_is_not_used(built_for, monkeypatch):
    # the checks read torch's objects by a layout compiled in: a module of another torch could give wrong pointers
    other = types.ModuleType("paper_2403_04206_amd._rows")
    other.rows = lambda t, K, P, grads: (1, 2, 0)
    if built_for is not None:
        other.built_for = built_for
    monkeypatch.setitem(sys.modules, other.__name__, other)
    spec = importlib.util.spec_from_file_location("paper_2403_04206_amd.grawa_again", grawa.__file__)
    again = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(again)
    assert again._native_rows is not other.rows and again._native_rows(torch.zeros(2, 4), 2, 4, False) is None


def test_native_checks_are_rebuilt_when_their_source_is_newer(tmp_path, monkeypatch):
    source, module, built = tmp_path / "rows.cpp", tmp_path / "rows.so", []
    source.write_text("")
    monkeypatch.setattr(buildlib, "ROWS_SOURCE", str(source))
    monkeypatch.setattr(buildlib, "ROWS", str(module))
    monkeypatch.setattr(buildlib, "needs_build", lambda: False)
    monkeypatch.setattr(buildlib, "build_rows", lambda: built.append(module.write_text("")))
    buildlib.build(force=False)
    assert len(built) == 1                               # not there
    os.utime(source, (1, 1))
    buildlib.build(force=False)
    assert len(built) == 1                               # up to date
    os.utime(module, (0, 0))
    buildlib.build(force=False)
    assert len(built) == 2                               # older than its source


def test_a_build_without_the_native_checks(tmp_path, monkeypatch, capfd):
    # no compiler for them: the library is built all the same, and a module of an older source is not left to be loaded
    module = tmp_path / "rows.so"
    module.write_text("")
    monkeypatch.setattr(buildlib, "ROWS", str(module))
    monkeypatch.setattr(buildlib, "build_library", lambda verbose=False: None)
    monkeypatch.setenv("PATH", str(tmp_path))
    assert buildlib.build(force=True) == buildlib.LIB
    assert not module.exists() and "not built" in capfd.readouterr().err


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
    assert seen == [None, None]                          # no storage of their own: the Python checks refuse them too
