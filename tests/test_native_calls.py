"""The native marshalling of the binding against its ctypes form: the same outcome for every kind of argument (no GPU
needed: a NULL context is refused by the library before anything else is looked at)."""
import ctypes
import inspect
import re

import numpy as np
import pytest
import torch

import paper_2406_19707_amd as ig
from paper_2406_19707_amd import binding


def outcome(f):
    try:
        return f()
    except Exception as e:        # noqa: BLE001 -- its type and text are what is compared
        return type(e), str(e)


class Odd(torch.Tensor):
    pass


@pytest.fixture(scope="module")
def native():
    if binding.os.environ.get("IG_LIBRARY"):
        pytest.skip("another build of the library is under test")
    fn = binding._Entries().ig_pool_touch
    assert type(fn).__name__ == "builtin_function_or_method", "the native module is missing: build it"
    return fn


@pytest.mark.parametrize("what", ["tensor", "view", "parameter", "subclass", "transposed", "numpy", "numpy strided", "address",
                                  "none", "text", "float stride", "numpy stride", "no descriptor", "other structure",
                                  "too few", "empty tensor"])
def test_same_outcome_as_through_ctypes(native, what):
    d, t = ig.IgDesc(B=1, H=1, d=64, r=8, N=8), torch.zeros(64, dtype=torch.int32)
    args = [None, d, t, 8, t, t, 255, 0]
    if what == "view":
        args[2] = t[8:16]
    elif what == "parameter":
        args[2] = torch.nn.Parameter(torch.zeros(4))
    elif what == "subclass":
        args[2] = torch.zeros(4).as_subclass(Odd)
    elif what == "transposed":
        args[2] = torch.zeros(4, 4).t()
    elif what == "numpy":
        args[2] = np.zeros(4, np.int32)
    elif what == "numpy strided":
        args[2] = np.zeros((4, 4), np.int32)[:, 1]
    elif what == "address":
        args[2] = t.data_ptr()
    elif what == "none":
        args[2] = None
    elif what == "text":
        args[2] = "x"
    elif what == "float stride":
        args[3] = 2.5
    elif what == "numpy stride":
        args[3] = np.int64(8)
    elif what == "no descriptor":
        args[1] = None
    elif what == "other structure":
        args[1] = ig.IgLayerIO()
    elif what == "too few":
        args.pop()
    elif what == "empty tensor":
        args[2] = torch.zeros(0)
    want = outcome(lambda: binding._through_ctypes("ig_pool_touch", *args))
    assert outcome(lambda: native(*args)) == want
    if what in ("tensor", "view", "parameter", "subclass", "numpy", "address", "none", "empty tensor"):
        assert want == ig.IG_EINVAL


@pytest.mark.parametrize("number", [np.int64(8), np.array(8), torch.tensor(8), torch.tensor([8], dtype=torch.int32)], ids=repr)
@pytest.mark.parametrize("form", ["native", "ctypes"])
def test_a_number_is_passed_by_value_whatever_holds_it(native, monkeypatch, number, form):
    """Both integers of the call, next to a tensor that does go by its address."""
    t, got = torch.zeros(8, dtype=torch.int32), []
    real = binding.lib().ig_pool_touch

    @ctypes.CFUNCTYPE(real.restype, *real.argtypes)
    def record(ctx, desc, sel_idx, sel_stride, sel_cnt, counters, counter_max, stream):
        got.append((sel_idx, sel_stride, counter_max))
        return 0
    record.argtypes = real.argtypes

    class Library:
        ig_pool_touch = record
    monkeypatch.setattr(binding, "lib", lambda: Library)
    args = (None, ig.IgDesc(B=1, H=1, d=64, r=8, N=8), t, number, t, t, number, 0)
    call = native if form == "native" else lambda *a: binding._through_ctypes("ig_pool_touch", *a)
    assert call(*args) == 0
    assert got == [(t.data_ptr(), 8, 8)]


@pytest.mark.parametrize("wrong", [torch.zeros(4, dtype=torch.int32), np.zeros(4, np.int32), torch.zeros(1), None, 2.5, "x"], ids=repr)
def test_what_is_no_whole_number_is_refused(native, wrong):
    t = torch.zeros(8, dtype=torch.int32)
    args = (None, ig.IgDesc(B=1, H=1, d=64, r=8, N=8), t, wrong, t, t, 255, 0)
    for call in (native, lambda *a: binding._through_ctypes("ig_pool_touch", *a)):
        with pytest.raises((ctypes.ArgumentError, TypeError)):
            call(*args)


def test_another_torch_than_the_modules_own_goes_through_ctypes(native, monkeypatch):
    from paper_2406_19707_amd import _ig_call
    monkeypatch.setattr(_ig_call, "built_for", "0.0")
    assert type(binding._Entries().ig_pool_touch).__name__ == "partial"


@pytest.mark.parametrize("missing", ["torch", "python_variable.h", "Python.h"])
def test_the_build_goes_on_without_the_module(missing, tmp_path, monkeypatch, capsys):
    from paper_2406_19707_amd import build
    stale = tmp_path / "_ig_call.so"
    stale.write_bytes(b"of another library")
    find, exists = build.importlib.util.find_spec, build.os.path.exists
    monkeypatch.setattr(build, "CALL", str(stale))
    monkeypatch.setattr(build.importlib.util, "find_spec", lambda n: None if n == missing else find(n))
    monkeypatch.setattr(build.os.path, "exists", lambda p: not str(p).endswith("/" + missing) and exists(p))
    build._build_call()
    assert not stale.exists() and "ctypes" in capsys.readouterr().out


def test_every_device_entry_point_has_a_native_form(native):
    """Every entry point that the binding's methods call through the native module or ctypes, no more and no fewer."""
    from paper_2406_19707_amd import _ig_call
    used = set(re.findall(r"_entries\.(ig_\w+)", inspect.getsource(binding)))
    assert len(used) >= 24 and used == {n for n in dir(_ig_call) if n.startswith("ig_")}
    assert used <= set(ig.EXPORTS)
