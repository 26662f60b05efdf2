"""The native view builder against binding.views: the same names in the same
order, and each view the same slice of the same storage with the same dtype,
sizes, strides and relation to the buffer, for file layouts, device layouts
and buffers that start inside a larger allocation."""

import os

import pytest
import torch

from paper_2401_14351_amd import binding, synth


@pytest.fixture(scope="module")
def L():
    if not os.path.exists(binding.LIB_PATH):
        pytest.skip("libsllm.so not built")
    return binding.lib()


def test_builder_is_built(L):
    """What the other tests compare is the native form (it is optional otherwise)."""
    assert binding._views_ext() is not None


@pytest.mark.parametrize("why", ["missing", "another torch", "no torch named"])
def test_without_the_builder(L, tmp_path, monkeypatch, why):
    """Views are built in Python where the builder is missing or was made for
    another Python or torch."""
    import sys

    import paper_2401_14351_amd as package

    if why == "missing":
        monkeypatch.setitem(sys.modules, "paper_2401_14351_amd._views", None)
        monkeypatch.delattr(package, "_views", raising=False)
    elif why == "no torch named":  # a builder from before it named its torch
        monkeypatch.delattr(binding._views_ext(), "TORCH_VERSION")
    else:
        monkeypatch.setattr(binding._views_ext(), "TORCH_VERSION", "1.0", raising=False)
    binding._views_ext.cache_clear()
    spec = synth.tiny(56, n=20, alignment=16)
    binding.convert(((t.name, t.dtype, t.shape, d) for t, d in zip(spec.tensors, synth.materialize(spec))), str(tmp_path), 16)
    try:
        with binding.Checkpoint(str(tmp_path), index_only=True) as ck:
            monkeypatch.setattr(ck, "load_into", lambda buf, stream: None)
            buf = torch.zeros(ck.total_bytes, dtype=torch.uint8)
            assert binding._views_ext() is None
            same(ck.load_with_views(buf), binding.views(buf, ck.tensors()))
    finally:
        monkeypatch.undo()
        binding._views_ext.cache_clear()


def test_library_builds_without_torch(monkeypatch):
    """The view builder alone needs torch's headers."""
    import sys

    from paper_2401_14351_amd import build

    monkeypatch.setitem(sys.modules, "torch", None)
    assert build.views_command("x") is None


def same(a, b):
    assert list(a) == list(b)
    for name in a:
        x, y = a[name], b[name]
        assert (x.dtype, x.shape, x.stride(), x.storage_offset()) == (y.dtype, y.shape, y.stride(), y.storage_offset()), name
        assert x.untyped_storage().data_ptr() == y.untyped_storage().data_ptr(), name
        assert x.is_inference() == y.is_inference() and x.requires_grad == y.requires_grad, name
        assert (x._base is None) == (y._base is None), name
        assert x.is_inference() or x._version == y._version, name


@pytest.mark.parametrize("A,A2", [(1, 0), (2, 0), (16, 0), (4096, 256), (1, 16)])
@pytest.mark.parametrize("start", [0, 1, 2, 4, 48])
def test_same_as_python(L, tmp_path, A, A2, start):
    spec = synth.tiny(51, n=60, alignment=A, max_bytes=4000)
    binding.convert(((t.name, t.dtype, t.shape, d) for t, d in zip(spec.tensors, synth.materialize(spec))), str(tmp_path), A)
    with binding.Checkpoint(str(tmp_path), index_only=True, dev_alignment=A2) as ck:
        buf = torch.zeros(start + ck.total_bytes + 7, dtype=torch.uint8)[start:]
        same(ck._views(buf, ck._table()), binding.views(buf, ck.tensors()))
        with torch.inference_mode():
            fresh = torch.zeros(ck.total_bytes, dtype=torch.uint8)
            same(ck._views(fresh, ck._table()), binding.views(fresh, ck.tensors()))
        got = ck._views(buf, ck._table())
        next(v for v in got.values() if v.numel()).fill_(1)  # views share the buffer's bytes and its version
        assert buf.any() and buf._version == 1


def test_refuses_what_python_refuses(L, tmp_path):
    spec = synth.tiny(52, n=10, alignment=16)
    binding.convert(((t.name, t.dtype, t.shape, d) for t, d in zip(spec.tensors, synth.materialize(spec))), str(tmp_path), 16)
    with binding.Checkpoint(str(tmp_path), index_only=True) as ck:
        for bad in (torch.zeros(4096, dtype=torch.float32), torch.zeros(64, 64, dtype=torch.uint8),
                    torch.zeros(8192, dtype=torch.uint8)[::2]):
            with pytest.raises(ValueError):
                ck._views(bad, ck._table())
        short = torch.zeros(8, dtype=torch.uint8)
        for build in (lambda: binding.views(short, ck.tensors()), lambda: ck._views(short, ck._table())):
            with pytest.raises(RuntimeError):
                build()


def test_function_modes_see_the_calls(L, tmp_path):
    spec = synth.tiny(53, n=6, alignment=16)
    binding.convert(((t.name, t.dtype, t.shape, d) for t, d in zip(spec.tensors, synth.materialize(spec))), str(tmp_path), 16)
    calls = []

    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            calls.append(func)
            return func(*args, **(kwargs or {}))

    with binding.Checkpoint(str(tmp_path), index_only=True) as ck:
        buf = torch.zeros(ck.total_bytes, dtype=torch.uint8)
        with Mode():
            ck._views(buf, ck._table())
        assert torch.Tensor.as_strided in calls


@pytest.mark.parametrize("n", [10, 3000])
@pytest.mark.parametrize("native", [True, False])
def test_handle_closed_after_the_load(L, tmp_path, monkeypatch, n, native):
    """after_load may close the handle, which owns the names: with the load on a
    helper thread the views are whole all the same, and without one the call
    fails as on any closed handle."""
    spec = synth.tiny(54, n=n, alignment=16, max_bytes=64)
    binding.convert(((t.name, t.dtype, t.shape, d) for t, d in zip(spec.tensors, synth.materialize(spec))), str(tmp_path), 16)
    want = [t.name for t in spec.tensors]
    for threaded in (True, False):
        for limit in ("_THREADED_VIEWS_MIN", "_THREADED_PYTHON_VIEWS_MIN"):
            monkeypatch.setattr(binding, limit, 0 if threaded else 1 << 30, raising=False)
        ck = binding.Checkpoint(str(tmp_path), index_only=True)
        buf = torch.zeros(ck.total_bytes, dtype=torch.uint8)
        if not native:
            buf = buf.as_subclass(type("Buffer", (torch.Tensor,), {}))
        monkeypatch.setattr(ck, "load_into", lambda buf, stream: None)
        if threaded:
            assert list(ck.load_with_views(buf, None, after_load=ck.close)) == want
        else:
            with pytest.raises(binding.SllmError) as ei:
                ck.load_with_views(buf, None, after_load=ck.close)
            assert ei.value.code == -1


def test_errors_of_the_names_callback(L, tmp_path):
    spec = synth.tiny(55, n=10, alignment=16)
    binding.convert(((t.name, t.dtype, t.shape, d) for t, d in zip(spec.tensors, synth.materialize(spec))), str(tmp_path), 16)

    def bad():
        raise KeyError("stop")

    with binding.Checkpoint(str(tmp_path), index_only=True) as ck:
        with pytest.raises(KeyError):
            ck._views(torch.zeros(ck.total_bytes, dtype=torch.uint8), ck._table(), bad)


class Mode(torch.overrides.TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


@pytest.mark.parametrize("where,native", [("plain", True), ("device", True), ("default device", True), ("nested", False),
                                          ("mode", False), ("subclass", False)])
def test_which_form_and_thread(L, tmp_path, monkeypatch, where, native):
    """Under torch.device(...) and torch.set_default_device the views are built
    natively; other function modes and subclasses get the Python form, for which
    a helper thread pays from 1,024 tensors on."""
    import threading

    binding.convert(((f"t{i}", "i8", (0,), b"") for i in range(2000)), str(tmp_path), 16)
    started, forms = [], []
    monkeypatch.setattr(threading.Thread, "start", lambda self, start=threading.Thread.start: (started.append(self.name), start(self)))
    monkeypatch.setattr(binding, "views", lambda *a, f=binding.views: (forms.append("python"), f(*a))[1])
    with binding.Checkpoint(str(tmp_path), index_only=True) as ck:
        monkeypatch.setattr(ck, "load_into", lambda buf, stream: None)
        buf = torch.zeros(64, dtype=torch.uint8)
        if where == "subclass":
            buf = buf.as_subclass(type("Buffer", (torch.Tensor,), {}))

        def go():
            assert len(ck.load_with_views(buf)) == 2000

        if where == "device":
            with torch.device("cpu"):
                go()
        elif where == "default device":
            torch.set_default_device("cpu")
            try:
                go()
            finally:
                torch.set_default_device(None)
        elif where == "nested":
            with torch.device("cpu"), Mode():
                go()
        elif where == "mode":
            with Mode():
                go()
        else:
            go()
    assert forms == ([] if native else ["python"])
    assert started == ([] if native else ["sllm-load"])
