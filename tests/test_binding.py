"""The Python binding's descriptions of tensors against torch's own: which
layouts count as float-float planes, and where the planes are (host tensors
are enough: nothing is launched)."""
import itertools

import pytest
import torch

import paper_cs_0603115_amd as ff


def _layouts():
    """(2, ...) tensors of many shapes and strides, among them dimensions of
    one element and of none, expanded, transposed and shifted ones."""
    base = torch.arange(4096, dtype=torch.float32)
    for dims in range(0, 4):
        for shape in itertools.product((0, 1, 2, 3), repeat=dims):
            for strides in itertools.product((0, 1, 2, 3, 6, 9), repeat=dims):
                for plane in (0, 1, 7, 100):
                    yield base.as_strided((2, *shape), (plane, *strides), 5)


def test_plane_contiguity_is_torchs():
    n = 0
    for t in _layouts():
        want = t[0].is_contiguous() and t[1].is_contiguous()
        assert ff._dense(t.shape, t.stride(), 1) == want, (t.shape, t.stride())
        n += 1
    assert n > 10000


def test_plane_addresses_are_torchs():
    for t in itertools.islice(_layouts(), 0, None, 37):
        if t.numel():
            assert ff._planes(t) == (t[0].data_ptr(), t[1].data_ptr()), (t.shape, t.stride())


@pytest.mark.parametrize("shape", [(), (0,), (1,), (5,), (1024,), (1025,), (3, 4), (0, 3), (2, 1, 5)])
def test_ff_empty_and_zeros_share_a_layout(shape):
    a, b = ff.ff_empty(shape, device="cpu"), ff.ff_zeros(shape, device="cpu")
    assert a.shape == b.shape == (2, *shape) and a.stride() == b.stride()
    assert a.stride(0) % ff.PLANE_ALIGN == 0 and not b.any()
    a.fill_(1.0)                       # both planes lie within the storage
    assert float(a.sum()) == a.numel()


def test_ff_empty_takes_any_iterable_of_sizes():
    for shape in ([3, 5], (3, 5), torch.Size((3, 5)), (d for d in (3, 5)), map(int, "35"),
                  {3: "rows", 5: "columns"}, torch.tensor([3, 5])):
        assert ff.ff_empty(shape, device="cpu").shape == (2, 3, 5)
    assert ff.ff_zeros(iter([4]), device="cpu").shape == (2, 4)


def test_stream_argument_by_position_and_keyword(monkeypatch):
    # the wrapper finds the stream wherever the caller put it
    seen = []

    class Entered:
        def __enter__(self):
            seen.append("entered")

        def __exit__(self, *exc):
            return False

    monkeypatch.setattr(ff, "_torch_stream", lambda s: s)
    monkeypatch.setattr(torch.cuda, "stream", lambda s: Entered())

    @ff._on_stream
    def wrapper(a, out=None, stream=None, more=1):
        return a, out, stream, more

    assert wrapper(1) == (1, None, None, 1) and not seen
    assert wrapper(1, None, "s") == (1, None, "s", 1) and len(seen) == 1
    assert wrapper(1, stream="s", more=2) == (1, None, "s", 2) and len(seen) == 2
    assert wrapper(1, 2, None, 3) == (1, 2, None, 3) and len(seen) == 2


@pytest.mark.parametrize("algo", [0, 1, 2])
def test_product_workspace_of_empty_sizes(algo):
    for shape in itertools.product((0, 1, 5), repeat=3):
        assert ff.ff_gemm_workspace_size(*shape, algo) >= 0


def test_binding_without_torchs_short_cuts(monkeypatch):
    # a torch without the private names: the public calls serve
    import importlib
    import sys

    class Stream:
        cuda_stream = 1234

    for name in ("_cuda_getDevice", "_cuda_getCurrentRawStream"):
        monkeypatch.delattr(torch._C, name, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda index: Stream)
    spec = importlib.util.spec_from_file_location(
        "ff_without_short_cuts", ff.__file__, submodule_search_locations=list(ff.__path__))
    mod = importlib.util.module_from_spec(spec)
    monkeypatch.setitem(sys.modules, spec.name, mod)
    spec.loader.exec_module(mod)
    assert mod._current_device() == 3 and mod._current_raw_stream(3) == 1234
    seen = []

    class Lib:
        @staticmethod
        def ff_entry(*args):
            seen.append(args)
            return 0

    monkeypatch.setattr(mod, "lib", Lib)
    mod._enqueue("ff_entry", torch.device("cuda", 3), None, 7, 8)
    mod._enqueue("ff_entry", torch.device("cuda", 3), Stream, 9)
    assert seen == [(7, 8, 1234), (9, 1234)]
