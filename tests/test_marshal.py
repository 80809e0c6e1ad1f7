"""The binding's marshalling in C++: it answers plain calls only and leaves everything else, errors included, to Python."""
import ctypes

import numpy as np
import pytest

from .helpers import dev, ensure_built, host

N, K, g, M = 256, 512, 128, 2


@pytest.fixture(scope="module")
def B():
    B = ensure_built()
    B.lib()
    return B


def tensors(device):
    import torch
    return dict(qweight=torch.zeros(N * K // 8, dtype=torch.int32, device=device), scales=torch.ones(N * K // g, dtype=torch.float16, device=device),
                zeros=torch.zeros(N, dtype=torch.int32, device=device), x=torch.zeros((M, K), dtype=torch.bfloat16, device=device),
                y=torch.zeros((M, N), dtype=torch.bfloat16, device=device))


def test_is_built(B):
    from paper_2412_01034_amd import _marshal
    assert B._linear_native is _marshal.w4a16_linear


def test_calls_that_are_not_plain_are_left_to_python(B):
    t = tensors("cpu")
    args = [N, K, g, *t.values(), M, None]
    assert B._linear_native(*args) is None                        # not on the GPU
    assert B._linear_native(*args[:-1]) is None                   # an argument less
    for i, v in ((0, -1), (0, 1 << 40), (1, 512.0), (2, 0), (3, None), (6, np.zeros(4)), (9, 5)):
        assert B._linear_native(*args[:i], v, *args[i + 1:]) is None
    for bad in (None, 5, "items"):
        assert B._conv_batch_native(bad, 1) is None and B._linear_batch_native(bad, 1, 1, None) is None
    assert B._conv_batch_native((B.qail_conv_item * 1)(), -1) is None
    assert B._linear_batch_native((B.qail_w4a16_item * 1)(), 1, 1, t["x"]) is None
    with pytest.raises(ValueError, match="device tensor expected"):
        B.qail_w4a16_linear(N, K, g, **t, M=M)
    with pytest.raises(ValueError, match="qweight: .* bytes given"):
        B.qail_w4a16_linear(N, K, g, **{**t, "qweight": t["qweight"][:1]}, M=M)


@pytest.mark.parametrize("built_for", [None, "python", "torch", "items"])
def test_a_module_built_for_something_else_is_left_alone(B, monkeypatch, built_for):
    from paper_2412_01034_amd import _marshal
    same = _marshal.built_for
    assert same == B._marshal_for()
    for name in ("_linear_native", "_linear_batch_native", "_conv_batch_native"):
        monkeypatch.setattr(B, name, B._not_plain)
    if built_for is None:   # as one from before it said so
        monkeypatch.delattr(_marshal, "built_for")
    else:
        other = {"python": (same[0] + 1, *same[1:]), "torch": (same[0], "2.0 0", *same[2:]), "items": (*same[:3], same[3] + 8, same[4])}
        monkeypatch.setattr(_marshal, "built_for", other[built_for])
    B._use_native(B.lib())
    assert B._linear_native is B._linear_batch_native is B._conv_batch_native is B._not_plain


@pytest.mark.parametrize("error", [RuntimeError("no Python.h"), FileNotFoundError("g++"), ImportError("torch"), None])
def test_library_is_built_without_the_marshalling(monkeypatch, tmp_path, capsys, error):
    from paper_2412_01034_amd import build

    def run(cmd):
        with open(cmd[cmd.index("-o") + 1], "w") as f:
            f.write(cmd[0])
        return ""

    def marshal():
        if error is not None:
            raise error
        open(build.MARSHAL, "w").close()

    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libqail.so"))
    monkeypatch.setattr(build, "MARSHAL", str(tmp_path / "_marshal.here.so"))
    monkeypatch.setattr(build, "_run", run)
    monkeypatch.setattr(build, "build_marshal", marshal)
    (tmp_path / "_marshal.so").touch()   # of an earlier build: not what is here now
    assert build.build_library() == build.LIB and (tmp_path / "libqail.so").exists()
    assert [p.name for p in tmp_path.glob("_marshal*")] == ([] if error else ["_marshal.here.so"])
    assert (str(error) in capsys.readouterr().err) == (error is not None)


@pytest.mark.gpu
def test_status_of_the_library_comes_back(B):
    with pytest.raises(B.QailError):   # NULL pointers
        B.qail_w4a4_conv_batch((B.qail_conv_item * 1)(), 1)
    with pytest.raises(B.QailError):
        B.qail_w4a16_linear_batch((B.qail_w4a16_item * 1)(), 1, 1)
    with pytest.raises(ctypes.ArgumentError):   # items of another kind are no items
        B.qail_w4a4_conv_batch((B.qail_w4a16_item * 1)(), 1)


@pytest.mark.gpu
def test_same_results_and_errors_as_the_way_through_python(B, monkeypatch):
    import torch
    t = tensors("cuda")
    rng = np.random.default_rng(5)
    t["qweight"].copy_(dev(rng.integers(0, 2**32, N * K // 8, dtype=np.uint32)))
    t["x"].copy_(torch.from_numpy(rng.standard_normal((M, K)).astype(np.float32)))
    items = B.make_w4a16_items([dict(N=N, K=K, group_size=g, **t)], M)

    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    def results():
        out = []
        for run in (lambda: B.qail_w4a16_linear(N, K, g, **t, M=M), lambda: B.qail_w4a16_linear_batch(items, 1, M)):
            t["y"].fill_(7.0)
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                run()
                out.append(t["y"].clone())
            side.synchronize()
        return [host(y, np.uint16) for y in out]

    native = results()
    with Mode():
        assert B._linear_native(N, K, g, *t.values(), M, None) is None
        moded = results()
    monkeypatch.setattr(B, "_linear_native", B._not_plain)
    monkeypatch.setattr(B, "_linear_batch_native", B._not_plain)
    for a, b, c in zip(native, results(), moded):
        assert np.array_equal(a, b) and np.array_equal(a, c) and len(np.unique(a)) > 10
    monkeypatch.undo()
    for bad in (dict(x=t["x"].t().contiguous().t()), dict(y=t["y"][:1]), dict(scales=t["scales"].cpu())):
        with pytest.raises(ValueError):
            B.qail_w4a16_linear(N, K, g, **{**t, **bad}, M=M)
