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


def plain_calls(B):
    """The three calls on data that tells results apart: what their items point to, and of each the native function, the public
    call and the output."""
    import torch
    t = tensors("cuda")
    rng = np.random.default_rng(5)
    t["qweight"].copy_(dev(rng.integers(0, 2**32, N * K // 8, dtype=np.uint32)))
    t["x"].copy_(torch.from_numpy(rng.standard_normal((M, K)).astype(np.float32)))
    items = B.make_w4a16_items([dict(N=N, K=K, group_size=g, **t)], M)
    conv = dict(B=2, H=9, W=7, Cin=64, Cout=40, KH=3, KW=3, stride=1, pad=1, a_u4=dev(rng.integers(0, 2**32, 2 * 9 * 7 * 64 // 8, dtype=np.uint32)),
                w_s4=dev(rng.integers(0, 2**32, 40 * 9 * 64 // 8, dtype=np.uint32)),
                acc_out=torch.empty(2 * 9 * 7 * 40, dtype=torch.int32, device="cuda"))
    conv_items = B.make_conv_items([conv])
    return (t, conv), [(lambda: B._linear_native(N, K, g, *t.values(), M, None), lambda: B.qail_w4a16_linear(N, K, g, **t, M=M), t["y"]),
                       (lambda: B._linear_batch_native(items, 1, M, None), lambda: B.qail_w4a16_linear_batch(items, 1, M), t["y"]),
                       (lambda: B._conv_batch_native(conv_items, 1), lambda: B.qail_w4a4_conv_batch(conv_items, 1), conv["acc_out"])]


@pytest.mark.gpu
def test_plain_calls_are_taken_with_the_same_results_as_the_way_through_python(B, monkeypatch):
    import torch
    (t, conv), calls = plain_calls(B)

    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    def results(way):
        found = []
        for call in calls:
            call[2].fill_(7)
            assert call[way]() == (0 if way == 0 else None)   # the native function answers; the public one has nothing to say
            found.append(host(call[2], np.uint32 if call[2].dtype == torch.int32 else np.uint16).copy())
        return found

    native, public = results(0), results(1)
    with Mode():
        assert all(call[0]() is None for call in calls)
        moded = results(1)
    for name in ("_linear_native", "_linear_batch_native", "_conv_batch_native"):
        monkeypatch.setattr(B, name, B._not_plain)
    for a, b, c, d in zip(native, public, moded, results(1)):
        assert np.array_equal(a, b) and np.array_equal(a, c) and np.array_equal(a, d) and len(np.unique(a)) > 10
    monkeypatch.undo()
    for bad in (dict(x=t["x"].t().contiguous().t()), dict(y=t["y"][:1]), dict(scales=t["scales"].cpu())):
        with pytest.raises(ValueError):
            B.qail_w4a16_linear(N, K, g, **{**t, **bad}, M=M)


@pytest.mark.gpu
def test_plain_calls_go_to_the_current_stream(B):
    """A stream under capture runs nothing: what is launched there is in the graph, what is launched elsewhere is not."""
    import torch
    held, calls = plain_calls(B)
    for native, _, out in calls:
        assert native() == 0   # (the first launch of a kernel loads it, which a capture does not allow)
        want = out.clone()
        torch.cuda.synchronize()
        out.fill_(7)
        torch.cuda.synchronize()
        graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.graph(graph, stream=side):
            status = native()
        torch.cuda.synchronize()
        assert status == 0 and (out == 7).all()
        for _ in range(2):
            out.fill_(7)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
