"""The tiled W4A4 kernel at the edges of its set-up and of its fused epilogue, bit for bit against the oracle.

Set-up: fewer K steps than the ring's first fill, filters that are not square, 32 taps, more padding than filter (taps and
rows that lie outside the image altogether).  Epilogue: values that the clamps of the quick quotient have to place."""
import numpy as np
import pytest

from oracle import qail_oracle as O
from paper_2412_01034_amd import synth

from .helpers import dev, ensure_built, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    return ensure_built()


# enough output tiles for the tiled kernel; in 128-code steps:
SHAPES = [
    synth.ConvShape("one step", 32, 30, 31, 32, 64, 1, 1, 1, 0),
    synth.ConvShape("three steps", 32, 30, 31, 32, 64, 3, 3, 1, 1),
    synth.ConvShape("a row of taps", 32, 30, 29, 64, 72, 1, 5, 1, 2),
    synth.ConvShape("a column of taps", 32, 30, 31, 64, 64, 7, 1, 1, 3),
    synth.ConvShape("32 taps", 32, 33, 37, 32, 64, 4, 8, 1, 3),              # K split between two groups
    synth.ConvShape("more padding than filter", 24, 28, 30, 64, 64, 2, 3, 1, 4),
    synth.ConvShape("one more step than the ring holds", 32, 61, 59, 128, 64, 2, 2, 2, 0),
]


@pytest.mark.parametrize("s", SHAPES, ids=[s.name for s in SHAPES])
def test_set_up_and_epilogue_edges(B, s):
    import torch
    geom = (s.B, s.H, s.W, s.Cin, s.Cout, s.KH, s.KW, s.stride, s.pad)
    rng = np.random.default_rng(s.K)
    aw = O.pack_nibbles(synth.random_codes((s.B, s.H, s.W, s.Cin), 0, 15, 81).astype(np.uint8))
    ww = O.pack_nibbles(synth.random_codes((s.Cout, s.K), -8, 7, 82))
    # the first and the last image whole (every border), and pixels of the others
    per = s.OH * s.OW
    rows = np.unique(np.concatenate([np.arange(per), np.arange(s.M - per, s.M), rng.integers(0, s.M, 500)]))
    ref = O.w4a4_conv_acc_rows(aw, ww, *geom, rows)
    acc = torch.full((s.M * s.Cout,), 0x55555555, dtype=torch.int32, device="cuda")
    B.qail_w4a4_gemm(*geom, dev(aw), dev(ww), acc_out=acc)
    torch.cuda.synchronize()
    assert np.array_equal(host(acc, np.int32).reshape(s.M, s.Cout)[rows], ref)

    # a step that spreads the codes, and channels whose bias is no ordinary number
    scale = (rng.random(s.Cout) * 1e-2 + 1e-3).astype(np.float32)
    bias = rng.standard_normal(s.Cout).astype(np.float32)
    bias[:7] = [np.inf, -np.inf, np.nan, 3e38, -3e38, -0.0, 1e-45]
    s_out = np.float32((ref * scale).max() / 18.0)
    codes = rng.integers(0, 16, size=(s.M, s.Cout)).astype(np.uint8)
    for res in (False, True):
        out = torch.full((s.M * s.Cout // 8,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
        B.qail_w4a4_conv_u4(*geom, dev(aw), dev(ww), dev(scale), dev(bias), float(s_out), out,
                            res_u4=dev(O.pack_nibbles(codes)) if res else None, res_scale=0.75 * float(s_out))
        torch.cuda.synchronize()
        kw = dict(res_codes=codes[rows], res_scale=np.float32(0.75 * float(s_out))) if res else {}
        with np.errstate(invalid="ignore", over="ignore"):
            want = O.fused_requant_u4(ref, scale, np.where(np.isnan(bias), -np.inf, bias), s_out, **kw)   # the ReLU makes 0 of a NaN
        assert len(np.unique(want)) >= 12
        assert np.array_equal(host(out, np.uint32).reshape(s.M, s.Cout // 8)[rows], O.pack_nibbles(want))
