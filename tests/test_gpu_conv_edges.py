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


# Every shape of the tiled kernel, with tiles that are cut off in both directions and a K that is no whole number of
# steps.  Columns: K split between groups of waves or not, waves' own tile, slots of the ring.
VARIANTS = [
    ("four groups", 4, (12, 20, 21, 352, 72, 3, 1, 1)),
    ("two groups of four waves", 4, (12, 20, 21, 224, 72, 3, 1, 1)),
    ("32 x 32 a wave", 4, (24, 28, 29, 96, 72, 3, 1, 1)),
    ("two groups of two waves", 4, (12, 28, 29, 224, 72, 3, 1, 1)),
    ("128 x 64, three slots", 4, (48, 33, 32, 32, 40, 3, 1, 1)),
    ("128 x 64, two slots", 4, (97, 33, 32, 32, 40, 3, 1, 1)),
    ("64 x 128, three slots", 4, (24, 33, 32, 32, 72, 3, 1, 1)),
    ("64 x 128, two slots", 4, (49, 33, 32, 64, 72, 1, 1, 0)),
    ("128 x 128", 4, (49, 33, 32, 32, 72, 3, 1, 1)),
    ("bytes, four groups", 8, (12, 20, 21, 176, 72, 3, 1, 1)),
    ("bytes, two groups of four waves", 8, (12, 20, 21, 112, 70, 3, 1, 1)),
    ("bytes, 32 x 32 a wave", 8, (24, 28, 29, 48, 72, 3, 1, 1)),
    ("bytes, two groups of four waves, more tiles", 8, (12, 28, 29, 112, 71, 3, 1, 1)),
    ("bytes, two groups of two waves", 8, (24, 28, 29, 128, 71, 3, 1, 1)),
    ("bytes, 32 x 32 a wave, ragged rows", 8, (24, 28, 29, 48, 141, 3, 1, 1)),
    ("bytes, 64 x 128, few steps", 8, (49, 33, 32, 16, 260, 3, 1, 1)),
    ("bytes, 128 x 64", 8, (48, 33, 32, 48, 40, 3, 1, 1)),
    ("bytes, 64 x 128", 8, (24, 33, 32, 48, 72, 3, 1, 1)),
    ("bytes, 128 x 128, three slots or, with one output, two", 8, (49, 33, 32, 48, 73, 3, 1, 1)),
    ("bytes, 128 x 128, three slots", 8, (100, 33, 32, 48, 72, 3, 1, 1)),
]


@pytest.mark.parametrize("bits,dims", [v[1:] for v in VARIANTS], ids=[v[0] for v in VARIANTS])
def test_tiled_variants(B, bits, dims):
    import torch
    nb, H, W, cin, cout, taps, stride, pad = dims
    s = synth.ConvShape("v", nb, H, W, cin, cout, taps, taps, stride, pad)
    geom = (nb, H, W, cin, cout, taps, taps, stride, pad)
    rng = np.random.default_rng(s.K + s.M)
    if bits == 4:
        aw = O.pack_nibbles(synth.random_codes((nb, H, W, cin), 0, 15, 91).astype(np.uint8))
        ww = O.pack_nibbles(synth.random_codes((cout, s.K), -7, 7, 92))   # of mean zero, so that sums of both signs come out
        plain, acc_rows = B.qail_w4a4_gemm, O.w4a4_conv_acc_rows
    else:
        aw = O.pack_bytes(synth.random_codes((nb, H, W, cin), -127, 127, 93))
        ww = O.pack_bytes(synth.random_codes((cout, s.K), -127, 127, 94))
        plain, acc_rows = B.qail_w8a8_gemm, O.w8a8_conv_acc_rows
    # the ends of the first and the last tiles, and pixels of all
    rows = np.unique(np.concatenate([np.arange(130), np.arange(s.M - 130, s.M), rng.integers(0, s.M, 300)]))
    ref = acc_rows(aw, ww, *geom, rows)
    scale = (rng.random(cout) * 1e-2 + 1e-3).astype(np.float32)
    bias = rng.standard_normal(cout).astype(np.float32)
    acc = torch.full((s.M * cout,), 0x55555555, dtype=torch.int32, device="cuda")
    y = torch.full((s.M * cout,), 7.0, device="cuda")
    a, w, sc, bi = dev(aw), dev(ww), dev(scale), dev(bias)
    plain(*geom, a, w, acc_out=acc, scale=sc, bias=bi, y_out=y)
    torch.cuda.synchronize()
    assert np.array_equal(host(acc, np.int32).reshape(s.M, cout)[rows], ref)
    assert np.array_equal(host(y, np.float32).reshape(s.M, cout)[rows], O.requant_f32(ref, scale, bias))
    # one output: bytes go by how many there are
    acc.fill_(0x55555555)
    plain(*geom, a, w, acc_out=acc)
    torch.cuda.synchronize()
    assert np.array_equal(host(acc, np.int32).reshape(s.M, cout)[rows], ref)
    if bits == 8 or cout % 8:
        return
    # fused, with each kind of shortcut; the step at an ordinary size (both ways to a code) and beyond what is quick
    codes = rng.integers(0, 16, size=(s.M, cout)).astype(np.uint8)
    real = rng.standard_normal((s.M, cout)).astype(np.float32) * np.float32((ref * scale).max() / 4)
    real.reshape(-1)[rng.integers(0, real.size, 2000)] = np.repeat(np.float32([np.inf, -np.inf, 3e38, 1e-45]), 500)
    for power in (0, 110, -110):
        k = np.float32(2.0) ** np.float32(power)
        s_out, r_step = np.float32((ref * scale).max() / 18.0) * k, np.float32((ref * scale).max() / 30.0) * k
        for res in (None, "codes", "floats"):
            out = torch.full((s.M * cout // 8,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
            kw, okw = {}, {}
            with np.errstate(invalid="ignore", over="ignore", under="ignore"):
                if res == "codes":
                    kw, okw = dict(res_u4=dev(O.pack_nibbles(codes)), res_scale=float(r_step)), dict(res_codes=codes[rows], res_scale=r_step)
                elif res == "floats":
                    kw, okw = dict(res_f32=dev(real * k)), dict(res_f32=(real * k)[rows])
                B.qail_w4a4_conv_u4(*geom, a, w, dev(scale * k), dev(bias * k), float(s_out), out, **kw)
                torch.cuda.synchronize()
                want = O.fused_requant_u4(ref, scale * k, bias * k, s_out, **okw)
            assert len(np.unique(want)) >= 10
            assert np.array_equal(host(out, np.uint32).reshape(s.M, cout // 8)[rows], O.pack_nibbles(want)), (power, res)
