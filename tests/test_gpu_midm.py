"""The kernel for medium batches (5 <= M <= 64): one pass over K, x staged step by step, K parts added in LDS.

Lists and shapes at its edges: row blocks full and ragged, columns that end inside a tile, one step of K and step counts
that the K parts do not divide, blocks of one tile and of several, both group sizes, bytes; and lists that run every compiled
variant between them (tests/midm_lists.py, which tests/test_dispatch.py holds against the library).  Against the oracle."""
import numpy as np
import pytest

from oracle import qail_oracle as O
from paper_2412_01034_amd import synth

from .helpers import dev, ensure_built, host, w4a16_norm_err, ws_for
from .midm_lists import EDGE_M, EDGES, LISTS

pytestmark = pytest.mark.gpu

TOL = 2e-3                          # of the norm product: fp32 sums, one rounding to bf16 (2^-9 of a value far below that product)
TOL_TINY_K = 2.0 ** -8 * 1.01       # few k: a dot product may be almost aligned, the output's rounding alone counts


@pytest.fixture(scope="module")
def B():
    return ensure_built()


def make(B, bits, N, K, g, M, seed):
    import torch
    w = synth.llm_weight(N, K, seed, outlier_frac=0.01)
    xb = synth.llm_activation_bf16(M, K, seed + 1, outlier_frac=0.005)
    e = dict(N=N, K=K, group_size=g, x=dev(xb), y=torch.full((M * N,), 0x7FC0, dtype=torch.int16, device="cuda"))
    nx = np.sqrt((O.bf16_bits_to_f64(xb) ** 2).sum(axis=1))
    if bits == 4:
        q, s, z = O.quantize_w4_asym_group(w, g)
        qw, zw = O.pack_w4a16(q, z)
        e.update(qweight=dev(qw), scales=dev(s.view(np.uint16)), zeros=dev(zw))
        return e, O.w4a16_linear(xb, qw, s, zw, g), O.w4a16_row_norms(xb, qw, s, zw, g)
    q, s = O.quantize_w8_sym_group(w, g)
    e.update(qweight=dev(O.pack_bytes(q)), scales=dev(s.view(np.uint16)))
    wh = q.astype(np.float64) * np.repeat(s.astype(np.float64), g, axis=1)
    return e, O.w8a16_linear(xb, q, s, g), (nx, np.sqrt((wh ** 2).sum(axis=1)))


def run(B, bits, ents, M):
    import torch
    if bits == 4:
        items = B.make_w4a16_items(ents, M)
        B.qail_w4a16_linear_batch(items, len(ents), M, ws_for(B, B.qail_w4a16_batch_workspace(items, len(ents), M)))
    else:
        items = B.make_w8a16_items(ents, M)
        B.qail_w8a16_linear_batch(items, len(ents), M, ws_for(B, B.qail_w8a16_batch_workspace(items, len(ents), M)))
    torch.cuda.synchronize()


@pytest.mark.parametrize("M", EDGE_M)
@pytest.mark.parametrize("bits,shapes", [(bits, shapes) for bits, shapes, _ in EDGES])
def test_lists_and_edges(B, bits, shapes, M):
    made = [make(B, bits, N, K, g, M, 3000 + 10 * i + M) for i, (N, K, g) in enumerate(shapes)]
    ents = [m[0] for m in made]
    run(B, bits, ents, M)
    first = [host(e["y"], np.uint16).copy() for e in ents]
    for e in ents:
        e["y"].fill_(0x7FC0)
    run(B, bits, ents, M)
    for (e, ref, (nx, nw)), y0 in zip(made, first):
        y = host(e["y"], np.uint16)
        assert np.array_equal(y, y0), "run to run"
        tol = TOL if e["K"] >= 512 else TOL_TINY_K
        assert w4a16_norm_err(y.reshape(M, e["N"]), ref, nx, nw) <= tol, (e["N"], e["K"], e["group_size"])


@pytest.mark.parametrize("bits,M,shapes", LISTS)
def test_every_variant(B, bits, M, shapes):
    """Random codes, scales and zero-points (every bit pattern of a code word is a weight).  All results are written and repeat bit
    for bit; the oracle is asked for a column out of every tile, as far as six million weights of an item go."""
    import torch
    rng = np.random.default_rng(M + sum(N + K for N, K, _ in shapes))
    gen = torch.Generator(device="cuda").manual_seed(int(rng.integers(1 << 30)))
    ents = []
    for N, K, g in shapes:
        G = K // g
        x = synth.llm_activation_bf16(M, K, int(rng.integers(1 << 30)), outlier_frac=0.005)
        ents.append(dict(N=N, K=K, group_size=g, x=dev(x), y=torch.full((M * N,), 0x7FC0, dtype=torch.int16, device="cuda"),
                         qweight=torch.randint(-2 ** 31, 2 ** 31, (N, K * bits // 32), dtype=torch.int32, device="cuda", generator=gen),
                         scales=(torch.rand((N, G), device="cuda", generator=gen) * 1e-2 + 1e-3).half(),
                         zeros=torch.randint(-2 ** 31, 2 ** 31, (N, (G + 7) // 8), dtype=torch.int32, device="cuda", generator=gen)))
    run(B, bits, ents, M)
    first = [e["y"].clone() for e in ents]
    for e in ents:
        e["y"].fill_(0x7FC0)
    run(B, bits, ents, M)
    for e, y0 in zip(ents, first):
        N, K, g = e["N"], e["K"], e["group_size"]
        assert torch.equal(e["y"], y0), "run to run"
        assert bool(torch.isfinite(y0.view(torch.bfloat16)).all())
        tiles = rng.permutation((N + 15) // 16)[:max(1, 6_000_000 // K)]
        n = np.unique(np.r_[0, N - 1, np.minimum(16 * tiles + rng.integers(0, 16, tiles.size), N - 1)])
        pick = torch.from_numpy(n).cuda()
        q, s, z = (host(e[k][pick], d) for k, d in (("qweight", np.uint32), ("scales", np.float16), ("zeros", np.uint32)))
        xb = host(e["x"], np.uint16).reshape(M, K)
        nx = np.sqrt((O.bf16_bits_to_f64(xb) ** 2).sum(axis=1))
        if bits == 4:
            ref, (_, nw) = O.w4a16_linear(xb, q, s, z, g), O.w4a16_row_norms(xb, q, s, z, g)
        else:
            codes = q.view(np.int8).reshape(n.size, K)
            ref = O.w8a16_linear(xb, codes, s, g)
            nw = np.sqrt(((codes.astype(np.float64) * np.repeat(s.astype(np.float64), g, axis=1)) ** 2).sum(axis=1))
        y = host(y0, np.uint16).reshape(M, N)[:, n]
        assert w4a16_norm_err(y, ref, nx, nw) <= (TOL if K >= 512 else TOL_TINY_K), (N, K)


@pytest.mark.parametrize("bits,g,M", [(4, 64, 16), (4, 64, 33), (4, 128, 40), (8, 128, 50)])
def test_rows_do_not_reach_each_other(B, bits, g, M):
    """A row of x that holds infinities and NaN gives NaN in its own results only; a row of zeros gives zeros."""
    N, K = 300, 1024
    e, ref, (nx, nw) = make(B, bits, N, K, g, M, 4000 + M)
    x = e["x"].view(M, K)
    x[3] = 0x7F80                   # +inf
    x[4] = 0x7FC0                   # NaN
    x[2] = 0
    run(B, bits, [e], M)
    y = (host(e["y"], np.uint16).reshape(M, N).astype(np.uint32) << 16).view(np.float32)
    assert np.all(np.isnan(y[3]) | np.isinf(y[3])) and np.all(np.isnan(y[4])) and np.all(y[2] == 0)
    rest = [m for m in range(M) if m not in (2, 3, 4)]
    assert w4a16_norm_err(host(e["y"], np.uint16).reshape(M, N)[rest], ref[rest], nx[rest], nw) <= TOL


@pytest.mark.parametrize("bits,shapes", [(4, [(256, 256, 128)] * 4 + [(520, 10880, 128)] * 8),
                                         (8, [(256, 256, 128)] * 3 + [(520, 10880, 128)] * 6)])
def test_lists_shared_with_the_matrix_core_gemm_stay_in_their_workspace(B, bits, shapes):
    """This kernel takes the first linears, the GEMM (85 groups) the others: it writes nothing past the workspace asked for."""
    import torch
    M, past = 48, 16 << 20
    made = [make(B, bits, N, K, g, M, 5000 + 10 * i) for i, (N, K, g) in enumerate(shapes)]
    ents = [m[0] for m in made]
    name = "w4a16" if bits == 4 else "w8a16"
    items = getattr(B, f"make_{name}_items")(ents, M)
    need = getattr(B, f"qail_{name}_batch_workspace")(items, len(ents), M)
    ws = torch.full((need + past,), 0x5A, dtype=torch.uint8, device="cuda")
    getattr(B, f"qail_{name}_linear_batch")(items, len(ents), M, ws[:need])
    torch.cuda.synchronize()
    assert bool((ws[need:] == 0x5A).all())
    for e, ref, (nx, nw) in made:
        assert w4a16_norm_err(host(e["y"], np.uint16).reshape(M, e["N"]), ref, nx, nw) <= (TOL if e["K"] >= 512 else TOL_TINY_K)


@pytest.mark.parametrize("bits,g,M", [(4, 64, 16), (4, 64, 40), (4, 128, 40), (8, 128, 40), (8, 128, 50)])
def test_rows_of_any_size(B, bits, g, M):
    """Rows of x from 2^-110 to just below the largest bf16 number: no sum on the way overflows or falls out of fp32's range."""
    import torch
    N, K = 300, 1024
    # 2^-10: the weights (their scales are fp16 numbers below 2^-14, exact in the oracle), so that results are representable
    w = synth.llm_weight(N, K, 6000) * np.float32(2.0 ** -10)
    rng = np.random.default_rng(6001)
    x = rng.uniform(0.5, 1.99, size=(M, K)) * np.where(rng.random((M, K)) < 0.05, -1.0, 1.0)   # mostly of one sign: the offset's sums grow with K
    x *= 2.0 ** np.linspace(-110, 127, M).round()[:, None]
    xb = synth.f32_to_bf16_bits(x.astype(np.float32))
    assert np.isfinite(O.bf16_bits_to_f64(xb)).all()
    e = dict(N=N, K=K, group_size=g, x=dev(xb), y=torch.full((M * N,), 0x7FC0, dtype=torch.int16, device="cuda"))
    nx = np.sqrt((O.bf16_bits_to_f64(xb) ** 2).sum(axis=1))
    if bits == 4:
        q, s, z = O.quantize_w4_asym_group(w, g)
        qw, zw = O.pack_w4a16(q, z)
        e.update(qweight=dev(qw), scales=dev(s.view(np.uint16)), zeros=dev(zw))
        ref, (_, nw) = O.w4a16_linear(xb, qw, s, zw, g), O.w4a16_row_norms(xb, qw, s, zw, g)
    else:
        q, s = O.quantize_w8_sym_group(w, g)
        e.update(qweight=dev(O.pack_bytes(q)), scales=dev(s.view(np.uint16)))
        ref = O.w8a16_linear(xb, q, s, g)
        nw = np.sqrt(((q.astype(np.float64) * np.repeat(s.astype(np.float64), g, axis=1)) ** 2).sum(axis=1))
    run(B, bits, [e], M)
    y = host(e["y"], np.uint16).reshape(M, N)
    assert w4a16_norm_err(y, ref, nx, nw) <= TOL
