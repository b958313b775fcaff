"""At most 16 tokens on the 16-row matrix instructions, all formats and both layouts: token counts on either side of 16, output channels at the
edges of half blocks, of whole blocks and of the grid that takes halves (4096 on 256 compute units), K at the edges of the kernels' rings and
wavefront ranges, an odd number of K steps, partial last tiles.  Every output against the FP64 product of the dequantized codes (32-bit
sums of exact products: 1e-6 of the norm for MXFP4; FP16 products of the other formats, chains of up to 2048: 1e-5), BF16 outputs the FP32
ones rounded to nearest even, nothing past row M or column N written."""
import numpy as np
import pytest

from oracle import wush_int4_oracle as I4
from oracle import wush_nvfp4_oracle as NV
from oracle import wush_oracle as O
from tests.test_gpu_token_groups import _tiled

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2512_00956_amd as P
    P.lib()
    return P


def _operands(P, fmt, layout, M, K, N):
    """(call(Y, out_dtype), reference of columns `cols`, cols)"""
    import torch
    rng = np.random.default_rng(M + K + N)
    xc, wc = rng.integers(0, 16, (M, K), dtype=np.uint8), rng.integers(0, 16, (N, K), dtype=np.uint8)
    X, W = O.pack_codes(xc), O.pack_codes(wc)
    cols = np.unique(np.concatenate([np.linspace(0, N - 1, 200), np.arange(max(0, N - 40), N)]).astype(int))
    if fmt == "mxfp4":
        xs, ws = rng.integers(110, 140, (M, K // 32), dtype=np.uint8), rng.integers(110, 140, (N, K // 32), dtype=np.uint8)
        ref = O.linear_dequant(xc, xs, wc[cols], ws[cols])
    elif fmt == "nvfp4":
        xs, ws = rng.integers(30, 100, (M, K // 16), dtype=np.uint8), rng.integers(30, 100, (N, K // 16), dtype=np.uint8)
        ref = NV.linear_dequant(xc, xs, np.float32(0.5), wc[cols], ws[cols], np.float32(0.25))
    else:
        xs, ws = (O.bf16_values_to_bits(O.round_to_bf16(rng.uniform(0.5, 2.0, (n, K // 32)))) for n in (M, N))
        ref = I4.linear_dequant(I4.unpack_codes(X), xs, I4.unpack_codes(W[cols]), ws[cols])
        xs, ws = (np.ascontiguousarray(s).view(np.uint8).reshape(-1, K // 16) for s in (xs, ws))
    if layout:
        xt, wt = _tiled(P, X, xs, M, K, fmt), _tiled(P, W, ws, N, K, fmt)
    else:
        xt, wt = ([torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in p] for p in ((X, xs), (W, ws)))
    ts = [torch.tensor([v], dtype=torch.float32, device="cuda") for v in (0.5, 0.25)]

    def call(Y, out):
        if fmt == "mxfp4":
            P.wush_linear(*xt, *wt, Y, P.default_fmt(out_dtype=out, layout=layout), K=K)
        elif fmt == "nvfp4":
            P.wush_linear_nvfp4(*xt, ts[0], *wt, ts[1], Y, layout, out, K=K)
        else:
            P.wush_linear_int4(*xt, *wt, Y, layout, out, K=K)
    return call, ref, cols


def _outputs(call, M, N, out):
    import torch
    Y = torch.full((M + 1, N + 3), 7.0, dtype=torch.float32 if out else torch.bfloat16, device="cuda")
    call(Y[:M, :N], out)
    assert (Y[M:] == 7.0).all() and (Y[:, N:] == 7.0).all()
    return Y[:M, :N].cpu()


SIZES = {("mxfp4", 1): [(1, 256, 1), (16, 512, 17), (15, 2048, 4096), (16, 2304, 4097), (1, 4352, 4095), (16, 8448, 70), (17, 2304, 100)],
         ("mxfp4", 0): [(1, 288, 1), (16, 1056, 17), (15, 2048, 4096), (16, 2080, 4097), (1, 2336, 4095), (16, 4128, 4130), (16, 8416, 70),
                        (17, 2080, 100)],
         ("w4", 1): [(1, 64, 1), (16, 192, 17), (15, 2048, 300), (16, 2112, 300), (1, 4160, 95), (16, 576, 24640), (17, 2112, 100)],
         ("w4", 0): [(1, 64, 1), (16, 192, 17), (15, 1024, 300), (16, 1088, 300), (9, 4160, 95), (16, 576, 1030), (17, 1088, 100)]}


@pytest.mark.parametrize("fmt,layout,M,K,N", [(f, lay, *s) for (kind, lay), sizes in SIZES.items()
                                              for f in (("mxfp4",) if kind == "mxfp4" else ("nvfp4", "int4")) for s in sizes])
def test_sixteen_tokens(P, fmt, layout, M, K, N):
    import torch
    call, ref, cols = _operands(P, fmt, layout, M, K, N)
    y = _outputs(call, M, N, 1)
    assert O.rel_fro(y.double().numpy()[:, cols], ref) <= (1e-6 if fmt == "mxfp4" else 1e-5)
    assert torch.equal(_outputs(call, M, N, 0), y.bfloat16())


# canonical MXFP4 layers of more blocks of 32 channels than compute units, on either side of the lines: (tokens, K, blocks a compute unit, channels
# past them, streams)
@pytest.mark.parametrize("M,K,rounds,more,streams", [(4, 2560, 2, 32, True), (4, 2816, 2, 32, False), (4, 2816, 2, 0, True), (5, 2560, 1, 32, False),
                                                     (16, 12288, 1, 32, True), (16, 12032, 1, 32, False), (1, 12288, 2, 32, False)])
def test_wide_canonical_layers(P, M, K, rounds, more, streams):
    import torch
    N = 32 * torch.cuda.get_device_properties(0).multi_processor_count * rounds + more
    call, ref, cols = _operands(P, "mxfp4", 0, M, K, N)
    y = _outputs(call, M, N, 1)
    P.wush_debug_set(P.WUSH_DEBUG_GEMM_SKINNY, 0)
    try:
        tiles = _outputs(call, M, N, 1)
    finally:
        P.wush_debug_set(P.WUSH_DEBUG_GEMM_SKINNY, -1)
    for out in (y, tiles):
        assert O.rel_fro(out.double().numpy()[:, cols], ref) <= 1e-6
    # the kernels add K in different orders: of the 30000 outputs and more some differ in their last bits, and none where both are the tiles
    assert torch.equal(y, tiles) != streams


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("M", [1, 16, 17])
@pytest.mark.parametrize("K", [64, 128, 192, 1088])
def test_int4_infinite_scale_in_the_last_step(P, layout, M, K):
    """An output of positive codes, one group of whose weights has an infinite scale, is infinite: what stands in for the missing step of
    an odd number has to be zero in both operands.  The other outputs are exact (code 1 in every place: K)."""
    import torch
    N = 40
    X, W = (np.full((n, K // 2), 0x11, dtype=np.uint8) for n in (M, N))
    xs, ws = (O.bf16_values_to_bits(np.ones((n, K // 32))) for n in (M, N))
    ws[5, -1] = 0x7F80
    xs, ws = (np.ascontiguousarray(s).view(np.uint8).reshape(-1, K // 16) for s in (xs, ws))
    if layout:
        args = (*_tiled(P, X, xs, M, K, "int4"), *_tiled(P, W, ws, N, K, "int4"))
    else:
        args = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (X, xs, W, ws)]
    Y = torch.empty((M, N), dtype=torch.float32, device="cuda")
    P.wush_linear_int4(*args, Y, layout, 1, K=K)
    ref = torch.full((M, N), float(K))
    ref[:, 5] = float("inf")
    assert torch.equal(Y.cpu(), ref)


@pytest.mark.parametrize("layout,M", [(0, 1), (1, 3), (1, 20), (1, 40)])
def test_more_blocks_than_a_grid_is_wide(P, layout, M):
    """2^20 blocks of 32 channels and three more, the last one partial: the grid goes on along z.  The channels on either side of the line and the
    last ones against a call of those alone, bit for bit."""
    import torch
    K, N, C = 256, (1 << 25) + 77, 8
    g = torch.Generator(device="cuda").manual_seed(M)
    rows, tokens = N + -N % 256, M + -M % 256                # as many as a tiled operand has
    X, W = (torch.randint(0, 256, (r, K // 2), dtype=torch.uint8, device="cuda", generator=g) for r in (tokens, rows))
    xs, ws = (torch.randint(110, 140, (r, C), dtype=torch.uint8, device="cuda", generator=g) for r in (tokens, rows))
    fmt = P.default_fmt(out_dtype=0, layout=layout)          # random bytes are an operand in either layout; a block of 32 rows is contiguous

    def call(first, n):
        Y = torch.full((M, n + 3), 7.0, dtype=torch.bfloat16, device="cuda")
        last = first + n + -n % 256
        w = W[first:last] if layout else W[first:first + n]
        s = ws[first:last] if layout else ws[first:first + n]
        x, t = (X, xs) if layout else (X[:M], xs[:M])
        P.wush_linear(x, t, w, s, Y[:, :n], fmt, K=K)
        assert (Y[:, n:] == 7.0).all()
        return Y[:, :n]
    P.wush_debug_set(P.WUSH_DEBUG_GEMM_SKINNY, 1)            # 40 tokens of so many channels take the tiles by themselves
    try:
        Y = call(0, N)
        for first in (0, (1 << 25) - 64):
            part = Y[:, first:first + 141]
            assert torch.equal(part, call(first, 141)[:, :part.shape[1]])
    finally:
        P.wush_debug_set(P.WUSH_DEBUG_GEMM_SKINNY, -1)
    assert torch.isfinite(Y).all()


@pytest.mark.parametrize("schedule", [2, 3, 4, 6])
@pytest.mark.parametrize("fmt", ["nvfp4", "int4"])
@pytest.mark.parametrize("layout,M", [(0, 1), (1, 3), (1, 16), (0, 17), (1, 40), (1, 70)])
def test_w4_more_blocks_than_workgroups(P, fmt, layout, M, schedule):
    """The streaming kernels of these formats launch 4096 workgroups side by side at most, each of which goes on to further blocks: one weight block
    at a time (schedule 3), two (4, 6) or, shared activations, four (2).  The channels on either side of the lines and the last ones against a
    call of those alone, bit for bit."""
    import torch
    K, N = 64, 4096 * 4 * 32 + 101
    g = torch.Generator(device="cuda").manual_seed(M)

    def operand(rows):
        q, s = (torch.randint(lo, hi, (rows + -rows % 32, n), dtype=torch.uint8, device="cuda", generator=g) for lo, hi, n in ((0, 256, K // 2), (30, 100, K // 16)))
        if fmt == "int4":
            s = (torch.rand((s.shape[0], K // 32), device="cuda", generator=g) + 0.5).bfloat16().view(torch.uint8)
        return q, s
    x, w = operand(M), operand(N)                            # random bytes are an operand in either layout; a block of 32 rows is contiguous
    ts = [torch.tensor([v], dtype=torch.float32, device="cuda") for v in (0.5, 0.25)]

    def call(first, n):
        Y = torch.full((M, n + 3), 7.0, dtype=torch.bfloat16, device="cuda")
        wq, ws = (t[first:first + n + -n % 32] for t in w)
        if fmt == "nvfp4":
            P.wush_linear_nvfp4(*x, ts[0], wq, ws, ts[1], Y[:, :n], layout, 0, K=K)
        else:
            P.wush_linear_int4(*x, wq, ws, Y[:, :n], layout, 0, K=K)
        assert (Y[:, n:] == 7.0).all()
        return Y[:, :n]
    P.wush_debug_set(P.WUSH_DEBUG_W4_SKINNY, schedule)
    try:
        Y = call(0, N)
        for first in (0, 4096 * 32 - 64, 4096 * 64 - 64, 4096 * 128 - 64):
            assert torch.equal(Y[:, first:first + 165], call(first, min(165, N - first))), first
    finally:
        P.wush_debug_set(P.WUSH_DEBUG_W4_SKINNY, -1)
    assert torch.isfinite(Y).all()
