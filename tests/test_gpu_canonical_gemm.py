"""The canonical-layout GEMM with every tile shape forced, at the edges of its tiles and steps (rows and columns past the
end, K below, at and past a step of 256, a partial last step of 1..7 groups, odd row strides): every output against the
FP64 product of the dequantized codes.  32-bit sums of exact products: FP32 output within 1e-6 of the norm; BF16 output is
the FP32 output rounded to nearest even, bit for bit; nothing past column N or row M is written."""
import numpy as np
import pytest

from oracle import wush_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2512_00956_amd as P
    P.lib()
    return P


@pytest.fixture(scope="module")
def G():
    from tests import gpu_util
    return gpu_util


SHAPES = [(1, 32, 1), (5, 96, 70), (64, 256, 64), (65, 288, 129), (257, 512, 257), (130, 32 * 23, 300), (300, 1280, 520),
          (33, 32 * 47, 1000)]


@pytest.mark.parametrize("tile", [-1, 0, 1, 2, 3, 4])
@pytest.mark.parametrize("M,K,N", SHAPES)
def test_every_tile_shape(P, G, M, K, N, tile):
    import torch
    rng = np.random.default_rng(M + K + N)
    xc, wc = rng.integers(0, 16, (M, K), dtype=np.uint8), rng.integers(0, 16, (N, K), dtype=np.uint8)
    xs, ws = rng.integers(118, 130, (M, K // 32), dtype=np.uint8), rng.integers(118, 130, (N, K // 32), dtype=np.uint8)
    ref = O.linear_dequant(xc, xs, wc, ws)
    args = (G.u8_dev(O.pack_codes(xc)), G.u8_dev(xs), G.u8_dev(O.pack_codes(wc)), G.u8_dev(ws))
    try:
        P.wush_debug_set(P.WUSH_DEBUG_GEMM_TILE, tile)
        for pad in (0, 3, 8):
            y = {}
            for out, dtype in ((1, torch.float32), (0, torch.bfloat16)):
                Y = torch.full((M + 1, N + pad), 7.0, dtype=dtype, device="cuda")
                P.wush_linear(*args, Y[:M, :N], P.default_fmt(out_dtype=out))
                torch.cuda.synchronize()
                assert (Y[M:] == 7.0).all() and (Y[:, N:] == 7.0).all(), (out, pad)
                y[out] = Y[:M, :N].cpu()
            assert O.rel_fro(y[1].double().numpy(), ref) <= 1e-6, pad
            assert torch.equal(y[0], y[1].bfloat16()), pad
    finally:
        P.wush_debug_set(P.WUSH_DEBUG_GEMM_TILE, -1)


# (tokens, K, output channels, row stride past them, FP32 output) -> the kernel that the default takes, on either side of the rule's
# lines: one wavefront per tile, the pipelined tiles, or (at most 256 blocks of 32 x 32 outputs) the streaming one
SHORT_K = [(2, 128, 520, 0, 1, "one"), (3, 128, 520, 0, 1, "stream"), (2, 160, 520, 0, 1, "stream"), (17, 480, 520, 3, 1, "stream"),
           (16, 128, 8256, 0, 0, "one"), (17, 128, 8256, 0, 0, "one"), (2048, 64, 8192, 0, 0, "one"),
           (2048, 96, 8184, 0, 0, "one"), (2048, 96, 8192, 0, 0, "pipe"), (2048, 96, 8192, 0, 1, "one"),
           (3072, 96, 8191, 0, 0, "one"), (3072, 96, 8193, 0, 0, "pipe"), (3072, 64, 8193, 0, 1, "one"), (3072, 128, 8193, 0, 1, "pipe"),
           (2047, 160, 8192, 0, 1, "pipe"), (2048, 160, 8192, 0, 1, "one"), (2048, 160, 8192, 0, 0, "pipe"),
           (2048, 192, 8191, 0, 1, "one"), (2048, 192, 8193, 0, 1, "pipe"), (1024, 192, 8191, 0, 0, "one"), (1024, 192, 8193, 0, 0, "pipe"),
           (128, 224, 2077, 0, 0, "one"), (129, 224, 2077, 0, 0, "pipe"),
           (16, 480, 8256, 0, 0, "one"), (17, 288, 8256, 0, 0, "pipe"), (16, 544, 8256, 0, 0, "pipe"), (16, 512, 8256, 0, 0, "pipe"),
           (64, 480, 4161, 0, 0, "one"), (65, 352, 4161, 0, 0, "pipe"), (65, 288, 4161, 0, 0, "one"), (65, 352, 4161, 0, 1, "one"),
           (65, 416, 4161, 0, 1, "pipe"), (256, 288, 8191, 0, 0, "one"), (256, 288, 8193, 0, 0, "pipe")]


@pytest.mark.parametrize("M,K,N,pad,out,kernel", SHORT_K)
def test_short_k_dispatch(P, G, M, K, N, pad, out, kernel):
    """Every kernel that could take the layer against the FP64 product where the default changes from one to the other, and the
    default's bits.  BF16 outputs: within the rounding, 2^-9 of the norm."""
    import torch
    rng = np.random.default_rng(M + K + N)
    xc, wc = rng.integers(0, 16, (M, K), dtype=np.uint8), rng.integers(0, 16, (N, K), dtype=np.uint8)
    xs, ws = rng.integers(110, 140, (M, K // 32), dtype=np.uint8), rng.integers(110, 140, (N, K // 32), dtype=np.uint8)
    args = (G.u8_dev(O.pack_codes(xc)), G.u8_dev(xs), G.u8_dev(O.pack_codes(wc)), G.u8_dev(ws))
    streams = ((M + 31) // 32) * ((N + 31) // 32) <= 256
    y = {}
    for run, simple, skinny in (("default", -1, -1), ("one", 1, -1), ("pipe", 0, 0)) + ((("stream", 0, -1),) if streams else ()):
        Y = torch.full((M + 1, N + pad), 7.0, dtype=torch.float32 if out else torch.bfloat16, device="cuda")
        P.wush_debug_set(P.WUSH_DEBUG_GEMM_SIMPLE, simple)
        P.wush_debug_set(P.WUSH_DEBUG_GEMM_SKINNY, skinny)
        try:
            P.wush_linear(*args, Y[:M, :N], P.default_fmt(out_dtype=out))
        finally:
            P.wush_debug_set(P.WUSH_DEBUG_GEMM_SIMPLE, -1)
            P.wush_debug_set(P.WUSH_DEBUG_GEMM_SKINNY, -1)
        assert (Y[M:] == 7.0).all() and (Y[:, N:] == 7.0).all()
        y[run] = Y[:M, :N].cpu()
    rows = np.unique(np.linspace(0, M - 1, 64).astype(int))
    ref = O.linear_dequant(xc[rows], xs[rows], wc, ws)
    for run in y:
        assert O.rel_fro(y[run].double().numpy()[rows], ref) <= (1e-6 if out else 2.0 ** -9), run
    assert torch.equal(y["default"], y[kernel])
    # They add K in different orders.  Up to K = 128 the bits may agree all the same (a thousand BF16 outputs: at 160 as well).
    if K > 128:
        assert not torch.equal(y["pipe"], y["one"])
        assert not streams or not torch.equal(y["stream"], y["one"])
