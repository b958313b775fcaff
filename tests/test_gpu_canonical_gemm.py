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


# (tokens, K, output channels, row stride past them) -> the kernel with one wavefront per tile (True) or the pipelined one, on
# either side of the rule's lines
SHORT_K = [(64, 128, 520, 0, True), (64, 160, 520, 0, False), (64, 224, 520, 3, True), (64, 256, 520, 3, False),
           (16, 288, 520, 0, True), (17, 288, 520, 0, False), (17, 480, 520, 3, True), (17, 512, 520, 3, False), (16, 512, 520, 0, False),
           (16, 544, 520, 3, False), (2048, 480, 2056, 3, False), (2047, 480, 2048, 3, True), (2048, 160, 8192, 0, True),
           (2047, 160, 8192, 0, False)]


@pytest.mark.parametrize("M,K,N,pad,one_wave", SHORT_K)
def test_short_k_dispatch(P, G, M, K, N, pad, one_wave):
    """Both kernels against the FP64 product where the default changes from one to the other, and the default's bits."""
    import torch
    rng = np.random.default_rng(M + K + N)
    xc, wc = rng.integers(0, 16, (M, K), dtype=np.uint8), rng.integers(0, 16, (N, K), dtype=np.uint8)
    xs, ws = rng.integers(110, 140, (M, K // 32), dtype=np.uint8), rng.integers(110, 140, (N, K // 32), dtype=np.uint8)
    args = (G.u8_dev(O.pack_codes(xc)), G.u8_dev(xs), G.u8_dev(O.pack_codes(wc)), G.u8_dev(ws))
    y = {}
    for forced in (-1, 0, 1):
        Y = torch.full((M + 1, N + pad), 7.0, dtype=torch.float32, device="cuda")
        P.wush_debug_set(P.WUSH_DEBUG_GEMM_SIMPLE, forced)
        try:
            P.wush_linear(*args, Y[:M, :N], P.default_fmt(out_dtype=1))
        finally:
            P.wush_debug_set(P.WUSH_DEBUG_GEMM_SIMPLE, -1)
        assert (Y[M:] == 7.0).all() and (Y[:, N:] == 7.0).all()
        y[forced] = Y[:M, :N].cpu()
    rows = np.unique(np.linspace(0, M - 1, 64).astype(int))
    ref = O.linear_dequant(xc[rows], xs[rows], wc, ws)
    for forced in (0, 1):
        assert O.rel_fro(y[forced].double().numpy()[rows], ref) <= 1e-6
    assert torch.equal(y[-1], y[1 if one_wave else 0])
    if K > 128:
        assert not torch.equal(y[0], y[1])      # they add K in different orders
