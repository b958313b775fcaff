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
