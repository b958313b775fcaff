"""Outputs of the tiled MXFP4 GEMM at every alignment of a row (row strides and first columns off 16 bytes, a last chunk of
1..7 columns, rows past the end), with every tile shape forced: FP32 output within 1e-6 of the norm (32-bit sums of exact
products), BF16 output the FP32 output rounded to nearest even, bit for bit, and nothing outside the M x N outputs written."""
import numpy as np
import pytest

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


def _check(P, args, ref, M, K, N, layout, tile, tol):
    import torch
    P.wush_debug_set(P.WUSH_DEBUG_GEMM_TILE, tile)
    try:
        for pad, first in ((0, 0), (1, 0), (4, 1), (8, 3), (16, 8)):
            y = {}
            for out, dtype in ((1, torch.float32), (0, torch.bfloat16)):
                whole = torch.full((M + 2, N + pad), 7.0, dtype=dtype, device="cuda")
                P.wush_linear(*args, whole[1:M + 1, first:first + N], P.default_fmt(out_dtype=out, layout=layout), K=K)
                torch.cuda.synchronize()
                y[out] = whole[1:M + 1, first:first + N].cpu()
                whole[1:M + 1, first:first + N] = 7.0
                assert (whole == 7.0).all(), (out, pad, first)
            assert O.rel_fro(y[1].double().numpy(), ref) <= tol, (pad, first)
            assert torch.equal(y[0], y[1].bfloat16()), (pad, first)
    finally:
        P.wush_debug_set(P.WUSH_DEBUG_GEMM_TILE, -1)


def _codes(M, K, N):
    rng = np.random.default_rng(M + K + N)
    xc, wc = rng.integers(0, 16, (M, K), dtype=np.uint8), rng.integers(0, 16, (N, K), dtype=np.uint8)
    xs, ws = rng.integers(118, 130, (M, K // 32), dtype=np.uint8), rng.integers(118, 130, (N, K // 32), dtype=np.uint8)
    return O.pack_codes(xc), xs, O.pack_codes(wc), ws, O.linear_dequant(xc, xs, wc, ws)


@pytest.mark.parametrize("tile", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N", [(129, 256, 1), (140, 512, 259), (257, 256, 390), (300, 256, 520)])
def test_row_alignments(P, M, K, N, tile):
    X, xs, W, ws, ref = _codes(M, K, N)
    _check(P, (*_tiled(P, X, xs, M, K, "mxfp4"), *_tiled(P, W, ws, N, K, "mxfp4")), ref, M, K, N, 1, tile, 1e-6)


@pytest.mark.parametrize("layout,tile", [(1, t) for t in range(4)] + [(0, t) for t in range(5)])
@pytest.mark.parametrize("M,K,N", [(161, 4096, 264), (161, 8192, 259)])
def test_long_k(P, M, K, N, layout, tile):
    """K from which rows at multiples of 16 bytes (4096) and at any (8192) leave in streaming stores; 2 sqrt(K) 2^-24 of the norm."""
    import torch
    X, xs, W, ws, ref = _codes(M, K, N)
    if layout:
        args = (*_tiled(P, X, xs, M, K, "mxfp4"), *_tiled(P, W, ws, N, K, "mxfp4"))
    else:
        args = tuple(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (X, xs, W, ws))
    _check(P, args, ref, M, K, N, layout, tile, 2 * K ** 0.5 * 2.0 ** -24)
