"""Outputs of the NVFP4 / INT4 tile kernels at every alignment of a row (row strides and first columns off 16 bytes, a last
chunk of 1..7 columns, rows past the end), for every tile width, both layouts, with W in registers (K a multiple of 128) and staged:
FP32 output against the FP64 product of the dequantized codes (FP32 accumulation of exact products, K <= 256: 1e-6 of the
norm; K = 8192, whose rows leave in streaming stores: 2 sqrt(K) 2^-24), BF16 output the FP32 output rounded to nearest even, bit
for bit, and nothing outside the M x N outputs written."""
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


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("fmt", ["nvfp4", "int4"])
@pytest.mark.parametrize("width", [2, 3, 4])
@pytest.mark.parametrize("M,K,N", [(129, 128, 1), (140, 192, 259), (257, 256, 390), (290, 64, 520), (161, 8192, 259)])
def test_row_alignments(P, M, K, N, width, fmt, layout):
    import torch
    rng = np.random.default_rng(M + K + N)
    xc, wc = rng.integers(0, 16, (M, K), dtype=np.uint8), rng.integers(0, 16, (N, K), dtype=np.uint8)
    X, W = O.pack_codes(xc), O.pack_codes(wc)
    ts = [torch.tensor([v], dtype=torch.float32, device="cuda") for v in (0.5, 0.25)]
    if fmt == "nvfp4":
        xs, ws = rng.integers(30, 100, (M, K // 16), dtype=np.uint8), rng.integers(30, 100, (N, K // 16), dtype=np.uint8)
        ref = NV.linear_dequant(xc, xs, np.float32(0.5), wc, ws, np.float32(0.25))
    else:
        xs, ws = (O.bf16_values_to_bits(O.round_to_bf16(rng.uniform(0.5, 2.0, (n, K // 32)))) for n in (M, N))
        ref = I4.linear_dequant(I4.unpack_codes(X), xs, I4.unpack_codes(W), ws)
        xs, ws = (np.ascontiguousarray(s).view(np.uint8).reshape(-1, K // 16) for s in (xs, ws))
    if layout:
        xt, wt = _tiled(P, X, xs, M, K, fmt), _tiled(P, W, ws, N, K, fmt)
    else:
        xt, wt = ([torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in p] for p in ((X, xs), (W, ws)))
    P.wush_debug_set(P.WUSH_DEBUG_W4_SKINNY, 0)
    P.wush_debug_set(P.WUSH_DEBUG_W4_WIDTH, width)
    try:
        for pad, first in ((0, 0), (1, 0), (4, 1), (32, 8)):
            y = {}
            for out, dtype in ((1, torch.float32), (0, torch.bfloat16)):
                whole = torch.full((M + 2, N + pad), 7.0, dtype=dtype, device="cuda")
                Y = whole[1:M + 1, first:first + N]
                if fmt == "nvfp4":
                    P.wush_linear_nvfp4(*xt, ts[0], *wt, ts[1], Y, layout, out, K=K)
                else:
                    P.wush_linear_int4(*xt, *wt, Y, layout, out, K=K)
                torch.cuda.synchronize()
                y[out] = Y.cpu()
                Y[:] = 7.0
                assert (whole == 7.0).all(), (out, pad, first)
            assert O.rel_fro(y[1].double().numpy(), ref) <= (1e-6 if K <= 256 else 2 * K ** 0.5 * 2.0 ** -24), (pad, first)
            assert torch.equal(y[0], y[1].bfloat16()), (pad, first)
    finally:
        P.wush_debug_set(P.WUSH_DEBUG_W4_SKINNY, -1)
        P.wush_debug_set(P.WUSH_DEBUG_W4_WIDTH, -1)
