"""Outputs of the weight-streaming GEMMs at every alignment of a row (row strides and first columns off the four outputs a
lane stores at once, a last 1..3 channels, tokens past a row block), for every format and layout that streams: MXFP4 tiled with one, two and
four row blocks per workgroup and canonical, NVFP4 and INT4 in both layouts with K split across the waves and with shared
activations, one and several groups of tokens.  FP32 output against the FP64 product of the dequantized codes (FP32 sums of at
most 576 exact products: sqrt(576) 2^-24 = 1.4e-6 of the norm, 2e-6 asked), BF16 output the FP32 output rounded to nearest even,
bit for bit, and nothing outside the M x N outputs written."""
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


def _operands(P, rng, M, K, N, fmt, layout, rows):
    """Device operands of both sides and the FP64 product of the given rows (tensor scales 0.5 and 0.25)."""
    import torch
    xc, wc = rng.integers(0, 16, (M, K), dtype=np.uint8), rng.integers(0, 16, (N, K), dtype=np.uint8)
    X, W = O.pack_codes(xc), O.pack_codes(wc)
    if fmt == "mxfp4":
        xs, ws = rng.integers(118, 130, (M, K // 32), dtype=np.uint8), rng.integers(118, 130, (N, K // 32), dtype=np.uint8)
        ref = O.linear_dequant(xc[rows], xs[rows], wc, ws)
    elif fmt == "nvfp4":
        xs, ws = rng.integers(30, 100, (M, K // 16), dtype=np.uint8), rng.integers(30, 100, (N, K // 16), dtype=np.uint8)
        ref = NV.linear_dequant(xc[rows], xs[rows], np.float32(0.5), wc, ws, np.float32(0.25))
    else:
        xs, ws = (O.bf16_values_to_bits(O.round_to_bf16(rng.uniform(0.5, 2.0, (n, K // 32)))) for n in (M, N))
        ref = I4.linear_dequant(I4.unpack_codes(X[rows]), xs[rows], I4.unpack_codes(W), ws)
        xs, ws = (np.ascontiguousarray(s).view(np.uint8).reshape(-1, K // 16) for s in (xs, ws))
    if layout:
        return (*_tiled(P, X, xs, M, K, fmt), *_tiled(P, W, ws, N, K, fmt)), ref
    return tuple(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (X, xs, W, ws)), ref


def _check(P, args, ref, M, K, N, fmt, layout, rows):
    import torch
    ts = [torch.tensor([v], dtype=torch.float32, device="cuda") for v in (0.5, 0.25)]
    for pad, first in ((0, 0), (1, 0), (4, 1), (6, 2), (8, 3)):
        y = {}
        for out, dtype in ((1, torch.float32), (0, torch.bfloat16)):
            whole = torch.full((M + 2, N + pad), 7.0, dtype=dtype, device="cuda")
            Y = whole[1:M + 1, first:first + N]
            if fmt == "mxfp4":
                P.wush_linear(*args, Y, P.default_fmt(out_dtype=out, layout=layout), K=K)
            elif fmt == "nvfp4":
                P.wush_linear_nvfp4(args[0], args[1], ts[0], args[2], args[3], ts[1], Y, layout, out, K=K)
            else:
                P.wush_linear_int4(*args, Y, layout, out, K=K)
            torch.cuda.synchronize()
            y[out] = Y.cpu()
            Y[:] = 7.0
            assert (whole == 7.0).all(), (out, pad, first)
        assert O.rel_fro(y[1].double().numpy()[rows], ref) <= 2e-6, (pad, first)
        assert torch.equal(y[0], y[1].bfloat16()), (pad, first)


# tiled: 1, 2 and 4 row blocks per workgroup (256 compute units), the last with the last workgroups' blocks past the tokens
MXFP4 = [(3, 256, 1, 1), (33, 512, 35, 1), (161, 256, 70, 1), (130, 512, 2051, 1), (130, 256, 4099, 1), (100, 512, 8201, 1),
         (1, 32, 3, 0), (33, 288, 70, 0), (65, 576, 130, 0), (200, 96, 1001, 0)]


@pytest.mark.parametrize("M,K,N,layout", MXFP4)
def test_mxfp4(P, M, K, N, layout):
    rows = np.unique(np.linspace(0, M - 1, 64).astype(int))
    args, ref = _operands(P, np.random.default_rng(M + K + N), M, K, N, "mxfp4", layout, rows)
    switch, value = (P.WUSH_DEBUG_GEMM_SKINNY, 1) if layout else (P.WUSH_DEBUG_GEMM_SIMPLE, 0)
    P.wush_debug_set(switch, value)
    try:
        _check(P, args, ref, M, K, N, "mxfp4", layout, rows)
    finally:
        P.wush_debug_set(switch, -1)


# shared activations; K split with 1 x 1, 1 x 2, 2 x 1, 2 x 2 blocks of tokens and channels per workgroup (at most 16 tokens: one of 16)
@pytest.mark.parametrize("schedule", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("fmt", ["nvfp4", "int4"])
@pytest.mark.parametrize("M,K,N", [(3, 64, 1), (19, 64, 1), (33, 576, 35), (70, 256, 131), (300, 320, 130), (257, 128, 261)])
def test_w4(P, M, K, N, fmt, layout, schedule):
    rows = np.unique(np.linspace(0, M - 1, 64).astype(int))
    args, ref = _operands(P, np.random.default_rng(M + K + N), M, K, N, fmt, layout, rows)
    P.wush_debug_set(P.WUSH_DEBUG_W4_SKINNY, schedule)
    try:
        _check(P, args, ref, M, K, N, fmt, layout, rows)
    finally:
        P.wush_debug_set(P.WUSH_DEBUG_W4_SKINNY, -1)
