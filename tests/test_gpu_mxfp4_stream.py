"""MXFP4 layers of few 32 x 32 blocks of outputs, which the streaming kernels take: tiled operands beyond 128 tokens (one, two and
four row blocks per workgroup) and canonical ones (whole, partial and no whole K tiles, rows whose scales start at odd bytes), on either
side of the lines where the tiles take over.  Every output against the FP64 product of the dequantized codes (32-bit sums of exact products: 1e-6
of the norm), nothing past row M or column N written; which kernel the default took shows in its bits (they add K in different orders)."""
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


# (tokens, K, output channels, layout, the default streams), 256 compute units
SIZES = [(129, 1280, 70, 1, True), (256, 1024, 1024, 1, True), (257, 1024, 1024, 1, True), (513, 512, 1536, 1, True), (513, 512, 1632, 1, False),
         (1000, 1024, 260, 1, True), (1024, 1024, 1024, 1, True), (1025, 1024, 70, 1, False),
         (449, 512, 1984, 1, True), (768, 1024, 1344, 1, False),
         (1, 1056, 1, 0, True), (33, 544, 130, 0, True), (63, 800, 4096, 0, True), (65, 1024, 4096, 0, False),
         (256, 1024, 1024, 0, True), (257, 1024, 1024, 0, False), (300, 1504, 70, 0, True)]


@pytest.mark.parametrize("M,K,N,layout,streams", SIZES)
def test_streaming(P, M, K, N, layout, streams):
    import torch
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    rng = np.random.default_rng(M + K + N)
    xc, wc = rng.integers(0, 16, (M, K), dtype=np.uint8), rng.integers(0, 16, (N, K), dtype=np.uint8)
    xs, ws = rng.integers(110, 140, (M, K // 32), dtype=np.uint8), rng.integers(110, 140, (N, K // 32), dtype=np.uint8)
    if layout:
        args = (*_tiled(P, O.pack_codes(xc), xs, M, K, "mxfp4"), *_tiled(P, O.pack_codes(wc), ws, N, K, "mxfp4"))
    else:
        args = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (O.pack_codes(xc), xs, O.pack_codes(wc), ws)]
    y = {}
    for forced in (-1, 0):
        Y = torch.full((M + 1, N + 3), 7.0, dtype=torch.float32, device="cuda")
        P.wush_debug_set(P.WUSH_DEBUG_GEMM_SKINNY, forced)
        try:
            P.wush_linear(*args, Y[:M, :N], P.default_fmt(out_dtype=1, layout=layout), K=K)
        finally:
            P.wush_debug_set(P.WUSH_DEBUG_GEMM_SKINNY, -1)
        assert (Y[M:] == 7.0).all() and (Y[:, N:] == 7.0).all()
        y[forced] = Y[:M, :N].cpu()
    rows = np.unique(np.linspace(0, M - 1, 300).astype(int))
    ref = O.linear_dequant(xc[rows], xs[rows], wc, ws)
    for forced in (-1, 0):
        assert O.rel_fro(y[forced].double().numpy()[rows], ref) <= 1e-6
    if N > 1:                                   # a single sum may round alike in both orders
        assert torch.equal(y[-1], y[0]) != streams
