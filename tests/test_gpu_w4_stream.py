"""NVFP4 / INT4 layers the weight-streaming kernel takes beyond 128 tokens and in the canonical layout: token counts around its row
blocks, a last block of channels and of tokens that is not whole, K ranges shorter than a workgroup's waves, both schedules, every number of
blocks per workgroup and the default, long K, every output against the FP64 product of the dequantized codes (FP32 accumulation of exact FP16
products, chains of at most 2048 of them: 1e-5 of the norm) and nothing past row M written.  The default's bits say which kernel ran."""
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


# (tokens, K, output channels, layout, the default streams; None: K too short to tell by the bits)
# At most 16 tokens take 16-row kernels of one token block, whatever blocks of tokens are forced: two of them need 17.
SIZES = [(129, 1088, 70, 1, True), (160, 64, 512, 1, None), (300, 512, 130, 1, True), (321, 256, 4100, 1, True),
         (1, 64, 1, 0, None), (1, 1088, 70, 0, True), (31, 512, 2048, 0, True), (33, 192, 8200, 0, None), (100, 256, 130, 0, True),
         (16, 512, 8224, 0, True), (48, 512, 4128, 0, True), (33, 512, 8200, 0, True), (300, 512, 1030, 0, True),
         (17, 64, 1, 0, None), (17, 64, 1, 1, None), (17, 1088, 70, 0, True), (20, 512, 8224, 0, True), (17, 8128, 70, 1, True),
         (130, 1024, 300, 0, True), (1, 8128, 70, 1, True), (33, 8192, 70, 1, True), (70, 8256, 33, 1, True), (2048, 256, 8192, 1, False), (2048, 256, 8192, 0, False)]


@pytest.mark.parametrize("fmt", ["nvfp4", "int4"])
@pytest.mark.parametrize("M,K,N,layout,streams", SIZES)
def test_streaming(P, M, K, N, layout, streams, fmt):
    import torch
    rng = np.random.default_rng(M + K + N)
    xc, wc = rng.integers(0, 16, (M, K), dtype=np.uint8), rng.integers(0, 16, (N, K), dtype=np.uint8)
    X, W = O.pack_codes(xc), O.pack_codes(wc)
    ts = [torch.tensor([v], dtype=torch.float32, device="cuda") for v in (0.5, 0.25)]
    rows = np.unique(np.linspace(0, M - 1, 330).astype(int))
    if fmt == "nvfp4":
        xs, ws = rng.integers(30, 100, (M, K // 16), dtype=np.uint8), rng.integers(30, 100, (N, K // 16), dtype=np.uint8)
        ref = NV.linear_dequant(xc[rows], xs[rows], np.float32(0.5), wc, ws, np.float32(0.25))
    else:
        xs, ws = (O.bf16_values_to_bits(O.round_to_bf16(rng.uniform(0.5, 2.0, (n, K // 32)))) for n in (M, N))
        ref = I4.linear_dequant(I4.unpack_codes(X[rows]), xs[rows], I4.unpack_codes(W), ws)
        xs, ws = (np.ascontiguousarray(s).view(np.uint8).reshape(-1, K // 16) for s in (xs, ws))
    if layout:
        xt, wt = _tiled(P, X, xs, M, K, fmt), _tiled(P, W, ws, N, K, fmt)
    else:
        xt, wt = ([torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in p] for p in ((X, xs), (W, ws)))
    y = {}
    for forced in range(-1, 7):
        Y = torch.full((M + 1, N), 7.0, dtype=torch.float32, device="cuda")
        P.wush_debug_set(P.WUSH_DEBUG_W4_SKINNY, forced)
        try:
            if fmt == "nvfp4":
                P.wush_linear_nvfp4(*xt, ts[0], *wt, ts[1], Y[:M], layout, 1, K=K)
            else:
                P.wush_linear_int4(*xt, *wt, Y[:M], layout, 1, K=K)
        finally:
            P.wush_debug_set(P.WUSH_DEBUG_W4_SKINNY, -1)
        y[forced] = Y[:M].cpu()
        assert (Y[M:] == 7.0).all()
        assert O.rel_fro(y[forced].double().numpy()[rows], ref) <= 1e-5, forced
    for blocks in (3, 4, 5, 6):                 # tokens and channels per workgroup: the same sums
        assert torch.equal(y[blocks], y[1]), blocks
    if K >= 256:                                # the kernels add K in different orders
        assert not torch.equal(y[0], y[1])
        assert torch.equal(y[-1], y[0]) != streams
