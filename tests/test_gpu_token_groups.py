"""Weight-streaming GEMMs whose workgroups take only part of the tokens (few output channels) or two weight blocks at a
time: every token count around a row block of 32, layer widths on either side of the dispatch's lines (256 compute units:
32-channel blocks x row blocks against 256 and 768), every output against the FP64 product of the dequantized codes.  MXFP4: FP32 sums
of exact products; NVFP4 and INT4: FP32 accumulation of exact FP16 products, K <= 1024 (1e-5 of the norm)."""
import numpy as np
import pytest

from oracle import wush_int4_oracle as I4
from oracle import wush_nvfp4_oracle as NV
from oracle import wush_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2512_00956_amd as P
    P.lib()
    return P


def _tiled(P, q, s, rows, K, fmt):
    """Tiled buffers of canonical codes and scale bytes (the layouts' definitions: the 16-byte group and scale byte orders
    wush_unpack_tiled* undo), padded as the packed sizes say."""
    import torch
    if fmt == "mxfp4":
        cb, sb = P.wush_packed_sizes(rows, K, P.default_fmt(layout=1))
    else:
        cb, sb = P.wush_packed_sizes_nvfp4(rows, K, 1)
    qt, st = np.zeros(cb, np.uint8), np.zeros(sb, np.uint8)
    r = np.arange(rows)[:, None]
    if fmt == "mxfp4":
        g, KT = np.arange(K // 32)[None, :], K // 256
        rb, ri, kt, kh, kk = r // 32, r % 32, g // 8, (g // 4) % 2, g % 4
        chunk = ((((rb * KT + kt) * 4 + kk) * 64) + kh * 32 + ri) * 16
        st[(((rb * KT + kt) * 64) + kh * 32 + ri) * 4 + kk] = s
    else:
        g, KT = np.arange(K // 32)[None, :], K // 64
        rb, ri, kt = r // 32, r % 32, g // 2
        chunk = (((rb * KT + kt) * 2 + g % 2) * 32 + ri) * 16
        b = np.arange(K // 16)[None, :]
        st[((rb * KT + b // 4) * 32 + ri) * 4 + b % 4] = s
    qt[chunk[..., None] + np.arange(16)] = q.reshape(rows, K // 32, 16)
    return torch.from_numpy(qt).cuda(), torch.from_numpy(st).cuda()


SIZES = [(M, K, N) for M in (1, 32, 33, 64, 65, 96, 100, 128) for (K, N) in ((512, 70), (256, 2048), (1024, 4100))] + [
    (16, 256, 24608), (40, 256, 24608), (100, 256, 24608), (70, 256, 8200)]


@pytest.mark.parametrize("fmt", ["mxfp4", "nvfp4", "int4"])
@pytest.mark.parametrize("M,K,N", SIZES)
def test_few_tokens(P, M, K, N, fmt):
    import torch
    rng = np.random.default_rng(M + K + N)
    xc, wc = rng.integers(0, 16, (M, K), dtype=np.uint8), rng.integers(0, 16, (N, K), dtype=np.uint8)
    X, W = O.pack_codes(xc), O.pack_codes(wc)
    Y = torch.full((M + 1, N), 7.0, dtype=torch.float32, device="cuda")
    if fmt == "mxfp4":
        xs, ws = rng.integers(120, 130, (M, K // 32), dtype=np.uint8), rng.integers(120, 130, (N, K // 32), dtype=np.uint8)
        ref = O.linear_dequant(xc, xs, wc, ws)
        P.wush_debug_set(P.WUSH_DEBUG_GEMM_SKINNY, 1)
        try:
            P.wush_linear(*_tiled(P, X, xs, M, K, fmt), *_tiled(P, W, ws, N, K, fmt), Y[:M], P.default_fmt(out_dtype=1, layout=1), K=K)
        finally:
            P.wush_debug_set(P.WUSH_DEBUG_GEMM_SKINNY, -1)
    elif fmt == "nvfp4":
        xs, ws = rng.integers(30, 100, (M, K // 16), dtype=np.uint8), rng.integers(30, 100, (N, K // 16), dtype=np.uint8)
        ref = NV.linear_dequant(xc, xs, np.float32(0.5), wc, ws, np.float32(0.25))
        tsx, tsw = (torch.tensor([v], dtype=torch.float32, device="cuda") for v in (0.5, 0.25))
        xt, wt = _tiled(P, X, xs, M, K, fmt), _tiled(P, W, ws, N, K, fmt)
        P.wush_linear_nvfp4(*xt, tsx, *wt, tsw, Y[:M], 1, 1, K=K)
    else:
        xs, ws = (O.bf16_values_to_bits(O.round_to_bf16(rng.uniform(0.5, 2.0, (n, K // 32)))) for n in (M, N))
        ref = I4.linear_dequant(I4.unpack_codes(X), xs, I4.unpack_codes(W), ws)
        xt = _tiled(P, X, np.ascontiguousarray(xs).view(np.uint8).reshape(M, K // 16), M, K, fmt)
        wt = _tiled(P, W, np.ascontiguousarray(ws).view(np.uint8).reshape(N, K // 16), N, K, fmt)
        P.wush_linear_int4(*xt, *wt, Y[:M], 1, 1, K=K)
    torch.cuda.synchronize()
    assert O.rel_fro(Y[:M].double().cpu().numpy(), ref) <= 1e-5
    assert (Y[M:] == 7.0).all()


# blocks of 32 output channels per compute unit (256 of them) -> schedule (1: K split over a workgroup's waves, 2: activations
# shared), on either side of every line of the rule
SCHEDULES = [("int4", 5, 1), ("int4", 6, 1), ("int4", 6.125, 2), ("int4", 8, 2), ("int4", 8.125, 1), ("int4", 9, 1), ("int4", 9.125, 2),
             ("nvfp4", 6.875, 1), ("nvfp4", 7, 2), ("nvfp4", 8, 2), ("nvfp4", 8.125, 1), ("nvfp4", 10, 1), ("nvfp4", 10.125, 2)]


@pytest.mark.parametrize("fmt,blocks,schedule", SCHEDULES)
def test_schedule_by_output_channels(P, fmt, blocks, schedule):
    """65..128 tokens: the schedules add K in different orders, so the default's bits tell which one ran."""
    import torch
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    M, K, N = 70, 512, int(32 * 256 * blocks)
    g = torch.Generator(device="cuda").manual_seed(N)
    size = lambda rows: P.wush_packed_sizes_nvfp4(rows, K, 1)
    codes = lambda rows: torch.randint(0, 256, (size(rows)[0],), dtype=torch.uint8, device="cuda", generator=g)
    if fmt == "nvfp4":
        scales = lambda rows: torch.randint(30, 100, (size(rows)[1],), dtype=torch.uint8, device="cuda", generator=g)
    else:
        scales = lambda rows: (torch.rand(size(rows)[1] // 2, device="cuda", generator=g) + 0.5).bfloat16().view(torch.uint8)
    X, W, ts = (codes(M), scales(M)), (codes(N), scales(N)), torch.ones(1, device="cuda")
    y = {}
    for forced in (-1, 1, 2):
        Y = torch.empty(M, N, device="cuda")
        P.wush_debug_set(P.WUSH_DEBUG_W4_SKINNY, forced)
        try:
            if fmt == "nvfp4":
                P.wush_linear_nvfp4(*X, ts, *W, ts, Y, 1, 1, K=K)
            else:
                P.wush_linear_int4(*X, *W, Y, 1, 1, K=K)
        finally:
            P.wush_debug_set(P.WUSH_DEBUG_W4_SKINNY, -1)
        y[forced] = Y
    assert not torch.equal(y[1], y[2]) and torch.equal(y[-1], y[schedule])
