"""Weight preparation at the edges of its tiles (16 rows per wavefront, four blocks of 32 channels per workgroup) and at
the ends of the scale range, where the 32-bit decisions give way to FP64 ones: every code and scale byte against the
oracle's FP64 definition (differences only next to a rounding boundary: 1e-9 of the group's maximum, as the other weight
tests)."""
import numpy as np
import pytest

import wush_inputs as I
from oracle import wush_int4_oracle as I4
from oracle import wush_nvfp4_oracle as NV
from oracle import wush_oracle as O
from tests import kernel_models as KM

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


SHAPES = [(1, 32), (15, 96), (16, 128), (17, 160), (33, 288), (700, 32 * 9)]


def _weights(N, K, spread):
    rng = np.random.default_rng(7 * N + K)
    w = rng.standard_normal((N, K))
    if spread:
        # rows from the smallest magnitudes (scale byte 0) to the largest a row can have and stay finite, a zero row
        e = np.linspace(-132.0, 121.0, N) if N > 1 else np.array([-130.0])
        w = np.ldexp(w, np.round(e).astype(int)[:, None])
        w[N // 2] = 0.0
    return O.round_to_bf16(w)


@pytest.mark.parametrize("N,K", SHAPES)
@pytest.mark.parametrize("spread", [False, True])
@pytest.mark.parametrize("rule", ["nosat", "ocp_floor"])
def test_mxfp4(P, G, N, K, spread, rule):
    W = _weights(N, K, spread)
    Tb = I.make_transforms_random(K // 32, 5)
    T = O.bf16_bits_to_f64(Tb)
    Wq, Ws, ws = G.empty_u8(N, K // 2), G.empty_u8(N, K // 32), G.empty_u8(P.wush_prepare_weight_workspace(N, K))
    fmt = P.default_fmt(scale_rule={"nosat": 0, "ocp_floor": 1}[rule])
    P.wush_prepare_weight(G.bf16_dev(O.bf16_values_to_bits(W)), G.bf16_dev(Tb), Wq, Ws, ws, fmt)
    P.wush_workspace_status(ws, K)
    Wt = O.transform_weight(W, T)
    cr, sr = O.quantize_mxfp4(Wt, rule)
    rate, unexplained = G.code_mismatch_report(Wt, O.unpack_codes(G.host(Wq)), G.host(Ws), cr, sr, tol=1e-9)
    assert rate <= 1e-4 and unexplained == 0, (rate, unexplained)


@pytest.mark.parametrize("N,K", SHAPES)
def test_nvfp4(P, G, N, K):
    import torch
    W = _weights(N, K, False) * np.exp2(np.round(np.linspace(-12, 3, N)))[:, None]     # small groups: subnormal scales, byte 0
    Tb = I.make_transforms_random(K // 16, 6, block=16)
    T = O.bf16_bits_to_f64(Tb)
    Wq, Ws, ws = G.empty_u8(N, K // 2), G.empty_u8(N, K // 16), G.empty_u8(P.wush_prepare_weight_nvfp4_workspace(K))
    tsw = torch.zeros(1, dtype=torch.float32, device="cuda")
    P.wush_prepare_weight_nvfp4(G.bf16_dev(O.bf16_values_to_bits(W)), G.bf16_dev(Tb), Wq, Ws, tsw, ws)
    P.wush_prepare_weight_nvfp4_status(ws, K)
    Wt = NV.transform_weight(W, T)
    ts = np.float32(tsw.cpu().numpy()[0])
    assert abs(float(ts) - float(NV.tensor_scale(Wt))) <= 1.2e-7 * float(ts)
    cr, sr = NV.quantize_nvfp4(Wt, ts)
    rate, unexplained = KM.nvfp4_explained(Wt, ts, O.unpack_codes(G.host(Wq)), G.host(Ws), cr, sr, tol=1e-9)
    assert rate <= 1e-4 and unexplained == 0, (rate, unexplained)


@pytest.mark.parametrize("N,K", SHAPES)
def test_int4(P, G, N, K):
    W = _weights(N, K, False) * np.exp2(np.round(np.linspace(-20, 20, N)))[:, None]
    Tb = I.make_transforms_random(K // 32, 8)
    T = O.bf16_bits_to_f64(Tb)
    Wq, Ws, ws = G.empty_u8(N, K // 2), G.empty_u8(N, K // 16), G.empty_u8(P.wush_prepare_weight_workspace(N, K))
    P.wush_prepare_weight_int4(G.bf16_dev(O.bf16_values_to_bits(W)), G.bf16_dev(Tb), Wq, Ws, ws)
    P.wush_workspace_status(ws, K)
    Wt = O.transform_weight(W, T)
    qr, sr = I4.quantize_int4(Wt)
    sg = G.host(Ws).view(np.uint16).reshape(N, K // 32)
    rate, unexplained = KM.int4_explained(Wt, I4.unpack_codes(G.host(Wq)), sg, qr, sr, tol=1e-9)
    assert rate <= 1e-4 and unexplained == 0, (rate, unexplained)


# Transformed weights past FP32's range (finite weights, a transform that is legitimate BF16): one group whose maximum lies
# in 2^128 .. 2^129, one from 2^129 on, groups that lie far above altogether (the scale byte saturates at 254, the codes
# at 6), each next to ordinary rows of the same 16-row tile.
def _beyond_float(scale_exp):
    rng = np.random.default_rng(3)
    N, K = 33, 160
    T = np.broadcast_to(O.round_to_bf16(np.ldexp(O.hadamard(), scale_exp)), (K // 32, 32, 32)).copy()
    W = rng.standard_normal((N, K))
    if scale_exp == 0:
        for row, e in ((2, 126.0), (3, 126.75), (17, 127.0)):        # maxima 31 w / sqrt(32): 2^128.45, 2^129.2, 2^129.45
            W[row] = 2.0 ** e
            W[row, ::32] = 1.0
    else:
        W *= np.ldexp(1.0, np.where(np.arange(N) % 3 == 0, 100, 0))[:, None]
    return O.round_to_bf16(W), T


@pytest.mark.parametrize("scale_exp", [0, -40, -100])
@pytest.mark.parametrize("rule", ["nosat", "ocp_floor"])
def test_mxfp4_past_float_range(P, G, scale_exp, rule):
    W, T = _beyond_float(scale_exp)
    N, K = W.shape
    Wt = O.transform_weight(W, T)
    assert np.isfinite(W).all() and np.abs(Wt).max() >= 2.0 ** 129
    Wq, Ws, ws = G.empty_u8(N, K // 2), G.empty_u8(N, K // 32), G.empty_u8(P.wush_prepare_weight_workspace(N, K))
    fmt = P.default_fmt(scale_rule={"nosat": 0, "ocp_floor": 1}[rule])
    P.wush_prepare_weight(G.bf16_dev(O.bf16_values_to_bits(W)), G.bf16_dev(O.bf16_values_to_bits(T)), Wq, Ws, ws, fmt)
    P.wush_workspace_status(ws, K)
    cr, sr = O.quantize_mxfp4(Wt, rule)
    # a BF16 Hadamard block has few bits, so codes do fall on exact ties, which a summation order decides: 1e-9 as above
    rate, unexplained = G.code_mismatch_report(Wt, O.unpack_codes(G.host(Wq)), G.host(Ws), cr, sr, tol=1e-9)
    assert np.array_equal(G.host(Ws), sr) and rate <= 1e-2 and unexplained == 0, (rate, unexplained)


def test_non_finite_weights(P, G):
    """An infinite weight saturates its group (byte 254, codes of magnitude 6); a NaN counts as no magnitude (code 0); other
    rows of the tile are what they are without them."""
    import torch
    rng = np.random.default_rng(4)
    N, K = 20, 64
    Tb = O.bf16_values_to_bits(O.round_to_bf16(np.broadcast_to(O.hadamard(), (2, 32, 32)).copy()))
    T16 = O.bf16_values_to_bits(O.round_to_bf16(np.broadcast_to(O.hadamard(16), (4, 16, 16)).copy()))
    bits = O.bf16_values_to_bits(O.round_to_bf16(rng.standard_normal((N, K))))
    clean = bits.copy()
    bits[3, 5], bits[9, 40] = 0x7F80, 0x7FC0
    out = {}
    for name, w in (("clean", clean), ("dirty", bits)):
        Wq, Ws, ws = G.empty_u8(N, K // 2), G.empty_u8(N, K // 32), G.empty_u8(P.wush_prepare_weight_workspace(N, K))
        P.wush_prepare_weight(G.bf16_dev(w), G.bf16_dev(Tb), Wq, Ws, ws)
        out[name] = O.unpack_codes(G.host(Wq)), G.host(Ws)
    c, s = out["dirty"]
    assert (c[3, :32] & 7 == 7).all() and s[3, 0] == 254
    assert (c[9, 32:] & 7 == 0).all() and s[9, 1] == 0
    keep = np.ones((N, 2), bool)
    keep[3, 0] = keep[9, 1] = False
    assert (out["clean"][1] == s)[keep].all() and (out["clean"][0] == c).reshape(N, 2, 32)[keep].all()
    # NVFP4: the NaN's group of 16 only (an infinite weight would leave no tensor scale)
    bits[3, 5] = clean[3, 5]
    for name, w in (("clean", clean), ("dirty", bits)):
        Wq, Ws, ws = G.empty_u8(N, K // 2), G.empty_u8(N, K // 16), G.empty_u8(P.wush_prepare_weight_nvfp4_workspace(K))
        ts = torch.zeros(1, dtype=torch.float32, device="cuda")
        P.wush_prepare_weight_nvfp4(G.bf16_dev(w), G.bf16_dev(T16), Wq, Ws, ts, ws)
        out[name] = O.unpack_codes(G.host(Wq)), G.host(Ws), float(ts)
    c, s, ts = out["dirty"]
    assert (c[9, 32:48] & 7 == 0).all() and s[9, 2] == 0
    keep = np.ones((N, 4), bool)
    keep[9, 2] = False
    if ts == out["clean"][2]:
        assert (out["clean"][1] == s)[keep].all() and (out["clean"][0] == c).reshape(N, 4, 16)[keep].all()
