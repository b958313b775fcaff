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
