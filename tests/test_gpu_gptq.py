"""GPU parity of wush_prepare_weight_gptq (Alg. 2, GPTQ case) against the FP64 oracle.

The schedule is sequential with feedback: a transform entry that lands on the other side of a
BF16 rounding boundary, or a weight code that flips at an exact tie, changes everything after
it a little.  Both sides are FP64 with different summation orders (1e-16 relative), so such an
event needs a value within 1e-15 of a boundary: on the layers below none occurs and the outputs
are identical (also on the full c2 layer, 25 million codes).  The bars are set at that level:
at most 1e-4 of the transform entries (each one BF16 step apart), of the scales and of the codes
may differ -- on these sizes that is a handful of elements at most, where a wrong index in the
propagation of a single block shifts every later block (a tenth of all codes or more) -- and the
output error GPTQ minimizes must equal the oracle's to 1e-6 when nothing differs, 1e-3 otherwise.
"""
import numpy as np
import pytest

import wush_inputs as I
from oracle import wush_gptq_oracle as Q
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


def _layer(M, K, N, Mc, seed_mix=7, n_outlier=3):
    cfg = I.scaled(I.CONFIGS["c2"], M=M, K=K, N=N, calib_tokens=Mc, n_outlier=n_outlier)
    L = I.make_layer(cfg)
    # correlate the channels (the generator draws them independently; GPTQ's propagation acts on correlations);
    # the mixed calibration set is rounded to BF16 again because that is what both sides read
    rng = np.random.default_rng(seed_mix)
    mix = np.eye(K) + 0.3 * rng.standard_normal((K, K)) / np.sqrt(K)
    Xc = O.round_to_bf16(O.bf16_bits_to_f64(L["X_cal"]) @ mix)
    X = O.round_to_bf16(O.bf16_bits_to_f64(L["X"]) @ mix)
    return O.bf16_bits_to_f64(L["W"]), Xc, X


def _run_gpu(P, G, W, Xc, lam, layout=0, T_given=None):
    import torch
    N, K = W.shape
    fmt = P.default_fmt(layout=layout)
    Wd, Xd = G.bf16_dev(O.bf16_values_to_bits(W)), G.bf16_dev(O.bf16_values_to_bits(Xc))
    if T_given is None:
        Td = torch.full((K // 32, 32, 32), float("nan"), dtype=torch.bfloat16, device="cuda")
    else:
        Td = G.bf16_dev(O.bf16_values_to_bits(T_given))
    cb, sb = P.wush_packed_sizes(N, K, fmt)
    Wq = torch.full((cb,), 0xEE, dtype=torch.uint8, device="cuda")
    Ws = torch.full((sb,), 0xEE, dtype=torch.uint8, device="cuda")
    wsp = torch.empty(P.wush_prepare_weight_gptq_workspace(N, K), dtype=torch.uint8, device="cuda")
    P.wush_prepare_weight_gptq(Wd, Xd, lam, Td, Wq, Ws, wsp, fmt, transform_given=T_given is not None)
    P.wush_prepare_weight_gptq_status(wsp, N, K)
    if layout:
        q, s = G.empty_u8(N, K // 2), G.empty_u8(N, K // 32)
        P.wush_unpack_tiled(Wq, Ws, N, K, q, s)
    else:
        q, s = Wq.view(N, K // 2), Ws.view(N, K // 32)
    torch.cuda.synchronize()
    return O.bf16_bits_to_f64(G.host(Td)), O.unpack_codes(G.host(q)), G.host(s)


def _compare(T_gpu, c_gpu, s_gpu, T_ref, c_ref, s_ref, W, X, what):
    dT = T_gpu != T_ref
    step = np.abs(T_gpu - T_ref) / np.maximum(np.abs(T_ref), 1e-30)
    print(f"{what}: T entries differing {dT.mean():.2e} (max relative step {step.max():.2e}), "
          f"scales differing {np.mean(s_gpu != s_ref):.2e}, codes differing {np.mean(c_gpu != c_ref):.2e}")
    n_diff = int(dT.sum()) + int(np.sum(s_gpu != s_ref)) + int(np.sum(c_gpu != c_ref))
    assert dT.mean() <= 1e-4 and step.max() <= 2.0 ** -7          # at most one BF16 step
    assert np.mean(s_gpu != s_ref) <= 1e-4
    assert np.mean(c_gpu != c_ref) <= 1e-4
    l_gpu, l_ref = Q.proxy_loss(T_gpu, c_gpu, s_gpu, W, X), Q.proxy_loss(T_ref, c_ref, s_ref, W, X)
    print(f"{what}: weight-only output MSE  oracle {l_ref:.5e}  GPU {l_gpu:.5e}  ({n_diff} differing values)")
    assert abs(l_gpu - l_ref) <= (1e-6 if n_diff == 0 else 1e-3) * l_ref
    return l_gpu


@pytest.mark.parametrize("N,K,Mc,layout", [(48, 128, 400, 0), (300, 512, 1024, 1), (77, 416, 1000, 0)])
def test_gptq_wush_against_oracle(P, G, N, K, Mc, layout):
    W, Xc, X = _layer(64, K, N, Mc)
    T_ref, c_ref, s_ref = Q.gptq_wush_layer(W, Xc, 1e-2)
    T_gpu, c_gpu, s_gpu = _run_gpu(P, G, W, Xc, 1e-2, layout)
    l_gptq = _compare(T_gpu, c_gpu, s_gpu, T_ref, c_ref, s_ref, W, X, f"N={N} K={K}")
    # and it does what it is for: lower output error than the RTN case on the same layer
    T0 = O.round_to_bf16(O.build_transforms(W, Xc, 1e-2))
    c0, s0 = O.quantize_mxfp4(O.transform_weight(W, T0))
    assert l_gptq < Q.proxy_loss(T0, c0, s0, W, X)


@pytest.mark.parametrize("transform", ["hadamard", "identity"])
def test_gptq_with_a_given_transform(P, G, transform):
    N, K, Mc = 96, 256, 800
    W, Xc, X = _layer(64, K, N, Mc)
    T_ref, c_ref, s_ref = Q.gptq_wush_layer(W, Xc, 1e-2, transform=transform)
    T_gpu, c_gpu, s_gpu = _run_gpu(P, G, W, Xc, 1e-2, 0, T_given=T_ref)
    assert np.array_equal(T_gpu, T_ref)                            # an input: untouched
    _compare(T_gpu, c_gpu, s_gpu, T_ref, c_ref, s_ref, W, X, transform)


def test_gptq_reports_a_hessian_that_is_not_positive_definite(P, G):
    import torch
    N, K = 32, 64
    W, _, _ = _layer(8, K, N, 64)
    Xc = np.zeros((64, K))
    Wd, Xd = G.bf16_dev(O.bf16_values_to_bits(W)), G.bf16_dev(O.bf16_values_to_bits(Xc))
    Td = torch.zeros((K // 32, 32, 32), dtype=torch.bfloat16, device="cuda")
    Wq, Ws = G.empty_u8(N, K // 2), G.empty_u8(N, K // 32)
    wsp = torch.empty(P.wush_prepare_weight_gptq_workspace(N, K), dtype=torch.uint8, device="cuda")
    P.wush_prepare_weight_gptq(Wd, Xd, 0.0, Td, Wq, Ws, wsp)
    with pytest.raises(P.WushError) as ei:
        P.wush_prepare_weight_gptq_status(wsp, N, K)
    assert ei.value.code == 7


def test_gptq_layer_runs_through_the_online_path(P, G):
    """The outputs plug into the unchanged online path: quantize activations with the returned T,
    multiply with the returned codes; the W4A4 layer loss beats RTN + Hadamard (direction of the paper's tables)."""
    import torch
    M, K, N, Mc = 64, 512, 256, 2048
    W, Xc, X = _layer(M, K, N, Mc)
    fmt = P.default_fmt(layout=1)
    T_gpu, c_gpu, s_gpu = _run_gpu(P, G, W, Xc, 1e-2, 1)
    Td = G.bf16_dev(O.bf16_values_to_bits(T_gpu))
    Wd, Xcd = G.bf16_dev(O.bf16_values_to_bits(W)), G.bf16_dev(O.bf16_values_to_bits(Xc))
    cb, sb = P.wush_packed_sizes(N, K, fmt)
    Wq, Ws = G.empty_u8(cb), G.empty_u8(sb)
    wsp = torch.empty(P.wush_prepare_weight_gptq_workspace(N, K), dtype=torch.uint8, device="cuda")
    Td2 = torch.empty_like(Td)
    P.wush_prepare_weight_gptq(Wd, Xcd, 1e-2, Td2, Wq, Ws, wsp, fmt)
    assert torch.equal(Td2, Td)                                    # reproducible
    xcb, xsb = P.wush_packed_sizes(M, K, fmt)
    Xq, Xs = G.empty_u8(xcb), G.empty_u8(xsb)
    Xd = G.bf16_dev(O.bf16_values_to_bits(X))
    P.wush_quantize_act(Xd, Td, Xq, Xs, fmt)
    Y = torch.empty((M, N), dtype=torch.float32, device="cuda")
    P.wush_linear(Xq, Xs, Wq, Ws, Y, P.default_fmt(out_dtype=1, layout=1), K=K)
    torch.cuda.synchronize()
    y = G.host(Y).astype(np.float64)
    xc, xs = O.quantize_mxfp4(O.transform_act(X, T_gpu))
    ref = O.dequantize(xc, xs) @ O.dequantize(c_gpu, s_gpu).T
    assert O.rel_fro(y, ref) <= 2e-3
    exact = X @ W.T
    l_gw = O.layer_loss(y, exact)
    l_rh = O.layer_loss(O.layer_forward(X, W, O.round_to_bf16(O.hadamard_transforms(K // 32))), exact)
    print(f"W4A4 layer loss: RTN-H {l_rh:.4e}  GPTQ-WUSH (GPU) {l_gw:.4e}")
    assert l_gw < l_rh


def test_gptq_c2_full_size(P, G):
    """The c2 layer in full (K=4096, N=6144, 4096 calibration tokens): the oracle redoes the whole schedule."""
    import time
    cfg = I.CONFIGS["c2"]
    L = I.make_layer(cfg)
    W, Xc = O.bf16_bits_to_f64(L["W"]), O.bf16_bits_to_f64(L["X_cal"])
    X = O.bf16_bits_to_f64(L["X"][:256])
    t0 = time.perf_counter()
    T_gpu, c_gpu, s_gpu = _run_gpu(P, G, W, Xc, 1e-2, 1)
    t1 = time.perf_counter()
    T_ref, c_ref, s_ref = Q.gptq_wush_layer(W, Xc, 1e-2)
    t2 = time.perf_counter()
    print(f"c2 GPTQ case: GPU call incl. transfers {t1 - t0:.2f} s, oracle {t2 - t1:.1f} s")
    _compare(T_gpu, c_gpu, s_gpu, T_ref, c_ref, s_ref, W, X, "c2")


# sizes at the edges of the kernels: one row and one block; more rows than one pass of the row workgroups takes (64 of
# 128 rows below K = 1024); K from 1024 on (warm-started SVD, buffers inside the Hessian's) with an odd number of blocks and
# fewer rows than a wavefront's tile; every position inside the groups of blocks whose errors travel together
@pytest.mark.parametrize("N,K,Mc", [(1, 32, 64), (9000, 64, 128), (13, 1056, 300), (40, 32 * 11, 400)])
def test_gptq_edge_sizes(P, G, N, K, Mc):
    W, Xc, X = _layer(64, K, N, Mc)
    T, c, s = _run_gpu(P, G, W, Xc, 1e-2)
    Tr, cr, sr = Q.gptq_wush_layer(W, Xc, 1e-2)
    _compare(T, c, s, Tr, cr, sr, W, X, f"N={N} K={K}")


def test_gptq_scales_beyond_float_range(P, G):
    """Rows whose group maxima lie outside the range the 32-bit decisions cover (scale bytes below 8), a zero row."""
    rng = np.random.default_rng(11)
    N, K = 48, 128
    W = np.ldexp(rng.standard_normal((N, K)), np.round(np.linspace(-131, -100, N)).astype(int)[:, None])
    W[7] = 0.0
    W = O.round_to_bf16(W)
    Xc = O.round_to_bf16(rng.standard_normal((400, K)))
    T0 = np.broadcast_to(O.round_to_bf16(O.hadamard()), (K // 32, 32, 32)).copy()
    T, c, s = _run_gpu(P, G, W, Xc, 1e-2, T_given=T0)
    _, cr, sr = Q.gptq_wush_layer(W, Xc, 1e-2, transform="hadamard")
    same = (c == cr) | (((c & 7) == 0) & ((cr & 7) == 0))      # +-0 have one magnitude
    assert np.mean(s != sr) <= 1e-4 and np.mean(~same) <= 1e-4, (np.mean(s != sr), np.mean(~same))


@pytest.mark.parametrize("scale_exp", [0, -40])
def test_gptq_past_float_range(P, G, scale_exp):
    """Transformed weights from 2^128 on beside ordinary rows: groups with one such maximum (transform of unit size), groups
    that lie above altogether (a transform of 2^-40 and rows of 2^100)."""
    rng = np.random.default_rng(12)
    N, K = 40, 96
    W = rng.standard_normal((N, K))
    if scale_exp == 0:
        W[[5, 21]] = [[2.0 ** 126.0], [2.0 ** 127.0]]
        W[[5, 21], ::32] = 1.0
    else:
        W *= np.ldexp(1.0, np.where(np.arange(N) % 3 == 0, 100, 0))[:, None]
    W = O.round_to_bf16(W)
    Xc = O.round_to_bf16(rng.standard_normal((400, K)))
    T0 = np.broadcast_to(O.round_to_bf16(np.ldexp(O.hadamard(), scale_exp)), (K // 32, 32, 32)).copy()
    _, c, s = _run_gpu(P, G, W, Xc, 1e-2, T_given=T0)
    _, cr, sr = Q.gptq_wush_layer(W, Xc, 1e-2, transform=T0)
    # behind the maximum of a row of 2^126 or 2^127 the subroutine propagates that element's rounding error, 2^53 times less:
    # those codes and the later blocks' scales may tie otherwise
    big = [5, 21] if scale_exp == 0 else []
    assert np.array_equal(s[:, 0], sr[:, 0]) and np.array_equal(c[:, 0], cr[:, 0])
    rest = np.setdiff1d(np.arange(N), big)
    assert np.mean((s != sr)[rest]) <= 1e-4 and np.mean((c != cr)[rest]) <= 1e-4, (np.mean(s != sr), np.mean((c != cr)[rest]))


@pytest.mark.parametrize("K", [32, 96])
def test_gptq_equal_channels_are_flagged(P, G, K):
    """lambda = 0 and calibration channels that are all the same: the Hessian is c^2 everywhere, exactly, and not positive
    definite, whatever c."""
    import torch
    W = G.bf16_dev(O.bf16_values_to_bits(O.round_to_bf16(np.random.default_rng(2).standard_normal((32, K)))))
    T = G.bf16_dev(O.bf16_values_to_bits(O.round_to_bf16(np.broadcast_to(O.hadamard(), (K // 32, 32, 32)).copy())))
    q, s = G.empty_u8(32, K // 2), G.empty_u8(32, K // 32)
    ws = torch.empty(P.wush_prepare_weight_gptq_workspace(32, K), dtype=torch.uint8, device="cuda")
    missed = []
    for c in range(1, 64):
        X = torch.full((64, K), float(c), dtype=torch.bfloat16, device="cuda")
        P.wush_prepare_weight_gptq(W, X, 0.0, T, q, s, ws, transform_given=True)
        try:
            P.wush_prepare_weight_gptq_status(ws, 32, K)
            missed.append(c)
        except P.WushError as e:
            assert e.code == 7
    assert missed == []


def _dense_turn(tangent, N=1024, K=1024):
    """A layer whose block 1, at its turn, needs a rotation by `tangent` between every two of the directions it starts from.  The calibration moments
    are exact: I, but 1/2 I between blocks 0 and 1 and (1/4 + 49/64) I in block 1, so block 1's weights lose 32/65 of block 0's errors E.  Those
    are made part of them, W_1 = F + E B with F orthogonal to E, such that the moment of W_1 is diag(d), the one of what W_1
    then is diag(d) + P, with P_ij = |d_i - d_j| tan(2 theta) / 2."""
    rng = np.random.default_rng(int(1e4 * tangent))
    Xc = np.ones((1, 1))
    while Xc.shape[0] < K:
        Xc = np.block([[Xc, Xc], [Xc, -Xc]])
    Xc[:, 32:64] = 0.5 * Xc[:, :32] + 0.875 * Xc[:, 32:64]
    W = O.round_to_bf16(rng.standard_normal((N, K)) * np.where(np.arange(K) < 32, 8.0, 1.0))
    T, codes, scales = Q.gptq_wush_layer(W[:, :64], Xc[:, :64], 0.0)
    E = O.dequantize(codes[:, :32], scales[:, :1]) @ T[0] - W[:, :32]
    d, e, S = 1.31 - 0.01 * np.arange(32), -32.0 / 65.0, E.T @ E / N
    P = np.abs(d[:, None] - d) * tangent / (1.0 - tangent ** 2)
    SB = (P - e * e * S) / (2.0 * e)
    F = rng.standard_normal((N, 32))
    F = np.linalg.qr(F - E @ np.linalg.solve(E.T @ E, E.T @ F))[0] * np.sqrt(N)
    W[:, 32:64] = O.round_to_bf16(F @ np.linalg.cholesky(np.diag(d) - SB @ np.linalg.solve(S, SB)).T + E @ np.linalg.solve(S, SB))
    return W, Xc


@pytest.mark.parametrize("tangent", [0.1, 0.12, 0.1475, 0.18])
def test_gptq_block_that_turns_by_many_angles_at_once(P, G, tangent):
    """31 tangents a row add up: the rotation by all of them at once is far from orthogonal as it is first formed, and its correction takes six
    to eight steps or is refused (0.18).  One that is not orthogonal leaves other singular values, off by 2e-7 (0.1), 1e-3 (0.12) and 1e-2
    (0.1475) with four steps."""
    W, Xc = _dense_turn(tangent)
    T, c, s = _run_gpu(P, G, W, Xc, 0.0)
    Tr, cr, sr = Q.gptq_wush_layer(W, Xc, 0.0)
    _compare(T, c, s, Tr, cr, sr, W, Xc, f"tangent {tangent}")


@pytest.mark.parametrize("spread", [60, 120])
def test_gptq_given_transform_whose_inverse_needs_elimination(P, G, spread):
    """inv(T) comes from the factor of T T^T and Newton steps from X near it.  With rows of T that are 2^0 to 2^-spread of one size, T X - I is 2^spread
    times rounding in some entries, too far for the steps, and T is inverted by elimination.  H = I exactly and lambda = 0, so the
    group scales are those of W inv(T): FP64 throughout, and no AbsMax within 1e-4 of a power of two."""
    import torch
    N, K = 1024, 32
    rng = np.random.default_rng(3)
    W = O.round_to_bf16(rng.standard_normal((N, K)))
    T = O.round_to_bf16(rng.standard_normal((K, K)) + 4.0 * np.eye(K)) * np.exp2(-np.round(np.linspace(0, spread, K)))[:, None]
    amax = np.abs(np.linalg.solve(T.T, W.T)).max(axis=0)
    assert np.abs(T @ np.linalg.inv(T) - np.eye(K)).max() > 1.0            # whichever way it is computed
    assert np.abs(amax / np.exp2(np.round(np.log2(amax))) - 1.0).min() > 1e-4
    Xc = O.hadamard(K) * np.sqrt(K)
    Wd, Xd, Td = (G.bf16_dev(O.bf16_values_to_bits(np.ascontiguousarray(O.round_to_bf16(a)))) for a in (W, Xc, T[None]))
    q, s = G.empty_u8(N, K // 2), G.empty_u8(N, K // 32)
    ws = torch.full((P.wush_prepare_weight_gptq_workspace(N, K),), 255, dtype=torch.uint8, device="cuda")     # NaN, should nothing be written
    P.wush_prepare_weight_gptq(Wd, Xd, 0.0, Td, q, s, ws, P.default_fmt(), transform_given=True)
    P.wush_prepare_weight_gptq_status(ws, N, K)
    assert np.array_equal(G.host(s)[:, 0], O.scale_bytes(amax, "nosat"))
