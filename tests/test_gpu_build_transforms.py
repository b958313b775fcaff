"""GPU parity of the on-device transform construction (Alg. 1 + the moment step
of Alg. 2, RTN case) against the oracle's FP64 construction.

The unrounded FP64 T must agree to ~1e-9 of the block's largest entry (both
sides are FP64; only summation order and the SVD algorithm differ).  The BF16
result must equal the oracle's rounded T except for entries whose FP64 value sits
within that distance of a BF16 rounding boundary.
"""
import numpy as np
import pytest

import wush_inputs as I
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


CASES = {
    "c1": (I.CONFIGS["c1"], 1e-2),
    "c1_lam0": (I.CONFIGS["c1"], 0.0),
    "ragged_rows": (I.scaled(I.CONFIGS["c1"], K=32 * 5, N=77, calib_tokens=333, n_outlier=2), 1e-4),
    "c2_cut": (I.scaled(I.CONFIGS["c2"], K=1024, N=1536, calib_tokens=4096, n_outlier=5), 1e-2),
    "c3_cut": (I.scaled(I.CONFIGS["c3"], K=32 * 20, N=512, calib_tokens=3000, n_outlier=6), 1e-2),
}


def _gpu_transforms(P, G, L, lam):
    import torch
    cfg = L["cfg"]
    C = cfg.C
    T = torch.empty((C, 32, 32), dtype=torch.bfloat16, device="cuda")
    T64 = torch.full((C, 32, 32), float("nan"), dtype=torch.float64, device="cuda")
    ws = G.empty_u8(P.wush_build_transforms_workspace(cfg.K))
    P.wush_build_transforms(G.bf16_dev(L["W"]), G.bf16_dev(L["X_cal"]), lam, T, ws, T_f64=T64)
    P.wush_build_transforms_status(ws, cfg.K)
    return G.host(T), T64.cpu().numpy()


@pytest.mark.parametrize("name", list(CASES))
def test_build_transforms_matches_oracle(P, G, name):
    cfg, lam = CASES[name]
    L = I.make_layer(cfg)
    W, Xc = O.bf16_bits_to_f64(L["W"]), O.bf16_bits_to_f64(L["X_cal"])
    T_ref = O.build_transforms(W, Xc, lam)
    t_bits, t64 = _gpu_transforms(P, G, L, lam)
    assert np.isfinite(t64).all()
    scale = np.max(np.abs(T_ref), axis=(1, 2), keepdims=True)
    err = np.max(np.abs(t64 - T_ref) / scale)
    assert err <= 1e-9, err
    # BF16 output: identical to the oracle's rounding except at rounding boundaries
    ref_bits = O.bf16_values_to_bits(O.round_to_bf16(T_ref))
    diff = t_bits != ref_bits
    assert diff.mean() <= 1e-4
    if diff.any():
        ulp = np.abs(O.bf16_bits_to_f64(t_bits)[diff] - O.bf16_bits_to_f64(ref_bits)[diff])
        gap = np.abs(np.abs(t64[diff] - T_ref[diff]))
        assert np.all(ulp <= np.abs(T_ref[diff]) * 2.0 ** -7) and np.all(gap <= 1e-9 * scale.repeat(32, 1).repeat(32, 2)[diff])
    # the device-built transforms satisfy the paper's identities on their own
    b = cfg.C // 2
    sl = slice(32 * b, 32 * b + 32)
    Wp, Xp, U, s, V = O.wush_factors(O.second_moment(W[:, sl]), O.second_moment(Xc[:, sl]), lam)
    eq = t64[b] @ O.damped(O.second_moment(Xc[:, sl]), lam) @ t64[b].T
    assert np.allclose(np.diag(eq), s.sum() / 32, rtol=1e-8)
    assert O.fp_model_objective(t64[b], Wp, Xp) == pytest.approx(s.sum() ** 2 / 32, rel=1e-8)


def test_device_built_transforms_drive_the_layer(P, G):
    """Whole offline + online path on the device: build T, prepare W, quantize X, GEMM."""
    import torch
    cfg = CASES["c2_cut"][0]
    cfg = I.scaled(cfg, M=300)
    L = I.make_layer(cfg)
    M, K, N = cfg.M, cfg.K, cfg.N
    t_bits, _ = _gpu_transforms(P, G, L, 1e-2)
    T = O.bf16_bits_to_f64(t_bits)
    Td = G.bf16_dev(t_bits)
    Xq, Xs = G.empty_u8(M, K // 2), G.empty_u8(M, K // 32)
    Wq, Ws = G.empty_u8(N, K // 2), G.empty_u8(N, K // 32)
    ws = G.empty_u8(P.wush_prepare_weight_workspace(N, K))
    Y = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    P.wush_prepare_weight(G.bf16_dev(L["W"]), Td, Wq, Ws, ws)
    P.wush_workspace_status(ws, K)
    P.wush_quantize_act(G.bf16_dev(L["X"]), Td, Xq, Xs)
    P.wush_linear(Xq, Xs, Wq, Ws, Y)
    torch.cuda.synchronize()
    X, W = O.bf16_bits_to_f64(L["X"]), O.bf16_bits_to_f64(L["W"])
    y = O.bf16_bits_to_f64(G.host(Y))
    assert O.rel_fro(y, O.layer_forward(X, W, T)) <= 2e-3
    # and it beats the plain Hadamard transform on the same data, as the oracle does
    Th = O.round_to_bf16(O.hadamard_transforms(cfg.C))
    exact = X @ W.T
    assert O.layer_loss(y, exact) < O.layer_loss(O.layer_forward(X, W, Th), exact)


def test_build_transforms_flags_indefinite_moment(P, G):
    """lambda = 0 with fewer calibration tokens than channels: M_X is singular."""
    import torch
    cfg = I.scaled(I.CONFIGS["c1"], K=64, N=64, calib_tokens=8, n_outlier=1)
    L = I.make_layer(cfg)
    T = torch.empty((2, 32, 32), dtype=torch.bfloat16, device="cuda")
    ws = G.empty_u8(P.wush_build_transforms_workspace(64))
    P.wush_build_transforms(G.bf16_dev(L["W"]), G.bf16_dev(L["X_cal"]), 0.0, T, ws)
    with pytest.raises(P.WushError) as ei:
        P.wush_build_transforms_status(ws, 64)
    assert ei.value.code == 7


@pytest.mark.parametrize("name", ["c1", "c1_lam0", "ragged_rows", "c2_cut"])
def test_build_transforms_16_matches_oracle(P, G, name):
    """The same construction with 16 x 16 blocks (the NVFP4 variant)."""
    import torch
    cfg, lam = CASES[name]
    L = I.make_layer(cfg)
    W, Xc = O.bf16_bits_to_f64(L["W"]), O.bf16_bits_to_f64(L["X_cal"])
    C16 = cfg.K // 16
    T_ref = np.empty((C16, 16, 16))
    for b in range(C16):
        sl = slice(16 * b, 16 * b + 16)
        T_ref[b] = O.wush_block(O.second_moment(W[:, sl]), O.second_moment(Xc[:, sl]), lam)
    T = torch.empty((C16, 16, 16), dtype=torch.bfloat16, device="cuda")
    T64 = torch.full((C16, 16, 16), float("nan"), dtype=torch.float64, device="cuda")
    ws = G.empty_u8(P.wush_build_transforms_workspace(cfg.K))
    P.wush_build_transforms_nvfp4(G.bf16_dev(L["W"]), G.bf16_dev(L["X_cal"]), lam, T, ws, T_f64=T64)
    P.wush_build_transforms_status(ws, cfg.K)
    t_bits, t64 = G.host(T), T64.cpu().numpy()
    assert np.isfinite(t64).all()
    scale = np.max(np.abs(T_ref), axis=(1, 2), keepdims=True)
    assert np.max(np.abs(t64 - T_ref) / scale) <= 1e-9
    ref_bits = O.bf16_values_to_bits(O.round_to_bf16(T_ref))
    diff = t_bits != ref_bits
    assert diff.mean() <= 1e-4
    if diff.any():
        assert np.all(np.abs(t64[diff] - T_ref[diff]) <= 1e-9 * scale.repeat(16, 1).repeat(16, 2)[diff])
    # the identities of the construction hold for a 16-block as well
    b = C16 // 2
    sl = slice(16 * b, 16 * b + 16)
    Wp, Xp, U, s, V = O.wush_factors(O.second_moment(W[:, sl]), O.second_moment(Xc[:, sl]), lam)
    eq = t64[b] @ O.damped(O.second_moment(Xc[:, sl]), lam) @ t64[b].T
    assert np.allclose(np.diag(eq), s.sum() / 16, rtol=1e-8)
    assert O.fp_model_objective(t64[b], Wp, Xp) == pytest.approx(s.sum() ** 2 / 16, rel=1e-8)


@pytest.mark.parametrize("rows", [(33, 128), (129, 127), (128, 1025), (257, 33), (512, 500), (512, 513)])
def test_row_splits_without_rows_are_not_read(P, G, rows):
    """Row counts around the splits of 128 rows, a workspace full of NaN: partial moments of splits that hold no rows stay
    unwritten and must not be read (the bar of the parity test above); four splits and five, on either side of the kernel for few."""
    import torch
    cfg = I.scaled(I.CONFIGS["c1"], K=96, N=rows[0], calib_tokens=rows[1], n_outlier=2)
    L = I.make_layer(cfg)
    T = torch.empty((3, 32, 32), dtype=torch.bfloat16, device="cuda")
    T64 = torch.empty((3, 32, 32), dtype=torch.float64, device="cuda")
    ws = torch.full((P.wush_build_transforms_workspace(96),), 255, dtype=torch.uint8, device="cuda")
    P.wush_build_transforms(G.bf16_dev(L["W"]), G.bf16_dev(L["X_cal"]), 1e-2, T, ws, T_f64=T64)
    P.wush_build_transforms_status(ws, 96)
    T_ref = O.build_transforms(O.bf16_bits_to_f64(L["W"]), O.bf16_bits_to_f64(L["X_cal"]), 1e-2)
    assert np.max(np.abs(T64.cpu().numpy() - T_ref) / np.max(np.abs(T_ref), axis=(1, 2), keepdims=True)) <= 1e-9


@pytest.mark.parametrize("block", [32, 16])
@pytest.mark.parametrize("clusters", [1, 2])
@pytest.mark.parametrize("noise_exp", [None, -28, -22, -16])
def test_repeated_singular_values(P, G, block, clusters, noise_exp):
    """Blocks whose singular values repeat (one group, or two a factor of 2 apart) or nearly do, M_W = I exactly: the columns of
    U stay orthogonal to FP64 accuracy however the rotations inside a group fall.  With W' = I, H T = S^(-1/2) U^T; the two
    products with H sum `block` rounded terms each, 2 block^2 2^-53 in the Gram matrix at most."""
    import torch
    rng = np.random.default_rng(17)
    Hs = O.hadamard(block) * np.sqrt(block)
    X = Hs * (1.0 + (np.arange(block) >= block // 2) * (clusters - 1))
    if noise_exp is not None:
        X = np.concatenate([X, np.ldexp(rng.standard_normal((32, block)), noise_exp)])
    reps = 32 // block
    W, X = np.tile(Hs, (1, reps)), np.tile(X, (1, reps))
    T = torch.empty((reps, block, block), dtype=torch.bfloat16, device="cuda")
    T64 = torch.full((reps, block, block), float("nan"), dtype=torch.float64, device="cuda")
    ws = G.empty_u8(P.wush_build_transforms_workspace(32))
    build = P.wush_build_transforms if block == 32 else P.wush_build_transforms_nvfp4
    bits = [G.bf16_dev(O.bf16_values_to_bits(O.round_to_bf16(a))) for a in (W, X)]
    build(*bits, 0.0, T, ws, T_f64=T64)
    P.wush_build_transforms_status(ws, 32)
    for t in T64.cpu().numpy():
        ut = O.hadamard(block) @ t
        ut /= np.linalg.norm(ut, axis=1, keepdims=True)
        err = np.max(np.abs(ut @ ut.T - np.eye(block)))
        assert err <= 2 * block * block * 2.0 ** -53, err


@pytest.mark.parametrize("block", [32, 16])
def test_equal_channels_are_flagged(P, G, block):
    """lambda = 0 and channels that are all the same: the moment is c^2 everywhere, exactly, and every step of the factorization
    behind the first meets a pivot of exactly zero, whatever c."""
    import torch
    build = P.wush_build_transforms if block == 32 else P.wush_build_transforms_nvfp4
    W = G.bf16_dev(O.bf16_values_to_bits(O.round_to_bf16(np.random.default_rng(2).standard_normal((64, 32)))))
    T = torch.empty((32 // block, block, block), dtype=torch.bfloat16, device="cuda")
    ws = G.empty_u8(P.wush_build_transforms_workspace(32))
    missed = []
    for c in range(1, 128):
        X = torch.full((64, 32), float(c), dtype=torch.bfloat16, device="cuda")
        for args in ((W, X), (X, W)):
            build(*args, 0.0, T, ws)
            try:
                P.wush_build_transforms_status(ws, 32)
                missed.append(c)
            except P.WushError as e:
                assert e.code == 7
    assert missed == []


@pytest.mark.parametrize("block", [32, 16])
@pytest.mark.parametrize("spread", [0.0, 1.0, 2.5])
@pytest.mark.parametrize("rows", [40, 2000])
def test_transforms_diagonalize_graded_moments(P, G, block, spread, rows):
    """Channels whose scales spread over exp(spread N(0, 1)), lambda = 0: H^T T M_X T^T H = S is diagonal.  Its off-diagonal entries relative to
    the diagonal ones: what the right rotations lack of orthogonality, some 50 rounds and steps of 32 rounded terms each, 50 x 32 x 2^-53 = 2e-13,
    and T's own rounding.  An entry of T is a sum over the rows S^(-1/2) U^T W'^T of either sign, rounded relative to the largest; a row
    comes back with 2^-53 of that, the square root of the singular values' ratio, and meets the largest direction of M_X, the same again:
    2^-53 x ratio for each of the 2 x 32 terms of a pair of rows.  The check itself is in long double."""
    import torch
    rng = np.random.default_rng(rows + int(10 * spread))
    K = 64
    W, X = (O.round_to_bf16(rng.standard_normal((rows, K)) * s) for s in (1.0, np.exp(spread * rng.standard_normal(K))))
    T = torch.empty((K // block, block, block), dtype=torch.bfloat16, device="cuda")
    T64 = torch.full((K // block, block, block), float("nan"), dtype=torch.float64, device="cuda")
    ws = G.empty_u8(P.wush_build_transforms_workspace(K))
    build = P.wush_build_transforms if block == 32 else P.wush_build_transforms_nvfp4
    build(*(G.bf16_dev(O.bf16_values_to_bits(a)) for a in (W, X)), 0.0, T, ws, T_f64=T64)
    P.wush_build_transforms_status(ws, K)
    H = O.hadamard(block).astype(np.longdouble)
    for i, t in enumerate(T64.cpu().numpy().astype(np.longdouble)):
        x = X[:, block * i:block * (i + 1)].astype(np.longdouble)
        S = H.T @ t @ (x.T @ x / rows) @ t.T @ H
        d = np.sqrt(np.diag(S))
        off, ratio = np.max(np.abs(S / np.outer(d, d) - np.eye(block))), (d.max() / d.min()) ** 2
        assert off <= 2e-13 + 64 * 2.0 ** -53 * ratio, (off, ratio)
