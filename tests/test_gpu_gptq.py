"""GPU parity of the MR-GPTQ sweep (fp4_gptq_quantize_weights) against the NumPy oracle (oracle/gptq.py).

The sweep rounds a running value that carries the accumulated updates of every earlier column; the kernel keeps it in
fp32, the oracle in fp64.  Where all the arithmetic is exact in both (dyadic weights and factor entries, errors pushed
one step only) the codes must be bit-exact.  On realistic inputs a rounding may flip where the running value sits
within fp32 noise of a grid midpoint, and a flip changes what later columns of that row see -- so the bar there is: the
scale bytes are the round-to-nearest ones bit for bit, nearly all codes equal the oracle's, and the quantity GPTQ
minimises, the layer's output error tr(dW H dW^T), is the oracle's within 1e-3 relative.
"""
import sys

import numpy as np
import pytest

from paper_2509_23202_amd import inputs
from tests.gpu_util import MX, NV, to_dev, to_dev_bf16, unpack

pytestmark = pytest.mark.gpu


def say(msg):
    print("[case] " + msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def fp4():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2509_23202_amd import binding
    return binding


@pytest.fixture(scope="module")
def gptq():
    from oracle import gptq
    return gptq


def np_(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("N,K", [(5, 64), (70, 256), (150, 1088)])
def test_sweep_is_bit_exact_where_the_arithmetic_is_exact(fp4, oracle, gptq, N, K):
    """Weights on a 2^-6 lattice, no rotation, unit diagonal, and every even column (in visiting order) pushing its error
    onto a few later odd columns with factors +-2^-3, +-2^-4 (odd columns push nothing): every product and sum is exact
    in fp32, so the codes must equal the oracle's everywhere -- across the 64-column block boundaries and (K = 1088)
    the 512-column outer blocks of the update kernel, through a random visiting order, with ragged row groups."""
    import torch
    rng = np.random.default_rng(K)
    w = (rng.integers(-200, 201, (N, K)) / 64.0).astype(np.float32)
    wb = inputs.f32_to_bf16_bits(w)
    assert np.array_equal(inputs.bf16_bits_to_f32(wb), w)      # the lattice values are bf16 numbers
    perm = rng.permutation(K).astype(np.int32)
    U = np.eye(K, dtype=np.float32)
    for j in range(0, K, 2):
        for d, mag in ((1, 0.125), (3, 0.0625), (65, 0.125), (131, 0.0625), (513, 0.125), (701, 0.0625)):
            if j + d < K:
                U[j, j + d] = mag * rng.choice([-1.0, 1.0])
    y = oracle.rotate(wb, 1)
    _, scales, _ = oracle.quantize(y, MX)
    want, _ = gptq.sweep(y, scales, MX, None, U, perm)
    rtn, _, _ = oracle.quantize(y, MX)
    say(f"gptq exact lattice case N={N} K={K}")
    c, s, _ = fp4.fp4_gptq_quantize_weights(to_dev_bf16(wb), 1, MX, to_dev(U), to_dev(perm))
    torch.cuda.synchronize()
    assert np.array_equal(np_(s).reshape(N, -1), scales)
    assert np.array_equal(np_(c).reshape(N, -1), want)
    assert (want != rtn).mean() > 0.02          # the pushed errors did change codes


@pytest.mark.parametrize("fmt", [MX, NV])
def test_diagonal_factor_gives_round_to_nearest(fp4, oracle, fmt):
    import torch
    N, K, b = 33, 512, 32
    wb = inputs.RECIPES[6].w(N, K, salt=9)
    U = np.diag(np.random.default_rng(1).uniform(0.5, 2.0, K)).astype(np.float32)
    say(f"gptq diagonal fmt={fmt}")
    c, s, T = fp4.fp4_gptq_quantize_weights(to_dev_bf16(wb), b, fmt, to_dev(U), None)
    c0, s0, T0 = fp4.fp4_quantize_weights(to_dev_bf16(wb), b, fmt)
    torch.cuda.synchronize()
    assert np.array_equal(np_(s), np_(s0))
    if fmt == NV:
        assert np_(T)[0] == np_(T0)[0]
    diff = unpack(np_(c).reshape(N, -1)) != unpack(np_(c0).reshape(N, -1))
    # MXFP4: w / s is exact both ways.  NVFP4: the quantizer multiplies by a rounded reciprocal, the sweep divides
    assert diff.mean() <= (0.0 if fmt == MX else 1e-4)


@pytest.mark.parametrize("fmt,policy,b", [(MX, "absmax", 32), (MX, "mse", 128), (MX, "round43", 32), (NV, "absmax", 16), (NV, "mse", 32),
                                          (NV, "mse_alt", 16), (NV, "mse_alt", 1)])
def test_sweep_matches_the_oracle_on_synthetic_hessians(fp4, oracle, gptq, fmt, policy, b):
    import torch
    N, K, T = 100, 512, 1024
    r = inputs.RECIPES[6]
    wb, xb = r.w(N, K, salt=40), r.x(T, K, salt=41)
    X = oracle.rotate(xb, b).astype(np.float64)
    H = X.T @ X
    perm = gptq.act_order(H).astype(np.int32)
    U = gptq.inverse_factor(H, perm, damp=1e-2).astype(np.float32)
    y = oracle.rotate(wb, b)
    if policy == "mse_alt":   # the grid of Ingredient 1 in full: group scales and tensor scale by alternating optimisation
        c_rtn, scales, sT, _ = oracle.quantize_nvfp4_alternating(y, 3)
    else:
        c_rtn, scales, sT = oracle.quantize(y, fmt, policy=policy)
    want, _ = gptq.sweep(y, scales, fmt, sT, U, perm)
    flags = {"absmax": 0, "mse": fp4.SCALE_MSE, "round43": fp4.SCALE_ROUND43, "mse_alt": fp4.SCALE_MSE | fp4.SCALE_FIT_TENSOR}[policy]
    say(f"gptq synthetic fmt={fmt} policy={policy} b={b}")
    c, s, Tg = fp4.fp4_gptq_quantize_weights(to_dev_bf16(wb), b, fmt, to_dev(U), to_dev(perm), flags=flags)
    torch.cuda.synchronize()
    got_c, got_s = np_(c).reshape(N, -1), np_(s).reshape(N, -1)
    assert (got_s != scales).mean() <= 1e-3
    if fmt == NV:
        assert abs(float(np_(Tg)[0]) - float(sT)) <= 2 * np.spacing(np.float32(sT))
    rows_ok = (got_s == scales).all(axis=1)
    diff = unpack(got_c) != unpack(want)
    e_got = gptq.layer_error(y[rows_ok], got_c[rows_ok], scales[rows_ok], fmt, sT, H)
    e_ref = gptq.layer_error(y[rows_ok], want[rows_ok], scales[rows_ok], fmt, sT, H)
    e_rtn = gptq.layer_error(y[rows_ok], c_rtn[rows_ok], scales[rows_ok], fmt, sT, H)
    say(f"   codes differing from the oracle: {diff[rows_ok].mean():.2e}; layer error {e_got:.6e} vs oracle {e_ref:.6e} (round-to-nearest {e_rtn:.4e})")
    assert diff[rows_ok].mean() <= 1e-3
    assert abs(e_got - e_ref) <= 1e-3 * e_ref
    assert e_got < 0.8 * e_rtn


def test_gptq_on_the_fitted_scale_range(fp4, oracle, gptq):
    """MR-GPTQ with the scale byte fitted to the tensor's range as the fixed grid (appendix on MXFP scale fitting, table:
    MR-GPTQ on MXFP4-dagger): the grid is the library's own (bytes and the 256 scale values it publishes; its parity
    with the oracle's fit is tested with the quantizer), the sweep is compared with the oracle's sweep on that grid."""
    import torch
    b, N, K, T = 32, 100, 512, 1024
    r = inputs.RECIPES[6]
    wb, xb = r.w(N, K, salt=60), r.x(T, K, salt=61)
    X = oracle.rotate(xb, b).astype(np.float64)
    H = X.T @ X
    perm = gptq.act_order(H).astype(np.int32)
    U = gptq.inverse_factor(H, perm, damp=1e-2).astype(np.float32)
    y = oracle.rotate(wb, b)
    say("gptq on the fitted scale range")
    c, s, ts = fp4.fp4_gptq_quantize_weights(to_dev_bf16(wb), b, MX, to_dev(U), to_dev(perm), flags=fp4.SCALE_FIT_RANGE)
    c0, s0, ts0 = fp4.fp4_quantize_weights(to_dev_bf16(wb), b, MX, flags=fp4.SCALE_FIT_RANGE)
    torch.cuda.synchronize()
    assert torch.equal(s, s0) and torch.equal(ts, ts0)          # the grid is the round-to-nearest call's, bit for bit
    got_c, q, table = np_(c).reshape(N, -1), np_(s).reshape(N, -1), np_(ts)[2:258].astype(np.float64)
    want, _ = gptq.sweep(y, q, MX, None, U, perm, table=table)
    diff = unpack(got_c) != unpack(want)
    e_got = gptq.layer_error(y, got_c, q, MX, None, H, table=table)
    e_ref = gptq.layer_error(y, want, q, MX, None, H, table=table)
    e_rtn = gptq.layer_error(y, np_(c0).reshape(N, -1), q, MX, None, H, table=table)
    say(f"   codes differing from the oracle: {diff.mean():.2e}; layer error {e_got:.6e} vs oracle {e_ref:.6e} (round-to-nearest {e_rtn:.4e})")
    assert diff.mean() <= 1e-3
    assert abs(e_got - e_ref) <= 1e-3 * e_ref
    assert e_got < 0.8 * e_rtn


def test_gptq_argument_validation(fp4):
    import torch
    w = torch.zeros((16, 128), dtype=torch.bfloat16, device="cuda")
    U = torch.eye(128, dtype=torch.float32, device="cuda")
    with pytest.raises(Exception):
        fp4.fp4_gptq_quantize_weights(w, 32, MX, U, None, flags=fp4.LAYOUT_GEMM)
    w96 = torch.zeros((16, 96), dtype=torch.bfloat16, device="cuda")
    U96 = torch.eye(96, dtype=torch.float32, device="cuda")
    with pytest.raises(Exception):
        fp4.fp4_gptq_quantize_weights(w96, 32, MX, U96, None)
    with pytest.raises(Exception):
        fp4.fp4_gptq_quantize_weights(w, 32, MX, U, None, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))


def synthetic_hessian(oracle, K, T, b, salt):
    xb = inputs.RECIPES[6].x(T, K, salt=salt)
    X = oracle.rotate(xb, b).astype(np.float64)
    return X.T @ X


@pytest.mark.parametrize("K", [64, 200, 320, 512, 1088])
def test_prepare_matches_the_oracle_order_and_factor(fp4, oracle, gptq, K):
    """Order: the same permutation as a stable descending sort of the diagonal.  Factor: fp32 blocked Cholesky and
    triangular inversion against NumPy in fp64 -- compared as matrices and through the identity U^T U A = I that
    defines it.  K = 200 and 320 have a ragged last block / an odd number of blocks (the doubling levels' tails)."""
    import torch
    b = 8 if K == 200 else 32
    H = synthetic_hessian(oracle, K, 2 * K + 100, b, salt=50 + K)
    H32 = H.astype(np.float32)
    say(f"gptq prepare K={K}")
    perm, U = fp4.fp4_gptq_prepare(to_dev(H32), 1e-2, True)
    torch.cuda.synchronize()
    perm, U = np_(perm), np_(U).astype(np.float64)
    want_perm = gptq.act_order(H32.astype(np.float64))
    assert np.array_equal(perm, want_perm)
    want_U = gptq.inverse_factor(H32.astype(np.float64), want_perm, damp=1e-2)
    assert np.all(np.tril(U, -1) == 0)
    rel = np.linalg.norm(U - want_U) / np.linalg.norm(want_U)
    A = H32.astype(np.float64)[np.ix_(want_perm, want_perm)]
    A[np.diag_indices(K)] += 1e-2 * np.mean(np.diag(A))
    resid = np.abs(U.T @ U @ A - np.eye(K)).max()
    say(f"   relative error of U {rel:.2e}; max |U^T U A - I| {resid:.2e}")
    assert rel <= 5e-4 and resid <= 2e-3
    # no re-ordering on request
    perm0, U0 = fp4.fp4_gptq_prepare(to_dev(H32), 1e-2, False)
    torch.cuda.synchronize()
    assert np.array_equal(np_(perm0), np.arange(K))
    want_U0 = gptq.inverse_factor(H32.astype(np.float64), np.arange(K), damp=1e-2)
    assert np.linalg.norm(np_(U0) - want_U0) / np.linalg.norm(want_U0) <= 5e-4


@pytest.mark.parametrize("K", [1, 2, 16, 127, 128, 129, 255, 257, 400])
def test_prepare_at_the_edges_of_its_blocks(fp4, gptq, K):
    """Sizes around the 128-column blocks of the elimination and the 16-column steps inside them.  Bounds as above."""
    import torch
    rng = np.random.default_rng(500 + K)
    X = rng.standard_normal((2 * K + 10, K)) * rng.uniform(0.2, 3.0, K)
    H32 = (X.T @ X).astype(np.float32)
    H32 = np.tril(H32) + np.tril(H32, -1).T
    say(f"gptq prepare edges K={K}")
    perm, U = fp4.fp4_gptq_prepare(to_dev(H32), 1e-2, True)
    torch.cuda.synchronize()
    perm, U = np_(perm), np_(U).astype(np.float64)
    H64 = H32.astype(np.float64)
    want_perm = gptq.act_order(H64)
    assert np.array_equal(perm, want_perm)
    want_U = gptq.inverse_factor(H64, want_perm, damp=1e-2)
    assert np.all(np.tril(U, -1) == 0)
    assert np.linalg.norm(U - want_U) / np.linalg.norm(want_U) <= 5e-4
    A = H64[np.ix_(want_perm, want_perm)] + 1e-2 * np.mean(np.diag(H64)) * np.eye(K)
    assert np.abs(U.T @ U @ A - np.eye(K)).max() <= 2e-3


@pytest.mark.parametrize("K", [1, 128, 129, 256, 272, 384, 400])
def test_prepare_stays_inside_its_workspace(fp4, K):
    """The size in the header, around whole blocks of 128: the same factor, and nothing behind it is written."""
    import torch
    say(f"gptq prepare workspace K={K}")
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    x = torch.randn(2 * K + 8, K, device="cuda", generator=g)
    H = x.t().contiguous() @ x
    H = ((H + H.t()) * 0.5).contiguous()
    need = fp4.workspace_bytes(fp4.OP_GPTQ_PREPARE, 0, 0, K, MX)
    room = torch.full((need + 65536,), 0xa5, dtype=torch.uint8, device="cuda")
    perm, U = fp4.fp4_gptq_prepare(H, 1e-2, True)
    perm2, U2 = fp4.fp4_gptq_prepare(H, 1e-2, True, workspace=room[:need])
    torch.cuda.synchronize()
    assert torch.equal(perm, perm2) and torch.equal(U, U2)
    assert bool((room[need:] == 0xa5).all())


@pytest.mark.parametrize("log2_scale", [-124, -60, 110])
def test_prepare_of_very_small_and_large_hessians(fp4, gptq, log2_scale):
    """The factor scales with the Hessian, also where pivots are subnormal in binary32 (mean of the diagonal 2^-124; they still
    hold 17 bits).  Bound as above."""
    import torch
    K = 300
    rng = np.random.default_rng(900)
    X = rng.standard_normal((2 * K, K)) * rng.uniform(0.1, 2.0, K)
    H = X.T @ X
    H32 = (H / np.mean(np.diag(H)) * 2.0 ** log2_scale).astype(np.float32)
    H32 = np.tril(H32) + np.tril(H32, -1).T
    say(f"gptq prepare at 2^{log2_scale}")
    perm, U = fp4.fp4_gptq_prepare(to_dev(H32), 1e-2, True)
    torch.cuda.synchronize()
    perm, U = np_(perm), np_(U).astype(np.float64)
    H64 = H32.astype(np.float64)
    want_perm = gptq.act_order(H64)
    assert np.array_equal(perm, want_perm)
    want_U = gptq.inverse_factor(H64, want_perm, damp=1e-2)
    assert np.linalg.norm(U - want_U) / np.linalg.norm(want_U) <= 5e-4


def test_prepare_orders_equal_diagonal_entries_by_index(fp4, gptq):
    import torch
    K = 128
    d = np.repeat(np.array([3.0, 1.0, 2.0, 3.0], dtype=np.float32), K // 4)
    H = np.diag(d).astype(np.float32)
    perm, U = fp4.fp4_gptq_prepare(to_dev(H), 1e-2, True)
    torch.cuda.synchronize()
    assert np.array_equal(np_(perm), gptq.act_order(H.astype(np.float64)))
    lam = 1e-2 * d.mean()
    assert np.allclose(np.diag(np_(U)), 1.0 / np.sqrt(d[np_(perm)] + lam), rtol=1e-6)


@pytest.mark.parametrize("fmt,policy", [(MX, "mse"), (NV, "absmax")])
def test_hessian_to_codes_entirely_on_the_gpu(fp4, oracle, gptq, fmt, policy):
    """H -> fp4_gptq_prepare -> fp4_gptq_quantize_weights against the oracle's whole quantizer (fp64 factor): same
    order, layer error within 1% of the oracle's and far below round-to-nearest."""
    import torch
    N, K, b = 96, 768, 32
    wb = inputs.RECIPES[6].w(N, K, salt=70)
    H = synthetic_hessian(oracle, K, 2048, b, salt=71).astype(np.float32)
    say(f"gptq whole path fmt={fmt} policy={policy}")
    perm, U = fp4.fp4_gptq_prepare(to_dev(H), 1e-2, True)
    flags = {"absmax": 0, "mse": fp4.SCALE_MSE}[policy]
    c, s, T = fp4.fp4_gptq_quantize_weights(to_dev_bf16(wb), b, fmt, U, perm, flags=flags)
    torch.cuda.synchronize()
    H64 = H.astype(np.float64)
    want_c, want_s, sT, want_perm, _ = gptq.mr_gptq(wb, H64, b, fmt, policy=policy)
    assert np.array_equal(np_(perm), want_perm)
    got_c, got_s = np_(c).reshape(N, -1), np_(s).reshape(N, -1)
    ok = (got_s == want_s).all(axis=1)
    assert ok.mean() >= 0.98
    y = oracle.rotate(wb, b)
    c_rtn, _, _ = oracle.quantize(y, fmt, policy=policy)
    e_got = gptq.layer_error(y[ok], got_c[ok], want_s[ok], fmt, sT, H64)
    e_ref = gptq.layer_error(y[ok], want_c[ok], want_s[ok], fmt, sT, H64)
    e_rtn = gptq.layer_error(y[ok], c_rtn[ok], want_s[ok], fmt, sT, H64)
    diff = (unpack(got_c) != unpack(want_c))[ok].mean()
    say(f"   codes differing from the oracle: {diff:.2e}; layer error {e_got:.5e} vs oracle {e_ref:.5e} (round-to-nearest {e_rtn:.3e})")
    assert abs(e_got - e_ref) <= 1e-2 * e_ref
    assert e_got < 0.8 * e_rtn


@pytest.mark.parametrize("b", [1, 32, 128])
def test_hessian_accumulation_matches_the_fp64_product(fp4, oracle, b):
    """H = (X H_b)^T (X H_b) in fp32 against the oracle's rotation and a NumPy fp64 product; every entry within
    2e-5 of sqrt(H_ii H_jj) (its Cauchy-Schwarz scale; 700 terms of fp32 rounding each), symmetric, and two batches of
    rows accumulate to the same matrix."""
    import torch
    T, K = 700, 384
    xb = inputs.RECIPES[6].x(T, K, salt=90 + b)
    X = oracle.rotate(xb, b).astype(np.float64)
    want = X.T @ X
    say(f"gptq hessian b={b}")
    H = fp4.fp4_gptq_accumulate_hessian(to_dev_bf16(xb), b)
    H2 = fp4.fp4_gptq_accumulate_hessian(to_dev_bf16(xb[:300]), b)
    H2 = fp4.fp4_gptq_accumulate_hessian(to_dev_bf16(xb[300:]), b, H2)
    torch.cuda.synchronize()
    scale = np.sqrt(np.outer(np.diag(want), np.diag(want)))
    for got in (np_(H).astype(np.float64), np_(H2).astype(np.float64)):
        assert np.all(np.abs(got - want) <= 2e-5 * scale)
        assert np.array_equal(got, got.T)


@pytest.mark.parametrize("T,K,b", [(1, 2, 1), (63, 130, 1), (65, 140, 1), (64, 128, 128), (200, 144, 16), (129, 448, 64), (1100, 384, 128), (2300, 640, 32)])
def test_hessian_tiles_and_split_rows(fp4, oracle, T, K, b):
    """Tile edges (K below, at and beyond a tile of 128; K not a multiple of eight, where rows are not 16-byte aligned), row
    counts around a stage of 64, and enough rows for the tiles' sums to be split into parts; fresh and accumulated.
    Bound: fp32 rounding of T terms, 2e-5 of the Cauchy-Schwarz scale at 700 of them as above, growing with their root."""
    import torch
    xb = inputs.RECIPES[6].x(T, K, salt=300 + T)
    X = oracle.rotate(xb, b).astype(np.float64)
    want = X.T @ X
    say(f"gptq hessian T={T} K={K} b={b}")
    H = fp4.fp4_gptq_accumulate_hessian(to_dev_bf16(xb), b)
    H2 = fp4.fp4_gptq_accumulate_hessian(to_dev_bf16(xb), b, H.clone())
    torch.cuda.synchronize()
    scale = np.sqrt(np.outer(np.diag(want), np.diag(want)))
    for got, times in ((np_(H).astype(np.float64), 1), (np_(H2).astype(np.float64), 2)):
        assert np.all(np.abs(got - times * want) <= 2e-5 * times * max(1.0, (T / 700) ** 0.5) * scale)
        assert np.array_equal(got, got.T)


# (pairs of tiles are taken where they fill the chip: 256 compute units)
PAIRS = [(2048, 4096, 16), (2050, 4224, 128), (2081, 4096, 64), (2113, 4080, 16), (4130, 3600, 16), (4200, 3456, 128), (4096, 5120, 32), (2100, 6144, 64)]


@pytest.mark.parametrize("T,K,b,kind", [(*s, "loud channels") for s in PAIRS] + [(*s, kind) for s in (PAIRS[0], PAIRS[1], PAIRS[4]) for kind in ("rows", "quiet channels")])
def test_hessian_in_pairs_of_tiles(fp4, T, K, b, kind):
    """Full and partial rounds of pairs, an odd number of tile rows, a last tile that is not whole, every remainder of stages by a group
    of four, rows behind the last whole stage; fresh and accumulated, against the fp64 product of rows rotated in fp64.  Rows of one size with loud channels; rows whose
    sizes differ by up to 2^40, so that neighbouring groups' scales do; quiet channels beside loud ones in every block, as in the test of those.
    Bound: (42 + T / 128) 2^-24 of sqrt(h_ii h_jj), as of many rows at the edges of stages and groups: 3.5e-6 to 4.4e-6 here.  Without one of the two products of a high half and a
    low one, computed in fp64 for three of the shapes: 2.2e-5 to 3.4e-5, rows of different size 1.0e-4 to 1.6e-4."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(T + K)
    x = torch.randn(T, K, device="cuda", generator=g)
    if kind == "rows":
        x *= 2.0 ** torch.randint(-20, 21, (T, 1), device="cuda", generator=g)
    elif kind == "quiet channels":
        x *= 2.0 ** -18
        x[::64] = (1.0 + torch.rand(len(x[::64]), K // b, device="cuda", generator=g)).repeat_interleave(b, dim=1)
    else:
        x[:, torch.randperm(K, device="cuda", generator=g)[:K // 200]] *= 50.0
    x = x.bfloat16()
    h = torch.ones(1, 1, dtype=torch.float64, device="cuda")
    while h.shape[0] < b:
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)], 0)
    rotated = ((x.double().view(-1, b) @ h) / b ** 0.5).view(T, K)
    want = rotated.t() @ rotated
    say(f"gptq hessian in pairs T={T} K={K} b={b} {kind}")
    H = fp4.fp4_gptq_accumulate_hessian(x, b)
    H2 = fp4.fp4_gptq_accumulate_hessian(x, b, H.clone())
    d = want.diagonal().sqrt()
    for got, times in ((H, 1), (H2, 2)):
        worst = ((got.double() - times * want).abs() / (d[:, None] * d[None, :])).max().item()
        say(f"   largest error over sqrt(h_ii h_jj): {worst:.2e}")
        assert worst <= times * (42 + T / 128) * 2.0 ** -24
        assert torch.equal(got, got.t())


def common_mode_rows(kind, T, K, b, salt):
    """Calibration rows whose channels have something in common inside a rotation block, as bf16 bits: the rotation moves it
    into a few channels and the others keep what little is left."""
    rng = np.random.default_rng(700 + salt)
    if kind == "offset":          # one constant under unit noise
        x = 100.0 + rng.standard_normal((T, K))
    elif kind == "factor":        # one zero-mean value per row and block, 0.2 % of noise per channel
        f = rng.standard_normal((T, K // b))
        x = np.repeat(f, b, axis=1) * (1.0 + 0.002 * rng.standard_normal((T, K)))
    elif kind == "walsh":         # the same, with the signs of a rotated channel
        f = rng.standard_normal((T, K // b))
        signs = np.where(np.array([bin(i & 5).count("1") & 1 for i in range(b)]), -1.0, 1.0)
        x = np.repeat(f, b, axis=1) * np.tile(signs, K // b) * (1.0 + 0.01 * rng.standard_normal((T, K)))
    else:                         # "constant": every row constant within a block but for its last element
        x = np.repeat(rng.uniform(1.0, 2.0, (T, K // b)), b, axis=1)
        x[:, b - 1::b] *= 1.0 + 2.0 ** -7
    return inputs.f32_to_bf16_bits(x.astype(np.float32))


@pytest.mark.parametrize("kind", ["offset", "factor", "walsh", "constant"])
@pytest.mark.parametrize("T,K,b", [(1, 128, 128), (700, 256, 16), (1500, 320, 32), (1500, 320, 64), (4100, 384, 128),
                                   (70, 1808, 16), (97, 3344, 16), (41, 4112, 16)])
def test_hessian_of_rows_with_a_common_component_in_a_block(fp4, oracle, kind, T, K, b):
    """Rotated channels of very different size beside each other: every entry is accurate on the scale of ITS two rotated
    channels, not of the largest one in the block, and no diagonal entry is negative; fresh and accumulated.  The last three
    sizes have tiles of 64 x 64, of 128 x 128, and of 128 x 128 with some of 32 x 32 left over.  Bound as above."""
    import torch
    xb = common_mode_rows(kind, T, K, b, salt=T + b)
    X = oracle.rotate(xb, b).astype(np.float64)
    want = X.T @ X
    say(f"gptq hessian {kind} T={T} K={K} b={b}")
    H = fp4.fp4_gptq_accumulate_hessian(to_dev_bf16(xb), b)
    H2 = fp4.fp4_gptq_accumulate_hessian(to_dev_bf16(xb), b, H.clone())
    torch.cuda.synchronize()
    scale = np.sqrt(np.outer(np.diag(want), np.diag(want)))
    for got, times in ((np_(H).astype(np.float64), 1), (np_(H2).astype(np.float64), 2)):
        say(f"   largest error over sqrt(h_ii h_jj): {(np.abs(got - times * want) / np.where(scale > 0, scale, np.inf)).max():.2e}")
        assert np.all(np.diag(got) >= 0.0)
        assert np.all(np.abs(got - times * want) <= 2e-5 * times * max(1.0, (T / 700) ** 0.5) * scale)
        assert np.array_equal(got, got.T)


@pytest.mark.parametrize("T,K,b", [(1408, 144, 16), (1409, 1744, 16), (1540, 256, 128), (800, 2416, 16), (1475, 4112, 16), (1130, 1264, 16), (1700, 912, 16)])
def test_hessian_of_many_rows_at_the_edges_of_stages_and_groups(fp4, oracle, T, K, b):
    """Rows kept as two scaled fp16 halves: row counts around whole stages of 32 and groups of four, and the rows behind them that
    are rotated on the spot (33 to 63 of them); tiles of 32, of 64, of 128, and two of them; rows whose sizes differ by up to 2^40, so that the scales of
    neighbouring groups do.  Bound relative to sqrt(h_ii h_jj) >= sum |x_i x_j|: both halves 2^-23 of either value, sums of 32 rows
    cut off at 2^-23, four of those added, then T / 128 of the groups' sums, each rounded to 2^-24; and 2 x 4 roundings of the rotated
    values on either side of the oracle's, of partial sums not larger than four times the value in the root mean square."""
    import torch
    x = np.random.default_rng(T).standard_normal((T, K)) * 2.0 ** np.random.default_rng(K).integers(-20, 21, (T, 1))
    xb = inputs.f32_to_bf16_bits(x.astype(np.float32))
    X = oracle.rotate(xb, b).astype(np.float64)
    want = X.T @ X
    say(f"gptq hessian T={T} K={K} b={b}")
    H = fp4.fp4_gptq_accumulate_hessian(to_dev_bf16(xb), b)
    H2 = fp4.fp4_gptq_accumulate_hessian(to_dev_bf16(xb), b, H.clone())
    torch.cuda.synchronize()
    scale = np.sqrt(np.outer(np.diag(want), np.diag(want)))
    for got, times in ((np_(H).astype(np.float64), 1), (np_(H2).astype(np.float64), 2)):
        say(f"   largest error over sqrt(h_ii h_jj): {(np.abs(got - times * want) / scale).max():.2e}")
        assert np.all(np.abs(got - times * want) <= times * (42 + T / 128) * 2.0 ** -24 * scale)
        assert np.array_equal(got, got.T)


@pytest.mark.parametrize("T,K", [(768, 2416), (1099, 2416), (1099, 4112)])
def test_hessian_of_fewer_rows_keeps_24_bits_of_a_rotated_value(fp4, T, K):
    """One row that is not zero, of integers whose rotated sums are exact and take up to 24 bits: below 1100 rows values are kept whole.
    Bound: of three bf16 parts (2^-9 and 2^-17 of the value at most behind the first) the products left out are 2^-25 of the whole, and
    the MFMA's result is cut off to 24 bits, 2^-23."""
    import torch
    rng = np.random.default_rng(T + K)
    row = rng.integers(128, 256, K) * 2.0 ** rng.integers(0, 13, K) * rng.choice([-1.0, 1.0], K)
    x = np.zeros((T, K), dtype=np.float32)
    x[T // 2] = row
    h = np.array([[(-1) ** bin(i & j).count("1") for j in range(16)] for i in range(16)])
    y = (row.reshape(-1, 16) @ h).reshape(-1)
    want = np.outer(y, y) / 16.0
    say(f"gptq hessian one row of {T}, K={K}")
    H = fp4.fp4_gptq_accumulate_hessian(to_dev_bf16(inputs.f32_to_bf16_bits(x)), 16)
    torch.cuda.synchronize()
    err = np.abs(np_(H).astype(np.float64) - want)
    say(f"   largest relative error: {(err / np.maximum(np.abs(want), 1.0)).max():.2e}")
    assert np.all(err <= 1.3 * 2.0 ** -23 * np.abs(want))


@pytest.mark.parametrize("log2_quiet", [8, 18, 30])
@pytest.mark.parametrize("T,K,b", [(1408, 144, 16), (1700, 912, 16), (1540, 256, 128), (1475, 4112, 16)])
def test_hessian_of_many_rows_with_quiet_channels_in_a_block(fp4, oracle, T, K, b, log2_quiet):
    """Every 64th row is constant within a block, which the rotation turns into one loud channel and exact zeros; the others are noise of
    2^-log2_quiet of that.  All other channels of the block are as quiet, and their entries as accurate on their own scale as any: the
    bound of the test above."""
    import torch
    rng = np.random.default_rng(T + log2_quiet)
    x = rng.standard_normal((T, K)) * 2.0 ** -log2_quiet
    x[::64] = np.repeat(rng.uniform(1.0, 2.0, (x[::64].shape[0], K // b)), b, axis=1)
    xb = inputs.f32_to_bf16_bits(x.astype(np.float32))
    X = oracle.rotate(xb, b).astype(np.float64)
    want = X.T @ X
    say(f"gptq hessian quiet channels T={T} K={K} b={b} 2^-{log2_quiet}")
    H = fp4.fp4_gptq_accumulate_hessian(to_dev_bf16(xb), b)
    torch.cuda.synchronize()
    got, scale = np_(H).astype(np.float64), np.sqrt(np.outer(np.diag(want), np.diag(want)))
    say(f"   largest error over sqrt(h_ii h_jj): {(np.abs(got - want) / scale).max():.2e}")
    assert np.all(np.abs(got - want) <= (42 + T / 128) * 2.0 ** -24 * scale)
    assert np.array_equal(got, got.T)


@pytest.mark.parametrize("log2_size", [-56, 56])
@pytest.mark.parametrize("T,K,b", [(1540, 256, 128), (1475, 4112, 16)])
def test_hessian_of_many_very_small_and_large_rows(fp4, T, K, b, log2_size):
    """Rows times 2^+-56: entries up to 2^123 and down to those of diagonals near 2^-102.  Every step is a power of two away from that of
    the same rows without the factor, and nothing leaves the range of normal numbers (entries below 2^-126 aside: half of their last
    place), so the entries are 2^+-112 times theirs."""
    import torch
    xb = inputs.f32_to_bf16_bits(np.random.default_rng(T).standard_normal((T, K)).astype(np.float32))
    x = to_dev_bf16(xb)
    say(f"gptq hessian T={T} K={K} b={b} times 2^{log2_size}")
    H = fp4.fp4_gptq_accumulate_hessian(x, b)
    big = fp4.fp4_gptq_accumulate_hessian((x * 2.0 ** log2_size).bfloat16(), b)
    torch.cuda.synchronize()
    H, big = np_(H).astype(np.float64), np_(big).astype(np.float64)
    assert np.isfinite(big).all()
    assert np.all(np.abs(big - np.ldexp(H, 2 * log2_size)) <= 2.0 ** -149)


def test_calibration_rows_to_codes_entirely_on_the_gpu(fp4, oracle, gptq):
    import torch
    N, K, T, b = 64, 512, 1536, 32
    r = inputs.RECIPES[6]
    wb, xb = r.w(N, K, salt=95), r.x(T, K, salt=96)
    say("gptq calibration rows -> codes")
    H = fp4.fp4_gptq_accumulate_hessian(to_dev_bf16(xb), b)
    perm, U = fp4.fp4_gptq_prepare(H, 1e-2, True)
    c, s, _ = fp4.fp4_gptq_quantize_weights(to_dev_bf16(wb), b, MX, U, perm)
    torch.cuda.synchronize()
    X = oracle.rotate(xb, b).astype(np.float64)
    H64 = X.T @ X
    want_c, want_s, sT, want_perm, _ = gptq.mr_gptq(wb, H64, b, MX)
    assert np.array_equal(np_(perm), want_perm)
    got_c, got_s = np_(c).reshape(N, -1), np_(s).reshape(N, -1)
    assert np.array_equal(got_s, want_s)
    y = oracle.rotate(wb, b)
    c_rtn, _, _ = oracle.quantize(y, MX)
    e_got = gptq.layer_error(y, got_c, want_s, MX, sT, H64)
    e_ref = gptq.layer_error(y, want_c, want_s, MX, sT, H64)
    e_rtn = gptq.layer_error(y, c_rtn, want_s, MX, sT, H64)
    say(f"   codes differing: {(unpack(got_c) != unpack(want_c)).mean():.2e}; layer error {e_got:.5e} vs oracle {e_ref:.5e} (round-to-nearest {e_rtn:.3e})")
    assert abs(e_got - e_ref) <= 1e-2 * e_ref and e_got < 0.8 * e_rtn


@pytest.mark.parametrize("N,K,b", [(40, 1088, 1), (17, 1600, 64)])
def test_rows_of_any_size_do_not_disturb_each_other(fp4, oracle, gptq, N, K, b):
    """Rows times powers of two up to 2^40 apart, one row zero: power-of-two scales follow, and the codes are the same -- every
    step of the sweep is exact under such a factor, also the scaled pairs of halves that an outer block's errors leave in."""
    import torch
    rng = np.random.default_rng(N)
    w = rng.standard_normal((N, K)).astype(np.float32)
    w[N // 2] = 0.0
    k = rng.integers(-20, 21, (N, 1))
    U = np.triu(rng.standard_normal((K, K)) * 0.02, 1) * 2.0 ** rng.integers(-16, 1, (1, K))   # (larger entries: the errors grow without bound)
    U[np.diag_indices(K)] = rng.uniform(0.5, 2.0, K)
    perm = rng.permutation(K).astype(np.int32)
    say(f"gptq row scales N={N} K={K}")
    got = []
    for x in (w, np.ldexp(w, k).astype(np.float32)):
        c, s, _ = fp4.fp4_gptq_quantize_weights(to_dev_bf16(inputs.f32_to_bf16_bits(x)), b, MX, to_dev(U.astype(np.float32)), to_dev(perm))
        torch.cuda.synchronize()
        got.append((np_(c).reshape(N, -1), np_(s).reshape(N, -1).astype(np.int64)))
    assert np.array_equal(got[0][0], got[1][0])
    live = np.arange(N) != N // 2
    assert np.array_equal(got[0][1][live] + k[live], got[1][1][live])


@pytest.mark.parametrize("N,K,b", [(40, 1088, 1), (17, 1600, 64)])
def test_rows_of_the_smallest_and_largest_size(fp4, N, K, b):
    """The same with rows 2^190 apart: running values and updates stay between 2^-126 and 2^127."""
    import torch
    rng = np.random.default_rng(N)
    w = rng.standard_normal((N, K)).astype(np.float32)
    k = rng.integers(-70, 121, (N, 1))
    k[0], k[-1] = -70, 120
    U = np.triu(rng.standard_normal((K, K)) * 0.02, 1) * 2.0 ** rng.integers(-16, 1, (1, K))
    U[np.diag_indices(K)] = rng.uniform(0.5, 2.0, K)
    say(f"gptq row scales N={N} K={K} 2^-70 .. 2^120")
    got = []
    for x in (w, np.ldexp(w, k).astype(np.float32)):
        c, s, _ = fp4.fp4_gptq_quantize_weights(to_dev_bf16(inputs.f32_to_bf16_bits(x)), b, MX, to_dev(U.astype(np.float32)), None)
        torch.cuda.synchronize()
        got.append((np_(c).reshape(N, -1), np_(s).reshape(N, -1).astype(np.int64)))
    assert np.array_equal(got[0][0], got[1][0])
    assert np.array_equal(got[0][1] + k, got[1][1])


@pytest.mark.parametrize("N,K", [(1, 576), (128, 640), (129, 704), (127, 1600)])
def test_update_behind_an_outer_block_at_the_edges_of_its_tiles(fp4, oracle, gptq, N, K):
    """A dense factor with full 24-bit entries, so that everything behind column 512 has its values from the 128 x 128 tiles
    of the update: one row, whole and ragged tiles, a last tile of 64 columns.  The update is as exact as a binary32 sum, so
    codes differ only where the running value is within binary32 noise of a midpoint: the bound of the tests above."""
    import torch
    rng = np.random.default_rng(N + K)
    w = rng.standard_normal((N, K)).astype(np.float32)
    wb = inputs.f32_to_bf16_bits(w)
    U = np.triu(rng.standard_normal((K, K)) * 0.02, 1).astype(np.float32)
    U[np.diag_indices(K)] = rng.uniform(0.5, 2.0, K).astype(np.float32)
    perm = rng.permutation(K).astype(np.int32)
    y = oracle.rotate(wb, 1)
    _, scales, _ = oracle.quantize(y, MX)
    want, _ = gptq.sweep(y, scales, MX, None, U, perm)
    say(f"gptq dense factor N={N} K={K}")
    c, s, _ = fp4.fp4_gptq_quantize_weights(to_dev_bf16(wb), 1, MX, to_dev(U), to_dev(perm))
    torch.cuda.synchronize()
    assert np.array_equal(np_(s).reshape(N, -1), scales)
    diff = unpack(np_(c).reshape(N, -1)) != unpack(want)
    say(f"   codes differing from the oracle: {diff.mean():.2e}")
    assert diff.mean() <= 1e-3


@pytest.mark.parametrize("fmt,b", [(MX, 1), (NV, 16)])
@pytest.mark.parametrize("N,K", [(1, 576), (16, 512), (128, 640), (130, 1600), (40, 1088)])
def test_sweep_in_the_least_workspace(fp4, fmt, b, N, K):
    """Without room for the prepared operands of the update: the same codes, and nothing written behind the workspace."""
    import torch
    say(f"gptq least workspace N={N} K={K} fmt={fmt}")
    g = torch.Generator(device="cuda")
    g.manual_seed(N + K)
    w = torch.randn(N, K, device="cuda", generator=g).bfloat16()
    U = torch.triu(torch.randn(K, K, device="cuda", generator=g) * 0.02, 1) + torch.diag(0.5 + torch.rand(K, device="cuda", generator=g))
    perm = torch.randperm(K, device="cuda", generator=g).int()
    up = lambda n: (n + 255) // 256 * 256
    full = fp4.workspace_bytes(fp4.OP_GPTQ, N, 0, K, fmt)
    need = full - 2080 * ((N + 15) // 16 * 16 + K) + up(2048 * N)
    room = torch.full((full + 65536,), 0xa5, dtype=torch.uint8, device="cuda")
    want = fp4.fp4_gptq_quantize_weights(w, b, fmt, U, perm)
    got = fp4.fp4_gptq_quantize_weights(w, b, fmt, U, perm, workspace=room[:need])
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(want, got) if x is not None)
    assert bool((room[need:] == 0xa5).all())


@pytest.mark.parametrize("log2_loud", [12, 40, -40])
def test_update_with_channels_of_two_kinds_that_have_nothing_in_common(fp4, oracle, gptq, log2_loud):
    """H = D C D with channels of two kinds that C keeps apart, the one 2^log2_loud times as loud: the factor's columns are divided by D,
    so the errors of the loud columns are that much larger than those of the quiet ones among them, on which alone the
    other quiet columns depend.  Codes as in the test above, of either kind."""
    import torch
    N, K = 130, 1600
    rng = np.random.default_rng(50 + log2_loud)
    wb = inputs.f32_to_bf16_bits(rng.standard_normal((N, K)).astype(np.float32))
    loud = rng.random(K) < 0.5
    U = np.triu(rng.standard_normal((K, K)) * 0.02, 1) * (loud[:, None] == loud[None, :])
    U[np.diag_indices(K)] = rng.uniform(0.5, 2.0, K)
    U = (U * np.where(loud, 2.0 ** -log2_loud, 1.0)[None, :]).astype(np.float32)
    perm = np.arange(K, dtype=np.int32)
    y = oracle.rotate(wb, 1)
    _, scales, _ = oracle.quantize(y, MX)
    want, _ = gptq.sweep(y, scales, MX, None, U, perm)
    say(f"gptq two kinds of channels 2^{log2_loud}")
    c, s, _ = fp4.fp4_gptq_quantize_weights(to_dev_bf16(wb), 1, MX, to_dev(U), to_dev(perm))
    torch.cuda.synchronize()
    diff = unpack(np_(c).reshape(N, -1)) != unpack(want)
    say(f"   codes differing from the oracle: loud {diff[:, loud].mean():.2e}, quiet {diff[:, ~loud].mean():.2e}")
    assert diff[:, loud].mean() <= 1e-3 and diff[:, ~loud].mean() <= 1e-3


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("at", [40, 616, 1130])
def test_sweep_keeps_the_codes_of_columns_visited_before_a_non_finite_weight(fp4, oracle, value, at):
    """A non-finite weight spoils the columns of its row that are visited after it (their running values carry its error),
    not those visited before it, in the same 64-column block either; other rows see nothing of it."""
    import torch
    N, K, row = 35, 1152, 17
    rng = np.random.default_rng(at)
    w = rng.standard_normal((N, K)).astype(np.float32)
    U = np.triu(rng.standard_normal((K, K)) * 0.02, 1).astype(np.float32)
    U[np.diag_indices(K)] = rng.uniform(0.5, 2.0, K).astype(np.float32)
    say(f"gptq non-finite weight {value} at {at}")
    codes = []
    for v in (w[row, at], value):
        w[row, at] = v
        c, s, _ = fp4.fp4_gptq_quantize_weights(to_dev_bf16(inputs.f32_to_bf16_bits(w)), 1, MX, to_dev(U), None)
        torch.cuda.synchronize()
        codes.append(unpack(np_(c).reshape(N, -1)))
    group = at // 32 * 32      # (the columns of its own group may have another scale)
    assert np.array_equal(codes[0][row, :group], codes[1][row, :group])
    others = np.arange(N) != row
    assert np.array_equal(codes[0][others], codes[1][others])


def test_sweep_at_layer_size_on_sampled_rows(fp4, oracle, gptq):
    """A whole [4096, 4096] layer through the library (the benchmark's shape: 64 blocks, 8 outer blocks), checked against the
    oracle on 32 sampled rows -- rows never interact, so the oracle sweeps just those rows with the same factor."""
    import torch
    N, K, T, b = 4096, 4096, 4608, 32
    r = inputs.RECIPES[6]
    wb = r.w(N, K, salt=120)
    H = synthetic_hessian(oracle, K, T, b, salt=121)
    perm = gptq.act_order(H).astype(np.int32)
    U = gptq.inverse_factor(H, perm, damp=1e-2).astype(np.float32)
    say("gptq layer size: N = K = 4096")
    c, s, _ = fp4.fp4_gptq_quantize_weights(to_dev_bf16(wb), b, MX, to_dev(U), to_dev(perm))
    torch.cuda.synchronize()
    rows = np.sort(np.random.default_rng(5).choice(N, 32, replace=False))
    y = oracle.rotate(wb[rows], b)
    c_rtn, scales, _ = oracle.quantize(y, MX)
    want, _ = gptq.sweep(y, scales, MX, None, U, perm)
    got_c, got_s = np_(c).reshape(N, -1)[rows], np_(s).reshape(N, -1)[rows]
    ok = (got_s == scales).all(axis=1)
    assert ok.mean() >= 0.9
    diff = (unpack(got_c) != unpack(want))[ok].mean()
    e_got = gptq.layer_error(y[ok], got_c[ok], scales[ok], MX, None, H)
    e_ref = gptq.layer_error(y[ok], want[ok], scales[ok], MX, None, H)
    e_rtn = gptq.layer_error(y[ok], c_rtn[ok], scales[ok], MX, None, H)
    say(f"   codes differing from the oracle: {diff:.2e}; layer error {e_got:.5e} vs oracle {e_ref:.5e} (round-to-nearest {e_rtn:.3e})")
    assert diff <= 1e-3 and abs(e_got - e_ref) <= 2e-3 * e_ref and e_got < 0.8 * e_rtn


def test_prepare_at_layer_size(fp4, oracle, gptq):
    """K = 4096 (64 diagonal blocks, six doubling levels of the triangular inversion) against the fp64 factor, and the
    defining identity on 64 sampled columns."""
    import torch
    K = 4096
    H32 = synthetic_hessian(oracle, K, 4608, 32, salt=121).astype(np.float32)
    say("gptq prepare K=4096")
    perm, U = fp4.fp4_gptq_prepare(to_dev(H32), 1e-2, True)
    torch.cuda.synchronize()
    perm, U = np_(perm), np_(U).astype(np.float64)
    H64 = H32.astype(np.float64)
    want_perm = gptq.act_order(H64)
    assert np.array_equal(perm, want_perm)
    want_U = gptq.inverse_factor(H64, want_perm, damp=1e-2)
    rel = np.linalg.norm(U - want_U) / np.linalg.norm(want_U)
    A = H64[np.ix_(want_perm, want_perm)]
    A[np.diag_indices(K)] += 1e-2 * np.mean(np.diag(A))
    cols = np.sort(np.random.default_rng(6).choice(K, 64, replace=False))
    resid = np.abs(U.T @ (U @ A[:, cols]) - np.eye(K)[:, cols]).max()
    say(f"   relative error of U {rel:.2e}; max |U^T U A - I| on 64 columns {resid:.2e}")
    assert rel <= 1e-3 and resid <= 5e-3


def test_widest_layer_of_the_benchmark_model(fp4, oracle, gptq):
    """K = 14336 (the down projection: 224 diagonal blocks, eight doubling levels, an 822 MB factor): the order against
    the oracle's, the factor through the identity that defines it, U^T U (H_perm + lambda I) = I, on sampled columns
    (an fp64 inverse of this size is minutes of CPU), and the sweep of 48 rows with that factor against the oracle's
    sweep of 12 of them.  The Hessian is a rank-96 Gram matrix plus a positive diagonal, built directly."""
    import torch
    K, N, b = 14336, 48, 32
    rng = np.random.default_rng(140)
    V = rng.standard_normal((K, 96)) * rng.uniform(0.3, 2.0, (K, 1))
    H64 = V @ V.T / 96.0
    H64[np.diag_indices(K)] += rng.uniform(0.5, 2.0, K)
    H32 = H64.astype(np.float32)
    H64 = H32.astype(np.float64)
    say("gptq prepare K=14336")
    perm_d, U_d = fp4.fp4_gptq_prepare(to_dev(H32), 1e-2, True)
    torch.cuda.synchronize()
    perm = np_(perm_d)
    want_perm = gptq.act_order(H64)
    assert np.array_equal(perm, want_perm)
    U = np_(U_d).astype(np.float64)
    assert np.all(np.diag(U) > 0)
    cols = np.sort(rng.choice(K, 16, replace=False))
    A_cols = H64[np.ix_(want_perm, want_perm[cols])]
    A_cols[cols, np.arange(16)] += 1e-2 * np.mean(np.diag(H64))
    E = np.zeros((K, 16))
    E[cols, np.arange(16)] = 1.0
    resid = np.abs(U.T @ (U @ A_cols) - E).max()
    below = max(np.abs(U[r, :r]).max() for r in (1, K // 2, K - 1))
    say(f"   max |U^T U A - I| on 16 columns {resid:.2e}")
    assert resid <= 5e-3 and below == 0.0

    wb = inputs.RECIPES[6].w(N, K, salt=141)
    say("gptq sweep N=48 K=14336")
    c, s, _ = fp4.fp4_gptq_quantize_weights(to_dev_bf16(wb), b, MX, U_d, perm_d)
    torch.cuda.synchronize()
    rows = np.arange(0, N, 4)
    y = oracle.rotate(wb[rows], b)
    c_rtn, scales, _ = oracle.quantize(y, MX)
    want, _ = gptq.sweep(y, scales, MX, None, U, perm)
    got_c, got_s = np_(c).reshape(N, -1)[rows], np_(s).reshape(N, -1)[rows]
    ok = (got_s == scales).all(axis=1)
    assert ok.mean() >= 0.9
    diff = (unpack(got_c) != unpack(want))[ok].mean()
    e_got = gptq.layer_error(y[ok], got_c[ok], scales[ok], MX, None, H64)
    e_ref = gptq.layer_error(y[ok], want[ok], scales[ok], MX, None, H64)
    e_rtn = gptq.layer_error(y[ok], c_rtn[ok], scales[ok], MX, None, H64)
    say(f"   codes differing from the oracle: {diff:.2e}; layer error {e_got:.5e} vs oracle {e_ref:.5e} (round-to-nearest {e_rtn:.3e})")
    assert diff <= 1e-3 and abs(e_got - e_ref) <= 2e-3 * e_ref and e_got < 0.9 * e_rtn
