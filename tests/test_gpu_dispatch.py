"""Parity of single kernels and of the branches of their dispatch, at the sizes where they can go wrong: edges of
tiles, remainders, the smallest and the largest of their ranges.  Workspaces start as NaN patterns, so a kernel that
reads what no kernel of its own call wrote shows."""
import math

import numpy as np
import pytest
import torch

import csat_inputs as gen
import paper_2507_02957_amd as csat
from oracle import csat_oracle as orc
from tests.gpu_harness import DEV, TOL, DeviceProblem, assert_close, to_dev, to_np
from tests.test_gpu_parity import _mu, _small, _support_check, options  # noqa: F401  (options: fixture)

pytestmark = pytest.mark.gpu


def _problem(w, Q, K, V, Phi):
    p = DeviceProblem(w, Q, K, V, Phi)
    p.ws.fill_(0xFF)
    return p


@pytest.mark.parametrize("iters", [0, 3])
@pytest.mark.parametrize("d", [64, 128])
def test_separate_matrices_read_only_what_the_call_wrote(d, iters):
    """V~ for a separate value matrix needs V transposed in this call, also where the synthesis reads V as it is."""
    w = _small("kv_fresh", B=1, H=2, n_q=70, n=200, d=d, m=48, dtype="bf16", iters=iters)
    Q, K, V = gen.make_qkv(w)
    PhiV = gen.make_workload_phi(w)
    PhiK = gen.quantize(gen.make_phi("rademacher", w.m, w.n, seed=7), w.dtype)
    mu = _mu(PhiV)
    ref = orc.forward(Q, K, V, PhiV, w.lam, mu, iters, Phi_K=PhiK)
    p = _problem(w, Q, K, V, PhiV)
    C, Z = p.empty(p.BH, w.n_q, w.d), p.empty(p.BH, w.n_q, w.d)
    csat.csat_forward_kv(p.dims, p.Q, p.K, p.V, to_dev(PhiK, w.dtype), p.Phi, w.lam, mu, iters, C, Z, None, p.ws)
    torch.cuda.synchronize()
    assert_close("Z", to_np(Z), ref["Z"], TOL[w.dtype])
    assert_close("C", to_np(C), ref["C"] if iters else ref["Z"], TOL[w.dtype])


# n_q around a wavefront's 32 rows and a workgroup's 256; m around a tile, around the last pair of tiles and on both
# sides of what fits LDS (d = 64: 20 tiles; d = 128: 10)
Z_ONLY_CASES = [(1, 5, 5, 32), (33, 31, 31, 32), (32, 33, 33, 64), (257, 96, 64, 64), (70, 640, 640, 64), (70, 641, 641, 64),
                (300, 1100, 1055, 64), (65, 200, 97, 96), (40, 320, 320, 128), (290, 330, 321, 128), (1, 400, 353, 128),
                # the lines between that kernel and the three for a short query side at d = 128
                (64, 740, 737, 128), (65, 740, 737, 128), (64, 736, 736, 128), (255, 490, 490, 128), (256, 490, 490, 128), (33, 480, 480, 128)]


@pytest.mark.parametrize("n_q,n,m,d", Z_ONLY_CASES)
def test_compressed_attention_without_the_attention_matrix(n_q, n, m, d, options):
    """Z when A~ is not asked for (a kernel of its own in bf16) against the oracle and against the call that asks for it."""
    w = _small("z_only", B=1, H=3, n_q=n_q, n=n, d=d, m=m, dtype="bf16")
    Q, K, V = gen.make_qkv(w)
    Phi = gen.make_workload_phi(w)
    p = _problem(w, Q, K, V, Phi)
    Kc, Vc = p.measure()
    A, Z = orc.compressed_attention(Q, to_np(Kc), to_np(Vc))
    Zg = p.empty(p.BH, n_q, d)
    p.ws.fill_(0xFF)
    csat.csat_compressed_attention(p.dims, p.Q, Kc, Vc, None, Zg, p.ws)
    torch.cuda.synchronize()
    assert_close("Z", to_np(Zg), Z, TOL["bf16"])
    _, Zf = p.attention(Kc, Vc)
    assert_close("Z against the call with A~", to_np(Zg), to_np(Zf), TOL["bf16"])
    # the block without iterations: the (hi | lo) pair of K~ through the same kernel
    mu = _mu(Phi)
    ref = orc.forward(Q, K, V, Phi, w.lam, mu, 0)
    C, Z0, _ = p.forward(w.lam, mu, 0, want_x=False)
    assert_close("C (no iterations)", to_np(C), ref["Z"], TOL["bf16"])
    assert torch.equal(C, Z0)


def test_compressed_attention_moves_its_reference_score():
    """Scores that grow along m by far more than 2^8 from one pair of tiles to the next (the kernel without A~ rescales its
    output then), and by less than that (it does not)."""
    d, m, n_q = 64, 224, 64
    w = _small("z_growing", B=1, H=2, n_q=n_q, n=256, d=d, m=m, dtype="bf16")
    rng = np.random.default_rng(3)
    Q = gen.quantize(rng.standard_normal((2, n_q, d)).astype(np.float32), "bf16")
    ramp = np.stack([np.linspace(0.0, 12.0, m), np.linspace(0.0, 0.6, m)])
    Kc = gen.quantize((Q[:, :1] * ramp[:, :, None] + 0.1 * rng.standard_normal((2, m, d))).astype(np.float32), "bf16")
    Vc = gen.quantize(rng.standard_normal((2, m, d)).astype(np.float32), "bf16")
    p = _problem(w, Q, Q[:, :1].repeat(256, 1), Q[:, :1].repeat(256, 1), gen.make_workload_phi(w))
    _, Z = orc.compressed_attention(Q, Kc, Vc)
    Zg = p.empty(2, n_q, d)
    csat.csat_compressed_attention(p.dims, p.Q, to_dev(Kc, "bf16"), to_dev(Vc, "bf16"), None, Zg, p.ws)
    torch.cuda.synchronize()
    assert_close("Z", to_np(Zg), Z, TOL["bf16"])


# the row's first finite score in the second pair of tiles, in the last tile, nowhere in one row
@pytest.mark.parametrize("d,m,first", [(64, 128, 64), (64, 200, 193), (128, 330, 300), (32, 700, 129)])
def test_compressed_attention_with_scores_of_minus_infinity(d, m, first):
    """Scores of -inf have weight 0 wherever they come in the row, also where a row of the same tile has finite ones
    there; a row without any finite score is NaN, as its softmax is."""
    n_q = 70
    w = _small("z_minus_inf", B=1, H=2, n_q=n_q, n=max(m, 256), d=d, m=m, dtype="bf16")
    rng = np.random.default_rng(m)
    Q = gen.quantize(rng.uniform(0.5, 2.0, (2, n_q, d)).astype(np.float32), "bf16")
    Q[:, 1::3] *= 2.0 ** -124                                # these rows' scores are finite everywhere
    Kc = gen.quantize(rng.standard_normal((2, m, d)).astype(np.float32), "bf16")
    Vc = gen.quantize(rng.standard_normal((2, m, d)).astype(np.float32), "bf16")
    Kc[:, :first] = -2.0 ** 127                              # (times 0.5 to 2, summed over d: beyond the largest float)
    Kc[1, first::2] = -2.0 ** 127
    p = _problem(w, Q, np.zeros((2, w.n, d), np.float32), np.zeros((2, w.n, d), np.float32), gen.make_workload_phi(w))
    s = np.matmul(Q.astype(np.float64), Kc.astype(np.float64).transpose(0, 2, 1)) / np.sqrt(d)
    s[s < -1e38] = -np.inf
    e = np.exp(s - s.max(-1, keepdims=True))
    want = np.matmul(e / e.sum(-1, keepdims=True), Vc.astype(np.float64))
    assert np.isinf(s[:, 0, :first]).all() and np.isfinite(s[:, 1]).all() and np.isfinite(s[0, 0, first:]).all()
    Zg = p.empty(2, n_q, d)
    csat.csat_compressed_attention(p.dims, p.Q, to_dev(Kc, "bf16"), to_dev(Vc, "bf16"), None, Zg, p.ws)
    torch.cuda.synchronize()
    assert_close("Z", to_np(Zg), want, TOL["bf16"])
    if m <= 512:
        _, Zf = p.attention(to_dev(Kc, "bf16"), to_dev(Vc, "bf16"))
        assert_close("Z with A~", to_np(Zf), want, TOL["bf16"])
    Kc[:] = -2.0 ** 127                                      # no finite score but in the small rows
    csat.csat_compressed_attention(p.dims, p.Q, to_dev(Kc, "bf16"), to_dev(Vc, "bf16"), None, Zg, p.ws)
    torch.cuda.synchronize()
    Z = to_np(Zg)
    assert np.isnan(Z[:, 0::3]).all() and np.isfinite(Z[:, 1::3]).all()


@pytest.mark.parametrize("d,m", [(64, 16), (64, 256), (128, 390), (96, 1000)])
def test_compressed_attention_of_large_values(d, m):
    """Values of V~ whose sum over m is beyond the largest float, but not their average: equal scores, and scores that rise
    by less than the kernel moves its reference for."""
    n_q = 64
    w = _small("z_large_values", B=1, H=2, n_q=n_q, n=max(m, 256), d=d, m=m, dtype="bf16")
    rng = np.random.default_rng(m)
    Q = gen.quantize(rng.standard_normal((2, n_q, d)).astype(np.float32), "bf16")
    Kc = np.zeros((2, m, d), np.float32)
    Kc[1] = gen.quantize((np.linspace(0.0, 4.0, m)[:, None] * Q[1, :1] / np.sqrt(d)).astype(np.float32), "bf16")
    Vc = gen.quantize((rng.uniform(0.5, 1.0, (2, m, d)) * 3e38).astype(np.float32), "bf16")
    p = _problem(w, Q, np.zeros((2, w.n, d), np.float32), np.zeros((2, w.n, d), np.float32), gen.make_workload_phi(w))
    _, want = orc.compressed_attention(Q, Kc, Vc)
    Zg = p.empty(2, n_q, d)
    csat.csat_compressed_attention(p.dims, p.Q, to_dev(Kc, "bf16"), to_dev(Vc, "bf16"), None, Zg, p.ws)
    torch.cuda.synchronize()
    assert_close("Z", to_np(Zg), want, TOL["bf16"])


# few workgroups and a long contraction: two groups of wavefronts split it (from n = 512 on at d = 128; at d = 64 from 1024 on
# where the last round of 512 is at least three quarters full, and from 2048 on always)
@pytest.mark.parametrize("n,m,d,zero_iters", [(511, 40, 64, True), (512, 40, 64, True), (700, 97, 128, True), (1025, 64, 128, False),
                                              (511, 40, 128, True), (512, 40, 128, False), (1024, 40, 64, True), (1408, 70, 64, False), (1409, 70, 64, True), (2050, 33, 64, True),
                                              (1500, 33, 64, False), (4097, 65, 64, True)])
def test_measurement_with_a_split_contraction(n, m, d, zero_iters, options):
    w = _small("split", B=1, H=3, n_q=40, n=n, d=d, m=m, dtype="bf16", iters=0 if zero_iters else 2, lam=0.02)
    Q, K, V = gen.make_qkv(w)
    Phi = gen.make_workload_phi(w)
    mu = _mu(Phi)
    ref = orc.forward(Q, K, V, Phi, w.lam, mu, w.iters)
    p = _problem(w, Q, K, V, Phi)
    Kc, Vc = p.measure()
    assert_close("Kc", to_np(Kc), ref["Kc"], TOL["bf16"])
    assert_close("Vc", to_np(Vc), ref["Vc"], TOL["bf16"])
    p.ws.fill_(0xFF)
    C, Z, _ = p.forward(w.lam, mu, w.iters, want_x=False)              # K~ as a pair and as fragments
    assert_close("Z", to_np(Z), ref["Z"], TOL["bf16"])
    C2, _, _ = p.forward(w.lam, mu, w.iters, want_z=False, want_x=False)   # K~ only
    assert_close("C", to_np(C2), to_np(C), TOL["bf16"])


# (n_q, n, m, iterations, decoder kernel): chunk counts on both sides of every instance's, one tile of m and eight, the
# largest Phi that fits LDS (80 chunk-tiles) and the first that does not, a ragged last row tile, one iteration
RESIDENT_CASES = [(33, 65, 8, 3, 5), (31, 96, 33, 4, 5), (70, 97, 96, 3, 5), (64, 160, 129, 2, 5), (40, 161, 160, 3, 5),
                  (97, 224, 224, 2, 5), (50, 225, 200, 3, 5), (129, 288, 256, 1, 5), (33, 289, 192, 3, 5), (32, 384, 161, 2, 5),
                  (20, 385, 160, 3, 5), (65, 512, 32, 3, 5), (40, 513, 32, 2, 6), (40, 385, 161, 2, 6), (64, 200, 200, 1, 5)]


@pytest.mark.parametrize("n_q,n,m,iters,kernel", RESIDENT_CASES)
def test_decoder_with_phi_in_lds(n_q, n, m, iters, kernel, options):
    """Small problems keep Phi in LDS and the iterate in registers: the bits of the decoder that streams both, and the
    oracle.  lambda small enough for a dense iterate in every chunk."""
    w = _small("resident", B=2, H=3, n_q=n_q, n=n, d=64, m=m, dtype="bf16", iters=iters, lam=0.002)
    Q, K, V = gen.make_qkv(w)
    Phi = gen.make_workload_phi(w)
    mu = _mu(Phi)
    p = _problem(w, Q, K, V, Phi)
    C, _, X = p.forward(w.lam, mu, iters)
    assert csat.csat_profile_decoder_kernel() == kernel
    assert csat.csat_decoder_status(p.ws) == 0
    ref = orc.forward(Q, K, V, Phi, w.lam, mu, iters)
    assert_close("X", to_np(X), ref["X"], TOL["bf16"])
    assert_close("C", to_np(C), ref["C"], TOL["bf16"])
    options("fused_thin", 1)
    options("synthesis", 1)       # (that decoder can also form C itself, in another summation order)
    p.ws.fill_(0xFF)
    C1, _, X1 = p.forward(w.lam, mu, iters)
    assert csat.csat_profile_decoder_kernel() != 5
    same = torch.equal(X, X1) and torch.equal(C, C1)
    assert same


def test_decoder_with_phi_in_lds_keeps_infinities_out_of_the_pads(options):
    """11 chunks on the instance for 12, and a synthesis that reads the operand's pads: an infinite row of positive products is
    infinite, as on the decoder that streams Phi, not NaN."""
    n_q, n, m, d = 260, 352, 64, 136
    w = _small("resident_pads", B=1, H=1, n_q=n_q, n=n, d=d, m=m, dtype="bf16", iters=1)
    rng = np.random.default_rng(1)
    draw = lambda *s: gen.quantize(rng.uniform(0.5, 1.0, s).astype(np.float32), "bf16")
    p = _problem(w, draw(1, n_q, d), draw(1, n, d), draw(1, n, d), draw(m, n))
    Y = rng.uniform(0.5, 1.0, (1, n_q, m)).astype(np.float32)
    Y[0, 5, 7] = np.inf
    out = []
    for thin, kernel in ((0, (5,)), (1, (0, 1, 3, 4))):
        options("fused_thin", thin)
        X, C = p.recover(to_dev(Y, "f32"), 0.01, 0.01, 1)
        torch.cuda.synchronize()
        assert csat.csat_profile_decoder_kernel() in kernel
        out.append((to_np(X), to_np(C)))
    assert np.isposinf(out[1][1][0, 5]).all()
    for a, b in zip(*out):
        assert (np.isposinf(a) == np.isposinf(b)).all() and (np.isfinite(a) == np.isfinite(b)).all()


# (rows, n, m): rows around the 128-row tile, columns around the 64-wide one, contractions around a step of 32 and shorter
FLOAT_PRODUCTS = [(127, 130, 96), (128, 64, 64), (129, 65, 33), (5, 9, 8), (257, 1056, 130), (33, 33, 31), (1, 31, 1), (1025, 1099, 1000)]


@pytest.mark.parametrize("rows,n,m", FLOAT_PRODUCTS)
def test_float_products_keep_float_precision(rows, n, m, options):
    """The float decoder's products run as six bf16 ones over the operands' three parts.  One iteration without a
    threshold is X = mu Phi^T y, and C = X V.  Bound per element: dropped products 2^-24 of sum |a b| (reached by operands
    like 1 + 2^-8 - 2^-17, whose parts are 1, 2^-8 and -2^-17: one row holds only such), one rounding (2^-24) of a partial sum per
    16 of the contraction and three at the end; 2^-23 for the iterate itself."""
    w = _small("f32_products", B=1, H=1, n_q=rows, n=n, d=64, m=m, dtype="f32", iters=1)
    Q, K, V = gen.make_qkv(w)
    Phi = gen.make_workload_phi(w)
    p = _problem(w, Q, K, V, Phi)
    Y = np.random.default_rng(rows).standard_normal((rows, m)).astype(np.float32)
    Y[rows // 4] = 1 + 2.0 ** -8 - 2.0 ** -17
    X, C = p.empty(1, rows, n, dtype=torch.float32), p.empty(1, rows, w.d)

    def decode(y):
        p.ws.fill_(0xFF)
        csat.csat_recover(p.dims, to_dev(y, "f32"), p.Phi, 0.0, 0.5, 1, X, p.V, C, p.ws)
        return X.clone(), C.clone()

    def bound(k):
        return 2.0 ** -24 + 2.0 ** -24 * (k / 16 + 3)

    Xg, Cg = (to_np(t)[0].astype(np.float64) for t in decode(Y))
    P, V64 = Phi.astype(np.float64), V.reshape(n, w.d).astype(np.float64)
    want = 0.5 * (Y.astype(np.float64) @ P)
    slack = (bound(m) + 2.0 ** -23) * 0.5 * (np.abs(Y) @ np.abs(P))
    assert (np.abs(Xg - want) <= slack).all()
    assert (np.abs(Cg - Xg @ V64) <= bound(n) * (np.abs(Xg) @ np.abs(V64))).all()
    # infinities, NaN and the largest floats come out as the float MFMA has them
    Y[0, 0], Y[rows // 2, m - 1], Y[rows // 3, m // 2], Y[rows - 1, 0] = np.inf, -np.inf, 3.4e38, np.nan
    Xg, Cg = decode(Y)
    options("gemm", 1)
    Xo, Co = decode(Y)
    for got, old in ((Xg, Xo), (Cg, Co)):
        same = torch.equal(got.isnan(), old.isnan()) and torch.equal(got.isposinf(), old.isposinf()) and torch.equal(got.isneginf(), old.isneginf())
        assert same
    assert rows == 1 or Xo.isinf().any()


@pytest.mark.parametrize("rows,n,m,iters", [(130, 300, 100, 1), (130, 300, 100, 3), (70, 128, 64, 3), (40, 161, 128, 2)])
@pytest.mark.parametrize("scale", [1e-33, 1e-37])
def test_float_decoder_of_small_numbers(rows, n, m, iters, scale):
    """Measurements near the smallest floats, in every row or in some rows of a tile (beside ordinary ones): their bf16
    parts would not hold all of their bits.  Without a threshold X is linear in y, so its error in a row is held to the
    row's own size: at most m / 2 (n / 2) roundings of 2^-24 in a product, one product of each kind per iteration, and C's."""
    w = _small("f32_small_numbers", B=1, H=1, n_q=rows, n=n, d=64, m=m, dtype="f32", iters=iters)
    Q, K, V = gen.make_qkv(w)
    Phi = gen.make_workload_phi(w)
    mu = _mu(Phi)
    p = _problem(w, Q, K, V, Phi)
    P, V64 = Phi.astype(np.float64), V.reshape(n, w.d).astype(np.float64)
    for mixed in (False, True):
        Y = np.random.default_rng(rows).standard_normal((rows, m)) * scale
        if mixed:
            Y[::2] /= scale
        Y = Y.astype(np.float32)
        X, C = p.empty(1, rows, n, dtype=torch.float32), p.empty(1, rows, w.d)
        csat.csat_recover(p.dims, to_dev(Y, "f32"), p.Phi, 0.0, mu, iters, X, p.V, C, p.ws)
        torch.cuda.synchronize()
        x = np.zeros((rows, n))
        for _ in range(iters):
            x = x + mu * ((Y.astype(np.float64) - x @ P.T) @ P)
        bound = 2.0 ** -24 * (m / 2 + n / 2 + 4) * iters
        for got, want in ((to_np(X)[0], x), (to_np(C)[0], x @ V64)):
            assert (np.linalg.norm(got - want, axis=-1) <= bound * np.linalg.norm(want, axis=-1)).all()


# (n_q, n, m, iterations, in LDS): chunks per wavefront below, at and beyond one, idle wavefronts, one to four tiles of m,
# the largest Phi that fits and the first that does not, ragged rows, unaligned n
FLOAT_RESIDENT_CASES = [(33, 40, 8, 2, True), (32, 128, 32, 5, True), (50, 131, 64, 4, True), (64, 160, 128, 3, True), (7, 161, 128, 3, False),
                        (40, 224, 96, 3, True), (31, 225, 96, 2, False), (70, 350, 64, 3, True), (20, 353, 64, 3, False), (33, 736, 32, 3, True),
                        (20, 737, 32, 2, False), (96, 97, 97, 6, True), (40, 128, 64, 1, False), (1, 20, 20, 3, True)]


@pytest.mark.parametrize("n_q,n,m,iters,resident", FLOAT_RESIDENT_CASES)
def test_float_decoder_with_phi_in_lds(n_q, n, m, iters, resident, options):
    """Small float problems in one launch: codes, support and context against the oracle, forward and stage call."""
    w = _small("f32_resident", B=2, H=3, n_q=n_q, n=n, d=64, m=m, dtype="f32", iters=iters, lam=0.01)
    Q, K, V = gen.make_qkv(w)
    Phi = gen.make_workload_phi(w)
    mu = _mu(Phi)
    p = _problem(w, Q, K, V, Phi)
    C, _, X = p.forward(w.lam, mu, iters)
    assert csat.csat_profile_decoder_kernel() == (5 if resident else -1)
    assert csat.csat_decoder_status(p.ws) == 0
    ref = orc.forward(Q, K, V, Phi, w.lam, mu, iters)
    assert_close("X", to_np(X), ref["X"], TOL["f32"])
    assert_close("C", to_np(C), ref["C"], TOL["f32"])
    _support_check(w.name, to_np(X), ref, mu * w.lam)
    Y = to_dev(ref["A"].astype(np.float32), "f32")
    Xr, Cr = p.empty(p.BH, n_q, n, dtype=torch.float32), p.empty(p.BH, n_q, w.d)
    p.ws.fill_(0xFF)
    csat.csat_recover(p.dims, Y, p.Phi, w.lam, mu, iters, Xr, p.V, Cr, p.ws)
    torch.cuda.synchronize()
    assert_close("X (stage call)", to_np(Xr), ref["X"], TOL["f32"])
    assert_close("C (stage call)", to_np(Cr), ref["C"], TOL["f32"])
    # a NaN, infinities and a huge value in y: what the float products make of them
    Y[0, 0, 0], Y[1, n_q // 2, m - 1], Y[2, n_q - 1, m // 2], Y[3, 0, 0] = float("inf"), float("-inf"), float("nan"), 1e30
    out = []
    for gemm in (0, 1):
        options("gemm", gemm)
        csat.csat_recover(p.dims, Y, p.Phi, w.lam, mu, iters, Xr, p.V, Cr, p.ws)
        torch.cuda.synchronize()
        out.append((Xr.clone(), Cr.clone()))
    for got, old in zip(*out):
        same = torch.equal(got.isnan(), old.isnan()) and torch.equal(got.isinf(), old.isinf())
        assert same
        fine = old.isfinite()
        rows_ok = fine.all(-1) & (old.abs().amax(-1) < 1e20)
        assert_close("finite rows", to_np(got[rows_ok]), to_np(old[rows_ok]), TOL["f32"])


@pytest.mark.parametrize("n_q,n,m", [(40, 128, 64), (33, 224, 96), (70, 65, 20), (20, 160, 128)])
def test_float_decoder_in_lds_leaves_the_range_of_float(n_q, n, m, options):
    """Finite inputs whose iterates overflow, in some rows of a tile from the first residual on and in others later: what
    the float products make of them (sums of one sign, so that the order of a sum does not matter).  -inf after two
    iterations, 0 after three (the threshold takes a NaN to 0), finite again after four."""
    w = _small("f32_overflow", B=1, H=2, n_q=n_q, n=n, d=64, m=m, dtype="f32", lam=0.01)
    rng = np.random.default_rng(n)
    Phi = (rng.uniform(0.5, 1.0, (m, n)) * 1e15).astype(np.float32)
    Q, K, V = gen.make_qkv(w)
    p = _problem(w, Q, K, V, Phi)
    Y = (rng.uniform(0.5, 1.0, (2, n_q, m)) * 1e10).astype(np.float32)
    Y[:, 1::3] *= 1e-30                                        # these rows stay finite for two iterations
    X, C = p.empty(2, n_q, n, dtype=torch.float32), p.empty(2, n_q, w.d)
    for iters in (2, 3, 4, 5):
        out = []
        for gemm in (0, 1):
            options("gemm", gemm)
            p.ws.fill_(0xFF)
            csat.csat_recover(p.dims, to_dev(Y, "f32"), p.Phi, w.lam, 1.0, iters, X, p.V, C, p.ws)
            torch.cuda.synchronize()
            assert csat.csat_profile_decoder_kernel() == (-1 if gemm else 5)
            out.append((to_np(X), to_np(C)))
        (Xg, Cg), (Xo, Co) = out
        if iters == 2:
            assert np.isneginf(Xo[:, 0]).all() and np.isfinite(Xo[:, 1]).all()
        for got, old in ((Xg, Xo), (Cg, Co)):
            assert (np.isnan(got) == np.isnan(old)).all() and (np.isposinf(got) == np.isposinf(old)).all() and (np.isneginf(got) == np.isneginf(old)).all()
            rows_ok = np.isfinite(old).all(-1)
            if rows_ok.any():
                assert_close(f"finite rows, {iters} iterations", got[rows_ok], old[rows_ok], TOL["f32"], slices_axis0=False)


# (rows, m, iterations, in LDS): two or three iterations of more than four tiles per CU go to the products if Phi is more than
# one tile of m
@pytest.mark.parametrize("rows,m,iters,resident", [(32768, 40, 2, True), (32769, 40, 3, False), (32769, 32, 2, True), (32769, 40, 4, True)])
def test_float_decoder_of_many_rows(rows, m, iters, resident):
    n, d = 70, 8
    dims = csat.make_dims(1, 1, rows, n, d, m, "f32")
    Phi = gen.make_phi("gaussian", m, n, seed=5).astype(np.float32)
    mu = _mu(Phi)
    Y = np.random.default_rng(m).standard_normal((rows, m)).astype(np.float32)
    X = torch.empty(rows, n, device=DEV)
    ws = torch.empty(csat.csat_workspace_bytes(dims, iters), dtype=torch.uint8, device=DEV).fill_(0xFF)
    csat.csat_recover(dims, to_dev(Y, "f32"), to_dev(Phi, "f32"), 0.1, mu, iters, X, None, None, ws)
    torch.cuda.synchronize()
    assert csat.csat_profile_decoder_kernel() == (5 if resident else -1)
    at = np.array([0, 31, 32, rows // 2, rows - 2, rows - 1])
    P, x = Phi.astype(np.float64), np.zeros((len(at), n))
    for _ in range(iters):
        u = x + mu * ((Y[at].astype(np.float64) - x @ P.T) @ P)
        x = np.sign(u) * np.maximum(np.abs(u) - mu * 0.1, 0)
    assert_close("X", to_np(X[torch.from_numpy(at).to(DEV)]), x, TOL["f32"], slices_axis0=False)


# widths around the lanes a row gets (four columns each: 1, 2, 4 ... 64), one beyond a wavefront's 256 columns; aligned and not
@pytest.mark.parametrize("dtype,m", [("f32", 3), ("f32", 8), ("f32", 9), ("f32", 33), ("f32", 64), ("f32", 130), ("f32", 257), ("bf16", 20), ("bf16", 63), ("bf16", 300)])
def test_row_packing_widths(dtype, m, options):
    """One iteration without a threshold is X = mu Phi^T y on the packed rows of y and the packed Phi; the workspace holds
    NaN patterns, so a pad that was not written shows."""
    rows, n = 37, max(m, 40) + 1
    w = _small("pack_widths", B=1, H=1, n_q=rows, n=n, d=8, m=m, dtype=dtype, iters=1)
    Q, K, V = gen.make_qkv(w)
    Phi = gen.make_workload_phi(w)
    p = _problem(w, Q, K, V, Phi)
    options("decoder", 1)
    Y = gen.quantize(np.random.default_rng(m).standard_normal((1, rows, m)).astype(np.float32), dtype)
    X = p.empty(1, rows, n, dtype=torch.float32)
    csat.csat_recover(p.dims, to_dev(Y, "f32"), p.Phi, 0.0, 0.5, 1, X, None, None, p.ws)
    torch.cuda.synchronize()
    assert_close("X", to_np(X)[0], 0.5 * (Y[0].astype(np.float64) @ Phi.astype(np.float64)), TOL[dtype], slices_axis0=False)


def test_more_rows_than_wavefronts_fit_a_launch():
    """2^26 rows of eight: a wavefront per row would be more threads than a launch may have."""
    rows, n, m, d = (1 << 26) + 70, 9, 8, 8
    free, _ = torch.cuda.mem_get_info()
    if free < 40 << 30:
        pytest.skip("needs 40 GB")
    dims = csat.make_dims(1, 1, rows, n, d, m, "f32")
    Phi = gen.make_phi("gaussian", m, n, seed=3)
    V = np.random.default_rng(4).standard_normal((n, d)).astype(np.float32)
    Y = torch.randn(rows, m, device=DEV)
    C = torch.empty(rows, d, device=DEV)
    ws = torch.empty(csat.csat_workspace_bytes(dims, 1), dtype=torch.uint8, device=DEV)
    csat.csat_recover(dims, Y, to_dev(Phi, "f32"), 0.0, 0.5, 1, None, to_dev(V, "f32"), C, ws)
    torch.cuda.synchronize()
    at = torch.tensor([0, 1, rows // 2, rows - 65, rows - 1], device=DEV)
    y = to_np(Y[at])
    assert_close("C", to_np(C[at]), 0.5 * (y @ Phi.astype(np.float64)) @ V.astype(np.float64), TOL["f32"], slices_axis0=False)


# (n_q, n, m, iterations): the fewest chunks this decoder gets, one to thirteen tiles of m (odd and even), odd and even
# chunk counts modulo its ring of five, a ragged last chunk and row tile, one and two iterations
SHARED_TILE_CASES = [(33, 513, 20, 4), (40, 544, 64, 3), (64, 577, 90, 1), (31, 700, 128, 2), (70, 609, 160, 5), (32, 416, 416, 3), (5, 500, 390, 4),
                     (97, 900, 217, 3), (160, 1600, 392, 2), (33, 353, 300, 6), (20, 330, 330, 2), (45, 1333, 352, 3)]


@pytest.mark.parametrize("tiles,iters,kernel", [(130, 3, 2), (130, 4, 6), (128, 2, 6)])
def test_few_iterations_over_an_iterate_beyond_the_infinity_cache(tiles, iters, kernel, options):
    """Two or three iterations over more than 256 MB of iterate stay with one wavefront per 32-row tile; same bits."""
    rows, n, m, d = 32 * tiles, 16384, 40, 64
    dims = csat.make_dims(1, 1, rows, n, d, m, "bf16")
    Phi = gen.quantize(gen.make_phi("gaussian", m, n, seed=9).astype(np.float32), "bf16")
    rng = np.random.default_rng(tiles)
    Y = to_dev(rng.standard_normal((rows, m)).astype(np.float32), "f32")
    V = to_dev(gen.quantize(rng.standard_normal((n, d)).astype(np.float32), "bf16"), "bf16")
    ws = torch.empty(csat.csat_workspace_bytes(dims, iters), dtype=torch.uint8, device=DEV).fill_(0xFF)
    C, C1 = torch.empty(rows, d, dtype=torch.bfloat16, device=DEV), torch.empty(rows, d, dtype=torch.bfloat16, device=DEV)
    csat.csat_recover(dims, Y, to_dev(Phi, "bf16"), 0.05, 0.002, iters, None, V, C, ws)
    assert csat.csat_profile_decoder_kernel() == kernel
    assert csat.csat_decoder_status(ws) == 0
    options("fused_thin", 1)
    csat.csat_recover(dims, Y, to_dev(Phi, "bf16"), 0.05, 0.002, iters, None, V, C1, ws)
    torch.cuda.synchronize()
    assert csat.csat_profile_decoder_kernel() in (0, 1)
    assert C.isfinite().all() and C.abs().max() > 0
    assert torch.equal(C, C1)


@pytest.mark.parametrize("n_q,n,m,iters", SHARED_TILE_CASES)
def test_decoder_with_a_tile_shared_by_eight_wavefronts(n_q, n, m, iters, options):
    """Launches with few rows and a Phi too large for LDS: the bits of the 128-row decoder, and the oracle."""
    w = _small("shared_tile", B=2, H=3, n_q=n_q, n=n, d=64, m=m, dtype="bf16", iters=iters, lam=0.002)
    Q, K, V = gen.make_qkv(w)
    Phi = gen.make_workload_phi(w)
    mu = _mu(Phi)
    p = _problem(w, Q, K, V, Phi)
    C, _, X = p.forward(w.lam, mu, iters)
    assert csat.csat_profile_decoder_kernel() == 6
    assert csat.csat_decoder_status(p.ws) == 0
    ref = orc.forward(Q, K, V, Phi, w.lam, mu, iters)
    assert_close("X", to_np(X), ref["X"], TOL["bf16"])
    assert_close("C", to_np(C), ref["C"], TOL["bf16"])
    options("fused_thin", 1)
    options("synthesis", 1)
    p.ws.fill_(0xFF)
    C1, _, X1 = p.forward(w.lam, mu, iters)
    assert csat.csat_profile_decoder_kernel() in (0, 1, 3, 4)
    same = torch.equal(X, X1) and torch.equal(C, C1)
    assert same


# (n_q, n, m, iterations, workgroups per tile): one tile and 96, one to thirteen tiles of m (odd and even), shares of unequal length,
# ragged last chunk and row tile, the fewest iterations and more
MEMBER_CASES = [(5, 1600, 392, 8, 5), (33, 1571, 197, 8, 5), (70, 3000, 130, 6, 8), (40, 4500, 20, 7, 9), (200, 1333, 352, 6, 4), (512, 1000, 416, 8, 2),
                (31, 2000, 64, 5, 7), (3, 8192, 90, 4, 13), (100, 1800, 300, 5, 6), (20, 16384, 20, 5, 16),
                # the lines: four iterations; 20 us of a call to be saved; two workgroups for every CU's one tile
                (5, 1600, 392, 4, 5), (5, 1600, 392, 3, 1), (300, 900, 200, 8, 3), (300, 900, 200, 7, 1), (682, 1600, 392, 8, 2), (683, 1600, 392, 8, 1)]
SHARED_MEMBER_CASES = [c[:4] for c in MEMBER_CASES if c[4] > 1]


@pytest.mark.parametrize("n_q,n,m,iters,members", MEMBER_CASES)
def test_decoder_with_a_tile_shared_by_workgroups(n_q, n, m, iters, members):
    """Fewer row tiles than CUs: several workgroups share a tile and exchange their parts of the residual; against the oracle, and
    the same bits in every call."""
    w = _small("shared_members", B=2, H=3, n_q=n_q, n=n, d=64, m=m, dtype="bf16", iters=iters, lam=0.002)
    Q, K, V = gen.make_qkv(w)
    Phi = gen.make_workload_phi(w)
    mu = _mu(Phi)
    p = _problem(w, Q, K, V, Phi)
    C, _, X = p.forward(w.lam, mu, iters)
    assert csat.csat_profile_decoder_kernel() == 6 and csat.csat_profile_launch_form("decoder_members") == members
    assert csat.csat_decoder_status(p.ws) == 0
    ref = orc.forward(Q, K, V, Phi, w.lam, mu, iters)
    assert_close("X", to_np(X), ref["X"], TOL["bf16"])
    assert_close("C", to_np(C), ref["C"], TOL["bf16"])
    p.ws.fill_(0xFF)
    C1, _, X1 = p.forward(w.lam, mu, iters)
    assert torch.equal(X, X1) and torch.equal(C, C1)


@pytest.mark.parametrize("n_q,n,m,iters", SHARED_MEMBER_CASES)
def test_workgroups_that_share_a_tile_hold_the_same_residual(n_q, n, m, iters):
    """The second half of Phi's columns repeats the first: each pair meets the same residual in shares of different workgroups,
    so the iterate's halves agree bit for bit."""
    h, rows = n // 2, 6 * n_q
    dims = csat.make_dims(1, 6, n_q, n, 64, m, "bf16")
    g = torch.Generator(device=DEV).manual_seed(n)
    half = torch.randn(m, h, generator=g, device=DEV) / n ** 0.5
    Phi = torch.cat([half, half, torch.zeros(m, n - 2 * h, device=DEV)], 1).bfloat16()
    Y = torch.randn(rows, m, generator=g, device=DEV)
    ws = torch.empty(csat.csat_workspace_bytes(dims, iters), dtype=torch.uint8, device=DEV).fill_(0xFF)
    X = torch.empty(rows, n, device=DEV)
    csat.csat_recover(dims, Y, Phi, (m / n) ** 0.5, 0.2, iters, X, None, None, ws)      # (lambda: the spread of Phi^T y)
    torch.cuda.synchronize()
    assert csat.csat_profile_launch_form("decoder_members") > 1 and csat.csat_decoder_status(ws) == 0
    assert X.isfinite().all() and 0.02 < float((X != 0).float().mean()) < 0.98
    assert torch.equal(X[:, :h], X[:, h:2 * h])


@pytest.mark.parametrize("n_q,n,m,iters,members", [(512, 1000, 416, 8, 2), (5, 1600, 392, 8, 5), (20, 16384, 20, 5, 16)])
def test_a_wait_of_workgroups_that_share_a_tile_runs_out(n_q, n, m, iters, members, options):
    """Two, five and sixteen workgroups to a tile.  Their waits for each other are bounded: one that runs out is reported and the
    outputs hold NaN (forced from the host: the error record set before the launch; a limit of no polls, under which whoever is
    first to an exchange gives up and goes on), every kernel ends normally, and the next call on the workspace is clean."""
    w = _small("members_give_up", B=2, H=3, n_q=n_q, n=n, d=64, m=m, dtype="bf16", iters=iters, lam=0.002)
    Q, K, V = gen.make_qkv(w)
    Phi = gen.make_workload_phi(w)
    mu = _mu(Phi)
    p = _problem(w, Q, K, V, Phi)
    C0, _, X0 = p.forward(w.lam, mu, iters)
    assert csat.csat_profile_launch_form("decoder_members") == members and csat.csat_decoder_status(p.ws) == 0
    for option, value, fails in (("inject_decoder_error", 1, True), ("fused_spin_limit", -1, True), ("fused_spin_limit", 1 << 22, False)):
        options(option, value)
        C, _, X = p.forward(w.lam, mu, iters)
        assert csat.csat_profile_launch_form("decoder_members") == members
        assert csat.csat_decoder_status(p.ws) == (csat.CSAT_ERR_TIMEOUT if fails else 0)
        options(option, 0)
        if fails:
            assert torch.isnan(X).all() and torch.isnan(C.float()).all()
            C, _, X = p.forward(w.lam, mu, iters)
            assert csat.csat_decoder_status(p.ws) == 0
        assert torch.equal(C, C0) and torch.equal(X, X0)


def test_tiles_shared_by_workgroups_on_two_streams_and_in_a_graph():
    """Two calls at once, together more workgroups than CUs, so that workgroups of one tile may start apart; then one of them as replays
    of a captured graph, whose counter and flags its own kernels clear: the bits of the call alone each time."""
    problems = []
    for n_q, n, m, iters, members in ((512, 1000, 416, 8, 2), (200, 1333, 352, 8, 4)):
        w = _small("members_streams", B=2, H=3, n_q=n_q, n=n, d=64, m=m, dtype="bf16", iters=iters, lam=0.002)
        Q, K, V = gen.make_qkv(w)
        Phi = gen.make_workload_phi(w)
        p = _problem(w, Q, K, V, Phi)
        args = (p.dims, p.Q, p.K, p.V, p.Phi, w.lam, _mu(Phi), iters)
        C0, _, X0 = p.forward(w.lam, args[6], iters)
        assert csat.csat_profile_launch_form("decoder_members") == members
        problems.append((p, args, C0, X0, torch.empty_like(C0), torch.empty_like(X0), torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(5):
        for p, args, _, _, C, X, stream in problems:
            with torch.cuda.stream(stream):
                csat.csat_forward(*args, C, None, X, p.ws)
    torch.cuda.synchronize()
    for p, args, C0, X0, C, X, stream in problems:
        assert csat.csat_decoder_status(p.ws) == 0
        assert torch.equal(C, C0) and torch.equal(X, X0)
    p, args, C0, X0, C, X, stream = problems[0]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        csat.csat_forward(*args, C, None, X, p.ws)
    for _ in range(3):
        C.zero_(), X.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert csat.csat_decoder_status(p.ws) == 0 and torch.equal(C, C0) and torch.equal(X, X0)
        p.forward(args[5], args[6], args[7] - 1)               # eager work on the same workspace in between


# (type, heads, n_q, n, d, m, forms of the small-tile products in measurement, attention and synthesis): contractions of less than a
# step, one, eight and nine steps, and with a ragged last one; tiles of one row and column, whole ones and one more; both
# tile sizes in bf16; the output product where it is one; the line (96 of the 128-wide tiles in float, 64 in bf16)
FEW_TILE_CASES = [("f32", 1, 1, 70, 8, 5, 1, 0, 5), ("f32", 2, 33, 256, 64, 64, 1, 0, 5), ("f32", 1, 32, 289, 40, 31, 1, 0, 5), ("f32", 3, 65, 1571, 80, 97, 1, 1, 5),
                  ("f32", 1, 100, 4099, 128, 300, 1, 1, 5), ("f32", 48, 128, 300, 64, 96, 1, 0, 5), ("f32", 49, 256, 300, 64, 96, 0, 0, 0),
                  ("bf16", 1, 1, 67, 8, 5, 1, 0, 1), ("bf16", 2, 33, 512, 80, 64, 1, 0, 1), ("bf16", 3, 64, 577, 32, 33, 1, 0, 1), ("bf16", 10, 70, 1571, 80, 197, 1, 1, 1),
                  ("bf16", 4, 40, 2050, 96, 1000, 2, 1, 1), ("bf16", 32, 128, 300, 80, 96, 2, 0, 1), ("bf16", 33, 256, 300, 80, 96, 0, 0, 0)]


@pytest.mark.parametrize("dtype,heads,n_q,n,d,m,measurement,attention,synthesis", FEW_TILE_CASES)
def test_products_of_few_tiles(dtype, heads, n_q, n, d, m, measurement, attention, synthesis, options):
    """Measurement, output product and synthesis whose tiles would leave most CUs idle, against float64 on the same operands; the
    synthesis also where operands are infinite, NaN or tiny: finite where the 128-wide kernels' result is."""
    rng = np.random.default_rng(n)
    q = lambda *s: gen.quantize(rng.standard_normal(s).astype(np.float32), dtype)    # noqa: E731
    Phi = gen.quantize((rng.standard_normal((m, n)) / np.sqrt(m)).astype(np.float32), dtype)
    Q, K, V = q(heads, n_q, d), q(heads, n, d), q(heads, n, d)
    dims = csat.make_dims(1, heads, n_q, n, d, m, dtype)
    ws = torch.empty(csat.csat_workspace_bytes(dims, 1), dtype=torch.uint8, device=DEV).fill_(0xFF)
    empty = lambda *s: torch.empty(*s, dtype=to_dev(Q, dtype).dtype, device=DEV)     # noqa: E731
    Kc, Vc, Z, C = empty(heads, m, d), empty(heads, m, d), empty(heads, n_q, d), empty(heads, n_q, d)
    A, X = torch.empty(heads, n_q, m, device=DEV), torch.empty(heads, n_q, n, device=DEV)
    csat.csat_measure(dims, to_dev(Phi, dtype), to_dev(K, dtype), to_dev(V, dtype), Kc, Vc, ws)
    assert csat.csat_profile_launch_form("small_tiles") == measurement
    P64, rel = Phi.astype(np.float64), 2e-6 if dtype == "f32" else 4e-3          # 24 bits over K terms; one rounding to bf16
    assert_close("K~", to_np(Kc), P64 @ K, rel)
    assert_close("V~", to_np(Vc), P64 @ V, rel)
    csat.csat_compressed_attention(dims, to_dev(Q, dtype), Kc, Vc, A, Z, ws)
    assert csat.csat_profile_launch_form("small_tiles") == attention
    torch.cuda.synchronize()
    assert_close("Z", to_np(Z), to_np(A).astype(np.float64) @ to_np(Vc), 2 * rel)      # (bf16: A~ rounded once too)
    # 1e-33: sums below 2^-90, where the split products are not used, and well above the smallest normal float (at 1e-37 they
    # are subnormal, 1.4e-45 apart, which is up to 7.6e-6 of them)
    for special in (None, np.inf, np.nan, 1e-33):
        Vs = V.copy()
        if special is not None:
            Vs[0, n // 2, d // 2] = special
        if special == 1e-33:
            Vs[0] *= np.float32(1e-33)
        got = []
        for gemm in (0, 1):
            options("gemm", gemm)
            csat.csat_recover(dims, A, to_dev(Phi, dtype), 0.0, 0.01, 1, X, to_dev(Vs, dtype), C, ws)
            assert csat.csat_profile_launch_form("small_tiles") == (0 if gemm else synthesis)
            torch.cuda.synchronize()
            got.append(to_np(C).astype(np.float64))
        options("gemm", 0)
        assert (np.isnan(got[0]) == np.isnan(got[1])).all() and (np.isinf(got[0]) == np.isinf(got[1])).all()
        if special is None or special == 1e-33:
            assert_close("C", got[0], to_np(X).astype(np.float64) @ Vs, 2 * rel)


@pytest.mark.parametrize("heads,n_q,n,d,m", [(1, 1, 8, 8, 4), (2, 33, 32, 64, 16), (8, 300, 31, 128, 20), (96, 128, 32, 64, 32)])
def test_synthesis_over_one_step_keeps_exact_products(heads, n_q, n, d, m, options):
    """Float C = X V over at most 32 columns and 128 features, few tiles: products of float, not of its bf16 parts, so the bits of
    the 128-wide kernel (one chain there and here), on dense rows and on rows of one coefficient."""
    rng = np.random.default_rng(n_q)
    dims = csat.make_dims(1, heads, n_q, n, d, m, "f32")
    Phi = torch.eye(m, n, device=DEV)
    V = to_dev(rng.standard_normal((heads, n, d)).astype(np.float32), "f32")
    ws = torch.empty(csat.csat_workspace_bytes(dims, 1), dtype=torch.uint8, device=DEV).fill_(0xFF)
    for sparse in (False, True):
        Y = rng.standard_normal((heads, n_q, m)).astype(np.float32)
        if sparse:
            Y *= np.arange(m) == rng.integers(0, m, (heads, n_q, 1))
        out = []
        for gemm in (0, 1):
            options("gemm", gemm)
            X, C = torch.empty(heads, n_q, n, device=DEV), torch.empty(heads, n_q, d, device=DEV)
            csat.csat_recover(dims, to_dev(Y, "f32"), Phi, 0.0, 1.0, 1, X, V, C, ws)
            torch.cuda.synchronize()
            out.append((X, C))
        assert torch.equal(out[0][0], to_dev(np.pad(Y, ((0, 0), (0, 0), (0, n - m))), "f32"))
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("heads,n_q,n,d", [(2, 78, 271, 8), (1, 135, 358, 128), (8, 216, 700, 96)])
def test_synthesis_of_sparse_rows_rounds_once(heads, n_q, n, d):
    """Float C = X V on small tiles, three coefficients per row in K steps of different wavefronts: their first products (8 bits each) sum
    exactly but for wide spreads of their exponents, so the result is rounded once: at most 2^-24 / sqrt(3) of it in the 2-norm (as the
    kernel with one chain per sum: 2.7e-8; with every wavefront's sum rounded before they meet it was 4.2e-8 to 5.2e-8)."""
    g = torch.Generator(device=DEV).manual_seed(n)
    dims = csat.make_dims(1, heads, n_q, n, d, n, "f32")
    at = torch.rand(heads, n_q, n, generator=g, device=DEV).topk(3, -1).indices
    Y = torch.zeros(heads, n_q, n, device=DEV).scatter_(-1, at, torch.randn(heads, n_q, 3, generator=g, device=DEV))
    V = torch.randn(heads, n, d, generator=g, device=DEV)
    ws = torch.empty(csat.csat_workspace_bytes(dims, 1), dtype=torch.uint8, device=DEV).fill_(0xFF)
    X, C = torch.empty(heads, n_q, n, device=DEV), torch.empty(heads, n_q, d, device=DEV)
    csat.csat_recover(dims, Y, torch.eye(n, device=DEV), 0.0, 1.0, 1, X, V, C, ws)
    assert csat.csat_profile_launch_form("small_tiles") == 5
    torch.cuda.synchronize()
    assert torch.equal(X, Y)
    ref = to_np(Y).astype(np.float64) @ to_np(V).astype(np.float64)
    assert np.linalg.norm(to_np(C) - ref) <= 2.0 ** -24 / np.sqrt(3) * np.linalg.norm(ref)


# (type, heads, n_q, m, d, wavefronts per workgroup): eight, four and two (more workgroups than CUs with fewer; four at most); K~ in LDS as a
# whole and in parts; 0: the three kernels
WAVE_CASES = [("f32", 600, 70, 40, 32, 8), ("f32", 140, 200, 100, 64, 8), ("f32", 192, 120, 73, 64, 4), ("f32", 3, 200, 100, 64, 2),
              ("f32", 70, 250, 390, 64, 4), ("f32", 40, 250, 390, 64, 2), ("bf16", 600, 70, 40, 80, 8),
              ("bf16", 300, 250, 200, 80, 8), ("bf16", 5, 250, 200, 80, 2), ("bf16", 4, 300, 1024, 80, 2), ("bf16", 3, 33, 600, 96, 0)]


@pytest.mark.parametrize("dtype,heads,n_q,m,d,waves", WAVE_CASES)
def test_attention_at_every_number_of_wavefronts(dtype, heads, n_q, m, d, waves):
    """The one-kernel attention against float64 on the same operands, at the workgroup sizes that the number of row tiles picks."""
    rng = np.random.default_rng(heads)
    q = lambda *s: gen.quantize(rng.standard_normal(s).astype(np.float32), dtype)    # noqa: E731
    Q, Kc, Vc = q(heads, n_q, d), q(heads, m, d), q(heads, m, d)
    dims = csat.make_dims(1, heads, n_q, max(m, n_q), d, m, dtype)
    ws = torch.empty(csat.csat_workspace_bytes(dims, 0), dtype=torch.uint8, device=DEV).fill_(0xFF)
    A, Z = torch.empty(heads, n_q, m, device=DEV), torch.empty(heads, n_q, d, dtype=to_dev(Q, dtype).dtype, device=DEV)
    csat.csat_compressed_attention(dims, to_dev(Q, dtype), to_dev(Kc, dtype), to_dev(Vc, dtype), A, Z, ws)
    assert csat.csat_profile_launch_form("attention_waves") == waves
    torch.cuda.synchronize()
    want_a, want_z = orc.compressed_attention(Q, Kc, Vc)
    # scores of |s| <= 40 to 2^-24 each way, then exp2 and the sum; Z in bf16: the weights and the result rounded once
    assert_close("A", to_np(A), want_a, 2e-5)
    assert_close("Z", to_np(Z), want_z, 2e-5 if dtype == "f32" else 1e-2)


@pytest.mark.parametrize("rows,n,m,iters", [(33000, 320, 160, 3), (33001, 300, 136, 2), (13000, 1600, 200, 3), (13007, 1530, 130, 1)])
def test_unrolled_decoder_on_the_wider_tile(rows, n, m, iters):
    """Row and column counts whose layers run 256 x 320 tiles: the bits that slices of the rows (too few for it) get on 256 x 256."""
    rng = np.random.default_rng(rows)
    bf = lambda *s: to_dev(gen.quantize(rng.standard_normal(s).astype(np.float32), "bf16"), "bf16")     # noqa: E731
    g = torch.Generator(device=DEV).manual_seed(rows)
    Y = torch.randn(1, rows, m, generator=g, device=DEV)
    V, B = bf(1, n, 64), (bf(n, m) * 0.05)
    S = (torch.eye(n, device=DEV) + 0.3 / n ** 0.5 * torch.randn(n, n, generator=g, device=DEV)).bfloat16()
    thetas = [0.2 + 0.1 * t for t in range(iters)]

    def decode(y):
        r = y.shape[1]
        dims = csat.make_dims(1, 1, r, n, 64, m, "bf16")
        ws = torch.empty(csat.csat_lista_workspace_bytes(dims, iters), dtype=torch.uint8, device=DEV).fill_(0xFF)
        X, C = torch.empty(1, r, n, device=DEV), torch.empty(1, r, 64, dtype=torch.bfloat16, device=DEV)
        csat.csat_recover_lista(dims, y.clone(), S, B, thetas, X, V, C, ws)
        assert csat.csat_profile_launch_form("lista_tile") == (320 if r == rows else 256)
        torch.cuda.synchronize()
        return X, C

    X, C = decode(Y)
    assert X.isfinite().all() and 0.05 < float((X != 0).float().mean()) < 0.95
    for r0 in (0, 7936, rows - 300):
        Xs, Cs = decode(Y[:, r0:r0 + 300])
        assert torch.equal(X[:, r0:r0 + 300], Xs) and torch.equal(C[:, r0:r0 + 300], Cs)


# (n_q, n, m, picks): a ragged last group of columns, more picks than a batch of eight, every column picked in the end (m = n = picks)
PICK_CASES = [(90, 128, 100, 5), (100, 130, 129, 9), (128, 32, 32, 32), (90, 300, 64, 17), (256, 513, 40, 3), (87, 257, 20, 20),
              (2730, 128, 20, 5), (2731, 128, 20, 5), (1365, 257, 30, 9), (1366, 512, 30, 9), (90, 512, 40, 3)]


@pytest.mark.parametrize("n_q,n,m,picks", PICK_CASES)
def test_matching_pursuit_picks_in_the_product(n_q, n, m, picks, options):
    """bf16: the largest correlation is found where the correlations are formed.  The picks of the search over stored correlations
    (forced; rows whose picks agree are compared in full and few may not), no column twice, coefficients consistent."""
    w = _small("omp_picks", B=1, H=3, n_q=n_q, n=n, d=64, m=m, dtype="bf16")
    Q, K, V = gen.make_qkv(w)
    Phi = gen.make_workload_phi(w)
    p = _problem(w, Q, K, V, Phi)
    rng = np.random.default_rng(n)
    Y = to_dev(rng.standard_normal((3, n_q, m)).astype(np.float32), "f32")
    ws = torch.empty(csat.csat_omp_workspace_bytes(p.dims, picks), dtype=torch.uint8, device=DEV)
    out = []
    for gemm in (0, 1):
        options("gemm", gemm)
        ws.fill_(0xFF)
        X, S, C = p.empty(3, n_q, n, dtype=torch.float32), p.empty(3, n_q, picks, dtype=torch.int32), p.empty(3, n_q, w.d)
        csat.csat_recover_omp(p.dims, Y, p.Phi, picks, X, S, p.V, C, ws)
        torch.cuda.synchronize()
        out.append([to_np(t) for t in (X, S, C)])
    (X, S, C), (X1, S1, C1) = out
    assert (S >= 0).all() and (S < n).all() and (np.diff(np.sort(S, -1), axis=-1) > 0).all()
    agree = (S == S1).all(-1)
    assert agree.mean() > 0.9
    assert_close("X", X[agree], X1[agree], TOL["f32"])
    assert_close("C", C[agree], C1[agree], TOL["bf16"])
    assert_close("C = X V", C, X.astype(np.float64) @ V.reshape(3, n, w.d).astype(np.float64), TOL["bf16"])


# (rows, n, m, picks): 1 to 16 slabs of 64 rows of Phi and their chunks per step, rings of two and three steps, four and eight
# wavefronts; whole row blocks (rows past 256 of them) with and without a cut remainder; 8, 9, 16 and 17 picks; a chunk of one column
PICK_KERNEL_CASES = [(33, 129, 64, 8), (300, 97, 65, 9), (40, 193, 192, 16), (70, 255, 250, 17), (257, 353, 300, 3), (90, 450, 448, 8),
                     (130, 545, 512, 4), (90, 640, 600, 9), (20, 833, 832, 2), (150, 900, 890, 3), (60, 1056, 1024, 10), (65600, 200, 150, 2),
                     (131072, 65, 40, 2), (131200, 33, 8, 3)]


# (rows, n, m, picks): row blocks that are fewer than the XCDs or not a multiple of them, more candidates than lanes, four and eight
# wavefronts
FEW_ROW_PICK_CASES = [(1, 16384, 64, 3), (70, 16384, 130, 2), (300, 8192, 512, 3), (500, 9000, 576, 2), (130, 5000, 1000, 3), (1100, 4096, 900, 2),
                      (2304, 4100, 200, 2), (4600, 2048, 40, 2)]


@pytest.mark.parametrize("rows,n,m,picks", FEW_ROW_PICK_CASES)
def test_matching_pursuit_shares_the_columns_over_the_chip(rows, n, m, picks, options):
    """Few row blocks: as many shares of the columns as give most CUs one, and the picks of the search over stored correlations."""
    blocks = -(-rows // (256 if m <= 512 else 128))
    _pick_forms_agree(rows, n, m, picks, options, lambda: csat.csat_profile_launch_form("omp_shares") * blocks >= 128)


# (rows, n, m, picks): m > 512 and enough rows and columns for rounds of 256 x 256 tiles; ragged tiles and last 128 columns, 8, 9 and 17
# picks, more candidates than lanes
TILE_PICK_CASES = [(1024, 16384, 640, 3), (1021, 16001, 577, 2), (2045, 8180, 1000, 8), (4090, 4090, 830, 9), (16400, 2049, 700, 17), (4097, 4500, 1024, 2)]


@pytest.mark.parametrize("rows,n,m,picks", TILE_PICK_CASES)
def test_matching_pursuit_picks_on_large_tiles(rows, n, m, picks, options):
    """bf16, long columns and whole rounds of tiles: the pick in the large-tile product, with the picks, coefficients and output of the
    search over stored correlations."""
    _pick_forms_agree(rows, n, m, picks, options, lambda: csat.csat_profile_launch_form("omp_pick") == 3)


@pytest.mark.parametrize("rows,n,m,picks", PICK_KERNEL_CASES)
def test_matching_pursuit_picks_while_the_columns_pass(rows, n, m, picks, options):
    """bf16: each row's largest correlation is kept while the columns of Phi pass.  The same sums in the same order as the
    product with stored correlations and their search (forced), so the same picks, coefficients and output."""
    _pick_forms_agree(rows, n, m, picks, options, lambda: csat.csat_profile_launch_form("omp_pick") == 2)


def _pick_forms_agree(rows, n, m, picks, options, form):
    d = 64
    dims = csat.make_dims(1, 1, rows, n, d, m, "bf16")
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    Phi = (torch.randn(m, n, generator=g, device=DEV) / m ** 0.5).bfloat16()
    V = torch.randn(n, d, generator=g, device=DEV).bfloat16()
    Y = torch.randn(rows, m, generator=g, device=DEV)
    ws = torch.empty(csat.csat_omp_workspace_bytes(dims, picks), dtype=torch.uint8, device=DEV)
    out = []
    for gemm in (0, 1):
        options("gemm", gemm)
        ws.fill_(0xFF)
        X, C = torch.empty(rows, n, device=DEV), torch.empty(rows, d, dtype=torch.bfloat16, device=DEV)
        S = torch.empty(rows, picks, dtype=torch.int32, device=DEV)
        csat.csat_recover_omp(dims, Y, Phi, picks, X, S, V, C, ws)
        assert form() == (gemm == 0)
        torch.cuda.synchronize()
        out.append((S, X, C))
    S, X, C = out[0]
    assert (S >= 0).all() and (S < n).all() and (S.sort(-1).values.diff(dim=-1) > 0).all()
    assert X.isfinite().all() and (X != 0).any()
    for a, b in zip(*out):
        assert torch.equal(a, b)


# (type, rows, few, n, m, picks): one to sixteen values of an m-vector per lane, up to eight picks and beyond
REFIT_CASES = [("f32", 900, 40, 700, 60, 8), ("f32", 1500, 90, 900, 300, 9), ("f32", 700, 100, 1500, 700, 4), ("bf16", 700, 20, 700, 64, 8), ("bf16", 2000, 60, 1100, 128, 6),
               ("bf16", 1000, 30, 1000, 190, 4), ("bf16", 3000, 200, 16384, 1000, 2)]


@pytest.mark.parametrize("dtype,rows,few,n,m,picks", REFIT_CASES)
def test_matching_pursuit_few_rows_store_their_vectors(dtype, rows, few, n, m, picks):
    """Few rows of many columns: the orthonormal vectors stored, Phi's columns not packed; the bits that the same rows get among
    more, whose vectors are formed again."""
    t = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    g = torch.Generator(device=DEV).manual_seed(n)
    Phi = (torch.randn(m, n, generator=g, device=DEV) / m ** 0.5).to(t)
    V = torch.randn(n, 64, generator=g, device=DEV).to(t)
    Y = torch.randn(rows, m, generator=g, device=DEV)

    def decode(y, stored):
        r = y.shape[0]
        dims = csat.make_dims(1, 1, r, n, 64, m, dtype)
        ws = torch.empty(csat.csat_omp_workspace_bytes(dims, picks), dtype=torch.uint8, device=DEV).fill_(0xFF)
        X, C, S = torch.empty(r, n, device=DEV), torch.empty(r, 64, dtype=t, device=DEV), torch.empty(r, picks, dtype=torch.int32, device=DEV)
        csat.csat_recover_omp(dims, y, Phi, picks, X, S, V, C, ws)
        assert csat.csat_profile_launch_form("omp_refit") == (2 if stored else 1)
        torch.cuda.synchronize()
        return X, C, S

    whole = decode(Y, False)
    assert whole[0].isfinite().all() and (whole[2].sort(-1).values.diff(dim=-1) > 0).all()
    for a, b in zip(whole, decode(Y[rows - few:].contiguous(), True)):
        assert torch.equal(a[rows - few:], b)


@pytest.mark.parametrize("dtype,picks", [("f32", 1), ("f32", 5), ("f32", 12), ("bf16", 4), ("bf16", 12)])
def test_matching_pursuit_sums_alike_in_every_lane(dtype, picks):
    """m = 64, one value of an m-vector per lane: with the two halves of the measurements exchanged, every sum of the refit has the same
    two operands at its first step and the same ones after, so rows that pick the same columns get the same coefficients, bit for bit."""
    rows, n, m = 2000, 300, 64
    t = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    g = torch.Generator(device=DEV).manual_seed(picks)
    Phi = (torch.randn(m, n, generator=g, device=DEV) / m ** 0.5).to(t)
    Y = torch.randn(rows, m, generator=g, device=DEV)
    dims = csat.make_dims(1, 1, rows, n, 64, m, dtype)
    out = []
    for shift in (0, 32):
        ws = torch.empty(csat.csat_omp_workspace_bytes(dims, picks), dtype=torch.uint8, device=DEV).fill_(0xFF)
        X, S = torch.empty(rows, n, device=DEV), torch.empty(rows, picks, dtype=torch.int32, device=DEV)
        csat.csat_recover_omp(dims, Y.roll(shift, 1).contiguous(), Phi.roll(shift, 0).contiguous(), picks, X, S, None, None, ws)
        torch.cuda.synchronize()
        out.append((X, S))
    (X, S), (X1, S1) = out
    same = (S == S1).all(-1)             # (correlations are summed in another order: near-ties may go the other way)
    assert float(same.float().mean()) > 0.98
    assert torch.equal(X[same], X1[same])


# (n, m, iterations): every length of the register-resident transforms, n at and off multiples of the thread count, just
# above half the length and equal to it, one and two iterations
HADAMARD_CASES = [(257, 30, 3), (512, 512, 2), (513, 100, 1), (1000, 64, 4), (1088, 200, 3), (2048, 300, 2), (2049, 90, 3), (4100, 1000, 2), (8200, 40, 2)]


@pytest.mark.parametrize("n,m,iters", HADAMARD_CASES)
def test_transform_decoder_lengths(n, m, iters, options):
    """The transform-based decoder with the iterate in registers against the one in LDS (same transforms, another order
    of their stages) and, where the explicit matrix is small, the oracle."""
    w = _small("hadamard_lengths", B=1, H=2, n_q=9, n=n, d=64, m=m, dtype="f32", iters=iters, lam=0.002)
    Q, K, V = gen.make_qkv(w)
    rows, signs = _selection(m, n)
    p = _problem(w, Q, K, V, np.zeros((m, n), np.float32))
    Y = np.random.default_rng(m).standard_normal((2, 9, m)).astype(np.float32) * 0.1
    N = len(signs)
    mu = m / N
    out = []
    for choice in (0, 1):
        options("hadamard", choice)
        p.ws.fill_(0xFF)
        X, C = p.empty(2, 9, n, dtype=torch.float32), p.empty(2, 9, w.d)
        csat.csat_recover_hadamard(p.dims, to_dev(Y, "f32"), to_dev_raw(rows), to_dev_raw(signs), w.lam, mu, iters, X, p.V, C, p.ws)
        torch.cuda.synchronize()
        out.append((to_np(X), to_np(C)))
    for name, a, b in zip("XC", *out):
        assert_close(name, a, b, TOL["f32"])
    if N <= 2048:
        i, j = rows[:, None].astype(np.int64), np.arange(n)[None, :]
        bits = np.zeros(i.shape[:1] + j.shape[1:], np.int64)
        both = i & j
        while both.any():
            bits ^= both & 1
            both >>= 1
        P = (1 - 2 * bits) * signs[:n] / np.sqrt(m)
        x = np.zeros((18, n))
        for _ in range(iters):
            u = x + mu * ((Y.reshape(18, m) - x @ P.T) @ P)
            x = np.sign(u) * np.maximum(np.abs(u) - mu * w.lam, 0)
        assert_close("X against float64", out[0][0].reshape(18, n), x, TOL["f32"])


def _selection(m, n):
    N = 1 << (n - 1).bit_length()
    rng = np.random.default_rng(m + n)
    return np.sort(rng.permutation(N)[:m]).astype(np.int32), (rng.integers(0, 2, N) * 2 - 1).astype(np.int8)


def to_dev_raw(a):
    return torch.from_numpy(a).to(DEV)


# (heads, n_q, n, m, d, layers): rows of 64 R columns for the instances' R and one more, a last group of rows that is not whole, several
# heads to a group, two layers, d that is not the synthesis kernel's
LISTA_SUPPORT_CASES = [(3, 87, 256, 130, 64, 4), (1, 259, 257, 136, 64, 2), (7, 75, 512, 200, 64, 5), (2, 391, 770, 160, 128, 3), (1, 1026, 1025, 200, 64, 3),
                       (2, 833, 1600, 392, 64, 6), (5, 330, 1639, 150, 80, 3), (3, 701, 2049, 256, 64, 3), (1, 2561, 2561, 136, 64, 2), (1, 4101, 4096, 130, 64, 2)]


@pytest.mark.parametrize("heads,n_q,n,m,d,layers", LISTA_SUPPORT_CASES)
def test_unrolled_decoder_over_the_support(heads, n_q, n, m, d, layers, options):
    """Layers that gather S's columns for the non-zero coefficients only: against float64 and against the layers over all columns."""
    g = torch.Generator(device=DEV).manual_seed(n)
    rows = heads * n_q
    randn = lambda *s: torch.randn(*s, generator=g, device=DEV)                     # noqa: E731
    Y, B = randn(heads, n_q, m), (randn(n, m) * 0.05).bfloat16()
    Y *= torch.rand(heads, n_q, 1, generator=g, device=DEV) ** 2                    # rows of a few and rows of many coefficients
    S = (torch.eye(n, device=DEV) + 0.3 / n ** 0.5 * randn(n, n)).bfloat16()
    V = randn(heads, n, d).bfloat16()
    theta = 2.0 * 0.05 * m ** 0.5
    thetas = [theta * (1.0 - 0.1 * t) for t in range(layers)]
    dims = csat.make_dims(1, heads, n_q, n, d, m, "bf16")

    def decode(choice, y=Y, s=S):
        options("support", choice)
        ws = torch.empty(csat.csat_lista_workspace_bytes(dims, layers), dtype=torch.uint8, device=DEV).fill_(0xFF)
        X, C = torch.empty(heads, n_q, n, device=DEV), torch.empty(heads, n_q, d, dtype=torch.bfloat16, device=DEV)
        csat.csat_recover_lista(dims, y.clone(), s, B, thetas, X, V, C, ws)
        torch.cuda.synchronize()
        return X, C

    X, C = decode(2)
    W = torch.matmul(Y.bfloat16().double().view(rows, m), B.double().t().contiguous())
    D = (S.float() - torch.eye(n, device=DEV)).bfloat16().double().t().contiguous()
    x = torch.zeros(rows, n, dtype=torch.float64, device=DEV)
    for th in thetas:
        u = W + x + torch.matmul(x.float().bfloat16().double(), D)
        x = u.sign() * (u.abs() - th).clamp_min(0.0)
    density = float((x != 0).double().mean())
    assert 0.001 < density < 0.1
    # the same roundings as in float64 here but for the float sums: 1e-6 of |u| <= 4 |x|, and a coefficient whose rounding to bf16
    # falls the other way, one of 2^-8 of itself in about 1e-3 of them and layer
    assert float((X.double().view(rows, n) - x).norm() / x.norm()) < 1e-3
    want = torch.matmul(x.float().bfloat16().double().view(heads, n_q, n), V.double())
    assert float((C.double() - want).norm() / want.norm()) < 3e-3       # (and C to bf16: 2^-9 each, at most)
    X1, C1 = decode(1)
    assert float((X1 - X).norm() / X.norm()) < 1e-3 and float((C1.float() - C.float()).norm() / C.float().norm()) < 4e-3
    Xr, Cr = decode(2)
    assert torch.equal(X, Xr) and torch.equal(C, Cr)
    # a matrix with an infinity or NaN, whose products with zeros are NaN, stays on the layers over all columns
    for bad in (float("inf"), float("nan")):
        Sb = S.clone()
        Sb[n // 2, n - 1] = bad
        got, old = decode(2, s=Sb), decode(1, s=Sb)
        assert all(torch.equal(p.isnan(), q.isnan()) and torch.equal(p.nan_to_num(), q.nan_to_num()) for p, q in zip(got, old))
    # an infinite measurement reaches its own row only
    Yb = Y.clone()
    Yb[heads - 1, n_q - 1, 3] = float("inf")
    Xb, Cb = decode(2, y=Yb)
    assert torch.equal(Xb.view(rows, n)[:-1], X.view(rows, n)[:-1]) and torch.equal(Cb.view(rows, d)[:-1], C.view(rows, d)[:-1])
    assert not Xb.view(rows, n)[-1].isfinite().all()


# (n_q, n, m, iterations): m around the instances' 512, 640, 768 and 1024 and small ones (asked for); last groups of rows that are not whole;
# the residual over all columns as one product and split along K; columns that are not whole tiles; more than 1024 columns
RESIDUAL_SUPPORT_CASES = [(300, 600, 130, 3), (331, 1100, 513, 4), (130, 1500, 640, 3), (257, 1300, 641, 2), (1001, 2048, 768, 3), (90, 2111, 1000, 5),
                          (258, 1280, 1024, 3)]


@pytest.mark.parametrize("n_q,n,m,iters", RESIDUAL_SUPPORT_CASES)
def test_residual_over_the_support(n_q, n, m, iters, options):
    """The large-tile decoder with its residual over the non-zero coefficients: against the oracle, and against the product over all columns."""
    w = _small("residual_support", B=1, H=3, n_q=n_q, n=n, d=64, m=m, dtype="bf16", iters=iters, seed=n)
    Q, K, V = gen.make_qkv(w)
    Phi = gen.make_workload_phi(w)
    mu = _mu(Phi)
    p = _problem(w, Q, K, V, Phi)
    A, _ = p.attention(*p.measure())
    first = np.abs(np.einsum("hqm,mn->hqn", to_np(A), Phi.astype(np.float64)))
    lam = float(np.quantile(first, 0.985))
    options("decoder", 1)
    options("support", 2)
    p.ws.fill_(0xFF)
    C, _, X = p.forward(lam, mu, iters)
    assert csat.csat_profile_decoder_kernel() == -1
    ref = orc.forward(Q, K, V, Phi, lam, mu, iters)
    assert 0.001 < float((ref["X"] != 0).mean()) < 0.1
    assert_close("X", to_np(X), ref["X"], TOL["bf16"])
    assert_close("C", to_np(C), ref["C"], TOL["bf16"])
    p.ws.fill_(0xFF)
    C2, _, X2 = p.forward(lam, mu, iters)
    assert torch.equal(X, X2) and torch.equal(C, C2)
    # the stage call has its measurement rows as the caller holds them
    Xs, Cs = p.recover(A, lam, mu, iters)
    options("support", 1)
    C1, _, X1 = p.forward(lam, mu, iters)
    X1s, C1s = p.recover(A, lam, mu, iters)
    # the residual is the same up to its float sums, so that one in about 2^8 of its elements is rounded to bf16 the other way: 2^-8 * 2^-4
    # of the residual, times what the threshold leaves of u (here up to 10)
    for got, old in ((X, X1), (Xs, X1s), (C.float(), C1.float()), (Cs.float(), C1s.float())):
        assert float((got - old).norm() / old.norm()) < 5e-3
    # an infinite measurement reaches its own row only
    Ab = A.clone()
    Ab[2, n_q - 1, 1] = float("inf")
    options("support", 2)
    Xb, _ = p.recover(Ab, lam, mu, iters)
    assert torch.equal(Xb.view(-1, n)[:-1], Xs.view(-1, n)[:-1]) and not Xb.view(-1, n)[-1].isfinite().all()


# (dtype, n_q, n, m, d, iterations, columns of Phi the rows lean on): rows for 128-row groups on the two-chunk decoder with the synthesis inside it and
# outside, the large-tile decoder with and without its product split along K, float; counts that are not whole tiles, and none at all
SCREEN_CASES = [("bf16", 2816, 1600, 392, 64, 4, 0.2), ("bf16", 2800, 700, 200, 128, 5, 0.4), ("bf16", 2816, 330, 100, 64, 3, 0.3), ("bf16", 700, 900, 500, 64, 4, 0.3),
                ("bf16", 5000, 800, 450, 80, 3, 0.1), ("bf16", 2816, 1600, 392, 64, 4, 0.0), ("f32", 900, 700, 150, 64, 4, 0.3), ("f32", 1100, 333, 75, 72, 3, 0.4),
                ("bf16", 2816, 1600, 392, 64, 4, 0.9)]


@pytest.mark.parametrize("dtype,n_q,n,m,d,iters,share", SCREEN_CASES)
def test_rows_without_coefficients_left_out(dtype, n_q, n, m, d, iters, share, options):
    """Rows with |Phi^T y| <= lambda have x = 0 throughout and are left out of the decoder: C is zero there and the decoder's elsewhere."""
    heads = 3
    g = torch.Generator(device=DEV).manual_seed(n + m)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    Phi = (torch.randn(m, n, generator=g, device=DEV) / m ** 0.5).to(t)
    rows = heads * n_q
    Y = 0.002 * torch.randn(rows, m, generator=g, device=DEV)
    lean = torch.rand(rows, generator=g, device=DEV) < share
    cols = torch.randint(0, n, (rows, 3), generator=g, device=DEV)
    Y[lean] += 0.4 * Phi.float().t()[cols[lean]].sum(1)
    mu, lam = 0.25 * m / n, 0.1
    V = torch.randn(heads, n, d, generator=g, device=DEV).to(t)
    dims = csat.make_dims(1, heads, n_q, n, d, m, dtype)

    def decode(choice, y=Y):
        options("screen", choice)
        ws = torch.empty(csat.csat_workspace_bytes(dims, iters), dtype=torch.uint8, device=DEV).fill_(0xFF)
        C = torch.empty(heads, n_q, d, dtype=t, device=DEV).fill_(7.0)
        csat.csat_recover(dims, y.view(heads, n_q, m).clone(), Phi, lam, mu, iters, None, V, C, ws)
        assert csat.csat_decoder_status(ws) == 0
        return C.view(rows, d)

    C, C1 = decode(2), decode(1)
    x = torch.zeros(rows, n, dtype=torch.float64, device=DEV)
    P = Phi.double()
    for _ in range(iters):
        u = x + mu * torch.matmul(Y.double() - torch.matmul(x, P.t().contiguous()), P)
        x = u.sign() * (u.abs() - mu * lam).clamp_min(0.0)
    want = torch.matmul(x.view(heads, n_q, n), V.double()).view(rows, d)
    zero = (x == 0).all(1)
    assert bool((C[zero] == 0).all()) and (share == 0.0) == bool(zero.all())
    assert torch.equal(decode(2), C)
    if share > 0:
        assert float((C.double() - want).norm() / want.norm()) < (2e-2 if dtype == "bf16" else 1e-5)
        # the same roundings; sums of the synthesis in another order
        assert float((C.float() - C1.float()).norm() / C1.float().norm()) < (4e-3 if dtype == "bf16" else 2e-6)
    # NaN and infinities stay with their rows
    Yb = Y.clone()
    i, j = int(zero.nonzero()[0]), int(zero.nonzero()[-1])
    Yb[i, 0], Yb[j, m - 1] = float("nan"), float("inf")
    Cb = decode(2, Yb)
    same = torch.ones(rows, dtype=torch.bool, device=DEV)
    same[i] = same[j] = False
    # (float: a tile of rows with such a one is computed on the float MFMA, in other sums: 2^-24 of u each, |u| up to 10 |x|)
    assert torch.equal(Cb[same], C[same]) if dtype == "bf16" else float((Cb[same] - C[same]).norm()) <= 2e-6 * float(C[same].norm())
    old = decode(1, Yb)
    assert torch.equal(Cb.isnan(), old.isnan()) and torch.equal(Cb.isinf(), old.isinf())


# (n_q, n, m, iterations): m on both sides of the instances' 256 and 512, rows of a few and of many coefficients, groups of rows and pieces of
# columns that are not whole
@pytest.mark.parametrize("n_q,n,m,iters", [(90, 300, 75, 3), (333, 1100, 256, 4), (101, 2049, 257, 3), (259, 1300, 512, 3), (130, 1601, 513, 2), (67, 1300, 1000, 3)])
def test_float_residual_over_the_support(n_q, n, m, iters, options):
    """The float decoder with its residual over the non-zero coefficients: no further from float64 than with the product over all columns."""
    heads = 2
    g = torch.Generator(device=DEV).manual_seed(n + m)
    rows = heads * n_q
    Phi = torch.randn(m, n, generator=g, device=DEV) / m ** 0.5
    Y = 0.02 * torch.randn(rows, m, generator=g, device=DEV) * torch.rand(rows, 1, generator=g, device=DEV) ** 3
    cols = torch.randint(0, n, (rows, 4), generator=g, device=DEV)
    Y += 0.3 * Phi.t()[cols].sum(1)
    lam, mu = 0.05, float(1.0 / torch.linalg.matrix_norm(Phi.double(), 2) ** 2)
    V = torch.randn(heads, n, 64, generator=g, device=DEV)
    dims = csat.make_dims(1, heads, n_q, n, 64, m, "f32")

    def decode(choice, y=Y, phi=Phi):
        options("support", choice)
        ws = torch.empty(csat.csat_workspace_bytes(dims, iters), dtype=torch.uint8, device=DEV).fill_(0xFF)
        X, C = torch.empty(heads, n_q, n, device=DEV), torch.empty(heads, n_q, 64, device=DEV)
        csat.csat_recover(dims, y.view(heads, n_q, m).clone(), phi, lam, mu, iters, X, V, C, ws)
        torch.cuda.synchronize()
        return X.view(rows, n), C

    X, C = decode(2)
    X1, C1 = decode(1)
    x = torch.zeros(rows, n, dtype=torch.float64, device=DEV)
    P, mu64, theta = Phi.double(), float(np.float32(mu)), float(np.float32(mu) * np.float32(lam))
    for _ in range(iters):
        u = x + mu64 * torch.matmul(Y.double() - torch.matmul(x, P.t().contiguous()), P)
        x = u.sign() * (u.abs() - theta).clamp_min(0.0)
    assert 0.0005 < float((x != 0).double().mean()) < 0.5
    err, err1 = (float((v.double() - x).norm() / x.norm()) for v in (X, X1))
    assert err <= 1.1 * err1 and err < 1e-5       # (a tenth: the update's sums, equal on both sides but for their operands' last bits)
    again = decode(2)
    assert torch.equal(again[0], X) and torch.equal(again[1], C)
    # a matrix with an infinity stays on the product over all columns, NaN and infinities in a row with that row
    bad = Phi.clone()
    bad[m // 2, n - 1] = float("inf")
    got, old = decode(2, phi=bad), decode(1, phi=bad)
    assert all(torch.equal(p.isnan(), q.isnan()) and torch.equal(p.isinf(), q.isinf()) for p, q in zip(got, old))
    Yb = Y.clone()
    Yb[3, 0], Yb[rows - 1, m - 1] = float("nan"), float("inf")
    got, old = decode(2, y=Yb), decode(1, y=Yb)
    assert all(torch.equal(p.isnan(), q.isnan()) and torch.equal(p.isinf(), q.isinf()) for p, q in zip(got, old))


@pytest.mark.parametrize("dtype,n_q,n,m", [("bf16", 2816, 700, 200), ("bf16", 1100, 900, 500), ("f32", 900, 700, 300)])
def test_packed_rows_and_support_in_a_graph(dtype, n_q, n, m, options):
    """What the device decides, it decides in every replay anew: replays over changed measurements against the eager call."""
    heads, iters, d = 3, 4, 64
    g = torch.Generator(device=DEV).manual_seed(n)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    Phi = (torch.randn(m, n, generator=g, device=DEV) / m ** 0.5).to(t)
    V = torch.randn(heads, n, d, generator=g, device=DEV).to(t)
    rows = heads * n_q
    dims = csat.make_dims(1, heads, n_q, n, d, m, dtype)
    options("screen", 2)
    options("support", 2)

    def measurements(share):
        Y = 0.002 * torch.randn(rows, m, generator=g, device=DEV)
        lean = torch.rand(rows, generator=g, device=DEV) < share
        Y[lean] += 0.4 * Phi.float().t()[torch.randint(0, n, (rows,), generator=g, device=DEV)[lean]]
        return Y.view(heads, n_q, m)

    Y = measurements(0.2)
    ws = torch.empty(csat.csat_workspace_bytes(dims, iters), dtype=torch.uint8, device=DEV).fill_(0xFF)
    C = torch.empty(heads, n_q, d, dtype=t, device=DEV)
    call = lambda: csat.csat_recover(dims, Y, Phi, 0.1, 0.25 * m / n, iters, None, V, C, ws)      # noqa: E731
    call()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call()
    for share in (0.3, 0.0, 0.9, 0.1):      # (0.9: too many rows to pack)
        Y.copy_(measurements(share))
        call()
        torch.cuda.synchronize()
        want = C.clone()
        C.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, want) and (share == 0.0) == (not bool(C.any()))


# (dtype, heads, n_q, n, m, iterations, share of rows with coefficients, packed, parts, apart): residual products that are not split along K, of row
# tiles that are no multiple of eight (their grid is padded), for all rows and for packed ones; the kernel over the support as a launch of its
# own (more than 1.2e11 products a residual); split along K with packed rows; float with packed rows
RESIDUAL_EITHER_CASES = [("bf16", 3, 258, 832, 600, 4, 1.0, False, 1, False), ("bf16", 3, 1001, 1216, 1024, 3, 0.5, False, 1, False),
                         ("bf16", 3, 938, 832, 600, 4, 0.38, True, 1, False), ("bf16", 1, 2305, 1216, 1000, 3, 0.3, True, 1, False),
                         ("bf16", 3, 700, 960, 600, 4, 0.3, True, 5, False),
                         ("bf16", 3, 20011, 3100, 660, 3, 0.5, False, 1, True), ("bf16", 3, 20011, 2050, 1000, 3, 0.5, False, 1, True),
                         ("bf16", 3, 20011, 3100, 660, 3, 0.3, True, 1, True), ("f32", 3, 1700, 900, 392, 4, 0.3, True, 0, False),
                         ("f32", 2, 1300, 1600, 600, 3, 0.3, True, 0, False)]


@pytest.mark.parametrize("dtype,heads,n_q,n,m,iters,share,packed,parts,apart", RESIDUAL_EITHER_CASES)
def test_residual_over_the_support_without_x(dtype, heads, n_q, n, m, iters, share, packed, parts, apart, options):
    """C of the products' decoder with its residual over the support, every row against float64 and against the product over all columns."""
    g = torch.Generator(device=DEV).manual_seed(n + m)
    t, bf16 = (torch.bfloat16, True) if dtype == "bf16" else (torch.float32, False)
    Phi = (torch.randn(m, n, generator=g, device=DEV) / m ** 0.5).to(t)
    rows, d = heads * n_q, 64
    Y = 0.002 * torch.randn(rows, m, generator=g, device=DEV)
    lean = torch.rand(rows, generator=g, device=DEV) < share
    cols = torch.randint(0, n, (rows, 3), generator=g, device=DEV)
    Y[lean] += 0.4 * Phi.float().t()[cols[lean]].sum(1)
    mu, lam = 0.25 * m / n, 0.13
    V = torch.randn(heads, n, d, generator=g, device=DEV).to(t)
    dims = csat.make_dims(1, heads, n_q, n, d, m, dtype)
    options("screen", 2 if packed else 1)

    def decode(choice):
        options("support", choice)
        ws = torch.empty(csat.csat_workspace_bytes(dims, iters), dtype=torch.uint8, device=DEV).fill_(0xFF)
        C = torch.empty(heads, n_q, d, dtype=t, device=DEV).fill_(7.0)
        csat.csat_recover(dims, Y.view(heads, n_q, m), Phi, lam, mu, iters, None, V, C, ws)
        assert csat.csat_profile_launch_form("residual") == (parts + (16 if apart and choice == 2 else 0))
        return C, ws[:256].view(torch.int32).tolist()

    C, words = decode(2)
    C1, _ = decode(1)
    x = torch.zeros(rows, n, dtype=torch.float64, device=DEV)
    P = Phi.double()
    for _ in range(iters):
        u = x + mu * torch.matmul(Y.double() - torch.matmul(x, P.t().contiguous()), P)
        x = u.sign() * (u.abs() - mu * lam).clamp_min(0.0)
    stay = int((x != 0).any(1).sum())
    # the device's words: non-zero pieces counted and none that forbids; the rows that it packed, none of them with coefficients left out
    assert words[8] > 0 and words[9] == 0
    assert words[16] == 0 and stay <= words[18] <= rows // 2 - 256 if packed else words[16] == -1
    want = torch.matmul(x.view(heads, n_q, n), V.double()).view(rows, d)
    assert float((C.double().view(rows, d) - want).norm() / want.norm()) < (2e-2 if bf16 else 1e-5)
    # the same roundings but for the residual's sums (bf16: as test_residual_over_the_support), row by row on the scale of the largest
    diff, size = (C.float() - C1.float()).view(rows, d).norm(dim=1), C1.float().view(rows, d).norm(dim=1)
    assert float(diff.max()) < (3e-2 if bf16 else 1e-5) * float(size.max()) and float(diff.norm() / size.norm()) < (5e-3 if bf16 else 2e-6)
    assert torch.equal(decode(2)[0], C)


# (what runs, dtype, heads, n_q, n, m, d): rows left out, on the two-chunk decoder, the large-tile pair and in float; the unrolled decoder over its support,
# with both kernels of its synthesis
@pytest.mark.parametrize("op,dtype,heads,n_q,n,m,d", [("screen", "bf16", 3, 2816, 700, 200, 64), ("screen", "bf16", 3, 700, 900, 500, 72), ("screen", "f32", 3, 900, 700, 150, 64),
                                                      ("lista", "bf16", 3, 391, 770, 160, 128), ("lista", "bf16", 3, 391, 770, 160, 72)])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_infinities_and_nan_of_v(op, dtype, heads, n_q, n, m, d, bad, options):
    """Zero times an infinity or NaN is NaN: C is what the product over all coefficients gives, in the last element of V as in the first."""
    g = torch.Generator(device=DEV).manual_seed(n + d)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    Phi = (torch.randn(m, n, generator=g, device=DEV) / m ** 0.5).to(t)
    Y = 0.002 * torch.randn(heads, n_q, m, generator=g, device=DEV)
    lean = torch.rand(heads, n_q, generator=g, device=DEV) < 0.3
    Y[lean] += 0.4 * Phi.float().t()[torch.randint(0, n, (int(lean.sum()),), generator=g, device=DEV)]
    mu, lam, iters = 0.25 * m / n, 0.13, 3
    S, B = (torch.eye(n, device=DEV) - mu * torch.matmul(Phi.float().t().contiguous(), Phi.float())).to(t), (mu * Phi.float().t()).to(t).contiguous()
    dims = csat.make_dims(1, heads, n_q, n, d, m, dtype)
    V = torch.randn(heads, n, d, generator=g, device=DEV).to(t)

    def decode(v, choice):
        options("screen" if op == "screen" else "support", choice)
        ws = torch.empty(max(csat.csat_workspace_bytes(dims, iters), csat.csat_lista_workspace_bytes(dims, iters)), dtype=torch.uint8, device=DEV).fill_(0xFF)
        C = torch.empty(heads, n_q, d, dtype=t, device=DEV).fill_(7.0)
        if op == "screen":
            csat.csat_recover(dims, Y, Phi, lam, mu, iters, None, v, C, ws)
        else:
            csat.csat_recover_lista(dims, Y, S, B, [mu * lam] * iters, None, v, C, ws)
        return C, ws[:256].view(torch.int32).tolist()

    C, words = decode(V, 2)
    assert C.isfinite().all() and (words[16] == 0 if op == "screen" else words[9] == 0)
    for h, j, k in ((0, 0, 0), (heads - 1, n - 1, d - 1), (1, n // 2, 5)):
        Vb = V.clone()
        Vb[h, j, k] = bad
        got, want = decode(Vb, 2)[0], decode(Vb, 1)[0]
        assert want[h, :, k].isnan().sum() > n_q // 2 and want.isfinite().sum() == want.numel() - n_q
        assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.nan_to_num(), want.nan_to_num())


@pytest.mark.parametrize("n", [161, 330, 1000])
def test_packed_rows_of_a_square_matrix(n, options):
    """m = n in float: a row of y is longer in the workspace than one of the iterate, so fewer than half of the rows fit packed.  The oracle is the decoder
    over all rows; nothing is written behind the workspace."""
    heads, n_q, d, iters, m = 3, 2816, 64, 3, n
    g = torch.Generator(device=DEV).manual_seed(n)
    Phi = torch.randn(m, n, generator=g, device=DEV) / m ** 0.5
    V = torch.randn(heads, n, d, generator=g, device=DEV)
    dims = csat.make_dims(1, heads, n_q, n, d, m, "f32")
    rows, wb = heads * n_q, csat.csat_workspace_bytes(dims, iters)
    fit = min(rows // 2, rows // 2 * ((n + 7) // 8 * 8) // ((m + 31) // 32 * 32)) - 256      # (rows: a multiple of 256)
    for stay in (fit // 2, fit - 3, fit, fit + 1, rows // 2 - 256, rows // 2):
        Y = torch.zeros(rows, m, device=DEV)
        lean = torch.randperm(rows, generator=g, device=DEV)[:stay]
        Y[lean] = 0.4 * Phi.t()[torch.randint(0, n, (stay,), generator=g, device=DEV)]
        out = []
        for choice in (2, 1):
            options("screen", choice)
            ws = torch.full((wb + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
            C = torch.empty(heads, n_q, d, device=DEV).fill_(7.0)
            csat.csat_recover(dims, Y.view(heads, n_q, m), Phi, 0.1, 0.1, iters, None, V, C, ws[:wb])
            assert bool((ws[wb:] == 0xA5).all())
            out.append((C, ws[:256].view(torch.int32).tolist()))
        (C, words), (C1, _) = out
        assert words[18] == stay and (words[16] == 0) == (stay <= fit)
        assert float((C - C1).norm() / C1.norm()) < 2e-6      # (sums of the synthesis in another order)


# thresholds of lambda from .. to, the lowest in the middle or at the end; whether the device is asked at all
@pytest.mark.parametrize("first,low,last,asked", [(1.25, 0.9, 0.75, True), (1.25, 0.75, 0.32, True), (1.25, 0.75, 0.3, False), (1.25, 0.3, 1.0, False), (0.0, 0.5, 1.0, True)])
def test_unrolled_decoder_whose_thresholds_fall(first, low, last, asked, options):
    """Thresholds that fall far below the first layer's leave an iterate that its count says nothing of: such a call stays on the layers over all columns."""
    heads, n_q, n, m, d, layers = 8, 701, 700, 200, 64, 21
    g = torch.Generator(device=DEV).manual_seed(d)
    Phi = torch.randn(m, n, generator=g, device=DEV) / m ** 0.5
    mu = float(1.0 / torch.linalg.matrix_norm(Phi, 2) ** 2)
    S, B = (torch.eye(n, device=DEV) - mu * torch.matmul(Phi.t().contiguous(), Phi)).bfloat16(), (mu * Phi.t()).bfloat16().contiguous()
    Y = 0.02 * torch.randn(heads, n_q, m, generator=g, device=DEV)
    Y += 0.4 * Phi.t()[torch.randint(0, n, (heads, n_q), generator=g, device=DEV)]
    V = torch.randn(heads, n, d, generator=g, device=DEV).bfloat16()
    half = layers // 2
    thetas = [mu * 0.1 * (first + (low - first) * t / half if t < half else low + (last - low) * (t - half) / half) for t in range(layers)]
    dims = csat.make_dims(1, heads, n_q, n, d, m, "bf16")

    def decode(choice):
        options("support", choice)
        ws = torch.empty(csat.csat_lista_workspace_bytes(dims, layers), dtype=torch.uint8, device=DEV).fill_(0xFF)
        X, C = torch.empty(heads, n_q, n, device=DEV), torch.empty(heads, n_q, d, dtype=torch.bfloat16, device=DEV)
        csat.csat_recover_lista(dims, Y, S, B, thetas, X, V, C, ws)
        return X, C, ws[:256].view(torch.int32).tolist()

    X, C, words = decode(0)
    X1, C1, _ = decode(1)
    # (the words of the status block that bench.py reads what ran from)
    assert words[9:11] == [0, int(words[8] <= heads * n_q / 4 * 24)] if asked else words[9:11] == [-1, -1]
    if words[10] != 1:
        assert torch.equal(X, X1) and torch.equal(C, C1)
    else:      # as test_unrolled_decoder_over_the_support
        assert float((X1 - X).norm() / X.norm()) < 1e-3 and float((C1.float() - C.float()).norm() / C.float().norm()) < 4e-3


def test_count_of_a_dense_iterate_does_not_wrap(options):
    """Just below 2^32 elements of a float iterate, all of them non-zero: every eighth row, counted eight times, is more than a word holds."""
    heads, n_q, n, m, d, iters = 5, 42949, 20000, 256, 64, 2
    rows = heads * n_q
    assert rows * n < 2 ** 32 < (rows + 7) // 8 * 8 * n
    g = torch.Generator(device=DEV).manual_seed(n)
    Phi = torch.randn(m, n, generator=g, device=DEV) / m ** 0.5
    Y = torch.randn(heads, n_q, m, generator=g, device=DEV)
    V = torch.randn(heads, n, d, generator=g, device=DEV)
    dims = csat.make_dims(1, heads, n_q, n, d, m, "f32")
    ws = torch.empty(csat.csat_workspace_bytes(dims, iters), dtype=torch.uint8, device=DEV)
    ws[:256].fill_(0xFF)
    C = torch.empty(heads, n_q, d, device=DEV)
    csat.csat_recover(dims, Y, Phi, 0.0, 0.25 * m / n, iters, None, V, C, ws)
    count, not_sparse = ws[:256].view(torch.int32).tolist()[8:10]
    assert not_sparse != 0 or count % 2 ** 32 > 0.025 * rows * n
    # x after two iterations from zero, of some rows
    P, mu = Phi.double(), 0.25 * m / n
    y = Y.view(rows, m)[[0, rows // 2, rows - 1]].double()
    x = mu * torch.matmul(y, P)
    x = x + mu * torch.matmul(y - torch.matmul(x, P.t().contiguous()), P)
    want = torch.stack([torch.matmul(x[i], V[h].double()) for i, h in enumerate((0, rows // 2 // n_q, heads - 1))])
    got = C.view(rows, d)[[0, rows // 2, rows - 1]].double()
    assert float((got - want).norm() / want.norm()) < 1e-5


@pytest.mark.parametrize("every,packs", [(64, True), (1, False)])
def test_sample_of_rows_meets_every_place_in_a_head(every, packs, options):
    """Heads of a multiple of 64 rows whose every 64th has coefficients: the sample that decides on packing is not of those alone."""
    heads, n_q, n, m, d, iters = 48, 2048, 700, 200, 64, 50
    g = torch.Generator(device=DEV).manual_seed(every)
    Phi = (torch.randn(m, n, generator=g, device=DEV) / m ** 0.5).bfloat16()
    Y = torch.zeros(heads, n_q, m, device=DEV)
    Y[:, ::every] = 0.4 * Phi.float().t()[torch.randint(0, n, (heads, n_q // every), generator=g, device=DEV)]
    V = torch.randn(heads, n, d, generator=g, device=DEV).bfloat16()
    dims = csat.make_dims(1, heads, n_q, n, d, m, "bf16")
    out = []
    for choice in (0, 1):
        options("screen", choice)
        ws = torch.empty(csat.csat_workspace_bytes(dims, iters), dtype=torch.uint8, device=DEV).fill_(0xFF)
        C = torch.empty(heads, n_q, d, dtype=torch.bfloat16, device=DEV)
        csat.csat_recover(dims, Y, Phi, 0.1, 0.25 * m / n, iters, None, V, C, ws)
        out.append((C.float(), ws[:256].view(torch.int32).tolist()))
    (C, words), (C1, _) = out
    assert (words[16] == 0) == packs and (not packs or words[18] == heads * n_q // every)
    assert float((C - C1).norm() / C1.norm()) < 4e-3      # as test_rows_without_coefficients_left_out


# (n_q, n, m, iterations): three heads of rows that take fewer rounds on the wider tile, last tiles of rows and of columns that are not whole; the
# two-chunk decoder and the large-tile pair
@pytest.mark.parametrize("n_q,n,m,iters", [(4099, 1571, 392, 3), (4096, 1600, 264, 3), (4100, 1300, 640, 3)])
def test_rows_left_out_are_found_on_wide_tiles(n_q, n, m, iters, options):
    """Every row that leans on one column of Phi stays, whichever element of a tile that is, and no other; C against float64."""
    heads, d = 3, 64
    g = torch.Generator(device=DEV).manual_seed(n + m)
    Phi = (torch.randn(m, n, generator=g, device=DEV) / m ** 0.5).bfloat16()
    rows = heads * n_q
    lean = torch.rand(rows, generator=g, device=DEV) < 0.3
    cols = torch.randint(0, n, (rows,), generator=g, device=DEV)
    Y = 0.002 * torch.randn(rows, m, generator=g, device=DEV)
    Y[lean] += 0.3 * Phi.float().t()[cols[lean]]
    # 0.3 |phi|^2 on that column, at most 0.3 |phi_i phi_j| on the others: the rest is noise of 0.002
    mu, lam = 0.25 * m / n, 0.18
    peak = torch.matmul(Y.double(), Phi.double()).abs().amax(1)
    assert bool(((peak > 1.02 * lam) == lean).all()) and not bool(((peak - lam).abs() < 0.02 * lam).any())
    V = torch.randn(heads, n, d, generator=g, device=DEV).bfloat16()
    dims = csat.make_dims(1, heads, n_q, n, d, m, "bf16")
    options("screen", 2)
    ws = torch.empty(csat.csat_workspace_bytes(dims, iters), dtype=torch.uint8, device=DEV).fill_(0xFF)
    C = torch.empty(heads, n_q, d, dtype=torch.bfloat16, device=DEV).fill_(7.0)
    csat.csat_recover(dims, Y.view(heads, n_q, m), Phi, lam, mu, iters, None, V, C, ws)
    assert csat.csat_profile_launch_form("screen_tile") == 320
    words = ws[:256].view(torch.int32).tolist()
    assert words[16] == 0 and words[18] == int(lean.sum())
    x = torch.zeros(rows, n, dtype=torch.float64, device=DEV)
    P = Phi.double()
    for _ in range(iters):
        u = x + mu * torch.matmul(Y.double() - torch.matmul(x, P.t().contiguous()), P)
        x = u.sign() * (u.abs() - mu * lam).clamp_min(0.0)
    want = torch.matmul(x.view(heads, n_q, n), V.double()).view(rows, d)
    C = C.view(rows, d)
    assert bool((C[~lean] == 0).all()) and float((C.double() - want).norm() / want.norm()) < 2e-2


# (rows, n, m, columns that a row leans on, whether the residual runs over the support, share of the rows, the others left out): products of one and of
# two rounds of tiles, whose few steps leave little to win, few rows of long columns, and packed rows
@pytest.mark.parametrize("rows,n,m,lean,sparse,share", [(12800, 2000, 1000, 3, False, 1.0), (12800, 2000, 1000, 0.5, True, 1.0), (28544, 1824, 744, 2, True, 1.0), (28544, 1824, 744, 5, False, 1.0),
                                                        (3432, 13713, 1024, 8, True, 1.0), (3432, 13713, 1024, 16, False, 1.0),
                                                        (28544, 1824, 744, 3, True, 0.2), (28544, 1824, 744, 5, False, 0.2), (12800, 2000, 1000, 3, True, 0.1)])
def test_residual_over_the_support_where_it_is_quicker(rows, n, m, lean, sparse, share, options):
    """The density up to which the residual's kernel over the support takes the product's place, as the device notes."""
    d, iters = 64, 3
    g = torch.Generator(device=DEV).manual_seed(n)
    Phi = (torch.randn(m, n, generator=g, device=DEV) / m ** 0.5).bfloat16()
    Y = 0.002 * torch.randn(rows, m, generator=g, device=DEV)
    stay = torch.rand(rows, 1, generator=g, device=DEV) < share
    for _ in range(max(1, int(lean))):
        some = stay & (torch.rand(rows, 1, generator=g, device=DEV) < lean)
        Y += some * 0.4 * Phi.float().t()[torch.randint(0, n, (rows,), generator=g, device=DEV)]
    V = torch.randn(8, n, d, generator=g, device=DEV).bfloat16()
    dims = csat.make_dims(1, 8, rows // 8, n, d, m, "bf16")
    options("screen", 1 if share == 1.0 else 2)
    out = []
    for choice in (0, 1, 2):
        options("support", choice)
        ws = torch.empty(csat.csat_workspace_bytes(dims, iters), dtype=torch.uint8, device=DEV).fill_(0xFF)
        C = torch.empty(8, rows // 8, d, dtype=torch.bfloat16, device=DEV)
        csat.csat_recover(dims, Y.view(8, rows // 8, m), Phi, 0.25, 0.25 * m / n, iters, None, V, C, ws)
        assert csat.csat_profile_launch_form("residual") == 1
        out.append((C, ws[:256].view(torch.int32).tolist()))
    (C, words), (C1, words1), (C2, words2) = out
    # pieces of four rows that the first iteration leaves, almost all of a column each; of packed rows as many as of all rows so dense
    assert 0.9 * lean * rows < words2[8] < 1.1 * lean * rows and words[9] == 0
    assert words2[18] == (-1 if share == 1.0 else int(stay.sum()))
    assert words[10] == int(sparse) and words1[10] == -1 and words2[10] == 1
    assert torch.equal(C, C2 if sparse else C1)


@pytest.mark.parametrize("left,packs", [(46, True), (50, False), (51, False)])
def test_sample_near_half_of_the_rows(left, packs, options):
    """Rows left of every 101, in heads and sample alike: below half of them they are packed, however near the sample comes to it."""
    heads, n_q, n, m, d, iters = 48, 2048, 700, 200, 64, 50
    rows = heads * n_q
    g = torch.Generator(device=DEV).manual_seed(left)
    Phi = (torch.randn(m, n, generator=g, device=DEV) / m ** 0.5).bfloat16()
    lean = torch.arange(rows, device=DEV) * 37 % 101 < left
    Y = torch.zeros(rows, m, device=DEV)
    Y[lean] = 0.4 * Phi.float().t()[torch.randint(0, n, (int(lean.sum()),), generator=g, device=DEV)]
    V = torch.randn(heads, n, d, generator=g, device=DEV).bfloat16()
    dims = csat.make_dims(1, heads, n_q, n, d, m, "bf16")
    out = []
    for choice in (0, 1):
        options("screen", choice)
        ws = torch.empty(csat.csat_workspace_bytes(dims, iters), dtype=torch.uint8, device=DEV).fill_(0xFF)
        C = torch.empty(heads, n_q, d, dtype=torch.bfloat16, device=DEV)
        csat.csat_recover(dims, Y.view(heads, n_q, m), Phi, 0.1, 0.25 * m / n, iters, None, V, C, ws)
        out.append((C.float(), ws[:256].view(torch.int32).tolist()))
    (C, words), (C1, _) = out
    assert (words[16] == 0) == packs and (not packs or words[18] == int(lean.sum()))
    assert float((C - C1).norm() / C1.norm()) < 4e-3      # as test_rows_without_coefficients_left_out


# (heads, n_q, n, m, layers, threshold in standard deviations of the first layer's u, over the support): short rows, all but dense or not, and long rows
@pytest.mark.parametrize("heads,n_q,n,m,layers,sigmas,sparse", [(192, 96, 96, 65, 25, 0.01, False), (192, 96, 96, 65, 25, 1.5, True), (48, 1000, 108, 65, 25, 0.3, False),
                                                                (48, 1000, 108, 65, 25, 2.0, True), (4, 3178, 3052, 400, 11, 3.0, False), (4, 3178, 3052, 400, 11, 3.6, True)])
def test_unrolled_decoder_over_the_support_where_it_is_quicker(heads, n_q, n, m, layers, sigmas, sparse, options):
    """The density up to which the layers run over the support: in short rows a share of their columns."""
    g = torch.Generator(device=DEV).manual_seed(n + int(sigmas * 10))
    rows, d = heads * n_q, 64
    Y, B = torch.randn(rows, m, generator=g, device=DEV), (0.05 * torch.randn(n, m, generator=g, device=DEV)).bfloat16()
    S = (0.9 * torch.eye(n, device=DEV)).bfloat16()
    V = torch.randn(heads, n, d, generator=g, device=DEV).bfloat16()
    theta = sigmas * 0.05 * m ** 0.5
    dims = csat.make_dims(1, heads, n_q, n, d, m, "bf16")
    out = []
    for choice in (0, 1, 2):
        options("support", choice)
        ws = torch.empty(csat.csat_lista_workspace_bytes(dims, layers), dtype=torch.uint8, device=DEV).fill_(0xFF)
        C = torch.empty(heads, n_q, d, dtype=torch.bfloat16, device=DEV)
        csat.csat_recover_lista(dims, Y.view(heads, n_q, m), S, B, [theta] * layers, None, V, C, ws)
        out.append((C, ws[:256].view(torch.int32).tolist()))
    (C, words), (C1, words1), (C2, words2) = out
    # the first layer leaves a float4 where one of its four is above (columns of B differ in length by a few per cent)
    above = math.erfc(sigmas / 2 ** 0.5)
    assert abs(words[8] / (rows / 4 * n * (1 - (1 - above) ** 4)) - 1) < 0.25 and words[9] == 0
    assert words[10] == int(sparse) and words1[10] == -1 and words2[10] == 1
    assert torch.equal(C, C2 if sparse else C1)
    assert float((C1.float() - C2.float()).norm() / C1.float().norm()) < 4e-3      # as test_unrolled_decoder_over_the_support
