"""Per-operator parity on the GPU through the C ABI: each fused kernel against
the oracle's definition of the same operator on the same seeded inputs.
Tolerances: fp32 mode 1e-5 (forward-type results) / 1e-4 (gradient-type);
bf16 mode 2e-2 / 3e-2 relative Frobenius; masks bit-exact."""
import numpy as np
import pytest
import torch

import paper_2303_04759_amd as raf
from oracle import layer as L
from oracle.philox import dropout_keep
from workloads.synthetic import round_to_bf16

from gemm_shapes import SHAPES
from gpu_util import announce, cdtype, host, rel_fro, to_dev

pytestmark = pytest.mark.gpu

FWD_TOL = {0: 1e-5, 1: 2e-2}
BWD_TOL = {0: 1e-4, 1: 3e-2}


def cfg_for(B, S, H, precision, p=0.1, causal=0, heads=None, eps=1e-5, seed=77, layer_id=2):
    return dict(batch=B, seq=S, hidden=H, heads=heads or H // 64, ffn=4 * H, pre_ln=0, causal=causal, gelu_tanh=0,
                precision=precision, ln_eps=eps, dropout_p=p, seed=seed, layer_id=layer_id)


def rnd(rng, shape, precision, scale=1.0):
    a = (scale * rng.standard_normal(shape)).astype(np.float32)
    return round_to_bf16(a) if precision == 1 else a


# ------------------------------------------------------------------ masks --
@pytest.mark.parametrize("site,n,p,step", [(1, 1000, 0.1, 1), (2, 4096 * 768, 0.1, 3), (3, 777, 0.5, (7 << 32) | 9),
                                           (1, 8, 0.0, 0), (2, 12345, 0.999, 2)])
def test_dropout_mask_bit_exact(site, n, p, step):
    announce("mask", site, n, p, step)
    cfg = cfg_for(1, 32, 64, 0, p=p, seed=0xDEADBEEF12345678, layer_id=0xABCDE)
    out = torch.zeros(n, dtype=torch.uint8, device="cuda")
    raf.raf_debug_dropout_mask(raf.make_desc(cfg), site, step, out, n)
    torch.cuda.synchronize()
    ref = dropout_keep(cfg["seed"], cfg["layer_id"], site, step, n, p)
    assert np.array_equal(out.cpu().numpy().astype(bool), ref)


# ------------------------------------------------------------------- gemm --
GEMM_SHAPES = [(32, 32, 32), (64, 96, 64), (160, 224, 96), (256, 128, 192), (128, 64, 128), (416, 320, 64),
               (256, 384, 768), (160, 96, 320), (384, 64, 512)]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("ak,bk", [(1, 1), (1, 0), (0, 0), (0, 1)])
@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_gemm_layouts(precision, ak, bk, M, N, K):
    announce("gemm", precision, ak, bk, M, N, K)
    rng = np.random.default_rng(M * 7 + N * 3 + K + ak * 2 + bk)
    A = rnd(rng, (M, K), precision)
    Bm = rnd(rng, (K, N), precision)
    dt = cdtype(precision)
    a_dev = to_dev(A if ak else A.T, dt)
    b_dev = to_dev(Bm.T if bk else Bm, dt)
    c = torch.zeros(M, N, dtype=dt, device="cuda")
    raf.raf_op_gemm(precision, M, N, K, a_dev, a_dev.shape[1], ak, b_dev, b_dev.shape[1], bk, c, N, alpha=0.5)
    torch.cuda.synchronize()
    ref = 0.5 * (A.astype(np.float64) @ Bm.astype(np.float64))
    assert rel_fro(host(c), ref) <= (1e-5 if precision == 0 else 4e-3)


# K-major x K-major bf16 products large enough that the launcher leaves the 128x128 tile, with partial last row tiles and
# full layer shapes: the 128x96, 128x144 and 256x144 tiles of the rings, the 256x192 ones of single k-steps and the
# 256x192 and 256x256 ones of the ping-pong kernel.
TILE_FAMILY_SHAPES = [(992, 2304, 128), (1984, 2304, 64), (2016, 3072, 64), (3968, 2304, 64), (3968, 3072, 64),
                      (4096, 768, 768), (4096, 2304, 768), (4096, 3072, 128), (4096, 768, 3072),
                      (4096, 4096, 1024), (3968, 4096, 64), (2016, 8192, 128)]


@pytest.mark.parametrize("M,N,K", TILE_FAMILY_SHAPES)
def test_gemm_tile_family(M, N, K):
    announce("gemm-tile-family", M, N, K)
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    A = rnd(rng, (M, K), 1)
    W = rnd(rng, (N, K), 1, 0.1)
    bias = rng.standard_normal(N).astype(np.float32)
    a_dev, w_dev, b_dev = to_dev(A, torch.bfloat16), to_dev(W, torch.bfloat16), torch.from_numpy(bias).cuda()
    c = torch.zeros(M, N, dtype=torch.bfloat16, device="cuda")
    raf.raf_op_gemm(1, M, N, K, a_dev, K, 1, w_dev, K, 1, c, N, epilogue=raf.EPI_BIAS, bias=b_dev)
    torch.cuda.synchronize()
    ref = A.astype(np.float64) @ W.astype(np.float64).T + bias
    got = host(c)
    assert rel_fro(got, ref) <= 4e-3
    # element-wise as well: a misplaced block would hide in a Frobenius norm of this size
    assert np.max(np.abs(got - ref)) <= 0.02 * (1.0 + np.max(np.abs(ref)))


def test_gemm_256x256_tile_epilogues():
    """The epilogues with a second operand or a second output on the largest tile (2016 x 8192: 8 x 32 tiles of
    256 x 256, the last row of tiles partial)."""
    announce("gemm 256x256 epilogues")
    rng = np.random.default_rng(256)
    M, N, K = 2016, 8192, 128
    bf = torch.bfloat16
    A, W = rnd(rng, (M, K), 1), rnd(rng, (N, K), 1, 0.1)
    bias = rng.standard_normal(N).astype(np.float32)
    a_dev, w_dev, b_dev = to_dev(A, bf), to_dev(W, bf), torch.from_numpy(bias).cuda()
    lin = A.astype(np.float64) @ W.astype(np.float64).T
    tol = 6e-3
    c = torch.zeros(M, N, dtype=bf, device="cuda")
    dsave = torch.zeros(M, N, dtype=bf, device="cuda")
    raf.raf_op_gemm(1, M, N, K, a_dev, K, 1, w_dev, K, 1, c, N, epilogue=raf.EPI_BIAS_GELU_DERIV, bias=b_dev, aux=dsave)
    assert rel_fro(host(c), L.gelu(lin + bias, False)) <= 2 * tol
    assert rel_fro(host(dsave), L.gelu_grad(lin + bias, False)) <= 2 * tol
    raf.raf_op_gemm(1, M, N, K, a_dev, K, 1, w_dev, K, 1, c, N, epilogue=raf.EPI_MUL_AUX, aux=dsave)
    got, ref = host(c), lin * host(dsave)
    assert rel_fro(got, ref) <= 2 * tol
    assert np.max(np.abs(got - ref)) <= 0.03 * (1.0 + np.max(np.abs(ref)))
    R = rnd(rng, (M, N), 1)
    raf.raf_op_gemm(1, M, N, K, a_dev, K, 1, w_dev, K, 1, c, N, epilogue=raf.EPI_ADD_RES, aux=to_dev(R, bf))
    got, ref = host(c), lin + R
    assert rel_fro(got, ref) <= tol
    assert np.max(np.abs(got - ref)) <= 0.02 * (1.0 + np.max(np.abs(ref)))


# Contractions that end in half a k-step, over the tiles of the split kernel with ragged last tiles and contractions shorter
# than the wavefronts' shares, over the rings and over the ping-pong kernel (gemm_shapes.py lists which shape reaches which
# kernel).  Bound per element: bf16 rounding of the result (2^-9 relative, twice that for the stored pre-activation path)
# and float32 accumulation of K products.
@pytest.mark.parametrize("epi", ["bias", "gelu_pair", "residual"])
@pytest.mark.parametrize("M,N,K", [(32, 32, 32), (64, 768, 800), (128, 768, 352), (256, 768, 800), (96, 3072, 96),
                                   (480, 1056, 352), (1056, 480, 352), (992, 736, 1056), (992, 1024, 1056),
                                   (992, 1440, 1568), (4064, 768, 96), (1984, 2304, 96), (8160, 768, 96),
                                   (3968, 2304, 96), (3968, 3072, 96), (2016, 8192, 96), (4064, 1024, 96),
                                   (3968, 3072, 1568)])
def test_gemm_split_tiles_and_half_steps(M, N, K, epi):
    announce("gemm-split", M, N, K, epi)
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    A, W = rnd(rng, (M, K), 1), rnd(rng, (N, K), 1, 0.1)
    bias = rng.standard_normal(N).astype(np.float32)
    a_dev, w_dev, b_dev = to_dev(A, torch.bfloat16), to_dev(W, torch.bfloat16), torch.from_numpy(bias).cuda()
    lin = A.astype(np.float64) @ W.astype(np.float64).T
    slack = K * 2.0 ** -24 * (np.abs(A).astype(np.float64) @ np.abs(W).astype(np.float64).T) + 1e-6
    c = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")

    def check(ref, extra=0.0):
        err = np.abs(host(c) - ref)
        assert (err <= 2.0 ** -8 * np.abs(ref) + slack + extra).all(), float(err.max())
    if epi == "bias":
        raf.raf_op_gemm(1, M, N, K, a_dev, K, 1, w_dev, K, 1, c, N, epilogue=raf.EPI_BIAS, bias=b_dev)
        check(lin + bias)
    elif epi == "gelu_pair":
        # the fast erf form: |gelu error| <= 2.6e-5 (times |u| <= 40 here), gelu' is read back and applied
        d = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        raf.raf_op_gemm(1, M, N, K, a_dev, K, 1, w_dev, K, 1, c, N, epilogue=raf.EPI_BIAS_GELU_DERIV, bias=b_dev, aux=d)
        check(L.gelu(lin + bias, False), 2e-3)
        raf.raf_op_gemm(1, M, N, K, a_dev, K, 1, w_dev, K, 1, c, N, epilogue=raf.EPI_MUL_AUX, aux=d)
        check(lin * host(d))
    else:
        R = rnd(rng, (M, N), 1)
        raf.raf_op_gemm(1, M, N, K, a_dev, K, 1, w_dev, K, 1, c, N, epilogue=raf.EPI_ADD_RES, aux=to_dev(R, torch.bfloat16))
        check(lin + R)


# The ping-pong kernel: each of its three tiles (256x128, 256x192, 256x256 by the widths), ragged in both directions and
# with a last group of two tile rows; two and three k-steps, which run its end without its main loop, and more, odd and
# even, with and without half a step at the end.  Bounds as above.
@pytest.mark.parametrize("epi", ["bias", "gelu_pair", "residual"])
@pytest.mark.parametrize("K", [96, 128, 160, 192, 256, 352, 448])
@pytest.mark.parametrize("N", [2016, 3040, 4064])
def test_gemm_pingpong_tiles(N, K, epi):
    test_gemm_split_tiles_and_half_steps(3488, N, K, epi)


# Every kernel and tile with whole and with half k-steps at the end.  Bounds as above.
@pytest.mark.parametrize("epi", ["bias", "gelu_pair", "residual"])
@pytest.mark.parametrize("M,N,K", [s[:3] for s in SHAPES])
def test_gemm_every_kernel_and_tile(M, N, K, epi):
    test_gemm_split_tiles_and_half_steps(M, N, K, epi)


# A panel wider than the ping-pong kernel's offsets reach stays on the 256x192 ring: rows of A 2^20 + 8 values apart.
@pytest.mark.parametrize("K", [32, 96, 192])
def test_gemm_rows_far_apart(K):
    announce("gemm-rows-far-apart", K)
    M, N, ld = 224, 49152, (1 << 20) + 8
    rng = np.random.default_rng(K)
    A, W = rnd(rng, (M, K), 1), rnd(rng, (N, K), 1, 0.1)
    wide = torch.empty(M, ld, dtype=torch.bfloat16, device="cuda")
    wide[:, :K] = to_dev(A, torch.bfloat16)
    c = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    raf.raf_op_gemm(1, M, N, K, wide, ld, 1, to_dev(W, torch.bfloat16), K, 1, c, N)
    ref = A.astype(np.float64) @ W.astype(np.float64).T
    slack = K * 2.0 ** -24 * (np.abs(A).astype(np.float64) @ np.abs(W).astype(np.float64).T) + 1e-6
    err = np.abs(host(c) - ref)
    assert (err <= 2.0 ** -8 * np.abs(ref) + slack).all(), float(err.max())


# Leading dimensions other than the contraction: padded rows (the ping-pong kernel sizes its buffer descriptors from them),
# one row repeated and rows stored backwards.  Bounds as above; the padding holds nan, which no result may see.
@pytest.mark.parametrize("M,N,K", [(3488, 4064, 192), (3488, 3040, 96), (256, 768, 800)])
@pytest.mark.parametrize("form", ["padded", "repeated", "backwards"])
def test_gemm_leading_dimensions(M, N, K, form):
    announce("gemm-ld", M, N, K, form)
    rng = np.random.default_rng(M + N + K)
    A, W = rnd(rng, (M, K), 1), rnd(rng, (N, K), 1, 0.1)
    lda, ldb = {"padded": (K + 40, K + 264), "repeated": (0, K), "backwards": (-K, -K)}[form]
    if form == "padded":
        a_dev, w_dev = (torch.full((r, ld), float("nan"), dtype=torch.bfloat16, device="cuda") for r, ld in ((M, lda), (N, ldb)))
        a_dev[:, :K], w_dev[:, :K] = to_dev(A, torch.bfloat16), to_dev(W, torch.bfloat16)
        a0, w0 = a_dev, w_dev
    else:
        a_dev, w_dev = to_dev(A, torch.bfloat16), to_dev(W, torch.bfloat16)
        a0, w0 = (a_dev, w_dev) if form == "repeated" else (a_dev[M - 1], w_dev[N - 1])   # the calls start at row 0
        A, W = (np.repeat(A[:1], M, axis=0), W) if form == "repeated" else (A[::-1], W[::-1])
    c = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    raf.raf_op_gemm(1, M, N, K, a0, lda, 1, w0, ldb, 1, c, N)
    ref = A.astype(np.float64) @ W.astype(np.float64).T
    slack = K * 2.0 ** -24 * (np.abs(A).astype(np.float64) @ np.abs(W).astype(np.float64).T) + 1e-6
    err = np.abs(host(c) - ref)
    assert (err <= 2.0 ** -8 * np.abs(ref) + slack).all(), float(err.max())


# The accurate forms on the split kernel, the one-exponential ones on a ring and on the ping-pong kernel.
@pytest.mark.parametrize("M,N,K", [(64, 64, 64), (1056, 992, 192), (1184, 3392, 192)])
def test_gemm_gelu_epilogue_at_the_ends_of_the_range(M, N, K):
    """GeLU and its derivative far from zero, at infinity and at nan: rows of zeros, so that u is the bias."""
    announce("gemm-gelu-range", M, N, K)
    bf = torch.bfloat16
    bias = torch.zeros(N)
    bias[:7] = torch.tensor([1e4, -1e4, 1e30, -1e30, float("inf"), float("nan"), 3e38])
    a, w = (torch.zeros(n, K, dtype=bf, device="cuda") for n in (M, N))
    for tanh in (0, 1):
        c, d = (torch.zeros(M, N, dtype=bf, device="cuda") for _ in range(2))
        raf.raf_op_gemm(1, M, N, K, a, K, 1, w, K, 1, c, N, epilogue=raf.EPI_BIAS_GELU_DERIV, bias=bias.cuda(), aux=d,
                        gelu_tanh=tanh)
        y, dy = host(c)[0], host(d)[0]
        want = bias.to(bf).double().numpy()
        assert np.array_equal(y[[0, 2, 4]], want[[0, 2, 4]]) and y[1] == 0 and np.isnan(y[5])
        assert dy[0] == 1 and dy[1] == 0 and np.isnan(dy[5])
        if not tanh:   # the tanh form's cubes overflow
            assert y[3] == 0 and dy[2] == 1 and dy[3] == 0 and y[6] == want[6] and dy[6] == 1
        assert np.array_equal(y[7:], np.zeros(N - 7)) and np.all(dy[7:] == 0.5)


# Products of half a k-step and of fewer than 128 rows or columns have the accurate GeLU on every kernel: in the tails, where
# the one-exponential form is off by up to 2.6e-5, each element within bf16 rounding and 4e-7 |u| (erf to 3e-7, halved, and
# float32 rounding).  Rows of zeros, so that u is the bias.
@pytest.mark.parametrize("M,N,K", [(1120, 928, 352), (1440, 2752, 352), (3968, 3072, 32), (96, 17632, 64), (64, 928, 352)])
def test_gemm_gelu_tails_of_odd_and_narrow_products(M, N, K):
    announce("gemm-gelu-tails", M, N, K)
    bf = torch.bfloat16
    a, w = (torch.zeros(n, K, dtype=bf, device="cuda") for n in (M, N))
    u = torch.linspace(-6.0, 6.0, N)
    u_bf = u.to(bf).double().numpy()
    c, aux = (torch.zeros(M, N, dtype=bf, device="cuda") for _ in range(2))

    def check(got, ref, at):
        assert (np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 4e-7 * (1.0 + np.abs(at))).all(), float(np.abs(got - ref).max())
    raf.raf_op_gemm(1, M, N, K, a, K, 1, w, K, 1, c, N, epilogue=raf.EPI_BIAS_GELU_DERIV, bias=u.cuda(), aux=aux)
    u64 = u.double().numpy()
    check(host(c), L.gelu(u64, False)[None, :], u64)
    check(host(aux), L.gelu_grad(u64, False)[None, :], u64)
    raf.raf_op_gemm(1, M, N, K, a, K, 1, w, K, 1, c, N, epilogue=raf.EPI_BIAS_GELU, bias=u.cuda(), aux=aux)
    check(host(c), L.gelu(u_bf, False)[None, :], u_bf)
    one = torch.zeros(M, K, dtype=bf, device="cuda")
    one[:, 0] = 1
    w[:, 0] = 1
    aux.copy_(u.to(bf).cuda().expand(M, N))
    raf.raf_op_gemm(1, M, N, K, one, K, 1, w, K, 1, c, N, epilogue=raf.EPI_MUL_GELU_GRAD, aux=aux)
    check(host(c), L.gelu_grad(u_bf, False)[None, :], u_bf)


# weight-gradient form (C = A^T B, both operands row-major over the contraction, float output).  Short contractions take
# the register-staged kernel; deep ones, and short ones of more than 256 tiles, the producer/consumer kernel: full 256x128
# tiles, a partial last tile in each direction, half a k-step, one and many
@pytest.mark.parametrize("M,N,K", [(256, 128, 64), (768, 768, 4096), (800, 160, 320), (2304, 768, 512),
                                   (256, 128, 32), (288, 160, 352), (128, 128, 96), (256, 128, 576), (288, 160, 544),
                                   (128, 128, 1056), (5248, 832, 32), (5152, 928, 64), (5152, 928, 352)])
def test_gemm_wgrad_form(M, N, K):
    announce("gemm-wgrad", M, N, K)
    rng = np.random.default_rng(M + 5 * N + 11 * K)
    Y = rnd(rng, (K, M), 1)
    X = rnd(rng, (K, N), 1)
    cf = torch.zeros(M, N, dtype=torch.float32, device="cuda")
    raf.raf_op_gemm(1, M, N, K, to_dev(Y, torch.bfloat16), M, 0, to_dev(X, torch.bfloat16), N, 0, cf, N, out_f32=1)
    torch.cuda.synchronize()
    ref = Y.astype(np.float64).T @ X.astype(np.float64)
    got = host(cf)
    assert rel_fro(got, ref) <= 1e-5
    assert np.max(np.abs(got - ref)) <= 1e-4 * (1.0 + np.max(np.abs(ref)))


@pytest.mark.parametrize("precision", [0, 1])
def test_gemm_epilogues_and_f32_out(precision):
    announce("gemm-epilogues", precision)
    rng = np.random.default_rng(5)
    M, N, K = 192, 160, 128
    dt = cdtype(precision)
    A, W = rnd(rng, (M, K), precision), rnd(rng, (N, K), precision, 0.1)
    bias = rng.standard_normal(N).astype(np.float32)
    a_dev, w_dev, b_dev = to_dev(A, dt), to_dev(W, dt), torch.from_numpy(bias).cuda()
    lin = A.astype(np.float64) @ W.astype(np.float64).T
    tol = 1e-5 if precision == 0 else 6e-3
    # bias
    c = torch.zeros(M, N, dtype=dt, device="cuda")
    raf.raf_op_gemm(precision, M, N, K, a_dev, K, 1, w_dev, K, 1, c, N, epilogue=raf.EPI_BIAS, bias=b_dev)
    assert rel_fro(host(c), lin + bias) <= tol
    # bias + gelu, pre-activation saved
    for tanh_form in (0, 1):
        u = torch.zeros(M, N, dtype=dt, device="cuda")
        raf.raf_op_gemm(precision, M, N, K, a_dev, K, 1, w_dev, K, 1, c, N, epilogue=raf.EPI_BIAS_GELU, bias=b_dev,
                        aux=u, gelu_tanh=tanh_form)
        assert rel_fro(host(u), lin + bias) <= tol
        assert rel_fro(host(c), L.gelu(lin + bias, bool(tanh_form))) <= 2 * tol
        # multiply by gelu'(u)
        raf.raf_op_gemm(precision, M, N, K, a_dev, K, 1, w_dev, K, 1, c, N, epilogue=raf.EPI_MUL_GELU_GRAD, aux=u,
                        gelu_tanh=tanh_form)
        assert rel_fro(host(c), lin * L.gelu_grad(host(u), bool(tanh_form))) <= 2 * tol
        # forward / backward pair that saves gelu'(pre-activation) instead of the pre-activation
        dsave = torch.zeros(M, N, dtype=dt, device="cuda")
        raf.raf_op_gemm(precision, M, N, K, a_dev, K, 1, w_dev, K, 1, c, N, epilogue=raf.EPI_BIAS_GELU_DERIV,
                        bias=b_dev, aux=dsave, gelu_tanh=tanh_form)
        assert rel_fro(host(c), L.gelu(lin + bias, bool(tanh_form))) <= 2 * tol
        assert rel_fro(host(dsave), L.gelu_grad(lin + bias, bool(tanh_form))) <= 2 * tol
        raf.raf_op_gemm(precision, M, N, K, a_dev, K, 1, w_dev, K, 1, c, N, epilogue=raf.EPI_MUL_AUX, aux=dsave)
        assert rel_fro(host(c), lin * host(dsave)) <= 2 * tol
    # residual add
    R = rnd(rng, (M, N), precision)
    r_dev = to_dev(R, dt)
    raf.raf_op_gemm(precision, M, N, K, a_dev, K, 1, w_dev, K, 1, c, N, epilogue=raf.EPI_ADD_RES, aux=r_dev)
    assert rel_fro(host(c), lin + R) <= tol
    # float output (weight-gradient form: both operands row-major over the contraction)
    X = rnd(rng, (K, N), precision)
    Y = rnd(rng, (K, M), precision)
    cf = torch.zeros(M, N, dtype=torch.float32, device="cuda")
    raf.raf_op_gemm(precision, M, N, K, to_dev(Y, dt), M, 0, to_dev(X, dt), N, 0, cf, N, out_f32=1)
    torch.cuda.synchronize()
    assert rel_fro(host(cf), Y.astype(np.float64).T @ X.astype(np.float64)) <= 1e-5


# Full-precision products at sizes where the tile choice (by rounds over 256 CUs) takes each of its tiles, with ragged
# last rows and columns and contractions that end inside a ring stage: 64x192, 64x144, 64x96, 64x64, 64x48, 32x32.
# The bound is float32 accumulation in any order: |error| <= K 2^-24 sum |a||b| per element, and per norm far less.
@pytest.mark.parametrize("ak,bk", [(1, 1), (1, 0), (0, 0), (0, 1)])
@pytest.mark.parametrize("M,N,K", [(992, 3040, 96), (992, 2272, 160), (992, 1504, 64), (992, 992, 32), (992, 736, 224),
                                   (32, 64, 288), (64, 32, 32)])
def test_gemm_f32_tiles(M, N, K, ak, bk):
    announce("gemm-f32-tiles", M, N, K, ak, bk)
    rng = np.random.default_rng(M + N + K + 2 * ak + bk)
    A, Bm = rnd(rng, (M, K), 0), rnd(rng, (K, N), 0)
    a_dev, b_dev = to_dev(A if ak else A.T, torch.float32), to_dev(Bm.T if bk else Bm, torch.float32)
    c = torch.full((M, N), float("nan"), device="cuda")
    raf.raf_op_gemm(0, M, N, K, a_dev, a_dev.shape[1], ak, b_dev, b_dev.shape[1], bk, c, N)
    torch.cuda.synchronize()
    A64, B64 = A.astype(np.float64), Bm.astype(np.float64)
    err = np.abs(host(c) - A64 @ B64)
    assert (err <= K * 2.0 ** -24 * (np.abs(A64) @ np.abs(B64))).all(), float(err.max())
    assert rel_fro(host(c), A64 @ B64) <= 1e-6


# ---------------------------------------------------------------- softmax --
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("B,S,causal,p", [(2, 32, 0, 0.0), (3, 96, 1, 0.1), (2, 128, 0, 0.1), (1, 512, 0, 0.1),
                                          (1, 1024, 1, 0.2), (1, 2048, 0, 0.1)])
def test_softmax_fwd_bwd(precision, B, S, causal, p):
    announce("softmax", precision, B, S, causal, p)
    nh = 2
    cfg = cfg_for(B, S, 64 * nh, precision, p=p, causal=causal)
    desc = raf.make_desc(cfg)
    rng = np.random.default_rng(S + causal)
    dt = cdtype(precision)
    s = rnd(rng, (B, nh, S, S), precision, 3.0)
    lens = np.array([S, max(1, S // 3), 0][:B], dtype=np.int32)     # full, ragged, and an empty sequence
    step = 11
    s_dev, lens_dev = to_dev(s, dt), torch.from_numpy(lens).cuda()
    prob, prob_d = torch.zeros_like(s_dev), torch.zeros_like(s_dev)
    raf.raf_op_softmax_fwd(desc, s_dev, lens_dev, prob, prob_d, step)
    torch.cuda.synchronize()
    masked = L.attention_masked(B, S, lens, bool(causal))
    ref = L.masked_softmax(s.astype(np.float64), masked)
    keep = dropout_keep(cfg["seed"], cfg["layer_id"], 1, step, B * nh * S * S, p).reshape(B, nh, S, S)
    got, got_d = host(prob), host(prob_d)
    assert rel_fro(got, ref) <= FWD_TOL[precision]
    assert rel_fro(got_d, ref * keep / (1 - p)) <= FWD_TOL[precision]
    assert ((got == 0) == (ref == 0)).all() or precision == 1     # structural zeros: masked entries
    assert (got[np.broadcast_to(masked, got.shape)] == 0).all()
    assert (got_d[~keep] == 0).all()
    # backward: the device works on the probabilities it saved, the reference is the oracle's adjoint on the
    # oracle's own probabilities
    dpd = rnd(rng, (B, nh, S, S), precision)
    ds = torch.zeros_like(s_dev)
    raf.raf_op_softmax_bwd(desc, prob, prob_d, to_dev(dpd, dt), ds, 0.125)
    torch.cuda.synchronize()
    ref_ds = 0.125 * L.softmax_dropout_bwd(ref, keep, 1.0 / (1 - p), dpd.astype(np.float64))
    assert rel_fro(host(ds), ref_ds) <= BWD_TOL[precision]
    assert (host(ds)[np.broadcast_to(masked, got.shape)] == 0).all()


# -------------------------------------------------------------- attention --
@pytest.mark.parametrize("B,S,nh,causal,p", [(2, 32, 1, 0, 0.0), (3, 64, 2, 1, 0.1), (3, 96, 3, 0, 0.1),
                                             (3, 128, 2, 1, 0.2), (3, 160, 2, 0, 0.1), (3, 256, 2, 1, 0.1),
                                             (2, 416, 1, 1, 0.1), (3, 512, 2, 0, 0.1), (1, 1024, 1, 1, 0.1),
                                             (2, 2048, 1, 0, 0.1), (1, 4096, 1, 1, 0.0)])
def test_attention_core_fwd_bwd(B, S, nh, causal, p):
    """The on-chip attention kernels (one block of keys for S <= 128, blockwise with running statistics beyond)
    against the oracle's attention core: context, then dQ | dK | dV, with key padding (a full, a ragged and an
    empty sequence), causal masks and dropout."""
    announce("attention", B, S, nh, causal, p)
    H = 64 * nh
    cfg = cfg_for(B, S, H, 1, p=p, causal=causal)
    desc = raf.make_desc(cfg)
    rng = np.random.default_rng(1000 * S + nh + causal)
    qkv = rnd(rng, (B * S, 3 * H), 1, 1.5)
    dctx = rnd(rng, (B * S, H), 1)
    lens = np.array([S, max(1, S // 3), 0][:B], dtype=np.int32)
    step = 5
    bf = torch.bfloat16
    qkv_d, dctx_d, lens_d = to_dev(qkv, bf), to_dev(dctx, bf), torch.from_numpy(lens).cuda()
    ctx = torch.full((B * S, H), 7.0, device="cuda", dtype=bf)
    dqkv = torch.full((B * S, 3 * H), 7.0, device="cuda", dtype=bf)
    lse = torch.zeros(B * nh * S, device="cuda", dtype=torch.float32)
    dvec = torch.zeros(B * nh * S, device="cuda", dtype=torch.float32)
    raf.raf_op_attention_fwd(desc, qkv_d, lens_d, ctx, lse, step)
    raf.raf_op_attention_bwd(desc, dctx_d, qkv_d, ctx, lse, lens_d, dqkv, dvec, step)
    torch.cuda.synchronize()
    ref_c, A = L.attention_core_forward(cfg, qkv, lens, step)
    ref_dqkv, _ = L.attention_core_backward(cfg, A, dctx)
    assert rel_fro(host(ctx), ref_c) <= FWD_TOL[1]
    got = host(dqkv)
    for blk, name in enumerate(("dQ", "dK", "dV")):
        g, r = got[:, blk * H:(blk + 1) * H], ref_dqkv[:, blk * H:(blk + 1) * H]
        assert rel_fro(g, r) <= BWD_TOL[1], name
    # the empty sequence: no admissible key, so context and every gradient of that sequence are exactly zero
    if B == 3:
        assert (host(ctx)[2 * S:] == 0).all() and (got[2 * S:] == 0).all()
    # keys beyond a sequence's length receive no gradient
    if B >= 2:
        L1 = int(lens[1])
        assert (got[S + L1:2 * S, H:] == 0).all()


@pytest.mark.parametrize("B,S,nh,causal,p", [(3, 160, 2, 0, 0.1), (3, 256, 2, 1, 0.1), (2, 416, 1, 1, 0.3),
                                             (3, 512, 2, 0, 0.2), (1, 1024, 1, 1, 0.1)])
def test_attention_keep_bits_stand_in_for_the_generator(B, S, nh, causal, p):
    """Blockwise attention with a keep buffer: the forward call leaves the keep decisions of dropout site 1 (checked
    against the mask the generator gives, wherever a key block is visited), and the backward call that reads them gives
    the results of the one that generates them again, bit for bit.  The latter is checked against the oracle above."""
    announce("attention keep bits", B, S, nh, causal, p)
    H = 64 * nh
    cfg = cfg_for(B, S, H, 1, p=p, causal=causal)
    desc = raf.make_desc(cfg)
    rng = np.random.default_rng(7000 * S + nh + causal)
    bf = torch.bfloat16
    qkv_d = to_dev(rnd(rng, (B * S, 3 * H), 1, 1.5), bf)
    dctx_d = to_dev(rnd(rng, (B * S, H), 1), bf)
    lens = np.array([S, max(1, S // 3), 0][:B], dtype=np.int32)
    lens_d = torch.from_numpy(lens).cuda()
    step = 9
    nkb = (S + 127) // 128
    nbytes = raf.raf_op_attention_keep_bytes(desc)
    assert nbytes == B * nh * S * nkb * 16
    assert raf.raf_op_attention_keep_bytes(raf.make_desc(dict(cfg, dropout_p=0.0))) == 0
    assert raf.raf_op_attention_keep_bytes(raf.make_desc(dict(cfg, seq=128))) == 0
    out = {}
    for with_keep in (False, True):
        ctx = torch.full((B * S, H), 7.0, device="cuda", dtype=bf)
        dqkv = torch.full((B * S, 3 * H), 7.0, device="cuda", dtype=bf)
        lse = torch.zeros(B * nh * S, device="cuda", dtype=torch.float32)
        dvec = torch.zeros(B * nh * S, device="cuda", dtype=torch.float32)
        keep = torch.zeros(nbytes // 4, device="cuda", dtype=torch.int32) if with_keep else None
        raf.raf_op_attention_fwd(desc, qkv_d, lens_d, ctx, lse, step, keep=keep)
        raf.raf_op_attention_bwd(desc, dctx_d, qkv_d, ctx, lse, lens_d, dqkv, dvec, step, keep=keep)
        torch.cuda.synchronize()
        out[with_keep] = (ctx, lse, dqkv, keep)
    for a, b in zip(out[False][:3], out[True][:3]):
        assert torch.equal(a, b)
    # the stored bits: bit 8u + e of dword g of (row, key block jb) is key 128 jb + 32u + 8g + e
    w = out[True][3].cpu().numpy().view(np.uint32).reshape(B, nh, S, nkb, 4)
    bits = (w[..., None] >> np.arange(32, dtype=np.uint32)) & 1              # [B, nh, S, nkb, g, 8u + e]
    bits = bits.reshape(B, nh, S, nkb, 4, 4, 8).transpose(0, 1, 2, 3, 5, 4, 6)   # -> [.., nkb, u, g, e]
    bits = bits.reshape(B, nh, S, nkb * 128)[..., :S].astype(bool)
    mask = torch.zeros(B * nh * S * S, dtype=torch.uint8, device="cuda")
    raf.raf_debug_dropout_mask(desc, 1, step, mask, mask.numel())
    mask = mask.cpu().numpy().reshape(B, nh, S, S).astype(bool)
    rows = np.arange(S)
    q_end = np.minimum((rows // 128 + 1) * 128, S)
    visited = 0
    for b in range(B):
        # key blocks the forward kernel visits for a query row: those that start below the length (and, under a
        # causal mask, below the end of the row's 128-query block)
        kmax = np.minimum(int(lens[b]), q_end) if causal else np.full(S, int(lens[b]))
        seen = (np.arange(S)[None, :] // 128 * 128) < kmax[:, None]           # [query, key]
        visited += int(seen.sum())
        for h in range(nh):
            assert (bits[b, h][seen] == mask[b, h][seen]).all(), (b, h)
            assert not bits[b, h][~seen].any()                                # never written
    assert visited > 0


# -------------------------------------------------------------- layernorm --
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("rows,H,p", [(64, 128, 0.0), (100, 768, 0.1), (37, 1024, 0.1), (9, 2048, 0.3), (5, 4096, 0.1),
                                      (33, 64, 0.1)])
def test_dropout_residual_ln_fwd_bwd(precision, rows, H, p):
    announce("ln", precision, rows, H, p)
    cfg = cfg_for(1, 32, H, precision, p=p, eps=1e-5)
    desc = raf.make_desc(cfg)
    rng = np.random.default_rng(rows + H)
    dt = cdtype(precision)
    a, res = rnd(rng, (rows, H), precision), rnd(rng, (rows, H), precision)
    gamma = (1 + 0.2 * rng.standard_normal(H)).astype(np.float32)
    beta = (0.1 * rng.standard_normal(H)).astype(np.float32)
    step, site = 4, 3
    a_d, r_d = to_dev(a, dt), to_dev(res, dt)
    g_d, b_d = torch.from_numpy(gamma).cuda(), torch.from_numpy(beta).cuda()
    out, z = torch.zeros_like(a_d), torch.zeros_like(a_d)
    mu = torch.zeros(rows, device="cuda")
    rstd = torch.zeros(rows, device="cuda")
    raf.raf_op_dropout_residual_ln_fwd(desc, site, rows, a_d, r_d, g_d, b_d, out, z, mu, rstd, step)
    torch.cuda.synchronize()
    keep = dropout_keep(cfg["seed"], cfg["layer_id"], site, step, rows * H, p).reshape(rows, H)
    z_ref = res.astype(np.float64) + a.astype(np.float64) * keep / (1 - p)
    o_ref, xhat, rstd_ref = L.layernorm(z_ref, gamma.astype(np.float64), beta.astype(np.float64), 1e-5)
    assert rel_fro(host(z), z_ref) <= FWD_TOL[precision]
    assert rel_fro(host(out), o_ref) <= FWD_TOL[precision]
    assert rel_fro(host(rstd), rstd_ref.reshape(-1)) <= FWD_TOL[precision]
    assert rel_fro(host(mu), z_ref.mean(-1)) <= FWD_TOL[precision] * 10 + 1e-6
    # variants: plain LN (no a), and no LN (gamma NULL)
    out2 = torch.zeros_like(a_d)
    raf.raf_op_dropout_residual_ln_fwd(desc, 0, rows, None, r_d, g_d, b_d, out2, None, mu, rstd, step)
    o2, _, _ = L.layernorm(res.astype(np.float64), gamma.astype(np.float64), beta.astype(np.float64), 1e-5)
    assert rel_fro(host(out2), o2) <= FWD_TOL[precision]
    out3 = torch.zeros_like(a_d)
    raf.raf_op_dropout_residual_ln_fwd(desc, site, rows, a_d, r_d, None, None, out3, None, None, None, step)
    assert rel_fro(host(out3), z_ref) <= FWD_TOL[precision]

    # backward against the adjoint of the same operator, on the z / statistics the device saved
    raf.raf_op_dropout_residual_ln_fwd(desc, site, rows, a_d, r_d, g_d, b_d, out, z, mu, rstd, step)
    dout, dout2, dres = (rnd(rng, (rows, H), precision) for _ in range(3))
    nf = raf.raf_op_ln_bwd_partial_floats(H, rows)
    assert nf > 0
    partial = torch.zeros(nf, device="cuda")
    dz, da = torch.zeros_like(a_d), torch.zeros_like(a_d)
    dg, db, dbias = (torch.zeros(H, device="cuda") for _ in range(3))
    raf.raf_op_dropout_residual_ln_bwd(desc, 2, rows, to_dev(dout, dt), to_dev(dout2, dt), z, mu, rstd, g_d,
                                       to_dev(dres, dt), dz, da, dg, db, dbias, partial, step)
    torch.cuda.synchronize()
    zz = host(z)
    _, xh, rs = L.layernorm(zz, gamma.astype(np.float64), beta.astype(np.float64), 1e-5)
    g_in = dout.astype(np.float64) + dout2
    dz_ref, dg_ref, db_ref = L.layernorm_bwd(g_in, xh, rs, gamma.astype(np.float64))
    dz_ref = dz_ref + dres
    keep2 = dropout_keep(cfg["seed"], cfg["layer_id"], 2, step, rows * H, p).reshape(rows, H)
    da_ref = dz_ref * keep2 / (1 - p)
    tol = BWD_TOL[precision]
    assert rel_fro(host(dz), dz_ref) <= tol
    assert rel_fro(host(da), da_ref) <= tol
    assert (host(da)[~keep2] == 0).all()
    assert rel_fro(host(dg), dg_ref) <= tol
    assert rel_fro(host(db), db_ref) <= tol
    assert rel_fro(host(dbias), da_ref.sum(0)) <= tol
    # no-LN variant: da = dout * keep / (1-p), column sums only
    raf.raf_op_dropout_residual_ln_bwd(desc, 3, rows, to_dev(dout, dt), None, None, None, None, None, None, None, da,
                                       None, None, dbias, partial, step)
    torch.cuda.synchronize()
    assert rel_fro(host(da), dout.astype(np.float64) * keep / (1 - p)) <= tol
    assert rel_fro(host(dbias), (dout.astype(np.float64) * keep / (1 - p)).sum(0)) <= tol


# ------------------------------------------------------------------- adam --
def test_adam_multi_tensor_matches_oracle():
    announce("adam")
    from oracle.adam import adam_step
    rng = np.random.default_rng(2)
    sizes = [1, 3, 4, 5, 4096, 4097, 16384 + 7, 768 * 64, 0, 12]
    sizes = sizes + [33 + i for i in range(60)]        # more tensors than one launch holds
    W = [rng.standard_normal(n).astype(np.float32) for n in sizes]
    Mo = [np.zeros(n, np.float32) for n in sizes]
    Vo = [np.zeros(n, np.float32) for n in sizes]
    dev = lambda a: torch.from_numpy(a.copy()).cuda()
    Wd, Md, Vd = [dev(w) for w in W], [dev(m) for m in Mo], [dev(v) for v in Vo]
    Ld = [torch.zeros(n, dtype=torch.bfloat16, device="cuda") if i % 2 == 0 else None for i, n in enumerate(sizes)]
    W64, M64, V64 = [w.astype(np.float64) for w in W], [m.astype(np.float64) for m in Mo], [v.astype(np.float64) for v in Vo]
    for t in (1, 2, 3):
        G = [(1024 * rng.standard_normal(n)).astype(np.float32) for n in sizes]
        Gd = [dev(g) for g in G]
        lst, cnt = raf.make_adam_list(zip(Wd, Gd, Md, Vd, Ld))
        raf.raf_adam_step(lst, cnt, 1e-3, 0.9, 0.999, 1e-8, 0.01, t, 1.0 / 1024)
        torch.cuda.synchronize()
        for i, n in enumerate(sizes):
            if n == 0:
                continue
            w_new, M64[i], V64[i] = adam_step(W64[i], G[i], M64[i], V64[i], t, 1e-3, 0.9, 0.999, 1e-8, 0.01, 1.0 / 1024)
            # the master weight is stored in float: the update is exact to 1e-4 of itself plus one
            # float rounding of the weight
            err = np.linalg.norm(host(Wd[i]) - w_new)
            assert err <= 1e-4 * np.linalg.norm(w_new - W64[i]) + 1.2e-7 * np.linalg.norm(w_new), (t, i)
            assert rel_fro(host(Md[i]), M64[i]) <= 1e-5 and rel_fro(host(Vd[i]), V64[i]) <= 1e-5
            W64[i] = host(Wd[i])         # continue from the stored (float-rounded) weights
            if Ld[i] is not None:    # the low-precision copy is the rounded master, bit for bit
                assert torch.equal(Ld[i], Wd[i].to(torch.bfloat16))


def test_adam_device_table_is_one_launch_with_the_same_results():
    """raf_adam_step_table (tensor table in device memory, any number of tensors in one launch) against raf_adam_step
    (table in the kernel arguments, 48 tensors per launch) on 150 tensors of odd sizes, some empty, some with a
    transposed copy: bit for bit, static and with the step count read from a scaler state."""
    import ctypes as C
    announce("adam device table")
    rng = np.random.default_rng(9)
    sizes = [(5,), (0,), (4096,), (72, 200), (33,), (4097,), (320, 1056), (0,), (768, 64)] + [(17 + 3 * i,) for i in range(141)]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()

    def build():
        ent = []
        r = np.random.default_rng(10)
        for sh in sizes:
            w, g = r.standard_normal(sh).astype(np.float32), (8 * r.standard_normal(sh)).astype(np.float32)
            m, v = (0.1 * r.standard_normal(sh)).astype(np.float32), (r.standard_normal(sh) ** 2).astype(np.float32)
            two = len(sh) == 2
            ent.append((dev(w), dev(g), dev(m), dev(v), torch.zeros(*sh, dtype=torch.bfloat16, device="cuda") if two else None,
                        torch.zeros(sh[1], sh[0], dtype=torch.bfloat16, device="cuda") if two else None))
        return ent
    for dynamic in (False, True):
        a, b = build(), build()
        la, ca = raf.make_adam_list(a)
        lb, cb = raf.make_adam_list(b)
        table = torch.zeros(raf.raf_adam_table_bytes(lb, cb), dtype=torch.uint8, device="cuda")
        raf.raf_adam_table_fill(lb, cb, table)
        state = None
        if dynamic:
            state = torch.zeros(C.sizeof(raf.ScalerState), dtype=torch.uint8, device="cuda")
            raf.raf_scaler_init(state, 8.0)
        for t in (1, 2):
            if dynamic:
                raf.raf_adam_step_scaled(la, ca, 1e-3, 0.9, 0.999, 1e-8, 0.01, state)
                raf.raf_adam_step_table(lb, cb, table, 1e-3, 0.9, 0.999, 1e-8, 0.01, 0, 0.0, state)
                raf.raf_scaler_update(state, 2.0, 0.5, 100)
            else:
                raf.raf_adam_step(la, ca, 1e-3, 0.9, 0.999, 1e-8, 0.01, t, 1.0 / 8)
                raf.raf_adam_step_table(lb, cb, table, 1e-3, 0.9, 0.999, 1e-8, 0.01, t, 1.0 / 8)
            torch.cuda.synchronize()
            for i, (ea, eb) in enumerate(zip(a, b)):
                for k in (0, 2, 3, 4, 5):
                    if ea[k] is not None:
                        assert torch.equal(ea[k], eb[k]), (dynamic, t, i, k)
            assert not torch.equal(a[2][0], torch.from_numpy(np.zeros(4096, np.float32)).cuda())


def test_adam_transposed_copy_is_the_exact_transpose_and_changes_nothing_else():
    """Tensors with a transposed bf16 copy are walked in 64 x 64 tiles: same update as the flat walk, bit for bit, the
    copy is the transpose of the bf16 weights, and elements outside ragged edge tiles are left alone."""
    announce("adam transposed copy")
    rng = np.random.default_rng(5)
    shapes = [(8, 8), (64, 64), (72, 200), (320, 1056), (768, 2304), (136, 40)]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    for t in (1, 2):
        flat, tiled = [], []
        for (r, c) in shapes:
            w = rng.standard_normal((r, c)).astype(np.float32)
            g = (64 * rng.standard_normal((r, c))).astype(np.float32)
            m = (0.1 * rng.standard_normal((r, c))).astype(np.float32)
            v = (rng.standard_normal((r, c)) ** 2).astype(np.float32)
            for dst, with_t in ((flat, False), (tiled, True)):
                wd, gd, md, vd = dev(w), dev(g), dev(m), dev(v)
                ld = torch.zeros(r, c, dtype=torch.bfloat16, device="cuda")
                # the transposed copy sits inside a guarded buffer: nothing outside [c, r] may be written
                guard = torch.full((c * r + 128,), 7.0, dtype=torch.bfloat16, device="cuda")
                dst.append((wd, gd, md, vd, ld, guard[64:64 + c * r].view(c, r) if with_t else None, guard))
        for group in (flat, tiled):
            lst, cnt = raf.make_adam_list([e[:6] for e in group])
            raf.raf_adam_step(lst, cnt, 1e-3, 0.9, 0.999, 1e-8, 0.01, t, 1.0 / 64)
        torch.cuda.synchronize()
        for a, b in zip(flat, tiled):
            for k in range(5):
                if k != 1:
                    assert torch.equal(a[k], b[k]), (t, tuple(a[0].shape), k)
            assert torch.equal(b[5], b[4].t()), (t, tuple(a[0].shape))
            assert (b[6][:64] == 7.0).all() and (b[6][-64:] == 7.0).all()
    # the matrix view must cover the tensor, with both sides multiples of 8
    wd = torch.zeros(16, 24, device="cuda")
    bad = raf.AdamTensor(wd.data_ptr(), wd.data_ptr(), wd.data_ptr(), wd.data_ptr(), None, 16 * 24, wd.data_ptr(), 16, 20)
    with pytest.raises(raf.RafError):
        raf.raf_adam_step((raf.AdamTensor * 1)(bad), 1, 1e-3, 0.9, 0.999, 1e-8, 0.0, 1, 1.0)
    bad.rows, bad.cols = 12, 32
    with pytest.raises(raf.RafError):
        raf.raf_adam_step((raf.AdamTensor * 1)(bad), 1, 1e-3, 0.9, 0.999, 1e-8, 0.0, 1, 1.0)


def test_loss_seed():
    announce("loss-seed")
    rng = np.random.default_rng(3)
    for precision in (0, 1):
        n = 64 * 128
        y, G = rnd(rng, n, precision), rnd(rng, n, precision)
        dt = cdtype(precision)
        loss = torch.zeros(1, device="cuda")
        dy = torch.zeros(n, dtype=dt, device="cuda")
        part = torch.zeros(raf.RAF_LOSS_PARTIALS, device="cuda")
        raf.raf_loss_seed(precision, to_dev(y, dt), to_dev(G, dt), n, 1024.0, loss, dy, part)
        torch.cuda.synchronize()
        ref_loss, ref_dy = L.loss_and_seed(y.astype(np.float64), G.astype(np.float64), 1024.0)
        assert abs(float(loss.item()) - ref_loss) <= 1e-5 * np.abs(y.astype(np.float64) * G).sum()
        assert np.array_equal(host(dy), ref_dy)      # power-of-two scale: exact
