"""GPU parity: every stage of the HIP path against the CPU oracle on the same
seeded inputs, through the C boundary.  Integer results (quantized tensors,
32-bit sums, token ids) must match bit for bit; float outputs are produced by
the same single-FMA formula from the same integers and are expected to be
identical, with 1e-5 relative as the stated bar.
"""
import ctypes
import functools

import numpy as np
import pytest
import torch

import oracle
import workloads
import paper_1805_12096_amd as mq

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
QT = {8: torch.int8, 16: torch.int16}


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU; there is no CPU fallback"
    mq.load_library()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def gpu_quantize(x, bits, scale=None, want_rowsum=False):
    """abs-max -> scale -> quant_int on the GPU; returns (q, scale, rowsum) device tensors."""
    xd = dev(x) if isinstance(x, np.ndarray) else x
    rows, cols = xd.shape
    s = torch.empty(1, dtype=torch.float32, device=DEV)
    if scale is None:
        mq.mq_absmax_f32(xd, xd.numel(), s)
        mq.mq_scale_from_amax(s, bits, s)
    else:
        s.fill_(float(scale))
    q = torch.empty((rows, cols), dtype=QT[bits], device=DEV)
    rs = torch.empty(rows, dtype=torch.int32, device=DEV) if (want_rowsum or bits == 16) else None
    mq.mq_quantize_f32(xd, rows, cols, bits, s, q, rs)
    return q, s, rs


def gpu_linear(A, Wt, bits, bias=None, relu=False, sA=None, sW=None, amax=False):
    pw = mq.prepare_weight(dev(Wt), bits, transposed=True,
                           scale=None if sW is None else torch.tensor([sW], dtype=torch.float32, device=DEV))
    q, s, rs = gpu_quantize(A, bits, sA)
    M, K = A.shape
    N = Wt.shape[0]
    C = torch.empty((M, N), dtype=torch.int32, device=DEV)
    mq.mq_gemm_i32(q, rs, pw.packed, bits, M, N, K, C)
    Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    am = torch.zeros(1, dtype=torch.float32, device=DEV) if amax else None
    mq.mq_gemm_dequant(q, rs, pw.packed, bits, M, N, K, s, pw.scale, None if bias is None else dev(bias),
                       relu, Y, am)
    qW = torch.empty((N, K), dtype=QT[bits], device=DEV)
    mq.mq_unpack_weight(pw.packed, bits, N, K, qW)
    return {"qA": host(q), "sA": host(s)[0], "sW": host(pw.scale)[0], "qW": host(qW), "acc": host(C),
            "Y": host(Y), "rowsum": None if rs is None else host(rs),
            "amax": None if am is None else host(am)[0]}


def assert_linear_matches(g, o):
    assert g["sA"] == o["sA"] and g["sW"] == o["sW"]
    assert np.array_equal(g["qA"], o["qA"])
    assert np.array_equal(g["qW"], o["qW"])
    assert np.array_equal(g["acc"], o["acc"])
    if g["rowsum"] is not None:
        assert np.array_equal(g["rowsum"], o["qA"].astype(np.int64).sum(1).astype(np.int32))
    tol = 1e-5 * np.abs(o["Y"]) + 1e-30
    assert np.all(np.abs(g["Y"] - o["Y"]) <= tol)
    assert np.array_equal(g["Y"], o["Y"]), "expected bit-identical float outputs"
    if g["amax"] is not None:
        assert g["amax"] == np.abs(o["Y"]).max()


# ------------------------------------------------------------------ quant_int

@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("shape", [(1, 1), (3, 7), (5, 64), (17, 513), (300, 512), (64, 2048), (1, 100003)])
def test_absmax_scale_quantize(bits, shape):
    rng = np.random.default_rng(shape[0] * 7919 + shape[1] + bits)
    x = rng.standard_normal(shape, dtype=np.float32) * np.float32(0.7)
    for rowsum in (False, True):
        q, s, rs = gpu_quantize(x, bits, want_rowsum=rowsum)
        oq, os_ = oracle.quant_int_absmax(x, bits)
        assert host(s)[0] == os_
        assert np.array_equal(host(q), oq)
        if rs is not None:
            assert np.array_equal(host(rs), oq.astype(np.int64).sum(1).astype(np.int32))


def test_quantize_fixed_multipliers_ties_clip_and_nan():
    # the paper's multipliers: 2^10 for 16 bit, 127/2 for 8 bit after clipping to [-2, 2]
    ties16 = (np.arange(-4000, 4000, dtype=np.float32) + np.float32(0.5)) / np.float32(1024)
    big = np.array([31.99, 32.0, 40.0, -40.0, 1e30, -1e30, np.inf, -np.inf, np.nan, 0.0, -0.0], dtype=np.float32)
    x = np.concatenate([ties16, big])[None, :]
    for bits, scale in [(16, 1024.0), (8, 63.5), (8, 1.0), (16, 1.0)]:
        q, _, _ = gpu_quantize(x, bits, scale=scale)
        assert np.array_equal(host(q), oracle.quant_int(x, bits, scale))
    z = np.zeros((4, 33), dtype=np.float32)
    q, s, _ = gpu_quantize(z, 8)
    assert host(s)[0] == 1.0 and not host(q).any()
    xn = np.array([[1.0, np.nan, -3.0, 2.0]], dtype=np.float32)
    q, s, _ = gpu_quantize(xn, 16)
    assert host(s)[0] == oracle.scale_from_amax(oracle.absmax(xn), 16)
    assert np.array_equal(host(q), oracle.quant_int(xn, 16, host(s)[0]))


@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("N,K", [(1, 1), (33, 65), (70, 50), (512, 512), (100, 1000)])
def test_prepare_weight_both_layouts_and_memoization(bits, N, K):
    rng = np.random.default_rng(N * 31 + K + bits)
    Wt = rng.standard_normal((N, K), dtype=np.float32) * np.float32(0.05)
    oq, os_ = oracle.quant_int_absmax(Wt, bits)
    pa = mq.prepare_weight(dev(Wt), bits, transposed=True)
    pb = mq.prepare_weight(dev(np.ascontiguousarray(Wt.T)), bits, transposed=False)
    pc = mq.prepare_weight(dev(Wt), bits, transposed=True)       # preparing again changes nothing
    assert host(pa.scale)[0] == os_ == host(pb.scale)[0]
    assert torch.equal(pa.packed, pb.packed) and torch.equal(pa.packed, pc.packed)
    q = torch.empty((N, K), dtype=QT[bits], device=DEV)
    mq.mq_unpack_weight(pa.packed, bits, N, K, q)
    assert np.array_equal(host(q), oq)
    if bits == 16:      # appended column sums
        Np = (N + 31) // 32 * 32
        cs = host(pa.packed)[-4 * Np:].view(np.int32)
        want = np.zeros(Np, dtype=np.int32)
        want[:N] = oq.astype(np.int64).sum(1)
        assert np.array_equal(cs, want)


# ------------------------------------------------------------------- dot'_int

def gpu_dot_int(qA, qB):
    """Exact integer operands through the GPU product: integers are fed as floats with multiplier 1."""
    bits = 8 if qA.dtype == np.int8 else 16
    one = torch.ones(1, dtype=torch.float32, device=DEV)
    pw = mq.prepare_weight(dev(qB.astype(np.float32)), bits, transposed=True, scale=one)
    qd = dev(qA)
    M, K = qA.shape
    N = qB.shape[0]
    rs = dev(qA.astype(np.int64).sum(1).astype(np.int32)) if bits == 16 else None
    C = torch.empty((M, N), dtype=torch.int32, device=DEV)
    mq.mq_gemm_i32(qd, rs, pw.packed, bits, M, N, K, C)
    return host(C)


SHAPES = [(1, 1, 1), (1, 5, 3), (7, 1, 16), (5, 3, 1), (32, 32, 32), (33, 31, 65), (64, 64, 64), (128, 128, 128),
          (129, 130, 80), (200, 260, 1000), (300, 70, 512), (45, 517, 96), (2, 1000, 2048)]


@pytest.mark.parametrize("dtype", [np.int8, np.int16])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_gemm_i32_full_range_integers(dtype, M, N, K):
    rng = np.random.default_rng(M * 1000003 + N * 1009 + K)
    lim = 127 if dtype == np.int8 else 32767
    qA = rng.integers(-lim, lim + 1, size=(M, K)).astype(dtype)
    qB = rng.integers(-lim, lim + 1, size=(N, K)).astype(dtype)
    want, over = oracle.dot_int(qA, qB, return_overflow=True)
    got = gpu_dot_int(qA, qB)
    assert np.array_equal(got, want)
    if dtype == np.int16 and K >= 512:
        assert over > 0          # the wrap-around path is really exercised


def test_gemm_i32_extremes_and_wrap():
    # all operands at +-32767: every sum wraps many times; int16 minimum -32768 as an A operand too
    for a, b, K in [(32767, 32767, 3), (32767, -32767, 4096), (-32768, 32767, 777), (-32768, -32767, 64)]:
        qA = np.full((40, K), a, dtype=np.int16)
        qB = np.full((37, K), b, dtype=np.int16)
        assert np.array_equal(gpu_dot_int(qA, qB), oracle.dot_int(qA, qB))
    qA = np.full((33, 100), -127, dtype=np.int8)
    qB = np.full((5, 100), 127, dtype=np.int8)
    assert np.all(gpu_dot_int(qA, qB) == -127 * 127 * 100)


def test_gemm_i32_one_hot_layout():
    # one non-zero per operand: exposes any mix-up of rows, columns or K slices
    for dtype in (np.int8, np.int16):
        M, N, K = 70, 90, 200
        for (m, n, k) in [(0, 0, 0), (69, 89, 199), (31, 32, 15), (32, 31, 16), (40, 64, 63), (5, 70, 64), (63, 33, 127)]:
            qA = np.zeros((M, K), dtype=dtype)
            qB = np.zeros((N, K), dtype=dtype)
            qA[m, k] = 3
            qB[n, k] = -5
            got = gpu_dot_int(qA, qB)
            want = np.zeros((M, N), dtype=np.int32)
            want[m, n] = -15
            assert np.array_equal(got, want), (dtype, m, n, k)


# ------------------------------------------------------------- fused epilogue

@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("M,N,K,relu,bias", [(1, 1, 1, False, True), (37, 53, 129, True, True),
                                             (130, 200, 192, False, False), (300, 512, 512, True, True),
                                             (64, 96, 2048, False, True)])
def test_linear_pipeline(bits, M, N, K, relu, bias):
    p = workloads.random_problem(M + N + K + bits, M, N, K)
    b = p["bias"] if bias else None
    o = oracle.linear(p["A"], p["Wt"], bits, b, relu)
    g = gpu_linear(p["A"], p["Wt"], bits, b, relu, amax=True)
    assert_linear_matches(g, o)


def test_linear_paper_multipliers():
    # 16 bit with 2^10 on both operands (no overflow), 8 bit with 63.5 on inputs clipped to [-2, 2]
    p = workloads.random_problem(5, 100, 150, 512, a_sigma=1.0, w_sigma=0.05)
    o = oracle.linear(p["A"], p["Wt"], 16, p["bias"], False, sA=1024.0, sW=1024.0)
    assert o["overflow_count"] == 0
    assert_linear_matches(gpu_linear(p["A"], p["Wt"], 16, p["bias"], False, sA=1024.0, sW=1024.0), o)
    A, W = np.clip(p["A"], -2, 2), np.clip(p["Wt"] * 10, -2, 2)
    o = oracle.linear(A, W, 8, p["bias"], True, sA=63.5, sW=63.5)
    assert_linear_matches(gpu_linear(A, W, 8, p["bias"], True, sA=63.5, sW=63.5), o)


def test_mq_linear_f32_is_the_composition():
    for bits in (8, 16):
        p = workloads.random_problem(77 + bits, 90, 130, 256)
        o = oracle.linear(p["A"], p["Wt"], bits, p["bias"], True)
        pw = mq.prepare_weight(dev(p["Wt"]), bits)
        M, K = p["A"].shape
        N = p["Wt"].shape[0]
        nbytes = mq.mq_linear_ws_bytes(bits, M, K)
        ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
        Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
        am = torch.zeros(1, dtype=torch.float32, device=DEV)
        mq.mq_linear_f32(dev(p["A"]), M, K, None, pw.packed, pw.scale, bits, N, dev(p["bias"]), True, Y, am, ws, nbytes)
        assert np.array_equal(host(Y), o["Y"])
        assert host(am)[0] == o["Y"].max()


@pytest.mark.parametrize("M,N,K,relu,fixed", [(300, 2048, 512, True, False), (300, 512, 512, False, False),
                                              (300, 1024, 1024, False, False), (1, 1, 32, False, False),
                                              (33, 70, 96, True, False), (512, 100, 768, False, True),
                                              (300, 512, 2048, False, False), (77, 40, 100, True, False),
                                              (290, 333, 992, True, True)])
def test_mq_linear_f32_decode_sizes(M, N, K, relu, fixed):
    # few rows, 8 bit: quant_int runs inside the product kernel when K is a multiple of 32 up to 1024
    # (the other shapes here take the separate quantizer); either way the oracle's linear layer, bit for bit
    p = workloads.random_problem(M * 7 + N * 3 + K, M, N, K)
    A = np.clip(p["A"], -2, 2) if fixed else p["A"]
    o = oracle.linear(A, p["Wt"], 8, p["bias"], relu, sA=63.5 if fixed else None)
    pw = mq.prepare_weight(dev(p["Wt"]), 8)
    nbytes = mq.mq_linear_ws_bytes(8, M, K)
    ws = torch.full((nbytes,), 0x5A, dtype=torch.uint8, device=DEV)
    Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    am = torch.zeros(1, dtype=torch.float32, device=DEV)
    sA = torch.full((1,), 63.5, dtype=torch.float32, device=DEV) if fixed else None
    for bias in (dev(p["bias"]), None):
        want = o["Y"] if bias is not None else oracle.linear(A, p["Wt"], 8, None, relu, sA=63.5 if fixed else None)["Y"]
        am.zero_()
        mq.mq_linear_f32(dev(A), M, K, sA, pw.packed, pw.scale, 8, N, bias, relu, Y, am, ws, nbytes)
        assert np.array_equal(host(Y), want)
        assert host(am)[0] == np.abs(want).max()


def test_decode_sized_products_random_shapes():
    # seeded random shapes (rows <= 512, any width, K a multiple of 32 up to 1024): the in-kernel quantizer through
    # mq_linear_f32, and the split-K / loader-wave kernels forced through the packed entry point, against the oracle
    rng = np.random.default_rng(20241127)
    qws = torch.empty(mq.mq_quantize_absmax_ws_bytes(), dtype=torch.uint8, device=DEV)
    try:
        for it in range(12):
            M, N, K = int(rng.integers(1, 513)), int(rng.integers(1, 2500)), int(rng.integers(1, 33)) * 32
            relu, fixed = bool(rng.integers(0, 2)), bool(rng.integers(0, 2))
            p = workloads.random_problem(1000 + it, M, N, K)
            A = np.clip(p["A"], -2, 2) if fixed else p["A"]
            o = oracle.linear(A, p["Wt"], 8, p["bias"], relu, sA=63.5 if fixed else None)
            pw = mq.prepare_weight(dev(p["Wt"]), 8)
            nb = mq.mq_linear_ws_bytes(8, M, K)
            ws = torch.full((nb,), 0x77, dtype=torch.uint8, device=DEV)
            Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
            am = torch.zeros(1, dtype=torch.float32, device=DEV)
            sA = torch.full((1,), 63.5, dtype=torch.float32, device=DEV) if fixed else None
            mq.mq_linear_f32(dev(A), M, K, sA, pw.packed, pw.scale, 8, N, dev(p["bias"]), relu, Y, am, ws, nb)
            assert np.array_equal(host(Y), o["Y"]), (M, N, K, relu, fixed)
            assert host(am)[0] == np.abs(o["Y"]).max()
            q = torch.empty(mq.mq_packed_bytes(8, M, K), dtype=torch.uint8, device=DEV)
            s = torch.empty(1, dtype=torch.float32, device=DEV)
            mq.mq_quantize_absmax_pack_f32(dev(p["A"]), M, K, 8, q, s, qws, qws.numel())
            o2 = oracle.linear(p["A"], p["Wt"], 8, p["bias"], relu)
            for v in (10, 11, 12, 13, 14):
                mq.mq_set_gemm_variant(v)
                mq.mq_gemm_dequant_packed(q, pw.packed, 8, M, N, K, s, pw.scale, dev(p["bias"]), relu, Y, None)
                assert np.array_equal(host(Y), o2["Y"]), (M, N, K, relu, v)
    finally:
        mq.mq_set_gemm_variant(0)


def test_mq_linear_f32_decode_sizes_special_values():
    # quant_int inside the product kernel: ties to even, clipping, infinities, NaN -> 0, an all-zero input
    M, N, K = 40, 48, 64
    rng = np.random.default_rng(4242)
    A = rng.standard_normal((M, K), dtype=np.float32)
    A[0, :8] = (np.arange(8, dtype=np.float32) + np.float32(0.5)) / np.float32(63.5)      # x * 63.5 = k + 0.5
    A[1, :6] = [np.inf, -np.inf, np.nan, 1e30, -1e30, -0.0]
    A[2, :] = 0.0
    Wt = rng.standard_normal((N, K), dtype=np.float32) * np.float32(0.05)
    bias = rng.standard_normal(N, dtype=np.float32) * np.float32(0.1)
    pw = mq.prepare_weight(dev(Wt), 8)
    nbytes = mq.mq_linear_ws_bytes(8, M, K)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    sA = torch.full((1,), 63.5, dtype=torch.float32, device=DEV)
    want = oracle.linear(A, Wt, 8, bias, False, sA=63.5)
    mq.mq_linear_f32(dev(A), M, K, sA, pw.packed, pw.scale, 8, N, dev(bias), False, Y, None, ws, nbytes)
    assert np.array_equal(host(Y), want["Y"])
    Z = np.zeros((M, K), dtype=np.float32)                     # abs-max of zeros: multiplier 1, output = bias
    mq.mq_linear_f32(dev(Z), M, K, None, pw.packed, pw.scale, 8, N, dev(bias), False, Y, None, ws, nbytes)
    assert np.array_equal(host(Y), oracle.linear(Z, Wt, 8, bias, False)["Y"])
    B = A.copy()
    B[1, :6] = [3.0, -3.0, np.nan, 2.5, -2.5, -0.0]            # abs-max skips the NaN
    mq.mq_linear_f32(dev(B), M, K, None, pw.packed, pw.scale, 8, N, dev(bias), False, Y, None, ws, nbytes)
    assert np.array_equal(host(Y), oracle.linear(B, Wt, 8, bias, False)["Y"])


@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("M,N,K,relu,fixed", [(1, 1, 4, False, False), (8, 33, 60, True, False), (9, 64, 256, False, True),
                                              (32, 31, 260, True, True), (1, 512, 512, False, False),
                                              (32, 512, 1024, False, False), (31, 70, 1028, True, False),
                                              (16, 40, 2048, False, True), (17, 40, 2044, False, False),
                                              (16, 32, 4096, False, False), (17, 32, 4096, True, False)])
def test_mq_linear_f32_of_one_row_block(M, N, K, relu, fixed, bits):
    # one launch up to 32 rows (K a multiple of 4; every edge of its waves, pieces and row counts), with NaN and
    # infinities (fixed multiplier) or NaN and a lone maximum (abs-max); an in-place call takes the separate quantizer
    p = workloads.random_problem(M * 5 + N * 3 + K + bits, M, N, K)
    A = p["A"].copy()
    A[0, 0], A[-1, -1] = np.nan, 7.25
    if fixed:
        A[-1, 1:3] = [np.inf, -np.inf]
    s0 = None if not fixed else 1024.0 if bits == 16 else 63.5
    pw = mq.prepare_weight(dev(p["Wt"]), bits)
    nb = mq.mq_linear_ws_bytes(bits, M, K)
    ws = torch.full((nb,), 0x5A, dtype=torch.uint8, device=DEV)
    am = torch.zeros(1, dtype=torch.float32, device=DEV)
    sA = torch.full((1,), s0, dtype=torch.float32, device=DEV) if fixed else None
    for bias in (p["bias"], None):
        want = oracle.linear(A, p["Wt"], bits, bias, relu, sA=s0)["Y"]
        Y = torch.full((M + 1, N), -3.0, dtype=torch.float32, device=DEV)
        am.zero_()
        mq.mq_linear_f32(dev(A), M, K, sA, pw.packed, pw.scale, bits, N, None if bias is None else dev(bias), relu, Y[:M], am, ws, nb)
        assert np.array_equal(host(Y[:M]), want) and (host(Y[M]) == -3.0).all()
        assert host(am)[0] == np.abs(want).max()
    if N == K and bits == 16:
        B = dev(A)
        mq.mq_linear_f32(B, M, K, sA, pw.packed, pw.scale, 16, N, None, relu, B, None, ws, nb)
        assert np.array_equal(host(B), want)


@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("fixed", [False, True])
@pytest.mark.parametrize("M,K", [(20, 512), (32, 256), (33, 512), (300, 512), (512, 1024), (600, 512)])
def test_mq_linear_f32_in_place(M, K, fixed, bits):
    # Y on top of A, and Y beginning in the middle of A: no workgroup may read rows that another one has already replaced,
    # whichever form serves these sizes otherwise (one launch, quant_int in the operand fetch, separate quantizer)
    p = workloads.random_problem(M + K + bits, M, K, K)
    s0 = None if not fixed else 1024.0 if bits == 16 else 63.5
    pw = mq.prepare_weight(dev(p["Wt"]), bits)
    nb = mq.mq_linear_ws_bytes(bits, M, K)
    ws = torch.full((nb,), 0x5A, dtype=torch.uint8, device=DEV)
    sA = torch.full((1,), s0, dtype=torch.float32, device=DEV) if fixed else None
    want = oracle.linear(p["A"], p["Wt"], bits, p["bias"], False, sA=s0)["Y"]
    for first in (0, M // 2):
        both = torch.zeros((M + first, K), dtype=torch.float32, device=DEV)
        both[:M] = dev(p["A"])
        mq.mq_linear_f32(both[:M], M, K, sA, pw.packed, pw.scale, bits, K, dev(p["bias"]), False, both[first:], None, ws, nb)
        assert np.array_equal(host(both[first:]), want)
        assert np.array_equal(host(both[:first]), p["A"][:first])


@pytest.mark.parametrize("bits,M,K", [(8, 20, 64), (8, 40, 64), (8, 300, 1024), (8, 600, 64), (16, 20, 64), (16, 40, 64)])
@pytest.mark.parametrize("top", [1e-38, 3e-37, 1e-42])
def test_mq_linear_f32_of_tiny_values(bits, M, K, top):
    # a maximum so small that Qmax / max is infinite: the dequantizing factor is 0 and every result its bias, whatever
    # the form that serves the size makes of the infinite products
    p = workloads.random_problem(M + K + bits, M, 48, K)
    A = np.clip(p["A"], -1, 1).astype(np.float32) * np.float32(top)
    pw = mq.prepare_weight(dev(p["Wt"]), bits)
    nb = mq.mq_linear_ws_bytes(bits, M, K)
    ws, Y = torch.empty(nb, dtype=torch.uint8, device=DEV), torch.empty((M, 48), dtype=torch.float32, device=DEV)
    mq.mq_linear_f32(dev(A), M, K, None, pw.packed, pw.scale, bits, 48, dev(p["bias"]), False, Y, None, ws, nb)
    assert np.array_equal(host(Y), np.broadcast_to(p["bias"], (M, 48)))
    assert np.array_equal(host(Y), oracle.linear(A, p["Wt"], bits, p["bias"])["Y"])


@functools.lru_cache(None)
def hip_runtime():
    """The HIP runtime this process runs on (the one torch has loaded)."""
    with open("/proc/self/maps") as f:
        return ctypes.CDLL(next(line.split()[-1] for line in f if "libamdhip64" in line))


class KernelNode(ctypes.Structure):              # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint * 3),
                ("params", ctypes.c_void_p), ("lds", ctypes.c_uint)]


def launched_grids(call):
    """(workgroups, threads of one) of the kernels that call(stream) enqueues: the nodes of a graph captured from it, after
    one call that really runs."""
    hip, graph, n = hip_runtime(), ctypes.c_void_p(), ctypes.c_size_t()
    stream = torch.cuda.Stream()
    call(stream)
    torch.cuda.synchronize()
    assert hip.hipStreamBeginCapture(ctypes.c_void_p(stream.cuda_stream), 1) == 0
    try:
        call(stream)
    finally:
        assert hip.hipStreamEndCapture(ctypes.c_void_p(stream.cuda_stream), ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    grids = []
    for node in nodes:
        k = KernelNode()
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(k)) == 0
        grids.append((k.grid[0] * k.grid[1] * k.grid[2], k.block[0]))
    assert hip.hipGraphDestroy(graph) == 0
    return grids


def launches(call):
    return len(launched_grids(call))


def tune(bits, M, N, K):
    nb = mq.mq_autotune_ws_bytes(bits, M, N, K)
    return mq.mq_autotune_gemm(bits, M, N, K, 2, torch.empty(nb, dtype=torch.uint8, device=DEV), nb)[0]


@pytest.mark.parametrize("bits,M,N,K,before,after", [(16, 11, 72, 92, 1, 3), (8, 11, 72, 92, 1, 3), (8, 11, 72, 1036, 1, 3),
                                                     (8, 11, 72, 96, 1, 1), (16, 43, 72, 92, 3, 3)])
def test_a_tuned_or_forced_variant_is_the_product_that_runs(bits, M, N, K, before, after):
    # Up to 32 rows one launch does everything, until the caller has named a packed product for the shape: then abs-max,
    # quantizer and that product run.  (8 bit with K a multiple of 32 up to 1024 never takes a packed product.)
    p = workloads.random_problem(M + N + K, M, N, K)
    pw, A = mq.prepare_weight(dev(p["Wt"]), bits), dev(p["A"])
    nb = mq.mq_linear_ws_bytes(bits, M, K)
    ws, Y = torch.empty(nb, dtype=torch.uint8, device=DEV), torch.empty((M, N), dtype=torch.float32, device=DEV)

    def call(stream):
        mq.mq_linear_f32(A, M, K, None, pw.packed, pw.scale, bits, N, None, False, Y, None, ws, nb, stream)

    want = oracle.linear(p["A"], p["Wt"], bits)["Y"]
    assert launches(call) == before and np.array_equal(host(Y), want)
    try:
        mq.mq_set_gemm_variant(1)
        Y.fill_(-3.0)
        assert launches(call) == after and np.array_equal(host(Y), want)
    finally:
        mq.mq_set_gemm_variant(0)
    tune(bits, M, N, K)
    Y.fill_(-3.0)
    assert launches(call) == after and np.array_equal(host(Y), want)


@pytest.mark.parametrize("bits,M,N,K,fixed,count", [
    (8, 32, 40, 512, True, 1), (8, 9, 40, 544, True, 1), (8, 32, 70, 1024, True, 1), (8, 9, 40, 516, True, 1),
    (8, 32, 40, 1020, True, 1), (8, 16, 40, 1028, True, 1), (8, 17, 40, 1028, True, 2), (8, 16, 40, 2048, True, 1),
    (8, 32, 40, 2048, True, 2), (8, 1, 40, 2052, True, 2), (8, 16, 40, 4096, True, 2), (8, 32, 40, 2048, False, 1),
    (8, 16, 40, 4096, False, 1), (8, 17, 40, 4096, False, 3), (16, 32, 40, 1024, True, 1), (16, 16, 40, 1028, True, 1),
    (16, 17, 40, 1028, True, 2), (16, 32, 40, 1664, True, 2), (16, 32, 40, 1668, True, 1), (16, 32, 40, 2048, False, 1)])
def test_mq_linear_f32_of_few_rows_on_both_sides_of_its_lines(bits, M, N, K, fixed, count):
    # which form serves up to 32 rows, seen by its launches, and that both sides of each line give the oracle's results
    p = workloads.random_problem(M + N + K, M, N, K)
    s0 = None if not fixed else 1024.0 if bits == 16 else 40.0
    pw, A = mq.prepare_weight(dev(p["Wt"]), bits), dev(p["A"])
    sA = torch.full((1,), s0, dtype=torch.float32, device=DEV) if fixed else None
    nb = mq.mq_linear_ws_bytes(bits, M, K)
    ws, Y = torch.full((nb,), 0x5A, dtype=torch.uint8, device=DEV), torch.full((M, N), -3.0, dtype=torch.float32, device=DEV)
    bias = dev(p["bias"])
    assert launches(lambda stream: mq.mq_linear_f32(A, M, K, sA, pw.packed, pw.scale, bits, N, bias, False, Y, None, ws, nb,
                                                    stream)) == count
    assert np.array_equal(host(Y), oracle.linear(p["A"], p["Wt"], bits, p["bias"], False, sA=s0)["Y"])


# -------------------------------------------------------------------- arg-max

def gpu_greedy(Hd, E, pw=None):
    pw = pw or mq.prepare_weight(dev(E), 8)
    q, s, _ = gpu_quantize(Hd, 8)
    M, K = Hd.shape
    N = E.shape[0]
    nbytes = mq.mq_argmax_ws_bytes(M, N)
    ws = torch.full((nbytes,), 0xAB, dtype=torch.uint8, device=DEV)     # contents must not matter
    tok = torch.empty(M, dtype=torch.int32, device=DEV)
    val = torch.empty(M, dtype=torch.float32, device=DEV)
    mq.mq_gemm_argmax(q, pw.packed, M, N, K, s, pw.scale, tok, val, ws, nbytes)
    return host(tok), host(val)


# 70 000 words are more units per workgroup than the pipeline holds stages: the loop that refills slots
@pytest.mark.parametrize("M,V,d", [(1, 1, 1), (3, 17, 8), (12, 777, 64), (33, 4100, 96), (300, 3000, 512), (130, 129, 512),
                                   (20, 70000, 64), (40, 150001, 32)])
def test_greedy_output_layer_small(M, V, d):
    c = workloads.config3(M=M, V=V, d=d, seed_extra=M + V)
    o = oracle.greedy_output_layer(c["Hd"], c["E"])
    tok, val = gpu_greedy(c["Hd"], c["E"])
    assert np.array_equal(tok, o["tok"])
    assert np.array_equal(val, o["maxlogit"])


# Row-major hidden states: widths around the streaming kernel's two sizes (512, 1024), with and without a last group of
# less than 64, beyond it (the tiled kernel), fewer and more sentences than a workgroup's chunk, more units than stages.
@pytest.mark.parametrize("M,V,d", [(1, 40, 16), (300, 3000, 1024), (257, 5000, 1008), (17, 777, 528), (600, 9000, 1024),
                                   (3, 70000, 544), (400, 2000, 496), (700, 1500, 512), (300, 3000, 1040), (33, 2000, 1023)])
def test_greedy_output_layer_row_major_widths(M, V, d):
    c = workloads.config3(M=M, V=V, d=d, seed_extra=M + V + d)
    o = oracle.greedy_output_layer(c["Hd"], c["E"])
    tok, val = gpu_greedy(c["Hd"], c["E"])
    assert np.array_equal(tok, o["tok"])
    assert np.array_equal(val, o["maxlogit"])


@pytest.mark.parametrize("d", [512, 1024])
def test_greedy_output_layer_extreme_sums(d):
    # sums of +-127 * 127 * d, the ends of the range a key's sum field holds, and ties between them
    M, V = 20, 600
    Hd = np.ones((M, d), dtype=np.float32)
    Hd[1::2] = -1
    E = np.full((V, d), -1, dtype=np.float32)
    o = oracle.greedy_output_layer(Hd, E)
    tok, val = gpu_greedy(Hd, E)
    assert np.array_equal(tok, o["tok"]) and np.array_equal(val, o["maxlogit"])
    E[[77, 78, 400]] = 1
    o = oracle.greedy_output_layer(Hd, E)
    assert o["tok"][0] == 77 and o["tok"][1] == 0 and o["acc"].max() == 127 * 127 * d
    tok, val = gpu_greedy(Hd, E)
    assert np.array_equal(tok, o["tok"]) and np.array_equal(val, o["maxlogit"])


def test_greedy_planted_winner_and_ties():
    c = workloads.config3(M=40, V=2085, d=128, seed_extra=9)
    Hd, E = c["Hd"].copy(), c["E"].copy()
    emax = np.abs(E).max()
    for m, j in [(0, 2084), (7, 5), (39, 1024)]:
        E[j] = Hd[m] * (emax / np.abs(Hd[m]).max()) * np.float32(0.999)
    # duplicates across different tiles and lanes: the lowest index has to win
    E[3] = E[1024]
    E[2080] = E[1024]
    E[1] = E[2084]
    o = oracle.greedy_output_layer(Hd, E)
    assert o["tok"][0] == 1 and o["tok"][7] == 5 and o["tok"][39] == 3
    tok, val = gpu_greedy(Hd, E)
    assert np.array_equal(tok, o["tok"]) and np.array_equal(val, o["maxlogit"])
    # all-equal logits (zero hidden state): index 0 everywhere
    tok, val = gpu_greedy(np.zeros((5, 128), dtype=np.float32), E)
    assert not tok.any() and not val.any()
    # all-negative rows: padding columns (zeros) must never win
    Hneg = np.abs(Hd[:4])
    Eneg = -np.abs(E[:70])           # 70 columns: 58 padded candidates in the last tile
    o = oracle.greedy_output_layer(Hneg, Eneg)
    assert (o["acc"] < 0).all()
    tok, val = gpu_greedy(Hneg, Eneg)
    assert np.array_equal(tok, o["tok"]) and np.array_equal(val, o["maxlogit"])


# ------------------------------------------------ benchmark workloads, full size

def test_config1_int16_single_product():
    c = workloads.config1()
    o = oracle.linear(c["A"], c["Wt"], 16, c["bias"])
    assert o["overflow_count"] > 0
    assert_linear_matches(gpu_linear(c["A"], c["Wt"], 16, c["bias"]), o)


def gpu_ffn(c, bits):
    """The launch sequence bench.py times: quantize, product+ReLU+abs-max, re-quantize, product."""
    A = dev(c["A"])
    M, d = A.shape
    f = c["W1t"].shape[0]
    p1 = mq.prepare_weight(dev(c["W1t"]), bits)
    p2 = mq.prepare_weight(dev(c["W2t"]), bits)
    b1, b2 = dev(c["b1"]), dev(c["b2"])
    s1 = torch.empty(1, dtype=torch.float32, device=DEV)
    mq.mq_absmax_f32(A, A.numel(), s1)
    mq.mq_scale_from_amax(s1, bits, s1)
    p_q1 = torch.empty(mq.mq_packed_bytes(bits, M, d), dtype=torch.uint8, device=DEV)
    mq.mq_quantize_pack_f32(A, M, d, bits, s1, p_q1)
    H = torch.empty((M, f), dtype=torch.float32, device=DEV)
    hmax = torch.zeros(1, dtype=torch.float32, device=DEV)
    mq.mq_gemm_dequant_packed(p_q1, p1.packed, bits, M, f, d, s1, p1.scale, b1, True, H, hmax)
    s2 = torch.empty(1, dtype=torch.float32, device=DEV)
    mq.mq_scale_from_amax(hmax, bits, s2)
    p_q2 = torch.empty(mq.mq_packed_bytes(bits, M, f), dtype=torch.uint8, device=DEV)
    mq.mq_quantize_pack_f32(H, M, f, bits, s2, p_q2)
    Y = torch.empty((M, d), dtype=torch.float32, device=DEV)
    mq.mq_gemm_dequant_packed(p_q2, p2.packed, bits, M, d, f, s2, p2.scale, b2, False, Y, None)
    # plain row-major views of the packed activations, for comparison with the oracle
    q1 = torch.empty((M, d), dtype=QT[bits], device=DEV)
    q2 = torch.empty((M, f), dtype=QT[bits], device=DEV)
    mq.mq_unpack_weight(p_q1, bits, M, d, q1)
    mq.mq_unpack_weight(p_q2, bits, M, f, q2)
    return {"q1": q1, "H": H, "s2": s2, "q2": q2, "Y": Y}


@functools.lru_cache(maxsize=None)
def oracle_ffn_full(cfg):
    """The oracle's whole FFN chain on ALL token rows of config 2 / config 4 (every value, the intermediate's
    multiplier included, comes from the oracle alone); computed once per test session."""
    bits = 8 if cfg == 2 else 16
    c = (workloads.config2 if cfg == 2 else workloads.config4)()
    o1 = oracle.linear(c["A"], c["W1t"], bits, c["b1"], True)
    s2 = oracle.scale_from_amax(oracle.absmax(o1["Y"]), bits)
    o2 = oracle.linear(o1["Y"], c["W2t"], bits, c["b2"], False, sA=s2)
    return c, o1, s2, o2


def oracle_ffn_rows(c, bits, rows, sA, s2):
    """Oracle on a subset of token rows, given the two per-tensor multipliers."""
    A = c["A"][rows]
    o1 = oracle.linear(A, c["W1t"], bits, c["b1"], True, sA=sA)
    o2 = oracle.linear(o1["Y"], c["W2t"], bits, c["b2"], False, sA=s2)
    return o1, o2


@pytest.mark.parametrize("cfg,bits", [(2, 8), (4, 16)])
def test_ffn_reduced_rows_full_chain(cfg, bits):
    c = (workloads.config2 if cfg == 2 else workloads.config4)(M=320)
    g = gpu_ffn(c, bits)
    o1 = oracle.linear(c["A"], c["W1t"], bits, c["b1"], True)
    s2 = oracle.scale_from_amax(oracle.absmax(o1["Y"]), bits)
    o2 = oracle.linear(o1["Y"], c["W2t"], bits, c["b2"], False, sA=s2)
    assert np.array_equal(host(g["q1"]), o1["qA"])
    assert np.array_equal(host(g["H"]), o1["Y"])
    assert host(g["s2"])[0] == s2
    assert np.array_equal(host(g["q2"]), o2["qA"])
    assert np.array_equal(host(g["Y"]), o2["Y"])


@pytest.mark.parametrize("cfg,bits", [(2, 8), (4, 16)])
def test_ffn_full_size_all_rows(cfg, bits):
    # M = 8192 as benchmarked, call by call; the oracle recomputes the whole chain on every token row and
    # supplies the intermediate's multiplier itself.
    c, o1, s2, o2 = oracle_ffn_full(cfg)
    g = gpu_ffn(c, bits)
    assert host(g["s2"])[0] == s2
    assert np.array_equal(host(g["q1"]), o1["qA"])
    assert np.array_equal(host(g["H"]), o1["Y"])
    assert np.array_equal(host(g["q2"]), o2["qA"])
    assert np.array_equal(host(g["Y"]), o2["Y"])


def test_config3_output_layer_full():
    c = workloads.config3()
    o = oracle.greedy_output_layer(c["Hd"], c["E"])
    tok, val = gpu_greedy(c["Hd"], c["E"])
    assert np.array_equal(tok, o["tok"])
    assert np.array_equal(val, o["maxlogit"])


def test_config5_decode_step_products():
    c = workloads.config5(layers=2)     # two of the six identical layers keep the oracle to seconds
    for g in c["gemms"]:
        o = oracle.linear(g["A"], g["Wt"], 8, g["bias"], g["relu"])
        r = gpu_linear(g["A"], g["Wt"], 8, g["bias"], g["relu"])
        assert np.array_equal(r["Y"], o["Y"]), g["name"]
    out = c["output"]
    o = oracle.greedy_output_layer(out["Hd"], out["E"])
    tok, val = gpu_greedy(out["Hd"], out["E"])
    assert np.array_equal(tok, o["tok"]) and np.array_equal(val, o["maxlogit"])


# ------------------------------------------- packed activations + packed product

def gpu_quantize_pack(x, bits, scale=None):
    xd = dev(x)
    rows, cols = xd.shape
    s = torch.empty(1, dtype=torch.float32, device=DEV)
    if scale is None:
        mq.mq_absmax_f32(xd, xd.numel(), s)
        mq.mq_scale_from_amax(s, bits, s)
    else:
        s.fill_(float(scale))
    packed = torch.full((mq.mq_packed_bytes(bits, rows, cols),), 0x5A, dtype=torch.uint8, device=DEV)
    mq.mq_quantize_pack_f32(xd, rows, cols, bits, s, packed)
    return packed, s


@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("shape", [(1, 1), (3, 7), (33, 65), (300, 512), (70, 2048), (257, 100), (8, 4099)])
def test_quantize_pack_matches_oracle(bits, shape):
    rng = np.random.default_rng(shape[0] * 131 + shape[1] + bits)
    x = rng.standard_normal(shape, dtype=np.float32) * np.float32(1.3)
    packed, s = gpu_quantize_pack(x, bits)
    oq, os_ = oracle.quant_int_absmax(x, bits)
    assert host(s)[0] == os_
    q = torch.empty(shape, dtype=QT[bits], device=DEV)
    mq.mq_unpack_weight(packed, bits, shape[0], shape[1], q)
    assert np.array_equal(host(q), oq)
    if bits == 16:
        Mp = (shape[0] + 31) // 32 * 32
        sums = host(packed)[-4 * Mp:].view(np.int32)
        assert np.array_equal(sums[:shape[0]], oq.astype(np.int64).sum(1).astype(np.int32))


@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("rows", [1, 8, 33])
@pytest.mark.parametrize("cols", [1, 2, 3, 4, 5, 6, 7, 9, 29, 31, 33, 62, 65, 67, 511, 513, 1022, 1157, 2050, 2307])
def test_quantizers_at_row_ends(bits, rows, cols):
    # rows that end anywhere in a vector of four, in a fragment, in a trip of four fragments, in a wave's part of K: all
    # three entry points give the oracle's integers; 8 bit: zero padding as in a prepared copy, 16 bit: the row sums, zero
    # for the padding rows
    rng = np.random.default_rng(rows * 7919 + cols * 3 + bits)
    x = rng.standard_normal((rows, cols), dtype=np.float32) * np.float32(2)
    x[-1, -1] = -9.5                                  # the largest magnitude is the last element of all
    x[rows // 2, max(cols - 3, 0)] = np.nan

    def check(packed, q):
        if bits == 8:
            one = torch.ones(1, dtype=torch.float32, device=DEV)
            assert torch.equal(packed, mq.prepare_weight(dev(q.astype(np.float32)), 8, scale=one).packed)
            return
        got = torch.empty((rows, cols), dtype=torch.int16, device=DEV)
        mq.mq_unpack_weight(packed, 16, rows, cols, got)
        assert np.array_equal(host(got), q)
        sums = np.zeros((rows + 31) // 32 * 32, dtype=np.int32)
        sums[:rows] = q.sum(1, dtype=np.int32)
        assert np.array_equal(host(packed)[-4 * len(sums):].view(np.int32), sums)

    x_inf = x.copy()                                  # a given multiplier: values beyond the range saturate
    x_inf[0, cols // 2], x_inf[-1, 0] = np.inf, -1e30
    packed, _ = gpu_quantize_pack(x_inf, bits, scale=63.5)
    check(packed, oracle.quant_int(x_inf, bits, 63.5))

    oq, os_ = oracle.quant_int_absmax(x, bits)
    xd, nb = dev(x), mq.mq_quantize_absmax_ws_bytes()
    for prepared in (False, True):
        ws = torch.full((nb,), 0x6D, dtype=torch.uint8, device=DEV)
        packed = torch.full((mq.mq_packed_bytes(bits, rows, cols),), 0x5A, dtype=torch.uint8, device=DEV)
        s = torch.empty(1, dtype=torch.float32, device=DEV)
        if prepared:
            mq.mq_quantize_absmax_ws_prepare(ws, nb)
            mq.mq_quantize_absmax_pack_f32_prepared(xd, rows, cols, bits, packed, s, ws, nb)
        else:
            mq.mq_quantize_absmax_pack_f32(xd, rows, cols, bits, packed, s, ws, nb)
        assert host(s)[0] == os_
        check(packed, oq)


@pytest.mark.parametrize("bits,rows,cols", [
    # a million elements and its neighbour; elements that fill no vector of four; both sides of twelve million; rows shared by 16
    # waves and by 4, short ones and ones of three elements in more items than the grid has waves
    (8, 1024, 1024), (16, 1024, 1024), (8, 1023, 1025), (16, 1023, 1025), (8, 2049, 2047), (16, 2049, 2047), (8, 6148, 2047),
    (16, 6147, 2047), (16, 6148, 2047), (16, 515, 4099), (8, 270001, 5), (16, 270001, 5), (8, 350003, 3), (16, 350003, 3)])
def test_absmax_and_quantizer_of_large_tensors(bits, rows, cols):
    # Two launches, the tensor dealt to the XCDs in runs of one workgroup: the largest magnitude in turn at the ends of the tensor,
    # of runs and of what fills no vector; the multiplier and, against the quantizer that is given it, every byte.
    n = rows * cols
    blocks = min((n + 2047) // 2048, 1024)
    run = (n // 4 + blocks - 1) // blocks * 4
    last = n // 4 * 4 // run * run
    x = np.random.default_rng(n + bits).standard_normal((rows, cols), dtype=np.float32).clip(-4, 4)
    xd, nb = dev(x), mq.mq_quantize_absmax_ws_bytes()
    flat = xd.view(-1)
    ws = torch.full((nb,), 0x6D, dtype=torch.uint8, device=DEV)
    got = torch.empty(mq.mq_packed_bytes(bits, rows, cols), dtype=torch.uint8, device=DEV)
    s, want = torch.empty(1, dtype=torch.float32, device=DEV), torch.empty_like(got)
    given = torch.full((1,), np.float32(127 if bits == 8 else 32767) / np.float32(9.5), dtype=torch.float32, device=DEV)
    try:
        mq.mq_set_quantize_single_pass(0)
        for at in sorted({0, 3, run - 1, run, blocks // 2 * run - 1, blocks // 2 * run, last - 1, last, n // 4 * 4 - 1, n // 4 * 4, n - 1}):
            if not 0 <= at < n:
                continue
            was = flat[at].clone()
            flat[at] = -9.5
            got.fill_(0x5A)
            mq.mq_quantize_absmax_pack_f32(xd, rows, cols, bits, got, s, ws, nb)
            mq.mq_quantize_pack_f32(xd, rows, cols, bits, given, want)
            assert torch.equal(s, given), at
            assert torch.equal(got, want), at
            flat[at] = was
        mq.mq_quantize_absmax_pack_f32(xd, rows, cols, bits, got, s, ws, nb)
    finally:
        mq.mq_set_quantize_single_pass(1)
    oq, os_ = oracle.quant_int_absmax(x, bits)
    q = torch.empty((rows, cols), dtype=QT[bits], device=DEV)
    mq.mq_unpack_weight(got, bits, rows, cols, q)
    assert host(s)[0] == os_ and np.array_equal(host(q), oq)
    if bits == 16:
        sums = host(got)[-4 * ((rows + 31) // 32 * 32):].view(np.int32)
        assert np.array_equal(sums[:rows], oq.sum(1, dtype=np.int32)) and not sums[rows:].any()


@pytest.mark.parametrize("rows", [1017, 1025, 2048, 2049])
@pytest.mark.parametrize("cols", [2047, 2052])
def test_quantize_pack_16_bit_waves_per_row_group(rows, cols):
    # 16-bit rows are shared by 16, 8 or 4 waves of a workgroup, by the number of row groups: both sides of the lines, a
    # number of fragments that 16 waves do not share evenly (the last ones get none), with and without abs-max
    rng = np.random.default_rng(rows + cols)
    x = rng.standard_normal((rows, cols), dtype=np.float32)
    oq, os_ = oracle.quant_int_absmax(x, 16)
    sums = np.zeros((rows + 31) // 32 * 32, dtype=np.int32)
    sums[:rows] = oq.sum(1, dtype=np.int32)
    nb = mq.mq_quantize_absmax_ws_bytes()
    ws, s = torch.full((nb,), 0x6D, dtype=torch.uint8, device=DEV), torch.empty(1, dtype=torch.float32, device=DEV)
    packed = torch.full((mq.mq_packed_bytes(16, rows, cols),), 0x5A, dtype=torch.uint8, device=DEV)
    try:
        mq.mq_set_quantize_single_pass(0)
        mq.mq_quantize_absmax_pack_f32(dev(x), rows, cols, 16, packed, s, ws, nb)
    finally:
        mq.mq_set_quantize_single_pass(1)
    assert host(s)[0] == os_
    for p in (packed, gpu_quantize_pack(x, 16, scale=os_)[0]):
        q = torch.empty((rows, cols), dtype=torch.int16, device=DEV)
        mq.mq_unpack_weight(p, 16, rows, cols, q)
        assert np.array_equal(host(q), oq)
        assert np.array_equal(host(p)[-4 * len(sums):].view(np.int32), sums)


def gpu_dot_int_packed(qA, qB):
    bits = 8 if qA.dtype == np.int8 else 16
    one = torch.ones(1, dtype=torch.float32, device=DEV)
    pw = mq.prepare_weight(dev(qB.astype(np.float32)), bits, transposed=True, scale=one)
    pa, _ = gpu_quantize_pack(qA.astype(np.float32), bits, scale=1.0)
    M, K = qA.shape
    N = qB.shape[0]
    C = torch.empty((M, N), dtype=torch.int32, device=DEV)
    mq.mq_gemm_i32_packed(pa, pw.packed, bits, M, N, K, C)
    return host(C)


PACKED_VARIANTS = {8: [0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14], 16: [0, 1, 2, 3, 4, 5, 6, 7, 8]}


@pytest.mark.parametrize("dtype", [np.int8, np.int16])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (33, 31, 65), (129, 130, 80), (300, 70, 512), (260, 517, 96),
                                   (2, 1000, 2048), (513, 258, 320), (300, 64, 4100), (70, 40, 9000),
                                   (320, 1030, 1024)])
def test_gemm_packed_full_range_all_variants(dtype, M, N, K):
    rng = np.random.default_rng(M * 1000003 + N * 1009 + K + 1)
    lim = 127 if dtype == np.int8 else 32767
    qA = rng.integers(-lim, lim + 1, size=(M, K)).astype(dtype)
    qB = rng.integers(-lim, lim + 1, size=(N, K)).astype(dtype)
    want = oracle.dot_int(qA, qB)
    try:
        for v in PACKED_VARIANTS[8 if dtype == np.int8 else 16]:
            mq.mq_set_gemm_variant(v)
            assert np.array_equal(gpu_dot_int_packed(qA, qB), want), f"variant {v}"
    finally:
        mq.mq_set_gemm_variant(0)


@pytest.mark.parametrize("dtype", [np.int8, np.int16])
@pytest.mark.parametrize("M,N,K", [(640, 1024, 96), (641, 1024, 96), (704, 1100, 70), (1500, 700, 160), (2049, 1024, 700),
                                   (4100, 1030, 96), (2304, 4096, 64), (3700, 1000, 2048), (4096, 1024, 1990),
                                   (504, 1030, 130), (513, 1030, 130), (1024, 1024, 96), (1025, 1024, 96), (2048, 250, 100), (2050, 250, 1000),
                                   (2050, 256, 500), (600, 878, 1100), (384, 1024, 2100), (1000, 1024, 2100)])
def test_gemm_packed_default_choice(dtype, M, N, K):
    # no forced variant: shapes on both sides of the lines where the default changes from the split-K kernel to the tiles
    # and from one tile size to the next
    rng = np.random.default_rng(M * 1009 + N + K)
    lim = 127 if dtype == np.int8 else 32767
    qA = rng.integers(-lim, lim + 1, size=(M, K)).astype(dtype)
    qB = rng.integers(-lim, lim + 1, size=(N, K)).astype(dtype)
    assert np.array_equal(gpu_dot_int_packed(qA, qB), oracle.dot_int(qA, qB))


@pytest.mark.parametrize("bits,M,N,K", [
    # up to one, two, three and more workgroups of one row block per compute unit; whole and half empty trips along K, waves
    # without a run; a last row block, column and band of tiles that are not full
    (8, 257, 1023, 511), (8, 255, 1025, 513), (8, 290, 2049, 1030), (8, 290, 2049, 1024), (8, 500, 1100, 1500), (8, 389, 1024, 4033),
    (8, 385, 700, 4096), (8, 385, 700, 3000), (8, 1409, 500, 1090), (8, 1201, 500, 1090), (8, 1217, 1056, 2100), (8, 70, 16400, 70),
    (16, 255, 1025, 500), (16, 300, 2017, 2048), (16, 260, 1025, 700), (16, 991, 1030, 530), (16, 1025, 1030, 130), (16, 40, 33, 3000)])
def test_split_k_shapes(bits, M, N, K):
    # the split-K kernels of a few hundred to a thousand rows, raw sums and dequantized with the maximum of |y|
    rng = np.random.default_rng(M * 31 + N * 7 + K + bits)
    lim = 127 if bits == 8 else 32767
    qA = rng.integers(-lim, lim + 1, size=(M, K)).astype(np.int8 if bits == 8 else np.int16)
    qB = rng.integers(-lim, lim + 1, size=(N, K)).astype(qA.dtype)
    p = workloads.random_problem(M + N + K, M, N, K)
    o = oracle.linear(p["A"], p["Wt"], bits, p["bias"], True)
    pw = mq.prepare_weight(dev(p["Wt"]), bits)
    pa, s = gpu_quantize_pack(p["A"], bits)
    Y, am = torch.empty((M, N), dtype=torch.float32, device=DEV), torch.zeros(1, dtype=torch.float32, device=DEV)
    try:
        mq.mq_set_gemm_variant(10 if bits == 8 else 6)
        assert np.array_equal(gpu_dot_int_packed(qA, qB), oracle.dot_int(qA, qB))
        mq.mq_gemm_dequant_packed(pa, pw.packed, bits, M, N, K, s, pw.scale, dev(p["bias"]), True, Y, am)
        top = o["Y"].max()
        words = [torch.full((1,), float(f * top), dtype=torch.float32, device=DEV) for f in (0.5, 2.0)]      # never lowered
        for w in words:
            mq.mq_gemm_dequant_packed(pa, pw.packed, bits, M, N, K, s, pw.scale, dev(p["bias"]), True, Y, w)
    finally:
        mq.mq_set_gemm_variant(0)
    assert np.array_equal(host(Y), o["Y"]) and host(am)[0] == top
    assert host(words[0])[0] == top and host(words[1])[0] == np.float32(2.0 * top)


@pytest.mark.parametrize("M,N,K", [(300, 2048, 512), (350, 2047, 480), (300, 2048, 1024), (330, 2040, 992), (150, 4096, 1024),
                                   (512, 2048, 1024), (250, 4090, 992), (290, 1030, 1024), (300, 4096, 1024), (32, 33000, 1024)])
@pytest.mark.parametrize("given", [False, True])
def test_quantizing_product_column_blocks(M, N, K, given):
    # quant_int in the operand fetch with one, two and three column blocks per workgroup on four and eight waves, and the
    # shapes beyond that go through the quantizer
    p = workloads.random_problem(M + N + K + 3, M, N, K)
    A = np.clip(p["A"], -2, 2)
    o = oracle.linear(A, p["Wt"], 8, p["bias"], False, sA=63.5 if given else None)
    pw = mq.prepare_weight(dev(p["Wt"]), 8)
    nb = mq.mq_linear_ws_bytes(8, M, K)
    ws, Y = torch.full((nb,), 0x77, dtype=torch.uint8, device=DEV), torch.empty((M, N), dtype=torch.float32, device=DEV)
    am = torch.zeros(1, dtype=torch.float32, device=DEV)
    sA = torch.full((1,), 63.5, dtype=torch.float32, device=DEV) if given else None
    mq.mq_linear_f32(dev(A), M, K, sA, pw.packed, pw.scale, 8, N, dev(p["bias"]), False, Y, am, ws, nb)
    assert np.array_equal(host(Y), o["Y"]) and host(am)[0] == np.abs(o["Y"]).max()


@pytest.mark.parametrize("M,N,K,count", [
    # one column block on four and on eight waves, two on eight, waves without a run, a half empty round, ragged rows and
    # columns; each with its neighbour that goes through the quantizer
    (33, 1, 32, 1), (384, 512, 512, 1), (1000, 512, 512, 1), (1025, 512, 512, 2), (70, 517, 96, 1), (70, 517, 100, 2), (200, 130, 544, 1),
    (250, 1000, 1024, 1), (500, 1024, 1024, 1), (520, 1024, 1024, 2), (290, 500, 1056, 1), (290, 510, 2048, 1), (530, 512, 2048, 2),
    (70, 60, 2080, 2)])
def test_quantizing_product_int16(M, N, K, count):
    # quant_int in the operand fetch in 16 bit: sums that wrap, ties and clipped values, infinities and NaN, max|y|; the bits of
    # the oracle, and the number of launches (without the abs-max one)
    p = workloads.random_problem(M + N + K + 5, M, N, K)
    pw = mq.prepare_weight(dev(p["Wt"]), 16)
    nb = mq.mq_linear_ws_bytes(16, M, K)
    ws, Y = torch.full((nb,), 0x77, dtype=torch.uint8, device=DEV), torch.empty((M, N), dtype=torch.float32, device=DEV)
    odd = p["A"].copy()
    odd[0, :4] = [np.nan, np.inf, -np.inf, 40.0]
    odd[M - 1, K - 1] = 0.5 / 1024
    given = torch.full((1,), 1024.0, dtype=torch.float32, device=DEV)
    for A, sA, bias, relu in ((p["A"], None, p["bias"], False), (odd, given, None, False), (p["A"] * 20, given, p["bias"], True),
                              (np.zeros_like(odd), None, p["bias"], False), (p["A"] * np.float32(1e-38), None, p["bias"], True)):
        o = oracle.linear(A, p["Wt"], 16, bias, relu, sA=None if sA is None else 1024.0)
        am = torch.zeros(1, dtype=torch.float32, device=DEV)
        Y.fill_(-3.0)
        x, b = dev(A), None if bias is None else dev(bias)

        def call(stream):
            mq.mq_linear_f32(x, M, K, sA, pw.packed, pw.scale, 16, N, b, relu, Y, am, ws, nb, stream)

        assert launches(call) == count + (sA is None)
        assert np.array_equal(host(Y), o["Y"]) and host(am)[0] == np.abs(o["Y"]).max(), (M, N, K, relu)


@pytest.mark.parametrize("bits,M,N,K,workgroups,threads", [
    (8, 384, 1024, 4096, 192, 512), (8, 512, 700, 700, 352, 512), (8, 300, 1536, 512, 480, 256), (16, 300, 1536, 512, 480, 256),
    (16, 300, 2048, 2048, 640, 256), (8, 1001, 512, 2048, 256, 512), (8, 1300, 512, 2048, 336, 512),      # split K ahead of the tiles
    (8, 5003, 100, 3000, 316, 512), (8, 8192, 128, 512, 1024, 256), (16, 5003, 100, 3000, 628, 256),      # ... few columns too
    (8, 12000, 100, 3000, 188, 256), (8, 8192, 512, 2048, 256, 256), (16, 9000, 100, 3000, 141, 256),     # tiles ahead of split K
    (16, 8192, 4096, 1024, 256, 512)])
def test_gemm_packed_default_configuration(bits, M, N, K, workgroups, threads):
    # which kernel serves shapes on which a wrong choice costs 15 % to 100 %: seen by its grid
    q = torch.zeros(mq.mq_packed_bytes(bits, M, K), dtype=torch.uint8, device=DEV)
    w = torch.zeros(mq.mq_packed_bytes(bits, N, K), dtype=torch.uint8, device=DEV)
    one, Y = torch.ones(1, dtype=torch.float32, device=DEV), torch.empty((M, N), dtype=torch.float32, device=DEV)
    got = launched_grids(lambda s: mq.mq_gemm_dequant_packed(q, w, bits, M, N, K, one, one, None, False, Y, None, s))
    assert got == [(workgroups, threads)]


@pytest.mark.parametrize("dtype", [np.int8, np.int16])
@pytest.mark.parametrize("K", [129, 192, 256, 320, 384, 448, 576, 640])
def test_gemm_packed_pipeline_boundaries_all_variants(dtype, K):
    # 3 to 10 K steps of 64: around every variant's ring depth (3, 4, 6 or 8 stages), where the main loop changes from
    # "everything issued by the prologue" to one peeled step to the steady loop
    M, N = 150, 140
    rng = np.random.default_rng(K * 7919 + (8 if dtype == np.int8 else 16))
    lim = 127 if dtype == np.int8 else 32767
    qA = rng.integers(-lim, lim + 1, size=(M, K)).astype(dtype)
    qB = rng.integers(-lim, lim + 1, size=(N, K)).astype(dtype)
    want = oracle.dot_int(qA, qB)
    try:
        for v in PACKED_VARIANTS[8 if dtype == np.int8 else 16]:
            mq.mq_set_gemm_variant(v)
            assert np.array_equal(gpu_dot_int_packed(qA, qB), want), f"variant {v}"
    finally:
        mq.mq_set_gemm_variant(0)


@pytest.mark.parametrize("M,N,K,relu", [(1, 1, 1, False), (37, 53, 64, True), (384, 512, 512, False), (130, 260, 1100, True)])
def test_int16_vector_alu_product_matches_oracle(M, N, K, relu):
    # variant 7 of the 16-bit packed products: the 16-bit dot instruction on the vector ALU instead of four 8-bit
    # matrix products.  Raw sums on full-range integers (runs of the extreme values planted, so that a pair of
    # products reaches 2 x 32767^2 and the sums wrap), then the dequantizing epilogue with bias, ReLU and the
    # abs-max by-product.
    rng = np.random.default_rng(M * 31 + N * 7 + K)
    qA = rng.integers(-32767, 32768, size=(M, K)).astype(np.int16)
    qB = rng.integers(-32767, 32768, size=(N, K)).astype(np.int16)
    qA[0, : min(K, 6)] = -32767
    qB[0, : min(K, 6)] = -32767
    qA[-1, -1], qB[-1, -1] = 32767, -32767
    p = workloads.random_problem(M + N + K + 7, M, N, K)
    o = oracle.linear(p["A"], p["Wt"], 16, p["bias"], relu)
    pw = mq.prepare_weight(dev(p["Wt"]), 16)
    pa, s = gpu_quantize_pack(p["A"], 16)
    Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    am = torch.zeros(1, dtype=torch.float32, device=DEV)
    try:
        mq.mq_set_gemm_variant(7)
        assert np.array_equal(gpu_dot_int_packed(qA, qB), oracle.dot_int(qA, qB))
        mq.mq_gemm_dequant_packed(pa, pw.packed, 16, M, N, K, s, pw.scale, dev(p["bias"]), relu, Y, am)
    finally:
        mq.mq_set_gemm_variant(0)
    assert np.array_equal(host(Y), o["Y"])
    assert host(am)[0] == np.abs(o["Y"]).max()


@pytest.mark.parametrize("M,N,K,relu,with_bias", [(4200, 2100, 200, True, True), (4097, 2049, 128, False, False),
                                                  (8200, 1100, 130, True, True), (300, 140, 1100, False, True),
                                                  (2100, 4200, 64, True, True)])
def test_int16_product_walking_through_several_tiles_matches_oracle(M, N, K, relu, with_bias):
    # variant 8 of the 16-bit packed products: one workgroup per compute unit that takes its tiles one after the other
    # and loads across tile boundaries.  The first three shapes have more 256 x 128 tiles than the chip has compute
    # units (289, 289 and 297, ragged in both directions), so workgroups take two tiles, with 4, 2 and 3 K steps per
    # tile (2 = the ring's look-ahead: every step of a tile already loads the next tile); then the one-tile case, and
    # a single K step, which the tile kernel takes over.
    rng = np.random.default_rng(M * 31 + N * 7 + K)
    qA = rng.integers(-32767, 32768, size=(M, K)).astype(np.int16)
    qB = rng.integers(-32767, 32768, size=(N, K)).astype(np.int16)
    qA[0, : min(K, 6)] = -32767
    qB[0, : min(K, 6)] = -32767
    qA[-1, -1], qB[-1, -1] = 32767, -32767
    p = workloads.random_problem(M + N + K + 8, M, N, K)
    bias = p["bias"] if with_bias else None
    o = oracle.linear(p["A"], p["Wt"], 16, bias, relu)
    pw = mq.prepare_weight(dev(p["Wt"]), 16)
    pa, s = gpu_quantize_pack(p["A"], 16)
    Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    am = torch.zeros(1, dtype=torch.float32, device=DEV)
    try:
        mq.mq_set_gemm_variant(8)
        assert np.array_equal(gpu_dot_int_packed(qA, qB), oracle.dot_int(qA, qB))
        mq.mq_gemm_dequant_packed(pa, pw.packed, 16, M, N, K, s, pw.scale, dev(bias) if with_bias else None, relu, Y, am)
    finally:
        mq.mq_set_gemm_variant(0)
    assert np.array_equal(host(Y), o["Y"])
    assert host(am)[0] == np.abs(o["Y"]).max()


def _seeded_shapes():
    rng = np.random.default_rng(2024)
    out = [(int(rng.integers(1, 1500)), int(rng.integers(1, 1500)), int(rng.integers(1, 700))) for _ in range(6)]
    out += [(int(rng.integers(3900, 4600)), int(rng.integers(2050, 2300)), int(rng.integers(65, 400))) for _ in range(4)]
    out += [(int(rng.integers(8100, 8300)), int(rng.integers(2050, 2200)), int(rng.integers(65, 200))) for _ in range(2)]
    return out


@pytest.mark.parametrize("idx,shape", list(enumerate(_seeded_shapes())))
def test_int16_walking_product_seeded_shapes(idx, shape):
    # variant 8 on shapes drawn from a seeded generator (ragged in every direction; the last six have more tiles than
    # compute units), through the library's own quantizer: 32-bit sums, dequantized outputs and max|y| against the oracle
    M, N, K = shape
    p = workloads.random_problem(1000 + idx, M, N, K)
    relu, with_bias = bool(idx % 2), idx % 3 != 0
    bias = p["bias"] if with_bias else None
    o = oracle.linear(p["A"], p["Wt"], 16, bias, relu)
    pw = mq.prepare_weight(dev(p["Wt"]), 16)
    pa, s = gpu_quantize_pack(p["A"], 16)
    Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    C = torch.empty((M, N), dtype=torch.int32, device=DEV)
    am = torch.zeros(1, dtype=torch.float32, device=DEV)
    try:
        mq.mq_set_gemm_variant(8)
        mq.mq_gemm_i32_packed(pa, pw.packed, 16, M, N, K, C)
        mq.mq_gemm_dequant_packed(pa, pw.packed, 16, M, N, K, s, pw.scale, dev(bias) if with_bias else None, relu, Y, am)
    finally:
        mq.mq_set_gemm_variant(0)
    assert np.array_equal(host(C), o["acc"])
    assert np.array_equal(host(Y), o["Y"])
    assert host(am)[0] == np.abs(o["Y"]).max()


def test_gemm_packed_one_hot_layout():
    # one non-zero per operand: checks where the direct-to-LDS copy puts each lane's bytes
    for dtype in (np.int8, np.int16):
        M, N, K = 70, 90, 200
        for (m, n, k) in [(0, 0, 0), (69, 89, 199), (31, 32, 15), (32, 31, 16), (40, 64, 63), (5, 70, 64), (63, 33, 127)]:
            qA = np.zeros((M, K), dtype=dtype)
            qB = np.zeros((N, K), dtype=dtype)
            qA[m, k] = 3
            qB[n, k] = -5
            want = np.zeros((M, N), dtype=np.int32)
            want[m, n] = -15
            assert np.array_equal(gpu_dot_int_packed(qA, qB), want), (dtype, m, n, k)


@pytest.mark.parametrize("M,N,K,relu", [(37, 53, 64, True), (300, 200, 320, False), (513, 258, 448, True),
                                        (1000, 130, 2048, False), (129, 512, 4100, True)])
def test_linear_pipeline_packed_k_split_over_wave_groups(M, N, K, relu):
    # variant 14: an odd number of 64-element K steps leaves the second wave group's last step empty; the
    # dequantizing epilogue with bias, ReLU and the abs-max by-product runs on the first group only
    p = workloads.random_problem(M + N + K + 14, M, N, K)
    o = oracle.linear(p["A"], p["Wt"], 8, p["bias"], relu)
    pw = mq.prepare_weight(dev(p["Wt"]), 8)
    pa, s = gpu_quantize_pack(p["A"], 8)
    Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    am = torch.zeros(1, dtype=torch.float32, device=DEV)
    try:
        mq.mq_set_gemm_variant(14)
        mq.mq_gemm_dequant_packed(pa, pw.packed, 8, M, N, K, s, pw.scale, dev(p["bias"]), relu, Y, am)
    finally:
        mq.mq_set_gemm_variant(0)
    assert np.array_equal(host(Y), o["Y"])
    assert host(am)[0] == np.abs(o["Y"]).max()


@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("M,N,K,relu", [(37, 53, 129, True), (300, 512, 512, True), (520, 300, 1024, False)])
def test_linear_pipeline_packed(bits, M, N, K, relu):
    p = workloads.random_problem(M + N + K + bits + 3, M, N, K)
    o = oracle.linear(p["A"], p["Wt"], bits, p["bias"], relu)
    pw = mq.prepare_weight(dev(p["Wt"]), bits)
    pa, s = gpu_quantize_pack(p["A"], bits)
    Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    am = torch.zeros(1, dtype=torch.float32, device=DEV)
    mq.mq_gemm_dequant_packed(pa, pw.packed, bits, M, N, K, s, pw.scale, dev(p["bias"]), relu, Y, am)
    assert np.array_equal(host(Y), o["Y"])
    assert host(am)[0] == np.abs(o["Y"]).max()


# ------------------------------------------------ decode-step arg-max kernel

def gpu_greedy_packed(Hd, E):
    pw = mq.prepare_weight(dev(E), 8)
    pa, s = gpu_quantize_pack(Hd, 8)
    M, K = Hd.shape
    N = E.shape[0]
    nbytes = mq.mq_argmax_ws_bytes(M, N)
    ws = torch.full((nbytes,), 0xCD, dtype=torch.uint8, device=DEV)     # contents must not matter
    tok = torch.full((M,), -7, dtype=torch.int32, device=DEV)
    val = torch.empty(M, dtype=torch.float32, device=DEV)
    mq.mq_gemm_argmax_packed(pa, pw.packed, M, N, K, s, pw.scale, tok, val, ws, nbytes)
    return host(tok), host(val)


@pytest.mark.parametrize("M,V,d", [(1, 1, 1), (3, 17, 8), (12, 777, 64), (33, 4100, 96), (130, 129, 512), (300, 3000, 512),
                                   (384, 9000, 192), (97, 20000, 128), (257, 33, 300), (320, 5000, 448),
                                   (261, 40000, 512)])
def test_greedy_packed_small(M, V, d):
    c = workloads.config3(M=M, V=V, d=d, seed_extra=M + V + 5)
    o = oracle.greedy_output_layer(c["Hd"], c["E"])
    tok, val = gpu_greedy_packed(c["Hd"], c["E"])
    assert np.array_equal(tok, o["tok"])
    assert np.array_equal(val, o["maxlogit"])


def test_greedy_packed_ties_padding_and_limits():
    c = workloads.config3(M=40, V=9000, d=128, seed_extra=11)
    Hd, E = c["Hd"].copy(), c["E"].copy()
    emax = np.abs(E).max()
    for m, j in [(0, 8999), (7, 5), (39, 4096)]:
        E[j] = Hd[m] * (emax / np.abs(Hd[m]).max()) * np.float32(0.999)
    E[3] = E[4096]          # duplicates in other vocabulary blocks, handled by other workgroups
    E[8990] = E[4096]
    E[1] = E[8999]
    o = oracle.greedy_output_layer(Hd, E)
    assert o["tok"][0] == 1 and o["tok"][7] == 5 and o["tok"][39] == 3
    tok, val = gpu_greedy_packed(Hd, E)
    assert np.array_equal(tok, o["tok"]) and np.array_equal(val, o["maxlogit"])
    tok, val = gpu_greedy_packed(np.zeros((5, 128), dtype=np.float32), E)
    assert not tok.any() and not val.any()
    Hneg, Eneg = np.abs(Hd[:4]), -np.abs(E[:70])      # all sums negative: zero padding must never win
    o = oracle.greedy_output_layer(Hneg, Eneg)
    tok, val = gpu_greedy_packed(Hneg, Eneg)
    assert np.array_equal(tok, o["tok"]) and np.array_equal(val, o["maxlogit"])
    # beyond the kernel's limits the call refuses instead of computing something else
    # (K = 576 > 512: the 32-bit keys of the streaming kernel could no longer hold the sums)
    wide = np.zeros((64, 576), dtype=np.float32)
    pw = mq.prepare_weight(dev(wide), 8)
    pa, s = gpu_quantize_pack(np.zeros((5, 576), dtype=np.float32), 8)
    nbytes = mq.mq_argmax_ws_bytes(5, 64)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    tok_t = torch.empty(5, dtype=torch.int32, device=DEV)
    val_t = torch.empty(5, dtype=torch.float32, device=DEV)
    with pytest.raises(mq.MqError) as e:
        mq.mq_gemm_argmax_packed(pa, pw.packed, 5, 64, 576, s, pw.scale, tok_t, val_t, ws, nbytes)
    assert e.value.status == 6


def test_config3_output_layer_full_packed():
    c = workloads.config3()
    o = oracle.greedy_output_layer(c["Hd"], c["E"])
    tok, val = gpu_greedy_packed(c["Hd"], c["E"])
    assert np.array_equal(tok, o["tok"])
    assert np.array_equal(val, o["maxlogit"])


def test_greedy_packed_more_rows_than_one_pass_holds():
    # 1000 rows: three chunks of rows in one launch, each over a third of the compute units
    c = workloads.config3(M=1000, V=5000, d=128, seed_extra=11)
    o = oracle.greedy_output_layer(c["Hd"], c["E"])
    tok, val = gpu_greedy_packed(c["Hd"], c["E"])
    assert np.array_equal(tok, o["tok"])
    assert np.array_equal(val, o["maxlogit"])


@pytest.mark.parametrize("M", [1, 33])
@pytest.mark.parametrize("columns", [1, 2, 15, 16, 17, 63, 64, 65, 240, 256])
def test_greedy_packed_every_column_of_candidates_counts(columns, M):
    # 16 words to a workgroup (up to 256 workgroups): the number of keys the reducing kernel loads goes by that count.
    # The best word of sentence m sits in another workgroup's share for each m, the last one's included.
    rng = np.random.default_rng(columns)
    V, d = 16 * columns - 3, 64
    Hd, E = rng.standard_normal((M, d), dtype=np.float32), rng.standard_normal((V, d), dtype=np.float32)
    for m in range(min(M, V)):
        E[V - 1 - m * V // M] = 3 * Hd[m]
    o = oracle.greedy_output_layer(Hd, E)
    tok, val = gpu_greedy_packed(Hd, E)
    assert np.array_equal(tok, o["tok"]) and np.array_equal(val, o["maxlogit"])


@pytest.mark.parametrize("M,V,d", [(6145, 300, 64), (6144 + 390, 4100, 96), (2 * 6144 + 1, 33, 32), (128 * 384 + 33, 33, 32)])
def test_greedy_packed_more_rows_than_one_launch_holds(M, V, d):
    # up to 128 chunks of 384 rows per launch: the launch behind the first one starts at a later row of the hidden states
    # and of both results, and reuses the workspace
    c = workloads.config3(M=M, V=V, d=d, seed_extra=M)
    o = oracle.greedy_output_layer(c["Hd"], c["E"])
    tok, val = gpu_greedy_packed(c["Hd"], c["E"])
    assert np.array_equal(tok, o["tok"])
    assert np.array_equal(val, o["maxlogit"])
    sl = np.arange(0, V, 3, dtype=np.int32)
    o = oracle.greedy_output_layer(c["Hd"], c["E"], shortlist=sl)
    tok, val = gpu_greedy_shortlist(c["Hd"], c["E"], sl)
    assert np.array_equal(tok, o["tok"])
    assert np.array_equal(val, o["maxlogit"])


@pytest.mark.parametrize("M,V,d,form", [(800, 400000, 16, "shortlist"), (800, 400000, 16, "packed"), (400, 270000, 528, "rows"),
                                        (800, 400000, 256, "rows")])
def test_greedy_vocabularies_that_leave_few_chunks_to_a_launch(M, V, d, form):
    # So many words that a chunk of rows needs a large share of the compute units: its neighbours go in launches of their own,
    # at a later row of the hidden states and of both results.  Checked against the oracle where the launches meet.
    rng = np.random.default_rng(V + d)
    Hd, E = rng.standard_normal((M, d), dtype=np.float32), rng.standard_normal((V, d), dtype=np.float32)
    if form == "rows":
        pw = mq.prepare_weight(dev(E), 8)
        q, s, _ = gpu_quantize(Hd, 8)
        nb = mq.mq_argmax_ws_bytes(M, V)
        ws = torch.full((nb,), 0xAB, dtype=torch.uint8, device=DEV)
        t, v = torch.empty(M, dtype=torch.int32, device=DEV), torch.empty(M, dtype=torch.float32, device=DEV)
        assert launches(lambda st: mq.mq_gemm_argmax(q, pw.packed, M, V, d, s, pw.scale, t, v, ws, nb, st)) >= 4
        tok, val = host(t), host(v)
    elif form == "packed":
        tok, val = gpu_greedy_packed(Hd, E)
    else:
        tok, val = gpu_greedy_shortlist(Hd, E, np.arange(V, dtype=np.int32))
    (qA, sA), (qW, sW) = oracle.quant_int_absmax(Hd, 8), oracle.quant_int_absmax(E, 8)
    for m in (0, 250, 380, 508, M - 8):                 # (chunks of 256 rows above a width of 512, of 384 up to it)
        want_tok, want_val = oracle.argmax_i32(oracle.dot_int(qA[m:m + 8], qW), sA, sW)
        assert np.array_equal(tok[m:m + 8], want_tok) and np.array_equal(val[m:m + 8], want_val)


@pytest.mark.parametrize("M,V,d,count", [(300, 3000, 1024, 2), (600, 9000, 1024, 3), (1000, 3000, 128, 3), (100, 2000, 128, 2),
                                         (385, 2500, 512, 2), (384, 2500, 512, 3), (200, 300, 640, 3), (17, 777, 528, 2),
                                         (257, 1777, 16, 3), (1023, 129, 48, 3), (900, 10000, 64, 3), (300, 20000, 512, 2)])
def test_greedy_row_major_takes_the_shorter_form(M, V, d, count):
    # the streaming kernel and its reduction (two launches) or the tiled product (three), ties planted in either
    rng = np.random.default_rng(M + V + d)
    Hd, E = rng.standard_normal((M, d), dtype=np.float32), rng.standard_normal((V, d), dtype=np.float32)
    E[V - 2] = E[V // 3]                                # equal sums: the lower index wins
    Hd[M // 2] = 4 * E[V // 3]
    pw = mq.prepare_weight(dev(E), 8)
    q, s, _ = gpu_quantize(Hd, 8)
    nb = mq.mq_argmax_ws_bytes(M, V)
    ws = torch.full((nb,), 0xAB, dtype=torch.uint8, device=DEV)
    tok, val = torch.empty(M, dtype=torch.int32, device=DEV), torch.empty(M, dtype=torch.float32, device=DEV)
    assert launches(lambda st: mq.mq_gemm_argmax(q, pw.packed, M, V, d, s, pw.scale, tok, val, ws, nb, st)) == count
    o = oracle.greedy_output_layer(Hd, E)
    assert np.array_equal(host(tok), o["tok"]) and np.array_equal(host(val), o["maxlogit"])
    assert host(tok)[M // 2] == V // 3


# ----------------------------------------------------------- fused FFN (8 bit)

def gpu_ffn_fused(c):
    A = dev(c["A"])
    M, d = A.shape
    f = c["W1t"].shape[0]
    p1 = mq.prepare_weight(dev(c["W1t"]), 8)
    p2 = mq.prepare_weight(dev(c["W2t"]), 8)
    nbytes = mq.mq_ffn_ws_bytes(M, d, f)
    ws = torch.full((nbytes,), 0x3C, dtype=torch.uint8, device=DEV)     # contents must not matter
    Y = torch.empty((M, d), dtype=torch.float32, device=DEV)
    mq.mq_ffn_i8_f32(A, M, d, f, p1.packed, p1.scale, dev(c["b1"]), p2.packed, p2.scale, dev(c["b2"]), Y, ws, nbytes)
    return host(Y)


@pytest.mark.parametrize("M,d,f", [(1, 1, 1), (37, 64, 200), (320, 512, 2048), (130, 96, 100), (513, 256, 384)])
def test_ffn_fused_matches_oracle_chain(M, d, f):
    c = workloads.ffn(2, M, d, f, 0.04, 8, seed_extra=M + d + f)
    o1 = oracle.linear(c["A"], c["W1t"], 8, c["b1"], True)
    s2 = oracle.scale_from_amax(oracle.absmax(o1["Y"]), 8)
    o2 = oracle.linear(o1["Y"], c["W2t"], 8, c["b2"], False, sA=s2)
    for v in (0, 1, 3, 4, 5, 7):
        try:
            mq.mq_set_gemm_variant(v)
            assert np.array_equal(gpu_ffn_fused(c), o2["Y"]), f"variant {v}"
        finally:
            mq.mq_set_gemm_variant(0)


@pytest.mark.parametrize("M,d,f", [(37, 64, 200), (700, 128, 600), (4352, 64, 4096)])
def test_ffn_single_pass_and_two_pass_agree_with_oracle(M, d, f):
    # The intermediate's multiplier needs max|H| over the whole tensor: one launch with a grid-wide
    # barrier when every tile is resident at once, two passes otherwise (the last shape has 272
    # tiles of 256 x 256, more than the chip holds).  Repeated calls reuse the workspace's counter.
    c = workloads.ffn(2, M, d, f, 0.04, 8, seed_extra=M + 2 * d + f)
    o1 = oracle.linear(c["A"], c["W1t"], 8, c["b1"], True)
    s2 = oracle.scale_from_amax(oracle.absmax(o1["Y"]), 8)
    o2 = oracle.linear(o1["Y"], c["W2t"], 8, c["b2"], False, sA=s2)
    try:
        for single in (1, 0, 1, 1):
            mq.mq_set_ffn_single_pass(single)
            assert np.array_equal(gpu_ffn_fused(c), o2["Y"]), f"single_pass={single}"
    finally:
        mq.mq_set_ffn_single_pass(1)


@pytest.mark.parametrize("bits,M,d,f", [(16, 70, 64, 600), (16, 70, 68, 600), (8, 700, 128, 600)])
def test_a_variant_named_by_another_thread_changes_no_result(bits, M, d, f):
    # Calls in which more than one launch depends on the product's configuration, while another thread forces one and takes it
    # back: who leaves the maxima of the intermediate (16 bit: the split-K kernel one a workgroup, the tiles in words of their
    # own; widths that are no multiple of 32, as others may quantize in the product's operand fetch and then look at no
    # configuration again) and how many there are (8 bit in two passes: one a tile) is settled once.
    import threading
    c = workloads.ffn(2 if bits == 8 else 4, M, d, f, 0.04, bits, seed_extra=M + f)
    W1, W2 = (mq.prepare_weight(dev(c[n]), bits) for n in ("W1t", "W2t"))
    A, b1, b2 = dev(c["A"]), dev(c["b1"]), dev(c["b2"])
    call, need = (mq.mq_ffn_i8_f32, mq.mq_ffn_ws_bytes) if bits == 8 else (mq.mq_ffn_i16_f32, mq.mq_ffn_i16_ws_bytes)
    nb = need(M, d, f)
    ws = torch.full((nb,), 0x7F, dtype=torch.uint8, device=DEV)         # (words nobody wrote: 3.4e38 as a maximum)
    Y, wrong = torch.empty((M, d), dtype=torch.float32, device=DEV), torch.zeros((), dtype=torch.int64, device=DEV)
    args = (A, M, d, f, W1.packed, W1.scale, b1, W2.packed, W2.scale, b2, Y, ws, nb)
    done = threading.Event()

    def name_variants():
        while not done.is_set():
            mq.mq_set_gemm_variant(1)
            mq.mq_set_gemm_variant(0)

    other = threading.Thread(target=name_variants)
    try:
        mq.mq_set_ffn_single_pass(0)
        call(*args)
        want = Y.clone()
        other.start()
        for _ in range(3000):
            call(*args)
            wrong += (Y != want).any()
    finally:
        done.set()
        if other.ident is not None:
            other.join()
        mq.mq_set_gemm_variant(0)
        mq.mq_set_ffn_single_pass(1)
    assert int(wrong) == 0


@pytest.mark.parametrize("M,d,f", [(1, 1, 1), (37, 64, 200), (300, 256, 520), (2100, 512, 96), (1, 32, 16400), (64, 1024, 4096),
                                   (250, 512, 2048), (129, 1024, 300)])
def test_ffn_int16_one_call_matches_oracle_chain(M, d, f):
    c = workloads.ffn(4, M, d, f, 0.03, 16, seed_extra=M + d + 3 * f)
    o1 = oracle.linear(c["A"], c["W1t"], 16, c["b1"], True)
    s2 = oracle.scale_from_amax(oracle.absmax(o1["Y"]), 16)
    o2 = oracle.linear(o1["Y"], c["W2t"], 16, c["b2"], False, sA=s2)
    A = dev(c["A"])
    p1 = mq.prepare_weight(dev(c["W1t"]), 16)
    p2 = mq.prepare_weight(dev(c["W2t"]), 16)
    nbytes = mq.mq_ffn_i16_ws_bytes(M, d, f)
    ws = torch.full((nbytes,), 0x3C, dtype=torch.uint8, device=DEV)     # contents must not matter
    for _ in range(2):
        Y = torch.empty((M, d), dtype=torch.float32, device=DEV)
        mq.mq_ffn_i16_f32(A, M, d, f, p1.packed, p1.scale, dev(c["b1"]), p2.packed, p2.scale, dev(c["b2"]), Y, ws,
                          nbytes)
        assert np.array_equal(host(Y), o2["Y"])


@pytest.mark.parametrize("M,d,f,count", [
    # quant_int in the first product's operand fetch (22 x 10 workgroups of the 256 allowed in the third); widths and numbers of
    # workgroups (29 x 10) that refuse it; of these, inputs of a million elements that one kernel quantizes (the last two: ragged
    # rows and columns)
    (37, 64, 200, 4), (70, 64, 600, 4), (300, 256, 520, 4), (700, 1024, 600, 4), (37, 68, 200, 5), (70, 68, 600, 5), (300, 260, 520, 5),
    (900, 1024, 600, 5), (1100, 500, 700, 5), (2100, 520, 96, 5), (3001, 512, 2048, 5)])
def test_ffn_int16_launches_and_oracle_chain(M, d, f, count):
    # which launches a call takes, with and without the kernels that wait, and the oracle's bits either way
    c = workloads.ffn(4, M, d, f, 0.03, 16, seed_extra=M + d + 3 * f)
    o1 = oracle.linear(c["A"], c["W1t"], 16, c["b1"], True)
    s2 = oracle.scale_from_amax(oracle.absmax(o1["Y"]), 16)
    o2 = oracle.linear(o1["Y"], c["W2t"], 16, c["b2"], False, sA=s2)
    A, b1, b2 = dev(c["A"]), dev(c["b1"]), dev(c["b2"])
    p1, p2 = (mq.prepare_weight(dev(c[n]), 16) for n in ("W1t", "W2t"))
    nb = mq.mq_ffn_i16_ws_bytes(M, d, f)
    ws, Y = torch.full((nb,), 0x3C, dtype=torch.uint8, device=DEV), torch.empty((M, d), dtype=torch.float32, device=DEV)

    def call(stream):
        mq.mq_ffn_i16_f32(A, M, d, f, p1.packed, p1.scale, b1, p2.packed, p2.scale, b2, Y, ws, nb, stream)

    absmax = min((M * d + 2047) // 2048, 1024)         # workgroups of an abs-max launch; the other first launch clears a few words
    try:
        for single in (1, 0):
            mq.mq_set_ffn_single_pass(single)
            Y.fill_(-3.0)
            grids = launched_grids(call)
            assert len(grids) == count
            assert (grids[0][0] != absmax) == (count == 5 and single == 1 and M * d >= 2 ** 20)
            assert np.array_equal(host(Y), o2["Y"])
    finally:
        mq.mq_set_ffn_single_pass(1)


def test_ffn_fused_full_size_equals_oracle_on_all_rows():
    # the one-call int8 block at M = 8192 against the oracle's whole chain, every row
    c, _, _, o2 = oracle_ffn_full(2)
    assert np.array_equal(gpu_ffn_fused(c), o2["Y"])


def test_ffn_int16_one_call_full_size_equals_oracle_on_all_rows():
    # mq_ffn_i16_f32 at the benchmark's 8192 x 1024 x 4096 against the oracle's whole chain, every row
    c, _, _, o2 = oracle_ffn_full(4)
    M, d = c["A"].shape
    f = c["W1t"].shape[0]
    p1 = mq.prepare_weight(dev(c["W1t"]), 16)
    p2 = mq.prepare_weight(dev(c["W2t"]), 16)
    nbytes = mq.mq_ffn_i16_ws_bytes(M, d, f)
    ws = torch.full((nbytes,), 0x3C, dtype=torch.uint8, device=DEV)
    Y = torch.empty((M, d), dtype=torch.float32, device=DEV)
    mq.mq_ffn_i16_f32(dev(c["A"]), M, d, f, p1.packed, p1.scale, dev(c["b1"]), p2.packed, p2.scale, dev(c["b2"]), Y, ws,
                      nbytes)
    assert np.array_equal(host(Y), o2["Y"])


def capture_graph(fn, reps):
    """HIP graph of `reps` consecutive calls of fn, captured the way bench.py does it."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        fn()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(reps):
            fn()
    return g


def test_ffn_block_replayed_as_a_graph_of_several_steps():
    # the launch configuration bench.py times: graphs of consecutive mq_ffn_i8_f32 calls at config 2's size.
    # Every replay (with eager work of the program's own and synchronizations in between, and a different input
    # each time) must give the eager call's bits; the eager result is pinned to the oracle on sampled rows.
    c = workloads.config2()
    M, d = c["A"].shape
    f = c["W1t"].shape[0]
    p1 = mq.prepare_weight(dev(c["W1t"]), 8)
    p2 = mq.prepare_weight(dev(c["W2t"]), 8)
    b1, b2 = dev(c["b1"]), dev(c["b2"])
    nbytes = mq.mq_ffn_ws_bytes(M, d, f)
    ws = torch.full((nbytes,), 0x3C, dtype=torch.uint8, device=DEV)
    A = dev(c["A"])
    Y = torch.empty((M, d), dtype=torch.float32, device=DEV)

    def step():
        mq.mq_ffn_i8_f32(A, M, d, f, p1.packed, p1.scale, b1, p2.packed, p2.scale, b2, Y, ws, nbytes)

    g = capture_graph(step, 3)
    base = dev(c["A"])
    for r, factor in enumerate((1.0, 0.5, -1.25, 1.0)):
        A.copy_(base * factor)                       # eager work between the replays
        step()
        torch.cuda.synchronize()
        want = Y.clone()
        Y.fill_(float("nan"))
        ws.fill_(0xA7 + r)                           # the workspace's contents must not matter either
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, want), f"replay {r}"
    _, _, _, o2 = oracle_ffn_full(2)               # the last replay ran on the unscaled input
    assert np.array_equal(host(Y), o2["Y"])


@pytest.mark.parametrize("M,d,f", [(1, 1, 1), (37, 64, 200), (320, 512, 2048), (2048, 512, 2048), (2048, 512, 16384),
                                   (2100, 512, 300), (8192, 512, 2048)])
def test_ffn_block_on_a_prepared_workspace(M, d, f):
    # mq_ffn_ws_prepare once, then calls that leave the agreement words as they found them: repeated calls with
    # changing inputs, the plain entry point mixed in, both switch positions of the single-pass kernels.  The
    # sizes cover: nothing single-pass (small), single-pass product only, both single-pass kernels (the last
    # ones), and a first product too large for one launch behind a single-pass quantizer (f = 16384).
    c = workloads.ffn(2, M, d, f, 0.04, 8, seed_extra=M + d + f + 5)
    p1 = mq.prepare_weight(dev(c["W1t"]), 8)
    p2 = mq.prepare_weight(dev(c["W2t"]), 8)
    b1, b2 = dev(c["b1"]), dev(c["b2"])
    nbytes = mq.mq_ffn_ws_bytes(M, d, f)
    ws = torch.full((nbytes,), 0x5B, dtype=torch.uint8, device=DEV)
    ws_plain = torch.full((nbytes,), 0x11, dtype=torch.uint8, device=DEV)
    Y = torch.empty((M, d), dtype=torch.float32, device=DEV)
    W = torch.empty((M, d), dtype=torch.float32, device=DEV)
    base = dev(c["A"])
    A = base.clone()
    mq.mq_ffn_ws_prepare(ws, nbytes, M, d, f)
    try:
        for r, (factor, kind) in enumerate([(1.0, "p"), (0.5, "p"), (-2.0, "plain"), (3.0, "p"), (1.0, "off"), (0.25, "p"),
                                            (1.0, "p")]):
            A.copy_(base * factor)
            mq.mq_ffn_i8_f32(A, M, d, f, p1.packed, p1.scale, b1, p2.packed, p2.scale, b2, W, ws_plain, nbytes)
            Y.fill_(float("nan"))
            if kind == "plain":        # the plain entry point on the prepared workspace: leaves it prepared
                mq.mq_ffn_i8_f32(A, M, d, f, p1.packed, p1.scale, b1, p2.packed, p2.scale, b2, Y, ws, nbytes)
            else:
                mq.mq_set_ffn_single_pass(0 if kind == "off" else 1)
                mq.mq_ffn_i8_f32_prepared(A, M, d, f, p1.packed, p1.scale, b1, p2.packed, p2.scale, b2, Y, ws, nbytes)
                mq.mq_set_ffn_single_pass(1)
            torch.cuda.synchronize()
            assert torch.equal(Y, W), f"call {r} ({kind})"
    finally:
        mq.mq_set_ffn_single_pass(1)
    # the last call ran on the unscaled input: pin it to the oracle's whole chain, every row, at every size
    o1 = oracle.linear(c["A"], c["W1t"], 8, c["b1"], True)
    s2 = oracle.scale_from_amax(oracle.absmax(o1["Y"]), 8)
    o2 = oracle.linear(o1["Y"], c["W2t"], 8, c["b2"], False, sA=s2)
    assert np.array_equal(host(Y), o2["Y"])


def test_ffn_block_on_a_prepared_workspace_replayed_as_a_graph():
    c = workloads.config2()
    M, d = c["A"].shape
    f = c["W1t"].shape[0]
    p1 = mq.prepare_weight(dev(c["W1t"]), 8)
    p2 = mq.prepare_weight(dev(c["W2t"]), 8)
    b1, b2 = dev(c["b1"]), dev(c["b2"])
    nbytes = mq.mq_ffn_ws_bytes(M, d, f)
    ws = torch.full((nbytes,), 0x3C, dtype=torch.uint8, device=DEV)
    ws_plain = torch.full((nbytes,), 0x3C, dtype=torch.uint8, device=DEV)
    A = dev(c["A"])
    Y = torch.empty((M, d), dtype=torch.float32, device=DEV)
    mq.mq_ffn_ws_prepare(ws, nbytes, M, d, f)

    def step():
        mq.mq_ffn_i8_f32_prepared(A, M, d, f, p1.packed, p1.scale, b1, p2.packed, p2.scale, b2, Y, ws, nbytes)

    g = capture_graph(step, 3)          # three consecutive blocks per replay: each relies on what the one before left
    base = dev(c["A"])
    for r, factor in enumerate((1.0, 0.5, -1.25, 1.0)):
        A.copy_(base * factor)           # eager work between the replays
        mq.mq_ffn_i8_f32(A, M, d, f, p1.packed, p1.scale, b1, p2.packed, p2.scale, b2, Y, ws_plain, nbytes)
        torch.cuda.synchronize()
        want = Y.clone()
        Y.fill_(float("nan"))
        g.replay()
        if r == 1:
            step()                       # an eager prepared call between replays
        torch.cuda.synchronize()
        assert torch.equal(Y, want), f"replay {r}"


@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("shape", [(1, 1), (33, 65), (300, 512), (300, 2048), (2000, 1024), (8192, 512), (70, 1030),
                                   (17000, 96), (384, 512), (48, 4096), (1000, 700), (8192, 1024)])
def test_quantize_absmax_pack(bits, shape):
    # Tensors that fit the registers of one resident grid are read once (the last shapes do not fit and take
    # the two-pass form anyway); with the switch off it is always two passes.  Both forms must give the
    # oracle's integers and multiplier and the same bytes, padding and appended row sums included.  Each
    # form is called twice on one workspace whose contents do not matter.
    rng = np.random.default_rng(shape[0] + shape[1] * 3 + bits)
    x = rng.standard_normal(shape, dtype=np.float32) * np.float32(0.3)
    oq, os_ = oracle.quant_int_absmax(x, bits)
    nb = mq.mq_quantize_absmax_ws_bytes()
    ws = torch.full((nb,), 0x7F, dtype=torch.uint8, device=DEV)
    outs = []
    try:
        for single in (2, 0, 2, 1):
            mq.mq_set_quantize_single_pass(single)
            s = torch.empty(1, dtype=torch.float32, device=DEV)
            packed = torch.full((mq.mq_packed_bytes(bits, *shape),), 0x5A, dtype=torch.uint8, device=DEV)
            mq.mq_quantize_absmax_pack_f32(dev(x), shape[0], shape[1], bits, packed, s, ws, nb)
            q = torch.empty(shape, dtype=QT[bits], device=DEV)
            mq.mq_unpack_weight(packed, bits, shape[0], shape[1], q)
            assert host(s)[0] == os_ and np.array_equal(host(q), oq)
            outs.append(packed)
    finally:
        mq.mq_set_quantize_single_pass(1)
    for o in outs[1:]:
        assert torch.equal(o, outs[0])


@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("shape", [(1, 1), (33, 65), (300, 512), (300, 2048), (2000, 1024), (8192, 512), (70, 1030),
                                   (17000, 96)])
def test_quantize_absmax_pack_on_a_prepared_workspace(bits, shape):
    # the workspace's agreement words are zeroed once; every call leaves them zero (the kernel that reads x once
    # cleans up after itself, the two-pass form never touches them): five calls in a row with changing inputs,
    # with the one-kernel form switched off in between, then three replays of a graph of two calls
    rng = np.random.default_rng(shape[0] * 7 + shape[1] + bits)
    base = rng.standard_normal(shape, dtype=np.float32) * np.float32(0.3)
    nb = mq.mq_quantize_absmax_ws_bytes()
    ws = torch.full((nb,), 0x6D, dtype=torch.uint8, device=DEV)
    ws_plain = torch.full((nb,), 0x6D, dtype=torch.uint8, device=DEV)
    mq.mq_quantize_absmax_ws_prepare(ws, nb)
    x = dev(base)
    s = torch.empty(1, dtype=torch.float32, device=DEV)
    s_plain = torch.empty(1, dtype=torch.float32, device=DEV)
    packed = torch.empty(mq.mq_packed_bytes(bits, *shape), dtype=torch.uint8, device=DEV)
    packed_plain = torch.empty_like(packed)

    def call():
        mq.mq_quantize_absmax_pack_f32_prepared(x, shape[0], shape[1], bits, packed, s, ws, nb)

    def check(tag):
        mq.mq_quantize_absmax_pack_f32(x, shape[0], shape[1], bits, packed_plain, s_plain, ws_plain, nb)
        torch.cuda.synchronize()
        assert torch.equal(s, s_plain) and torch.equal(packed, packed_plain), tag

    try:
        for r, (factor, single) in enumerate([(1.0, 1), (0.5, 1), (-3.0, 0), (2.0, 1), (1.0, 1)]):
            x.copy_(dev(base) * factor)
            packed.fill_(0x5A)
            mq.mq_set_quantize_single_pass(single)
            call()
            mq.mq_set_quantize_single_pass(1)
            check(f"call {r}")
    finally:
        mq.mq_set_quantize_single_pass(1)
    oq, os_ = oracle.quant_int_absmax(base, bits)
    q = torch.empty(shape, dtype=QT[bits], device=DEV)
    mq.mq_unpack_weight(packed, bits, shape[0], shape[1], q)
    assert host(s)[0] == os_ and np.array_equal(host(q), oq)
    g = capture_graph(call, 2)
    for r, factor in enumerate((0.75, -1.5, 1.0)):
        x.copy_(dev(base) * factor)
        packed.fill_(0x33)
        g.replay()
        check(f"replay {r}")


def test_prepared_quantizer_cleans_up_after_a_timed_out_agreement():
    # every workgroup gives up at once: the multiplier is NaN, all kernels end, and since the workgroups still count
    # themselves out the last one leaves the agreement words zero: the next call is right without preparing again
    shape = (2000, 1024)
    rng = np.random.default_rng(99)
    xh = rng.standard_normal(shape, dtype=np.float32)
    oq, os_ = oracle.quant_int_absmax(xh, 8)
    nb = mq.mq_quantize_absmax_ws_bytes()
    ws = torch.full((nb,), 0x42, dtype=torch.uint8, device=DEV)
    mq.mq_quantize_absmax_ws_prepare(ws, nb)
    x = dev(xh)
    s = torch.empty(1, dtype=torch.float32, device=DEV)
    packed = torch.empty(mq.mq_packed_bytes(8, *shape), dtype=torch.uint8, device=DEV)
    try:
        mq.mq_set_barrier_timeout_us(0)
        mq.mq_quantize_absmax_pack_f32_prepared(x, shape[0], shape[1], 8, packed, s, ws, nb)
        assert np.isnan(host(s)[0])
    finally:
        mq.mq_set_barrier_timeout_us(500000)
    assert not ws[: 4 * (8 * 256 + 64)].any().item()
    for _ in range(2):
        mq.mq_quantize_absmax_pack_f32_prepared(x, shape[0], shape[1], 8, packed, s, ws, nb)
        q = torch.empty(shape, dtype=torch.int8, device=DEV)
        mq.mq_unpack_weight(packed, 8, shape[0], shape[1], q)
        assert host(s)[0] == os_ and np.array_equal(host(q), oq)


def test_quantize_absmax_pack_skips_nan_and_handles_zero_tensor():
    x = np.zeros((40, 70), dtype=np.float32)
    nb = mq.mq_quantize_absmax_ws_bytes()
    ws = torch.empty(nb, dtype=torch.uint8, device=DEV)
    s = torch.empty(1, dtype=torch.float32, device=DEV)
    packed = torch.empty(mq.mq_packed_bytes(8, 40, 70), dtype=torch.uint8, device=DEV)
    mq.mq_quantize_absmax_pack_f32(dev(x), 40, 70, 8, packed, s, ws, nb)
    assert host(s)[0] == 1.0
    x[3, 5] = np.nan
    x[7, 9] = -2.5
    oq, os_ = oracle.quant_int_absmax(x, 8)
    mq.mq_quantize_absmax_pack_f32(dev(x), 40, 70, 8, packed, s, ws, nb)
    q = torch.empty((40, 70), dtype=torch.int8, device=DEV)
    mq.mq_unpack_weight(packed, 8, 40, 70, q)
    assert host(s)[0] == os_ and np.array_equal(host(q), oq)


def test_two_pass_requantizing_product():
    p = workloads.random_problem(404, 300, 520, 256)
    o = oracle.linear(p["A"], p["Wt"], 8, p["bias"], True)
    os2 = oracle.scale_from_amax(oracle.absmax(o["Y"]), 8)
    oq = oracle.quant_int(o["Y"], 8, os2)
    M, K = p["A"].shape
    N = p["Wt"].shape[0]
    pw = mq.prepare_weight(dev(p["Wt"]), 8)
    pa, s = gpu_quantize_pack(p["A"], 8)
    nb = mq.mq_gemm_amax_ws_bytes(M, N)
    ws = torch.full((nb,), 0x11, dtype=torch.uint8, device=DEV)
    bias = dev(p["bias"])
    s2 = torch.empty(1, dtype=torch.float32, device=DEV)
    out = torch.full((mq.mq_packed_bytes(8, M, N),), 0x22, dtype=torch.uint8, device=DEV)
    mq.mq_gemm_amax_packed(pa, pw.packed, M, N, K, s, pw.scale, bias, True, ws, nb)
    mq.mq_gemm_requant_packed(pa, pw.packed, M, N, K, s, pw.scale, bias, True, ws, nb, s2, out)
    q = torch.empty((M, N), dtype=torch.int8, device=DEV)
    mq.mq_unpack_weight(out, 8, M, N, q)
    assert host(s2)[0] == os2
    assert np.array_equal(host(q), oq)
    # padding of the packed output is zero: a prepared copy of the same integers has identical bytes
    ref = mq.prepare_weight(dev(oq.astype(np.float32)), 8, scale=torch.ones(1, dtype=torch.float32, device=DEV))
    assert torch.equal(out, ref.packed)


# (the last three: 256 tiles of 128 x 128; too many of those, so 256 x 128, ragged and whole; too many of those, so 256 x 256)
@pytest.mark.parametrize("shape", [(1, 1, 1), (300, 520, 256), (1000, 1100, 128), (512, 768, 192), (256, 256, 64),
                                   (2048, 2048, 64), (2060, 2048, 64), (2304, 2048, 128), (4100, 2048, 64)])
def test_single_pass_requantizing_product(shape):
    # one pass over the operands, the sums waiting in registers while the grid agrees on max|y|;
    # called twice on one workspace (it clears its two words itself)
    M, N, K = shape
    p = workloads.random_problem(405 + M, M, N, K)
    o = oracle.linear(p["A"], p["Wt"], 8, p["bias"], True)
    os2 = oracle.scale_from_amax(oracle.absmax(o["Y"]), 8)
    oq = oracle.quant_int(o["Y"], 8, os2)
    pw = mq.prepare_weight(dev(p["Wt"]), 8)
    pa, s = gpu_quantize_pack(p["A"], 8)
    nb = mq.mq_gemm_amax_ws_bytes(M, N)
    ws = torch.full((nb,), 0xA5, dtype=torch.uint8, device=DEV)
    bias = dev(p["bias"])
    ref = mq.prepare_weight(dev(oq.astype(np.float32)), 8, scale=torch.ones(1, dtype=torch.float32, device=DEV))
    for _ in range(2):
        s2 = torch.empty(1, dtype=torch.float32, device=DEV)
        out = torch.full((mq.mq_packed_bytes(8, M, N),), 0x22, dtype=torch.uint8, device=DEV)
        mq.mq_gemm_requant_single_packed(pa, pw.packed, M, N, K, s, pw.scale, bias, True, ws, nb, s2, out)
        assert host(s2)[0] == os2
        assert torch.equal(out, ref.packed)


@pytest.mark.parametrize("M,N,K,grid", [(31, 33, 31, (2, 512)), (32, 8192, 70, (256, 512)), (33, 4100, 300, (129, 512)),
                                        (200, 2000, 257, (252, 512)), (260, 2048, 1100, (192, 512)),
                                        (1030, 1000, 64, (144, 512)), (2048, 1024, 96, (256, 512)),
                                        (1001, 2050, 520, (136, 512)), (2048, 2048, 96, (256, 512)),
                                        # several trips along K for every wave, the last one not full
                                        (40, 100, 6000, (8, 512)), (200, 2000, 2130, (252, 512)), (260, 2048, 3000, (192, 512)),
                                        (257, 2760, 2300, (132, 512))])
def test_single_pass_requantizing_product_split_k(M, N, K, grid):
    # the forms of the split-K kernel in the order of size and the first tiles behind them, with and without ReLU and bias, a
    # NaN and infinities among the biases (max = inf: multiplier 0, every output 0)
    p = workloads.random_problem(77 + M, M, N, K)
    pw = mq.prepare_weight(dev(p["Wt"]), 8)
    pa, s = gpu_quantize_pack(p["A"], 8)
    nb = mq.mq_gemm_amax_ws_bytes(M, N)
    ws = torch.full((nb,), 0xA5, dtype=torch.uint8, device=DEV)
    out, s2 = torch.empty(mq.mq_packed_bytes(8, M, N), dtype=torch.uint8, device=DEV), torch.empty(1, dtype=torch.float32, device=DEV)
    nan, inf = p["bias"].copy(), p["bias"].copy()
    nan[N // 3], inf[N // 2] = np.nan, -np.inf
    for bias, relu in ((p["bias"], True), (None, False), (nan, False), (inf, True), (inf, False)):
        o = oracle.linear(p["A"], p["Wt"], 8, bias, relu)
        os2 = oracle.scale_from_amax(oracle.absmax(o["Y"]), 8)
        oq = oracle.quant_int(o["Y"], 8, os2)
        ref = mq.prepare_weight(dev(oq.astype(np.float32)), 8, scale=torch.ones(1, dtype=torch.float32, device=DEV))
        db = None if bias is None else dev(bias)
        out.fill_(0x22)

        def call(stream):
            mq.mq_gemm_requant_single_packed(pa, pw.packed, M, N, K, s, pw.scale, db, relu, ws, nb, s2, out, stream)

        grids = launched_grids(call)
        assert host(s2)[0] == os2
        assert torch.equal(out, ref.packed)
        assert tuple(grids[-1]) == grid


@pytest.mark.parametrize("shape", [(512, 768, 192), (300, 520, 256)])
def test_single_pass_requantizing_product_special_bias(shape):
    # whole tiles + ReLU take the kernel whose re-quantization is a single rounding addition per element;
    # a NaN bias (ReLU turns it into 0) and an infinite one (max = inf, multiplier 0, every output 0)
    # must come out as the clamp-and-NaN rule gives them.  The second shape takes the general kernel.
    M, N, K = shape
    p = workloads.random_problem(911 + M, M, N, K)
    pw = mq.prepare_weight(dev(p["Wt"]), 8)
    pa, s = gpu_quantize_pack(p["A"], 8)
    nb = mq.mq_gemm_amax_ws_bytes(M, N)
    ws = torch.full((nb,), 0xA5, dtype=torch.uint8, device=DEV)
    for special in (np.nan, np.inf):
        bias = p["bias"].copy()
        bias[N // 3] = special
        o = oracle.linear(p["A"], p["Wt"], 8, bias, True)
        os2 = oracle.scale_from_amax(oracle.absmax(o["Y"]), 8)
        oq = oracle.quant_int(o["Y"], 8, os2)
        ref = mq.prepare_weight(dev(oq.astype(np.float32)), 8, scale=torch.ones(1, dtype=torch.float32, device=DEV))
        s2 = torch.empty(1, dtype=torch.float32, device=DEV)
        out = torch.full((mq.mq_packed_bytes(8, M, N),), 0x22, dtype=torch.uint8, device=DEV)
        mq.mq_gemm_requant_single_packed(pa, pw.packed, M, N, K, s, pw.scale, dev(bias), True, ws, nb, s2, out)
        assert host(s2)[0] == os2
        assert torch.equal(out, ref.packed)


def test_single_pass_barrier_timeout_is_loud_and_recoverable():
    # With a zero time limit every workgroup that has to wait gives up at once: all kernels still end,
    # the output's multiplier is NaN (and so is everything a caller computes from it), and the next
    # call with the normal limit is correct again on the same workspace.
    c = workloads.ffn(2, 1000, 128, 1100, 0.04, 8, seed_extra=77)
    o1 = oracle.linear(c["A"], c["W1t"], 8, c["b1"], True)
    s2 = oracle.scale_from_amax(oracle.absmax(o1["Y"]), 8)
    o2 = oracle.linear(o1["Y"], c["W2t"], 8, c["b2"], False, sA=s2)
    try:
        mq.mq_set_barrier_timeout_us(0)
        assert np.all(np.isnan(gpu_ffn_fused(c)))
    finally:
        mq.mq_set_barrier_timeout_us(500000)
    assert np.array_equal(gpu_ffn_fused(c), o2["Y"])


def test_prepared_workspace_after_a_timed_out_agreement():
    # The same failure on a prepared workspace: the call that gave up is loud (NaN) and may leave the agreement words
    # in any state; after mq_ffn_ws_prepare the calls are right again.  (M d >= 2^20, so both single-pass kernels run.)
    M, d, f = 2048, 512, 640
    c = workloads.ffn(2, M, d, f, 0.04, 8, seed_extra=78)
    o1 = oracle.linear(c["A"], c["W1t"], 8, c["b1"], True)
    s2 = oracle.scale_from_amax(oracle.absmax(o1["Y"]), 8)
    o2 = oracle.linear(o1["Y"], c["W2t"], 8, c["b2"], False, sA=s2)
    p1 = mq.prepare_weight(dev(c["W1t"]), 8)
    p2 = mq.prepare_weight(dev(c["W2t"]), 8)
    A, b1, b2 = dev(c["A"]), dev(c["b1"]), dev(c["b2"])
    nbytes = mq.mq_ffn_ws_bytes(M, d, f)
    ws = torch.full((nbytes,), 0x77, dtype=torch.uint8, device=DEV)
    Y = torch.empty((M, d), dtype=torch.float32, device=DEV)

    def call():
        mq.mq_ffn_i8_f32_prepared(A, M, d, f, p1.packed, p1.scale, b1, p2.packed, p2.scale, b2, Y, ws, nbytes)
        torch.cuda.synchronize()
        return host(Y)

    mq.mq_ffn_ws_prepare(ws, nbytes, M, d, f)
    assert np.array_equal(call(), o2["Y"])
    try:
        mq.mq_set_barrier_timeout_us(0)
        assert np.all(np.isnan(call()))
    finally:
        mq.mq_set_barrier_timeout_us(500000)
    mq.mq_ffn_ws_prepare(ws, nbytes, M, d, f)
    assert np.array_equal(call(), o2["Y"])
    assert np.array_equal(call(), o2["Y"])


def test_single_pass_requantizing_product_refuses_what_does_not_fit():
    M, N, K = 4352, 4096, 64           # 272 tiles of 256 x 256
    pa = torch.zeros(mq.mq_packed_bytes(8, M, K), dtype=torch.uint8, device=DEV)
    pw = torch.zeros(mq.mq_packed_bytes(8, N, K), dtype=torch.uint8, device=DEV)
    one = torch.ones(1, dtype=torch.float32, device=DEV)
    nb = mq.mq_gemm_amax_ws_bytes(M, N)
    ws = torch.zeros(nb, dtype=torch.uint8, device=DEV)
    out = torch.zeros(mq.mq_packed_bytes(8, M, N), dtype=torch.uint8, device=DEV)
    with pytest.raises(mq.MqError):
        mq.mq_gemm_requant_single_packed(pa, pw, M, N, K, one, one, None, False, ws, nb, one.clone(), out)


# ------------------------------------------------ short-listed output layer

def gpu_greedy_shortlist(Hd, E, shortlist):
    pw = mq.prepare_weight(dev(E), 8)
    pa, s = gpu_quantize_pack(Hd, 8)
    M, K = Hd.shape
    N = E.shape[0]
    sl = dev(np.asarray(shortlist, dtype=np.int32))
    nbytes = mq.mq_argmax_ws_bytes(M, N)
    ws = torch.full((nbytes,), 0xEE, dtype=torch.uint8, device=DEV)
    tok = torch.full((M,), -7, dtype=torch.int32, device=DEV)
    val = torch.empty(M, dtype=torch.float32, device=DEV)
    mq.mq_gemm_argmax_shortlist(pa, pw.packed, sl, sl.numel(), M, N, K, s, pw.scale, tok, val, ws, nbytes)
    return host(tok), host(val)


@pytest.mark.parametrize("M,V,d,L", [(1, 1, 1, 1), (12, 777, 64, 1), (12, 777, 64, 15), (33, 4100, 96, 1000),
                                     (300, 36000, 512, 4321), (300, 36000, 512, 36000), (130, 9000, 192, 8999),
                                     (20, 150001, 32, 70000)])       # a list longer than the ring: slots refilled
def test_greedy_shortlist(M, V, d, L):
    c = workloads.config3(M=M, V=V, d=d, seed_extra=M + V + L)
    rng = np.random.default_rng(L + V)
    sl = np.sort(rng.choice(V, size=L, replace=False))
    o = oracle.greedy_output_layer(c["Hd"], c["E"], shortlist=sl)
    tok, val = gpu_greedy_shortlist(c["Hd"], c["E"], sl)
    assert np.array_equal(tok, o["tok"])
    assert np.array_equal(val, o["maxlogit"])


def test_greedy_shortlist_ties_and_frequent_plus_translations_shape():
    # list shaped like the paper's: the 100 most frequent ids plus 100 candidates per source word
    V, d, M = 36000, 512, 15
    c = workloads.config3(M=M, V=V, d=d, seed_extra=77)
    rng = np.random.default_rng(5)
    sl = np.unique(np.concatenate([np.arange(100), rng.integers(0, V, size=384 * 100 // 8)]))
    E = c["E"].copy()
    E[sl[40]] = E[sl[3000]]          # duplicate rows inside the list: the smaller id has to win
    E[sl[-1]] = E[sl[3000]]
    o = oracle.greedy_output_layer(c["Hd"], E, shortlist=sl)
    tok, val = gpu_greedy_shortlist(c["Hd"], E, sl)
    assert np.array_equal(tok, o["tok"]) and np.array_equal(val, o["maxlogit"])
    assert np.all(np.isin(tok, sl))


def test_greedy_shortlist_ids_outside_the_vocabulary_do_not_fault():
    # an id outside [0, N) is the caller's mistake; the kernel scores the nearest row in its place instead of reading
    # outside the embedding, and reports the id as listed if that candidate wins
    c = workloads.config3(M=9, V=500, d=64, seed_extra=3)
    bad = np.array([-7, 3, 17, 250, 100000], dtype=np.int32)
    good_clamped = np.array([0, 3, 17, 250, 499])
    o = oracle.greedy_output_layer(c["Hd"], c["E"], shortlist=np.unique(good_clamped))
    tok_bad, val_bad = gpu_greedy_shortlist(c["Hd"], c["E"], bad)
    assert np.array_equal(val_bad, o["maxlogit"])                       # rows 0 and 499 were scored in their place
    back = {-7: 0, 100000: 499}
    assert np.array_equal(np.array([back.get(int(t), int(t)) for t in tok_bad]), o["tok"])


# ---------------------------------- fixed multipliers (the paper's scheme) and auto-tuning

@pytest.mark.parametrize("M,d,f", [(1, 1, 1), (37, 64, 200), (300, 256, 520), (130, 96, 1000)])
def test_ffn_int16_with_the_fixed_multiplier(M, d, f):
    # the paper's 16-bit scheme (Section 4.2): every tensor multiplied by 2^10; the first product writes the
    # second one's input as packed 16-bit activations (byte planes + row sums) from its epilogue
    c = workloads.ffn(4, M, d, f, 0.03, 16, seed_extra=M + d + 7 * f)
    S = np.float32(1024.0)
    o1 = oracle.linear(c["A"], c["W1t"], 16, c["b1"], True, sA=S, sW=S)
    o2 = oracle.linear(o1["Y"], c["W2t"], 16, c["b2"], False, sA=S, sW=S)
    assert o1["overflow_count"] == 0 and o2["overflow_count"] == 0
    sc = torch.full((1,), 1024.0, dtype=torch.float32, device=DEV)
    p1 = mq.prepare_weight(dev(c["W1t"]), 16, scale=sc)
    p2 = mq.prepare_weight(dev(c["W2t"]), 16, scale=sc)
    qA = torch.empty(mq.mq_packed_bytes(16, M, d), dtype=torch.uint8, device=DEV)
    mq.mq_quantize_pack_f32(dev(c["A"]), M, d, 16, sc, qA)
    for _ in range(2):                                            # the row sums are cleared by the call itself
        qH = torch.full((mq.mq_packed_bytes(16, M, f),), 0x5D, dtype=torch.uint8, device=DEV)
        mq.mq_gemm_requant_fixed_packed_i16(qA, p1.packed, M, f, d, sc, sc, dev(c["b1"]), True, sc, qH)
        # identical bytes to the quantizer's packing of the oracle's intermediate (planes, padding, row sums)
        ref = torch.empty_like(qH)
        mq.mq_quantize_pack_f32(dev(o1["Y"]), M, f, 16, sc, ref)
        assert torch.equal(qH, ref)
        q = torch.empty((M, f), dtype=torch.int16, device=DEV)
        mq.mq_unpack_weight(qH, 16, M, f, q)
        assert np.array_equal(host(q), o2["qA"])
        Y = torch.empty((M, d), dtype=torch.float32, device=DEV)
        mq.mq_gemm_dequant_packed(qH, p2.packed, 16, M, d, f, sc, sc, dev(c["b2"]), False, Y, None)
        assert np.array_equal(host(Y), o2["Y"])
    # the same block in one call
    nb = mq.mq_ffn_i16_fixed_ws_bytes(M, d, f)
    ws = torch.full((nb,), 0x6E, dtype=torch.uint8, device=DEV)
    for _ in range(2):
        Y = torch.full((M, d), float("nan"), dtype=torch.float32, device=DEV)
        mq.mq_ffn_i16_fixed_f32(dev(c["A"]), M, d, f, sc, p1.packed, sc, dev(c["b1"]), sc, p2.packed, sc, dev(c["b2"]), Y,
                                ws, nb)
        assert np.array_equal(host(Y), o2["Y"])


@pytest.mark.parametrize("M,N,K,relu,grid", [(1, 33, 1, False, (2, 512)),              # an odd number of fragments: padding
                                             (33, 64, 70, True, (4, 512)), (255, 1024, 33, False, (256, 512)),
                                             (257, 1000, 520, False, (288, 256)), (5, 4100, 129, True, (129, 512)),
                                             (16384, 96, 5, False, (1536, 256)), (16385, 96, 5, False, (129, 512))])
def test_requantizing_int16_product_shapes(M, N, K, relu, grid):
    # split K with four or eight waves up to six workgroups per compute unit, tiles beyond: the bytes of the quantizer on the
    # oracle's result (planes, padding, row sums), with values beyond the 16-bit range, infinities among the biases and none
    p = workloads.random_problem(M + N + K, M, N, K)
    sc, s_out = (torch.full((1,), v, dtype=torch.float32, device=DEV) for v in (1024.0, 5000.0))
    pw = mq.prepare_weight(dev(p["Wt"]), 16, scale=sc)
    qA = torch.empty(mq.mq_packed_bytes(16, M, K), dtype=torch.uint8, device=DEV)
    mq.mq_quantize_pack_f32(dev(p["A"]), M, K, 16, sc, qA)
    bias = np.random.default_rng(N).normal(0, 6, N).astype(np.float32)
    bias[:2] = np.inf, -np.inf
    got = torch.empty(mq.mq_packed_bytes(16, M, N), dtype=torch.uint8, device=DEV)
    for b in (bias, None):
        o = oracle.linear(p["A"], p["Wt"], 16, b, relu, sA=np.float32(1024.0), sW=np.float32(1024.0))
        ref = torch.empty_like(got)
        mq.mq_quantize_pack_f32(dev(o["Y"]), M, N, 16, s_out, ref)
        got.fill_(0x5D)
        db = None if b is None else dev(b)

        def call(stream):
            mq.mq_gemm_requant_fixed_packed_i16(qA, pw.packed, M, N, K, sc, sc, db, relu, s_out, got, stream)

        grids = launched_grids(call)
        assert torch.equal(got, ref)
        assert tuple(grids[-1]) == grid


def test_ffn_int16_fixed_multiplier_full_size_equals_oracle_on_all_rows():
    # the paper's 16-bit scheme at the benchmark's 8192 x 1024 x 4096, one call, every row against the oracle;
    # with 2^10 no 32-bit sum wraps (Section 4.2 chose the multiplier for that)
    c = workloads.config4()
    M, d = c["A"].shape
    f = c["W1t"].shape[0]
    S = np.float32(1024.0)
    o1 = oracle.linear(c["A"], c["W1t"], 16, c["b1"], True, sA=S, sW=S)
    o2 = oracle.linear(o1["Y"], c["W2t"], 16, c["b2"], False, sA=S, sW=S)
    assert o1["overflow_count"] == 0 and o2["overflow_count"] == 0
    sc = torch.full((1,), 1024.0, dtype=torch.float32, device=DEV)
    p1 = mq.prepare_weight(dev(c["W1t"]), 16, scale=sc)
    p2 = mq.prepare_weight(dev(c["W2t"]), 16, scale=sc)
    nb = mq.mq_ffn_i16_fixed_ws_bytes(M, d, f)
    ws = torch.full((nb,), 0x6E, dtype=torch.uint8, device=DEV)
    Y = torch.full((M, d), float("nan"), dtype=torch.float32, device=DEV)
    mq.mq_ffn_i16_fixed_f32(dev(c["A"]), M, d, f, sc, p1.packed, sc, dev(c["b1"]), sc, p2.packed, sc, dev(c["b2"]), Y, ws, nb)
    assert np.array_equal(host(Y), o2["Y"])


def test_ffn_with_fixed_multipliers_single_pass():
    # Section 4.2: 8-bit inputs clipped to [-2, 2] and scaled by 127/2; no abs-max anywhere.  The
    # intermediate is quantized in the epilogue of the product that creates it.
    c = workloads.ffn(2, 200, 128, 384, 0.04, 8, seed_extra=5)
    A = c["A"] * np.float32(1.5)                  # some values beyond +-2: they saturate at +-127
    W1, W2 = c["W1t"] * np.float32(8), c["W2t"] * np.float32(8)
    fixed = np.float32(63.5)
    o1 = oracle.linear(A, W1, 8, c["b1"], True, sA=fixed, sW=fixed)
    assert np.abs(o1["qA"]).max() == 127 and (np.abs(A) > 2).any()
    oqH = oracle.quant_int(o1["Y"], 8, fixed)
    o2 = oracle.dequant_bias(oracle.dot_int(oqH, oracle.quant_int(W2, 8, fixed)), fixed, fixed, c["b2"], False)
    M, d = A.shape
    f = W1.shape[0]
    sc = torch.full((1,), 63.5, dtype=torch.float32, device=DEV)
    p1 = mq.prepare_weight(dev(W1), 8, scale=sc)
    p2 = mq.prepare_weight(dev(W2), 8, scale=sc)
    qA = torch.empty(mq.mq_packed_bytes(8, M, d), dtype=torch.uint8, device=DEV)
    mq.mq_quantize_pack_f32(dev(A), M, d, 8, sc, qA)
    qH = torch.full((mq.mq_packed_bytes(8, M, f),), 0x44, dtype=torch.uint8, device=DEV)
    mq.mq_gemm_requant_fixed_packed(qA, p1.packed, M, f, d, sc, p1.scale, dev(c["b1"]), True, sc, qH)
    Y = torch.empty((M, d), dtype=torch.float32, device=DEV)
    mq.mq_gemm_dequant_packed(qH, p2.packed, 8, M, d, f, sc, p2.scale, dev(c["b2"]), False, Y, None)
    q = torch.empty((M, f), dtype=torch.int8, device=DEV)
    mq.mq_unpack_weight(qH, 8, M, f, q)
    assert np.array_equal(host(q), oqH)
    assert np.array_equal(host(Y), o2)


def test_autotune_freezes_a_variant_and_results_stay_identical():
    M, N, K = 300, 512, 256
    p = workloads.random_problem(909, M, N, K)
    o = oracle.linear(p["A"], p["Wt"], 8, p["bias"], False)
    nbytes = mq.mq_autotune_ws_bytes(8, M, N, K)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    best, us = mq.mq_autotune_gemm(8, M, N, K, 20, ws, nbytes)
    assert 1 <= best <= 14 and us > 0
    pw = mq.prepare_weight(dev(p["Wt"]), 8)
    pa, s = gpu_quantize_pack(p["A"], 8)
    Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    mq.mq_gemm_dequant_packed(pa, pw.packed, 8, M, N, K, s, pw.scale, dev(p["bias"]), False, Y, None)
    assert np.array_equal(host(Y), o["Y"])
    best16, _ = mq.mq_autotune_gemm(16, 64, 96, 128, 5, torch.empty(mq.mq_autotune_ws_bytes(16, 64, 96, 128),
                                                                      dtype=torch.uint8, device=DEV),
                                    mq.mq_autotune_ws_bytes(16, 64, 96, 128))
    assert 1 <= best16 <= 6


# ------------------------------------------------ beam-search output layer

def gpu_topk(Hd, E, k, shortlist=None):
    pw = mq.prepare_weight(dev(E), 8)
    pa, s = gpu_quantize_pack(Hd, 8)
    M, K = Hd.shape
    N = E.shape[0]
    sl = None if shortlist is None else dev(np.asarray(shortlist, dtype=np.int32))
    nbytes = mq.mq_topk_ws_bytes(M, N, k)
    ws = torch.full((nbytes,), 0xC3, dtype=torch.uint8, device=DEV)
    tok = torch.full((M, k), -7, dtype=torch.int32, device=DEV)
    lp = torch.empty((M, k), dtype=torch.float32, device=DEV)
    mq.mq_gemm_topk_packed(pa, pw.packed, sl, 0 if sl is None else sl.numel(), M, N, K, s, pw.scale, k, tok, lp, ws,
                           nbytes)
    return host(tok), host(lp)


@pytest.mark.parametrize("k", [1, 2, 3, 4])
@pytest.mark.parametrize("M,V,d", [(1, 4, 1), (12, 777, 64), (33, 4100, 96), (300, 36000, 512), (130, 9000, 192),
                                   (600, 5000, 128), (12, 70000, 64), (1200, 3000, 64)])
def test_beam_output_layer_topk(M, V, d, k):
    # Table 2's b = 2 / b = 4 rows: the k best words per row, exact, with log-probabilities within 1e-4
    # (binary32 logits of magnitude <= ~30 here; the normaliser sums V terms in binary32).  M = 600 and 1200 go
    # through three and five chunks of rows (the last ones ragged), all in one launch.
    c = workloads.config3(M=M, V=V, d=d, seed_extra=M + V + k)
    o = oracle.topk_log_softmax(c["Hd"], c["E"], k)
    tok, lp = gpu_topk(c["Hd"], c["E"], k)
    assert np.array_equal(tok, o["tok"])
    assert np.allclose(lp, o["logprob"], rtol=0, atol=1e-4)


def test_beam_output_layer_ties_and_crowded_lanes():
    # all k best words in one accumulator register's stream: duplicates of the winning embedding row placed
    # one workgroup-stride (256 units of 16 words) apart land in the same register of the same lane
    c = workloads.config3(M=20, V=36000, d=64, seed_extra=123)
    E = c["E"].copy()
    h = c["Hd"][0] / np.abs(c["Hd"][0]).max() * np.abs(E).max()     # aligned with sentence 0, inside the abs-max
    for j in range(4):
        E[5 + 4096 * j] = h * (1.0 - 0.01 * j)
    E[5 + 4096 * 4] = h                                              # exact tie with the first, higher index
    o = oracle.topk_log_softmax(c["Hd"], E, 4)
    tok, lp = gpu_topk(c["Hd"], E, 4)
    assert list(o["tok"][0][:2]) == [5, 5 + 4096 * 4]
    assert np.array_equal(tok, o["tok"])
    assert np.allclose(lp, o["logprob"], rtol=0, atol=1e-4)


@pytest.mark.parametrize("k", [2, 4])
@pytest.mark.parametrize("M,V", [(520, 20000), (40, 9000)])
def test_beam_output_layer_growing_logits(M, V, k):
    # Embedding rows that grow with their index: later words exceed the running reference of the softmax normaliser
    # again and again (by more than its slack of 2^16), in chunks of rows that share the compute units and alone.
    # Logits reach about 60: one binary32 rounding of such a logit is 4e-6, a sum of V terms stays below 1e-4.
    c = workloads.config3(M=M, V=V, d=64, seed_extra=31 + k)
    E = np.ascontiguousarray(c["E"] * (30.0 * np.arange(V) / V)[:, None]).astype(np.float32)
    o = oracle.topk_log_softmax(c["Hd"], E, k)
    tok, lp = gpu_topk(c["Hd"], E, k)
    assert np.array_equal(tok, o["tok"])
    assert np.allclose(lp, o["logprob"], rtol=0, atol=1e-4)


@pytest.mark.parametrize("M,columns,units,more", [
    # around the ring of ten slots (9 units: nothing is refilled; 10: a refill that nobody reads), once and twice round it, with
    # an even and an odd number of units and columns of both lengths; one chunk of rows, and three whose 85 columns share XCDs
    (5, 256, 9, 0), (5, 256, 9, 3), (5, 256, 10, 0), (5, 256, 11, 255), (5, 256, 19, 1), (5, 256, 20, 0), (5, 256, 21, 7),
    (780, 85, 10, 84), (780, 85, 21, 1)])
def test_output_layer_units_of_a_workgroup(M, columns, units, more):
    V, d = 16 * (columns * units + more) - 3, 32
    c = workloads.config3(M=M, V=V, d=d, seed_extra=units + more)
    E = c["E"].copy()
    top = np.abs(E).max()
    for j, u in enumerate(sorted({0, units - 1, units, 9, 10})):       # best words of the last sentences in these units
        at = 16 * columns * u + 16 * (more // 2) + j
        if at < V:
            E[at] = c["Hd"][M - 1 - j] * (top / np.abs(c["Hd"][M - 1 - j]).max())
    o = oracle.greedy_output_layer(c["Hd"], E)
    tok, val = gpu_greedy_packed(c["Hd"], E)
    assert np.array_equal(tok, o["tok"]) and np.array_equal(val, o["maxlogit"])
    if M < 100:
        for k in (2, 4):
            o = oracle.topk_log_softmax(c["Hd"], E, k)
            tok, lp = gpu_topk(c["Hd"], E, k)
            assert np.array_equal(tok, o["tok"]) and np.allclose(lp, o["logprob"], rtol=0, atol=1e-4)
        wide = np.zeros((M, 528), dtype=np.float32), np.zeros((V, 528), dtype=np.float32)      # two stages a unit, 18 slots
        wide[0][:, 496:], wide[1][:, 496:] = c["Hd"], E
        o = oracle.greedy_output_layer(*wide)
        tok, val = gpu_greedy(*wide)[:2]
        assert np.array_equal(tok, o["tok"]) and np.array_equal(val, o["maxlogit"])


@pytest.mark.parametrize("k", [2, 4])
@pytest.mark.parametrize("V,L", [(9000, 1234), (120000, 60000)])     # the longer list refills the ring's slots
def test_beam_output_layer_with_shortlist(k, V, L):
    c = workloads.config3(M=64, V=V, d=128 if V < 10000 else 32, seed_extra=77)
    rng = np.random.default_rng(5)
    sl = np.sort(rng.choice(V, size=L, replace=False)).astype(np.int32)
    qE = c["E"][sl]
    # the short list is scored with the whole embedding's multiplier: quantize the whole, then gather
    full = oracle.greedy_output_layer(c["Hd"], c["E"])
    acc = oracle.dot_int(full["qA"], np.ascontiguousarray(full["qW"][sl]))
    y = oracle.dequant_bias(acc, full["sA"], full["sW"]).astype(np.float64)
    lse = np.log(np.exp(y - y.max(1, keepdims=True)).sum(1, keepdims=True)) + y.max(1, keepdims=True)
    order = np.argsort(-acc.astype(np.int64), axis=1, kind="stable")[:, :k]
    tok, lp = gpu_topk(c["Hd"], c["E"], k, shortlist=sl)
    assert np.array_equal(tok, sl[order])
    assert np.allclose(lp, np.take_along_axis(y, order, axis=1) - lse, rtol=0, atol=1e-4)
    del qE
