"""GPU parity of the float glue of the averaging-attention decode step and of the chained decoder layer
(Sections 3.1, 3.2) against oracle/glue.py, through the C boundary.

Tolerances.  The glue is binary32 on the GPU and binary64 in the oracle.  Element-wise operations make a
handful of roundings (relative 2^-24 each); the reductions sum d <= 2048 terms of magnitude O(1) in
binary32 (error below d * 2^-24 * max|term| ~ 1e-4 in the worst case, ~1e-6 typically).  Each operation
is therefore compared at 2e-5 absolute + 2e-5 relative on inputs of unit scale.  A chained layer feeds
glue results into quant_int: an input that sits within ~1e-7 of a rounding boundary can round to the
neighbouring integer on one side only (about 5e-6 of the elements: a 1-ulp difference times |x s| ~ 40),
which changes every output of that sentence's row in the next product by about |w| / s ~ 1e-3, and the
row then stays at that level through the following layers.  So chained results are compared per
sentence: no element beyond 5e-2, and only a small share of the rows (one product input has 150 000
elements, so about one row per product) beyond 1e-4.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads
from oracle import glue

mq = pytest.importorskip("paper_1805_12096_amd")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def host(t):
    return t.detach().cpu().numpy()


def close(a, b, tol=2e-5):
    return np.allclose(a, b, rtol=tol, atol=tol)


@pytest.mark.parametrize("t", [1, 2, 20, 97])
def test_running_average(t):
    rng = np.random.default_rng(t)
    g, x = rng.standard_normal((300, 512), dtype=np.float32), rng.standard_normal((300, 512), dtype=np.float32)
    out = torch.empty((300, 512), dtype=torch.float32, device=DEV)
    mq.mq_running_average_f32(dev(g), dev(x), g.size, t, out)
    assert close(host(out), glue.running_average(g, x, t), 1e-6)


def test_concat2_is_exact():
    rng = np.random.default_rng(5)
    a, b = rng.standard_normal((37, 96), dtype=np.float32), rng.standard_normal((37, 33), dtype=np.float32)
    out = torch.empty((37, 129), dtype=torch.float32, device=DEV)
    mq.mq_concat2_f32(dev(a), 96, dev(b), 33, 37, out)
    assert np.array_equal(host(out), np.concatenate([a, b], axis=1))


@pytest.mark.parametrize("M,d", [(1, 1), (5, 33), (300, 512), (64, 2048), (3, 8192)])
def test_add_layer_norm(M, d):
    rng = np.random.default_rng(M + d)
    a = (rng.standard_normal((M, d)) * 2 + 0.5).astype(np.float32)
    r = rng.standard_normal((M, d), dtype=np.float32)
    gamma, beta = (1 + 0.1 * rng.standard_normal(d)).astype(np.float32), (0.1 * rng.standard_normal(d)).astype(np.float32)
    y = torch.empty((M, d), dtype=torch.float32, device=DEV)
    mq.mq_add_layer_norm_f32(dev(a), dev(r), dev(gamma), dev(beta), M, d, 1e-6, y)
    assert close(host(y), glue.add_layer_norm(a, r, gamma, beta, 1e-6), 5e-5 if d > 1024 else 2e-5)


@pytest.mark.parametrize("M,d", [(2, 3), (300, 512), (17, 1000)])
def test_gate_mix_layer_norm(M, d):
    rng = np.random.default_rng(M * 7 + d)
    x, f = rng.standard_normal((M, d), dtype=np.float32), rng.standard_normal((M, d), dtype=np.float32)
    z = (rng.standard_normal((M, 2 * d)) * 3).astype(np.float32)
    gamma, beta = (1 + 0.1 * rng.standard_normal(d)).astype(np.float32), (0.1 * rng.standard_normal(d)).astype(np.float32)
    y = torch.empty((M, d), dtype=torch.float32, device=DEV)
    mq.mq_gate_mix_layer_norm_f32(dev(x), dev(f), dev(z), dev(gamma), dev(beta), M, d, 1e-6, y)
    assert close(host(y), glue.add_layer_norm(glue.gate_mix(x, f, z), x, gamma, beta, 1e-6))


@pytest.mark.parametrize("M,d", [(1, 256), (33, 512), (5, 768), (300, 1024)])
def test_layer_norm_kernels_give_the_same_bits(M, d):
    # rows that do not start on 16 bytes take the kernel with a thread per element; the order of the additions is the same
    rng = np.random.default_rng(M + d)

    def shifted(a):
        buf = torch.empty(a.size + 4, dtype=torch.float32, device=DEV)
        v = buf[1:1 + a.size].view(a.shape)
        v.copy_(dev(a))
        return v

    a, r, z = (rng.standard_normal(s, dtype=np.float32) for s in ((M, d), (M, d), (M, 2 * d)))
    gamma, beta = (1 + 0.1 * rng.standard_normal(d)).astype(np.float32), (0.1 * rng.standard_normal(d)).astype(np.float32)
    got = []
    for put in (dev, shifted):
        y1, y2 = (torch.empty((M, d), dtype=torch.float32, device=DEV) for _ in range(2))
        mq.mq_add_layer_norm_f32(put(a), put(r), put(gamma), put(beta), M, d, 1e-6, y1)
        mq.mq_gate_mix_layer_norm_f32(put(a), put(r), put(z), put(gamma), put(beta), M, d, 1e-6, y2)
        got.append((host(y1), host(y2)))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("M,S,d,heads", [(1, 1, 8, 1), (7, 5, 48, 3), (300, 25, 512, 8), (9, 130, 256, 4),
                                          (5, 7, 1024, 16), (6, 9, 512, 4), (4, 3, 256, 64), (3, 6, 512, 2),
                                          # around the trips of 32 source positions and 64 scores a head
                                          (3, 31, 512, 8), (2, 33, 512, 8), (5, 64, 512, 1), (2, 65, 1024, 4), (1, 17, 1024, 16),
                                          (3, 63, 256, 2), (3, 64, 256, 1), (2, 150, 256, 8), (4, 1, 1024, 8),
                                          # fewer positions than waves, and than rows of a trip; more sentences than compute units
                                          (600, 1, 512, 8), (300, 8, 1024, 16), (1, 9, 256, 4), (2, 24, 512, 8), (257, 26, 512, 8),
                                          # either side of where V is asked for ahead: 256 sentences, 12 positions
                                          (256, 13, 256, 4), (257, 13, 256, 4), (256, 12, 512, 8), (257, 33, 1024, 16),
                                          (9, 40, 1024, 16), (300, 70, 512, 8)])
def test_cross_attention(M, S, d, heads):
    rng = np.random.default_rng(M + S + d)
    q = rng.standard_normal((M, d), dtype=np.float32) * np.float32(2)
    K, V = rng.standard_normal((M, S, d), dtype=np.float32), rng.standard_normal((M, S, d), dtype=np.float32)
    ctx = torch.empty((M, d), dtype=torch.float32, device=DEV)
    mq.mq_cross_attention_f32(dev(q), dev(K), dev(V), M, S, d, heads, ctx)
    assert close(host(ctx), glue.cross_attention(q, K, V, heads))


def test_glue_argument_checks():
    x = torch.zeros((4, 8), dtype=torch.float32, device=DEV)
    with pytest.raises(mq.MqError):
        mq.mq_running_average_f32(x, x, 32, 0, x)                      # positions count from 1
    with pytest.raises(mq.MqError):
        mq.mq_cross_attention_f32(x, x, x, 4, 1, 8, 3, x)              # width not divisible by heads
    with pytest.raises(mq.MqError):
        mq.mq_add_layer_norm_f32(x, x, x, x, 1, 10000, 1e-6, x)        # row longer than the kernel keeps


# ------------------------------------------------------------ chained layer

def prepare_layer(P, d, ffn, aan_ffn):
    products = {}
    for name in ("aan_ffn1", "aan_ffn2", "aan_gate", "ctx_q", "ctx_o", "ffn1", "ffn2"):
        products[name] = (mq.prepare_weight(dev(P[name]["Wt"]), 8), dev(P[name]["bias"]))
    norms = {name: (dev(P[name]["gamma"]), dev(P[name]["beta"])) for name in ("ln1", "ln2", "ln3")}
    return mq.aan_layer(products, norms, d, ffn, aan_ffn)


def run_layer(layer, x, g_prev, t, K, V, heads, use_ffn=True, use_gate=True):
    M, d = x.shape
    S = K.shape[1]
    nb = mq.mq_aan_layer_ws_bytes(M, d, layer.c.ffn, layer.c.aan_ffn)
    ws = torch.full((nb,), 0x6B, dtype=torch.uint8, device=DEV)        # contents must not matter
    y = torch.empty((M, d), dtype=torch.float32, device=DEV)
    g = torch.empty((M, d), dtype=torch.float32, device=DEV)
    mq.mq_aan_layer_f32(layer, x, g_prev, t, K, V, M, S, heads, use_ffn, use_gate, glue.LN_EPS, y, g, ws, nb)
    return y, g


def assert_chained_close(got, want, what, max_rows_off):
    diff = np.abs(got.astype(np.float64) - want.astype(np.float64))
    assert diff.max() < 5e-2, f"{what}: max |diff| {diff.max()}"
    rows_off = (diff.max(axis=1) > 1e-4).mean()
    assert rows_off <= max_rows_off, f"{what}: {rows_off:.3f} of the rows beyond 1e-4"


@pytest.mark.parametrize("use_ffn,use_gate", [(True, True), (False, True), (False, False), (True, False)])
@pytest.mark.parametrize("shape", [dict(M=6, d=32, ffn=64, aan_ffn=48, S=4, heads=4),
                                   dict(M=300, d=512, ffn=2048, aan_ffn=2048, S=25, heads=8),
                                   dict(M=130, d=512, ffn=2048, aan_ffn=512, S=25, heads=8),
                                   dict(M=40, d=1024, ffn=160, aan_ffn=96, S=5, heads=16),
                                   dict(M=24, d=48, ffn=40, aan_ffn=72, S=3, heads=4)])
def test_decoder_layer_matches_oracle(shape, use_ffn, use_gate):
    # the third shape is the paper's own averaging block (inner width = model width, Section 3.2); the fourth has a
    # gate input wider than the in-kernel quantizer takes (concatenated copy + separate quantizer), the fifth has
    # widths that are no multiples of 32 (no product of it quantizes in the kernel)
    c = workloads.config5_chained(M=shape["M"], layers=1, d=shape["d"], ffn=shape["ffn"], aan_ffn=shape["aan_ffn"],
                                  S=shape["S"], V=8, t=20, seed_extra=shape["M"])
    P, (K, V) = c["layers"][0], c["KV"][0]
    want_y, want_g = glue.aan_decoder_layer(c["x0"], c["g_prev"][0], 20, P, K, V, heads=shape["heads"],
                                            use_ffn=use_ffn, use_gate=use_gate)
    layer = prepare_layer(P, shape["d"], shape["ffn"], shape["aan_ffn"])
    y, g = run_layer(layer, dev(c["x0"]), dev(c["g_prev"][0]), 20, dev(K), dev(V), shape["heads"], use_ffn, use_gate)
    assert close(host(g), want_g, 1e-6)
    assert_chained_close(host(y), want_y, "layer output", 0.10)


def gpu_quant8(xd):
    """abs-max, multiplier and quant_int (8 bit) of a device tensor; returns (integers, multiplier) on the host."""
    rows, cols = xd.shape
    s = torch.empty(1, dtype=torch.float32, device=DEV)
    mq.mq_absmax_f32(xd, xd.numel(), s)
    mq.mq_scale_from_amax(s, 8, s)
    q = torch.empty((rows, cols), dtype=torch.int8, device=DEV)
    mq.mq_quantize_f32(xd, rows, cols, 8, s, q, None)
    return host(q), host(s)[0]


def assert_few_flips(xd, want_f32, what):
    """quant_int of a GPU glue result against quant_int of the oracle's value of the same tensor: the multipliers
    agree to a few ulps (the tensor's maximum is itself a glue result: a layer normalisation's binary32 sums leave
    it a few ulps from the binary64 value; 1e-6 relative is allowed), no integer differs by more than one, and only
    a handful differ at all (a binary32 glue result a few ulps from the binary64 one crosses a rounding boundary
    with probability ~ |x s| 2^-21 ~ 2e-5; 1e-4 of the elements are allowed)."""
    q, s = gpu_quant8(xd)
    oq, os_ = oracle.quant_int_absmax(want_f32, 8)
    assert abs(float(s) - float(os_)) <= 1e-6 * float(os_), what
    dq = q.astype(np.int32) - oq.astype(np.int32)
    assert np.abs(dq).max() <= 1, f"{what}: an integer differs by {np.abs(dq).max()}"
    allowed = max(3, int(1e-4 * dq.size))
    assert np.count_nonzero(dq) <= allowed, f"{what}: {np.count_nonzero(dq)} of {dq.size} integers flipped (allowed {allowed})"


def gpu_linear_f32(A, W, bias, relu):
    M, K = A.shape
    N = W.N
    nb = mq.mq_linear_ws_bytes(8, M, K)
    ws = torch.empty(nb, dtype=torch.uint8, device=DEV)
    Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    mq.mq_linear_f32(A, M, K, None, W.packed, W.scale, 8, N, bias, relu, Y, None, ws, nb)
    return Y


@pytest.mark.parametrize("shape", [dict(M=300, d=512, ffn=2048, aan_ffn=2048, S=25, heads=8),
                                   dict(M=130, d=512, ffn=2048, aan_ffn=512, S=25, heads=8),
                                   dict(M=24, d=48, ffn=40, aan_ffn=72, S=3, heads=4)])
def test_decoder_layer_stage_by_stage(shape):
    # The envelope of test_decoder_layer_matches_oracle is wide because one flipped integer moves a whole row of the
    # next product.  Here every stage is checked on the ORACLE's input for that stage, so nothing accumulates:
    #   glue stages: 2e-5 against the binary64 value, and quant_int of the GPU's result differs from quant_int of the
    #     oracle's in at most a handful of integers, each by one;
    #   products (quant_int -> dot'_int -> dequantize + bias): bit-identical;
    # and the one-call layer must give the bits of the same stages called one by one on the GPU.
    from test_oracle_glue_pins import hand_composed_layer
    M, d, heads, t = shape["M"], shape["d"], shape["heads"], 20
    c = workloads.config5_chained(M=M, layers=1, d=d, ffn=shape["ffn"], aan_ffn=shape["aan_ffn"], S=shape["S"], V=8,
                                  t=t, seed_extra=shape["M"] + 1)
    P, (K, V) = c["layers"][0], c["KV"][0]
    x, gp = c["x0"], c["g_prev"][0]
    r = hand_composed_layer(x, gp, t, P, K, V, heads)
    W = {}
    for name in ("aan_ffn1", "aan_ffn2", "aan_gate", "ctx_q", "ctx_o", "ffn1", "ffn2"):
        W[name] = mq.prepare_weight(dev(P[name]["Wt"]), 8)
        W[name].bias = dev(P[name]["bias"])
    ln = {n_: (dev(P[n_]["gamma"]), dev(P[n_]["beta"])) for n_ in ("ln1", "ln2", "ln3")}
    xd, gpd, Kd, Vd = dev(x), dev(gp), dev(K), dev(V)

    def f32buf(cols=d):
        return torch.empty((M, cols), dtype=torch.float32, device=DEV)

    def stages(src):
        """The layer's stages one call at a time; src(name, gpu_value) picks each stage's input."""
        o = {}
        o["g"] = f32buf()
        mq.mq_running_average_f32(gpd, xd, M * d, t, o["g"])
        o["h1"] = gpu_linear_f32(src("g", o["g"]), W["aan_ffn1"], W["aan_ffn1"].bias, True)
        o["f"] = gpu_linear_f32(src("h1", o["h1"]), W["aan_ffn2"], W["aan_ffn2"].bias, False)
        fin = src("f", o["f"])
        cat = f32buf(2 * d)
        mq.mq_concat2_f32(xd, d, fin, d, M, cat)
        o["z"] = gpu_linear_f32(cat, W["aan_gate"], W["aan_gate"].bias, False)
        o["y1"] = f32buf()
        mq.mq_gate_mix_layer_norm_f32(xd, fin, src("z", o["z"]), ln["ln1"][0], ln["ln1"][1], M, d, glue.LN_EPS, o["y1"])
        y1 = src("y1", o["y1"])
        o["q"] = gpu_linear_f32(y1, W["ctx_q"], W["ctx_q"].bias, False)
        o["ctx"] = f32buf()
        mq.mq_cross_attention_f32(src("q", o["q"]), Kd, Vd, M, shape["S"], d, heads, o["ctx"])
        o["o"] = gpu_linear_f32(src("ctx", o["ctx"]), W["ctx_o"], W["ctx_o"].bias, False)
        o["y2"] = f32buf()
        mq.mq_add_layer_norm_f32(src("o", o["o"]), y1, ln["ln2"][0], ln["ln2"][1], M, d, glue.LN_EPS, o["y2"])
        y2 = src("y2", o["y2"])
        o["h2"] = gpu_linear_f32(y2, W["ffn1"], W["ffn1"].bias, True)
        o["ff"] = gpu_linear_f32(src("h2", o["h2"]), W["ffn2"], W["ffn2"].bias, False)
        o["y3"] = f32buf()
        mq.mq_add_layer_norm_f32(src("ff", o["ff"]), y2, ln["ln3"][0], ln["ln3"][1], M, d, glue.LN_EPS, o["y3"])
        return o

    # every stage on the oracle's value of its input
    forced = stages(lambda name, gpu_value: dev(r[name]))
    torch.cuda.synchronize()
    for name in ("h1", "f", "z", "q", "o", "h2", "ff"):
        assert np.array_equal(host(forced[name]), r[name]), f"product {name} on the oracle's input"
    assert close(host(forced["g"]), r["g"], 1e-6)
    for name in ("y1", "ctx", "y2", "y3"):
        assert close(host(forced[name]), r[name]), f"glue {name} on the oracle's input"
    for name in ("g", "y1", "ctx", "y2"):              # the glue results that enter quant_int
        assert_few_flips(forced[name], r[name], name)
    # the one-call layer against the same stages chained on the GPU's own values
    own = stages(lambda name, gpu_value: gpu_value)
    layer = prepare_layer(P, d, shape["ffn"], shape["aan_ffn"])
    y, g = run_layer(layer, xd, gpd, t, Kd, Vd, heads)
    torch.cuda.synchronize()
    assert torch.equal(g, own["g"]) and torch.equal(y, own["y3"])


@pytest.mark.parametrize("shape", [dict(M=1, d=512, ffn=2048, aan_ffn=2048, S=23, heads=8),
                                   dict(M=9, d=256, ffn=1028, aan_ffn=260, S=3, heads=4),
                                   dict(M=32, d=768, ffn=96, aan_ffn=2048, S=4, heads=12),
                                   dict(M=8, d=1024, ffn=4096, aan_ffn=1024, S=40, heads=16),
                                   dict(M=17, d=1024, ffn=4096, aan_ffn=64, S=2, heads=16)])
def test_decoder_layer_of_one_row_block_stage_by_stage(shape):
    # at most 32 sentences: average, normalisations, gate and quantizers run inside the products; the last shape's
    # second feed-forward product is beyond what that form holds and takes the quantizing launch
    test_decoder_layer_stage_by_stage(shape)


@pytest.mark.parametrize("shape", [dict(M=1, d=256, ffn=64, aan_ffn=2048, S=1, heads=1),       # one head as wide as it may be
                                   dict(M=8, d=256, ffn=2048, aan_ffn=64, S=64, heads=64),     # heads of four columns
                                   dict(M=7, d=512, ffn=192, aan_ffn=320, S=100, heads=32),
                                   dict(M=2, d=512, ffn=2048, aan_ffn=2048, S=33, heads=4),
                                   dict(M=8, d=1024, ffn=4096, aan_ffn=4096, S=17, heads=16),
                                   dict(M=3, d=1024, ffn=64, aan_ffn=1088, S=256, heads=16),
                                   dict(M=1, d=512, ffn=2048, aan_ffn=2048, S=512, heads=8),   # the longest source
                                   dict(M=1, d=1024, ffn=4096, aan_ffn=4096, S=190, heads=4),  # ... of the widest heads
                                   # where nine launches are ahead (eight sentences of 256 words, two heads: 47.1 us and 68.6)
                                   dict(M=1, d=1024, ffn=4096, aan_ffn=4096, S=191, heads=4, launches=9),
                                   dict(M=8, d=512, ffn=64, aan_ffn=64, S=512, heads=2, launches=9),
                                   dict(M=8, d=256, ffn=256, aan_ffn=256, S=8, heads=64, launches=9),
                                   dict(M=1, d=512, ffn=64, aan_ffn=64, S=513, heads=4, launches=9)])
def test_decoder_layer_of_a_few_rows(shape):
    # up to eight sentences: two launches, whose workgroups wait for each other's rows.  The bits of the launches stage by
    # stage (and of the route that a named variant takes), also when no row comes within the time a workgroup waits (each then
    # takes roles over and begins again, and ends when that fails, but for the one that computes the layer alone), when some
    # come and some do not, with NaN and infinities, and replayed.
    from test_gpu_parity import launches
    M, d, S, heads = (shape[k] for k in ("M", "d", "S", "heads"))
    test_decoder_layer_stage_by_stage(shape)
    c = workloads.config5_chained(M=M, layers=1, d=d, ffn=shape["ffn"], aan_ffn=shape["aan_ffn"], S=S, V=8, t=4, seed_extra=d)
    layer = prepare_layer(c["layers"][0], d, shape["ffn"], shape["aan_ffn"])
    K, V = (dev(a) for a in c["KV"][0])
    x, gp = dev(c["x0"]), dev(c["g_prev"][0])
    odd = x.clone()
    odd[0, 5], odd[-1, -1] = float("inf"), float("nan")

    def same(a, b):
        return torch.equal(torch.nan_to_num(a, 7.5, 8.5, 9.5), torch.nan_to_num(b, 7.5, 8.5, 9.5))

    try:
        mq.mq_set_gemm_variant(1)
        want, want_odd = run_layer(layer, x, gp, 4, K, V, heads), run_layer(layer, odd, gp, 4, K, V, heads)
    finally:
        mq.mq_set_gemm_variant(0)
    for xs, w in ((x, want), (odd, want_odd)):
        y, g = run_layer(layer, xs, gp, 4, K, V, heads)
        assert same(y, w[0]) and same(g, w[1])
    try:
        for us in (0, 1, 2, 4, 8) * 3:
            mq.mq_set_barrier_timeout_us(us)
            y, g = run_layer(layer, x, gp, 4, K, V, heads)
            torch.cuda.synchronize()
            assert torch.equal(y, want[0]) and torch.equal(g, want[1])
    finally:
        mq.mq_set_barrier_timeout_us(500000)
    nb = mq.mq_aan_layer_ws_bytes(M, d, shape["ffn"], shape["aan_ffn"])
    ws, y, g = torch.empty(nb, dtype=torch.uint8, device=DEV), torch.empty_like(x), torch.empty_like(x)

    def call(stream):
        mq.mq_aan_layer_f32(layer, x, gp, 4, K, V, M, S, heads, True, True, glue.LN_EPS, y, g, ws, nb, stream)

    assert launches(call) == shape.get("launches", 2)
    try:
        mq.mq_set_ffn_single_pass(0)                     # kernels that wait are switched off: the same bits in launches
        assert launches(call) == 9
        y0, g0 = run_layer(layer, x, gp, 4, K, V, heads)
        assert torch.equal(y0, want[0]) and torch.equal(g0, want[1])
    finally:
        mq.mq_set_ffn_single_pass(1)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(torch.cuda.current_stream())
    for _ in range(4):
        y.fill_(5.0)
        ws.fill_(0x3C)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want[0]) and torch.equal(g, want[1])


def test_decoder_layer_of_one_row_block_runs_the_variant_named():
    # the products of the layer that go through the packed products otherwise (wider than 1024) keep to a variant the
    # caller has forced or tuned, also up to 32 sentences, where one launch quantizes and multiplies: launches of the layer
    from test_gpu_parity import launches, tune
    M, d, ffn = 5, 768, 1056
    c = workloads.config5_chained(M=M, layers=1, V=8, d=d, ffn=ffn, aan_ffn=d, t=3)
    layer = prepare_layer(c["layers"][0], d, ffn, d)
    K, V = (dev(a) for a in c["KV"][0])
    x, gp = dev(c["x0"]), dev(c["g_prev"][0])
    want = run_layer(layer, x, gp, 3, K, V, 12)
    nb = mq.mq_aan_layer_ws_bytes(M, d, ffn, d)
    ws, y, g = torch.empty(nb, dtype=torch.uint8, device=DEV), torch.empty_like(x), torch.empty_like(x)

    def call(stream):
        mq.mq_aan_layer_f32(layer, x, gp, 3, K, V, M, K.shape[1], 12, True, True, glue.LN_EPS, y, g, ws, nb, stream)

    assert launches(call) == 9
    try:
        mq.mq_set_gemm_variant(1)
        several = launches(call)
        mq.mq_set_gemm_variant(15)                     # a variant that does not exist is refused
        with pytest.raises(mq.MqError) as e:
            call(torch.cuda.current_stream())
        assert e.value.status == 6
    finally:
        mq.mq_set_gemm_variant(0)
    assert several > 10                                # the gate's product (width 1536) and the second feed-forward product
    tune(8, M, d, ffn)
    assert launches(call) == 10                        # a quantizer and the tuned product in place of one launch
    y.fill_(-3.0)
    call(torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert torch.equal(y, want[0]) and torch.equal(g, want[1])


@pytest.mark.parametrize("M", [20, 33, 1])
def test_decoder_layer_updates_the_average_in_place(M):
    # g_out = g_prev: no workgroup may read an average that another one has already replaced.  The last elements hold the
    # largest average, and averaging them a second time would nearly double it.
    c = workloads.config5_chained(M=M, layers=1, V=8, t=20)
    layer = prepare_layer(c["layers"][0], 512, 2048, 2048)
    K, V = (dev(a) for a in c["KV"][0])
    x, g = dev(c["x0"]), dev(c["g_prev"][0])
    x[-1, -4:], g[-1, -4:] = 200.0, 0.0
    want_y, want_g = run_layer(layer, x, g, 20, K, V, 8)
    nb = mq.mq_aan_layer_ws_bytes(M, 512, 2048, 2048)
    ws, y = torch.empty(nb, dtype=torch.uint8, device=DEV), torch.empty_like(x)
    mq.mq_aan_layer_f32(layer, x, g, 20, K, V, M, K.shape[1], 8, True, True, glue.LN_EPS, y, g, ws, nb)
    assert torch.equal(g, want_g) and torch.equal(y, want_y)


def test_decoder_layer_and_output_layer_replayed_as_a_graph():
    # the launch configuration of bench.py's chained decode step: layers and the greedy output layer in one HIP
    # graph.  Every replay (other inputs, refilled workspaces, eager work in between) must give the eager bits.
    c = workloads.config5_chained(M=300, layers=2, V=5000)
    layers = [prepare_layer(P, 512, 2048, 2048) for P in c["layers"]]
    KV = [(dev(k), dev(v)) for k, v in c["KV"]]
    gp = [dev(g) for g in c["g_prev"]]
    gn = [torch.empty_like(g) for g in gp]
    M, d, V = 300, 512, 5000
    xs = [dev(c["x0"])] + [torch.empty((M, d), dtype=torch.float32, device=DEV) for _ in layers]
    nwl = mq.mq_aan_layer_ws_bytes(M, d, 2048, 2048)
    wsl = torch.full((nwl,), 0x11, dtype=torch.uint8, device=DEV)
    pe = mq.prepare_weight(dev(c["E"]), 8)
    qp = torch.empty(mq.mq_packed_bytes(8, M, d), dtype=torch.uint8, device=DEV)
    s = torch.empty(1, dtype=torch.float32, device=DEV)
    qn = mq.mq_quantize_absmax_ws_bytes()
    qws = torch.empty(qn, dtype=torch.uint8, device=DEV)
    nws = mq.mq_argmax_ws_bytes(M, V)
    ws = torch.empty(nws, dtype=torch.uint8, device=DEV)
    tok = torch.empty(M, dtype=torch.int32, device=DEV)
    val = torch.empty(M, dtype=torch.float32, device=DEV)

    def step():
        for l, layer in enumerate(layers):
            mq.mq_aan_layer_f32(layer, xs[l], gp[l], c["t"], KV[l][0], KV[l][1], M, 25, c["heads"], True, True,
                                glue.LN_EPS, xs[l + 1], gn[l], wsl, nwl)
        mq.mq_quantize_absmax_pack_f32(xs[-1], M, d, 8, qp, s, qws, qn)
        mq.mq_gemm_argmax_packed(qp, pe.packed, M, V, d, s, pe.scale, tok, val, ws, nws)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
        step()
    x0 = dev(c["x0"])
    for r, factor in enumerate((1.0, -0.75, 2.0)):
        xs[0].copy_(x0 * factor)
        step()
        torch.cuda.synchronize()
        want = (xs[-1].clone(), tok.clone(), val.clone(), gn[0].clone())
        for t_ in (xs[-1], val, gn[0]):
            t_.fill_(float("nan"))
        tok.fill_(-1)
        wsl.fill_(0x40 + r)
        ws.fill_(0x50 + r)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(xs[-1], want[0]) and torch.equal(tok, want[1]) and torch.equal(val, want[2]), f"replay {r}"
        assert torch.equal(gn[0], want[3])


def test_full_decode_step_matches_oracle():
    # Six layers with their real dependencies, then the tied output layer with greedy arg-max.
    # Per-tensor abs-max multipliers make a free-running chain sensitive: once a rounding flip reaches the
    # element that holds a tensor's maximum, that tensor's multiplier moves by ~1e-3 and every row of the
    # following products moves with it.  So each layer is checked tightly on the ORACLE's input for that
    # layer (what the kernels compute), and the free-running chain only statistically.
    c = workloads.config5_chained(M=300, layers=6, V=36000)
    x = dev(c["x0"])
    x_oracle = c["x0"]
    for l, P in enumerate(c["layers"]):
        layer = prepare_layer(P, 512, 2048, 2048)
        K, V, gp = dev(c["KV"][l][0]), dev(c["KV"][l][1]), dev(c["g_prev"][l])
        forced, g_forced = run_layer(layer, dev(x_oracle), gp, c["t"], K, V, c["heads"])
        x, _ = run_layer(layer, x, gp, c["t"], K, V, c["heads"])
        x_oracle, g_oracle = glue.aan_decoder_layer(x_oracle, c["g_prev"][l], c["t"], P, *c["KV"][l], heads=c["heads"])
        assert close(host(g_forced), g_oracle, 1e-6)
        assert_chained_close(host(forced), x_oracle, f"layer {l} on the oracle's input", 0.05)
    diff = host(x).astype(np.float64) - x_oracle
    assert np.sqrt((diff ** 2).mean()) < 5e-2 * np.sqrt((x_oracle.astype(np.float64) ** 2).mean())
    want = oracle.greedy_output_layer(x_oracle, c["E"])
    M, d = 300, 512
    pe = mq.prepare_weight(dev(c["E"]), 8)
    qp = torch.empty(mq.mq_packed_bytes(8, M, d), dtype=torch.uint8, device=DEV)
    s = torch.empty(1, dtype=torch.float32, device=DEV)
    qws = torch.empty(mq.mq_quantize_absmax_ws_bytes(), dtype=torch.uint8, device=DEV)
    mq.mq_quantize_absmax_pack_f32(x, M, d, 8, qp, s, qws, qws.numel())
    nws = mq.mq_argmax_ws_bytes(M, 36000)
    ws = torch.empty(nws, dtype=torch.uint8, device=DEV)
    tok = torch.empty(M, dtype=torch.int32, device=DEV)
    val = torch.empty(M, dtype=torch.float32, device=DEV)
    mq.mq_gemm_argmax_packed(qp, pe.packed, M, 36000, d, s, pe.scale, tok, val, ws, nws)
    # the GPU's own hidden state decides its tokens exactly (the integer path is bit-exact) ...
    own = oracle.greedy_output_layer(host(x), c["E"])
    assert np.array_equal(host(tok), own["tok"]) and np.array_equal(host(val), own["maxlogit"])
    # ... and most of them are the binary64 chain's tokens (random hidden states against a random embedding
    # have many near-ties; measured agreement 0.95)
    agree = host(tok) == want["tok"]
    assert agree.mean() >= 0.85, f"only {agree.mean():.3f} of the tokens agree with the binary64 chain"
