"""GPU parity of the training-side entry points (Alg. 1 / Alg. 2 backward and update, Sec. 2.1-2.3) against the CPU
oracle, through the C ABI.  The sums of the backward products run in the oracle's order, so they are compared bit
for bit; steps that go through an fp64 library function (exp, sqrt of a sum in another order) within 1e-6."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util
    return gpu_util


@pytest.fixture(scope="module")
def bnn():
    import paper_1706_09453_amd as b
    return b


@pytest.fixture(scope="module")
def T():
    from oracle import train_oracle
    return train_oracle


def _f32(M, N, fill=float("nan")):
    return torch.full((M, N), fill, dtype=torch.float32, device="cuda:0")


SHAPES = [(1, 1, 1), (3, 5, 7), (17, 33, 65), (64, 100, 257), (130, 440, 200), (70, 2048, 96), (300, 260, 1028)]


@pytest.mark.parametrize("wb", [32, 64])
@pytest.mark.parametrize("N,K", [(1, 1), (5, 3), (31, 64), (64, 65), (65, 33), (100, 257), (2048, 440), (1000, 2048)])
def test_pack_weights_transposed(G, bnn, oracle, N, K, wb):
    W = np.random.default_rng(N + K).standard_normal((N, K)).astype(np.float32)
    W[::3, ::5] = 0.0                                                   # Sign(0) = -1: bit 0
    out = G.word_tensor(K, N, wb)
    dW = G.to_dev(W)
    bnn.bnn_pack_weights_transposed(G.ptr(dW), N, K, wb, G.ptr(out), G.stream())
    assert np.array_equal(G.words_to_host(out, wb), oracle.pack_sign(np.ascontiguousarray(W.T), wb))


@pytest.mark.parametrize("R,C", [(1, 1), (3, 70), (64, 64), (65, 63), (130, 2048), (4096, 100)])
def test_transpose(G, bnn, R, C):
    A = np.random.default_rng(R * C).standard_normal((R, C)).astype(np.float32)
    out = _f32(C, R)
    dA = G.to_dev(A)
    bnn.bnn_transpose_f32(G.ptr(dA), R, C, G.ptr(out), G.stream())
    assert np.array_equal(out.cpu().numpy(), A.T)


@pytest.mark.parametrize("M,N", [(1, 1), (7, 10), (64, 3307), (300, 1000), (5, 4), (3001, 3), (70000, 1), (1, 70004), (2, 70001),
                                 (1023, 512), (1024, 511), (1024, 512), (1030, 701)])
def test_softmax_xent_grad(G, bnn, T, M, N):
    rng = np.random.default_rng(M + N)
    z = rng.standard_normal((M, N)) * 3
    logp = (z - np.log(np.exp(z).sum(1, keepdims=True))).astype(np.float32)
    labels = rng.integers(0, N, M).astype(np.int32)
    g = _f32(M, N)
    dlogp, dlabels = G.to_dev(logp), G.to_dev(labels)
    bnn.bnn_softmax_xent_grad(G.ptr(dlogp), G.ptr(dlabels), M, N, G.ptr(g), G.stream())
    assert np.max(np.abs(g.cpu().numpy() - T.softmax_xent_grad(logp, labels))) <= 1e-6


@pytest.mark.parametrize("k", [0.5, 1.0, 3.0])
def test_mask_grad(G, bnn, T, k):
    rng = np.random.default_rng(7)
    g = rng.standard_normal(100003).astype(np.float32)
    hh = (rng.standard_normal(100003) * 2).astype(np.float32)
    hh[:4] = [k, -k, np.nextafter(np.float32(k), np.float32(9)), np.nan]
    dg, dhh = G.to_dev(g), G.to_dev(hh)
    out = torch.full((g.size,), float("nan"), dtype=torch.float32, device="cuda:0")
    bnn.bnn_mask_grad(G.ptr(dg), G.ptr(dhh), g.size, k, G.ptr(out), G.stream())
    assert np.array_equal(out.cpu().numpy(), T.mask_grad(g, hh, k), equal_nan=True)
    bnn.bnn_mask_grad(G.ptr(dg), G.ptr(dhh), g.size, k, G.ptr(dg), G.stream())      # in place
    assert np.array_equal(dg.cpu().numpy(), T.mask_grad(g, hh, k), equal_nan=True)


def test_sigmoid_grad(G, bnn, T):
    rng = np.random.default_rng(3)
    g = rng.standard_normal(200001).astype(np.float32)
    h = (1.0 / (1.0 + np.exp(-rng.standard_normal(200001) * 3))).astype(np.float32)
    h[:3] = [0.0, 1.0, 0.5]
    dg, dh = G.to_dev(g), G.to_dev(h)
    out = torch.full((g.size,), float("nan"), dtype=torch.float32, device="cuda:0")
    bnn.bnn_sigmoid_grad(G.ptr(dg), G.ptr(dh), g.size, G.ptr(out), G.stream())
    assert np.array_equal(out.cpu().numpy(), T.sigmoid_grad(g, h))


@pytest.mark.parametrize("wb", [32, 64])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_backward_input_binw(G, bnn, oracle, T, M, N, K, wb):
    """g_h = g_hhat w^b through the transposed packed signs: the same ascending-n chain as the oracle's, identical bits."""
    rng = np.random.default_rng(M + N + K)
    g = rng.standard_normal((M, N)).astype(np.float32)
    W = rng.uniform(-1, 1, (N, K)).astype(np.float32)
    WpT = G.word_tensor(K, N, wb)
    dW, dg = G.to_dev(W), G.to_dev(g)
    bnn.bnn_pack_weights_transposed(G.ptr(dW), N, K, wb, G.ptr(WpT), G.stream())
    out = _f32(M, K)
    bnn.bnn_backward_input_binw(G.ptr(dg), G.ptr(WpT), M, N, K, wb, G.ptr(out), G.stream())
    want = T.backward_input_binw(g, np.where(W > 0, 1, -1).astype(np.int8))
    assert np.array_equal(out.cpu().numpy(), want)


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_backward_input_realw_and_weight_gradient(G, bnn, T, M, N, K):
    rng = np.random.default_rng(3 * M + N + K)
    g = rng.standard_normal((M, N)).astype(np.float32)
    W = (rng.standard_normal((N, K)) / np.sqrt(N)).astype(np.float32)
    h = rng.standard_normal((M, K)).astype(np.float32)
    dg, dW, dh = G.to_dev(g), G.to_dev(W), G.to_dev(h)
    Wt, gt, ht = _f32(K, N), _f32(N, M), _f32(K, M)
    bnn.bnn_transpose_f32(G.ptr(dW), N, K, G.ptr(Wt), G.stream())
    bnn.bnn_transpose_f32(G.ptr(dg), M, N, G.ptr(gt), G.stream())
    bnn.bnn_transpose_f32(G.ptr(dh), M, K, G.ptr(ht), G.stream())
    gh, gw, gr = _f32(M, K), _f32(N, K), torch.full((N,), float("nan"), dtype=torch.float32, device="cuda:0")
    bnn.bnn_backward_input_realw(G.ptr(dg), G.ptr(Wt), M, N, K, G.ptr(gh), G.stream())
    bnn.bnn_backward_weight(G.ptr(gt), G.ptr(ht), N, K, M, G.ptr(gw), G.stream())
    bnn.bnn_bias_grad(G.ptr(dg), M, N, G.ptr(gr), G.stream())
    assert np.array_equal(gh.cpu().numpy(), T.backward_input_realw(g, W))
    assert np.array_equal(gw.cpu().numpy(), T.backward_weight(g, h))
    assert np.array_equal(gr.cpu().numpy(), T.bias_grad(g))


def test_weight_gradient_of_a_binary_input(G, bnn, oracle, T):
    """g_w = g_hhat^T h with h the bits of a binary layer, read as -1/+1 and as 0/1 (unpacked, transposed, multiplied)."""
    M, N, K = 200, 96, 130
    rng = np.random.default_rng(11)
    g = rng.standard_normal((M, N)).astype(np.float32)
    words = oracle.pack_sign(rng.standard_normal((M, K)).astype(np.float32), 32)
    gt = _f32(N, M)
    dg, dwords = G.to_dev(g), G.to_dev(words)
    bnn.bnn_transpose_f32(G.ptr(dg), M, N, G.ptr(gt), G.stream())
    for zero_one in (False, True):
        hX = G.unpack_activations(dwords, K, 32, zero_one)
        ht, gw = _f32(K, M), _f32(N, K)
        bnn.bnn_transpose_f32(G.ptr(hX), M, K, G.ptr(ht), G.stream())
        bnn.bnn_backward_weight(G.ptr(gt), G.ptr(ht), N, K, M, G.ptr(gw), G.stream())
        assert np.array_equal(gw.cpu().numpy(), T.backward_weight(g, oracle.bits_to_real(words, K, 32, zero_one)))


@pytest.mark.parametrize("wb", [32, 64])
@pytest.mark.parametrize("M,N,K", SHAPES + [(4096, 64, 300)])
def test_weight_gradient_of_sign_units_by_add_and_subtract(G, bnn, oracle, T, M, N, K, wb):
    """g_w = g_hhat^T h for h = Sign(hhat_prev) from the bits of h^T packed along the frames: same bits as the product
    with the unpacked input."""
    rng = np.random.default_rng(M + 2 * N + K)
    g = rng.standard_normal((M, N)).astype(np.float32)
    hhat_prev = rng.standard_normal((M, K)).astype(np.float32)
    dg, dhh = G.to_dev(g), G.to_dev(hhat_prev)
    gt, HpT, gw = _f32(N, M), G.word_tensor(K, M, wb), _f32(N, K)
    bnn.bnn_transpose_f32(G.ptr(dg), M, N, G.ptr(gt), G.stream())
    bnn.bnn_pack_weights_transposed(G.ptr(dhh), M, K, wb, G.ptr(HpT), G.stream())
    bnn.bnn_backward_weight_binh(G.ptr(gt), G.ptr(HpT), N, K, M, wb, G.ptr(gw), G.stream())
    want = T.backward_weight(g, np.where(hhat_prev > 0, 1.0, -1.0).astype(np.float32))
    assert np.array_equal(gw.cpu().numpy(), want)


def _realx_i8(G, bnn, dX, dWp, M, K, N, wb, scale=None, bias=None):
    """bnn_layer_binw_realx_i8 with a fresh workspace; returns the fp32 outputs."""
    nbytes = bnn.bnn_layer_binw_realx_i8_workspace_bytes(M, K, N)
    assert nbytes > 0
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda:0")
    out = _f32(M, N)
    bnn.bnn_layer_binw_realx_i8(G.ptr(dX), G.ptr(dWp), 0 if scale is None else G.ptr(scale), 0 if bias is None else G.ptr(bias),
                                M, K, N, wb, G.ptr(out), G.ptr(ws), nbytes, G.stream())
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("wb", [32, 64])
@pytest.mark.parametrize("M,K,N", [(1, 1, 1), (3, 5, 7), (130, 440, 200), (128, 64, 256), (300, 2048, 700), (257, 1023, 129),
                                   (129, 8192, 65), (1000, 4096, 300), (2048, 256, 2048)])
def test_layer_binw_realx_on_the_int8_matrix_cores(G, bnn, oracle, M, K, N, wb):
    """The sign-selected sum from four digit planes: within K 2^-27 max|x| (or K 2^-101 for tiny frames) of the exact sum
    for every frame (the bound the header states; the fp64 sum of the oracle stands for the exact one), scale and bias
    applied by one fma."""
    rng = np.random.default_rng(M * 3 + K + N + wb)
    X = rng.standard_normal((M, K)).astype(np.float32)
    X[::5] *= np.exp(rng.uniform(-12, 12, (len(X[::5]), K))).astype(np.float32)      # wide range inside some frames
    X[1::7] *= np.float32(1e-30)
    W = rng.uniform(-1, 1, (N, K)).astype(np.float32)
    Wp = oracle.pack_sign(W, wb)
    scale = (rng.uniform(0.5, 1.5, N) * np.where(rng.random(N) < 0.2, -1, 1)).astype(np.float32)
    bias = rng.standard_normal(N).astype(np.float32)
    _, acc64 = oracle.realx_acc(X, oracle.unpack_pm1(Wp, K, wb))
    got = _realx_i8(G, bnn, G.to_dev(X), G.to_dev(Wp), M, K, N, wb)
    # (frames whose largest element is below 2^-74 are rounded to multiples of 2^-100)
    bound = K * np.maximum(2.0 ** -27 * np.abs(X).max(1, keepdims=True).astype(np.float64), 2.0 ** -101)
    assert np.all(np.abs(got.astype(np.float64) - acc64) <= bound + 2.0 ** -23 * np.abs(acc64))   # + the final rounding to fp32
    got = _realx_i8(G, bnn, G.to_dev(X), G.to_dev(Wp), M, K, N, wb, G.to_dev(scale), G.to_dev(bias))
    want = oracle.affine_f64(acc64, scale, bias)
    tol = np.abs(scale.astype(np.float64)) * bound + 2.0 ** -22 * (np.abs(want) + np.abs(bias))
    assert np.all(np.abs(got.astype(np.float64) - want) <= tol)


@pytest.mark.parametrize("K", [4, 508, 512, 516, 1024, 1028, 2048, 2052, 4096, 4100, 8188, 8192, 513])
@pytest.mark.parametrize("M", [1, 5])
def test_layer_binw_realx_int8_row_lengths(G, bnn, oracle, M, K):
    """Both sides of every length at which the quantisation takes another number of registers, and a ragged length: the
    same bound.  The largest element is the frame's last one, so a tail left out shows in every digit."""
    N = 33
    rng = np.random.default_rng(M + K)
    X = rng.standard_normal((M, K)).astype(np.float32)
    X[:, -1] = 7.5
    Wp = oracle.pack_sign(rng.uniform(-1, 1, (N, K)).astype(np.float32), 32)
    _, acc64 = oracle.realx_acc(X, oracle.unpack_pm1(Wp, K, 32))
    got = _realx_i8(G, bnn, G.to_dev(X), G.to_dev(Wp), M, K, N, 32)
    assert np.all(np.abs(got.astype(np.float64) - acc64) <= K * 2.0 ** -27 * 7.5 + 2.0 ** -23 * np.abs(acc64))


# 64 x 128 tiles, in the launch's order and (17 tile rows) in the XCDs'; 128 x 256 tiles; ragged
@pytest.mark.parametrize("M,N", [(1, 1), (65, 129), (1030, 200), (2049, 2049)])
@pytest.mark.parametrize("K", [3, 64, 65, 129, 193, 257, 320])       # one to five steps of 64 k, three of them in LDS
def test_layer_binw_realx_int8_tiles(G, bnn, oracle, M, N, K):
    """Integers of at most 2^14 as inputs: quantised without rounding, and the sums are below 2^24, so the result is exact."""
    rng = np.random.default_rng(M + K)
    X = rng.integers(-(1 << 14), 1 << 14, (M, K)).astype(np.float32)
    W = rng.uniform(-1, 1, (N, K)).astype(np.float32)
    Wp = oracle.pack_sign(W, 32)
    got = _realx_i8(G, bnn, G.to_dev(X), G.to_dev(Wp), M, K, N, 32)
    want = X.astype(np.float64) @ oracle.unpack_pm1(Wp, K, 32).T.astype(np.float64)   # |sum| <= 320 2^14 < 2^24
    assert np.array_equal(got.astype(np.float64), want)


def test_layer_binw_realx_int8_rows_that_cannot_be_quantised(G, bnn, oracle):
    """Frames with NaN, Inf or values beyond 2^90 take the fp32 sum in ascending k: the bits of bnn_layer_binw_realx."""
    M, K, N, wb = 140, 700, 300, 32
    rng = np.random.default_rng(3)
    X = rng.standard_normal((M, K)).astype(np.float32)
    X[3, 17] = np.inf
    X[4, 100] = np.nan
    X[5] *= np.float32(1e30)
    X[6] = 0.0
    W = rng.uniform(-1, 1, (N, K)).astype(np.float32)
    Wp = oracle.pack_sign(W, wb)
    dX, dWp = G.to_dev(X), G.to_dev(Wp)
    got = _realx_i8(G, bnn, dX, dWp, M, K, N, wb)
    with np.errstate(all="ignore"):
        acc32, acc64 = oracle.realx_acc(X, oracle.unpack_pm1(Wp, K, wb))
    for m in (3, 4, 5):
        assert np.array_equal(got[m].view(np.uint32), acc32[m].view(np.uint32)), m
    assert np.all(got[6] == 0.0)
    rest = np.ones(M, bool); rest[[3, 4, 5]] = False
    bound = K * 2.0 ** -27 * np.abs(X[rest]).max(1, keepdims=True).astype(np.float64)
    assert np.all(np.abs(got[rest].astype(np.float64) - acc64[rest]) <= bound + 2.0 ** -23 * np.abs(acc64[rest]))


@pytest.mark.parametrize("M,N,K", [(256, 300, 200), (1024, 512, 2048), (4096, 130, 257)])
def test_backward_products_on_the_int8_matrix_cores(G, bnn, oracle, T, M, N, K):
    """Both backward products of Alg. 1 through bnn_layer_binw_realx_i8 (g_h = g_hhat w^b with the transposed signs,
    g_w = g_hhat^T h with the bits of h^T): within M or N times 2^-27 of the largest gradient of the row of the oracle's
    product (whose own fp32 chain is further from the exact sum than that)."""
    rng = np.random.default_rng(M + N + K)
    g = (rng.standard_normal((M, N)) * np.exp(rng.uniform(-6, 0, (M, 1)))).astype(np.float32)   # frames of very different weight
    W = rng.uniform(-1, 1, (N, K)).astype(np.float32)
    hhat_prev = rng.standard_normal((M, K)).astype(np.float32)
    dg, dW, dhh = G.to_dev(g), G.to_dev(W), G.to_dev(hhat_prev)
    WpT, HpT, gt = G.word_tensor(K, N, 32), G.word_tensor(K, M, 32), _f32(N, M)
    bnn.bnn_pack_weights_transposed(G.ptr(dW), N, K, 32, G.ptr(WpT), G.stream())
    bnn.bnn_pack_weights_transposed(G.ptr(dhh), M, K, 32, G.ptr(HpT), G.stream())
    bnn.bnn_transpose_f32(G.ptr(dg), M, N, G.ptr(gt), G.stream())
    gh = _realx_i8(G, bnn, dg, WpT, M, N, K, 32)              # rows: frames, summed over the N outputs
    gw = _realx_i8(G, bnn, gt, HpT, N, M, K, 32)              # rows: outputs, summed over the M frames
    want_h = T.backward_input_binw(g, np.where(W > 0, 1, -1).astype(np.int8)).astype(np.float64)
    want_w = T.backward_weight(g, np.where(hhat_prev > 0, 1.0, -1.0).astype(np.float32)).astype(np.float64)
    u = 2.0 ** -24
    tol_h = (N * 2.0 ** -27 + N * u) * np.abs(g).max(1, keepdims=True) * 1.0 + N * u * np.abs(g).sum(1, keepdims=True)
    tol_w = (M * 2.0 ** -27) * np.abs(g).max(0)[:, None] + M * u * np.abs(g).sum(0)[:, None]
    assert np.all(np.abs(gh - want_h) <= tol_h)
    assert np.all(np.abs(gw - want_w) <= tol_w)
    # against the exact products (fp64; the oracle's fp32 chains are further from them than the matrix-core sums): the
    # bound the header states plus the one rounding to fp32
    g64, s_w, s_h = g.astype(np.float64), np.where(W > 0, 1.0, -1.0), np.where(hhat_prev > 0, 1.0, -1.0)
    exact_h, exact_w = g64 @ s_w, g64.T @ s_h
    assert np.all(np.abs(gh - exact_h) <= N * 2.0 ** -27 * np.abs(g64).max(1, keepdims=True) + 2.0 ** -23 * np.abs(exact_h))
    assert np.all(np.abs(gw - exact_w) <= M * 2.0 ** -27 * np.abs(g64).max(0)[:, None] + 2.0 ** -23 * np.abs(exact_w))


@pytest.mark.parametrize("M,N", [(1, 1), (255, 15), (256, 16), (257, 33), (513, 68), (1030, 20), (300, 12288), (1, 12289), (33, 12289),
                                 (70, 20000)])
def test_bias_grad_slabs(G, bnn, T, M, N):
    """Column sums at the edges of the 256-row slabs and of the 16-column workgroups, rows 16-byte aligned or not; with more
    than 12288 columns at the edges of the 32 rows that one wave per 64 columns requests at a time."""
    g = np.random.default_rng(M * N).standard_normal((M, N)).astype(np.float32)
    out = _f32(1, N)
    dg = G.to_dev(g)
    bnn.bnn_bias_grad(G.ptr(dg), M, N, G.ptr(out), G.stream())
    assert np.array_equal(out.cpu().numpy()[0], T.bias_grad(g))


def test_elementwise_kernels_on_unaligned_arrays(G, bnn, T):
    """Arrays at 4 bytes past a 16-byte boundary take the one-element accesses: the same values."""
    rng = np.random.default_rng(12)
    n = 4099
    a, h, w = (rng.standard_normal(n).astype(np.float32) for _ in range(3))
    da, dh, dw = (torch.cat([torch.zeros(1, device="cuda:0"), G.to_dev(v)]) for v in (a, h, w))
    pa, ph, pw = (t.data_ptr() + 4 for t in (da, dh, dw))
    bnn.bnn_update_clip(pw, pa, n, 0.1, 1, G.stream())
    assert np.array_equal(dw[1:].cpu().numpy(), T.update_clip(w, a, 0.1, True))
    bnn.bnn_sigmoid_grad(pa, ph, n, pw, G.stream())
    assert np.array_equal(dw[1:].cpu().numpy(), T.sigmoid_grad(a, h))
    ws, norm = torch.empty(2048, dtype=torch.uint8, device="cuda:0"), _f32(1, 1)
    bnn.bnn_grad_norm_clip(pa, n, 1.0, G.ptr(ws), G.ptr(norm), G.stream())
    want, want_norm = T.grad_norm_clip(a, 1.0)
    assert abs(float(norm) - float(want_norm)) <= 1e-6 * float(want_norm)
    assert np.max(np.abs(da[1:].cpu().numpy() - want)) <= 1e-6 * np.max(np.abs(want))
    bnn.bnn_mask_grad(ph, pw, n, 0.2, ph, G.stream())
    assert np.array_equal(dh[1:].cpu().numpy(), T.mask_grad(h, T.sigmoid_grad(a, h), 0.2))


@pytest.mark.parametrize("clip", [0, 1])
def test_update_clip(G, bnn, T, clip):
    rng = np.random.default_rng(5)
    w = rng.uniform(-1, 1, 300001).astype(np.float32)
    g = (rng.standard_normal(300001) * 30).astype(np.float32)
    dw, dg = G.to_dev(w), G.to_dev(g)
    bnn.bnn_update_clip(G.ptr(dw), G.ptr(dg), w.size, 0.008, clip, G.stream())
    want = T.update_clip(w, g, 0.008, bool(clip))
    assert np.array_equal(dw.cpu().numpy(), want)
    if clip:
        assert np.abs(want).max() == 1.0 and (np.abs(want) == 1.0).mean() > 0.01


@pytest.mark.parametrize("alpha", [15.0, 1e6])
@pytest.mark.parametrize("count", [1, 1000, 2048 * 440, 2048 * 2048 + 3])
def test_grad_norm_clip(G, bnn, T, count, alpha):
    g = (np.random.default_rng(count).standard_normal(count) * 0.05).astype(np.float32)
    dg = G.to_dev(g)
    ws = torch.empty(4096, dtype=torch.uint8, device="cuda:0")
    norm = torch.full((1,), float("nan"), dtype=torch.float32, device="cuda:0")
    bnn.bnn_grad_norm_clip(G.ptr(dg), count, alpha, G.ptr(ws), G.ptr(norm), G.stream())
    want, want_norm = T.grad_norm_clip(g, alpha)
    got_norm = float(norm.cpu().numpy()[0])
    assert abs(got_norm - float(want_norm)) <= 1e-6 * float(want_norm) + 1e-30
    got = dg.cpu().numpy()
    if float(want_norm) <= alpha:
        assert np.array_equal(got, g)                      # at or below the threshold: untouched
    else:
        assert np.max(np.abs(got - want)) <= 1e-6 * np.max(np.abs(want))
        assert abs(np.linalg.norm(got.astype(np.float64)) - alpha) <= 1e-4 * alpha


@pytest.mark.parametrize("count", [3, 1024 * 1024 * 4 + 5])
@pytest.mark.parametrize("at", [0, 4, 1024, 2044])
def test_grad_norm_clip_with_the_norm_inside_the_workspace(G, bnn, count, at):
    """norm_out among the 2048 bytes of partial sums: the same bits as with a float of its own."""
    g = G.to_dev((np.random.default_rng(count).standard_normal(count) * 20.0).astype(np.float32))
    want, norm, ws = g.clone(), _f32(1, 1), torch.empty(2048, dtype=torch.uint8, device="cuda:0")
    bnn.bnn_grad_norm_clip(G.ptr(want), count, 15.0, G.ptr(ws), G.ptr(norm), G.stream())
    bnn.bnn_grad_norm_clip(G.ptr(g), count, 15.0, G.ptr(ws), G.ptr(ws) + at, G.stream())
    assert torch.equal(ws[at:at + 4].view(torch.float32), norm.view(-1)) and float(norm) > 15.0
    assert torch.equal(g, want)


def test_semi_stochastic_binarize(G, bnn, T):
    rng = np.random.default_rng(9)
    w = rng.uniform(-1, 1, 500003).astype(np.float32)
    w[:3] = [0.0, 1.0, -1.0]
    u = rng.uniform(0, 1, w.size).astype(np.float32)
    dw, du = G.to_dev(w), G.to_dev(u)
    bnn.bnn_semi_stochastic_binarize(G.ptr(dw), G.ptr(du), w.size, G.stream())
    assert np.array_equal(dw.cpu().numpy(), T.semi_stochastic_binarize(w, u))


def test_one_training_step_of_a_binary_network(G, bnn, oracle, T):
    """Alg. 1 + Alg. 2 on a small (sign, sign, softmax) network with binary weights: forward with pre-activations kept,
    backward and update through the C ABI, every gradient and the updated weights against the oracle's."""
    import workloads
    cfg = workloads.NetConfig(21, "train", (40, 96, 64, 30), 70, "sign", 32)
    Ws, rs = workloads.make_net_params(cfg)
    X = workloads.make_frames(cfg)
    labels = np.random.default_rng(1).integers(0, 30, cfg.M).astype(np.int32)
    M, k_mask, eta, alpha = cfg.M, 1.0, 0.001, 15.0
    L = len(Ws)
    # ---- oracle (no per-layer scale: the paper's layer)
    hs, hhats = [X], []
    for l, (W, r) in enumerate(zip(Ws, rs)):
        Wb = np.where(W > 0, 1, -1).astype(np.int8)
        x_real = hs[-1] if l == 0 else oracle.bits_to_real(hs[-1], W.shape[1], 32, False)
        hhat = oracle.affine_f32(oracle.realx_acc(x_real, Wb, want64=False)[0], None, r)
        hhats.append(hhat)
        hs.append(oracle.pack_sign(hhat, 32) if l < L - 1 else oracle.log_softmax(hhat)[0])
    want_gw, want_gr = [None] * L, [None] * L
    g = T.softmax_xent_grad(hs[-1], labels)
    for l in range(L - 1, -1, -1):
        if l < L - 1:
            g = T.mask_grad(g, hhats[l], k_mask)
        x_real = hs[l] if l == 0 else oracle.bits_to_real(hs[l], Ws[l].shape[1], 32, False)
        want_gw[l], want_gr[l] = T.backward_weight(g, x_real), T.bias_grad(g)
        if l > 0:
            g = T.backward_input_binw(g, np.where(Ws[l] > 0, 1, -1).astype(np.int8))
    # ---- GPU, through the C ABI
    st = G.stream()
    dX, dlab = G.to_dev(X), G.to_dev(labels)
    dW = [G.to_dev(W) for W in Ws]
    dr = [G.to_dev(r) for r in rs]
    acts, hh = [dX], []
    for l in range(L):
        N, K = Ws[l].shape
        Wp = G.word_tensor(N, K, 32)
        bnn.bnn_pack_weights(G.ptr(dW[l]), N, K, 32, G.ptr(Wp), 0, st)
        z = _f32(M, N)
        if l == 0:
            bnn.bnn_layer_binw_realx(G.ptr(acts[-1]), G.ptr(Wp), 0, G.ptr(dr[l]), M, K, N, bnn.BNN_ACT_LINEAR, 32, G.ptr(z), st)
        else:
            bnn.bnn_layer_binw_binx(G.ptr(acts[-1]), G.ptr(Wp), 0, G.ptr(dr[l]), M, K, N, bnn.BNN_ACT_LINEAR, 32, G.ptr(z), st)
        hh.append(z)
        if l < L - 1:
            acts.append(G.pack_activations(z, 32))
    assert all(np.array_equal(a.cpu().numpy(), b) for a, b in zip(hh, hhats))
    logp = _f32(M, 30)
    N, K = Ws[-1].shape
    Wp = G.word_tensor(N, K, 32)
    bnn.bnn_pack_weights(G.ptr(dW[-1]), N, K, 32, G.ptr(Wp), 0, st)
    bnn.bnn_layer_binw_binx(G.ptr(acts[-1]), G.ptr(Wp), 0, G.ptr(dr[-1]), M, K, N, bnn.BNN_ACT_LOGSOFTMAX, 32, G.ptr(logp), st)
    dg, dlab = _f32(M, 30), G.to_dev(labels)
    bnn.bnn_softmax_xent_grad(G.ptr(logp), G.ptr(dlab), M, 30, G.ptr(dg), st)
    ws = torch.empty(4096, dtype=torch.uint8, device="cuda:0")
    norm = torch.zeros(1, dtype=torch.float32, device="cuda:0")
    for l in range(L - 1, -1, -1):
        N, K = Ws[l].shape
        if l < L - 1:
            bnn.bnn_mask_grad(G.ptr(dg), G.ptr(hh[l]), M * N, k_mask, G.ptr(dg), st)
        x_real = acts[l] if l == 0 else G.unpack_activations(acts[l], K, 32, False)
        gt, ht, gw = _f32(N, M), _f32(K, M), _f32(N, K)
        gr = torch.empty(N, dtype=torch.float32, device="cuda:0")
        bnn.bnn_transpose_f32(G.ptr(dg), M, N, G.ptr(gt), st)
        bnn.bnn_transpose_f32(G.ptr(x_real), M, K, G.ptr(ht), st)
        bnn.bnn_backward_weight(G.ptr(gt), G.ptr(ht), N, K, M, G.ptr(gw), st)
        bnn.bnn_bias_grad(G.ptr(dg), M, N, G.ptr(gr), st)
        tol = 2e-6 * float(np.max(np.abs(want_gw[l])))      # the Softmax gradient goes through exp: not bit for bit
        assert np.max(np.abs(gw.cpu().numpy() - want_gw[l])) <= tol, l
        assert np.max(np.abs(gr.cpu().numpy() - want_gr[l])) <= 2e-6 * float(np.max(np.abs(want_gr[l]))), l
        if l > 0:
            WpT = G.word_tensor(K, N, 32)
            bnn.bnn_pack_weights_transposed(G.ptr(dW[l]), N, K, 32, G.ptr(WpT), st)
            gh = _f32(M, K)
            bnn.bnn_backward_input_binw(G.ptr(dg), G.ptr(WpT), M, N, K, 32, G.ptr(gh), st)
            dg = gh
        # update: norm clip, Clip(w - eta g), bias
        bnn.bnn_grad_norm_clip(G.ptr(gw), N * K, alpha, G.ptr(ws), G.ptr(norm), st)
        bnn.bnn_update_clip(G.ptr(dW[l]), G.ptr(gw), N * K, eta, 1, st)
        bnn.bnn_update_clip(G.ptr(dr[l]), G.ptr(gr), N, eta, 0, st)
        want_w = T.update_clip(Ws[l], T.grad_norm_clip(want_gw[l], alpha)[0], eta, True)
        got_w = dW[l].cpu().numpy()
        assert np.max(np.abs(got_w - want_w)) <= 1e-6 and np.abs(got_w).max() <= 1.0
        assert np.mean(np.sign(got_w) == np.sign(want_w)) > 0.9999


def test_backward_of_the_paper_topology(G, bnn, oracle, T):
    """(sigma, b, b, sigma, delta) with real-valued input and Softmax weights and binary weights in between (Table 2,
    Sec. 3.1), small: the forward pass keeps pre-activations, the backward pass goes through every kind of step
    (Sigmoid derivative, Mask, both weight-gradient forms, both input-gradient forms).  Each gradient is checked
    against the oracle's, which is fed the GPU's own incoming gradient of that layer (layer-by-layer, so that the
    fp64 exp of the Softmax gradient cannot make later comparisons inexact)."""
    import workloads
    cfg = workloads.NetConfig(22, "train paper topology", (40, 64, 96, 64, 70, 30), 130,
                              ("sigmoid", "sign", "sign", "sigmoid"), 32, real_weight_layers=(0, 4))
    Ws, rs = workloads.make_net_params(cfg)
    X = workloads.make_frames(cfg)
    M, L, st = cfg.M, 5, G.stream()
    acts = ["sigmoid", "sign", "sign", "sigmoid", "logsoftmax"]
    labels = np.random.default_rng(2).integers(0, 30, M).astype(np.int32)
    # ---- forward on the GPU, keeping what the backward pass needs; checked against the oracle as it goes
    dX = G.to_dev(X)
    dW = [G.to_dev(W) for W in Ws]
    dr = [G.to_dev(r) for r in rs]
    h_real = [dX]          # real-valued input of layer l (frames, Sigmoid outputs) or None where the input is bits
    h_bits, hhat = [None], []
    for l in range(L):
        N, K = Ws[l].shape
        z = _f32(M, N)
        if l in cfg.real_weight_layers:
            bnn.bnn_layer_realw(G.ptr(h_real[l]), G.ptr(dW[l]), G.ptr(dr[l]), M, K, N, bnn.BNN_ACT_LINEAR, 32, G.ptr(z), st)
        else:
            Wp = G.word_tensor(N, K, 32)
            bnn.bnn_pack_weights(G.ptr(dW[l]), N, K, 32, G.ptr(Wp), 0, st)
            if h_real[l] is not None:
                bnn.bnn_layer_binw_realx(G.ptr(h_real[l]), G.ptr(Wp), 0, G.ptr(dr[l]), M, K, N, bnn.BNN_ACT_LINEAR, 32, G.ptr(z), st)
            else:
                bnn.bnn_layer_binw_binx(G.ptr(h_bits[l]), G.ptr(Wp), 0, G.ptr(dr[l]), M, K, N, bnn.BNN_ACT_LINEAR, 32, G.ptr(z), st)
        hhat.append(z)
        zh = z.cpu().numpy()
        if acts[l] == "sign":
            h_bits.append(G.pack_activations(z, 32)); h_real.append(None)
        elif acts[l] == "sigmoid":
            h_real.append(G.to_dev(oracle.sigmoid(zh))); h_bits.append(None)     # the oracle's Sigmoid of the GPU's h^
        else:
            logp = G.to_dev(oracle.log_softmax(zh)[0])
    # ---- backward
    dg, dlab = _f32(M, 30), G.to_dev(labels)
    bnn.bnn_softmax_xent_grad(G.ptr(logp), G.ptr(dlab), M, 30, G.ptr(dg), st)
    assert np.max(np.abs(dg.cpu().numpy() - T.softmax_xent_grad(logp.cpu().numpy(), labels))) <= 1e-6
    for l in range(L - 1, -1, -1):
        N, K = Ws[l].shape
        g_in = dg.cpu().numpy()                                  # the oracle continues from the GPU's gradient
        if acts[l] == "sign":
            bnn.bnn_mask_grad(G.ptr(dg), G.ptr(hhat[l]), M * N, 1.0, G.ptr(dg), st)
            want_g = T.mask_grad(g_in, hhat[l].cpu().numpy(), 1.0)
        elif acts[l] == "sigmoid":
            bnn.bnn_sigmoid_grad(G.ptr(dg), G.ptr(h_real[l + 1]), M * N, G.ptr(dg), st)
            want_g = T.sigmoid_grad(g_in, h_real[l + 1].cpu().numpy())
        else:
            want_g = g_in
        assert np.array_equal(dg.cpu().numpy(), want_g), l
        gt, gw = _f32(N, M), _f32(N, K)
        gr = torch.empty(N, dtype=torch.float32, device="cuda:0")
        bnn.bnn_transpose_f32(G.ptr(dg), M, N, G.ptr(gt), st)
        if h_real[l] is not None:                                 # real input: multiply kernel
            ht = _f32(K, M)
            bnn.bnn_transpose_f32(G.ptr(h_real[l]), M, K, G.ptr(ht), st)
            bnn.bnn_backward_weight(G.ptr(gt), G.ptr(ht), N, K, M, G.ptr(gw), st)
            want_gw = T.backward_weight(want_g, h_real[l].cpu().numpy())
        else:                                                     # input = Sign(h^ of the layer below): add/subtract kernel
            HpT = G.word_tensor(K, M, 32)
            bnn.bnn_pack_weights_transposed(G.ptr(hhat[l - 1]), M, K, 32, G.ptr(HpT), st)
            bnn.bnn_backward_weight_binh(G.ptr(gt), G.ptr(HpT), N, K, M, 32, G.ptr(gw), st)
            want_gw = T.backward_weight(want_g, np.where(hhat[l - 1].cpu().numpy() > 0, 1.0, -1.0).astype(np.float32))
        bnn.bnn_bias_grad(G.ptr(dg), M, N, G.ptr(gr), st)
        assert np.array_equal(gw.cpu().numpy(), want_gw), l
        assert np.array_equal(gr.cpu().numpy(), T.bias_grad(want_g)), l
        if l > 0:
            gh = _f32(M, K)
            if l in cfg.real_weight_layers:
                Wt = _f32(K, N)
                bnn.bnn_transpose_f32(G.ptr(dW[l]), N, K, G.ptr(Wt), st)
                bnn.bnn_backward_input_realw(G.ptr(dg), G.ptr(Wt), M, N, K, G.ptr(gh), st)
                want_gh = T.backward_input_realw(want_g, Ws[l])
            else:
                WpT = G.word_tensor(K, N, 32)
                bnn.bnn_pack_weights_transposed(G.ptr(dW[l]), N, K, 32, G.ptr(WpT), st)
                bnn.bnn_backward_input_binw(G.ptr(dg), G.ptr(WpT), M, N, K, 32, G.ptr(gh), st)
                want_gh = T.backward_input_binw(want_g, np.where(Ws[l] > 0, 1, -1).astype(np.int8))
            assert np.array_equal(gh.cpu().numpy(), want_gh), l
            dg = gh
