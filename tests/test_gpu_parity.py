"""Parity of the HIP library (called through its C ABI) against the CPU oracle,
element by element, on seeded inputs that span several tiles and ragged tails.
See parity_util.py for the comparison rules."""
import numpy as np
import pytest
import torch

import oracle
from paper_2203_15952_amd import binding as B
from paper_2203_15952_amd import inputs
from parity_util import REL_F, check_float_forward, check_forward, check_grad, unpack_mask

pytestmark = pytest.mark.gpu
F = np.float32


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def say(*a):
    print(*a, flush=True)


# ----------------------------------------------------------------------------
# quantizers
# ----------------------------------------------------------------------------
@pytest.mark.parametrize("shape", [(256, 256), (1000, 517), (1, 1), (3, 5), (2, 1027), (12800, 512)])
@pytest.mark.parametrize("bits", [8, 4])
def test_quantize_per_tensor(shape, bits):
    say("quantize per tensor", shape, bits)
    rng = np.random.default_rng(shape[0] * 7 + shape[1] + bits)
    x = rng.standard_normal(shape).astype(F)
    q_ref, s_ref = oracle.quantize(x, bits, oracle.AXIS_ALL)
    status = B.new_status()
    q, s, _ = B.aqt_quantize(dev(x), bits, B.AQT_AXIS_ALL, dev_status=status)
    np.testing.assert_array_equal(host(s), s_ref)
    np.testing.assert_array_equal(host(q), q_ref)
    assert host(status)[0] == 0
    # the masked variant takes the general kernels: same codes, all-ones mask
    q2, s2, mask = B.aqt_quantize(dev(x), bits, B.AQT_AXIS_ALL, want_mask=True)
    np.testing.assert_array_equal(host(q2), q_ref)
    np.testing.assert_array_equal(host(s2), s_ref)
    assert unpack_mask(host(mask), x.size).all()


@pytest.mark.parametrize("axis", [B.AQT_AXIS_ROWS, B.AQT_AXIS_COLS])
@pytest.mark.parametrize("shape", [(512, 2048), (77, 131), (1, 9), (9, 1)])
def test_quantize_per_channel(axis, shape):
    say("quantize per channel", axis, shape)
    rng = np.random.default_rng(shape[0] + 3 * shape[1] + axis)
    x = (rng.standard_normal(shape) * rng.uniform(0.1, 10, (1, shape[1]))).astype(F)
    q_ref, s_ref, m_ref = oracle.quantize(x, 4, axis, want_mask=True)
    q, s, mask = B.aqt_quantize(dev(x), 4, axis, want_mask=True)
    np.testing.assert_array_equal(host(s), s_ref)
    np.testing.assert_array_equal(host(q), q_ref)
    np.testing.assert_array_equal(unpack_mask(host(mask), x.size), m_ref.reshape(-1))


def test_quantize_strided_rows():
    say("quantize strided")
    rng = np.random.default_rng(21)
    big = rng.standard_normal((40, 100)).astype(F)
    x = big[:, :73]
    for axis in (B.AQT_AXIS_ALL, B.AQT_AXIS_ROWS, B.AQT_AXIS_COLS):
        q_ref, s_ref = oracle.quantize(np.ascontiguousarray(x), 8, axis)
        q, s, _ = B.aqt_quantize(dev(big), 8, axis, ldx=100, cols=73)
        np.testing.assert_array_equal(host(s), s_ref)
        np.testing.assert_array_equal(host(q), q_ref)


def test_quantize_ties_zero_groups_and_denormals():
    say("quantize ties / zeros / denormals")
    t = np.nextafter(F(0.5), F(0))
    x = np.array([[127.0, 0.5, -0.5, 1.5, -1.5, 2.5, -2.5, t, -t, -127.0]], F)
    q, s, _ = B.aqt_quantize(dev(x), 8, B.AQT_AXIS_ALL)
    assert host(s)[0] == 1.0
    assert host(q).tolist() == [[127, 1, 0, 2, -1, 3, -2, 1, 0, -127]]   # Fig. 2: floor(t + 0.5)
    z = np.zeros((4, 5), F)
    z[:, 1] = [1, -2, 3, -4]
    z[:, 3] = [1e-45, 0, -1e-45, 0]
    q_ref, s_ref, m_ref = oracle.quantize(z, 4, 0, want_mask=True)
    q, s, mask = B.aqt_quantize(dev(z), 4, B.AQT_AXIS_ROWS, want_mask=True)
    np.testing.assert_array_equal(host(q), q_ref)
    np.testing.assert_array_equal(host(s), s_ref)
    np.testing.assert_array_equal(unpack_mask(host(mask), z.size), m_ref.reshape(-1))
    q, s, _ = B.aqt_quantize(dev(np.zeros((8, 64), F)), 8, B.AQT_AXIS_ALL)
    assert host(s)[0] == 0 and not host(q).any()
    rng = np.random.default_rng(22)
    d = (rng.standard_normal((32, 96)) * 1e-38).astype(F)      # subnormal scale
    q_ref, s_ref = oracle.quantize(d, 8, oracle.AXIS_ALL)
    q, s, _ = B.aqt_quantize(dev(d), 8, B.AQT_AXIS_ALL)
    np.testing.assert_array_equal(host(s), s_ref)
    np.testing.assert_array_equal(host(q), q_ref)
    big = (rng.standard_normal((32, 96)) * 1e37).astype(F)
    q_ref, s_ref = oracle.quantize(big, 8, oracle.AXIS_ALL)
    q, s, _ = B.aqt_quantize(dev(big), 8, B.AQT_AXIS_ALL)
    np.testing.assert_array_equal(host(s), s_ref)
    np.testing.assert_array_equal(host(q), q_ref)


def test_nonfinite_sets_device_status():
    say("non-finite status")
    x = np.ones((64, 64), F)
    x[5, 7] = np.inf
    for axis in (B.AQT_AXIS_ALL, B.AQT_AXIS_ROWS, B.AQT_AXIS_COLS):
        status = B.new_status()
        B.aqt_quantize(dev(x), 8, axis, dev_status=status)
        assert host(status)[0] == B.AQT_ERR_NONFINITE
    x[5, 7] = np.nan
    status = B.new_status()
    B.aqt_quantize_weights(dev(x), 4, dev_status=status)
    assert host(status)[0] == B.AQT_ERR_NONFINITE


def test_quantize_with_scale_saturates_and_masks():
    say("quantize with external scale")
    rng = np.random.default_rng(23)
    x = (rng.standard_normal((50, 70)) * 3).astype(F)
    for axis, ns in ((B.AQT_AXIS_ALL, 1), (B.AQT_AXIS_ROWS, 70), (B.AQT_AXIS_COLS, 50)):
        scale = rng.uniform(0.2, 1.0, ns).astype(F)
        scale[0] = 0 if axis != B.AQT_AXIS_ALL else scale[0]
        q_ref, m_ref = oracle.quantize_with_scale(x, 4, axis, scale)
        assert 0 < m_ref.mean() < 1            # the case really saturates somewhere
        q, mask = B.aqt_quantize_with_scale(dev(x), 4, axis, dev(scale))
        np.testing.assert_array_equal(host(q), q_ref)
        np.testing.assert_array_equal(unpack_mask(host(mask), x.size), m_ref.reshape(-1))


@pytest.mark.parametrize("K,N", [(512, 2048), (256, 1024), (67, 45), (1, 1), (5, 33), (130, 31), (8, 64), (16, 36), (17, 33), (81, 64)])
@pytest.mark.parametrize("bits_w", [4, 8])
def test_quantize_weights_layouts(K, N, bits_w):
    say("quantize weights", K, N, bits_w)
    rng = np.random.default_rng(K + N + bits_w)
    w = (rng.standard_normal((K, N)) / np.sqrt(K)).astype(F)
    if N > 2:
        w[:, 2] = 0
    q_ref, s_ref, m_ref = oracle.quantize(w, bits_w, 0, want_mask=True)
    wq, s_w, wq_kn, mask = B.aqt_quantize_weights(dev(w), bits_w, want_mask=True)
    np.testing.assert_array_equal(host(s_w), s_ref)
    np.testing.assert_array_equal(host(wq_kn), q_ref)
    np.testing.assert_array_equal(unpack_mask(host(mask), w.size), m_ref.reshape(-1))
    if bits_w <= 4:
        np.testing.assert_array_equal(host(wq).reshape(N, (K + 1) // 2), oracle.pack_int4(q_ref))
    else:
        np.testing.assert_array_equal(host(wq).view(np.int8).reshape(N, K), q_ref.T)
    np.testing.assert_array_equal(host(B.aqt_unpack_weights(wq, K, N, bits_w)), q_ref)


# ----------------------------------------------------------------------------
# forward
# ----------------------------------------------------------------------------
FWD_CASES = [
    # M, K, N, bits_x, bits_w, epilogue, bias      (which kernel it lands on)
    (256, 256, 1024, 8, 4, 0, False),    # the single-layer config: 16 tiles of 128 x 128, split contraction
    (300, 128, 256, 8, 4, 0, True),      # ragged M
    (300, 128, 256, 8, 8, 1, True),      # int8 weights, Swish
    (200, 256, 512, 8, 4, 2, True),      # GLU
    (200, 384, 512, 8, 8, 2, False),     # odd number of fan-in stages
    (1100, 128, 128, 4, 4, 1, False),    # int4 activations, a single stage
    (130, 192, 256, 8, 4, 0, True),      # fan-in not a multiple of the tuned kernel's stage
    (37, 50, 23, 8, 4, 0, True),         # odd N
    (37, 51, 24, 8, 8, 2, True),         # odd K, GLU
    (5, 7, 3, 8, 4, 1, False),
    (1, 1, 1, 8, 8, 0, False),
    (2100, 128, 512, 8, 4, 1, True),     # tuned kernel (more than 32 tiles of 128 x 128, 64 from K = 512 on): one stage, ragged M
    (2176, 256, 512, 8, 8, 2, True),     # GLU on the tuned kernel, whole row tiles
    (1500, 640, 768, 8, 4, 2, False),    # the same with five stages, ragged M
    (4200, 256, 256, 4, 4, 0, True),
]


@pytest.mark.parametrize("M,K,N,bx,bw,epi,with_bias", FWD_CASES)
def test_dense_fwd_against_oracle(M, K, N, bx, bw, epi, with_bias):
    say("dense fwd", M, K, N, bx, bw, epi, with_bias)
    c = inputs.small_case(31 + M + K + N, M, K, N, bx, bw, epi, with_bias=with_bias, with_dy=False)
    ora = oracle.dense_fwd(c.x, c.w, bx, bw, c.bias, epi)
    bias = None if c.bias is None else dev(c.bias)
    # staged: quantize, quantize weights, contraction with accumulators exposed
    xq, s_x, _ = B.aqt_quantize(dev(c.x), bx, B.AQT_AXIS_ALL)
    wq, s_w, wq_kn, _ = B.aqt_quantize_weights(dev(c.w), bw)
    np.testing.assert_array_equal(host(xq), ora["xq"])
    np.testing.assert_array_equal(host(s_x), ora["s_x"])
    np.testing.assert_array_equal(host(wq_kn), ora["wq"])
    np.testing.assert_array_equal(host(s_w), ora["s_w"])
    y, acc = B.aqt_dense_fwd_q(xq, s_x, wq, s_w, N, bx, bw, bias=bias, epilogue=epi, want_acc=True)
    np.testing.assert_array_equal(host(acc), ora["acc"])
    check_forward(host(y), ora, ora["s_x"][0], ora["s_w"], c.bias, epi)
    # fused training forward: what is trained is what is served, bit for bit
    y2 = B.aqt_dense_fwd(dev(c.x), dev(c.w), bx, bw, bias=bias, epilogue=epi)
    np.testing.assert_array_equal(host(y2), host(y))


@pytest.mark.parametrize("M,K,N", [(1, 64, 4), (33, 64, 36), (31, 68, 2044), (256, 256, 1024), (97, 252, 100), (64, 132, 60),
                                   (32, 256, 64), (45, 260, 64), (40, 60, 64)])   # the last two: fan-ins next to the range
@pytest.mark.parametrize("bw,epi", [(8, 0), (4, 1), (3, 0)])
def test_small_dense_layers_quantize_inside_the_product(M, K, N, bw, epi):
    """Everything that the two quantizers and the product leave behind, in one launch behind the maxima: as called one by one."""
    say("dense in two launches", M, K, N, bw, epi)
    rng = np.random.default_rng(41 + M + K + N)
    x, w = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((K, N)).astype(np.float32)
    w[:, N // 2] = 0.0
    x_d, w_d, bias = dev(x), dev(w), dev(rng.standard_normal(N).astype(np.float32))
    xq, s_x, _ = B.aqt_quantize(x_d, 8, B.AQT_AXIS_ALL)
    wq, s_w, wq_kn, _ = B.aqt_quantize_weights(w_d, bw)
    want, _ = B.aqt_dense_fwd_q(xq, s_x, wq, s_w, N, 8, bw, bias=bias, epilogue=epi)
    sv, status = B.Saved(M, K, N, bw), B.new_status()
    for t in (sv.xq, sv.wq_packed, sv.wq_kn):
        t.fill_(85)
    y = B.aqt_dense_fwd(x_d, w_d, 8, bw, bias=bias, epilogue=epi, saved=sv, dev_status=status)
    for got, ref in ((sv.xq, xq), (sv.s_x, s_x), (sv.wq_packed, wq), (sv.s_w, s_w), (sv.wq_kn, wq_kn), (y, want)):
        np.testing.assert_array_equal(host(got).reshape(-1), host(ref).reshape(-1))
    assert host(status)[0] == 0
    for t in (x, w):   # a value that is not finite is reported, whichever tensor holds it
        keep, t[-1, -1] = t[-1, -1], np.nan
        status = B.new_status()
        B.aqt_dense_fwd(dev(x), dev(w), 8, bw, bias=bias, epilogue=epi, dev_status=status)
        assert host(status)[0] == B.AQT_ERR_NONFINITE
        t[-1, -1] = keep


def test_weights_of_more_than_two_to_the_35_elements():
    """More blocks than one grid dimension can hold: 2048 x (2^24 + 64), 137 GB, copies of one matrix side by side."""
    K, block, copies, rest = 2048, 1 << 16, 1 << 8, 64
    N = block * copies + rest
    if torch.cuda.mem_get_info()[0] < 230 << 30:
        pytest.skip("needs 230 GB of device memory")
    say("weights", K, N)
    gen = torch.Generator(device="cuda").manual_seed(44)
    one = torch.randn((K, block), device="cuda", generator=gen)
    w = torch.empty((K, N), device="cuda")
    w[:, : block * copies].unflatten(1, (copies, block)).copy_(one[:, None, :])
    w[:, block * copies:] = one[:, :rest]
    ref, s_ref, _, _ = B.aqt_quantize_weights(one, 4, want_kn=False)
    x = torch.randn((1, K), device="cuda", generator=gen)
    sv = B.Saved(1, K, block, 4)
    y_ref = B.aqt_dense_fwd(x, one, 8, 4, saved=sv)

    def check(wq, s_w, y=None):
        wq = wq.view(N, K // 2)
        for i in range(copies + 1):
            n = block if i < copies else rest
            at = slice(i * block, i * block + n)
            assert torch.equal(wq[at], ref.view(block, K // 2)[:n]) and torch.equal(s_w[at], s_ref[:n]), i
            assert y is None or torch.equal(y[0, at], y_ref[0, :n]), i

    wq, s_w, _, _ = B.aqt_quantize_weights(w, 4, want_kn=False)
    check(wq, s_w)
    wq.zero_()
    s_w.zero_()
    sv.wq_packed, sv.s_w, sv.wq_kn, sv.N = wq, s_w, None, N
    y = torch.empty((1, N), device="cuda")
    B.aqt_dense_fwd(x, w, 8, 4, y=y, saved=sv.refresh())
    check(wq, s_w, y)
    del w, wq
    torch.cuda.empty_cache()


@pytest.mark.parametrize("M,K,bw,epi", [(256, 256, 4, 0), (40, 64, 8, 1), (1000, 100, 8, 0), (300, 260, 4, 0), (512, 128, 4, 1)])
@pytest.mark.parametrize("where", ["x", "w", "dact", "codes"])
def test_dense_fwd_into_its_own_inputs(M, K, bw, epi, where):
    """What the product writes may lie over x or w, and the weights' codes over x: as the three calls in sequence."""
    say("dense in place", M, K, bw, epi, where)
    N, rng = K, np.random.default_rng(43 + M + K)
    x, w, bias = (dev(rng.standard_normal(s).astype(np.float32)) for s in ((M, K), (K, N), N))
    B.aqt_dense_fwd(x, w, 8, bw, bias=bias, epilogue=epi, saved=(ref := B.Saved(M, K, N, bw, dact=True)),
                    y=(want := torch.empty((M, N), device="cuda")))
    for _ in range(3):
        both = torch.empty(max(M, K), K, device="cuda")   # y over w needs M rows behind it
        sv = B.Saved(M, K, N, bw, dact=True)
        xi, wi, y = x, w, torch.empty((M, N), device="cuda")
        if where == "w":
            both[:K] = w
            wi, y = both[:K], both[:M]
        else:
            both[:M] = x
            xi = both[:M]
            if where == "x":
                y = xi
            elif where == "dact":
                sv.dact = xi
            else:
                sv.wq_kn = both.view(torch.int8).view(-1)[: K * N].view(K, N)
        B.aqt_dense_fwd(xi, wi, 8, bw, bias=bias, epilogue=epi, y=y, saved=sv.refresh())
        np.testing.assert_array_equal(host(y), host(want))
        names = ["xq", "s_x", "wq_packed", "s_w", "wq_kn"] + (["dact"] if epi else [])
        for name in names:
            np.testing.assert_array_equal(host(getattr(sv, name)), host(getattr(ref, name)), err_msg=name)


@pytest.mark.parametrize("M,K,N,bw,epi", [(300, 128, 256, 4, 1), (200, 256, 512, 8, 2), (16500, 1152, 1024, 4, 0),
                                          (12800, 512, 2048, 4, 1)])
def test_prepared_weights_serving_path(M, K, N, bw, epi):
    # weights re-ordered once, then the contraction without workspace: bit-identical to aqt_dense_fwd_q
    say("prepared weights", M, K, N, bw, epi)
    c = inputs.small_case(131 + M + N, M, K, N, 8, bw, epi, with_bias=True, with_dy=False)
    bias = dev(c.bias)
    xq, s_x, _ = B.aqt_quantize(dev(c.x), 8, B.AQT_AXIS_ALL)
    wq, s_w, _, _ = B.aqt_quantize_weights(dev(c.w), bw)
    y_ref, _ = B.aqt_dense_fwd_q(xq, s_x, wq, s_w, N, 8, bw, bias=bias, epilogue=epi)
    wprep = B.aqt_prepare_weights(wq, K, N, bw)
    assert wprep.numel() == K * N // (2 if bw <= 4 else 1)
    for _ in range(2):
        y = B.aqt_dense_fwd_q_prepared(xq, s_x, wprep, s_w, N, 8, bw, bias=bias, epilogue=epi)
        np.testing.assert_array_equal(host(y), host(y_ref))
    # shapes the matrix-core kernel does not take are refused
    assert B.lib().aqt_prepared_weight_bytes(100, 256, bw) == 0
    with pytest.raises(B.AqtError) as e:
        B.aqt_dense_fwd_q_prepared(xq[:100].contiguous(), s_x, wprep, s_w, N, 8, bw)
    assert e.value.status == B.AQT_ERR_UNSUPPORTED


def test_dense_fwd_big_tiles_sampled():
    # the wide tiles; compare whole row tiles and sampled accumulators and outputs
    say("dense fwd big tiles")
    M, K, N = 16384, 1024, 2048
    c = inputs.small_case(41, M, K, N, 8, 4, 0, with_dy=False)
    ora_xq, ora_sx = oracle.quantize(c.x, 8, oracle.AXIS_ALL)
    ora_wq, ora_sw = oracle.quantize(c.w, 4, 0)
    xq, s_x, _ = B.aqt_quantize(dev(c.x), 8, B.AQT_AXIS_ALL)
    wq, s_w, wq_kn, _ = B.aqt_quantize_weights(dev(c.w), 4)
    np.testing.assert_array_equal(host(xq), ora_xq)
    np.testing.assert_array_equal(host(wq_kn), ora_wq)
    y, acc = B.aqt_dense_fwd_q(xq, s_x, wq, s_w, N, 8, 4, want_acc=True)
    acc_h, y_h = host(acc), host(y)
    rows = tile_rows(M)
    ora = oracle.dense_fwd_q(ora_xq[rows], ora_sx[0], ora_wq, ora_sw)
    np.testing.assert_array_equal(acc_h[rows], ora["acc"])
    check_forward(y_h[rows], ora, ora_sx[0], ora_sw, None, 0)
    # an int64 library matmul of the codes on a row slab, plus scattered samples
    rows = np.r_[0:64, 8000:8064, M - 64:M]
    ref = ora_xq[rows].astype(np.int64) @ ora_wq.astype(np.int64)
    np.testing.assert_array_equal(acc_h[rows], ref)
    rng = np.random.default_rng(0)
    im, inn = rng.integers(0, M, 4000), rng.integers(0, N, 4000)
    a, pre = oracle.dense_fwd_q_sampled(ora_xq, ora_sx[0], ora_wq, ora_sw, im, inn)
    np.testing.assert_array_equal(acc_h[im, inn], a)
    assert (np.abs(y_h[im, inn] - pre) <= 1e-6 * np.abs(pre) + 1e-37).all()


# ----------------------------------------------------------------------------
# backward
# ----------------------------------------------------------------------------
BWD_CASES = [(256, 256, 1024, 8, 4),    # small problems on the tuned grid: split contraction, slabs of rows
             (300, 128, 256, 8, 8),     # ragged M; dW off the grid (float64 kernel)
             (37, 50, 23, 8, 4),        # off the grid
             (5, 7, 3, 8, 8),
             (1024, 512, 384, 8, 4),
             (1000, 1024, 1024, 8, 4),  # several slabs, ragged M
             (70, 128, 96, 8, 4)]       # too few rows for the grid


@pytest.mark.parametrize("M,K,N,bx,bw", BWD_CASES)
def test_dense_bwd_against_oracle(M, K, N, bx, bw):
    say("dense bwd", M, K, N, bx, bw)
    c = inputs.small_case(51 + M + K + N, M, K, N, bx, bw)
    ora = oracle.dense_fwd(c.x, c.w, bx, bw)
    g = oracle.dense_bwd(c.dy, ora["xq"], ora["s_x"][0], ora["wq"], ora["s_w"])
    sv = B.Saved(M, K, N, bw)
    B.aqt_dense_fwd(dev(c.x), dev(c.w), bx, bw, saved=sv)
    np.testing.assert_array_equal(host(sv.xq), ora["xq"])
    np.testing.assert_array_equal(host(sv.wq_kn), ora["wq"])
    dx, dw, db = B.aqt_dense_bwd(dev(c.dy), sv, bx, bw, want_dbias=True)
    check_grad(host(dx), g["dx"], g["dx_abs"], "dx")
    check_grad(host(dw), g["dw"], g["dw_abs"], "dw")
    check_grad(host(db), g["dbias"], np.abs(c.dy.astype(np.float64)).sum(0), "dbias")


@pytest.mark.parametrize("M,K,N", [(96, 64, 48),        # off the tuned grid
                                   (300, 256, 128)])     # a small problem on it (the tuned kernels: TUNED_BWD_CASES)
def test_dense_bwd_masks_and_zero_groups(M, K, N):
    say("dense bwd masks", M, K, N)
    c = inputs.small_case(61, M, K, N, 8, 4)
    c.w[:, 5] = 0
    # externally supplied, too small scales make both masks non-trivial
    s_x = np.array([0.02], F)
    s_w = np.full(N, 0.01, F)
    s_w[5] = 0
    xq_ref, mx_ref = oracle.quantize_with_scale(c.x, 8, oracle.AXIS_ALL, s_x)
    wq_ref, mw_ref = oracle.quantize_with_scale(c.w, 4, 0, s_w)
    assert 0 < mx_ref.mean() < 1 and 0 < mw_ref.mean() < 1
    g = oracle.dense_bwd(c.dy, xq_ref, s_x[0], wq_ref, s_w, mx_ref, mw_ref)
    sv = B.Saved(M, K, N, 4, masks=True)
    B.aqt_quantize_with_scale(dev(c.x), 8, B.AQT_AXIS_ALL, dev(s_x), q=sv.xq, clip_mask=sv.mask_x)
    B.aqt_quantize_with_scale(dev(c.w), 4, B.AQT_AXIS_ROWS, dev(s_w), q=sv.wq_kn, clip_mask=sv.mask_w)
    sv.s_x.copy_(dev(s_x))
    sv.s_w.copy_(dev(s_w))
    dx, dw, _ = B.aqt_dense_bwd(dev(c.dy), sv, 8, 4)
    dx_h, dw_h = host(dx), host(dw)
    check_grad(dx_h, g["dx"], g["dx_abs"], "dx")
    check_grad(dw_h, g["dw"], g["dw_abs"], "dw")
    assert (dx_h[mx_ref == 0] == 0).all() and (dw_h[mw_ref == 0] == 0).all()
    # no masks given: "scale is non-zero" on both sides, the zero channel still gets no gradient
    sv2 = B.Saved(M, K, N, 4)
    B.aqt_dense_fwd(dev(c.x), dev(c.w), 8, 4, saved=sv2)
    ora2 = oracle.dense_fwd(c.x, c.w, 8, 4)
    g2 = oracle.dense_bwd(c.dy, ora2["xq"], ora2["s_x"][0], ora2["wq"], ora2["s_w"])
    dx2, dw2, _ = B.aqt_dense_bwd(dev(c.dy), sv2, 8, 4)
    check_grad(host(dx2), g2["dx"], g2["dx_abs"], "dx")
    check_grad(host(dw2), g2["dw"], g2["dw_abs"], "dw")
    assert (host(dw2)[:, 5] == 0).all() and host(dw2)[:, 4].any()


TUNED_BWD_CASES = [
    # M, K, N                 dX from 65 tiles of 128 x 128 on; dW from 4e9 multiply-adds on
    (15301, 512, 512),     # dX on 128 x 128 tiles, dW on 256 x 256; the last row tile and the last stage in part
    (15360, 512, 512),     # the same with whole tiles and stages
    (61100, 512, 128),     # dX on 128 x 512 tiles, dW on 256 x 128, in part
    (61440, 512, 128),     # ... whole
    (4163, 512, 64),       # dX on 128 x 128 tiles, two stages; dW off the grid
]


@pytest.mark.parametrize("M,K,N", TUNED_BWD_CASES)
@pytest.mark.parametrize("masked,want_dbias", [(False, False), (True, True), (False, True)])
def test_tuned_backward_kernels_in_full(M, K, N, masked, want_dbias):
    """Every element of dX and dW against float64 products, with and without clip masks and the bias gradient's sums
    (dW's kernel and its fold have a form for each)."""
    say("tuned backward", M, K, N, masked, want_dbias)
    gen = torch.Generator(device="cuda").manual_seed(M + K + N)
    x, w = torch.randn((M, K), device="cuda", generator=gen), torch.randn((K, N), device="cuda", generator=gen)
    dy = torch.randn((M, N), device="cuda", generator=gen) + 0.1
    w[:, 5] = 0
    sv = B.Saved(M, K, N, 8, masks=masked)
    if masked:   # scales that are too small make both masks non-trivial
        sv.s_x.fill_(0.02)
        sv.s_w.fill_(0.02)
        B.aqt_quantize_with_scale(x, 8, B.AQT_AXIS_ALL, sv.s_x, q=sv.xq, clip_mask=sv.mask_x)
        B.aqt_quantize_with_scale(w, 8, B.AQT_AXIS_ROWS, sv.s_w, q=sv.wq_kn, clip_mask=sv.mask_w)
        pass_x, pass_w = (dev(unpack_mask(host(m), n).reshape(shape)) for m, n, shape in
                          ((sv.mask_x, M * K, (M, K)), (sv.mask_w, K * N, (K, N))))
        assert 0 < float(pass_x.double().mean()) < 1 and 0 < float(pass_w.double().mean()) < 1
    else:
        B.aqt_dense_fwd(x, w, 8, 8, saved=sv)
        pass_x, pass_w = 1.0, (sv.s_w != 0).double()
        assert int((sv.s_w == 0).sum()) == 1
    dx, dw, db = B.aqt_dense_bwd(dy, sv, 8, 8, want_dbias=want_dbias)
    dys, q, xq, d, sx = (dy * sv.s_w).double(), sv.wq_kn.double(), sv.xq.double(), dy.double(), sv.s_x.double()
    qt, xt = q.t().contiguous(), xq.t().contiguous()
    for what, got, ref, mag in (("dx", dx, (dys @ qt) * pass_x, dys.abs() @ qt.abs()),
                                ("dw", dw, sx * (xt @ d) * pass_w, sx * (xt.abs() @ d.abs()))):
        err = (got.double() - ref).abs()
        assert float(err.max()) <= 1e-4 * float(ref.abs().max()), what
        assert bool((err <= 1e-4 * mag + 1e-37).all()), what
        assert bool((got[ref == 0] == 0).all()), what
    if want_dbias:
        ref = d.sum(0)
        assert bool(((db.double() - ref).abs() <= 2.0 ** -24 * ref.abs() * 1.0001 + M * 2.0 ** -53 * d.abs().sum(0)).all())


DX_WIDE_CASES = [
    # M, K, N, masked        dX tiles need >= 512 (128 x 256) or >= 256 (128 x 512) of them
    (22016, 768, 64, False),     # 128 x 256 tiles, four wavefronts
    (16400, 1024, 96, False),    # 128 x 512 tiles, eight wavefronts, ragged M
    (16384, 512, 64, True),      # the same with a clip mask
]


@pytest.mark.parametrize("M,K,N,masked", DX_WIDE_CASES)
def test_dense_bwd_dx_wide_tiles_sampled(M, K, N, masked):
    say("dx wide tiles", M, K, N, masked)
    c = inputs.small_case(67 + K, M, K, N, 8, 4)
    sv = B.Saved(M, K, N, 4, masks=masked)
    if masked:
        # a scale that is too small for a few elements makes the mask non-trivial
        s_x = np.array([np.abs(c.x).max() / 127 / 1.5], F)
        xq_ref, mx_ref = oracle.quantize_with_scale(c.x, 8, oracle.AXIS_ALL, s_x)
        wq_ref, sw_ref = oracle.quantize(c.w, 4, 0)
        assert 0 < (mx_ref == 0).sum() < mx_ref.size
        B.aqt_quantize_with_scale(dev(c.x), 8, B.AQT_AXIS_ALL, dev(s_x), q=sv.xq, clip_mask=sv.mask_x)
        B.aqt_quantize_weights(dev(c.w), 4, wq_packed=sv.wq_packed, s_w=sv.s_w, wq_kn=sv.wq_kn,
                               clip_mask_w=sv.mask_w)
        sv.s_x.copy_(dev(s_x))
    else:
        wq_ref, sw_ref = oracle.quantize(c.w, 4, 0)
        mx_ref = None
        B.aqt_dense_fwd(dev(c.x), dev(c.w), 8, 4, saved=sv)
    dx, _, _ = B.aqt_dense_bwd(dev(c.dy), sv, 8, 4, want_dw=False)
    dx_h = host(dx)
    rng = np.random.default_rng(3)
    im = np.r_[rng.integers(0, M, 4000), [0, M - 1, M - 1]]
    ik = np.r_[rng.integers(0, K, 4000), [0, K - 1, 0]]
    r, ra = oracle.dense_bwd_dx_sampled(c.dy, wq_ref, sw_ref, im, ik)
    if masked:
        r = r * mx_ref[im, ik]
        assert (dx_h[mx_ref == 0] == 0).all()
    err = np.abs(dx_h[im, ik] - r)
    assert (err <= 1e-4 * ra + 1e-37).all() and err.max() <= 1e-4 * np.abs(r).max()
    # whole row tiles: the first, one in the middle, and the last one (shifted up when M is ragged)
    rows = tile_rows(M)
    xq_rows = np.zeros((rows.size, K), np.int8)     # unused by dX
    g = oracle.dense_bwd(c.dy[rows], xq_rows, 1.0, wq_ref, sw_ref, None if mx_ref is None else mx_ref[rows], None,
                         want_dw=False, want_dbias=False)
    check_grad(dx_h[rows], g["dx"], g["dx_abs"], "dx tiles")


def tile_rows(M, BM=128):
    """Rows of the first row tile, of one in the middle, and the last 2 * BM rows (the last
    tile, shifted up to end at row M when M is ragged, and what it overlaps)."""
    mid = (M // BM // 2) * BM
    return np.unique(np.r_[0:BM, mid:mid + BM, max(0, M - 2 * BM):M])


@pytest.mark.parametrize("M,K,N", [(4096, 512, 256), (16000, 512, 512)])   # small and tuned
def test_backward_is_bit_reproducible_and_stream_ordered(M, K, N):
    # dW folds its slabs in a fixed order: two runs give identical bits; the same work
    # enqueued on a side stream (the stream argument of the C ABI) gives them too
    say("bwd reproducible / side stream", M, K, N)
    c = inputs.small_case(71, M, K, N, 8, 4)
    sv = B.Saved(M, K, N, 4)
    x_d, w_d, dy_d = dev(c.x), dev(c.w), dev(c.dy)
    y1 = B.aqt_dense_fwd(x_d, w_d, 8, 4, saved=sv)
    dx1, dw1, _ = B.aqt_dense_bwd(dy_d, sv, 8, 4)
    dx2, dw2, _ = B.aqt_dense_bwd(dy_d, sv, 8, 4)
    np.testing.assert_array_equal(host(dw1), host(dw2))
    np.testing.assert_array_equal(host(dx1), host(dx2))
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        sv3 = B.Saved(M, K, N, 4)
        y3 = B.aqt_dense_fwd(x_d, w_d, 8, 4, saved=sv3)
        dx3, dw3, _ = B.aqt_dense_bwd(dy_d, sv3, 8, 4)
    side.synchronize()
    np.testing.assert_array_equal(host(y3), host(y1))
    np.testing.assert_array_equal(host(dw3), host(dw1))
    np.testing.assert_array_equal(host(dx3), host(dx1))


@pytest.mark.parametrize("M,K,N", [(2048, 512, 512), (8000, 512, 1024)])   # small and tuned
def test_twenty_runs_give_identical_bytes(M, K, N):
    # Every kernel is deterministic: integer maxima and integer sums do not depend on order, the float
    # reductions (dW slabs, column sums, row statistics) are folded in a fixed order, and the only atomics
    # are maxima and bit-wise ORs.  Twenty runs of each entry point must agree byte for byte.
    say("determinism x20", M, K, N)
    c = inputs.small_case(111, M, K, N, 8, 4, 1, with_bias=True)
    x_d, w_d, dy_d, b_d = dev(c.x), dev(c.w), dev(c.dy), dev(c.bias)
    first = None
    for run in range(20):
        sv = B.Saved(M, K, N, 4, masks=True, dact=True)
        y = B.aqt_dense_fwd(x_d, w_d, 8, 4, bias=b_d, epilogue=1, saved=sv)
        _, m = B.aqt_dense_fwd_q_absmax(sv.xq, sv.s_x, sv.wq_packed, sv.s_w, N, 8, 4, bias=b_d, epilogue=1)
        dx, dw, db = B.aqt_dense_bwd(dy_d, sv, 8, 4, epilogue=1, want_dbias=True)
        q_ln, s_ln, _, st_ln = B.aqt_layernorm_quantize(x_d, 8, want_stats=True)
        got = [host(t).tobytes() for t in (sv.xq, sv.s_x, sv.mask_x, sv.wq_packed, sv.wq_kn, sv.s_w, sv.mask_w,
                                           sv.dact, y, m, dx, dw, db, q_ln, s_ln, st_ln)]
        if first is None:
            first = got
        else:
            assert got == first, f"run {run} differs from run 0"


def test_dense_fwd_very_tall_input_indexing():
    # a million rows: tile bases are 64-bit, lane offsets 32-bit; compare sampled accumulators
    say("dense fwd tall")
    M, K, N = (1 << 20) + 5, 128, 128
    rng = np.random.default_rng(81)
    xq_h = rng.integers(-127, 128, (M, K), dtype=np.int8)
    w = (rng.standard_normal((K, N)) / np.sqrt(K)).astype(F)
    wq_ref, sw_ref = oracle.quantize(w, 4, 0)
    wq, s_w, _, _ = B.aqt_quantize_weights(dev(w), 4)
    s_x = np.array([0.03125], F)
    y, acc = B.aqt_dense_fwd_q(dev(xq_h), dev(s_x), wq, s_w, N, 8, 4, want_acc=True)
    acc_h, y_h = host(acc), host(y)
    im = np.r_[rng.integers(0, M, 3000), [0, M - 1, M - 6, 1 << 19]]
    inn = np.r_[rng.integers(0, N, 3000), [0, N - 1, 5, 77]]
    a, pre = oracle.dense_fwd_q_sampled(xq_h, s_x[0], wq_ref, sw_ref, im, inn)
    np.testing.assert_array_equal(acc_h[im, inn], a)
    assert (np.abs(y_h[im, inn] - pre) <= 1e-6 * np.abs(pre) + 1e-37).all()
    # the last rows, in full
    ref = xq_h[-200:].astype(np.int64) @ wq_ref.astype(np.int64)
    np.testing.assert_array_equal(acc_h[-200:], ref)


def test_argument_errors_on_device_buffers():
    say("argument errors")
    x = dev(np.ones((4, 4), F))
    with pytest.raises(B.AqtError) as e:
        B.aqt_quantize(x, 9, B.AQT_AXIS_ALL)
    assert e.value.status == B.AQT_ERR_UNSUPPORTED
    with pytest.raises(B.AqtError) as e:
        B.aqt_quantize(x, 8, 5)
    assert e.value.status == B.AQT_ERR_INVALID_ARG
    with pytest.raises(B.AqtError) as e:
        B.aqt_dense_fwd(x, x, 8, 4, ws=B.workspace(256))
    assert e.value.status == B.AQT_ERR_WORKSPACE


# ----------------------------------------------------------------------------
# producer-side abs-max and the one-pass quantizer that consumes it
# ----------------------------------------------------------------------------
ABSMAX_CASES = [
    # M, K, N, bits_w, epilogue, bias
    (300, 128, 256, 4, 1, True),        # ragged M, Swish
    (200, 256, 512, 8, 2, True),        # GLU: the maximum is over the gated outputs
    (4100, 384, 384, 4, 0, False),      # tuned kernel, the output spans more than one quantizer block
    (2100, 128, 512, 4, 1, True),       # tuned kernel, ragged M (shifted tile recomputes rows), Swish
    (2176, 256, 512, 8, 2, True),       # tuned kernel, GLU
    (37, 50, 23, 4, 1, True),           # odd N
    (1, 1, 1, 8, 0, False),
]


@pytest.mark.parametrize("M,K,N,bw,epi,with_bias", ABSMAX_CASES)
def test_fused_absmax_feeds_one_pass_quantizer(M, K, N, bw, epi, with_bias):
    say("fused absmax", M, K, N, bw, epi, with_bias)
    c = inputs.small_case(77 + M + N, M, K, N, 8, bw, epi, with_bias=with_bias, with_dy=False)
    bias = None if c.bias is None else dev(c.bias)
    xq, s_x, _ = B.aqt_quantize(dev(c.x), 8, B.AQT_AXIS_ALL)
    wq, s_w, _, _ = B.aqt_quantize_weights(dev(c.w), bw)
    y_ref, _ = B.aqt_dense_fwd_q(xq, s_x, wq, s_w, N, 8, bw, bias=bias, epilogue=epi)
    y, m = B.aqt_dense_fwd_q_absmax(xq, s_x, wq, s_w, N, 8, bw, bias=bias, epilogue=epi)
    y_h = host(y)
    np.testing.assert_array_equal(y_h, host(y_ref))                 # same outputs as the plain entry point
    assert host(m)[0] == np.abs(y_h).max()                          # the definition, on the very buffer written
    # the next layer's quantizer: one pass with the known maximum == the oracle on the same float32 buffer
    for bits in (8, 4):
        status = B.new_status()
        q, s, mask = B.aqt_quantize_with_absmax(y, bits, m, want_mask=(M * N < 100000), dev_status=status)
        q_ref, s_ref = oracle.quantize(y_h, bits, oracle.AXIS_ALL)
        np.testing.assert_array_equal(host(s), s_ref)
        np.testing.assert_array_equal(host(q), q_ref)
        assert host(status)[0] == 0
        q2, s2, _ = B.aqt_quantize(y, bits, B.AQT_AXIS_ALL)
        np.testing.assert_array_equal(host(q2), host(q))
        np.testing.assert_array_equal(host(s2), host(s))
        if mask is not None:
            assert unpack_mask(host(mask), M * N).all() or s_ref[0] == 0


def test_quantize_with_absmax_edge_cases():
    say("quantize with absmax edge cases")
    rng = np.random.default_rng(5)
    x = rng.standard_normal((33, 65)).astype(np.float32)
    x_d = dev(x)
    # a maximum that is too small saturates; codes and mask follow the external-scale oracle
    m_small = np.float32(np.abs(x).max() / 2)
    status = B.new_status()
    q, s, mask = B.aqt_quantize_with_absmax(x_d, 8, dev(np.array([m_small], np.float32)), want_mask=True,
                                            dev_status=status)
    s_ref = np.array([m_small / np.float32(127)], np.float32)
    q_ref, mask_ref = oracle.quantize_with_scale(x, 8, oracle.AXIS_ALL, s_ref)
    np.testing.assert_array_equal(host(s), s_ref)
    np.testing.assert_array_equal(host(q), q_ref)
    np.testing.assert_array_equal(unpack_mask(host(mask), x.size), mask_ref.reshape(-1))
    assert host(status)[0] == 0 and (mask_ref == 0).any()
    # zero maximum: scale 0, codes 0
    q, s, _ = B.aqt_quantize_with_absmax(x_d, 8, dev(np.zeros(1, np.float32)))
    assert host(s)[0] == 0 and not host(q).any()
    # non-finite and negative maxima are reported
    for bad in (np.inf, np.nan, -1.0):
        status = B.new_status()
        B.aqt_quantize_with_absmax(x_d, 8, dev(np.array([bad], np.float32)), dev_status=status)
        assert host(status)[0] == B.AQT_ERR_NONFINITE


# ----------------------------------------------------------------------------
# weight-only modes: float32 activations x integer weights
# ----------------------------------------------------------------------------
WONLY_CASES = [
    # M, K, N, bits_w, epilogue, bias       (which kernel it lands on)
    (256, 256, 1024, 4, 0, False),   # small problems on the tuned grid: split contraction; packed int4 weights
    (300, 96, 256, 8, 1, True),      # ragged M, int8 weights, Swish
    (200, 64, 512, 4, 2, True),      # GLU
    (200, 160, 256, 8, 2, False),
    (2176, 256, 512, 4, 0, False),   # tuned kernel (more than 64 tiles), 128 x 128 tiles, packed int4 weights
    (2100, 96, 640, 8, 1, True),     # ragged M, int8 weights, Swish, three contraction stages
    (2100, 64, 640, 4, 2, True),     # GLU: value and gate blocks in one tile
    (4000, 160, 384, 8, 2, False),
    (37, 50, 23, 4, 0, True),        # off the grid: float64 sums
    (37, 51, 24, 8, 2, True),
    (3, 1, 2, 4, 1, False),
]


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("top", [1.0, 3.7e-3, 2.0 ** -59, 2.0 ** -62, 2.0 ** 66, 1e-42, 3.0e38])
def test_codes_next_to_every_rounding_line(bits, top):
    """Values on and up to four units in the last place to either side of every line between two codes, with scales inside
    and outside of the range where the quantizer multiplies by a reciprocal, and a largest value below the tensor's."""
    say("rounding lines", bits, top)
    qmax = 2 ** (bits - 1) - 1
    s = np.float32(top) / np.float32(qmax)
    lines = ((np.arange(-qmax - 1, qmax + 1) + 0.5) * np.float64(s)).astype(np.float32)
    x = np.concatenate([lines, np.float32([top, -top, 0.0, -0.0])])
    for way in (np.float32(np.inf), np.float32(-np.inf)):
        v = lines
        for _ in range(4):
            v = np.nextafter(v, way)
            x = np.concatenate([x, v])
    x = np.clip(x, -np.float32(top), np.float32(top))
    x = np.resize(x, (9, 1100)).astype(np.float32)      # several groups of loads in a block, and a remainder
    q_ref, s_ref = oracle.quantize(x, bits, oracle.AXIS_ALL)
    q, sc, _ = B.aqt_quantize(dev(x), bits, B.AQT_AXIS_ALL)
    np.testing.assert_array_equal(host(sc), s_ref)
    np.testing.assert_array_equal(host(q), q_ref)
    m = np.float32([top])
    q1, s1, _ = B.aqt_quantize_with_absmax(dev(x), bits, dev(m))
    np.testing.assert_array_equal(host(q1), q_ref)
    small = np.float32([np.float32(top) * np.float32(0.37)])
    q2, s2, _ = B.aqt_quantize_with_absmax(dev(x), bits, dev(small))
    np.testing.assert_array_equal(host(q2), oracle.quantize_with_scale(x, bits, oracle.AXIS_ALL, host(s2))[0])


@pytest.mark.parametrize("M,K,N,bw,epi,with_bias", WONLY_CASES)
def test_dense_fwd_weight_only_against_oracle(M, K, N, bw, epi, with_bias):
    say("dense fwd weight-only", M, K, N, bw, epi, with_bias)
    c = inputs.small_case(91 + M + K + N, M, K, N, 8, bw, epi, with_bias=with_bias, with_dy=False)
    wq_ref, sw_ref = oracle.quantize(c.w, bw, 0)
    ora = oracle.dense_fwd_wonly(c.x, wq_ref, sw_ref, c.bias, epi)
    wq, s_w, wq_kn, _ = B.aqt_quantize_weights(dev(c.w), bw)
    np.testing.assert_array_equal(host(wq_kn), wq_ref)
    np.testing.assert_array_equal(host(s_w), sw_ref)
    y = B.aqt_dense_fwd_wonly(dev(c.x), wq, s_w, N, bw, bias=None if c.bias is None else dev(c.bias), epilogue=epi)
    check_float_forward(host(y), ora, epi)


WONLY_WIDE_CASES = [
    (16384, 128, 2048, 4, 0),        # 128 x 512 tiles, eight wavefronts
    (16500, 96, 1024, 8, 2),         # the same with GLU, ragged M
    (22016, 64, 768, 4, 1),          # 128 x 256 tiles (768 is not a multiple of 512)
]


@pytest.mark.parametrize("M,K,N,bw,epi", WONLY_WIDE_CASES)
def test_dense_fwd_weight_only_wide_tiles_sampled(M, K, N, bw, epi):
    say("dense fwd weight-only wide", M, K, N, bw, epi)
    c = inputs.small_case(97 + K + N, M, K, N, 8, bw, epi, with_dy=False)
    wq_ref, sw_ref = oracle.quantize(c.w, bw, 0)
    wq, s_w, _, _ = B.aqt_quantize_weights(dev(c.w), bw)
    y_h = host(B.aqt_dense_fwd_wonly(dev(c.x), wq, s_w, N, bw, epilogue=epi))
    rng = np.random.default_rng(9)
    out_cols = N // 2 if epi == 2 else N
    im = np.r_[rng.integers(0, M, 3000), [0, M - 1]]
    ij = np.r_[rng.integers(0, out_cols, 3000), [0, out_cols - 1]]
    pre, mag = oracle.dense_fwd_wonly_sampled(c.x, wq_ref, sw_ref, im, ij)
    got = y_h[im, ij].astype(np.float64)
    tol_v = REL_F * mag + 1e-37
    if epi == 0:
        assert (np.abs(got - pre) <= tol_v).all()
        assert np.abs(got - pre).max() <= REL_F * np.abs(pre).max()
    elif epi == 1:
        ref = pre / (1 + np.exp(-pre))
        assert (np.abs(got - ref) <= 1e-6 * np.abs(ref) + 1.1 * tol_v).all()
    else:
        gate, gmag = oracle.dense_fwd_wonly_sampled(c.x, wq_ref, sw_ref, im, ij + out_cols)
        sg = 1 / (1 + np.exp(-gate))
        ref = pre * sg
        tol = 1e-6 * np.abs(ref) + sg * tol_v + 0.25 * np.abs(pre) * (REL_F * gmag) + 1e-37
        assert (np.abs(got - ref) <= tol).all()
    # whole row tiles against the full oracle on those rows
    rows = tile_rows(M)
    ora = oracle.dense_fwd_wonly(c.x[rows], wq_ref, sw_ref, None, epi)
    check_float_forward(y_h[rows], ora, epi)


@pytest.mark.parametrize("layer", [0, 1])
def test_dense_fwd_weight_only_training_step_shapes(layer):
    # the two shapes the benchmark times this entry point on (16 and 64 contraction stages of 32)
    c = inputs.config5()[layer]
    say("dense fwd weight-only full size", c.M, c.K, c.N)
    wq_ref, sw_ref = oracle.quantize(c.w, c.bits_w, 0)
    wq, s_w, _, _ = B.aqt_quantize_weights(dev(c.w), c.bits_w)
    y_h = host(B.aqt_dense_fwd_wonly(dev(c.x), wq, s_w, c.N, c.bits_w))
    rng = np.random.default_rng(19)
    im = np.r_[rng.integers(0, c.M, 4000), [0, c.M - 1]]
    ij = np.r_[rng.integers(0, c.N, 4000), [0, c.N - 1]]
    pre, mag = oracle.dense_fwd_wonly_sampled(c.x, wq_ref, sw_ref, im, ij)
    err = np.abs(y_h[im, ij] - pre)
    assert (err <= REL_F * mag + 1e-37).all() and err.max() <= REL_F * np.abs(pre).max()
    say("   max err / bound:", float((err / (REL_F * mag + 1e-37)).max()))
    rows = tile_rows(c.M)
    ora = oracle.dense_fwd_wonly(c.x[rows], wq_ref, sw_ref, None, 0)
    check_float_forward(y_h[rows], ora, 0)


# 128 x 256 tiles are used from about 400 of them at a fan-in of 1024 or more (2048 below that)
WIDE_TILE_CASES = [
    # M, K, N, bits_x, bits_w, epilogue
    (16384, 1024, 1024, 8, 8, 2),    # GLU, value and gate halves in one tile, int8 weights
    (16500, 1152, 1024, 8, 4, 1),    # ragged M (shifted last row tile), Swish, nine stages
    (16384, 1024, 2048, 4, 4, 0),    # int4 x int4
    (33000, 128, 2048, 8, 4, 0),     # a single stage, ragged M, many tiles at a short fan-in
]


@pytest.mark.parametrize("M,K,N,bx,bw,epi", WIDE_TILE_CASES)
def test_dense_fwd_wide_tiles_sampled(M, K, N, bx, bw, epi):
    c = inputs.small_case(53 + K + N, M, K, N, bx, bw, epi, with_dy=False)
    run_full_size_case(c, n_samples=2000)


# ----------------------------------------------------------------------------
# the paper-shaped configurations at full size, in the launch configuration the
# benchmark times: quantizers compared in full, contractions on sampled outputs
# ----------------------------------------------------------------------------
def run_full_size_case(c, n_samples=3000, backward=False, full_dw=False):
    say("full size", c.name, c.M, c.K, c.N, c.bits_x, c.bits_w, c.epilogue)
    xq_ref, sx_ref = oracle.quantize(c.x, c.bits_x, oracle.AXIS_ALL)
    wq_ref, sw_ref = oracle.quantize(c.w, c.bits_w, 0)
    sv = B.Saved(c.M, c.K, c.N, c.bits_w)
    status = B.new_status()
    x_d, w_d = dev(c.x), dev(c.w)
    y = B.aqt_dense_fwd(x_d, w_d, c.bits_x, c.bits_w, epilogue=c.epilogue, saved=sv, dev_status=status)
    assert host(status)[0] == 0
    np.testing.assert_array_equal(host(sv.s_x), sx_ref)
    np.testing.assert_array_equal(host(sv.s_w), sw_ref)
    np.testing.assert_array_equal(host(sv.xq), xq_ref)
    np.testing.assert_array_equal(host(sv.wq_kn), wq_ref)
    if c.bits_w <= 4:
        np.testing.assert_array_equal(host(sv.wq_packed).reshape(c.N, -1), oracle.pack_int4(wq_ref))
    else:
        np.testing.assert_array_equal(host(sv.wq_packed).view(np.int8).reshape(c.N, c.K), wq_ref.T)
    _, acc = B.aqt_dense_fwd_q(sv.xq, sv.s_x, sv.wq_packed, sv.s_w, c.N, c.bits_x, c.bits_w, want_acc=True)
    acc_h, y_h = host(acc), host(y)
    del acc
    rng = np.random.default_rng(7)
    im = np.r_[rng.integers(0, c.M, n_samples), [0, c.M - 1]]
    out_cols = c.N // 2 if c.epilogue == 2 else c.N
    ij = np.r_[rng.integers(0, out_cols, n_samples), [0, out_cols - 1]]
    a, pre = oracle.dense_fwd_q_sampled(xq_ref, sx_ref[0], wq_ref, sw_ref, im, ij)
    np.testing.assert_array_equal(acc_h[im, ij], a)
    got = y_h[im, ij].astype(np.float64)
    tol_v = 1e-6 * np.abs(pre) + 1e-37
    if c.epilogue == 0:
        assert (np.abs(got - pre) <= tol_v).all()
    elif c.epilogue == 1:
        ref = pre / (1 + np.exp(-pre))
        assert (np.abs(got - ref) <= 1e-6 * np.abs(ref) + 1.1 * tol_v).all()
    else:
        a2, gate = oracle.dense_fwd_q_sampled(xq_ref, sx_ref[0], wq_ref, sw_ref, im, ij + out_cols)
        np.testing.assert_array_equal(acc_h[im, ij + out_cols], a2)
        sg = 1 / (1 + np.exp(-gate))
        ref = pre * sg
        tol = 1e-6 * np.abs(ref) + sg * tol_v + 0.25 * np.abs(pre) * (1e-6 * np.abs(gate)) + 1e-37
        assert (np.abs(got - ref) <= tol).all()
    # whole row tiles (first, middle, last): accumulators and outputs in full
    rows = tile_rows(c.M)
    ora = oracle.dense_fwd_q(xq_ref[rows], sx_ref[0], wq_ref, sw_ref, None, c.epilogue)
    np.testing.assert_array_equal(acc_h[rows], ora["acc"])
    check_forward(y_h[rows], ora, sx_ref[0], sw_ref, None, c.epilogue)
    del acc_h
    if backward:
        dy_d = dev(c.dy)
        dx, dw, _ = B.aqt_dense_bwd(dy_d, sv, c.bits_x, c.bits_w)
        dx_h, dw_h = host(dx), host(dw)
        ik = np.r_[rng.integers(0, c.K, n_samples), [0, c.K - 1]]
        r, ra = oracle.dense_bwd_dx_sampled(c.dy, wq_ref, sw_ref, im, ik)
        err = np.abs(dx_h[im, ik] - r)
        assert (err <= 1e-4 * ra + 1e-37).all() and err.max() <= 1e-4 * np.abs(r).max()
        n_dw = 400
        ik2, in2 = rng.integers(0, c.K, n_dw), rng.integers(0, c.N, n_dw)
        r, ra = oracle.dense_bwd_dw_sampled(c.dy, xq_ref, sx_ref[0], ik2, in2)
        err = np.abs(dw_h[ik2, in2] - r)
        assert (err <= 1e-4 * ra + 1e-37).all() and err.max() <= 1e-4 * np.abs(r).max()
        say("   bwd max err / 1e-4 bound:", float((err / (1e-4 * ra + 1e-37)).max()))
        g = oracle.dense_bwd(c.dy[rows], xq_ref[rows], sx_ref[0], wq_ref, sw_ref, want_dw=False, want_dbias=False)
        check_grad(dx_h[rows], g["dx"], g["dx_abs"], "dx tiles")
        if full_dw:      # every element of dW, all slabs and tiles
            g = oracle.dense_bwd(c.dy, xq_ref, sx_ref[0], wq_ref, sw_ref, want_dx=False, want_dbias=False)
            check_grad(dw_h, g["dw"], g["dw_abs"], "dw in full")


@pytest.mark.parametrize("cfg", [2, 3, 4])
def test_conformer_configs_full_size(cfg):
    for c in inputs.CONFIGS[cfg]():
        run_full_size_case(c)


def test_training_step_full_size():
    for c in inputs.config5():
        run_full_size_case(c, backward=True, full_dw=True)
        torch.cuda.empty_cache()


def test_fused_absmax_full_size_chain():
    # layer 1 of the training-step configuration with a Swish epilogue, its output quantized
    # for layer 2 in one pass: the launch configuration the benchmark's extra figures time
    c = inputs.config5()[0]
    say("fused absmax full size", c.M, c.K, c.N)
    xq, s_x, _ = B.aqt_quantize(dev(c.x), 8, B.AQT_AXIS_ALL)
    wq, s_w, _, _ = B.aqt_quantize_weights(dev(c.w), 4)
    y, m = B.aqt_dense_fwd_q_absmax(xq, s_x, wq, s_w, c.N, 8, 4, epilogue=B.AQT_EPI_SWISH)
    status = B.new_status()
    q, s, _ = B.aqt_quantize_with_absmax(y, 8, m, dev_status=status)
    y_h = host(y)
    assert host(m)[0] == np.abs(y_h).max()
    q_ref, s_ref = oracle.quantize(y_h, 8, oracle.AXIS_ALL)
    np.testing.assert_array_equal(host(s), s_ref)
    np.testing.assert_array_equal(host(q), q_ref)
    assert host(status)[0] == 0


def test_quantize_more_than_2_31_elements():
    # 64-bit indexing in the per-tensor quantizer: a tensor of 2^31 + 4100 floats (8.6 GB) made on
    # the device; the scale is checked against the definition, the codes on slices (head, the
    # 2^31 boundary, the ragged tail) against the oracle's element-wise half with that scale
    say("quantize > 2^31 elements")
    rows, cols = (1 << 19) + 1, 4100            # cols not a multiple of 4 rows apart: ragged runs
    n = rows * cols
    assert n > (1 << 31)
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.empty((rows, cols), dtype=torch.float32, device="cuda")
    x.normal_(generator=g)
    x[rows - 1, cols - 1] = -9.5                # the maximum sits in the very last element
    status = B.new_status()
    q, s, _ = B.aqt_quantize(x, 8, B.AQT_AXIS_ALL, dev_status=status)
    assert host(status)[0] == 0
    m = np.float32(x.abs().max().item())
    assert m == np.float32(9.5)
    s_ref = np.array([m / np.float32(127)], F)
    np.testing.assert_array_equal(host(s), s_ref)
    flat_x, flat_q = x.view(-1), q.view(-1)
    for lo, hi in [(0, 70000), ((1 << 31) - 40000, (1 << 31) + 40000), (n - 70001, n)]:
        xs = flat_x[lo:hi].cpu().numpy().reshape(1, -1)
        q_ref, _ = oracle.quantize_with_scale(xs, 8, oracle.AXIS_ALL, s_ref)
        np.testing.assert_array_equal(flat_q[lo:hi].cpu().numpy().reshape(1, -1), q_ref)
    assert int(flat_q[n - 1].item()) == -127
    del x, q
    torch.cuda.empty_cache()


@pytest.mark.parametrize("bx,bw", [(2, 2), (5, 3), (7, 6), (3, 8)])
def test_other_bit_widths_forward_and_backward(bx, bw):
    # Sec. 2.2 gives the rule for 8 and 4 bits; the same rule (qmax = 2^(b-1) - 1) is accepted for
    # any width in 2..8: codes stay inside [-qmax, qmax], weights up to 4 bits are stored packed
    say("other bit widths", bx, bw)
    for (M, K, N) in [(256, 128, 128), (33, 20, 11)]:
        c = inputs.small_case(100 * bx + bw + M, M, K, N, bx, bw, 0, with_bias=True)
        ora = oracle.dense_fwd(c.x, c.w, bx, bw, c.bias, 0)
        qx, qw = (1 << (bx - 1)) - 1, (1 << (bw - 1)) - 1
        assert np.abs(ora["xq"]).max() == qx and np.abs(ora["wq"]).max() == qw
        sv = B.Saved(M, K, N, bw)
        y = B.aqt_dense_fwd(dev(c.x), dev(c.w), bx, bw, bias=dev(c.bias), saved=sv)
        np.testing.assert_array_equal(host(sv.xq), ora["xq"])
        np.testing.assert_array_equal(host(sv.wq_kn), ora["wq"])
        np.testing.assert_array_equal(host(sv.s_x), ora["s_x"])
        np.testing.assert_array_equal(host(sv.s_w), ora["s_w"])
        np.testing.assert_array_equal(host(B.aqt_unpack_weights(sv.wq_packed, K, N, bw)), ora["wq"])
        _, acc = B.aqt_dense_fwd_q(sv.xq, sv.s_x, sv.wq_packed, sv.s_w, N, bx, bw, want_acc=True)
        np.testing.assert_array_equal(host(acc), ora["acc"])
        check_forward(host(y), ora, ora["s_x"][0], ora["s_w"], c.bias, 0)
        g = oracle.dense_bwd(c.dy, ora["xq"], ora["s_x"][0], ora["wq"], ora["s_w"])
        dx, dw, _ = B.aqt_dense_bwd(dev(c.dy), sv, bx, bw)
        check_grad(host(dx), g["dx"], g["dx_abs"], "dx")
        check_grad(host(dw), g["dw"], g["dw_abs"], "dw")
