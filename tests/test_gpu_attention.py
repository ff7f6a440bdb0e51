"""Parity of the self-attention module's pieces (the float attention core and the module as one
call) against the CPU oracle; the chain is checked stage by stage, each quantized stage with the
oracle fed the very float32 buffer the GPU stage consumed."""
import numpy as np
import pytest
import torch

import oracle
from paper_2203_15952_amd import binding as B
from parity_util import TINY, check_forward

pytestmark = pytest.mark.gpu
F = np.float32
U = 2.0 ** -24   # float32 unit round-off


def dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def say(*a):
    print(*a, flush=True)


def check_attention(ctx, qkv, B_, T, D, heads, left, right):
    """A scaled score is a float32 chain of dh multiply-adds and one more product: within
    e_s = (dh + 2) u of the sum of the magnitudes of its terms (smag).  exp turns that absolute error
    into a relative error of each weight (plus the exponential's own few u), numerator and normaliser
    are sums of at most T such weights, so their ratio is within 2 (2 e_s smag + (T + 16) u) of the
    float64 result, relative to sum_j p_j |v_j| (vmag)."""
    dh = D // heads
    ref, smag, vmag = oracle.attention(qkv.reshape(B_, T, 3 * D), heads, left, right, want_mags=True)
    rel = 2.0 * (2.0 * (dh + 2) * U * np.repeat(smag, dh, axis=2) + (T + 16) * U)
    bad = np.abs(ctx.reshape(B_, T, D).astype(np.float64) - ref) > rel * vmag + TINY
    assert not bad.any(), f"{bad.sum()} of {bad.size} attention outputs outside tolerance"


ATT_CASES = [
    # B, T, D, heads, left, right
    (32, 400, 512, 8, -1, -1),      # the self-attention configuration: 8 heads of 64, whole utterance
    (2, 70, 128, 2, 23, 0),         # causal with 23 frames of left context (Sec. 3.3); ragged tile
    (1, 130, 72, 2, -1, 3),         # heads of 36 (Conformer S), a little right context
    (3, 65, 12, 3, 5, 7),
    (1, 1, 1, 1, -1, -1),
    (2, 200, 256, 4, 30, 30),       # windows that skip whole key tiles
]


@pytest.mark.parametrize("B_,T,D,heads,left,right", ATT_CASES)
def test_attention_forward(B_, T, D, heads, left, right):
    say("attention", B_, T, D, heads, left, right)
    rng = np.random.default_rng(600 + T + D)
    qkv = rng.standard_normal((B_ * T, 3 * D)).astype(F)
    ctx, m = B.aqt_attention_fwd(dev(qkv), B_, T, heads, left=left, right=right, want_absmax=True)
    ctx_h = host(ctx)
    check_attention(ctx_h, qkv, B_, T, D, heads, left, right)
    assert host(m)[0] == np.abs(ctx_h).max()
    q, s, _ = B.aqt_quantize_with_absmax(ctx, 8, m)
    q_ref, s_ref = oracle.quantize(ctx_h, 8, oracle.AXIS_ALL)
    np.testing.assert_array_equal(host(s), s_ref)
    np.testing.assert_array_equal(host(q), q_ref)
    # same bits on a second run (the only atomic is a maximum)
    ctx2, _ = B.aqt_attention_fwd(dev(qkv), B_, T, heads, left=left, right=right)
    np.testing.assert_array_equal(host(ctx2), ctx_h)


def test_attention_window_of_the_frame_itself_returns_the_values():
    rng = np.random.default_rng(610)
    B_, T, D = 2, 100, 128
    qkv = rng.standard_normal((B_ * T, 3 * D)).astype(F)
    ctx, _ = B.aqt_attention_fwd(dev(qkv), B_, T, 2, left=0, right=0)
    np.testing.assert_array_equal(host(ctx), qkv[:, 2 * D:])


def test_attention_argument_errors():
    z = torch.zeros((8, 3 * 130), device="cuda")
    with pytest.raises(B.AqtError) as e:
        B.aqt_attention_fwd(z, 1, 8, 1)          # a head of 130 columns
    assert e.value.status == B.AQT_ERR_UNSUPPORTED
    with pytest.raises(B.AqtError) as e:
        B.aqt_attention_fwd(z, 1, 8, 4)          # 130 is not a multiple of 4 heads
    assert e.value.status == B.AQT_ERR_INVALID_ARG


def rows_of(M):
    mid = (M // 256) * 128
    return np.unique(np.r_[0:min(128, M), mid:min(mid + 128, M), max(0, M - 256):M])


@pytest.mark.parametrize("B_,T,D,heads,left,right,policy,outliers", [
    (32, 400, 512, 8, -1, -1, ((8, 8), (8, 8)), True),    # the self-attention configuration, int8 x int8
    (3, 70, 128, 4, 23, 0, ((4, 8), (8, 8)), False),      # causal, ragged, int4 projection weights
    (2, 19, 24, 2, -1, 2, ((8, 4), (4, 8)), False),       # shapes off the tuned grid
])
def test_mhsa_chain_stage_by_stage(B_, T, D, heads, left, right, policy, outliers):
    say("mhsa", B_, T, D, heads, left, right, policy)
    M = B_ * T
    rng = np.random.default_rng(700 + M)
    x = rng.standard_normal((M, D)).astype(F)
    if outliers:   # 1 % of the entries at +-8 standard deviations
        hit = rng.random((M, D)) < 0.01
        x[hit] = np.where(rng.random(int(hit.sum())) < 0.5, F(-8.0), F(8.0))
    gamma, beta = (1 + 0.1 * rng.standard_normal(D)).astype(F), (0.1 * rng.standard_normal(D)).astype(F)
    wqkv, bqkv = (rng.standard_normal((D, 3 * D)) / np.sqrt(D)).astype(F), (0.1 * rng.standard_normal(3 * D)).astype(F)
    wo, bo = (rng.standard_normal((D, D)) / np.sqrt(D)).astype(F), (0.1 * rng.standard_normal(D)).astype(F)
    (bw1, bx1), (bw2, bx2) = policy
    sv = B.MhsaSaved(B_, T, D, policy)
    status = B.new_status()
    x_d, g_d, b_d, wqkv_d, bqkv_d, wo_d, bo_d = (dev(a) for a in (x, gamma, beta, wqkv, bqkv, wo, bo))
    y = B.aqt_mhsa_fwd(x_d, wqkv_d, bqkv_d, wo_d, bo_d, sv, heads, left=left, right=right, gamma=g_d, beta=b_d,
                       dev_status=status)
    assert host(status)[0] == 0
    rows = rows_of(M)
    # stage 1: normalisation + quantizer
    q_a, s_a, xn_t, _ = B.aqt_layernorm_quantize(x_d, bx1, gamma=g_d, beta=b_d, eps=1e-6, want_y=True)
    xn = host(xn_t)
    ref = oracle.layernorm(x, gamma, beta, 1e-6)
    assert (np.abs(xn - ref) <= 1e-5 * (1 + np.abs(ref))).all()
    xq1, sx1 = oracle.quantize(xn, bx1, oracle.AXIS_ALL)
    np.testing.assert_array_equal(host(sv.qkv.s_x), sx1)
    np.testing.assert_array_equal(host(sv.qkv.xq), xq1)
    # stage 2: fused projection
    wq1, sw1 = oracle.quantize(wqkv, bw1, 0)
    np.testing.assert_array_equal(host(sv.qkv.wq_kn), wq1)
    qkv_h = host(sv.qkv_f)
    check_forward(qkv_h[rows], oracle.dense_fwd_q(xq1[rows], sx1[0], wq1, sw1, bqkv, 0), sx1[0], sw1, bqkv, 0)
    # stage 3: attention on the GPU's own projections
    ctx_h = host(sv.ctx)
    check_attention(ctx_h, qkv_h, B_, T, D, heads, left, right)
    # stage 4: quantizer on the GPU's own attention result; stage 5: output projection
    xq2, sx2 = oracle.quantize(ctx_h, bx2, oracle.AXIS_ALL)
    np.testing.assert_array_equal(host(sv.out.s_x), sx2)
    np.testing.assert_array_equal(host(sv.out.xq), xq2)
    wq2, sw2 = oracle.quantize(wo, bw2, 0)
    np.testing.assert_array_equal(host(sv.out.wq_kn), wq2)
    y_h = host(y)
    check_forward(y_h[rows], oracle.dense_fwd_q(xq2[rows], sx2[0], wq2, sw2, bo, 0), sx2[0], sw2, bo, 0)
    # the one call equals the same entry points called one by one, bit for bit
    wp1, s_w1, _, _ = B.aqt_quantize_weights(wqkv_d, bw1)
    qkv_b, _ = B.aqt_dense_fwd_q(q_a, s_a, wp1, s_w1, 3 * D, bx1, bw1, bias=bqkv_d)
    ctx_b, m_b = B.aqt_attention_fwd(qkv_b, B_, T, heads, left=left, right=right, want_absmax=True)
    q_b, sx_b, _ = B.aqt_quantize_with_absmax(ctx_b, bx2, m_b)
    wp2, s_w2, _, _ = B.aqt_quantize_weights(wo_d, bw2)
    y_b, _ = B.aqt_dense_fwd_q(q_b, sx_b, wp2, s_w2, D, bx2, bw2, bias=bo_d)
    np.testing.assert_array_equal(host(y_b), y_h)


@pytest.mark.parametrize("B_,T,D,heads,left,right", ATT_CASES)
def test_attention_backward(B_, T, D, heads, left, right):
    from parity_util import check_grad
    say("attention bwd", B_, T, D, heads, left, right)
    rng = np.random.default_rng(650 + T + D)
    M = B_ * T
    qkv = rng.standard_normal((M, 3 * D)).astype(F)
    dctx = (0.1 * rng.standard_normal((M, D))).astype(F)
    qkv_d, dctx_d = dev(qkv), dev(dctx)
    lse = torch.empty((M, heads), dtype=torch.float32, device="cuda")
    ctx, _ = B.aqt_attention_fwd(qkv_d, B_, T, heads, left=left, right=right, lse=lse)
    dqkv = B.aqt_attention_bwd(qkv_d, ctx, dctx_d, lse, B_, T, heads, left=left, right=right)
    ref, mag = oracle.attention_bwd(qkv.reshape(B_, T, 3 * D), dctx.reshape(B_, T, D), heads, left, right)
    got = host(dqkv).reshape(B_, T, 3 * D)
    for name, sl in (("dq", slice(0, D)), ("dk", slice(D, 2 * D)), ("dv", slice(2 * D, 3 * D))):
        check_grad(got[:, :, sl], ref[:, :, sl], mag[:, :, sl], name)
    # the forward with lse gives the same ctx as without; the backward has one summation order
    ctx0, _ = B.aqt_attention_fwd(qkv_d, B_, T, heads, left=left, right=right)
    np.testing.assert_array_equal(host(ctx0), host(ctx))
    dqkv2 = B.aqt_attention_bwd(qkv_d, ctx, dctx_d, lse, B_, T, heads, left=left, right=right)
    np.testing.assert_array_equal(host(dqkv2), host(dqkv))
    if M <= 400:   # lse is log2 of the sum of exponentials of the scaled scores
        dh = D // heads
        q, k = (qkv[:, i * D:(i + 1) * D].astype(np.float64).reshape(B_, T, heads, dh) for i in range(2))
        sc = np.einsum("bthd,bjhd->bthj", q, k) / np.sqrt(dh)
        t_i, j_i = np.arange(T)[:, None], np.arange(T)[None, :]
        ok = np.ones((T, T), bool)
        if left >= 0:
            ok &= j_i >= t_i - left
        if right >= 0:
            ok &= j_i <= t_i + right
        sc = np.where(ok[None, :, None, :], sc, -np.inf)
        want = np.log2(np.exp(sc - sc.max(-1, keepdims=True)).sum(-1)) + sc.max(-1) * np.log2(np.e)
        np.testing.assert_allclose(host(lse).reshape(B_, T, heads), want, rtol=0, atol=2e-5 * (1 + np.abs(want).max()))


@pytest.mark.parametrize("B_,T,D,heads,left,right,policy", [
    (8, 200, 512, 8, -1, -1, ((8, 8), (8, 8))),
    (3, 70, 128, 4, 23, 0, ((4, 8), (8, 8))),
    (2, 19, 24, 2, -1, 2, ((8, 4), (4, 8))),
])
def test_mhsa_backward_stage_by_stage(B_, T, D, heads, left, right, policy):
    from parity_util import check_grad
    say("mhsa bwd", B_, T, D, heads, left, right, policy)
    M = B_ * T
    rng = np.random.default_rng(750 + M)
    x = rng.standard_normal((M, D)).astype(F)
    wqkv, bqkv = (rng.standard_normal((D, 3 * D)) / np.sqrt(D)).astype(F), (0.1 * rng.standard_normal(3 * D)).astype(F)
    wo, bo = (rng.standard_normal((D, D)) / np.sqrt(D)).astype(F), (0.1 * rng.standard_normal(D)).astype(F)
    dy = (0.1 * rng.standard_normal((M, D))).astype(F)
    (bw1, bx1), (bw2, bx2) = policy
    sv = B.MhsaSaved(B_, T, D, policy, heads=heads)
    B.aqt_mhsa_fwd(dev(x), dev(wqkv), dev(bqkv), dev(wo), dev(bo), sv, heads, left=left, right=right)
    o = B.aqt_mhsa_bwd(dev(dy), sv, heads, left=left, right=right)
    # output projection against the oracle on the GPU's own codes
    xq2, sx2, wq2, sw2 = host(sv.out.xq), host(sv.out.s_x), host(sv.out.wq_kn), host(sv.out.s_w)
    g2 = oracle.dense_bwd(dy, xq2, sx2[0], wq2, sw2)
    check_grad(host(o["dwo"]), g2["dw"], g2["dw_abs"], "dwo")
    check_grad(host(o["dbo"]), g2["dbias"], np.abs(dy.astype(np.float64)).sum(0), "dbo")
    sv2 = B.Saved(M, D, D, bw2)
    sv2.xq.copy_(sv.out.xq); sv2.s_x.copy_(sv.out.s_x); sv2.wq_kn.copy_(sv.out.wq_kn); sv2.s_w.copy_(sv.out.s_w)
    dctx, _, _ = B.aqt_dense_bwd(dev(dy), sv2, bx2, bw2, want_dw=False)
    dctx_h = host(dctx)
    check_grad(dctx_h, g2["dx"], g2["dx_abs"], "dctx")
    # attention: the oracle fed the float32 gradient and projections the GPU used
    qkv_h = host(sv.qkv_f)
    dqkv = B.aqt_attention_bwd(sv.qkv_f, sv.ctx, dctx, sv.lse, B_, T, heads, left=left, right=right)
    ref, mag = oracle.attention_bwd(qkv_h.reshape(B_, T, 3 * D), dctx_h.reshape(B_, T, D), heads, left, right)
    dqkv_h = host(dqkv)
    check_grad(dqkv_h, ref.reshape(M, 3 * D), mag.reshape(M, 3 * D), "dqkv")
    # fused projection
    xq1, sx1, wq1, sw1 = host(sv.qkv.xq), host(sv.qkv.s_x), host(sv.qkv.wq_kn), host(sv.qkv.s_w)
    g1 = oracle.dense_bwd(dqkv_h, xq1, sx1[0], wq1, sw1)
    check_grad(host(o["dxn"]), g1["dx"], g1["dx_abs"], "dxn")
    check_grad(host(o["dwqkv"]), g1["dw"], g1["dw_abs"], "dwqkv")
    check_grad(host(o["dbqkv"]), g1["dbias"], np.abs(dqkv_h.astype(np.float64)).sum(0), "dbqkv")


# Copies of two utterances: a small batch takes the kernels of attention_few.hip and the backward's 32 rows to a workgroup, with this many
# copies (more than 512 workgroups from 16 queries and from 32 rows) 128 rows belong to one.
MANY = 90


@pytest.mark.parametrize("copies", [1, MANY])
@pytest.mark.parametrize("T", [1, 31, 33, 128, 161])
@pytest.mark.parametrize("dh,left,right", [(4, -1, -1), (16, 33, 0), (20, -1, 31), (32, 0, 64), (44, 32, 32), (52, -1, -1), (64, 95, 1)])
def test_attention_tile_edges(T, dh, left, right, copies):
    """Every step count of the kernels for vectorised rows (head widths up to 16, 32, 48 and 64, with and without a partial
    step) against tile remainders of the frames and window ends on and next to tile ends."""
    from parity_util import check_grad
    heads, D = 3, 3 * dh
    say("attention edges", T, dh, left, right, copies)
    rng = np.random.default_rng(660 + 100 * T + dh)
    qkv, dctx = rng.standard_normal((2 * T, 3 * D)).astype(F), rng.standard_normal((2 * T, D)).astype(F)
    B_, qkv_d, dctx_d = 2 * copies, dev(qkv).repeat(copies, 1), dev(dctx).repeat(copies, 1)
    M, pair = B_ * T, slice(-2 * T, None)   # the batch's last two utterances
    lse = torch.empty((M, heads), dtype=torch.float32, device="cuda")
    ctx, _ = B.aqt_attention_fwd(qkv_d, B_, T, heads, left=left, right=right, lse=lse)
    check_attention(host(ctx[pair]), qkv, 2, T, D, heads, left, right)
    got = host(B.aqt_attention_bwd(qkv_d, ctx, dctx_d, lse, B_, T, heads, left=left, right=right)[pair]).reshape(2, T, 3 * D)
    ref, mag = oracle.attention_bwd(qkv.reshape(2, T, 3 * D), dctx.reshape(2, T, D), heads, left, right)
    check_grad(got, ref, mag, "dqkv")
    # a tensor that is not 16-byte aligned takes the kernels for any layout
    ctx_odd, _ = B.aqt_attention_fwd(moved(qkv_d), B_, T, heads, left=left, right=right)
    np.testing.assert_array_equal(host(ctx_odd), host(ctx))   # the forwards share every product and sum


def moved(t):
    """The same values 4-byte aligned only: the kernels for any layout take them."""
    out = torch.empty(t.numel() + 1, device="cuda")[1:].view(t.shape)
    return out.copy_(t)


@pytest.mark.parametrize("dh", [16, 36, 64])
def test_backward_uses_the_probabilities_of_the_forward(dh):
    """Large scores: exp2(score - lse) repeats the forward's rounding, so what the two backwards make of one lse may differ by
    the float32 rounding of dv's sum over T products, (T + 4) u of the magnitudes each, but not by the scores' own error,
    which is 30 times that here."""
    T, heads = 40, 4
    D = heads * dh
    rng = np.random.default_rng(680 + dh)
    qkv = rng.standard_normal((2 * T, 3 * D)).astype(F)
    qkv[:, :2 * D] *= 8
    qkv_d, go = dev(qkv), dev(rng.standard_normal((2 * T, D)).astype(F))
    lse = torch.empty((2 * T, heads), device="cuda")
    ctx, _ = B.aqt_attention_fwd(qkv_d, 2, T, heads, lse=lse)

    def dv(q, g):
        return host(B.aqt_attention_bwd(q, ctx, g, lse, 2, T, heads))[:, 2 * D:].astype(np.float64)

    mag = dv(moved(qkv_d), go.abs())
    assert np.all(np.abs(dv(qkv_d, go) - dv(moved(qkv_d), go)) <= 2 * (T + 4) * U * mag * 1.001 + TINY)


BIG = F(3.4e38)   # rounds to an infinity in bf16


@pytest.mark.parametrize("copies", [1, MANY])
@pytest.mark.parametrize("what,value", [("q", np.nan), ("k", np.nan), ("k", np.inf), ("k", -BIG), ("v", np.inf), ("v", BIG)])
@pytest.mark.parametrize("dh,left,right", [(64, -1, -1), (12, 40, 70)])
def test_forward_takes_special_values_as_the_any_layout_kernel_does(what, value, dh, left, right, copies):
    """Whole tiles and tiles that a window cuts alike: a score that is NaN or below -1e29 counts as a masked key."""
    say("special values", what, value, dh, left, right, copies)
    T, heads = 100, 2
    D = heads * dh
    qkv = np.random.default_rng(690 + dh).standard_normal((2 * T, 3 * D)).astype(F)
    qkv[37, {"q": 0, "k": D, "v": 2 * D}[what] + 5] = value
    got = []
    batch, pair = dev(qkv).repeat(copies, 1), slice(-2 * T, None)
    for t in (batch, moved(batch)):
        lse = torch.empty((2 * T * copies, heads), device="cuda")
        ctx, m = B.aqt_attention_fwd(t, 2 * copies, T, heads, left=left, right=right, lse=lse, want_absmax=True)
        got.append((host(ctx[pair]), host(lse[pair]), host(m).view(np.int32)))
    if what == "v" and not np.isfinite(value) and left >= 0:
        # a masked key's probability is zero: zero times an infinity only where the key's half of a tile is formed at all
        seen = np.abs(np.arange(2 * T) - 37) <= 40
        got = [(c[seen], l, 0) for c, l, _ in got]
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("what,value", [("dctx", np.inf), ("dctx", -np.inf), ("v", np.inf), ("q", np.nan), ("k", np.inf)])
@pytest.mark.parametrize("dh", [16, 32, 36, 64])
@pytest.mark.parametrize("copies", [1, MANY])
def test_backward_keeps_what_is_infinite_and_what_is_finite(what, value, dh, copies):
    """An infinity has no bf16 terms: the same entries come out infinite (with their sign), NaN and finite as with float32
    products.  The finite ones differ by the rounding of sums of T products of order one (2 (T + dh + 8) u of the largest,
    the scores' amplification included: dP - D cancels)."""
    say("special values, backward", what, value, dh, copies)
    T, heads = 100, 2
    D = heads * dh
    rng = np.random.default_rng(691 + dh)
    qkv, go = rng.standard_normal((2 * T, 3 * D)).astype(F), rng.standard_normal((2 * T, D)).astype(F)
    if what == "dctx":
        go[37, 5] = value
    else:
        qkv[37, {"q": 0, "k": D, "v": 2 * D}[what] + 5] = value
    qkv_d, go_d, n = dev(qkv).repeat(copies, 1), dev(go).repeat(copies, 1), 2 * copies
    lse = torch.empty((n * T, heads), device="cuda")
    ctx, _ = B.aqt_attention_fwd(qkv_d, n, T, heads, lse=lse)
    a = host(B.aqt_attention_bwd(qkv_d, ctx, go_d, lse, n, T, heads)[-2 * T:])
    b = host(B.aqt_attention_bwd(moved(qkv_d), ctx, go_d, lse, n, T, heads)[-2 * T:])
    fine = np.isfinite(b)
    assert (~fine).any() and fine[T:].all()   # the other utterance is untouched
    np.testing.assert_array_equal(a[~fine], b[~fine])
    assert np.isfinite(a[fine]).all() and np.abs(a[fine] - b[fine]).max() <= 2 * (T + dh + 8) * U * np.abs(b[fine]).max()


@pytest.mark.parametrize("what", ["dctx", "v", "k", "q"])
@pytest.mark.parametrize("dh,T,left,right", [(64, 100, -1, -1), (32, 300, 30, 45), (36, 130, -1, 3), (4, 40, 5, -1)])
@pytest.mark.parametrize("copies", [1, MANY])
def test_backward_with_values_beyond_bf16(what, dh, T, left, right, copies):
    """Finite in float32, an infinity if rounded to bf16: the gradients stay finite and right."""
    from parity_util import check_grad
    say("beyond bf16", what, dh, T, left, right, copies)
    heads = 2
    D = heads * dh
    rng = np.random.default_rng(692 + dh)
    qkv, go = rng.standard_normal((2 * T, 3 * D)).astype(F), (1e-3 * rng.standard_normal((2 * T, D))).astype(F)
    if what == "dctx":
        qkv[:, 2 * D:] *= F(0.1)
        go[37, 2] = BIG
    else:
        at = {"q": 0, "k": D, "v": 2 * D}[what] + 2
        if what != "v":                        # the score's other factor is zero, so that the scores stay what they are
            qkv[:, {"q": D, "k": 0}[what] + 2] = 0.0
        qkv[37, at] = BIG
    qkv_d, go_d, n = dev(qkv).repeat(copies, 1), dev(go).repeat(copies, 1), 2 * copies
    lse = torch.empty((n * T, heads), device="cuda")
    ctx, _ = B.aqt_attention_fwd(qkv_d, n, T, heads, left=left, right=right, lse=lse)
    got = host(B.aqt_attention_bwd(qkv_d, ctx, go_d, lse, n, T, heads, left=left, right=right)[-2 * T:]).reshape(2, T, 3 * D)
    ref, mag = oracle.attention_bwd(qkv.reshape(2, T, 3 * D), go.reshape(2, T, D), heads, left, right)
    assert np.isfinite(got).all()
    check_grad(got, ref, mag, "dqkv")


@pytest.mark.parametrize("T,left,right", [(1, -1, -1), (16, 3, 0), (40, 23, 0), (65, -1, 2), (217, 40, 33), (230, -1, -1)])
@pytest.mark.parametrize("dh", [4, 20, 36, 64])
def test_few_utterances_have_the_bits_of_many(T, left, right, dh):
    """A small batch takes tiles of 16 queries, a large one of 128: every sum in the same order."""
    say("few and many", T, left, right, dh)
    heads = 2
    D, many = heads * dh, 300
    assert -(-T // 16) * heads * 2 <= 512 < -(-T // 16) * heads * many
    qkv = np.random.default_rng(695 + T + dh).standard_normal((2 * T, 3 * D)).astype(F)
    qkv[: T // 2] *= 6
    few_d = dev(qkv)
    many_d = few_d.view(1, 2 * T, 3 * D).expand(many // 2, -1, -1).contiguous().view(many * T, 3 * D)
    got = []
    for x, B_ in ((few_d, 2), (many_d, many)):
        lse = torch.empty((B_ * T, heads), device="cuda")
        ctx, m = B.aqt_attention_fwd(x, B_, T, heads, left=left, right=right, lse=lse, want_absmax=True)
        got.append((host(ctx[-2 * T:]), host(lse[-2 * T:]), host(m)))
    check_attention(got[0][0], qkv, 2, T, D, heads, left, right)
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("T", [1, 33, 95])
@pytest.mark.parametrize("D,bw", [(64, 8), (68, 4), (132, 8), (508, 4), (512, 8), (512, 4), (516, 8), (60, 4)])
def test_small_output_projections_quantize_inside_the_product(T, D, bw):
    """Row lengths on and next to the ends of the range whose product makes the codes itself, and of its slices: the module's
    codes, scale and result are those of the quantizer and the product called one by one, and an infinity is reported."""
    say("quantizer inside the product", T, D, bw)
    rng = np.random.default_rng(760 + T + D)
    heads, policy = D // 4 if D % 16 else 16, ((8, 8), (bw, 8))
    x, wqkv, wo, bo = (rng.standard_normal(s).astype(F) for s in ((T, D), (D, 3 * D), (D, D), (D,)))
    sv = B.MhsaSaved(1, T, D, policy)
    y = B.aqt_mhsa_fwd(dev(x), dev(wqkv), None, dev(wo), dev(bo), sv, heads)
    m = dev(np.float32([np.abs(host(sv.ctx)).max()]))
    q, s, _ = B.aqt_quantize_with_absmax(sv.ctx, 8, m)
    wp, s_w, _, _ = B.aqt_quantize_weights(dev(wo), bw)
    want, _ = B.aqt_dense_fwd_q(q, s, wp, s_w, D, 8, bw, bias=dev(bo))
    np.testing.assert_array_equal(host(sv.out.xq), host(q))
    np.testing.assert_array_equal(host(sv.out.s_x), host(s))
    np.testing.assert_array_equal(host(y), host(want))
    status = B.new_status()
    x[T // 2, 1] = np.inf
    B.aqt_mhsa_fwd(dev(x), dev(wqkv), None, dev(wo), dev(bo), sv, heads, dev_status=status)
    assert host(status)[0] == B.AQT_ERR_NONFINITE


@pytest.mark.parametrize("T,D", [(95, 64), (300, 144), (40, 512)])
def test_modules_may_leave_their_result_over_the_second_layers_input(T, D):
    """A program that only serves needs neither ctx, s nor h behind the call: y over them is what it is elsewhere."""
    say("module results over their scratch", T, D)
    rng = np.random.default_rng(790 + T + D)
    heads, H = D // 16, 2 * D
    p = ((8, 8), (8, 8))
    x, wq, wo, w1, wd, w2, f1, f2 = (dev(rng.standard_normal(s).astype(F)) for s in (
        (T, D), (D, 3 * D), (D, D), (D, 2 * D), (5, D), (D, D), (D, H), (H, D)))

    def mhsa(over):
        sv = B.MhsaSaved(1, T, D, p)
        return B.aqt_mhsa_fwd(x, wq, None, wo, None, sv, heads, y=sv.ctx if over else None)

    def conv(over):
        sv = B.ConvSaved(1, T, D, p)
        return B.aqt_conv_module_fwd(x, w1, None, wd, None, w2, None, sv, pad_left=2, y=sv.s if over else None)

    def ffn(over):
        sv = B.FfnSaved(T, D, H, p)
        return B.aqt_ffn_fwd(x, f1, None, f2, None, sv, y=sv.h.view(-1)[: T * D].view(T, D) if over else None)

    for call in (mhsa, conv, ffn):
        want = host(call(False))
        for _ in range(3):
            np.testing.assert_array_equal(host(call(True)), want, err_msg=call.__name__)


@pytest.mark.parametrize("T,left,right", [(1, -1, -1), (32, 5, 3), (33, -1, -1), (64, -1, -1), (129, 23, 0), (300, -1, 40), (420, -1, -1)])
@pytest.mark.parametrize("dh", [8, 20, 36, 64])
def test_backward_of_few_and_of_many_utterances(T, left, right, dh):
    """From 33 frames on a small batch gives 32 rows to a workgroup, whose wavefronts share the tiles, a large one 128: both against the oracle."""
    from parity_util import check_grad
    say("backward, few and many", T, left, right, dh)
    heads = 2
    D, many = heads * dh, 260
    rng = np.random.default_rng(696 + T + dh)
    qkv, dctx = rng.standard_normal((T, 3 * D)).astype(F), rng.standard_normal((T, D)).astype(F)
    ref, mag = oracle.attention_bwd(qkv.reshape(1, T, 3 * D), dctx.reshape(1, T, D), heads, left, right)
    for B_ in (1, many):
        q, g = (dev(a).view(1, T, -1).expand(B_, -1, -1).contiguous().view(B_ * T, -1) for a in (qkv, dctx))
        lse = torch.empty((B_ * T, heads), device="cuda")
        ctx, _ = B.aqt_attention_fwd(q, B_, T, heads, left=left, right=right, lse=lse)
        got = host(B.aqt_attention_bwd(q, ctx, g, lse, B_, T, heads, left=left, right=right))
        check_grad(got[-T:].reshape(1, T, 3 * D), ref, mag, "dqkv")
