"""One Conformer encoder layer as one call: bit-identical to its modules called in sequence (each of
which has its own stage-by-stage parity test against the oracle), and, end to end, close to the same
layer evaluated in float64 without any quantization (compared statistically, as a quantized chain
must be: a code that flips upstream changes everything downstream a little)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2203_15952_amd import binding as B

pytestmark = pytest.mark.gpu
F = np.float32


def dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def say(*a):
    print(*a, flush=True)


@pytest.mark.parametrize("n,alpha", [(1, 0.5), (1023, 1.0), (4096, 0.5), (12800 * 512, -0.25)])
def test_residual_add(n, alpha):
    rng = np.random.default_rng(n)
    x, m = rng.standard_normal(n).astype(F), rng.standard_normal(n).astype(F)
    out = B.aqt_residual_add(dev(x), dev(m), alpha)
    np.testing.assert_array_equal(host(out), x + F(alpha) * m)     # float32 product, then float32 sum


def layer_weights(seed, D, H, kw):
    rng = np.random.default_rng(seed)

    def mat(k, n):
        return (rng.standard_normal((k, n)) / np.sqrt(k)).astype(F)

    def vec(n, centre=0.0):
        return (centre + 0.1 * rng.standard_normal(n)).astype(F)

    w = {}
    for p in ("ffn1", "ffn2"):
        w.update({f"{p}_ln_g": vec(D, 1.0), f"{p}_ln_b": vec(D), f"{p}_w1": mat(D, H), f"{p}_b1": vec(H),
                  f"{p}_w2": mat(H, D), f"{p}_b2": vec(D)})
    w.update(att_ln_g=vec(D, 1.0), att_ln_b=vec(D), att_wqkv=mat(D, 3 * D), att_bqkv=vec(3 * D), att_wo=mat(D, D),
             att_bo=vec(D))
    w.update(conv_ln_g=vec(D, 1.0), conv_ln_b=vec(D), conv_w1=mat(D, 2 * D), conv_b1=vec(2 * D),
             conv_wdw=(rng.standard_normal((kw, D)) / np.sqrt(kw)).astype(F), conv_bdw=vec(D),
             conv_norm_scale=vec(D, 1.0), conv_norm_shift=vec(D), conv_w2=mat(D, D), conv_b2=vec(D))
    w.update(out_ln_g=vec(D, 1.0), out_ln_b=vec(D))
    return w


def float_layer(x, w, B_, T, D, heads, kw, pl, left, right):
    """The same encoder layer in float64 with no quantization anywhere."""
    f = {k: v.astype(np.float64) for k, v in w.items()}

    def swish(v):
        return v / (1.0 + np.exp(-v))

    def ffn(r, p):
        xn = oracle.layernorm(r.astype(F), w[f"{p}_ln_g"], w[f"{p}_ln_b"], 1e-6)
        return swish(xn @ f[f"{p}_w1"] + f[f"{p}_b1"]) @ f[f"{p}_w2"] + f[f"{p}_b2"]

    r1 = x + 0.5 * ffn(x, "ffn1")
    xn = oracle.layernorm(r1.astype(F), w["att_ln_g"], w["att_ln_b"], 1e-6)
    qkv = xn @ f["att_wqkv"] + f["att_bqkv"]
    ctx = oracle.attention(qkv.astype(F).reshape(B_, T, 3 * D), heads, left, right).reshape(-1, D)
    r2 = r1 + ctx @ f["att_wo"] + f["att_bo"]
    xn = oracle.layernorm(r2.astype(F), w["conv_ln_g"], w["conv_ln_b"], 1e-6)
    pre = xn @ f["conv_w1"] + f["conv_b1"]
    g = pre[:, :D] / (1.0 + np.exp(-pre[:, D:]))
    v = oracle.depthwise_conv(g.astype(F).reshape(B_, T, D), w["conv_wdw"], w["conv_bdw"], pad_left=pl).reshape(-1, D)
    s, _ = oracle.affine_swish(v, w["conv_norm_scale"], w["conv_norm_shift"])
    r3 = r2 + s @ f["conv_w2"] + f["conv_b2"]
    r4 = r3 + 0.5 * ffn(r3, "ffn2")
    return oracle.layernorm(r4.astype(F), w["out_ln_g"], w["out_ln_b"], 1e-6)


def run_layer(x_d, wd, policy, B_, T, D, H, heads, kw, pl, left, right):
    sv = B.LayerSaved(B_, T, D, H, policy, heads=heads)
    status = B.new_status()
    y = B.aqt_conformer_layer_fwd(x_d, wd, sv, B=B_, T=T, H=H, heads=heads, kw=kw, pad_left=pl, left=left, right=right,
                                  dev_status=status)
    assert host(status)[0] == 0
    return y, sv


def test_conformer_layer_equals_its_modules_in_sequence_and_tracks_the_float_layer():
    B_, T, D, H, heads, kw, pl, left, right = 6, 150, 256, 1024, 4, 15, 14, 23, 0
    M = B_ * T
    say("encoder layer", B_, T, D, H)
    w = layer_weights(800, D, H, kw)
    x = np.random.default_rng(801).standard_normal((M, D)).astype(F)
    wd = {k: dev(v) for k, v in w.items()}
    x_d = dev(x)
    ref = float_layer(x.astype(np.float64), w, B_, T, D, heads, kw, pl, left, right)
    errs = {}
    for name, pattern, bits_w in (("int8", B.AQT_POLICY_ALL, 8), ("int4 except attention", B.AQT_POLICY_EXCEPT_ATTENTION, 4),
                                  ("int4", B.AQT_POLICY_ALL, 4)):
        pol = B.aqt_policy_preset(pattern, 1, 0, bits_w, 8)[0]
        y, sv = run_layer(x_d, wd, pol, B_, T, D, H, heads, kw, pl, left, right)
        y_h = host(y)
        errs[name] = np.linalg.norm(y_h - ref) / np.linalg.norm(ref)
        say(" ", name, "relative error against the float layer", errs[name])
        # the same modules one by one
        def pair(a, b):
            return ((a.bits_w, a.bits_x), (b.bits_w, b.bits_x))
        f1 = B.FfnSaved(M, D, H, pair(pol.ffn1_in, pol.ffn1_out))
        m = B.aqt_ffn_fwd(x_d, wd["ffn1_w1"], wd["ffn1_b1"], wd["ffn1_w2"], wd["ffn1_b2"], f1, gamma=wd["ffn1_ln_g"],
                          beta=wd["ffn1_ln_b"])
        r1 = B.aqt_residual_add(x_d, m, 0.5)
        a = B.MhsaSaved(B_, T, D, pair(pol.attn_qkv, pol.attn_out))
        m = B.aqt_mhsa_fwd(r1, wd["att_wqkv"], wd["att_bqkv"], wd["att_wo"], wd["att_bo"], a, heads, left=left,
                           right=right, gamma=wd["att_ln_g"], beta=wd["att_ln_b"])
        r2 = B.aqt_residual_add(r1, m, 1.0)
        c = B.ConvSaved(B_, T, D, pair(pol.conv_pw1, pol.conv_pw2))
        m = B.aqt_conv_module_fwd(r2, wd["conv_w1"], wd["conv_b1"], wd["conv_wdw"], wd["conv_bdw"], wd["conv_w2"],
                                  wd["conv_b2"], c, pad_left=pl, gamma=wd["conv_ln_g"], beta=wd["conv_ln_b"],
                                  norm_scale=wd["conv_norm_scale"], norm_shift=wd["conv_norm_shift"])
        r3 = B.aqt_residual_add(r2, m, 1.0)
        f2 = B.FfnSaved(M, D, H, pair(pol.ffn2_in, pol.ffn2_out))
        m = B.aqt_ffn_fwd(r3, wd["ffn2_w1"], wd["ffn2_b1"], wd["ffn2_w2"], wd["ffn2_b2"], f2, gamma=wd["ffn2_ln_g"],
                          beta=wd["ffn2_ln_b"])
        r4 = B.aqt_residual_add(r3, m, 0.5)
        _, _, y2, _ = B.aqt_layernorm_quantize(r4, 8, gamma=wd["out_ln_g"], beta=wd["out_ln_b"], quantize=False,
                                               want_y=True)
        np.testing.assert_array_equal(host(y2), y_h)
        for got, want in zip(sv.r, (r1, r2, r3, r4)):
            np.testing.assert_array_equal(host(got), host(want))
    # int8 stays within a few per cent of the float layer; int4 weights cost more, and keeping the attention
    # projections at int8 (Table 2, E7) recovers part of it
    assert errs["int8"] < 0.03
    assert errs["int8"] < errs["int4 except attention"] < errs["int4"] < 0.25


def test_conformer_layer_rejects_float_activations_in_attention():
    B_, T, D, H = 1, 64, 128, 256
    pol = B.aqt_policy_preset(B.AQT_POLICY_ALL, 1, 0, 4, 0)[0]      # weight-only everywhere
    w = {k: dev(v) for k, v in layer_weights(1, D, H, 15).items()}
    sv = B.LayerSaved(B_, T, D, H, pol)
    with pytest.raises(B.AqtError) as e:
        B.aqt_conformer_layer_fwd(torch.zeros((B_ * T, D), device="cuda"), w, sv, B=B_, T=T, H=H, heads=2, kw=15,
                                  pad_left=14)
    assert e.value.status == B.AQT_ERR_UNSUPPORTED


def test_serving_form_on_prepared_weights_equals_the_training_forward():
    # "what you train is what you serve": with the weights quantized once and kept in matrix-core order, the
    # layer (and each module) gives the very bits of the call that quantizes its float32 weights every time
    B_, T, D, H, heads, kw, pl = 4, 160, 256, 1024, 4, 15, 14
    M = B_ * T
    say("serving form", B_, T, D, H)
    w = layer_weights(810, D, H, kw)
    wd = {k: dev(v) for k, v in w.items()}
    x_d = dev(np.random.default_rng(811).standard_normal((M, D)).astype(F))
    for pattern, bits_w in ((B.AQT_POLICY_ALL, 8), (B.AQT_POLICY_EXCEPT_ATTENTION, 4)):
        pol = B.aqt_policy_preset(pattern, 1, 0, bits_w, 8)[0]
        y_train, _ = run_layer(x_d, wd, pol, B_, T, D, H, heads, kw, pl, 23, 0)
        sv = B.LayerSaved(B_, T, D, H, pol).prepare(wd)
        assert sv.policy.ffn1_in.weights_ready == 1 and sv.ffn1.l1.wprep is not None
        no_w = {k: v for k, v in wd.items() if k not in ("ffn1_w1", "ffn1_w2", "ffn2_w1", "ffn2_w2", "att_wqkv", "att_wo",
                                                         "conv_w1", "conv_w2")}
        for _ in range(2):
            y_serve = B.aqt_conformer_layer_fwd(x_d, no_w, sv, B=B_, T=T, H=H, heads=heads, kw=kw, pad_left=pl, left=23,
                                                right=0)
            np.testing.assert_array_equal(host(y_serve), host(y_train))
    # a module alone, shapes off the tuned grid (no prepared operand exists: the packed codes are used as they are)
    Ms, Ds, Hs = 70, 40, 24
    rng = np.random.default_rng(812)
    xs = dev(rng.standard_normal((Ms, Ds)).astype(F))
    w1, w2 = dev((rng.standard_normal((Ds, Hs)) / 6).astype(F)), dev((rng.standard_normal((Hs, Ds)) / 5).astype(F))
    a = B.FfnSaved(Ms, Ds, Hs, ((4, 8), (8, 8)))
    y_a = B.aqt_ffn_fwd(xs, w1, None, w2, None, a)
    b = B.FfnSaved(Ms, Ds, Hs, ((4, 8), (8, 8))).prepare(w1, w2)
    assert b.l1.wprep is None
    y_b = B.aqt_ffn_fwd(xs, None, None, None, None, b)
    np.testing.assert_array_equal(host(y_b), host(y_a))
    # training mode without weights is an argument error
    with pytest.raises(B.AqtError) as e:
        B.aqt_ffn_fwd(xs, None, None, w2, None, a)
    assert e.value.status == B.AQT_ERR_INVALID_ARG


def test_layer_call_replays_from_a_hip_graph():
    # the library allocates nothing and only launches kernels on the caller's stream (its counters are cleared
    # by small kernels, not by memsets), so a whole layer can be recorded once and replayed; every replay is
    # checked against the eager result, with eager work and synchronisations in between
    B_, T, D, H, heads, kw, pl = 3, 130, 256, 512, 4, 15, 14
    M = B_ * T
    say("layer in a HIP graph", B_, T, D, H)
    wd = {k: dev(v) for k, v in layer_weights(820, D, H, kw).items()}
    pol = B.aqt_policy_preset(B.AQT_POLICY_EXCEPT_ATTENTION, 1, 0, 4, 8)[0]
    sv = B.LayerSaved(B_, T, D, H, pol)
    rng = np.random.default_rng(821)
    xs = [dev(rng.standard_normal((M, D)).astype(F)) for _ in range(3)]
    x_in = torch.empty_like(xs[0])
    y = torch.empty((M, D), dtype=torch.float32, device="cuda")
    ws = B.workspace(B.aqt_workspace_bytes(B.AQT_OP_CONFORMER_LAYER_FWD, M, D, H))
    status = B.new_status()

    def layer():
        B.aqt_conformer_layer_fwd(x_in, wd, sv, B=B_, T=T, H=H, heads=heads, kw=kw, pad_left=pl, left=23, right=0, y=y,
                                  ws=ws, dev_status=status)

    eager = []
    for x in xs:
        x_in.copy_(x)
        layer()
        eager.append(host(y).copy())
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        layer()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        layer()
    for rep in range(2):
        for x, want in zip(xs, eager):
            x_in.copy_(x)
            graph.replay()
            np.testing.assert_array_equal(host(y), want)
            B.aqt_residual_add(x_in, x_in, 0.5)          # unrelated eager work between replays
            torch.cuda.synchronize()
    assert host(status)[0] == 0


def torch_float_layer(x, w, B_, T, D, heads, kw, pl, left, right):
    """The encoder layer in float64 PyTorch on the CPU, no quantization, for its gradients by autograd."""
    import torch.nn.functional as Fn

    def ln(r, p):
        return Fn.layer_norm(r, (D,), w[f"{p}_ln_g"], w[f"{p}_ln_b"], eps=1e-6)

    def swish(v):
        return v * torch.sigmoid(v)

    def ffn(r, p):
        return swish(ln(r, p) @ w[f"{p}_w1"] + w[f"{p}_b1"]) @ w[f"{p}_w2"] + w[f"{p}_b2"]

    dh = D // heads
    r1 = x + 0.5 * ffn(x, "ffn1")
    qkv = (ln(r1, "att") @ w["att_wqkv"] + w["att_bqkv"]).reshape(B_, T, 3, heads, dh)
    sc = torch.einsum("bthd,bjhd->bhtj", qkv[:, :, 0], qkv[:, :, 1]) / dh ** 0.5
    t_i, j_i = torch.arange(T)[:, None], torch.arange(T)[None, :]
    ok = torch.ones((T, T), dtype=torch.bool)
    if left >= 0:
        ok &= j_i >= t_i - left
    if right >= 0:
        ok &= j_i <= t_i + right
    ctx = torch.einsum("bhtj,bjhd->bthd", torch.softmax(sc.masked_fill(~ok, float("-inf")), -1), qkv[:, :, 2])
    r2 = r1 + ctx.reshape(-1, D) @ w["att_wo"] + w["att_bo"]
    pre = ln(r2, "conv") @ w["conv_w1"] + w["conv_b1"]
    g = (pre[:, :D] * torch.sigmoid(pre[:, D:])).reshape(B_, T, D).transpose(1, 2)            # [B, D, T]
    v = Fn.conv1d(Fn.pad(g, (pl, kw - 1 - pl)), w["conv_wdw"].t().unsqueeze(1), w["conv_bdw"], groups=D)
    v = v.transpose(1, 2).reshape(-1, D)
    r3 = r2 + swish(v * w["conv_norm_scale"] + w["conv_norm_shift"]) @ w["conv_w2"] + w["conv_b2"]
    r4 = r3 + 0.5 * ffn(r3, "ffn2")
    return Fn.layer_norm(r4, (D,), w["out_ln_g"], w["out_ln_b"], eps=1e-6)


@pytest.mark.parametrize("D,heads", [(18, 2), (20, 1), (516, 12), (1032, 24)])
def test_conformer_layer_backward_halves_the_stream_gradient(D, heads):
    """Rows of every kernel of the normalisation's backward: the halves handed to the feed-forward modules are exact."""
    B_, T, H, kw, pl = 1, 5, 24, 3, 1
    say("encoder layer bwd, halves", D)
    wd = {k: dev(v) for k, v in layer_weights(840, D, H, kw).items()}
    rng = np.random.default_rng(841)
    x_d, dy_d = (dev(rng.standard_normal((B_ * T, D)).astype(F)) for _ in range(2))
    _, sv = run_layer(x_d, wd, B.aqt_policy_preset(B.AQT_POLICY_ALL, 1, 0, 8, 8)[0], B_, T, D, H, heads, kw, pl, -1, -1)
    dx, grads = B.aqt_conformer_layer_bwd(dy_d, x_d, wd, sv, B=B_, T=T, H=H, heads=heads, kw=kw, pad_left=pl, left=-1, right=-1)
    dr4, _, _ = B.aqt_layernorm_bwd(sv.r[3], sv.out_row_stats, dy_d, gamma=wd["out_ln_g"])
    dxn, dw1, _, _, _ = B.aqt_ffn_bwd(B.aqt_residual_add(dr4, dr4, -0.5), sv.ffn2)
    dr3, _, _ = B.aqt_layernorm_bwd(sv.r[2], sv.ffn2.row_stats, dxn, gamma=wd["ffn2_ln_g"], add=dr4)
    dr2, _, _ = B.aqt_layernorm_bwd(sv.r[1], sv.conv.row_stats, B.aqt_conv_module_bwd(dr3, sv.conv, wd["conv_wdw"], pad_left=pl)["dxn"],
                                    gamma=wd["conv_ln_g"], add=dr3)
    dr1, g_a, b_a = B.aqt_layernorm_bwd(sv.r[0], sv.att.row_stats, B.aqt_mhsa_bwd(dr2, sv.att, heads, left=-1, right=-1)["dxn"],
                                        gamma=wd["att_ln_g"], add=dr2)
    dxn1, dw1a, _, _, _ = B.aqt_ffn_bwd(B.aqt_residual_add(dr1, dr1, -0.5), sv.ffn1)
    want, _, _ = B.aqt_layernorm_bwd(x_d, sv.ffn1.row_stats, dxn1, gamma=wd["ffn1_ln_g"], add=dr1)
    for got, ref in ((dx, want), (grads["ffn2_w1"], dw1), (grads["ffn1_w1"], dw1a), (grads["att_ln_g"], g_a), (grads["att_ln_b"], b_a)):
        np.testing.assert_array_equal(host(got), host(ref))


def test_conformer_layer_backward_in_a_workspace_that_folds_each_normalisation():
    """Room for the column sums of one normalisation only: each is folded before the next, the same bits; less is refused."""
    B_, T, D, H, heads, kw, pl = 2, 33, 64, 256, 4, 5, 2
    M = B_ * T
    say("encoder layer bwd, small workspace")
    wd = {k: dev(v) for k, v in layer_weights(842, D, H, kw).items()}
    rng = np.random.default_rng(843)
    x_d, dy_d = (dev(rng.standard_normal((M, D)).astype(F)) for _ in range(2))
    _, sv = run_layer(x_d, wd, B.aqt_policy_preset(B.AQT_POLICY_ALL, 1, 0, 8, 8)[0], B_, T, D, H, heads, kw, pl, -1, -1)
    need = B.aqt_workspace_bytes(B.AQT_OP_CONFORMER_LAYER_BWD, M, D, H)
    spare = B.aqt_workspace_bytes(B.AQT_OP_CONFORMER_LAYER_BWD, M, D, H) - 4 * B.aqt_workspace_bytes(B.AQT_OP_LAYERNORM_BWD, M, D, 1)
    shape = dict(B=B_, T=T, H=H, heads=heads, kw=kw, pad_left=pl, left=-1, right=-1)
    got = [B.aqt_conformer_layer_bwd(dy_d, x_d, wd, sv, ws=B.workspace(n), **shape) for n in (need, spare)]
    np.testing.assert_array_equal(host(got[0][0]), host(got[1][0]))
    for k in got[0][1]:
        if got[0][1][k] is not None:
            np.testing.assert_array_equal(host(got[0][1][k]), host(got[1][1][k]), err_msg=k)
    with pytest.raises(B.AqtError):
        B.aqt_conformer_layer_bwd(dy_d, x_d, wd, sv, ws=B.workspace(need // 8), **shape)


def test_conformer_layer_backward_equals_its_modules_and_tracks_the_float_gradient():
    B_, T, D, H, heads, kw, pl, left, right = 4, 150, 256, 1024, 4, 15, 14, 23, 0
    M = B_ * T
    say("encoder layer bwd", B_, T, D, H)
    w = layer_weights(830, D, H, kw)
    rng = np.random.default_rng(831)
    x = rng.standard_normal((M, D)).astype(F)
    dy = (0.1 * rng.standard_normal((M, D))).astype(F)
    wd = {k: dev(v) for k, v in w.items()}
    x_d, dy_d = dev(x), dev(dy)
    # float64 reference gradients by autograd (CPU)
    wt = {k: torch.tensor(v, dtype=torch.float64, requires_grad=True) for k, v in w.items()}
    xt = torch.tensor(x, dtype=torch.float64, requires_grad=True)
    torch_float_layer(xt, wt, B_, T, D, heads, kw, pl, left, right).backward(torch.tensor(dy, dtype=torch.float64))
    errs = {}
    for name, bits_w in (("int8", 8), ("int4", 4)):
        pol = B.aqt_policy_preset(B.AQT_POLICY_ALL, 1, 0, bits_w, 8)[0]
        y, sv = run_layer(x_d, wd, pol, B_, T, D, H, heads, kw, pl, left, right)
        dx, grads = B.aqt_conformer_layer_bwd(dy_d, x_d, wd, sv, B=B_, T=T, H=H, heads=heads, kw=kw, pad_left=pl,
                                              left=left, right=right)
        assert set(grads) == set(w) - {"conv_norm_scale", "conv_norm_shift"}

        def rel(a, b):
            return float(np.linalg.norm(a - b) / np.linalg.norm(b))
        e = {"dx": rel(host(dx), xt.grad.numpy())}
        for k in grads:
            e[k] = rel(host(grads[k]), wt[k].grad.numpy())
        errs[name] = e
        say(" ", name, "dx", round(e["dx"], 4), "worst weight gradient", max(e, key=e.get), round(max(e.values()), 4))
        # the same backward through the public module calls, bit for bit
        def pair(a, b):
            return ((a.bits_w, a.bits_x), (b.bits_w, b.bits_x))
        dr4, g_o, b_o = B.aqt_layernorm_bwd(sv.r[3], sv.out_row_stats, dy_d, gamma=wd["out_ln_g"])
        half = B.aqt_residual_add(dr4, dr4, -0.5)                          # dr4 / 2, exactly
        dxn, dw1, db1, dw2, db2 = B.aqt_ffn_bwd(half, sv.ffn2)
        dr3, g_f2, _ = B.aqt_layernorm_bwd(sv.r[2], sv.ffn2.row_stats, dxn, gamma=wd["ffn2_ln_g"], add=dr4)
        c = B.aqt_conv_module_bwd(dr3, sv.conv, wd["conv_wdw"], pad_left=pl)
        dr2, _, _ = B.aqt_layernorm_bwd(sv.r[1], sv.conv.row_stats, c["dxn"], gamma=wd["conv_ln_g"], add=dr3)
        a = B.aqt_mhsa_bwd(dr2, sv.att, heads, left=left, right=right)
        dr1, _, _ = B.aqt_layernorm_bwd(sv.r[0], sv.att.row_stats, a["dxn"], gamma=wd["att_ln_g"], add=dr2)
        half = B.aqt_residual_add(dr1, dr1, -0.5)
        dxn1, dw1a, _, _, _ = B.aqt_ffn_bwd(half, sv.ffn1)
        dx_b, _, _ = B.aqt_layernorm_bwd(x_d, sv.ffn1.row_stats, dxn1, gamma=wd["ffn1_ln_g"], add=dr1)
        np.testing.assert_array_equal(host(dx_b), host(dx))
        for got, want in ((grads["out_ln_g"], g_o), (grads["out_ln_b"], b_o), (grads["ffn2_w1"], dw1),
                          (grads["ffn2_w2"], dw2), (grads["ffn2_ln_g"], g_f2), (grads["conv_wdw"], c["dw_dw"]),
                          (grads["conv_w1"], c["dw1"]), (grads["att_wqkv"], a["dwqkv"]), (grads["att_bo"], a["dbo"]),
                          (grads["ffn1_w1"], dw1a)):
            np.testing.assert_array_equal(host(got), host(want))
    # straight-through gradients of the int8 layer stay close to the float layer's true gradients; int4 is coarser
    assert errs["int8"]["dx"] < 0.05 and max(errs["int8"].values()) < 0.10
    assert errs["int8"]["dx"] < errs["int4"]["dx"] < 0.40


def test_native_quantization_aware_training_reduces_the_loss_and_serves_what_it_trained():
    # two encoder layers (the first with int4 weights), Adam on the float32 master weights, gradients from
    # aqt_conformer_layer_bwd; then the serving form on weights quantized once
    from paper_2203_15952_amd import train_demo
    out = train_demo.main(["--steps", "40", "--utterances", "4", "--frames", "96", "--d-model", "128", "--d-ff", "256",
                           "--heads", "2"])
    say(out)
    assert out["device_status"] == 0
    assert out["loss_last"] < 0.6 * out["loss_first"]
    assert out["served_equals_trained_bit_for_bit"]
    assert out["weight_bytes_quantized"] < 0.25 * out["weight_bytes_float32"]
