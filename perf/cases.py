"""The work this library is used for, as cases that can be timed: what a training program, a serving
program and a quantization pass call, through the public entry points of `paper_2203_15952_amd.binding`.

A case is a dict of plain values; its `kind` says which program it stands for:

  dense_fwd    one quantized dense layer, training forward (quantize x, quantize w, product, activation)
  dense_step   training step of the two linear layers K -> N and N -> K: forward and straight-through backward
  ffn_wonly    feed-forward module with integer weights and float32 activations (the weight-only modes)
  quantize     per-tensor abs-max quantizer alone
  layer_serve  Conformer encoder layer, forward, weights quantized once before
  layer_train  Conformer encoder layer, forward and backward, weights quantized in every step

Sizes run from one short utterance to 65536 tokens, model widths from 96 to 512 (the widths, head counts,
kernel sizes and contexts of the tests and of the demonstration programs), whole tiles and ragged sizes.
Values: activations N(0, 1) (with one per cent of outliers at +-8 where `outliers` is set), weights
N(0, 1 / fan-in), upstream gradients N(0, 0.01), biases and normalisation parameters as a trained model
has them.  Everything is drawn on the GPU from the seed.
"""
import math

import torch

from paper_2203_15952_amd import binding as B

EPILOGUE = {"none": B.AQT_EPI_NONE, "swish": B.AQT_EPI_SWISH, "glu": B.AQT_EPI_GLU}
PATTERN = {"all": B.AQT_POLICY_ALL, "except_attention": B.AQT_POLICY_EXCEPT_ATTENTION}


def listed():
    return [
        # one small layer, the single-layer configuration: a few launches
        dict(name="dense_small", kind="dense_fwd", M=256, K=256, N=1024, bits_w=4, epilogue="none", outliers=False),
        # the training step of the two feed-forward layers, the benchmark's configuration
        dict(name="step_65536", kind="dense_step", M=65536, K=512, N=2048, bits_w=4),
        # the same step where no size is a multiple of a tile: a projection to and from an odd-sized vocabulary
        dict(name="step_ragged", kind="dense_step", M=4099, K=520, N=1000, bits_w=8),
        # weight-only inference of a feed-forward module: int4 weights, float32 activations
        dict(name="weight_only_ffn", kind="ffn_wonly", M=12800, D=512, H=2048, bits_w=4),
        # a large activation tensor through the quantizer
        dict(name="quantize_large", kind="quantize", M=65536, K=2048, bits_x=8, outliers=True),
        # serving: one short utterance through a causal layer (latency), a batch, and a narrow model
        dict(name="serve_short", kind="layer_serve", B=1, T=40, D=512, heads=8, kw=15, causal=True, bits_w=4,
             pattern="except_attention"),
        dict(name="serve_batch", kind="layer_serve", B=32, T=400, D=512, heads=8, kw=32, causal=False, bits_w=4,
             pattern="except_attention"),
        dict(name="serve_narrow", kind="layer_serve", B=6, T=217, D=144, heads=4, kw=32, causal=False, bits_w=8,
             pattern="all"),
        # training: the demonstration's small causal model, the batch the configurations name, a narrow model,
        # and a large batch
        dict(name="train_small", kind="layer_train", B=8, T=128, D=256, heads=4, kw=15, causal=True, bits_w=4,
             pattern="all"),
        dict(name="train_batch", kind="layer_train", B=32, T=400, D=512, heads=8, kw=32, causal=False, bits_w=8,
             pattern="all"),
        dict(name="train_narrow", kind="layer_train", B=24, T=417, D=144, heads=4, kw=32, causal=False, bits_w=8,
             pattern="all"),
        dict(name="train_large", kind="layer_train", B=128, T=512, D=512, heads=8, kw=32, causal=False, bits_w=4,
             pattern="except_attention"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """Layer widths: powers-of-two multiples mostly, multiples of 8 often, anything now and then."""
    unit = rng.choice([128, 128, 8, 8, 1])
    return max(lo, min(hi, max(1, _log(rng, lo, hi) // unit) * unit))


def draw(rng):
    kind = rng.choice(["dense_fwd", "dense_step", "ffn_wonly", "quantize", "layer_serve", "layer_serve", "layer_train",
                       "layer_train"])
    if kind == "quantize":
        K = _width(rng, 64, 2048)
        return dict(kind=kind, M=_log(rng, 16, min(65536, 65536 * 2048 // K)), K=K, bits_x=rng.choice([8, 8, 4]),
                    outliers=rng.random() < 0.5)
    if kind in ("dense_fwd", "dense_step"):
        K, N = _width(rng, 64, 2048), _width(rng, 64, 2048)
        most = 65536 * 512 * 2048 if K % 128 == 0 and N % 128 == 0 else 4099 * 520 * 1000
        c = dict(kind=kind, M=_log(rng, 24, max(25, min(65536, most // (K * N)))), K=K, N=N, bits_w=rng.choice([4, 8]))
        if kind == "dense_fwd":
            c.update(epilogue=rng.choice(["none", "swish"] + (["glu"] if N % 2 == 0 else [])), outliers=rng.random() < 0.3)
        return c
    heads = rng.choice([2, 4, 8])
    dh = 4 * rng.randint(6, 16) if rng.random() < 0.5 else rng.choice([32, 64])
    D = min(512, max(96, heads * dh) // heads * heads)
    whole = D % 128 == 0
    if kind == "ffn_wonly":
        return dict(kind=kind, M=_log(rng, 24, 12800 if whole else 4099), D=D, H=4 * D, bits_w=rng.choice([4, 8]))
    while True:
        c = dict(kind=kind, B=_log(rng, 1, 128), T=_log(rng, 16, 1024), D=D, heads=heads, kw=rng.choice([15, 32]),
                 causal=rng.random() < 0.4, bits_w=rng.choice([4, 8]), pattern=rng.choice(["all", "except_attention"]))
        tokens = c["B"] * c["T"]
        if tokens * c["T"] <= 128 * 512 * 512 and tokens * D * D <= (65536 * 512 * 512 if whole else 24 * 417 * 144 * 144):
            return c


def _layer_shape(case):
    kw, causal = case["kw"], case["causal"]
    return dict(B=case["B"], T=case["T"], H=4 * case["D"], heads=case["heads"], kw=kw,
                pad_left=kw - 1 if causal else (kw - 1) // 2, left=23 if causal else -1, right=0 if causal else -1)


def _weights(mat, vec, D, H, kw):
    w = {}
    for p in ("ffn1", "ffn2"):
        w.update({p + "_ln_g": 1 + vec(D), p + "_ln_b": vec(D), p + "_w1": mat(D, H), p + "_b1": vec(H),
                  p + "_w2": mat(H, D), p + "_b2": vec(D)})
    w.update(att_ln_g=1 + vec(D), att_ln_b=vec(D), att_wqkv=mat(D, 3 * D), att_bqkv=vec(3 * D), att_wo=mat(D, D),
             att_bo=vec(D))
    w.update(conv_ln_g=1 + vec(D), conv_ln_b=vec(D), conv_w1=mat(D, 2 * D), conv_b1=vec(2 * D), conv_wdw=mat(kw, D),
             conv_bdw=vec(D), conv_norm_scale=1 + vec(D), conv_norm_shift=vec(D), conv_w2=mat(D, D), conv_b2=vec(D))
    w.update(out_ln_g=1 + vec(D), out_ln_b=vec(D))
    return w


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(*shape, std=1.0):
        t = torch.randn(shape, device="cuda", generator=gen)
        return t if std == 1.0 else t.mul_(std)

    def mat(k, n):
        return normal(k, n, std=k ** -0.5)

    def vec(n):
        return normal(n, std=0.1)

    def activations(m, k):
        x = normal(m, k)
        if case.get("outliers"):
            hit = torch.rand((m, k), device="cuda", generator=gen) < 0.01
            x = torch.where(hit, 8.0 * torch.sign(x), x).contiguous()
        return x

    def buffer(m, n):
        return torch.empty((m, n), dtype=torch.float32, device="cuda")

    kind = case["kind"]
    s = dict(case=case, kind=kind, status=B.new_status())
    if kind == "quantize":
        M, K = case["M"], case["K"]
        s.update(x=activations(M, K), q=torch.empty((M, K), dtype=torch.int8, device="cuda"), scale=torch.empty(1, device="cuda"),
                 ws=B.workspace(B.aqt_workspace_bytes(B.AQT_OP_QUANTIZE, M, K, 1)))
    elif kind == "dense_fwd":
        M, K, N, bw = case["M"], case["K"], case["N"], case["bits_w"]
        epi = EPILOGUE[case["epilogue"]]
        s.update(x=activations(M, K), w=mat(K, N), bias=vec(N), epi=epi, y=buffer(M, N // 2 if epi == B.AQT_EPI_GLU else N),
                 saved=B.Saved(M, K, N, bw), ws=B.workspace(B.aqt_workspace_bytes(B.AQT_OP_DENSE_FWD, M, K, N, 8, bw)))
    elif kind == "dense_step":
        M, bw = case["M"], case["bits_w"]
        s["layers"] = []
        for K, N in ((case["K"], case["N"]), (case["N"], case["K"])):
            s["layers"].append(dict(
                x=activations(M, K), w=mat(K, N), dy=normal(M, N, std=0.1), y=buffer(M, N), dx=buffer(M, K), dw=buffer(K, N),
                saved=B.Saved(M, K, N, bw), ws=B.workspace(B.aqt_workspace_bytes(B.AQT_OP_DENSE_FWD, M, K, N, 8, bw)),
                ws_b=B.workspace(B.aqt_workspace_bytes(B.AQT_OP_DENSE_BWD, M, K, N, 8, bw))))
    elif kind == "ffn_wonly":
        M, D, H, bw = case["M"], case["D"], case["H"], case["bits_w"]
        w1, b1, w2, b2 = mat(D, H), vec(H), mat(H, D), vec(D)
        saved = B.FfnSaved(M, D, H, ((bw, 0), (bw, 0))).prepare(w1, w2)
        s.update(x=activations(M, D), w=(w1, b1, w2, b2), gamma=1 + vec(D), beta=vec(D), y=buffer(M, D), saved=saved,
                 ws=B.workspace(B.aqt_workspace_bytes(B.AQT_OP_FFN_FWD, M, D, H)))
    else:
        M, D = case["B"] * case["T"], case["D"]
        shape = _layer_shape(case)
        H = shape["H"]
        w = _weights(mat, vec, D, H, case["kw"])
        policy = B.aqt_policy_preset(PATTERN[case["pattern"]], 1, 0, case["bits_w"], 8)[0]
        saved = B.LayerSaved(case["B"], case["T"], D, H, policy, heads=case["heads"])
        s.update(x=activations(M, D), w=w, shape=shape, saved=saved, y=buffer(M, D),
                 ws=B.workspace(B.aqt_workspace_bytes(B.AQT_OP_CONFORMER_LAYER_FWD, M, D, H)))
        if kind == "layer_serve":
            saved.prepare(w)
        else:
            s.update(dy=normal(M, D, std=0.1), ws_b=B.workspace(B.aqt_workspace_bytes(B.AQT_OP_CONFORMER_LAYER_BWD, M, D, H)))
    return s


def run(s):
    kind, case = s["kind"], s["case"]
    if kind == "quantize":
        B.aqt_quantize(s["x"], case["bits_x"], B.AQT_AXIS_ALL, q=s["q"], scale=s["scale"], ws=s["ws"], dev_status=s["status"])
        return dict(q=s["q"], scale=s["scale"])
    if kind == "dense_fwd":
        y = B.aqt_dense_fwd(s["x"], s["w"], 8, case["bits_w"], bias=s["bias"], epilogue=s["epi"], y=s["y"], saved=s["saved"],
                            ws=s["ws"], dev_status=s["status"])
        return dict(y=y, xq=s["saved"].xq, wq=s["saved"].wq_packed)
    if kind == "dense_step":
        out = []
        for a in s["layers"]:
            y = B.aqt_dense_fwd(a["x"], a["w"], 8, case["bits_w"], y=a["y"], saved=a["saved"], ws=a["ws"], dev_status=s["status"])
            dx, dw, _ = B.aqt_dense_bwd(a["dy"], a["saved"], 8, case["bits_w"], dx=a["dx"], dw=a["dw"], ws=a["ws_b"])
            out.append(dict(y=y, dx=dx, dw=dw))
        return out
    if kind == "ffn_wonly":
        return dict(y=B.aqt_ffn_fwd(s["x"], *s["w"], s["saved"], gamma=s["gamma"], beta=s["beta"], y=s["y"], ws=s["ws"],
                                    dev_status=s["status"]))
    y = B.aqt_conformer_layer_fwd(s["x"], s["w"], s["saved"], y=s["y"], ws=s["ws"], dev_status=s["status"], **s["shape"])
    if kind == "layer_serve":
        return dict(y=y)
    dx, grads = B.aqt_conformer_layer_bwd(s["dy"], s["x"], s["w"], s["saved"], ws=s["ws_b"], **s["shape"])
    return dict(y=y, dx=dx, grads=grads)


def _weight_bytes(n, bits_w):
    return n / 2 if bits_w <= 4 else n


def work(case):
    kind = case["kind"]
    if kind == "quantize":
        n = case["M"] * case["K"]
        return dict(bytes=5 * n, flops=0)
    if kind in ("dense_fwd", "dense_step"):
        M, K, N = case["M"], case["K"], case["N"]
        if kind == "dense_fwd":
            oc = N // 2 if case["epilogue"] == "glu" else N
            return dict(bytes=4 * M * K + 4 * K * N + 4 * M * oc + M * K + _weight_bytes(K * N, case["bits_w"]), flops=2 * M * K * N)
        # per layer: x, w and dy read, y, dx and dw written; three products
        return dict(bytes=2 * (4 * M * (K + K + N + N) + 8 * K * N), flops=2 * 3 * 2 * M * K * N)
    if kind == "ffn_wonly":
        M, D, H = case["M"], case["D"], case["H"]
        return dict(bytes=8 * M * D + _weight_bytes(2 * D * H, case["bits_w"]), flops=4 * M * D * H)
    D, T, Bc, kw = case["D"], case["T"], case["B"], case["kw"]
    M = Bc * T
    params = 2 * 2 * D * 4 * D + 4 * D * D + 3 * D * D
    keys = sum(min(t, 23) + 1 for t in range(T)) if case["causal"] else T * T      # (query, key) pairs per utterance
    dense, attention, conv = 2 * M * params, 4 * Bc * keys * D, 2 * M * D * kw
    if kind == "layer_serve":
        return dict(bytes=8 * M * D + _weight_bytes(params, case["bits_w"]), flops=dense + attention + conv)
    # forward and the two products of every dense layer's backward; the attention backward has five products to
    # the forward's two, the convolution two to one; x and dy read, y and dx written, weights and their gradients
    return dict(bytes=16 * M * D + 8 * params, flops=3 * dense + 3.5 * attention + 3 * conv)


def tolerance(case):
    kind = case["kind"]
    if kind == "quantize":
        return "exact"
    if kind == "dense_fwd":
        return dict(rel=1e-6, max=2e-5)           # codes and packed weights are whole values and exact
    if kind in ("dense_step", "ffn_wonly"):
        return dict(rel=2e-5, max=1e-3)           # float operand carried as two bf16 terms
    # a layer quantizes what it computed in float32: the last bit of a value can move its 8-bit code by one
    return dict(rel=1e-3, max=0.04)
