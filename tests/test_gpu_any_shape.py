"""GPU: the contractions of gemm_any.hip (any shape, straight from the caller's tensors) at the sizes where
they can go wrong: around the matrix-core steps and groups of the contraction, one row or channel over a
block, odd row lengths, every workgroup arrangement, one slab and several."""
import numpy as np
import pytest

import oracle
from paper_2203_15952_amd import binding as B
from paper_2203_15952_amd import inputs
from parity_util import check_float_forward, check_forward, check_grad

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return None if a is None else torch.from_numpy(a).cuda()


def host(t):
    return t.cpu().numpy()


SHAPES = [
    # M, K, N, bits_w, epilogue
    (40, 512, 2048, 4, 1),        # few rows, whole steps: four wavefronts share the contraction
    (1, 31, 1, 8, 0),             # less than one step, one channel
    (33, 33, 31, 4, 0),           # one beyond a step, odd packed rows
    (32, 128, 64, 8, 2),          # exactly one group and one tile; GLU halves of one block
    (65, 129, 34, 4, 2),          # GLU halves that end inside a block
    (31, 255, 65, 8, 1),          # whole steps that make no group, then a partial one
    (3, 517, 130, 4, 1),
    (700, 144, 2000, 8, 1),       # 64 x 128 tiles
    (1543, 100, 2052, 4, 0),      # 128 x 128 tiles, packed, partial last step
    (1537, 97, 2054, 8, 2),       # the same with GLU and odd rows
    (2051, 72, 46, 8, 0),         # several slabs of rows
    (20000, 144, 60, 8, 0),       # 128 x 64 tiles (odd number of 64-channel blocks); many slabs
    (9, 40, 4300, 4, 0),          # dX: a split contraction long enough for the float64 sums
    (130, 3, 2, 8, 0), (130, 2, 3, 4, 0), (9, 15, 17, 8, 1), (9, 31, 14, 4, 2), (200, 33, 5, 4, 0),   # rows shorter than a piece
    (300, 50, 6, 8, 2), (5000, 30, 31, 4, 1), (25000, 17, 129, 8, 0),
    (6, 4400, 33, 8, 0),          # the same for the weight-only forward
    (24700, 96, 130, 8, 0),       # 128 x 128 tiles, short contraction
]


@pytest.mark.parametrize("M,K,N,bw,epi", SHAPES)
def test_forward_and_backward(M, K, N, bw, epi):
    print("[any shape]", M, K, N, bw, epi, flush=True)
    c = inputs.small_case(17 + M + K + N, M, K, N, 8, bw, epi, with_bias=True)
    ora = oracle.dense_fwd(c.x, c.w, 8, bw, c.bias, epi)
    sv = B.Saved(M, K, N, bw)
    y = B.aqt_dense_fwd(dev(c.x), dev(c.w), 8, bw, bias=dev(c.bias), epilogue=epi, saved=sv)
    check_forward(host(y), ora, ora["s_x"][0], ora["s_w"], c.bias, epi)
    y2, acc = B.aqt_dense_fwd_q(sv.xq, sv.s_x, sv.wq_packed, sv.s_w, N, 8, bw, bias=dev(c.bias), epilogue=epi, want_acc=True)
    np.testing.assert_array_equal(host(acc), ora["acc"])
    np.testing.assert_array_equal(host(y2), host(y))
    _, m = B.aqt_dense_fwd_q_absmax(sv.xq, sv.s_x, sv.wq_packed, sv.s_w, N, 8, bw, bias=dev(c.bias), epilogue=epi)
    assert host(m)[0] == np.abs(host(y)).max()
    g = oracle.dense_bwd(c.dy, ora["xq"], ora["s_x"][0], ora["wq"], ora["s_w"])
    dx, dw, _ = B.aqt_dense_bwd(dev(c.dy), sv, 8, bw)
    check_grad(host(dx), g["dx"], g["dx_abs"], "dx")
    check_grad(host(dw), g["dw"], g["dw_abs"], "dw")
    if max(M, N) % 128 and max(K, N) % 128:   # off every tuned tile: the float64 sum to about one rounding
        for mine, ref, mag in ((host(dx), g["dx"], g["dx_abs"]), (host(dw), g["dw"], g["dw_abs"])):
            assert np.all(np.abs(mine - ref) <= 2.0 ** -22 * mag + 1e-37)


@pytest.mark.parametrize("M,K,N,bw,epi", SHAPES)
def test_weight_only_forward(M, K, N, bw, epi):
    print("[any shape, weight only]", M, K, N, bw, epi, flush=True)
    c = inputs.small_case(19 + M + K + N, M, K, N, 8, bw, epi, with_bias=True, with_dy=False)
    wq_ref, sw_ref = oracle.quantize(c.w, bw, 0)
    ora = oracle.dense_fwd_wonly(c.x, wq_ref, sw_ref, c.bias, epi)
    wq, s_w, _, _ = B.aqt_quantize_weights(dev(c.w), bw)
    y = B.aqt_dense_fwd_wonly(dev(c.x), wq, s_w, N, bw, bias=dev(c.bias), epilogue=epi)
    check_float_forward(host(y), ora, epi)


@pytest.mark.parametrize("M,K,N", [
    (15301, 512, 512),     # 256 x 256 dW tiles, the last stage of rows in part
    (61100, 512, 128),     # 256 x 128 tiles; most row tiles' slabs end with a turn that is not theirs
    (30528, 256, 512),     # whole stages, one row tile
    (4096, 2048, 512),     # more row tiles than stages in a slab would share evenly
    (1000, 520, 130),      # any-shape dW: partial tiles on every side
    (33, 129, 3),          # one slab of two slices, two row tiles, fewer than four columns
    (1, 1, 1), (64, 128, 128),
])
def test_bias_gradient_rides_on_dw(M, K, N):
    """The column sums taken inside the dW kernels are float64 sums rounded once: half a float32 ulp, plus the float64
    sums' own M * 2^-53 of the magnitudes.  Without dW they come from their own kernels."""
    import torch
    print("[bias gradient]", M, K, N, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(M + K + N)
    x = torch.randn((M, K), device="cuda", generator=gen)
    w = torch.randn((K, N), device="cuda", generator=gen)
    dy = torch.randn((M, N), device="cuda", generator=gen) + 0.3
    sv = B.Saved(M, K, N, 8)
    B.aqt_dense_fwd(x, w, 8, 8, saved=sv)
    ref = dy.double().sum(0)
    bound = 2.0 ** -24 * ref.abs() * 1.0001 + M * 2.0 ** -53 * dy.double().abs().sum(0)
    for want_dw in (True, False):
        _, _, db = B.aqt_dense_bwd(dy, sv, 8, 8, want_dx=False, want_dw=want_dw, want_dbias=True)
        assert bool(((db.double() - ref).abs() <= bound).all()), (want_dw, float(((db.double() - ref).abs() - bound).max()))
