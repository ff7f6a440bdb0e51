"""GPU: the contractions straight from the caller's tensors (gemm_any.hip: the forward for any shape and small problems
on the tuned kernels' grid; gemm_any_f64.hip and gemm_exact.hip: the float ones off that grid) at the sizes where they can go wrong: around the matrix-core steps and groups of the contraction, one row or channel over a
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
    (40, 512, 2048, 4, 1),        # few rows, whole steps: eight wavefronts share the contraction
    (1, 31, 1, 8, 0),             # less than one step, one channel
    (33, 33, 31, 4, 0),           # one beyond a step, odd packed rows
    (32, 128, 64, 8, 2),          # exactly one group and one tile; GLU halves of one block
    (65, 129, 34, 4, 2),          # GLU halves that end inside a block
    (31, 255, 65, 8, 1),          # whole steps that make no group, then a partial one
    (3, 517, 130, 4, 1),
    (700, 144, 2000, 8, 1),       # 64 x 128 tiles
    (1543, 100, 2052, 4, 0),      # the same, packed, partial last step
    (1537, 97, 2054, 8, 2),       # with GLU and odd rows
    (2051, 72, 46, 8, 0),         # several slabs of rows
    (20000, 144, 60, 8, 0),       # 128 x 64 tiles (odd number of 64-channel blocks); many slabs
    (9, 40, 4300, 4, 0),          # dX: a split contraction long enough for the float64 sums
    (130, 3, 2, 8, 0), (130, 2, 3, 4, 0), (9, 15, 17, 8, 1), (9, 31, 14, 4, 2), (200, 33, 5, 4, 0),   # rows shorter than a piece
    (300, 50, 6, 8, 2), (5000, 30, 31, 4, 1), (25000, 17, 129, 8, 0),
    (6, 4400, 33, 8, 0),          # the same for the weight-only forward
    (24700, 96, 130, 8, 0),       # 128 x 64 tiles, short contraction
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
    # off the tuned kernels' grid, which each product has its own of: the float64 sum to about one rounding
    for off, mine, ref, mag in ((M < 128 or K % 128 or N % 32, dx, g["dx"], g["dx_abs"]),
                                (K % 256 or N % 128, dw, g["dw"], g["dw_abs"])):
        if off:
            assert np.all(np.abs(host(mine) - ref) <= 2.0 ** -22 * mag + 1e-37)


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
    (1000, 520, 130),      # float64 dW: partial tiles on every side
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


def test_unaligned_single_slab_stays_in_its_workspace():
    """A fan-in on the tuned grid so wide that its row tiles outnumber the rows reserved at least, on a gradient that is
    4-byte aligned only: nothing behind the workspace is written, and the sums are right."""
    import torch
    M, K, N = 128, 8192, 2048
    print("[bias gradient, unaligned, one slab]", M, K, N, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    x, w = torch.randn((M, K), device="cuda", generator=gen), torch.randn((K, N), device="cuda", generator=gen)
    dy = torch.randn(M * N + 1, device="cuda", generator=gen)[1:].view(M, N)
    sv = B.Saved(M, K, N, 8)
    B.aqt_dense_fwd(x, w, 8, 8, saved=sv)
    need = B.aqt_workspace_bytes(B.AQT_OP_DENSE_BWD, M, K, N)
    ws = torch.full((need + (4 << 20),), 0x5A, dtype=torch.uint8, device="cuda")
    _, dw, db = B.aqt_dense_bwd(dy, sv, 8, 8, want_dx=False, want_dbias=True, ws=ws[:need])
    assert bool((ws[need:] == 0x5A).all())
    ref = dy.double().sum(0)
    assert bool(((db.double() - ref).abs() <= 2.0 ** -24 * ref.abs() * 1.0001 + M * 2.0 ** -53 * dy.double().abs().sum(0)).all())
    xq = sv.xq.double().t().contiguous()
    rounded_once(dw, sv.s_x.double() * (xq @ dy.double()), M, sv.s_x.double() * (xq.abs() @ dy.double().abs()))


def rounded_once(got, ref, terms, mag):
    """A float64 sum of `terms` products, rounded to float32 once: half a unit in the last place (2^-24 of the value; 2^-150
    below the normal range), and what the float64 additions themselves may lose of the magnitudes."""
    import torch
    bound = 2.0 ** -24 * (1 + 2.0 ** -20) * ref.abs() + 2.0 ** -149 + terms * 2.0 ** -53 * mag
    fine = torch.where(torch.isfinite(ref), (got.double() - ref).abs() <= bound, (got.double() == ref) | (got.isnan() & ref.isnan()))
    assert bool(fine.all()), (int((~fine).sum()), fine.numel())


def float64_products(M, K, N, moved=False, wild=False, change=None):
    """dX, dW and the weight-only forward of one layer with their float64 values; moved: tensors that are 4-byte aligned only;
    change: what is done to the float operands."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(M + 3 * K + N)

    def put(t):
        if not moved:
            return t
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")
        buf[1:].copy_(t.reshape(-1))
        return buf[1:].view(t.shape)

    x, w = torch.randn((M, K), device="cuda", generator=gen), torch.randn((K, N), device="cuda", generator=gen)
    dy, xf = torch.randn((M, N), device="cuda", generator=gen) + 0.2, torch.randn((M, K), device="cuda", generator=gen) + 0.2
    sv = B.Saved(M, K, N, 8)
    B.aqt_dense_fwd(x, w, 8, 8, saved=sv)
    if wild:   # infinities, the largest finite value, products and sums that float32 cannot hold but the result can
        for t in (dy, xf):
            t[0, 0], t[M // 2, 1], t[M - 1, 2] = float("inf"), 3.4028234e38, float("-inf")
            t[M // 3, 3:5] = torch.tensor([3.0e38, -3.0e38], device="cuda")
            t[1, :] = 1e-41
    if change:
        change(dy), change(xf)
    dy, xf = put(dy), put(xf)
    dx, dw, _ = B.aqt_dense_bwd(dy, sv, 8, 8)
    y = B.aqt_dense_fwd_wonly(xf, sv.wq_packed, sv.s_w, N, 8)
    dys, q, xq = (dy * sv.s_w).double(), sv.wq_kn.double(), sv.xq.double()
    sx, sw = sv.s_x.double(), sv.s_w.double()
    return dict(dx=(dx, dys @ q.t().contiguous(), N, dys.abs() @ q.abs().t().contiguous()),
                dw=(dw, sx * (xq.t().contiguous() @ dy.double()), M, sx * (xq.abs().t().contiguous() @ dy.double().abs())),
                y=(y, (xf.double() @ q) * sw, K, (xf.double().abs() @ q.abs()) * sw))


@pytest.mark.parametrize("M,K,N,off", [
    (4099, 520, 1000, "dx dw y"), (2051, 1002, 1000, "dx dw y"), (300, 2040, 1030, "dx dw y"), (40, 512, 2048, "dx y"),
    (20000, 384, 1536, "dw"),          # a fan-in that the tuned dW's tiles do not divide, several slabs
    (2000, 1100, 4300, "dx dw y"),     # many tiles, one slab
    (33, 130, 3, "dx dw y"), (1, 1, 1, "dx dw y"), (70, 2, 65, "dx dw y"), (65, 63, 64, "dx dw y"),
    (127, 1000, 1100, "dx dw y"), (128, 1000, 1100, "dx dw y"),          # digits: dW from two steps of rows on,
    (24500, 3, 60, "dx dw y"), (24500, 4, 60, "dx dw y"),                # and four fan-in positions
    (5000, 130, 127, "dx dw y"), (5000, 130, 128, "dx dw"), (5000, 127, 130, "dx dw y")])   # dX and weight-only from 128 positions on
def test_off_the_grid_sums_are_float64(M, K, N, off):
    """Shapes that the tuned kernels do not divide: the float64 sum, rounded to float32 once."""
    print("[float64 sums]", M, K, N, flush=True)
    for what, (got, ref, terms, mag) in float64_products(M, K, N).items():
        if what in off.split():
            rounded_once(got, ref, terms, mag)


def test_off_the_grid_by_alignment():
    """Sizes of the tuned kernels' grid on tensors that are not 16-byte aligned: float64 sums as well."""
    for M, K, N in ((512, 256, 256), (20000, 512, 512)):
        print("[float64 sums, 4-byte aligned]", M, K, N, flush=True)
        for got, ref, terms, mag in float64_products(M, K, N, moved=True).values():
            rounded_once(got, ref, terms, mag)


@pytest.mark.parametrize("M,K,N", [(300, 131, 77), (40, 512, 128)])
def test_off_the_grid_infinite_and_huge_values(M, K, N):
    """Infinities, the largest finite value and intermediate results beyond float32 come out as a float64 loop has them."""
    print("[float64 sums, wild values]", M, K, N, flush=True)
    for what, (got, ref, terms, mag) in float64_products(M, K, N, wild=True).items():
        if what == "dw" and K % 256 == 0:
            continue
        ref32 = ref.float().double()   # a float64 result beyond float32 is an infinity
        rounded_once(got, torch_where_finite(ref32, ref), terms, mag.nan_to_num(0.0, 0.0, 0.0))


@pytest.mark.parametrize("pattern", ["few", "many", "planes", "softmax", "row", "zeros"])
@pytest.mark.parametrize("M,K,N", [(1500, 345, 519), (7600, 67, 128), (500, 1001, 1024)])
def test_off_the_grid_values_far_apart(M, K, N, pattern):
    """Large enough for the digits of gemm_exact.hip, values further apart in a row or column than the digits reach: a few of
    them, most of them, over all of float32's range, as in a softmax's gradient, rows and columns with an infinity among ordinary ones, rows and columns of zeros."""
    import torch
    print("[float64 sums, values far apart]", M, K, N, pattern, flush=True)

    def change(t):
        gen = torch.Generator(device="cuda").manual_seed(t.shape[1])
        if pattern == "few":
            t[torch.rand(t.shape, device="cuda", generator=gen) < 2e-4] *= 2.0 ** -27
        elif pattern == "many":
            t *= torch.exp2(torch.randint(-60, 40, t.shape, device="cuda", generator=gen).float())
        elif pattern == "planes":
            t *= torch.exp2(torch.randint(-140, 90, t.shape, device="cuda", generator=gen).float())
        elif pattern == "softmax":
            t.copy_(torch.softmax(30 * t / t.std(), 1))
        elif pattern == "row":
            t[5, 7], t[M // 2 + 1, t.shape[1] - 1], t[M - 1, 3] = float("inf"), float("nan"), 3.0e38
        else:
            t[64:130], t[:, 10:30] = 0.0, 0.0
            t[3, :] *= 2.0 ** -140

    for what, (got, ref, terms, mag) in float64_products(M, K, N, change=change).items():
        off = {"dx": K % 128 or N % 32, "dw": K % 256 or N % 128, "y": N % 128 or K % 32}[what]
        if off:
            ref32 = ref.float().double()
            rounded_once(got, torch_where_finite(ref32, ref), terms, mag.nan_to_num(0.0, 0.0, 0.0))


def torch_where_finite(ref32, ref):
    import torch
    return torch.where(torch.isfinite(ref32), ref, ref32)


@pytest.mark.parametrize("M,K,N", [
    (300, 256, 1024),      # dX of 6 tiles, dW in slabs of 64 rows (one in part)
    (512, 256, 4160),      # dX: a contraction long enough to leave float32 sums on the way, 32 beyond whole steps
    (131, 128, 4256),      # the same with row tiles in part
    (122000, 256, 128),    # dW: as many slabs as it takes, of 512 rows
    (260, 4160, 256),      # the weight-only forward: as long a contraction
    (700, 1024, 256), (128, 256, 128),
])
def test_small_problems_on_the_tuned_grid(M, K, N):
    """Three bf16 terms and a code's one carry a product whole; sums run in float32 over at most 512 positions (32 steps of
    three passes, a rounding of the running sum each) and in float64 from there: (96 + 4) u of the magnitudes."""
    print("[small, on the grid]", M, K, N, flush=True)
    for what, (got, ref, terms, mag) in float64_products(M, K, N).items():
        if what == "dw" and (K % 256 or M * K * N >= 4000000000):
            continue
        if what == "y" and (N % 128 or -(-M // 128) * -(-N // 128) > 64):
            continue
        assert bool(((got.double() - ref).abs() <= 100 * 2.0 ** -24 * mag + 1e-37).all()), what


@pytest.mark.parametrize("M,K,N,bw,epi", [
    (800, 40, 1024, 8, 0), (799, 40, 992, 4, 0),                           # 800 and 775 split tiles
    (8192, 33, 130, 8, 1), (9217, 33, 130, 4, 0), (9217, 1000, 130, 8, 1),  # 256 and 290 tiles of 64 x 128, one round of 128 x 64
    (4099, 1499, 322, 8, 0), (4099, 1500, 322, 4, 2),                      # 195 of them; 1500 positions
    (10881, 250, 322, 8, 1), (10945, 257, 322, 4, 0), (21889, 250, 322, 8, 2),   # two rounds against three, six against five
    (6600, 999, 642, 8, 0), (6592, 1001, 642, 4, 1), (6593, 1002, 1300, 8, 2),   # 640 channels and more: around 1000 positions
    (2550, 1500, 2570, 4, 0), (2550, 1501, 2570, 4, 1), (2550, 1511, 2570, 4, 2), (2550, 1499, 2570, 4, 0),   # 128 x 128 with int4 weights
    (3000, 1500, 2040, 4, 1),                                              # not with half a round of them
    (2048, 128, 1024, 4, 1), (2049, 128, 1024, 8, 1)])                     # Swish on the tuned grid: 128 and 136 tiles
def test_forward_around_the_lines_between_arrangements(M, K, N, bw, epi):
    """Whatever tile a size takes: the integer sums are exact, the result is their de-quantization, the maximum is the result's."""
    import torch
    print("[arrangements]", M, K, N, bw, epi, flush=True)
    rng = np.random.default_rng(M + K + N)
    x, w = rng.standard_normal((M, K)).astype(np.float32), (rng.standard_normal((K, N)) * K ** -0.5).astype(np.float32)
    sv = B.Saved(M, K, N, bw)
    y = B.aqt_dense_fwd(dev(x), dev(w), 8, bw, epilogue=epi, saved=sv)
    y2, m = B.aqt_dense_fwd_q_absmax(sv.xq, sv.s_x, sv.wq_packed, sv.s_w, N, 8, bw, epilogue=epi)
    _, acc = B.aqt_dense_fwd_q(sv.xq, sv.s_x, sv.wq_packed, sv.s_w, N, 8, bw, epilogue=epi, want_acc=True)
    exact = torch.matmul(sv.xq.double(), sv.wq_kn.double().contiguous())   # whole numbers below 2^53
    assert torch.equal(acc.double(), exact)
    v = acc.float() * (sv.s_x * sv.s_w)
    h = N // 2
    want = v if epi == 0 else v * torch.sigmoid(v) if epi == 1 else v[:, :h] * torch.sigmoid(v[:, h:])
    # exp and the logistic function built on it: a few roundings each way
    assert torch.all((y - want).abs() <= 2e-6 * want.abs() + 1e-30)
    assert torch.equal(y2, y) and m[0] == y.abs().max()


@pytest.mark.parametrize("M,K,N", [(1, 256, 128), (31, 256, 128), (33, 512, 128), (255, 256, 384), (257, 256, 256), (513, 256, 128), (128, 256, 4096), (130, 256, 4224),
                                   (3072, 256, 256), (3073, 256, 256), (1907, 512, 1024), (1908, 512, 1024),
                                   (2048, 256, 128), (2049, 256, 128), (1809, 512, 1024), (1811, 512, 1024),   # rows of few tiles; products
                                   (64, 1024, 2048), (65, 1024, 2048), (64, 1024, 1024), (17, 2048, 2048), (300, 4096, 2048)])   # single slabs
def test_weight_gradient_of_few_rows(M, K, N):
    """One workgroup per tile up to 3072 rows and 10^9 products, slabs beyond (and where one slab is all): sums of at most 512 rows in float32 (as above), then float64."""
    import torch
    print("[dW, few rows]", M, K, N, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    x, w = torch.randn(M, K, device="cuda", generator=gen), torch.randn(K, N, device="cuda", generator=gen)
    dy = torch.randn(M, N, device="cuda", generator=gen)
    sv = B.Saved(M, K, N, 8)
    B.aqt_dense_fwd(x, w, 8, 8, saved=sv)
    _, dw, db = B.aqt_dense_bwd(dy, sv, 8, 8, want_dx=False, want_dbias=True)
    codes = (sv.xq.double().t().contiguous(), dy.double())
    ref, mag = sv.s_x.double() * (codes[0] @ codes[1]), sv.s_x.double() * (codes[0].abs() @ codes[1].abs())
    assert bool(((dw.double() - ref).abs() <= 100 * 2.0 ** -24 * mag + 1e-37).all())
    rb = dy.double().sum(0)
    assert bool(((db.double() - rb).abs() <= 2.0 ** -24 * rb.abs() + 1e-12 * dy.double().abs().sum(0)).all())
    again = B.aqt_dense_bwd(dy, sv, 8, 8, want_dx=False, want_dbias=True)
    assert torch.equal(again[1], dw) and torch.equal(again[2], db)
    # both gradients in one launch: the same sums as in launches of their own
    dx, _, _ = B.aqt_dense_bwd(dy, sv, 8, 8, want_dw=False)
    both = B.aqt_dense_bwd(dy, sv, 8, 8, want_dbias=True)
    assert torch.equal(both[0], dx) and torch.equal(both[1], dw) and torch.equal(both[2], db)


def fastest(call, calls=20, rounds=8):
    """us of one of `calls` calls in a row, the fastest of some rounds"""
    import torch
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = float("inf")
    for _ in range(rounds):
        a.record()
        for _ in range(calls):
            call()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / calls)
    return best


def test_weight_gradient_of_few_rows_is_not_slower_than_of_many():
    """A wide layer, where one slab of rows is all there are: the split kernel takes 86 us for 64 rows, the other one 20."""
    import torch
    K, N, us = 4096, 2048, []
    for M in (64, 1024):
        print("[dW time]", M, K, N, flush=True)
        sv = B.Saved(M, K, N, 8)
        B.aqt_dense_fwd(torch.randn(M, K, device="cuda"), torch.randn(K, N, device="cuda"), 8, 8, saved=sv)
        dy, dw = torch.randn(M, N, device="cuda"), torch.empty(K, N, device="cuda")
        ws = B.workspace(B.aqt_workspace_bytes(B.AQT_OP_DENSE_BWD, M, K, N))
        us.append(fastest(lambda: B.aqt_dense_bwd(dy, sv, 8, 8, want_dx=False, dw=dw, ws=ws)))
    assert us[0] <= us[1], us


def test_gradients_of_a_softmax_cost_at_most_a_second_plane():
    """Off the grid, logits of standard deviation 3 over 1000 channels: most values lie below the first six digits of their row's
    largest.  Two planes take 1.6 times the time of one; what they stand in for took five times."""
    import torch
    M, K, N = 4099, 520, 1000
    print("[digits, time of a softmax's gradient]", M, K, N, flush=True)
    sv = B.Saved(M, K, N, 8)
    B.aqt_dense_fwd(torch.randn(M, K, device="cuda"), torch.randn(K, N, device="cuda"), 8, 8, saved=sv)
    plain = torch.randn(M, N, device="cuda")
    peaked = torch.softmax(3 * torch.randn(M, N, device="cuda"), 1)
    peaked[torch.arange(M), torch.randint(0, N, (M,))] -= 1
    dx, dw = torch.empty(M, K, device="cuda"), torch.empty(K, N, device="cuda")
    ws = B.workspace(B.aqt_workspace_bytes(B.AQT_OP_DENSE_BWD, M, K, N))
    t = [fastest(lambda: B.aqt_dense_bwd(dy, sv, 8, 8, dx=dx, dw=dw, ws=ws)) for dy in (plain, peaked)]
    assert t[1] <= 2.5 * t[0], t


@pytest.mark.parametrize("M,K,N,bw", [(1, 1, 1, 8), (5, 64, 32, 4), (33, 70, 36, 8), (130, 2, 4, 4), (3, 517, 130, 4), (7, 1030, 8, 4),
                                      (9, 63, 31, 8), (2100, 65, 68, 8), (3, 8, 36, 4), (2, 16, 40, 8), (2, 17, 33, 4), (4, 80, 64, 4), (4, 81, 31, 8)])
@pytest.mark.parametrize("off", [0, 1])   # elements by which the weights and their [K,N] codes are off their alignment
def test_layer_quantizers_in_one_launch_pair(M, K, N, bw, off):
    import torch
    print("[layer quantizers]", M, K, N, bw, off, flush=True)
    c = inputs.small_case(23 + M + K + N, M, K, N, 8, bw, 0, with_bias=False, with_dy=False)
    if N > 2:
        c.w[:, 2] = 0
    q_ref, s_ref = oracle.quantize(c.w, bw, 0)
    x_ref, sx_ref = oracle.quantize(c.x, 8, -1)
    w = torch.empty(K * N + off, device="cuda")[off:].view(K, N)
    w.copy_(dev(c.w))
    sv = B.Saved(M, K, N, bw)
    sv.wq_kn = torch.empty(K * N + off, dtype=torch.int8, device="cuda")[off:].view(K, N)
    B.aqt_dense_fwd(dev(c.x), w, 8, bw, saved=sv.refresh())
    np.testing.assert_array_equal(host(sv.xq), x_ref)
    np.testing.assert_array_equal(host(sv.s_x), sx_ref)
    np.testing.assert_array_equal(host(sv.s_w), s_ref)
    np.testing.assert_array_equal(host(sv.wq_kn), q_ref)
    rows = oracle.pack_int4(q_ref) if bw <= 4 else q_ref.T.view(np.uint8)
    np.testing.assert_array_equal(host(sv.wq_packed).reshape(N, -1), rows)
    c.w[K // 2, N - 1] = np.inf   # one of the matrix's last channels, in neither first slab nor first tile
    status = B.new_status()
    B.aqt_dense_fwd(dev(c.x), dev(c.w), 8, bw, dev_status=status)
    assert int(status.item()) == B.AQT_ERR_NONFINITE
