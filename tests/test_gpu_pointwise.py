"""Depthwise convolution, pooling and split-K reduction kernels at the edges of their dispatch: filter sizes with and without
a kernel of their own, windows larger than the image, one-pixel maps, grids just below and above a band of eight workgroups,
average pooling around its batch of seven loads."""
import numpy as np
import pytest

import paper_2504_08795_amd as D
import workloads as wl
from gpu_helpers import GpuNet, oracle_logits, rel_err

pytestmark = pytest.mark.gpu
N = wl.nets
TOL = {"fp32": 5e-6, "bf16": 6e-3}  # 49 terms: 7 * 2^-24 of the row norm and a margin; bf16: one rounding (2^-9) and a margin


def _run(layer, weights, x, dtype):
    with GpuNet([layer], [weights], x.shape, dtype) as g:
        got = g.forward(x)
    return got, oracle_logits([layer], [weights], x, dtype)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("c,h,w,k,s,p", [(8, 1, 1, 3, 1, 1), (8, 2, 3, 3, 2, 1), (136, 31, 15, 3, 1, 1), (128, 32, 16, 3, 1, 1), (64, 33, 31, 3, 2, 0),
                                         (24, 9, 8, 5, 1, 2), (16, 7, 7, 7, 2, 3), (40, 5, 6, 1, 1, 0), (16, 4, 5, 3, 1, 2)])
def test_depthwise_filter_sizes(c, h, w, k, s, p, dtype):
    rng = np.random.default_rng(5)
    L = N.Layer(op=N.OP_CONV, c_in=c, c_out=c, k=k, stride=s, pad=p, groups=c, act=0, in_from=-1)
    wt = rng.normal(0, 1.0 / k, (c, 1, k, k)).astype(np.float32), rng.normal(0, 0.3, c).astype(np.float32)
    e_max, e_l2 = rel_err(*_run(L, wt, rng.normal(0, 1, (c, h, w)).astype(np.float32), dtype))
    assert e_max <= TOL[dtype] and e_l2 <= TOL[dtype], (e_max, e_l2)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("c,h,w,k,s,p", [(8, 1, 1, 3, 2, 1), (20, 11, 13, 3, 1, 1), (8, 5, 5, 2, 1, 1), (16, 9, 9, 2, 2, 0), (12, 8, 7, 4, 2, 1), (8, 6, 6, 5, 3, 2)])
def test_maxpool_filter_sizes(c, h, w, k, s, p, dtype):
    x = np.random.default_rng(6).normal(-2, 1, (c, h, w)).astype(np.float32)
    x[0, 0, 0], x[1, h - 1, w - 1] = -np.inf, np.finfo(np.float32).min
    got, want = _run(N.Layer(op=N.OP_MAXPOOL, c_in=c, c_out=c, k=k, stride=s, pad=p, in_from=-1), (None, None), x, dtype)
    np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("h,w", [(1, 1), (1, 3), (3, 9), (4, 7), (1, 29), (7, 8), (8, 14), (15, 15)])
def test_average_pool_sizes(h, w, dtype):
    x = np.random.default_rng(7).normal(0.5, 1, (72, h, w)).astype(np.float32)
    e_max, e_l2 = rel_err(*_run(N.Layer(op=N.OP_GAVGPOOL, c_in=72, c_out=72, in_from=-1), (None, None), x, dtype))
    assert e_max <= TOL[dtype] and e_l2 <= TOL[dtype], (e_max, e_l2)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("cin,h,w,cout,res", [(16, 5, 7, 20, False), (24, 6, 6, 12, True)])
def test_split_k_reduction(cin, h, w, cout, res, dtype):
    """Few tiles and many taps: K is split over workgroups into more slices than the reduction loads at once."""
    rng = np.random.default_rng(8)
    layers = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=1, stride=1, pad=0, act=0, in_from=-1),
              N.Layer(op=N.OP_CONV, c_in=cout, c_out=cout, k=7, stride=1, pad=3, act=1, in_from=0, res_from=0 if res else -1)]
    wts = [(rng.normal(0, (2.0 / (L.c_in * L.k * L.k)) ** 0.5, (L.c_out, L.c_in, L.k, L.k)).astype(np.float32), rng.normal(0, 0.3, L.c_out).astype(np.float32))
           for L in layers]
    x = rng.normal(0, 1, (cin, h, w)).astype(np.float32)
    with GpuNet(layers, wts, x.shape, dtype) as g:
        got = g.forward(x)
    e_max, e_l2 = rel_err(got, oracle_logits(layers, wts, x, dtype))
    tol = {"fp32": 2e-5, "bf16": 1.5e-2}[dtype]
    assert e_max <= tol and e_l2 <= tol, (e_max, e_l2)


@pytest.mark.parametrize("c", [1, 3])
def test_bf16_rounding(c):
    """fp32 inputs rounded to bf16 on their way in: ties both ways, the carry into the exponent, overflow, denormals, infinities."""
    bits = np.array([0x3f808000, 0x3f818000, 0x3f807fff, 0x3f808001, 0x3fffffff, 0x7f7fffff, 0xff7fffff, 0x7f7f7fff, 0x7f800000, 0xff800000, 0x80000000,
                     0x00018000, 0x00008000, 0x00008001, 0x807fffff, 0x00800000, 0xbf808000, 0xbf818000], np.uint32)
    x = np.resize(bits, (c, 3, 6)).view(np.float32)
    got, want = _run(N.Layer(op=N.OP_MAXPOOL, c_in=c, c_out=c, k=1, stride=1, pad=0, in_from=-1), (None, None), x, "bf16")
    np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("c,h,w,cout,k,s,p", [(1, 5, 4, 8, 3, 1, 1), (2, 9, 11, 40, 5, 2, 4), (4, 13, 7, 64, 7, 2, 3), (3, 40, 33, 96, 3, 2, 0), (3, 1, 1, 16, 1, 1, 0)])
def test_first_convolution_reads_the_image(c, h, w, cout, k, s, p, dtype):
    """One to four planes, padding wider than the window's centre, windows with most taps outside the image."""
    rng = np.random.default_rng(9)
    L = N.Layer(op=N.OP_CONV, c_in=c, c_out=cout, k=k, stride=s, pad=p, act=0, in_from=-1)
    wt = rng.normal(0, (2.0 / (c * k * k)) ** 0.5, (cout, c, k, k)).astype(np.float32), rng.normal(0, 0.3, cout).astype(np.float32)
    e_max, e_l2 = rel_err(*_run(L, wt, rng.normal(0, 1, (c, h, w)).astype(np.float32), dtype))
    assert e_max <= TOL[dtype] and e_l2 <= TOL[dtype], (e_max, e_l2)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("cin,h,w,cout,k,cus", [(960, 7, 7, 160, 1, 128), (256, 3, 5, 24, 3, 128), (512, 7, 7, 512, 3, 192), (2048, 7, 7, 512, 1, 256), (128, 1, 1, 20, 1, 128)])
def test_few_small_tiles(cin, h, w, cout, k, cus, dtype):
    """16-pixel tiles that do not fill the partition: up to 18 steps a wave, and just past it (512 channels, 3x3, fp32)."""
    rng = np.random.default_rng(10)
    L = N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=k, stride=1, pad=k // 2, act=0, in_from=-1)
    wt = rng.normal(0, (2.0 / (cin * k * k)) ** 0.5, (cout, cin, k, k)).astype(np.float32), rng.normal(0, 0.3, cout).astype(np.float32)
    x = rng.normal(0, 1, (cin, h, w)).astype(np.float32)
    with GpuNet([L], [wt], x.shape, dtype, plan_cus=cus) as g:
        got = g.forward(x)
        plan = D.daris_get_launch_plan(g.task, 0)
    steps = cin * k * k // (16 if dtype == "fp32" else 32) // plan["nw"]
    assert (plan["rows"] == 16) == (cin > 128 and steps <= 18), plan      # (the smallest one splits K in neither kernel)
    e_max, e_l2 = rel_err(got, oracle_logits([L], [wt], x, dtype))
    tol = {"fp32": 2e-5, "bf16": 6e-3}[dtype]  # sqrt(4608) * 2^-24 of the row norm and a margin; one bf16 rounding and a margin
    assert e_max <= tol and e_l2 <= tol, (e_max, e_l2)
