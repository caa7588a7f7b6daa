"""GPU parity of the split-operand convolution kernel (bf16 matrix cores, every
fp32 operand the sum of three parts), through the automatic choice on layers
that take it: every tile shape and kind of signature, ragged channels and
positions, filter lengths with and without an unrolled kernel, gates, no
bias.  The host bounds checker walks the same launches and asserts their tiles
(tests/test_split_bounds.py).

Tolerance: a sum of n products in fp32, in any order, rounds to about
2^-24 sqrt(n) of the largest outputs (random signs, unit-variance terms); twice
that, and the fp32 kernel's own error on the same layer may not be less than a
third of it."""
import numpy as np
import pytest
import torch

import oracle
import paper_2507_01040_amd as P
import workloads as W
from gpu_util import dev, normwise

pytestmark = pytest.mark.gpu

LIN, SUM, MEAN = P.AGG_LINEAR, P.AGG_SUM, P.AGG_MEAN
# (g, (B, C_in, C_out, d_image, d_filter), gate (mode, blades) or None, bias,
#  tile WCO.WPOS.NPT, with .16 where a wave has 16 channels instead of 32)
CASES = [
    ((1, 1), (4, 9, 62, 130, 3), None, True, "2.4.2"),
    ((1, 1), (1, 8, 64, 300, 3), (LIN, (0, 1, 2, 3)), True, "1.8.1"),
    ((1, -1), (10, 13, 61, 93, 3), None, False, "1.8.1"),
    ((-1, 1), (1, 24, 64, 128, 3), (MEAN, (3,)), True, "2.2.1"),
    ((-1, 1), (12, 16, 32, 67, 7), (LIN, (1, 3)), True, "1.8.1"),
    ((1, 1), (12, 16, 64, 98, 2), (SUM, (2, 1)), True, "2.4.2"),
    ((1, -1), (6, 13, 61, 90, 5), None, False, "1.4.1"),
    ((1, 1), (103, 7, 64, 19, 5), None, True, "2.2.2"),
    ((-1, 0), (4, 11, 62, 127, 3), (MEAN, (0, 2)), True, "2.4.2"),
    ((-1, -1), (1, 24, 64, 128, 3), None, True, "2.2.1"),
    ((0, 1), (1, 8, 64, 300, 3), (LIN, (3, 0, 1)), True, "1.8.1"),
    ((-1, -1), (6, 13, 61, 90, 5), None, False, "1.4.1"),
    ((1, 1, 1), (2, 16, 32, 26, 3), (MEAN, tuple(range(8))), True, "1.4.1"),
    ((1, 1, 1), (128, 8, 29, 12, 3), (LIN, (7, 0, 3)), True, "1.8.1"),
    ((1, 1, 1), (64, 7, 60, 10, 3), None, False, "1.4.1"),
    ((1, 1, 1), (5, 7, 32, 34, 3), (LIN, (7, 0, 3)), True, "1.4.1"),
    ((1, 1, 1), (9, 15, 29, 34, 2), None, False, "1.8.1"),
    ((1, -1, 1), (8, 6, 20, 34, 3), None, True, "1.8.1"),
    ((1, 0, 1), (64, 8, 60, 10, 3), (SUM, (4, 1)), True, "1.4.1"),
    ((-1,), (2000, 21, 62, 61, 17), (LIN, (1, 0)), True, "2.2.2"),
    ((1,), (700, 32, 64, 260, 5), None, False, "2.4.2"),
    ((-1,), (1024, 13, 64, 515, 9), (MEAN, (1,)), True, "2.4.4"),
    ((-1,), (5800, 32, 30, 60, 17), (SUM, (0, 1)), True, "1.8.2"),
    ((1,), (512, 93, 96, 200, 5), None, True, "1.4.2"),
    ((1, 1), (5, 13, 16, 258, 3), (LIN, (0, 1, 2, 3)), True, "1.8.1.16"),
    ((-1, 1), (8, 24, 11, 131, 5), None, True, "1.8.1.16"),
    ((1, -1), (8, 32, 16, 182, 3), (SUM, (3, 1)), False, "1.8.1.16"),
    ((-1, 0), (5, 12, 15, 258, 3), (MEAN, (0, 2)), True, "1.8.1.16"),
    ((1, 1), (4, 8, 16, 300, 3), None, True, "1.8.1.16"),
]
IDS = ["%s-%s" % ("".join(str(v) for v in g), "x".join(str(v) for v in s)) for g, s, _, _, _ in CASES]


def _inputs(g, shape, gate, bias, seed):
    B, C_in, C_out, d, df = shape
    _, x, f, b = W.random_conv_case(seed, len(g), g, B, C_in, C_out, d, df, bias_std=0.1)
    act = None
    if gate is not None:
        rng = np.random.default_rng(seed + 1)
        mode, blades = gate
        aw = rng.standard_normal((C_out, len(blades))).astype(np.float32) if mode == LIN else None
        ab = (0.1 * rng.standard_normal(C_out)).astype(np.float32) if mode == LIN else None
        act = (mode, blades, aw, ab)
    return x, f, (b if bias else None), act


def _run(g, x, f, b, act, algo):
    a = None if act is None else (act[0], act[1], None if act[2] is None else dev(act[2]),
                                  None if act[3] is None else dev(act[3]))
    k = len(g)
    d_out = x.shape[2] - f.shape[2] + 1
    y = torch.full((x.shape[0], f.shape[1]) + (d_out,) * k + (1 << k,), float("nan"),
                   dtype=torch.float32, device="cuda:0")
    P.conv_nd(dev(x), dev(f), None if b is None else dev(b), g, act=a, out=y, algo=algo)
    torch.cuda.synchronize()
    return y.cpu().numpy()


@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_conv_split(case):
    g, shape, gate, bias, _ = case
    print(g, shape, gate, flush=True)
    x, f, b, act = _inputs(g, shape, gate, bias, 4000 + sum(shape))
    y = _run(g, x, f, b, act, P.ALGO_AUTO)
    assert np.isfinite(y).all()
    z = _run(g, x, f, b, act, P.ALGO_MFMA)
    assert not np.array_equal(y, z)  # not the fp32 kernels' result
    sel = sorted({0, 1, 2, shape[0] // 2, shape[0] - 2, shape[0] - 1} & set(range(shape[0])))
    if len(g) > 1:
        sel = sorted({0, shape[0] - 1})
    ref = oracle.conv_nd(x[sel], f, np.zeros((shape[2], 1 << len(g)), np.float32) if b is None else b, g)
    if act is not None:
        ref = oracle.act(ref, *act)
    n = shape[1] * (1 << len(g)) * shape[4] ** len(g)
    e, ez = normwise(y[sel], ref), normwise(z[sel], ref)
    print("normwise %.2e, fp32 kernel %.2e" % (e, ez), flush=True)
    assert e <= 2.0 ** -23 * np.sqrt(n)
    assert e <= 3 * ez


def test_conv_split_non_finite_filters():
    # every blade of some filter infinite or NaN, also where the table's sign
    # is zero: the classes of the vector kernel
    for g, shape in (((-1, 0), (1, 8, 64, 300, 3)), ((1, 0, 1), (64, 8, 60, 10, 3)),
                     ((1, -1), (10, 13, 61, 93, 3))):
        k = len(g)
        x, f, _, _ = _inputs(g, shape, None, False, 79)
        for i in range(1 << k):
            f[(1, 3 * i) + (1,) * k + (i,)] = np.inf if i % 2 else np.nan
        y = _run(g, x, f, None, None, P.ALGO_AUTO)
        r = _run(g, x, f, None, None, P.ALGO_DIRECT)
        assert np.isnan(r).any() and np.isinf(r).any() and np.isfinite(r).any()
        np.testing.assert_array_equal(np.isnan(y), np.isnan(r))
        np.testing.assert_array_equal(y[np.isinf(r)], r[np.isinf(r)])


@pytest.mark.parametrize("g,shape", [
    ((1, 1), (1, 8, 64, 300, 3)), ((-1, 0), (1, 8, 64, 300, 3)), ((1, 1, 1), (2, 16, 32, 26, 3)),
    ((1, -1, 1), (2, 16, 32, 26, 3)), ((1, 1), (4, 8, 16, 300, 3)), ((-1, 0), (4, 8, 16, 300, 3)),
    ((1, 1, 1), (4, 16, 32, 34, 3))], ids=str)
def test_conv_split_non_finite(g, shape):
    # infinities, NaN, the largest floats and products past them: outputs that
    # bf16 parts cannot hold are those of the vector kernel, the others are
    # untouched
    k = len(g)
    x, f, b, _ = _inputs(g, shape, None, True, 77)
    big = np.float32(3.3e38)
    x[(0, 3) + (4,) * k] = np.inf
    x[(0, 2) + (9,) * k + (1,)] = np.nan
    x[(0, 1) + (14,) * k] = big
    x[(0, 5) + (24,) * k] = 3.4028235e38    # its high bf16 part is infinite, outputs are not
    x[(0, 4) + (20,) * k + (0,)] = -np.inf
    f[(0, 5) + (1,) * k] = 0.0              # zero filter against the values above
    f[(3, 6) + (0,) * k + (1,)] = 0.0
    # products past the largest float, one to an output (sums of several could
    # pass it in one order and not in another)
    f[(1, 9) + (2,) * k] = 0.0
    f[(1, 9) + (2,) * k + (0,)] = big
    y = _run(g, x, f, b, None, P.ALGO_AUTO)
    r = _run(g, x, f, b, None, P.ALGO_DIRECT)
    fin = np.isfinite(r)
    assert (~fin).any() and fin.any() and np.isposinf(r).any() and np.isnan(r).any()
    np.testing.assert_array_equal(np.isfinite(y), fin)
    np.testing.assert_array_equal(np.isnan(y), np.isnan(r))
    np.testing.assert_array_equal(y[np.isinf(r)], r[np.isinf(r)])
    huge = fin & (np.abs(r) > 1e30)
    assert huge.any()
    # a sum of up to n terms of size T rounds to 2^-24 n T; the terms of these
    # outputs are up to the largest float times the largest filter
    T = float(big) * max(1.0, float(np.abs(f[np.abs(f) < 1e30]).max()))
    assert np.max(np.abs(y[huge].astype(np.float64) - r[huge])) <= 2.0 ** -20 * T
    ok = fin & (np.abs(r) <= 1e30)
    # the others: as in test_conv_split, next to outputs of the usual size
    n = shape[1] * (1 << k) * 3 ** k
    usual = ok & (np.abs(r) < 1e3)
    assert np.max(np.abs(y[usual].astype(np.float64) - r[usual])) <= \
        2.0 ** -22 * np.sqrt(n) * np.max(np.abs(r[usual]))


# Layers whose blades differ in size, of every kind of signature: every blade
# keeps its own digits.
SCALED = [((1, 1), (1, 8, 64, 300, 3)), ((1, -1), (10, 13, 61, 93, 3)), ((-1, 1), (12, 16, 32, 67, 7)),
          ((-1, -1), (1, 24, 64, 128, 3)), ((1, 1), (4, 8, 16, 300, 3)),
          ((1, 1, 1), (2, 16, 32, 26, 3)), ((1, -1, 1), (8, 6, 20, 34, 3)),
          ((-1,), (2000, 21, 62, 61, 17))]


@pytest.mark.parametrize("even", [False, True], ids=["scalar", "even"])
@pytest.mark.parametrize("g,shape", SCALED, ids=str)
def test_conv_split_blades_of_different_size(g, shape, even):
    # inputs with blades 1e4, 1, 1, 1e-4, ... and filters of blade 0 (or of the
    # even blades, the others zero).  Each of the 6 C_in N_B / 16 accumulations
    # of a tap loses at most 2^-23 of a partial sum, and no partial sum of a
    # blade is far above the blade's largest output; the error of every blade
    # also stays within three times the fp32 kernel's.
    k = len(g)
    nb = 1 << k
    print(g, shape, even, flush=True)
    x, f, _, _ = _inputs(g, shape, None, False, 31)
    grade = [0, 1] if k == 1 else [0, 1, 1, 2] if k == 2 else [0, 1, 1, 1, 2, 2, 2, 3]
    for i in range(nb):
        x[..., i] *= np.float32(10.0 ** (4 - 4 * grade[i]) if k > 1 else (1e4, 1e-4)[i])
        if grade[i] % 2 or (i and not even):
            f[..., i] = 0.0
        elif i:
            f[..., i] *= np.float32(1e-4)
    y = _run(g, x, f, None, None, P.ALGO_AUTO)
    sel = sorted({0, shape[0] - 1})
    ref = oracle.conv_nd(x[sel], f, np.zeros((shape[2], nb), np.float32), g)
    z = _run(g, x, f, None, None, P.ALGO_MFMA)
    e, ez = (np.abs(v[sel] - ref).reshape(-1, nb).max(0) for v in (y, z))
    size = np.abs(ref).reshape(-1, nb).max(0)
    assert (size > 0).sum() >= nb // 2
    print("error over the blade's largest", e / np.maximum(size, 1e-300), "fp32 kernel",
          ez / np.maximum(size, 1e-300), flush=True)
    n_acc = 6 * -(-shape[1] * nb // 16) * shape[4] ** k
    assert (e <= n_acc * 2.0 ** -23 * size).all()
    assert (e <= 3 * ez).all()


def _time(run, reps):
    run()
    best = 1e9
    for _ in range(3):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            run()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / reps)
    return best


@pytest.mark.parametrize("g,shape", [
    ((1, 1), (8, 64, 64, 128, 3)), ((-1, 0), (4, 12, 16, 258, 3)), ((-1,), (1024, 64, 64, 60, 17)),
    ((1, 1, 1), (2, 32, 32, 32, 3))], ids=str)
def test_conv_split_masked_channel(g, shape):
    # an input channel of the lowest value in all images but one: every output of
    # those is computed again in fp32.  The outputs are the fp32 kernel's
    # but for the order of the sums (filters of that channel are zero for the
    # even output channels, which stay of the usual size), and the layer takes no
    # more than the kernel's own time and twice the fp32 kernel's.
    k = len(g)
    x, f, b, _ = _inputs(g, shape, None, True, 78)
    y0 = _run(g, x, f, b, None, P.ALGO_AUTO)
    x[1:, 1] = -3.4028235e38
    f[1, ::2] = 0.0
    y = _run(g, x, f, b, None, P.ALGO_AUTO)
    z = _run(g, x, f, b, None, P.ALGO_MFMA)
    fin = np.isfinite(z)
    np.testing.assert_array_equal(np.isfinite(y), fin)
    even = np.zeros_like(fin)
    even[:, ::2] = True
    assert fin[even].all() and np.isfinite(y0).all()
    n = shape[1] * (1 << k) * shape[4] ** k
    assert np.max(np.abs(y[even] - z[even])) <= 2.0 ** -22 * np.sqrt(n) * np.max(np.abs(z[even]))
    xt, ft, bt, x0 = dev(x), dev(f), dev(b), dev(np.zeros_like(x))
    out = torch.empty(y.shape, device="cuda:0")
    ms = [_time(lambda: P.conv_nd(v, ft, bt, g, out=out, algo=algo), 5)
          for v, algo in ((xt, P.ALGO_AUTO), (x0, P.ALGO_AUTO), (xt, P.ALGO_MFMA))]
    print("masked, plain, fp32 kernel: %.3f %.3f %.3f ms" % tuple(ms), flush=True)
    assert ms[0] <= ms[1] + 2 * ms[2]


@pytest.mark.parametrize("ex,ew", [(-118, 0), (-124, 0), (0, -118), (-60, -60), (-140, 20), (60, 40),
                                   (100, -20), (0, 110)], ids=str)
@pytest.mark.parametrize("g,shape", [((-1, -1), (1, 24, 64, 128, 3)), ((-1,), (2000, 21, 62, 61, 17)),
                                     ((1, 1, 1), (2, 16, 32, 26, 3))], ids=str)
def test_conv_split_operand_range(g, shape, ex, ew):
    # operands times powers of two, from where the low parts of bf16 run out
    # (subnormal inputs and sums past 2^96 among them): the tolerance of
    # test_conv_split; inputs below 2^-126 keep the bits that they have
    print(g, shape, ex, ew, flush=True)
    x, f, _, _ = _inputs(g, shape, None, False, 80)
    x, f = np.ldexp(x, ex), np.ldexp(f, ew)
    y = _run(g, x, f, None, None, P.ALGO_AUTO)
    sel = sorted({0, shape[0] - 1})
    xs, fs = np.ldexp(x[sel].astype(np.float64), -ex), np.ldexp(f.astype(np.float64), -ew)
    assert (xs.astype(np.float32) == xs).all() and (fs.astype(np.float32) == fs).all()
    ref = oracle.conv_nd(xs.astype(np.float32), fs.astype(np.float32),
                         np.zeros((shape[2], 1 << len(g)), np.float32), g)
    n = shape[1] * (1 << len(g)) * shape[4] ** len(g)
    e = normwise(np.ldexp(y[sel].astype(np.float64), -ex - ew), ref)
    print("normwise %.2e" % e, flush=True)
    assert e <= 2.0 ** -23 * np.sqrt(n)


# Tables with zeros: layers that stay with the fp32 tiles, as the split sums
# would be up to 1.05 times as far from 64 bits, and layers that do not (kind 7
# of the launch checker).
ZEROS = [((0, 1), (6, 3, 62, 100, 7), "1"), ((-1, 0), (6, 5, 62, 100, 7), "1"),
         ((0, 1), (6, 7, 62, 100, 7), "1"), ((1, 0), (6, 9, 62, 100, 7), "1"),
         ((0, 0, 1), (4, 32, 30, 30, 3), "1"), ((0, 1), (6, 11, 62, 100, 7), "7"),
         ((0, 1), (6, 10, 62, 100, 7), "7"), ((0, 1), (6, 13, 62, 100, 7), "7"),
         ((1, 0, -1), (4, 16, 30, 30, 3), "7"), ((1, 0, 1), (4, 5, 30, 30, 3), "7"),
         ((0, 1), (6, 7, 62, 100, 3), "7"), ((1, 0), (8, 9, 60, 130, 3), "7"),
         ((0, 0, -1), (4, 4, 30, 30, 3), "7"), ((0, 0, 1), (8, 12, 60, 34, 2), "7")]


@pytest.mark.parametrize("g,shape,kind", ZEROS, ids=str)
def test_conv_split_zero_signatures(g, shape, kind):
    # the automatic choice is no further from 64 bits than the fp32 tiles
    x, f, _, _ = _inputs(g, shape, None, False, 81)
    y = _run(g, x, f, None, None, P.ALGO_AUTO)
    z = _run(g, x, f, None, None, P.ALGO_MFMA)
    ref = oracle.conv_nd(x[:1], f, np.zeros((shape[2], 1 << len(g)), np.float32), g)
    e, ez = (np.linalg.norm(v[:1] - ref) / np.linalg.norm(ref) for v in (y, z))
    print("2-norm error %.2e, fp32 kernel %.2e" % (e, ez), flush=True)
    assert np.array_equal(y, z) == (kind == "1")
    assert e <= ez
