"""GPU parity of the split-operand linear kernel (bf16 matrix cores, every fp32
operand the sum of three parts) through clifford_linear: every width it takes,
a ragged last tile with guard rows past B, gates, no bias, zero signs, and
values that bf16 parts cannot hold.  tests/test_split_bounds.py walks the same
launches.

Tolerance: as for the convolution, 2^-23 sqrt(K) of the largest outputs for a
sum of K products, and no more than three times the convolution tile's own
error on the same rows."""
import numpy as np
import pytest
import torch

import oracle
import paper_2507_01040_amd as P
from gpu_util import dev, normwise

pytestmark = pytest.mark.gpu

LIN, SUM, MEAN = P.AGG_LINEAR, P.AGG_SUM, P.AGG_MEAN
B0 = 32768
# (g, B, C_in, C_out, gate or None, bias)
CASES = [
    ((1, 1), B0 + 17, 32, 32, None, True),
    ((-1, 0), B0 + 31, 32, 32, (LIN, (0, 1, 2, 3)), True),
    ((1, -1), 3 * B0 + 1, 16, 32, (SUM, (2, 1)), False),
    ((1, 1), B0, 32, 16, (MEAN, (3,)), True),
    ((0, 1), B0 + 1, 64, 16, None, False),
    ((-1,), B0 + 33, 64, 64, (LIN, (1, 0)), True),
    ((1,), B0 + 2, 128, 32, (MEAN, (0, 1)), True),
    ((-1,), B0 + 5, 32, 64, None, True),
    ((1, 1, 1), B0 + 9, 16, 16, (LIN, tuple(range(8))), True),
    ((0, -1, 1), B0 + 40, 8, 16, (SUM, (7, 4, 3)), True),
    ((1, -1, 1), B0 + 3, 32, 8, None, False),
]


def _inputs(g, B, C_in, C_out, gate, bias, seed):
    nb = 1 << len(g)
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((B, C_in, nb)).astype(np.float32)
    w = (rng.uniform(-1, 1, (C_in, C_out, nb)) / np.sqrt(C_in)).astype(np.float32)
    b = rng.standard_normal((C_out, nb)).astype(np.float32) if bias else None
    act = None
    if gate is not None:
        aw = rng.standard_normal((C_out, len(gate[1]))).astype(np.float32) if gate[0] == LIN else None
        ab = (0.1 * rng.standard_normal(C_out)).astype(np.float32) if gate[0] == LIN else None
        act = (gate[0], gate[1], aw, ab)
    return x, w, b, act


def _run(g, x, w, b, act, algo=None):
    """The rows of the output, after a check that the rows behind it stay as
    they were."""
    a = None if act is None else tuple(v if i < 2 or v is None else dev(v) for i, v in enumerate(act))
    B, C_out, nb = x.shape[0], w.shape[1], x.shape[-1]
    y = torch.full((B + 64, C_out, nb), float("nan"), device="cuda:0")
    xt, wt, bt = dev(x), dev(w), None if b is None else dev(b)
    if algo is None:
        P.linear(xt, wt, bt, g, act=a, out=y[:B])
    else:
        k = len(g)
        P.conv_nd(xt.reshape((B, -1) + (1,) * k + (nb,)), wt.reshape(w.shape[:2] + (1,) * k + (nb,)), bt,
                  g, act=a, out=y[:B].reshape((B, C_out) + (1,) * k + (nb,)), algo=algo)
    torch.cuda.synchronize()
    assert torch.isnan(y[B:]).all()
    return y[:B].cpu().numpy()


@pytest.mark.parametrize("case", CASES, ids=str)
def test_linear_split(case):
    g, B, C_in, C_out, gate, bias = case
    print(case, flush=True)
    x, w, b, act = _inputs(*case, seed=B + C_in)
    y = _run(g, x, w, b, act)
    assert np.isfinite(y).all()
    sel = np.unique(np.r_[0:64, B // 2:B // 2 + 64, B - 64:B])
    ref = oracle.linear(x[sel], w, np.zeros((C_out, x.shape[-1]), np.float32) if b is None else b, g)
    if act is not None:
        ref = oracle.act(ref[:, :, None, :], *act)[:, :, 0, :]
    z = _run(g, x[sel], w, b, act, P.ALGO_MFMA_TINY)
    e, ez = normwise(y[sel], ref), normwise(z, ref)
    print("normwise %.2e, fp32 kernel %.2e" % (e, ez), flush=True)
    assert e <= 2.0 ** -23 * np.sqrt(C_in * x.shape[-1])
    assert e <= 3 * ez
    # every row: against the fp32 tile within both bounds
    full = _run(g, x, w, b, act, P.ALGO_MFMA_TINY)
    assert np.max(np.abs(y - full)) <= 2.0 ** -22 * np.sqrt(C_in * x.shape[-1]) * np.max(np.abs(full))


@pytest.mark.parametrize("case", [((1, 1), B0 + 7, 32, 32, (LIN, (0, 2)), True),
                                  ((0, -1, 1), B0 + 7, 16, 16, None, True)], ids=str)
def test_linear_split_non_finite(case):
    # infinities, NaN and products past the largest float: those outputs are
    # the vector kernel's, the others untouched
    g, B = case[0], case[1]
    x, w, b, act = _inputs(*case, seed=5)
    x[3, 2] = np.inf
    x[40, 1, 1] = np.nan
    x[B - 1, 0, 0] = -np.inf
    x[77, 4, 0] = 3.3e38
    w[4, 3] = 0.0
    w[4, 3, 0] = 5.0          # 77: past the largest float
    w[2, 5] = 0.0             # 3: zero weights against infinities
    y = _run(g, x, w, b, act)
    r = _run(g, x, w, b, act, P.ALGO_DIRECT)
    assert not np.isfinite(r).all()
    np.testing.assert_array_equal(np.isnan(y), np.isnan(r))
    np.testing.assert_array_equal(np.isfinite(y), np.isfinite(r))
    np.testing.assert_array_equal(y[np.isinf(r)], r[np.isinf(r)])
    ok = np.isfinite(r) & (np.abs(r) < 1e3)
    assert np.max(np.abs(y[ok] - r[ok])) <= 1e-5 * np.max(np.abs(r[ok]))


@pytest.mark.parametrize("case", [((1, 1), 4 * B0 + 7, 32, 32, (LIN, (0, 2)), True),
                                  ((-1,), 4 * B0, 64, 32, None, False),
                                  ((0, -1, 1), 4 * B0 + 40, 16, 16, None, True)], ids=str)
def test_linear_split_masked_channel(case):
    # an input channel of the lowest value in all rows but 32: those are
    # computed again in fp32.  The outputs are the fp32 kernel's but for the
    # order of the sums (the channel's weights are zero for the even output
    # channels), in no more than the kernel's own time and the fp32 kernel's
    # twice.
    from test_conv_split_gpu import _time
    g, B, C_in, C_out = case[:4]
    x, w, b, act = _inputs(*case, seed=6)
    x0 = x.copy()
    x[32:, 1] = -3.4028235e38
    w[1, ::2] = 0.0
    y = _run(g, x, w, b, act)
    z = _run(g, x, w, b, act, P.ALGO_MFMA_STREAM)
    np.testing.assert_array_equal(np.isfinite(y), np.isfinite(z))
    assert np.isfinite(z[:, ::2]).all()
    assert np.max(np.abs(y[:, ::2] - z[:, ::2])) <= \
        2.0 ** -22 * np.sqrt(C_in * x.shape[-1]) * np.max(np.abs(z[:, ::2]))
    a = None if act is None else tuple(v if i < 2 or v is None else dev(v) for i, v in enumerate(act))
    wt, bt, out = dev(w), None if b is None else dev(b), torch.empty(y.shape, device="cuda:0")
    k, nb = len(g), x.shape[-1]
    one = (1,) * k + (nb,)
    ms = [_time(lambda: P.conv_nd(v.reshape(v.shape[:2] + one), wt.reshape(w.shape[:2] + one), bt, g,
                                  act=a, out=out.reshape(out.shape[:2] + one), algo=algo), 10)
          for v, algo in ((dev(x), P.ALGO_AUTO), (dev(x0), P.ALGO_AUTO), (dev(x), P.ALGO_MFMA_STREAM))]
    print("masked, plain, fp32 kernel: %.3f %.3f %.3f ms" % tuple(ms), flush=True)
    assert ms[0] <= ms[1] + 2 * ms[2]


@pytest.mark.parametrize("ex,ew", [(-118, 0), (-124, 0), (0, -118), (-140, 20), (60, 40), (0, 110)], ids=str)
def test_linear_split_operand_range(ex, ew):
    # as for the convolution
    g, B, C_in, C_out = (1, 1), B0 + 17, 32, 32
    x, w, _, _ = _inputs(g, B, C_in, C_out, None, False, 8)
    x, w = np.ldexp(x, ex), np.ldexp(w, ew)
    y = _run(g, x, w, None, None)
    sel = np.unique(np.r_[0:64, B - 64:B])
    xs, ws = np.ldexp(x[sel].astype(np.float64), -ex), np.ldexp(w.astype(np.float64), -ew)
    ref = oracle.linear(xs.astype(np.float32), ws.astype(np.float32), np.zeros((C_out, 4), np.float32), g)
    e = normwise(np.ldexp(y[sel].astype(np.float64), -ex - ew), ref)
    print("normwise %.2e" % e, flush=True)
    assert e <= 2.0 ** -23 * np.sqrt(4 * C_in)
