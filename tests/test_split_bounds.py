"""The split-operand convolution's launches (tests/test_conv_split_gpu.py and
the benchmark's layers), walked by the host bounds checker before any GPU sees
them: every load, LDS slot and store of its address arithmetic
(tests/hostcheck/check_conv_split.cpp), and the tile each layer takes.  The
layers of the other GPU tests that the automatic choice gives to the split
kernels, and random ones, are walked too."""
import os
import sys

import numpy as np

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

import paper_2507_01040_amd as P  # noqa: E402
import workloads as W  # noqa: E402
from hostcheck import build as HC  # noqa: E402
from test_host_bounds import conv_line  # noqa: E402


def _run(lines):
    return HC.run(lines)


def test_parity_cases():
    import test_conv_split_gpu as T
    lines = [conv_line(len(g), g, *shape, P.ALGO_AUTO, gate) for g, shape, gate, _, _ in T.CASES]
    for res, (g, shape, _, _, tile) in zip(_run(lines), T.CASES):
        f = res.split()
        assert f[0] == "ok" and f[4] == "7", (g, shape, res)
        t = f[5].split(".")
        assert ".".join(t[3:6] + (["16"] if t[7] == "16" else [])) == tile, (g, shape, res)


def test_zero_signatures():
    import test_conv_split_gpu as T
    lines = [conv_line(len(g), g, *shape, P.ALGO_AUTO) for g, shape, _ in T.ZEROS]
    for res, (g, shape, kind) in zip(_run(lines), T.ZEROS):
        f = res.split()
        assert f[0] == "ok" and f[4] == kind, (g, shape, res)


def test_benchmark_layers_and_sizes():
    # the benchmark's convolutions, and layers that stay with the fp32 kernels:
    # small ones, forced tiles, the vector kernel, linear layers
    lines, want = [], []
    for name in ("conv2d_c64_d128", "conv3d_c32_d32", "block2d_c64_d130", "block3d_c64_d36"):
        for s in W.WORKLOADS[name].layers:
            lines.append(conv_line(s.k, s.g, s.B, s.C_in, s.C_out, s.d_image, s.d_filter, P.ALGO_AUTO))
            want.append("7")
    big = (2, (1, 1), 8, 64, 64, 128, 3)
    for algo, kind in ((P.ALGO_MFMA, "1"), (P.ALGO_MFMA_WIDE, "1"), (P.ALGO_DIRECT, "3")):
        lines.append(conv_line(*big, algo))
        want.append(kind)
    # few steps: the K group full or not
    for g, shape, kind in (((-1, -1), (13, 3, 62, 324, 2), "1"), ((1, 1), (8, 3, 64, 406, 2), "1"),
                           ((-1, -1), (5, 4, 63, 488, 2), "7"), ((1, 1), (8, 3, 64, 258, 3), "7")):
        lines.append(conv_line(2, g, *shape, P.ALGO_AUTO))
        want.append(kind)
    for k, g, shape in ((2, (1, 1), (8, 4, 4, 16, 3)), (3, (1, 1, 1), (2, 8, 8, 12, 3)),
                        (2, (1, 1), (1000, 32, 32, 1, 1)), (1, (-1,), (64, 16, 16, 60, 17))):
        lines.append(conv_line(k, g, *shape, P.ALGO_AUTO))
        want.append("2" if k == 1 else "1")
    for line, res, kind in zip(lines, _run(lines), want):
        f = res.split()
        assert f[0] == "ok" and f[4] == kind, (line, res)


def test_observer_without_the_kind():
    # a checker that cannot walk the kernel is not handed it
    res = HC.run(["kinds 6", conv_line(2, (1, 1), 8, 64, 64, 128, 3, P.ALGO_AUTO)])[1].split()
    assert res[0] == "ok" and res[4] == "1", res


def test_linear_layers():
    # the automatic choice takes the split linear kernel for the GPU tests'
    # layers and the benchmark's, and keeps the fp32 kernels for smaller batches
    # and other widths; the forced choices (fp32 tiles, streamed) stay with the
    # fp32 streamed kernel at every batch size
    import test_linear_split_gpu as T
    S = P.ALGO_MFMA_STREAM
    cases = [(g, B, ci, co, gate, "8", "4", "4") for g, B, ci, co, gate, _ in T.CASES]
    cases += [((1, 1), 1 << 20, 32, 32, None, "8", "4", "4"),
              ((1, 1), 16383, 32, 32, None, "1", "1", "4"),
              ((1, 1), 18431, 32, 32, None, "4", "4", "4"),
              ((1, 1), 18432, 32, 32, None, "8", "4", "4"),
              ((1, 1, 1), 32768, 16, 16, None, "4", "4", "4"),
              ((-1,), 32768, 32, 64, None, "4", "4", "4"),
              ((-1,), 16384, 64, 32, None, "8", "4", "4"),
              ((1,), 1 << 21, 32, 32, None, "4", "4", "4"),
              ((1, 1), 1 << 18, 24, 32, None, "1", "1", None)]
    lines, want = [], []
    for g, B, ci, co, gate, *kinds in cases:
        for algo, kind in zip((P.ALGO_AUTO, P.ALGO_MFMA, S), kinds):
            if kind is not None:
                lines.append(conv_line(len(g), g, B, ci, co, 1, 1, algo, gate))
                want.append(kind)
    out = HC.run(lines)
    for line, res, kind in zip(lines, out, want):
        f = res.split()
        assert f[0] == "ok" and f[4] == kind, (line, res, kind)


def test_other_gpu_tests_layers():
    # the automatic choice on the layers of the other GPU tests
    import test_parity_gpu as T
    lines = [conv_line(2, g, *s, P.ALGO_AUTO)
             for g, s in T.WIDE16_CASES + T.DF5_CASES + T.NARROW10_CASES + T.SMALL_CHANNEL_WIDTH_CASES +
             T.WIDE64_CASES]
    lines += [conv_line(3, g, *s, P.ALGO_AUTO) for g, s in T.W3_8_CASES]
    lines += [conv_line(2, (1, 1), *s, P.ALGO_AUTO) for s in T.WIDE_STAGE + T.ROW_BLOCKS]
    lines += [conv_line(2, s[5], *s[:5], P.ALGO_AUTO) for s in T.SNUG]
    lines += [conv_line(2, (1, 1), B, C, C, d, 3, P.ALGO_AUTO)
              for B, C, d in ((2, 16, 2050), (1, 64, 2050), (1, 16, 4098), (1, 32, 3000))]
    lines += [conv_line(1, (-1,), B, ci, co, d, 17, P.ALGO_AUTO)
              for B, ci, co, d in ((1024, 64, 64, 60), (1000, 64, 62, 60), (1001, 64, 64, 61), (2048, 128, 128, 60))]
    out = _run(lines)
    for line, res in zip(lines, out):
        assert res.startswith("ok 0 "), (line, res)
    assert sum(res.split()[4] == "7" for res in out) >= 8


def test_random_layers():
    # layers of the sizes that the split kernels are for: ragged channels and
    # positions, every signature and filter length
    rng = np.random.default_rng(20)
    lines = []
    while len(lines) < 60:
        k = int(rng.choice([1, 2, 2, 3]))
        g = tuple(int(v) for v in rng.choice([-1, 1, 1, -1, 0], k))
        if not any(g):
            continue
        df = int(rng.choice([[5, 9, 17, 30], [2, 3, 3, 4, 5, 7], [2, 3, 3, 4]][k - 1]))
        d = df + int(np.exp(rng.uniform(np.log([16, 16, 6][k - 1]), np.log([600, 200, 30][k - 1]))))
        ci, co = (int(np.exp(rng.uniform(np.log(24), np.log(100)))) for _ in range(2))
        per = 2.0 * ci * co * 4 ** k * (df * (d - df + 1)) ** k  # FLOP of a batch entry
        B = max(1, int(np.exp(rng.uniform(np.log(2e10), np.log(1.5e11))) / per))
        if B * (ci + co) * d ** k * 2 ** k > 3e8:
            continue
        lines.append(conv_line(k, g, B, ci, co, d, df, P.ALGO_AUTO))
    for _ in range(20):
        k = int(rng.choice([1, 2, 3]))
        n, kk = [(128, 128), (128, 64), (64, 128), (64, 256)][int(rng.integers(4))]
        lines.append(conv_line(k, (1,) * k, int(np.exp(rng.uniform(np.log(16384), np.log(1 << 20)))),
                               kk >> k, n >> k, 1, 1, P.ALGO_AUTO))
    out = _run(lines)
    for line, res in zip(lines, out):
        assert res.startswith("ok 0 "), (line, res)
    kinds = [res.split()[4] for res in out]
    assert kinds.count("7") >= 25 and kinds.count("8") >= 10, kinds
