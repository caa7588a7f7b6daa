"""The split-operand convolution's launches (tests/test_conv_split_gpu.py and
the benchmark's layers), walked by the host bounds checker before any GPU sees
them: every load, LDS slot and store of its address arithmetic
(tests/hostcheck/check_conv_split.cpp), and the tile each layer takes.  An
observer has to say that it knows the kernel ("kinds 7"); without, the
automatic choice stays with the fp32 kernels, whose own tests assert them."""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

import paper_2507_01040_amd as P  # noqa: E402
import workloads as W  # noqa: E402
from hostcheck import build as HC  # noqa: E402
from test_host_bounds import conv_line  # noqa: E402


def _run(lines):
    out = HC.run(["kinds 7"] + lines)
    assert out[0].startswith("ok"), out[0]
    return out[1:]


def test_parity_cases():
    import test_conv_split_gpu as T
    lines = [conv_line(len(g), g, *shape, P.ALGO_AUTO, gate) for g, shape, gate, _, _ in T.CASES]
    for res, (g, shape, _, _, tile) in zip(_run(lines), T.CASES):
        f = res.split()
        assert f[0] == "ok" and f[4] == "7", (g, shape, res)
        t = f[5].split(".")
        assert ".".join(t[2:5] + (["16"] if t[6] == "16" else [])) == tile, (g, shape, res)


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
    res = HC.run([conv_line(2, (1, 1), 8, 64, 64, 128, 3, P.ALGO_AUTO)])[0].split()
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
    out = HC.run(["kinds 8"] + lines)[1:]
    for line, res, kind in zip(lines, out, want):
        f = res.split()
        assert f[0] == "ok" and f[4] == kind, (line, res, kind)
