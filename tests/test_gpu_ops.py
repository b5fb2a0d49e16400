"""Per-operator parity of the HIP kernels against the oracle, through the C ABI.

Each case feeds exact fp16 inputs into one operator (after an identity node
that puts the graph input into the sliced layout, where needed) and compares
the operator's output element by element with the oracle.  Shapes cover
several tiles plus ragged tails: channel counts that are not multiples of 8 or
16, pixel counts that are not multiples of the GEMM tile, batch > 1, strides,
dilations and the edge cases 1x1 spatial and a single pixel.
"""
import numpy as np
import pytest

import oracle
import workloads
from workloads import ACT_NONE, ACT_RELU, ACT_RELU6, NetBuilder

from gpu_util import (ISO_RTOL, ISO_RTOL_BF16, check_isolated, check_layer, isolated_reference, labels_check, log,
                      run_gpu)

pytestmark = pytest.mark.gpu


def sliced(g, x):
    """Identity activation: the graph input reaches the next op in sliced form."""
    return g.activation(x, ACT_NONE)


def run_case(name, g, target):
    desc = g.graph(name)
    log(f"[case] {name}")
    _, outs, nodes = run_gpu(desc, materialize_all=True)
    ref = oracle.run_graph(desc)
    return outs, nodes, ref


PW_CASES = [
    # n, h, w, cin, cout, act, residual
    (1, 7, 7, 32, 64, ACT_RELU6, False),
    (3, 5, 5, 12, 13, ACT_RELU, False),
    (1, 56, 56, 128, 128, ACT_RELU6, False),
    (2, 14, 14, 1024, 40, ACT_NONE, False),
    (1, 1, 1, 320, 256, ACT_RELU, False),
    (1, 13, 11, 96, 24, ACT_NONE, True),
    (4, 9, 9, 24, 144, ACT_RELU6, False),
    (2, 7, 7, 160, 160, ACT_NONE, True),
    (64, 7, 7, 64, 200, ACT_RELU6, False),
    # pipelined kernel: K not a multiple of 32, ragged pixel and channel tails,
    # a 128 x 128 tile with a residual epilogue, long K with 64 x 64 tiles
    (1, 13, 13, 200, 72, ACT_RELU6, False),
    (64, 14, 14, 96, 576, ACT_RELU6, True),
    (8, 14, 14, 512, 1024, ACT_RELU, True),
]


@pytest.mark.parametrize("n,h,w,cin,cout,act,res", PW_CASES)
def test_pointwise(n, h, w, cin, cout, act, res):
    g = NetBuilder(seed=cin + cout)
    x = sliced(g, g.input(n, h, w, cin, -1, 1))
    y = g.conv(x, cout, 1, act=act if not res else ACT_NONE)
    if res:
        r = sliced(g, g.input(n, h, w, cout, -2, 2))
        y = g.add(y, r, act=act)
    g.mark_output(y)
    outs, nodes, ref = run_case(f"pw_{n}x{h}x{w}x{cin}->{cout}_a{act}_r{int(res)}", g, y)
    check_isolated("pw", nodes[y], ref[y])
    check_isolated("pw out", outs[0], ref[y].reshape(outs[0].shape))


CONV_CASES = [
    # n, h, w, cin, cout, k, s, d, pads
    (1, 9, 9, 16, 32, 3, 1, 1, None),
    (2, 9, 10, 24, 40, 3, 2, 1, None),
    (1, 12, 12, 32, 16, 3, 1, 2, None),
    (1, 8, 8, 40, 24, 1, 2, 1, (0, 0, 0, 0)),
    (1, 11, 7, 8, 8, 5, 1, 1, None),
    (3, 6, 6, 13, 21, 3, 2, 1, (1, 1, 1, 1)),
]


@pytest.mark.parametrize("n,h,w,cin,cout,k,s,d,pads", CONV_CASES)
def test_conv_window(n, h, w, cin, cout, k, s, d, pads):
    g = NetBuilder(seed=k * 100 + cin)
    x = sliced(g, g.input(n, h, w, cin, -1, 1))
    y = g.conv(x, cout, k, s, d, act=ACT_RELU6, pads=pads)
    g.mark_output(y)
    outs, nodes, ref = run_case(f"conv_{n}x{h}x{w}x{cin}->{cout}_k{k}s{s}d{d}", g, y)
    check_isolated("conv", nodes[y], ref[y])


STEM_CASES = [
    # n, h, w, c, cout, k, s, fp16 input
    (1, 224, 224, 3, 32, 3, 2, False),
    (2, 15, 17, 3, 32, 3, 2, True),
    (1, 13, 13, 3, 24, 3, 1, False),
    (3, 10, 10, 4, 16, 2, 2, False),
    (1, 33, 31, 1, 64, 5, 2, True),
]


@pytest.mark.parametrize("n,h,w,c,cout,k,s,fp16", STEM_CASES)
def test_stem(n, h, w, c, cout, k, s, fp16):
    g = NetBuilder(seed=7)
    x = g.input(n, h, w, c, 0, 1, dtype=workloads.DTYPE_FP16 if fp16 else workloads.DTYPE_FP32)
    y = g.conv(x, cout, k, s, act=ACT_RELU6)
    g.mark_output(y)
    outs, nodes, ref = run_case(f"stem_{n}x{h}x{w}x{c}->{cout}_k{k}s{s}_f16{int(fp16)}", g, y)
    check_isolated("stem", nodes[y], ref[y])


DW_CASES = [
    # n, h, w, c, k, s, d
    (1, 56, 56, 128, 3, 1, 1),
    (1, 112, 112, 32, 3, 2, 1),
    (3, 7, 7, 13, 3, 1, 1),
    (2, 5, 5, 8, 3, 2, 1),
    (1, 1, 1, 24, 3, 1, 1),
    (1, 33, 33, 40, 3, 1, 2),
    (2, 14, 13, 64, 3, 2, 1),
    (1, 9, 9, 16, 5, 1, 1),
    (1, 17, 17, 8, 3, 2, 2),
]


@pytest.mark.parametrize("n,h,w,c,k,s,d", DW_CASES)
def test_depthwise(n, h, w, c, k, s, d):
    g = NetBuilder(seed=c + h)
    x = sliced(g, g.input(n, h, w, c, -1, 1))
    y = g.dw(x, k, s, d, act=ACT_RELU6)
    g.mark_output(y)
    outs, nodes, ref = run_case(f"dw_{n}x{h}x{w}x{c}_k{k}s{s}d{d}", g, y)
    check_isolated("dw", nodes[y], ref[y])


def test_depthwise_activations():
    for act in (ACT_NONE, ACT_RELU):
        g = NetBuilder(seed=3)
        x = sliced(g, g.input(2, 10, 10, 16, -4, 4))
        y = g.dw(x, 3, 1, act=act)
        g.mark_output(y)
        outs, nodes, ref = run_case(f"dw_act{act}", g, y)
        check_isolated("dw", nodes[y], ref[y])


@pytest.mark.parametrize("n,h,w,c", [(2, 7, 7, 40), (1, 33, 33, 320), (1, 1, 1, 8), (64, 7, 7, 1024),
                                      (2, 9, 9, 16), (3, 40, 40, 24)])
def test_global_avgpool(n, h, w, c):
    g = NetBuilder(seed=1)
    x = sliced(g, g.input(n, h, w, c, -1, 1))
    y = g.gap(x)
    g.mark_output(y)
    outs, nodes, ref = run_case(f"gap_{n}x{h}x{w}x{c}", g, y)
    check_isolated("gap", outs[0], ref[y].reshape(n, c))


@pytest.mark.parametrize("n,cin,cout", [(1, 1024, 1000), (3, 20, 7), (64, 1280, 1000), (5, 8, 16)])
def test_fc_softmax(n, cin, cout):
    g = NetBuilder(seed=2)
    x = sliced(g, g.input(n, 1, 1, cin, -1, 1))
    z = g.fc(x, cout)
    p = g.softmax(z)
    g.mark_output(z)
    g.mark_output(p)
    outs, nodes, ref = run_case(f"fc_{n}x{cin}->{cout}", g, p)
    check_isolated("fc", outs[0], ref[z].reshape(n, cout))
    np.testing.assert_allclose(outs[1], ref[p].reshape(n, cout), rtol=1e-5, atol=1e-7)
    np.testing.assert_allclose(outs[1].sum(1), 1.0, rtol=1e-5)


def test_standalone_add_and_activation():
    g = NetBuilder(seed=4)
    a = sliced(g, g.input(2, 6, 5, 13, -3, 3))
    b = sliced(g, g.input(2, 6, 5, 13, -3, 3))
    s = g.add(a, b, act=ACT_RELU6)
    t = g.activation(s, ACT_RELU)
    g.mark_output(t)
    desc = g.graph("add_act")
    log("[case] add_act unfused")
    _, outs, nodes = run_gpu(desc, fuse=False)
    ref = oracle.run_graph(desc)
    check_isolated("add", nodes[s], ref[s])
    check_isolated("act", outs[0], ref[t])


def test_concat_ragged():
    g = NetBuilder(seed=5)
    xs = [sliced(g, g.input(2, 5, 4, c, -1, 1)) for c in (16, 13, 5)]
    y = g.concat(xs)
    g.mark_output(y)
    outs, nodes, ref = run_case("concat_16_13_5", g, y)
    np.testing.assert_array_equal(outs[0], ref[y].astype(np.float32))


@pytest.mark.parametrize("n,h,w,c,oh,ow,align", [(2, 1, 1, 24, 4, 5, 1), (1, 5, 7, 13, 17, 13, 1),
                                                 (1, 33, 33, 21, 513, 513, 1), (1, 6, 4, 8, 9, 11, 0)])
def test_resize(n, h, w, c, oh, ow, align):
    g = NetBuilder(seed=6)
    x = sliced(g, g.input(n, h, w, c, -1, 1))
    y = g.resize(x, oh, ow, bool(align))
    g.mark_output(y)
    outs, nodes, ref = run_case(f"resize_{h}x{w}->{oh}x{ow}_a{align}", g, y)
    check_isolated("resize", outs[0], ref[y])


def test_argmax_exact():
    g = NetBuilder(seed=8)
    x = sliced(g, g.input(2, 9, 7, 21, -1, 1))
    y = g.argmax(x)
    g.mark_output(y)
    outs, nodes, ref = run_case("argmax", g, y)
    np.testing.assert_array_equal(outs[0], ref[y][..., 0])


def test_resize_argmax_fused():
    g = NetBuilder(seed=9)
    x = sliced(g, g.input(1, 33, 33, 21, -1, 1))
    up = g.resize(x, 513, 513, True)
    y = g.argmax(up)
    g.mark_output(y)
    desc = g.graph("resize_argmax")
    log("[case] resize_argmax")
    plan, outs, nodes = run_gpu(desc)
    assert plan.nodes()[-1]["kind"] == "resize_argmax"
    ref = oracle.run_graph(desc)
    bad, covered, raw = labels_check(outs[0], ref[up])
    assert bad == 0 and covered > 0.9, (bad, covered, raw)
    # grid points are exact copies of the input pixels: labels equal the input argmax
    np.testing.assert_array_equal(outs[0][0, ::16, ::16], ref[x].argmax(-1)[0])


def test_graph_cleanup_matches_oracle():
    # identities (activation NONE on a shared tensor, one-input concat,
    # same-size resize) are removed and both PADs fold into the convolutions
    # that consume them (Sec. 3.1); results follow the oracle on the graph as
    # written
    g = NetBuilder(seed=3)
    x = sliced(g, g.input(2, 9, 9, 16, -1, 1))
    a = g.conv(x, 32, 1)
    i3 = g.resize(g.concat([g.activation(a, ACT_NONE)]), 9, 9, True)
    c1 = g.conv(g.pad(i3, (0, 1, 0, 1)), 24, 3, s=2, pads=(0, 0, 0, 0))
    d1 = g.dw(g.pad(a, (1, 1, 1, 1)), 3, s=1, pads=(0, 0, 0, 0))
    y = g.add(g.gap(c1), g.gap(g.conv(g.gap(d1), 24, 1)))
    g.mark_output(y)
    desc = g.graph("cleanup")
    log("[case] graph cleanup")
    _, outs, nodes = run_gpu(desc, materialize_all=True)
    ref = oracle.run_graph(desc)
    kinds = [n["kind"] for n in __import__("paper_1907_01989_amd.engine", fromlist=["x"]).Plan(desc, bind=False).nodes()]
    assert "pad" not in kinds and "concat" not in kinds
    for t in (c1, d1):
        check_isolated(f"node {t}", nodes[t], isolated_reference(desc, t, nodes))
    ok, msg = check_layer("output", outs[0], ref[y].reshape(outs[0].shape))
    assert ok, msg


def test_pad_merged_into_stem_and_standalone_pad():
    g = NetBuilder(seed=11)
    x = g.input(1, 34, 34, 3, 0, 1, dtype=workloads.DTYPE_FP16)
    st = g.conv(g.pad(x, (0, 1, 0, 1)), 32, 3, s=2, pads=(0, 0, 0, 0))
    xs = sliced(g, g.input(2, 5, 6, 12, -1, 1, name="input2"))
    q = g.add(g.pad(xs, (1, 2, 0, 3)), g.pad(xs, (2, 1, 3, 0)), act=ACT_RELU)
    g.mark_output(st)
    g.mark_output(q)
    desc = g.graph("pads")
    log("[case] pad into stem + standalone pads")
    _, outs, nodes = run_gpu(desc, materialize_all=True)
    ref = oracle.run_graph(desc)
    check_isolated("stem", nodes[st], ref[st])
    check_isolated("pad add", nodes[q], ref[q])
    check_isolated("pad add out", outs[1], ref[q].reshape(outs[1].shape))


def test_greedy_and_materialized_runs_agree():
    desc = workloads.mobilenet_v2(2)
    log("[case] v2 b2 greedy vs naive arena")
    _, outs_a, _ = run_gpu(desc, materialize_all=False)
    _, outs_b, _ = run_gpu(desc, materialize_all=True)
    for a, b in zip(outs_a, outs_b):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("net,batch", [("mobilenet_v2", 2), ("deeplab", 1)])
def test_mcfp_arena_runs_agree_with_greedy(net, batch):
    # the minimum-cost-flow plan places tensors differently (Sec. 5); the
    # kernels and their inputs are the same, so the outputs are bit-identical
    from paper_1907_01989_amd import _binding as B
    desc = workloads.WORKLOADS[net](batch)
    log(f"[case] {net} b{batch} mcfp vs greedy arena")
    plan_m, outs_m, _ = run_gpu(desc, materialize_all=False, planner=B.PLANNER_MCFP)
    plan_g, outs_g, _ = run_gpu(desc, materialize_all=False, planner=B.PLANNER_GREEDY)
    assert plan_m.memory_report()[1] != plan_g.memory_report()[1]
    for a, b in zip(outs_m, outs_g):
        np.testing.assert_array_equal(a, b)


CONV_RING_CASES = [
    # n, h, w, cin, cout, k, s, d, pads, fuse-residual: every tile of the window GEMM's ring
    (1, 33, 33, 64, 64, 3, 1, 1, None, False),       # one tap per stage
    (2, 19, 17, 32, 72, 3, 2, 1, None, True),        # 4 slices: one tap per 4-slice stage, two per 8-slice stage
    (3, 9, 9, 24, 136, 3, 1, 2, None, False),        # taps change inside a stage, dilation 2
    (70, 3, 3, 8, 16, 3, 1, 1, None, False),         # one slice per tap, many images per tile
    (1, 130, 3, 128, 40, 3, 1, 1, (1, 1, 0, 2), False),   # taps wholly outside for some columns
    (1, 1, 1, 64, 32, 5, 1, 1, (2, 2, 2, 2), False),  # a single pixel, 24 of 25 taps outside
    (1, 12, 12, 16, 24, 6, 1, 1, (2, 3, 2, 3), False),   # more taps than the ring's mask holds
    (4, 16, 16, 40, 48, 1, 2, 1, (0, 0, 0, 0), False),   # strided 1x1
]


@pytest.mark.parametrize("n,h,w,cin,cout,k,s,d,pads,res", CONV_RING_CASES)
@pytest.mark.parametrize("dtype", [0, 1])
def test_conv_window_every_configuration(n, h, w, cin, cout, k, s, d, pads, res, dtype):
    from paper_1907_01989_amd import engine, _binding as B
    g = NetBuilder(seed=k * 100 + cin + cout)
    x = sliced(g, g.input(n, h, w, cin, -1, 1))
    y = g.conv(x, cout, k, s, d, act=ACT_NONE if res else ACT_RELU6, pads=pads)
    if res:
        oh, ow, _ = g.hwc(y)
        y = g.add(y, sliced(g, g.input(n, oh, ow, cout, -2, 2)), act=ACT_RELU)
    g.mark_output(y)
    desc = g.graph(f"ring_{n}x{h}x{w}x{cin}->{cout}_k{k}s{s}d{d}")
    if dtype:
        desc = workloads.as_bf16_graph(desc)
    ref = oracle.run_graph(desc)[y]
    plan = engine.Plan(desc, bind=False, dtype=dtype)
    i = [m["kind"] for m in plan.nodes()].index("conv_igemm")
    first = None
    for c in range(plan.node_configs()[i][1]):
        B.mgi_plan_set_node_config(plan.handle, i, c)
        log(f"[case] {desc['name']} dtype {dtype} {plan.node_configs()[i][2]}")
        _, outs, _ = run_gpu(desc, materialize_all=False, dtype=dtype, configs={i: c})
        if first is None:
            first = outs[0]
            check_isolated("conv", first, ref.reshape(first.shape), rtol=ISO_RTOL_BF16 if dtype else ISO_RTOL)
        np.testing.assert_array_equal(outs[0], first)


DW_INPUT_CASES = [
    # n, h, w, c, k, s, d: depthwise convolutions that read the NHWC graph input
    (1, 56, 56, 128, 3, 1, 1),
    (2, 9, 7, 8, 3, 1, 1),            # one slice
    (3, 13, 11, 24, 3, 2, 1),         # three slices (lanes past the last one)
    (1, 5, 6, 72, 3, 1, 2),           # nine slices, dilation 2
    (2, 17, 15, 40, 3, 2, 2),
    (1, 1, 1, 64, 3, 1, 1),
    (2, 10, 9, 104, 5, 1, 1),
    (5, 11, 14, 16, 5, 2, 1),
    (1, 3, 3, 48, 5, 1, 1),           # a plane smaller than the window
]


@pytest.mark.parametrize("n,h,w,c,k,s,d", DW_INPUT_CASES)
@pytest.mark.parametrize("src,dtype", [(0, 0), (2, 0), (0, 1), (2, 1)])
def test_depthwise_reads_the_graph_input(n, h, w, c, k, s, d, src, dtype):
    """In every configuration, aligned (the kernel reads the input itself) and
    not (the conversion kernel runs first): the oracle's result, and bit for
    bit that of a plan that keeps the converted tensor."""
    import torch
    from paper_1907_01989_amd import engine, _binding as B
    g = NetBuilder(seed=c + h)
    y = g.dw(g.input(n, h, w, c, -1, 1, dtype=src), k, s, d, act=ACT_RELU6)
    g.mark_output(y)
    desc = g.graph(f"dwin_{n}x{h}x{w}x{c}_k{k}s{s}d{d}")
    if dtype:
        desc = workloads.as_bf16_graph(desc)
    log(f"[case] {desc['name']} src {src} store {dtype}")
    ref = oracle.run_graph(desc)[y]
    _, kept, _ = run_gpu(desc, materialize_all=True, dtype=dtype)
    check_isolated("dw", kept[0], ref.reshape(kept[0].shape), rtol=ISO_RTOL_BF16 if dtype else ISO_RTOL)
    plan = engine.Plan(desc, dtype=dtype)
    i = [m["kind"] for m in plan.nodes()].index("dw_conv")
    x = plan.input_tensors()[0]
    for cfg in range(plan.node_configs()[i][1]):
        B.mgi_plan_set_node_config(plan.handle, i, cfg)
        for off in (0, 1):
            xb = torch.empty(x.numel() + off, dtype=x.dtype, device=x.device)
            xo = xb[off:].view(x.shape)
            xo.copy_(x)
            out = plan.run([xo])[0]
            torch.cuda.synchronize()
            np.testing.assert_array_equal(out.cpu().numpy(), kept[0], err_msg=f"config {cfg} offset {off}")


@pytest.mark.parametrize("n,h,w,c,oh,ow,align", [
    (1, 9, 11, 5, 70, 90, True),          # one row per thread
    (2, 13, 9, 21, 390, 345, True),       # two, an even number of rows
    (3, 12, 20, 9, 431, 421, False),      # four, a remainder; rows that share no source row at the end
    (1, 700, 30, 8, 701, 760, True),      # hardly any upsampling: no two rows share a source row
])
def test_resize_argmax_rows(n, h, w, c, oh, ow, align):
    g = NetBuilder(seed=n + c)
    x = sliced(g, g.input(n, h, w, c, -1, 1))
    up = g.resize(x, oh, ow, align)
    y = g.argmax(up)
    g.mark_output(y)
    desc = g.graph("resize_argmax")
    log(f"[case] resize_argmax {n}x{h}x{w}x{c} -> {oh}x{ow}")
    _, outs, _ = run_gpu(desc)
    ref = oracle.run_graph(desc)
    # exact fp16 inputs: the interpolation differs from float64 by a few fp32
    # roundings of values up to 1, and by the coordinate's rounding (at most
    # 2^-24 * h, on slopes of at most 2)
    bad, covered, _ = labels_check(outs[0], ref[up], margin=1e-3)
    assert bad == 0 and covered > 0.9


@pytest.mark.parametrize("chans", [(16, 24, 13), (8, 8), (40, 5)])
@pytest.mark.parametrize("dtype", [0, 1])
def test_concat_operands_written_in_place(chans, dtype):
    """Operands whose producers write them into the concatenated tensor, one
    of them read elsewhere too (also after the concatenation), against a plan
    that keeps and copies every tensor; and operands that cannot be (a ragged
    one in the middle, one used twice)."""
    from paper_1907_01989_amd import engine
    g = NetBuilder(seed=sum(chans))
    x = g.input(2, 9, 7, 24, -1, 1)
    parts = [g.conv(x, c, 1 + 2 * (i % 2)) for i, c in enumerate(chans)]
    parts[0] = g.dw(parts[0], 3)
    cat = g.concat(parts)
    z = g.conv(cat, 40, 1)
    late = g.conv(g.add(parts[0], g.conv(z, chans[0], 1)), 16, 1)
    odd = g.concat([g.conv(z, 13, 1), late, late])
    for t in (z, late, parts[-1], odd):
        g.mark_output(t)
    desc = g.graph(f"concat_{chans}")
    log(f"[case] {desc['name']} dtype {dtype}")
    _, kept, _ = run_gpu(desc, materialize_all=True, dtype=dtype)
    for planner in (0, 1, 2):
        _, outs, _ = run_gpu(desc, materialize_all=False, dtype=dtype, planner=planner)
        for o, k in zip(outs, kept):
            np.testing.assert_array_equal(o, k)


@pytest.mark.parametrize("n,h,w,c,s", [
    (64, 7, 7, 104, 1), (64, 7, 6, 168, 1),      # eight slices a workgroup (the last of five), two bands and one
    (33, 14, 13, 104, 1), (20, 30, 28, 40, 1),   # two slices, a last group of one; bands of sixteen and eight rows
    (6, 40, 40, 56, 1), (1, 9, 200, 24, 1),      # bands of four rows; single slices of wide rows
    (7, 61, 33, 24, 1),                          # a last band of five rows of eight
    (30, 29, 27, 56, 2), (40, 21, 19, 72, 2),    # stride 2
])
@pytest.mark.parametrize("dtype", [0, 1])
def test_depthwise_5x5_bands(n, h, w, c, s, dtype):
    # the bands chosen by size, from the sliced tensor and from the NHWC input
    for direct in (False, True):
        g = NetBuilder(seed=c + h)
        x = g.input(n, h, w, c, -1, 1, dtype=2 if dtype else 0)
        y = g.dw(x if direct else sliced(g, x), 5, s, act=ACT_RELU6)
        g.mark_output(y)
        desc = g.graph(f"dw5_{n}x{h}x{w}x{c}_s{s}_{int(direct)}")
        if dtype:
            desc = workloads.as_bf16_graph(desc)
        log(f"[case] {desc['name']} store {dtype}")
        ref = oracle.run_graph(desc)[y]
        _, outs, _ = run_gpu(desc, materialize_all=False, dtype=dtype)
        check_isolated("dw", outs[0], ref.reshape(outs[0].shape), rtol=ISO_RTOL_BF16 if dtype else ISO_RTOL)


@pytest.mark.parametrize("n,h,w,c,s,d", [(1, 7, 5, 24, 1, 1), (1, 14, 14, 96, 1, 2), (2, 9, 8, 40, 2, 1),
                                         (3, 33, 31, 64, 1, 1), (8, 56, 56, 128, 1, 1)])
@pytest.mark.parametrize("dtype", [0, 1])
def test_depthwise_every_row_count(n, h, w, c, s, d, dtype):
    # one row per thread on small grids, four (two) and eight (four) on large
    # ones: the same bits from the sliced tensor
    from paper_1907_01989_amd import engine, _binding as B
    g = NetBuilder(seed=c + h)
    y = g.dw(sliced(g, g.input(n, h, w, c, -1, 1)), 3, s, d, act=ACT_RELU6)
    g.mark_output(y)
    desc = g.graph(f"dwrows_{n}x{h}x{w}x{c}_s{s}d{d}")
    if dtype:
        desc = workloads.as_bf16_graph(desc)
    ref = oracle.run_graph(desc)[y]
    plan = engine.Plan(desc, bind=False, dtype=dtype)
    i = [m["kind"] for m in plan.nodes()].index("dw_conv")
    outs, names = [], []
    for cfg in range(plan.node_configs()[i][1]):
        B.mgi_plan_set_node_config(plan.handle, i, cfg)
        names.append(plan.node_configs()[i][2])
        _, o, _ = run_gpu(desc, materialize_all=False, dtype=dtype, configs={i: cfg})
        outs.append(o[0])
    log(f"[case] {desc['name']} dtype {dtype} {names}")
    assert ("rows1" in names) == (s == 2 or n * h < 200) and len(set(names)) == 3
    check_isolated("dw", outs[0], ref.reshape(outs[0].shape), rtol=ISO_RTOL_BF16 if dtype else ISO_RTOL)
    for o in outs[1:]:
        np.testing.assert_array_equal(o, outs[0])


@pytest.mark.parametrize("n,h,w,cin,cout", [(1, 7, 7, 776, 24), (3, 33, 31, 792, 24), (16, 28, 28, 872, 40), (2, 9, 9, 779, 16),
                                            (1, 1, 1, 1000, 48)])
@pytest.mark.parametrize("src,dtype", [(workloads.DTYPE_FP16, 0), (workloads.DTYPE_FP32, 0), (workloads.DTYPE_FP16, 1)])
def test_infinity_beside_the_k_tail(n, h, w, cin, cout, src, dtype):
    """Narrow pointwise products with K above 768 and not whole steps of 32: an
    infinity in the last real K slice meets that slice's weights only, not the
    zero weights of the padding behind it (the default configuration; finite
    inputs in every one, bit for bit)."""
    import torch
    from paper_1907_01989_amd import engine, _binding as B
    g = NetBuilder(seed=cin)
    t = g.conv(g.input(n, h, w, cin, 0.0, 1.0, dtype=src), cout, 1, act=ACT_NONE)
    g.mark_output(t)
    desc = g.graph("tail")
    plan = engine.Plan(desc, dtype=dtype)
    x = plan.input_tensors()[0]
    node = [i for i, k in enumerate(plan.nodes()) if k["kind"] == "pw_gemm"][0]
    first = None
    for c in range(plan.node_configs()[node][1]):
        B.mgi_plan_set_node_config(plan.handle, node, c)
        log(f"[case] tail {n}x{h}x{w} {cin}->{cout} input {src} store {dtype} {plan.node_configs()[node][2]}")
        y = plan.run([x])[0].cpu()
        if first is None:
            first = y
            store = torch.bfloat16 if dtype else torch.float16
            wt = torch.from_numpy(desc["ops"][t]["w"].reshape(cout, cin)).to(store).float()
            ref = x.cpu().to(store).double().reshape(-1, cin) @ wt.double().t() + torch.from_numpy(desc["ops"][t]["b"]).double()
            ok, msg = check_layer("tail", y.numpy().reshape(ref.shape), ref.numpy(), ISO_RTOL_BF16 if dtype else ISO_RTOL)
            assert ok, msg
        assert torch.equal(y, first), plan.node_configs()[node][2]
    B.mgi_plan_set_node_config(plan.handle, node, 0)
    x[n - 1, h - 1, w - 1, cin - 1] = float("inf")
    y = plan.run([x])[0].cpu().reshape(-1, cout)
    assert torch.equal(y[-1], wt[:, cin - 1] * float("inf"))
    assert torch.equal(y[:-1], first.reshape(-1, cout)[:-1])
    plan.close()
