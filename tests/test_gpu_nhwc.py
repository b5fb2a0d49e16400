"""Conversions between NHWC graph I/O and the sliced layout: exact copies up to
the storage rounding, for every lane mapping (1 to 8 slices of a wave), pixel
counts on both sides of a thread's and a workgroup's share, channel counts
that end inside a slice, and buffers that start off a 16-byte boundary."""
import numpy as np
import pytest

import workloads
from workloads import ACT_NONE, NetBuilder

from gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w,c", [(1, 1, 1, 8), (1, 5, 3, 13), (2, 9, 7, 16), (1, 8, 8, 24), (3, 7, 5, 36),
                                     (1, 33, 1, 72), (2, 6, 11, 100), (5, 13, 13, 136), (4, 96, 95, 64),
                                     (16, 57, 57, 4)])
@pytest.mark.parametrize("src,dtype", [(0, 0), (2, 0), (0, 1), (2, 1)])
def test_ingest_export(n, h, w, c, src, dtype):
    import torch
    from paper_1907_01989_amd import engine
    g = NetBuilder(seed=c)
    y = g.activation(g.input(n, h, w, c, -3, 3, dtype=src), ACT_NONE)
    g.mark_output(y)
    plan = engine.Plan(g.graph("io"), dtype=dtype)
    store = torch.bfloat16 if dtype else torch.float16
    x = plan.input_tensors()[0]
    if src == 2:
        x = x * 1.0009765                   # fp32 values between the storage type's
    want = x.to(store).float()
    for off in (0, 1):
        log(f"[case] io {n}x{h}x{w}x{c} src {src} store {dtype} offset {off}")
        xb = torch.empty(x.numel() + off, dtype=x.dtype, device=x.device)
        xo = xb[off:].view(x.shape)
        xo.copy_(x)
        yb = torch.full((x.numel() + off + 64,), 7.0, dtype=torch.float32, device=x.device)
        shape = (n, c) if h == w == 1 else (n, h, w, c)
        yo = yb[off:off + x.numel()].view(shape)
        plan.run([xo], [yo])
        torch.cuda.synchronize()
        np.testing.assert_array_equal(yo.cpu().numpy().reshape(-1), want.cpu().numpy().reshape(-1))
        assert bool((yb[off + x.numel():] == 7.0).all()) and bool((yb[:off] == 7.0).all())


DIRECT_CASES = [
    # n, h, w, cin, cout, window, residual
    (1, 1, 1, 8, 5, 1, False),
    (3, 9, 7, 40, 21, 1, False),            # channel tail of a 4-channel group, ragged tiles
    (2, 13, 13, 64, 136, 1, True),          # half a channel block at the end, residual
    (5, 14, 14, 96, 64, 1, True),
    (1, 33, 33, 24, 30, 3, False),          # implicit GEMM
    (2, 9, 9, 16, 72, 3, True),
]


@pytest.mark.parametrize("n,h,w,cin,cout,k,res", DIRECT_CASES)
@pytest.mark.parametrize("dtype", [0, 1])
def test_gemm_writes_nhwc_output(n, h, w, cin, cout, k, res, dtype):
    """The GEMM kernels' own NHWC fp32 store, in every configuration, against
    the sliced store and the export kernel (a plan that keeps every tensor),
    with and without another reader of the sliced tensor; and a run whose
    output buffer is its input buffer."""
    import torch
    from paper_1907_01989_amd import engine, _binding as B

    def net(second):
        g = NetBuilder(seed=cin + cout)
        x = g.input(n, h, w, cin, -1, 1, dtype=workloads.DTYPE_FP32)
        y = g.conv(x, cout, k, act=ACT_NONE)
        if res:
            y = g.add(y, g.activation(g.conv(x, cout, 1, act=ACT_NONE), workloads.ACT_RELU), act=ACT_NONE)
        g.mark_output(y)
        if second:
            g.mark_output(g.gap(y))
        return g.graph("direct")

    for second in (False, True):
        desc = net(second)
        ref_plan = engine.Plan(desc, dtype=dtype, materialize_all=True)
        x = ref_plan.input_tensors()
        ref = ref_plan.run(x)
        plan = engine.Plan(desc, dtype=dtype)
        for i, (kind, (_, ncfg, _)) in enumerate(zip([m["kind"] for m in plan.nodes()], plan.node_configs())):
            if kind not in ("pw_gemm", "conv_igemm"):
                continue
            for c in range(ncfg):
                B.mgi_plan_set_node_config(plan.handle, i, c)
                log(f"[case] direct {n}x{h}x{w}x{cin}->{cout} k{k} res{int(res)} dtype {dtype} "
                    f"{kind} {plan.node_configs()[i][2]} readers {1 + int(second)}")
                outs = [torch.full_like(o, 9.0) for o in ref]
                plan.run(x, outs)
                torch.cuda.synchronize()
                for o, r in zip(outs, ref):
                    np.testing.assert_array_equal(o.cpu().numpy(), r.cpu().numpy())
            B.mgi_plan_set_node_config(plan.handle, i, 0)


def test_output_in_the_input_buffer():
    """Input and output may share memory, whole or in part: every input value
    is read before an output value is written."""
    import torch
    from paper_1907_01989_amd import engine
    g = NetBuilder(seed=4)
    x = g.input(2, 17, 19, 48, -1, 1, dtype=workloads.DTYPE_FP32)
    g.mark_output(g.conv(g.dw(x, 3), 48))
    plan = engine.Plan(g.graph("inplace"))
    xs = plan.input_tensors()
    want = plan.run(xs)[0].cpu().numpy()
    for shift in (0, 64):
        log(f"[case] output buffer {shift} values into the input buffer")
        buf = torch.empty(xs[0].numel() + shift, dtype=torch.float32, device="cuda")
        xi = buf[:xs[0].numel()].view(xs[0].shape)
        xi.copy_(xs[0])
        yo = buf[shift:].view(xs[0].shape)
        plan.run([xi], [yo])
        torch.cuda.synchronize()
        np.testing.assert_array_equal(yo.cpu().numpy(), want)


def _inplace_net(kind, n, h, w, c, cout):
    g = NetBuilder(seed=c + cout)
    x = g.input(n, h, w, c, -1, 1, dtype=workloads.DTYPE_FP16)
    if kind == "pw":
        y = [g.conv(x, cout, 1)]
    elif kind == "block":                       # expansion, depthwise, projection, residual from the input
        t = g.conv(g.dw(g.conv(x, cout, 1), 3), c, 1, act=ACT_NONE)
        y = [g.add(t, x)]
    elif kind == "down":
        y = [g.dw(g.conv(x, cout, 1), 3, 2)]
    elif kind == "pool":
        y = [g.gap(g.conv(x, cout, 1))]
    elif kind == "conv":
        y = [g.conv(x, cout, 3)]
    else:                                       # two readers, one of them the pool
        y = [g.conv(x, cout, 1), g.gap(x), g.dw(x, 3)]
    for t in y:
        g.mark_output(t)
    return g.graph(kind)


@pytest.mark.parametrize("kind,n,h,w,c,cout", [
    ("pw", 1, 1, 1, 8, 16), ("pw", 3, 9, 7, 40, 72), ("pw", 2, 13, 13, 264, 136), ("pw", 1, 30, 30, 512, 40),
    ("pw", 37, 14, 14, 96, 520),
    ("block", 2, 14, 14, 24, 96), ("block", 1, 7, 7, 160, 320), ("block", 3, 29, 27, 32, 48),
    ("down", 2, 15, 15, 96, 192), ("down", 1, 28, 28, 40, 64),
    ("pool", 5, 7, 7, 320, 136), ("pool", 70, 3, 3, 72, 64), ("pool", 33, 7, 7, 512, 512),
    ("conv", 2, 12, 11, 32, 40), ("conv", 1, 9, 9, 64, 136), ("conv", 3, 5, 5, 24, 16),
    ("two", 2, 11, 10, 48, 24), ("two", 9, 7, 7, 16, 64),
])
def test_kernels_read_the_input_in_place(kind, n, h, w, c, cout):
    """Every configuration of every node that can read an NHWC fp16 input,
    against a plan that keeps the converted tensor; and an input off a 16-byte
    boundary, which is converted first."""
    import torch
    from paper_1907_01989_amd import engine, _binding as B
    desc = _inplace_net(kind, n, h, w, c, cout)
    ref_plan = engine.Plan(desc, materialize_all=True, fuse_pwdw=2, fuse_pool=2)
    x = ref_plan.input_tensors()[0]
    ref = ref_plan.run([x])
    plan = engine.Plan(desc, fuse_pwdw=2, fuse_pool=2)
    for i, (m, (_, ncfg, _)) in enumerate(zip(plan.nodes(), plan.node_configs())):
        for cfg in range(ncfg if ncfg > 1 or i == 0 else 0):
            B.mgi_plan_set_node_config(plan.handle, i, cfg)
            log(f"[case] in place {kind} {n}x{h}x{w}x{c}->{cout} node {i} {m['kind']} {plan.node_configs()[i][2]}")
            for off in (0, 1):
                xb = torch.empty(x.numel() + off, dtype=x.dtype, device=x.device)
                xo = xb[off:].view(x.shape)
                xo.copy_(x)
                outs = [torch.full_like(o, 9.0) for o in ref]
                plan.run([xo], outs)
                torch.cuda.synchronize()
                for o, r in zip(outs, ref):
                    np.testing.assert_array_equal(o.cpu().numpy(), r.cpu().numpy())
        B.mgi_plan_set_node_config(plan.handle, i, 0)


@pytest.mark.parametrize("kind,src,dtype", [("dw3", 0, 0), ("dw3", 2, 1), ("dw5", 2, 0), ("pw", 0, 0), ("conv", 0, 0)])
def test_tensors_not_written(kind, src, dtype):
    """What the workspace holds after a run tells which tensors were stored: with
    the input read in place and the output written by the GEMM, only the one
    between them; with an input off 16 bytes its converted form too; with an
    output over the input also the GEMM's sliced result."""
    import torch
    from paper_1907_01989_amd import engine, _binding as B
    n, h, w, c, cout = 2, 12, 11, 64, 48
    g = NetBuilder(seed=6)
    t = x = g.input(n, h, w, c, 0.5, 1.0, dtype=src)
    if kind in ("dw3", "dw5"):
        t = g.dw(t, int(kind[2]))
    elif kind == "conv":
        t = g.conv(t, c, 3)
    else:
        t = g.conv(t, c, 1)
    g.mark_output(g.conv(t, cout, 1))
    plan = engine.Plan(g.graph("stored"), planner=B.PLANNER_NAIVE, dtype=dtype)
    x = plan.input_tensors()[0]
    elems = n * h * w * np.array([c // 8, c // 8, cout // 8])        # converted input, middle, sliced output
    both = torch.empty(x.numel() * 2 + 4096, dtype=x.dtype, device=x.device)

    def stored(xo, yo):
        plan.ws.fill_(0xa5)                     # a small negative number in fp16 and bf16: no ReLU6 output
        plan.run([xo], [yo])
        torch.cuda.synchronize()
        base = plan._ws_ptr - plan.ws.data_ptr()
        words = plan.ws[base:base + plan.workspace_bytes // 16 * 16].view(-1, 16)
        return int((words != 0xa5).any(1).sum())

    want = plan.alloc_outputs()[0]
    log(f"[case] stored tensors {kind} src {src} store {dtype}")
    assert stored(x, want) == elems[1]
    off = torch.empty(x.numel() + 1, dtype=x.dtype, device=x.device)[1:].view(x.shape)
    off.copy_(x)
    y = torch.empty_like(want)
    assert stored(off, y) == elems[0] + elems[1]
    assert torch.equal(y, want)
    xo = both[:x.numel()].view(x.shape)
    xo.copy_(x)
    yo = both.view(torch.float32)[:want.numel()].view(want.shape)
    assert stored(xo, yo) == elems.sum()
    assert torch.equal(yo, want)
    plan.close()
