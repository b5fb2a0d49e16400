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
