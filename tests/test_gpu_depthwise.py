"""GPU tests of the depthwise kernels against the float64 oracle."""
import numpy as np
import pytest
import torch

from paper_1907_11210_amd import huge2 as h2
from paper_1907_11210_amd import workloads as wl
from paper_1907_11210_amd.workloads import Layer

import parity as P

pytestmark = pytest.mark.gpu


def L(name, tr, n, ci, h, w, co, k, st, pd, op, dl, layout, dtype):
    return Layer(name, tr, n, ci, h, w, co, k, k, st, pd, op, dl, layout, dtype, "none", ci)


LAYERS = [
    # 3x3 conv, chains of rows: a chain cut by the last row, one-row and one-column planes
    L("dw3_d1", False, 2, 16, 9, 7, 16, 3, 1, 1, 0, 1, "NHWC", "bf16"),
    L("dw3_d4_short", False, 1, 8, 5, 33, 8, 3, 1, 4, 0, 4, "NHWC", "bf16"),
    L("dw3_row", False, 3, 24, 1, 6, 24, 3, 1, 1, 0, 1, "NHWC", "bf16"),
    L("dw3_column", False, 1, 12, 17, 1, 12, 3, 1, 2, 0, 2, "NHWC", "f32"),
    L("dw3_s2", False, 2, 8, 18, 15, 8, 3, 2, 1, 0, 1, "NHWC", "bf16"),
    L("dw3_s2_d3", False, 1, 4, 20, 19, 4, 3, 2, 3, 0, 3, "NHWC", "f32"),
    L("dw3_s2_d2", False, 1, 6, 13, 14, 6, 3, 2, 2, 0, 2, "NCHW", "f32"),
    L("dw3_odd_channels", False, 2, 13, 10, 11, 13, 3, 1, 2, 0, 2, "NHWC", "bf16"),
    L("dw3_nchw", False, 2, 5, 19, 21, 5, 3, 1, 6, 0, 6, "NCHW", "bf16"),
    L("dw3_mult2", False, 1, 6, 9, 8, 12, 3, 1, 1, 0, 1, "NHWC", "bf16"),
    L("dw3_no_pad", False, 1, 8, 12, 12, 8, 3, 1, 0, 0, 3, "NHWC", "bf16"),
    # any size and stride, conv and transposed
    L("dw_s3", False, 1, 8, 14, 13, 8, 3, 3, 1, 0, 1, "NHWC", "f32"),
    L("dw_5x5", False, 2, 16, 9, 9, 16, 5, 1, 4, 0, 2, "NHWC", "bf16"),
    L("dwt_4x4", True, 2, 16, 6, 5, 16, 4, 2, 1, 0, 1, "NHWC", "bf16"),
    L("dwt_nchw_op", True, 1, 7, 4, 9, 7, 3, 2, 1, 1, 1, "NCHW", "bf16"),
    L("dwt_s3_d2", True, 1, 4, 5, 6, 8, 4, 3, 2, 2, 2, "NCHW", "f32"),
    L("dwt_s4_d2_zero_taps", True, 1, 8, 3, 4, 8, 3, 4, 1, 2, 2, "NHWC", "f32"),
    L("dwt_k2_s3_zero_taps", True, 1, 8, 4, 4, 8, 2, 3, 0, 2, 1, "NHWC", "bf16"),
]


def _inputs(layer, seed):
    dt = wl.torch_dtype(layer.dtype)
    return (wl.layer_input(layer, seed).to(dt), wl.random_weight(layer, seed + 1, 0.5).to(dt))


@pytest.mark.parametrize("chains", ["0", "1"])
@pytest.mark.parametrize("layer", LAYERS, ids=lambda l: l.name)
def test_depthwise_forms(layer, chains, monkeypatch):
    """Every dispatch of the depthwise kernels (3x3 row chains or any taps;
    16-byte channel pieces or one channel per thread) with bias and ReLU."""
    monkeypatch.setenv("HUGE2_DEPTHWISE_CHAINS", chains)
    layer = layer.with_(act="relu")
    P.say("case", layer)
    xq, wq = _inputs(layer, 7)
    bias = torch.linspace(-0.5, 0.5, layer.c_out)
    ref = P.oracle_full(layer, xq, wq, bias)
    absref = P.oracle_full(layer, xq, wq, bias, absolute=True)
    P.check(P.run_gpu(layer, xq, wq, bias, prefill_nan=True), ref, absref, layer.dtype, layer.name)
    plan = P.make_plan(layer, wq.contiguous().to(torch.device("cuda", 0)))
    try:
        rows3 = chains == "1" and layer.name.startswith("dw3")
        assert ("depthwise3" if rows3 else "depthwise ") in plan.kernel, plan.kernel
    finally:
        plan.close()


@pytest.mark.parametrize("layer,chains", [
    (L("dw_small", False, 3, 64, 52, 37, 64, 3, 2, 0, 0, 1, "NHWC", "bf16"), False),
    (L("dw_under", False, 4, 128, 64, 63, 128, 3, 1, 1, 0, 1, "NHWC", "bf16"), False),
    (L("dw_over", False, 8, 128, 64, 64, 128, 3, 1, 1, 0, 4, "NHWC", "f32"), True),
    (L("dw_under_one", False, 1, 63, 64, 64, 63, 3, 1, 1, 0, 1, "NCHW", "f32"), False),
    (L("dw_under_s2", False, 2, 128, 63, 63, 128, 3, 2, 1, 0, 1, "NCHW", "bf16"), False),
    (L("dw_over_one", False, 2, 128, 50, 50, 128, 3, 1, 1, 0, 1, "NCHW", "bf16"), True),
], ids=lambda v: getattr(v, "name", None))
def test_chains_by_size(layer, chains, monkeypatch):
    """Row chains where there are enough of them for the chip; the same bits
    either way."""
    P.say("case", layer)
    xq, wq = _inputs(layer, 11)
    def run():
        plan = P.make_plan(layer, wq.contiguous().to(torch.device("cuda", 0)))
        try:
            return plan.kernel, P.run_gpu(layer, xq, wq, plan=plan)
        finally:
            plan.close()
    kernel, y = run()
    assert ("depthwise3" in kernel) == chains, kernel
    monkeypatch.setenv("HUGE2_DEPTHWISE_CHAINS", "0" if chains else "1")
    kernel, other = run()
    assert ("depthwise3" in kernel) != chains, kernel
    assert np.array_equal(y, other)


@pytest.mark.parametrize("layer", [l for l in LAYERS if l.layout == "NHWC"][:5],
                         ids=lambda l: l.name)
def test_depthwise_unaligned(layer, monkeypatch):
    """Tensors that do not start on 16 bytes take one channel per thread and
    give the same bits: the taps are added in the same order."""
    P.say("case", layer)
    monkeypatch.setenv("HUGE2_DEPTHWISE_CHAINS", "1")
    dev = torch.device("cuda", 0)
    xq, wq = _inputs(layer, 9)
    x, w = wl.to_layout(xq, layer.layout).to(dev), wq.contiguous().to(dev)
    plan = P.make_plan(layer, w)
    try:
        y = plan(x)
        big = torch.zeros(x.numel() + 1, dtype=x.dtype, device=dev)
        big[1:] = x.flatten()
        out = torch.full((y.numel() + 1,), 7.0, dtype=y.dtype, device=dev)
        h2.huge2_plan_execute(plan._plan, big[1:].data_ptr(), 0, out[1:].data_ptr(),
                              torch.cuda.current_stream(dev).cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(out[1:].view(y.shape), y) and out[0].item() == 7.0
    finally:
        plan.close()


@pytest.mark.parametrize("chains", ["0", "1"])
@pytest.mark.parametrize("layout", ["NCHW", "NHWC"])
def test_depthwise_skips_padding(layout, chains, monkeypatch):
    """Products outside the input are skipped: an infinite weight whose tap
    lies in the padding leaves the outputs there finite."""
    monkeypatch.setenv("HUGE2_DEPTHWISE_CHAINS", chains)
    dev = torch.device("cuda", 0)
    layer = L("dw_inf", False, 1, 8, 6, 6, 8, 3, 1, 1, 0, 1, layout, "bf16")
    w = torch.full((8, 1, 3, 3), 0.25, dtype=torch.bfloat16)
    w[:, :, 0, 0] = float("inf")
    x = torch.ones(1, 8, 6, 6, dtype=torch.bfloat16)
    y = wl.from_layout(P.make_plan(layer, w.to(dev))(wl.to_layout(x, layout).to(dev)), layout)
    finite = torch.isfinite(y.float().cpu())
    want = torch.zeros(6, 6, dtype=torch.bool)
    want[0, :] = want[:, 0] = True
    assert bool((finite == want).all())
    assert np.isclose(y[0, 0, 0, 0].item(), 1.0)
