"""GPU tests of the wave-K form and of fp32 on the bf16 matrix cores."""
import time

import numpy as np
import pytest
import torch

from paper_1907_11210_amd import huge2 as h2
from paper_1907_11210_amd import workloads as wl
from paper_1907_11210_amd.workloads import Layer

import parity as P

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def L(name, tr, n, ci, h, w, co, k, st, pd, op, dl, layout, dtype):
    return Layer(name, tr, n, ci, h, w, co, k, k, st, pd, op, dl, layout, dtype)


# (layer, kernel): both sides of the rules' lines, ragged tiles and K tails
FORMS = [
    # one stage and one tile; fewer stages than waves; a stage more than eight
    (L("wk_1x1", False, 1, 8, 3, 5, 8, 1, 1, 0, 0, 1, "NHWC", "bf16"), "wavek_kernel 64x32"),
    (L("wk_7_stages", False, 1, 7 * 64, 4, 4, 40, 1, 1, 0, 0, 1, "NHWC", "bf16"), "wavek_kernel 64x32"),
    (L("wk_9_stages", False, 2, 70, 9, 9, 65, 3, 1, 1, 0, 1, "NCHW", "bf16"), "wavek_kernel 64x32"),
    (L("wk_listed_100", False, 1, 100, 17, 19, 33, 3, 1, 5, 0, 5, "NCHW", "bf16"), "wavek_kernel 64x32"),
    (L("wk_wide", False, 1, 520, 13, 11, 66, 3, 1, 2, 0, 2, "NHWC", "bf16"), "wavek_kernel 64x32"),
    (L("wk_wide_staged", False, 1, 710, 13, 11, 66, 3, 1, 2, 0, 2, "NCHW", "bf16"), "phase_gemm2"),
    (L("wk_ct_staged", True, 3, 1030, 7, 7, 72, 4, 2, 1, 0, 1, "NCHW", "bf16"), "wavek_kernel 64x32"),
    (L("wk_ct_nhwc", True, 3, 128, 8, 8, 72, 4, 2, 1, 0, 1, "NHWC", "bf16"), "wavek_kernel 64x32"),
    (L("quad_nhwc", True, 40, 64, 8, 8, 264, 4, 2, 1, 0, 1, "NHWC", "bf16"), "quad_kernel"),
    # the all-taps form's output rows: the fewest that fit, more, two to a compute unit
    (L("z_2_rows", True, 3, 24, 9, 10, 3, 4, 2, 1, 0, 1, "NCHW", "bf16"), "ztile_kernel ob2"),
    (L("z_4_rows", True, 20, 16, 16, 18, 3, 4, 2, 1, 0, 1, "NHWC", "bf16"), "ztile_kernel ob4"),
    (L("z_many", True, 260, 8, 6, 6, 3, 4, 2, 1, 0, 1, "NCHW", "bf16"), "ztile_kernel ob"),
    (L("wk_wide_tiles", False, 6, 264, 33, 33, 70, 3, 1, 2, 0, 2, "NHWC", "bf16"), "wavek_kernel 64x64"),
    (L("wk_f32", True, 1, 37, 5, 7, 21, 4, 2, 1, 0, 1, "NCHW", "f32"), "wavek_kernel 64x32"),
    (L("wk_f32_64", True, 9, 40, 14, 12, 100, 5, 2, 2, 1, 1, "NHWC", "f32"), "wavek_kernel 64x64"),
    (L("wk_no_taps", True, 1, 16, 4, 5, 24, 2, 3, 0, 2, 1, "NHWC", "f32"), "wavek_kernel"),
    (L("f32_128x64", False, 3, 20, 81, 75, 50, 3, 1, 2, 0, 2, "NCHW", "f32"), "f32_kernel 128x64"),
    (L("f32_128x32", True, 3, 10, 61, 59, 9, 3, 2, 1, 1, 1, "NHWC", "f32"), "f32_kernel 128x32"),
    (L("f32_64x128", True, 5, 165, 29, 31, 130, 4, 2, 1, 0, 1, "NCHW", "f32"), "f32_kernel 64x128"),
    (L("f32_128x128", True, 8, 20, 41, 43, 150, 3, 2, 1, 1, 1, "NHWC", "f32"), "f32_kernel 128x128"),
    # a K split across workgroups, more taps than the wave-K form holds
    (L("f32_splitk", False, 1, 600, 9, 9, 70, 3, 1, 1, 0, 1, "NCHW", "f32"), "f32_kernel 64x128"),
    # few tiles: K too long for the wave-K form, with and without enough channel
    # blocks to split it by, on both sides of 128 tiles; many tiles of a short K
    (L("f32_long_k", True, 5, 912, 17, 6, 8, 5, 2, 2, 1, 1, "NHWC", "f32"), "f32_kernel 128x32"),
    (L("f32_long_k64", False, 2, 330, 9, 7, 40, 4, 1, 1, 0, 1, "NCHW", "f32"), "f32_kernel 128x64"),
    (L("wk_f32_few_blocks", False, 2, 84, 18, 7, 14, 5, 2, 0, 0, 1, "NHWC", "f32"), "wavek_kernel 64x32"),
    (L("wk_f32_128_tiles", False, 2, 230, 65, 64, 9, 3, 1, 1, 0, 1, "NHWC", "f32"), "wavek_kernel 64x32"),
    (L("f32_short_k", True, 5, 16, 8, 29, 200, 4, 2, 1, 0, 1, "NCHW", "f32"), "f32_kernel 128x64"),
    # many tiles of a short K: the fp32 MFMA tiles
    (L("f32_mfma_narrow", True, 9, 20, 60, 41, 12, 3, 2, 1, 1, 1, "NHWC", "f32"), "phase_gemm_kernel 128x32"),
    (L("f32_mfma_narrow_nchw", False, 17, 70, 71, 69, 30, 1, 1, 0, 0, 1, "NCHW", "f32"), "phase_gemm_kernel 128x32"),
    (L("f32_mfma_one_stage", True, 4, 20, 44, 45, 140, 2, 2, 0, 0, 1, "NCHW", "f32"), "phase_gemm_kernel 128x128"),
    (L("f32_9x9", False, 1, 20, 21, 22, 40, 9, 1, 4, 0, 1, "NHWC", "f32"), "f32_kernel 128x64"),
]


def _inputs(layer, seed):
    dt = wl.torch_dtype(layer.dtype)
    return (wl.layer_input(layer, seed).to(dt), wl.random_weight(layer, seed + 1, 0.1).to(dt))


@pytest.mark.parametrize("layer,kernel", FORMS, ids=lambda v: getattr(v, "name", None))
def test_forms(layer, kernel):
    """Each form the size rules pick matches the oracle with bias and ReLU,
    writes every output and repeats bit for bit."""
    layer = layer.with_(act="relu")
    P.say("case", layer)
    xq, wq = _inputs(layer, 3)
    bias = torch.linspace(-0.5, 0.5, layer.c_out)
    ref = P.oracle_full(layer, xq, wq, bias)
    absref = P.oracle_full(layer, xq, wq, bias, absolute=True)
    y = P.run_gpu(layer, xq, wq, bias, prefill_nan=True)
    P.check(y, ref, absref, layer.dtype, layer.name)
    assert np.array_equal(y, P.run_gpu(layer, xq, wq, bias))
    if layer.dtype == "f32":
        # the parts hold all 24 bits and 2^-25 of a product is left out: the
        # sums in fp32 are what is left, within 2^-24 of the largest partial
        # sum per addition, random over at most 5400 of them
        assert np.all(np.abs(y - ref) <= 75 * 2.0 ** -24 * absref + 1e-30)
    plan = P.make_plan(layer, wq.to(DEV))
    try:
        assert kernel in plan.kernel, plan.kernel
    finally:
        plan.close()


@pytest.mark.parametrize("n,c_in,c_out,layout", [(64, 100, 1024, "NCHW"), (64, 128, 40, "NHWC"),
                                                 (7, 65, 300, "NCHW"), (33, 64, 96, "NHWC")])
def test_two_stages_keep_the_order_of_one_sum(n, c_in, c_out, layout, monkeypatch):
    """A projection of at most 128 channels gives the bits of the 32 x 256
    tile, whose workgroup sums all channels in one accumulator."""
    layer = L("proj", True, n, c_in, 1, 1, c_out, 4, 1, 0, 0, 1, layout, "bf16")
    P.say("case", layer)
    x, w = _inputs(layer, 17)
    def run():
        plan = P.make_plan(layer, w.to(DEV))
        try:
            return plan.kernel, P.run_gpu(layer, x, w, plan=plan)
        finally:
            plan.close()
    kernel, y = run()
    assert "wavek_kernel" in kernel
    monkeypatch.setenv("HUGE2_TILE", "5")
    kernel, want = run()
    assert " 32x256 " in kernel
    assert np.array_equal(y, want)


def test_projection_plan_in_time(monkeypatch):
    """A plan of 512 equal works is laid out about as fast as one of 64: a
    program with new weights pays for it."""
    layer = L("proj", True, 1, 100, 1, 1, 1024, 4, 1, 0, 0, 1, "NCHW", "bf16")
    P.say("case", layer)
    w = torch.zeros(100, 1024, 4, 4, dtype=torch.bfloat16, device=DEV)

    def us():
        t = []
        for _ in range(40):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            plan = P.make_plan(layer, w)
            t.append(time.perf_counter() - t0)
            plan.close()
        return sorted(t)[len(t) // 2] * 1e6
    us()
    many = us()
    monkeypatch.setenv("HUGE2_TILE", "5")
    few = us()
    P.say("us", many, few)
    assert many <= 1.8 * few  # (2.0 to 2.3 where each of them was placed by a scan)


F32 = [l for l, _ in FORMS if l.name in ("wk_f32", "f32_128x64", "f32_64x128", "f32_splitk")]


def _run(layer, x, w):
    return P.run_gpu(layer, x, w).astype(np.float64)


@pytest.mark.parametrize("layer", F32, ids=lambda l: l.name)
def test_fp32_non_finite(layer):
    """Infinities and NaN in x, and values that round to infinity in bf16,
    give what fp32 arithmetic gives: infinite operands have no finite parts,
    so these sums are formed again in fp32."""
    P.say("case", layer)
    x, w = _inputs(layer, 5)
    x, w = x.abs() + 0.1, w.abs() + 0.1  # one sign: the expected sums are known
    big = 3.4e38
    x[0, 1, 0, 0] = float("inf")
    x[0, 2, -1, -1] = float("nan")
    x[0, 0, 1, 1] = big
    w.view(-1)[:] *= 1e-3
    torch_f = torch.nn.functional
    xd, wd = x.double(), w.double()
    ref = (torch_f.conv_transpose2d(xd, wd, None, layer.stride, layer.pad, layer.out_pad)
           if layer.transposed else
           torch_f.conv2d(xd, wd, None, layer.stride, layer.pad, layer.dil)).numpy()
    y = _run(layer, x, w)
    assert np.array_equal(np.isnan(y), np.isnan(ref))
    assert np.array_equal(np.isinf(y), np.isinf(ref))
    fin = np.isfinite(ref)
    assert np.any(fin & (np.abs(ref) > 1e33))
    # (the oracle has no infinities to work with: a relative bound instead)
    assert np.all(np.abs(y[fin] - ref[fin]) <= 75 * 2.0 ** -24 * np.abs(ref[fin]))


@pytest.mark.parametrize("layer", [l for l, _ in FORMS if l.dtype == "f32"], ids=lambda l: l.name)
def test_fp32_formed_again(layer):
    """Sums beyond the scaled parts' range, every one of every fp32 tile, are
    fp32 sums all the same; an infinite and a NaN weight meet only the outputs
    that read them inside the input, on each of them."""
    P.say("case", layer)
    x, w = _inputs(layer, 19)
    x, w = x * 1e28, w.abs() + 0.1
    ref = P.oracle_full(layer, x, w)
    absref = P.oracle_full(layer, x, w, absolute=True)
    y = _run(layer, x, w)
    assert np.all(np.abs(y - ref) <= 75 * 2.0 ** -24 * absref)
    x = x.abs() + 1e-3
    for k, bad in ((0, float("inf")), (min(layer.c_out, 70) - 1, float("nan"))):
        w[(1, k) if layer.transposed else (k, 1)][-1, 0] = bad
    hit = torch.zeros_like(w)
    hit[~torch.isfinite(w)] = 1
    hit = P.oracle_full(layer, torch.ones_like(x), hit) > 0
    got = _run(layer, x, w)
    assert np.array_equal(~np.isfinite(got), hit)
    assert np.isposinf(got[:, 0][hit[:, 0]]).all()
    assert np.isnan(got[:, min(layer.c_out, 70) - 1][hit[:, min(layer.c_out, 70) - 1]]).all()


def _us(f):
    f()
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    a.record()
    for _ in range(4):
        f()
    b.record()
    torch.cuda.synchronize()
    return a.elapsed_time(b) * 250


@pytest.mark.parametrize("fill", [float("nan"), float("inf"), 1e30])
@pytest.mark.parametrize("n,c_in,hw,c_out", [(64, 512, 8, 256), (9, 264, 40, 40), (9, 128, 40, 24)])
def test_fp32_formed_again_in_time(n, c_in, hw, c_out, fill):
    """A layer all of whose sums are formed again takes about four times as
    long (64 x 128, 128 x 64 and wave-K tiles), not hundreds of times."""
    x = torch.randn(n, c_in, hw, hw, device=DEV)
    w = torch.rand(c_in, c_out, 4, 4, device=DEV) + 0.1
    bad = torch.full_like(x, fill)
    plan = h2.Plan(w, x.shape, True, 2, 1)
    try:
        y = plan(x)
        usual, redone = _us(lambda: plan(x, None, y)), _us(lambda: plan(bad, None, y))
        assert torch.isnan(y).all() if fill != fill else (y > 1e30).all()
        P.say("us", plan.kernel, usual, redone)
        assert redone <= 12 * usual
    finally:
        plan.close()


@pytest.mark.parametrize("layer", F32, ids=lambda l: l.name)
def test_fp32_infinite_weight(layer):
    x, w = _inputs(layer, 7)
    x = x.abs() + 0.1
    w = w.abs()
    w[1, 0, 0, 0] = float("inf")
    w[0, 1, -1, -1] = -float("inf")
    y = _run(layer, x, w)
    co = 0 if layer.transposed else 1
    out = y[:, [co, 1 - co]] if layer.transposed else y[:, [1, 0]]
    assert np.any(np.isposinf(out[:, 0])) and np.any(np.isneginf(out[:, 1]))
    assert not np.isnan(out).any()  # infinities of one sign per channel
    rest = np.delete(y, [0, 1], axis=1)
    assert np.isfinite(rest).all()


@pytest.mark.parametrize("layer", F32, ids=lambda l: l.name)
def test_fp32_large_weight(layer):
    """Finite weights that round to infinity in bf16 give finite sums, and
    nothing at all against a zero input."""
    P.say("case", layer)
    x, w = _inputs(layer, 9)
    x, w = x.abs() * 1e-2 + 1e-3, w.abs()
    x[0, 1] = 0
    a = (lambda c, k: (c, k)) if layer.transposed else (lambda c, k: (k, c))
    w[a(0, 0)] = 3.4e38  # output channel 0 alone: 3.4e36 and more
    w[a(2, 1)][0, 0] = -torch.finfo(torch.float32).max
    w[a(1, 2)] = 3.4e38  # meets the zeros only in the first image
    xd, wd = x.double(), w.double()
    f = torch.nn.functional
    ref = (f.conv_transpose2d(xd, wd, None, layer.stride, layer.pad, layer.out_pad)
           if layer.transposed else
           f.conv2d(xd, wd, None, layer.stride, layer.pad, layer.dil)).numpy()
    y = _run(layer, x, w)
    assert np.isfinite(ref).all() and (np.abs(ref) < 3e38).all()
    assert np.abs(ref[:, 0]).max() > 1e36 and np.abs(ref[0, 2]).max() < 1e3
    # (one sign a channel but for one tap, and fp32's subnormals)
    absref = (f.conv_transpose2d(xd, wd.abs(), None, layer.stride, layer.pad, layer.out_pad)
              if layer.transposed else
              f.conv2d(xd, wd.abs(), None, layer.stride, layer.pad, layer.dil)).numpy()
    assert np.all(np.abs(y - ref) <= 75 * 2.0 ** -24 * absref + 1e-30)


@pytest.mark.parametrize("scale", [1e-30, 1e-18, 1.0, 1e15])
@pytest.mark.parametrize("layer", F32[:2], ids=lambda l: l.name)
def test_fp32_scales(layer, scale):
    """The relative error stays that of fp32 sums from tiny to huge inputs."""
    x, w = _inputs(layer, 11)
    xs = (x.double() * scale).float()
    ref = P.oracle_full(layer, xs, w)
    y = _run(layer, xs, w)
    err = np.linalg.norm(y - ref) / np.linalg.norm(ref)
    assert err <= 1e-6, err


@pytest.mark.parametrize("small", ["x", "w"])
@pytest.mark.parametrize("scale", [1e-34, 1e-36, 3e-38, 1e-41, 1e27])
@pytest.mark.parametrize("layer", F32, ids=lambda l: l.name)
def test_fp32_ends_of_the_exponent_range(layer, scale, small):
    """Operands at the ends of fp32's exponents (subnormal ones, and ones that
    the scaled parts cannot hold) against operands that bring the sums back
    to ordinary size: the three parts lose no bit, so the error is that of
    fp32 sums all the same."""
    P.say("case", layer, scale, small)
    x, w = _inputs(layer, 11)
    other = min(1 / scale, 1e36)  # (1 / 1e-41 is no float)
    a, b = (scale, other) if small == "x" else (other, scale)
    x, w = (x.double() * a).float(), (w.double() * b).float()
    ref = P.oracle_full(layer, x, w)
    y = _run(layer, x, w)
    err = np.linalg.norm(y - ref) / np.linalg.norm(ref)
    assert err <= 1e-6, err


def test_fp32_noalloc_limit():
    """Weights of 56 MiB fit the no-allocation call's 64 MiB, whatever the
    parts that they are split into take; weights of 72 MiB do not."""
    def call(c_out, entry):
        layer = L("na_f32_%d" % c_out, True, 1, 1024, 2, 3, c_out, 4, 2, 1, 0, 1, "NHWC", "f32")
        P.say("case", layer)
        x, w = _inputs(layer, 13)
        x, w = wl.to_layout(x, "NHWC").to(DEV), w.to(DEV)
        desc = h2.make_desc(1, 1024, 2, 3, c_out, 4, 4, 2, 1, 0, 1, layout=h2.HUGE2_NHWC,
                            dtype=h2.HUGE2_F32)
        y = torch.full((1, 4, 6, c_out), float("nan"), device=DEV)
        entry(desc, x.data_ptr(), w.data_ptr(), 0, y.data_ptr(),
              torch.cuda.current_stream(DEV).cuda_stream)
        torch.cuda.synchronize()
        return y
    y = call(896, h2.huge2_conv2d_transpose_noalloc)
    assert torch.equal(y, call(896, h2.huge2_conv2d_transpose)) and torch.isfinite(y).all()
    with pytest.raises(h2.Huge2Error) as e:
        call(1152, h2.huge2_conv2d_transpose_noalloc)
    assert e.value.status == h2.HUGE2_ERR_UNSUPPORTED


@pytest.mark.parametrize("layout", ["NCHW", "NHWC"])
def test_short_all_phase_noalloc_limit(layout):
    """A layer of the all-phase form's shape whose weights fill the
    no-allocation call's 64 MiB, as that form needs no other buffer, is taken
    where the wave-K form runs it; one channel block more is not."""
    def call(c_out, entry):
        layer = L("na_bf16", True, 8, 2048, 4, 4, c_out, 4, 2, 1, 0, 1, layout, "bf16")
        P.say("case", layer)
        g = torch.Generator(DEV).manual_seed(c_out)
        x = torch.randn(P._x_shape(layer), generator=g, device=DEV).bfloat16()
        w = torch.randn(2048, c_out, 4, 4, generator=g, device=DEV).bfloat16()
        desc = h2.make_desc(8, 2048, 4, 4, c_out, 4, 4, 2, 1, 0, 1, dtype=h2.HUGE2_BF16,
                            layout=h2.HUGE2_NCHW if layout == "NCHW" else h2.HUGE2_NHWC)
        y = torch.full((8, c_out, 8, 8), float("nan"), device=DEV).bfloat16()
        entry(desc, x.data_ptr(), w.data_ptr(), 0, y.data_ptr(),
              torch.cuda.current_stream(DEV).cuda_stream)
        torch.cuda.synchronize()
        return y
    y = call(1024, h2.huge2_conv2d_transpose_noalloc)
    assert torch.equal(y, call(1024, h2.huge2_conv2d_transpose)) and torch.isfinite(y).all()
    with pytest.raises(h2.Huge2Error) as e:
        call(1056, h2.huge2_conv2d_transpose_noalloc)
    assert e.value.status == h2.HUGE2_ERR_UNSUPPORTED


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,c,h,w", [(1, 1, 1, 1), (2, 3, 7, 9), (3, 64, 8, 8), (1, 65, 5, 13),
                                     (2, 130, 11, 16), (1, 71, 9, 24)])
def test_nchw_staging(n, c, h, w, dtype):
    """A pointwise conv with the identity as weights gives back its staged
    input, bit for bit: ragged and whole tiles of both staging kernels."""
    P.say("case staging", n, c, h, w, dtype)
    dt = wl.torch_dtype(dtype)
    x = torch.randn(n, c, h, w, generator=torch.Generator().manual_seed(c)).to(dt).to(DEV)
    eye = torch.eye(c, device=DEV, dtype=dt).reshape(c, c, 1, 1).contiguous()
    plan = h2.Plan(eye, x.shape, False, 1, 0, 0, 1, "NCHW", "none")
    try:
        assert torch.equal(plan(x), x)
    finally:
        plan.close()
