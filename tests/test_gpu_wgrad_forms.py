"""GPU tests of the weight gradients' gather on any pixel count and of the
GEMM's tiles, against the float64 oracle."""
import numpy as np
import pytest
import torch

from paper_1907_11210_amd import huge2 as h2

import parity as P
import test_gpu_wgrad as W

pytestmark = pytest.mark.gpu

# name, transposed, n, c_in, h, w, c_out, r, s, stride, pad, out_pad, dil, dtype
CASES = [
    # small grids of an odd pixel count: pairs of images per workgroup, an odd
    # last one, a single image, pairs of elements across an image's end
    ("odd_pixels", False, 5, 12, 9, 7, 20, 3, 3, 1, 1, 0, 1, "bf16"),
    ("odd_one_image", False, 1, 9, 7, 5, 70, 3, 3, 1, 2, 0, 2, "bf16"),
    ("odd_many_channels", False, 7, 520, 5, 5, 24, 3, 3, 1, 1, 0, 1, "bf16"),
    ("even_pixels", True, 3, 33, 5, 6, 10, 4, 4, 2, 1, 0, 1, "bf16"),
    ("odd_f32", False, 3, 10, 11, 13, 33, 5, 5, 2, 2, 0, 1, "f32"),
    # a plane of almost 32 KiB, doubled to a pair of images
    ("odd_large_plane", False, 3, 5, 127, 127, 6, 3, 3, 1, 1, 0, 1, "bf16"),
    # few columns or rows, all on 64 x 64 tiles; 128 x 64 and more of both
    ("tile_64_64", False, 2, 60, 8, 9, 64, 1, 1, 1, 0, 0, 1, "bf16"),
    ("short_64_128", True, 2, 61, 6, 7, 17, 3, 3, 2, 1, 1, 1, "bf16"),
    ("short_128_64", True, 2, 130, 6, 7, 3, 4, 4, 2, 1, 0, 1, "bf16"),
    ("short_128_128", False, 3, 30, 12, 11, 129, 3, 3, 1, 1, 0, 1, "bf16"),
    ("tile_f32_128", False, 2, 30, 12, 11, 129, 3, 3, 1, 1, 0, 1, "f32"),
    ("tile_f32_64", False, 2, 66, 9, 9, 40, 1, 1, 1, 0, 0, 1, "f32"),
    # one K slice, fewer stages than the loads run ahead
    ("short_k", False, 1, 66, 4, 4, 66, 2, 2, 1, 0, 0, 1, "f32"),
]


# of an odd pixel count in 16 bits and several images: pairs of images
PAIRS = ("odd_pixels", "odd_many_channels", "odd_large_plane")


def _kernel(case):
    """The kernel that the case's plan names."""
    _, tr, n, ci, h, w, co, r, s, st, pd, op, dl, dt = case
    plan = h2.huge2_wgrad_plan_create(
        h2.make_desc(n, ci, h, w, co, r, s, st, pd, op, dl,
                     dtype=h2.HUGE2_BF16 if dt == "bf16" else h2.HUGE2_F32), tr)
    try:
        return h2.huge2_wgrad_plan_kernel(plan)
    finally:
        h2.huge2_wgrad_plan_destroy(plan)


@pytest.mark.parametrize("case", CASES, ids=lambda c: c[0])
def test_forms(case, monkeypatch):
    """Gathered through LDS or by the plain staging kernel
    (HUGE2_WGRAD_GATHER=0): the oracle's values, and the same bits."""
    P.say("case", case)
    xq, dyq = W._inputs(case, seed=21)
    ref, absref = W._oracle(case, xq, dyq), W._oracle(case, xq, dyq, absolute=True)
    monkeypatch.setenv("HUGE2_WGRAD_GATHER", "2")
    assert int(_kernel(case).split("gather")[1]) >= (2 if case[0] in PAIRS else 1)
    got = W._gpu(case, xq, dyq)
    P.check(got, ref, absref, case[-1], case[0])
    if case[-1] == "f32":
        # three bf16 parts leave 2^-25 of a product out; the fp32 sums of at
        # most 512 terms round within 2^-24 of the largest partial sum each
        assert np.all(np.abs(got - ref) <= 24 * 2.0 ** -24 * absref + 1e-30)
    monkeypatch.setenv("HUGE2_WGRAD_GATHER", "0")
    assert "gather0" in _kernel(case)
    assert np.array_equal(got, W._gpu(case, xq, dyq))


@pytest.mark.parametrize("case", [c for c in CASES if c[0] in ("odd_pixels", "odd_large_plane")],
                         ids=lambda c: c[0])
def test_gather_of_a_last_single_image(case, monkeypatch):
    """Chunks of two images of an odd pixel count, the last of one: the pair's
    second half is not there to read."""
    P.say("case", case)
    xq, dyq = W._inputs(case, seed=22)
    monkeypatch.setenv("HUGE2_WGRAD_CHUNK", "2")
    monkeypatch.setenv("HUGE2_WGRAD_GATHER", "2")
    assert "gather2" in _kernel(case)
    got = W._gpu(case, xq, dyq)
    P.check(got, W._oracle(case, xq, dyq), W._oracle(case, xq, dyq, absolute=True), case[-1], case[0])
    monkeypatch.setenv("HUGE2_WGRAD_GATHER", "0")
    assert np.array_equal(got, W._gpu(case, xq, dyq))


@pytest.mark.parametrize("n,gather", [(2, "gather0"), (12, "gather2")])
def test_gather_by_workgroups(n, gather):
    """Off multiples of 8 pixels the gather is taken where it has a workgroup
    for every compute unit."""
    case = ("workgroups", False, n, 136, 62, 28, 20, 4, 4, 1, 1, 0, 1, "bf16")
    P.say("case", case)
    assert gather in _kernel(case)


# enough work for wide tiles (from 4096 tiles of 64 x 64 times 128-byte stages)
TILES = [
    ("64x128", False, 8, 61, 60, 61, 60, 3, 3, 1, 1, 0, 1, "bf16"),
    ("128x64", False, 4, 3, 124, 124, 1030, 4, 4, 2, 1, 0, 1, "bf16"),
    ("128x128", True, 6, 100, 49, 50, 61, 3, 3, 1, 1, 0, 1, "bf16"),
]


@pytest.mark.parametrize("case", TILES, ids=lambda c: c[0])
def test_wide_tiles(case):
    """The 64 x 128, 128 x 64 and 128 x 128 tiles with remainders on both
    sides, against sums in float64."""
    P.say("case", case)
    assert "kernel " + case[0] + " " in _kernel(case)
    name, tr, n, ci, h, w, co, r, s, st, pd, op, dl, dt = case
    xq, dyq = W._inputs(case, seed=27)
    # per tap, a product of two matrices: the small tensor and the large one's tap
    sm, bg = (xq, dyq) if tr else (dyq, xq)
    bg = torch.nn.functional.pad(bg.double(), (pd, r, pd, r))
    hs, ws = sm.shape[2:]
    a = sm.double().transpose(0, 1).flatten(1)
    ref = np.empty(tuple(W._w_shape(case)))
    absref = np.empty_like(ref)
    for kh in range(r):
        for kw in range(s):
            b = bg[:, :, kh:kh + (hs - 1) * st + 1:st, kw:kw + (ws - 1) * st + 1:st]
            b = b.transpose(0, 1).flatten(1).t().contiguous()
            ref[:, :, kh, kw] = (a @ b).numpy()
            absref[:, :, kh, kw] = (a.abs() @ b.abs()).numpy()
    P.check(W._gpu(case, xq, dyq), ref, absref, case[-1], case[0])


@pytest.mark.parametrize("scale", [1e-36, 1e-41, 1e27])
@pytest.mark.parametrize("case", [c for c in CASES if c[0] in ("odd_f32", "tile_f32_128")],
                         ids=lambda c: c[0])
def test_ends_of_the_exponent_range(case, scale):
    """x at the ends of fp32's exponents against errors that bring the sums
    back to ordinary size: the error is that of fp32 sums all the same."""
    P.say("case", case, scale)
    xq, dyq = W._inputs(case, seed=25)
    xq, dyq = (xq.double() * scale).float(), (dyq.double() * min(1 / scale, 1e36)).float()
    ref = W._oracle(case, xq, dyq)
    err = np.linalg.norm(W._gpu(case, xq, dyq) - ref) / np.linalg.norm(ref)
    assert err <= 1e-6, err


@pytest.mark.parametrize("case", [c for c in CASES if c[0] in ("odd_f32", "tile_f32_128")],
                         ids=lambda c: c[0])
def test_non_finite(case):
    """An infinity and a NaN in x reach the gradients that fp32 arithmetic
    gives them, and no others."""
    P.say("case", case)
    xq, dyq = W._inputs(case, seed=23)
    xq, dyq = xq.abs() + 0.1, dyq.abs() + 0.1
    clean = W._gpu(case, xq, dyq)
    xq[0, 1, 5, 5] = float("inf")
    xq[0, 2, 5, 5] = float("nan")
    got = W._gpu(case, xq, dyq)
    assert np.isfinite(clean).all()
    assert np.isposinf(got[:, 1]).any() and not np.isneginf(got).any()
    assert np.isnan(got[:, 2]).any()
    rest = np.delete(got, [1, 2], axis=1)
    assert np.array_equal(rest, np.delete(clean, [1, 2], axis=1))


def test_non_finite_in_time():
    """Gradients whose sums are all formed again (errors of NaN) take a few
    times as long, not tens of times."""
    dev = torch.device("cuda", 0)
    n, ci, h, co = 64, 512, 8, 256
    x, dy = torch.randn(n, ci, h, h, device=dev), torch.randn(n, co, 2 * h, 2 * h, device=dev)
    bad = torch.full_like(dy, float("nan"))
    dw = torch.empty(ci, co, 4, 4, device=dev)
    plan = h2.huge2_wgrad_plan_create(h2.make_desc(n, ci, h, h, co, 4, 4, 2, 1), True)

    def us(e):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        for i in range(5):
            if i == 1:
                a.record()
            h2.huge2_wgrad_execute(plan, x.data_ptr(), e.data_ptr(), dw.data_ptr(),
                                   torch.cuda.current_stream(dev).cuda_stream)
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) * 250
    try:
        usual, redone = us(dy), us(bad)
        P.say("us", usual, redone)
        assert torch.isnan(dw).all()
        assert redone <= 12 * usual
    finally:
        h2.huge2_wgrad_plan_destroy(plan)


def test_many_columns():
    """5.5M columns (beyond 65535 tiles of 64) of a one-pixel layer: every
    gradient is one product, rounded once."""
    P.say("case many columns")
    dev = torch.device("cuda", 0)
    g = torch.Generator(dev).manual_seed(3)
    x = torch.randn(1, 128, 1, 1, generator=g, device=dev).bfloat16()
    dy = torch.randn(1, 32768, 13, 13, generator=g, device=dev).bfloat16()
    dw = h2.conv2d_transpose_wgrad(x, dy, (128, 32768, 13, 13), 1, 0)
    want = torch.outer(x.flatten().float(), dy.flatten().float()).bfloat16()
    assert torch.equal(dw.view(128, -1), want)
