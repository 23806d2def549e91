"""Float convolutions on three bf16 terms (conv_triple.hip) against the CPU
oracle and against the float kernels.

Bound.  The products of the first terms add up in a float accumulator that is
rounded once per 16 reduction elements (32 in the 16-row tiles), the small ones
in another; the splits' partials and the bias add a few roundings more.  For
operands of random sign these roundings are independent and the running sum is
at most the result's size in the mean, so the 2-norm error is about
2^-24 sqrt(R / 16) of the result's norm plus the last rounding.  A missing
product of any order (2^-9, 2^-18 of a term) is above it.  Each single output is
within its worst case: the two accumulators' R / 16 additions and a few more,
each off by at most 2^-23 (the instructions may cut instead of rounding) of the
sum of the terms' sizes, and each product by 2^-24.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_1408_5093_amd as cc

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV)


def _close(got, ref, R, what):
    torch.cuda.synchronize()
    got = got.double().cpu().numpy()
    assert got.shape == ref.shape and np.all(np.isfinite(got)), what
    rel = np.linalg.norm(got - ref) / max(np.linalg.norm(ref), 1e-300)
    bound = (2 + np.sqrt(R / 16)) * 2.0 ** -24
    assert rel <= bound, f"{what}: {rel:.2e} > {bound:.2e}"


def _each(got, ref, sizes, R, what):
    """sizes: the same sum over the absolute values of its terms."""
    torch.cuda.synchronize()
    err = np.abs(got.double().cpu().numpy() - ref)
    bound = (R / 16 + 8) * 2.0 ** -23 * sizes + 2.0 ** -149
    assert np.all(err <= bound), f"{what}: an output is off by {(err / bound).max():.2f} bounds"


def _case(c, seed=0):
    N, C, H, W, K, kh, kw, sh, sw, ph, pw, g = c
    rng = np.random.default_rng([1408, seed] + list(c))
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = (rng.standard_normal((K, C // g, kh, kw)) * 0.3).astype(np.float32)
    b = rng.standard_normal(K).astype(np.float32)
    Ho, Wo = (H + 2 * ph - kh) // sh + 1, (W + 2 * pw - kw) // sw + 1
    gd = rng.standard_normal((N, K, Ho, Wo)).astype(np.float32)
    top = np.maximum(rng.standard_normal(gd.shape), 0).astype(np.float32)
    return x, w, b, gd, top


# N, C, H, W, K, kh, kw, sh, sw, ph, pw, group
CASES = [
    (1, 8, 5, 5, 8, 3, 3, 1, 1, 1, 1, 1),       # one ragged tile, one unit per tap
    (2, 5, 9, 7, 13, 3, 2, 1, 1, 1, 0, 1),      # padded channels both ways
    (3, 32, 13, 13, 64, 3, 3, 1, 1, 1, 1, 1),   # whole 32-channel stages
    (2, 96, 15, 11, 96, 5, 5, 1, 1, 2, 2, 2),   # 48 channels per group: half stages
    (2, 40, 12, 9, 130, 3, 3, 2, 2, 1, 1, 1),   # strided, rows past a 128-row tile
    (1, 64, 20, 17, 192, 1, 1, 1, 1, 0, 0, 1),  # 1x1, 96-row tiles
    (2, 16, 19, 23, 48, 7, 5, 3, 2, 3, 1, 2),   # unequal strides, phase-stacked rows
    (1, 24, 3, 256, 20, 1, 3, 1, 1, 0, 1, 1),   # rows of 256 pixels, the staging's limit
    (2, 8, 6, 6, 9, 2, 2, 3, 3, 0, 0, 1),       # stride past the kernel: unread pixels
    (5, 12, 4, 4, 24, 4, 4, 1, 1, 3, 3, 3),     # pad wider than the image's margin
]


@pytest.mark.parametrize("c", CASES)
@pytest.mark.parametrize("relu", [False, True])
def test_terms_parity(overrides, c, relu):
    overrides.setenv("CAFFE_CONV_X3", "7")
    N, C, H, W, K, kh, kw, sh, sw, ph, pw, g = c
    x, w, b, gd, top = _case(c)
    R = (C // g) * kh * kw
    y = cc.conv_forward(_t(x), _t(w), _t(b), (sh, sw), (ph, pw), g, relu)
    ref = oracle.conv_forward(x, w, b, (sh, sw), (ph, pw), g, relu)
    _close(y, ref, R, "forward")
    ax, aw, agd = (np.abs(a) for a in (x, w, gd))
    _each(y, ref, oracle.conv_forward(ax, aw, np.abs(b), (sh, sw), (ph, pw), g, False), R,
          "forward")
    dx, dw, db = cc.conv_backward(_t(x), _t(w), _t(gd), _t(top), (sh, sw), (ph, pw), g, relu)
    rx, rw, rb = oracle.conv_backward(x, w, gd, top=top, stride=(sh, sw), pad=(ph, pw), group=g,
                                      relu=relu)
    _close(dx, rx, (K // g) * kh * kw, "data gradient")
    _close(dw, rw, gd.size // K, "weight gradient")
    _close(db, rb, gd.size // K, "bias gradient")
    sx, sw_, _ = oracle.conv_backward(ax, aw, agd, top=top, stride=(sh, sw), pad=(ph, pw), group=g,
                                      relu=relu)
    _each(dx, rx, sx, (K // g) * kh * kw, "data gradient")
    _each(dw, rw, sw_, gd.size // K, "weight gradient")


@pytest.mark.parametrize("tile", range(4))
@pytest.mark.parametrize("how", [{"SPLITS": 3}, {"TAIL_SPLITS": 2, "TAIL_UNITS": 3}])
def test_terms_tiles_and_splits(overrides, tile, how):
    """Every tile with an even split and with a tail split of its reduction."""
    overrides.setenv("CAFFE_CONV_X3", "7")
    overrides.setenv("CAFFE_X3_FWD_TILE", str(tile))
    overrides.setenv("CAFFE_X3_DGRAD_TILE", str(tile))
    overrides.setenv("CAFFE_X3_WGRAD_TILE", str(min(tile, 2)))
    if "SPLITS" in how:
        for k in ("FWD", "DGRAD", "WGRAD"):
            overrides.setenv(f"CAFFE_X3_{k}_SPLITS", str(how["SPLITS"]))
    else:
        for k, v in how.items():
            overrides.setenv(f"CAFFE_X3_{k}", str(v))
    c = (3, 64, 21, 19, 140, 3, 3, 1, 1, 1, 1, 2)
    N, C, H, W, K, kh, kw, sh, sw, ph, pw, g = c
    x, w, b, gd, top = _case(c)
    y = cc.conv_forward(_t(x), _t(w), _t(b), 1, 1, g, True)
    _close(y, oracle.conv_forward(x, w, b, 1, 1, g, True), 32 * 9, "forward")
    xs = np.abs(x) * (x > -0.5)
    dx, dw, _ = cc.conv_backward(_t(xs), _t(w), _t(gd), _t(top), 1, 1, g, True,
                                 flags=cc.BACKWARD_MASK_BOTTOM_DIFF)
    rx, rw, _ = oracle.conv_backward(xs, w, gd, top=top, stride=1, pad=1, group=g, relu=True)
    _close(dx, rx * (xs > 0), 70 * 9, "masked data gradient")
    _close(dw, rw, N * H * W, "weight gradient")


@pytest.mark.parametrize("stride", [1, 2])
def test_terms_non_finite_as_float(overrides, stride):
    """Infinities, NaN and the largest floats give what the float kernels
    give, element by element (with a stride the data gradient's phases have
    taps that don't exist, zeros in both paths)."""
    c = (2, 48, 11, 12, 40, 3, 3, stride, stride, 1, 1, 2)
    x, w, b, gd, top = _case(c)
    x[0, 3, 2, 5], x[0, 30, 9, 9], x[1, 4, 4, 4] = np.inf, -np.inf, np.nan
    x[1, 7, 10, 0], x[0, 9, 0, 0] = 3.4e38, 0.0
    w[3, 2, 1, 1], w[21, 5, 0, 0], w[30, 1, 2, 2] = np.inf, -np.inf, np.nan
    w[4] *= 1e-30
    w[5, :, 1, 1] = 1.0
    gd[0, 11, 3, 3], gd[1, 25, 0, 0], gd[1, 2, 5, 5] = np.inf, -np.inf, np.nan
    outs = []
    for mode in ("0", "7"):
        overrides.setenv("CAFFE_CONV_X3", mode)
        with np.errstate(all="ignore"):
            y = cc.conv_forward(_t(x), _t(w), _t(b), stride, 1, 2, False)
            outs.append([y] + list(cc.conv_backward(_t(x), _t(w), _t(gd), None, stride, 1, 2,
                                                    False)))
    torch.cuda.synchronize()
    for a, t in zip(*outs):
        assert torch.equal(torch.isnan(a), torch.isnan(t))
        assert torch.equal(torch.isposinf(a), torch.isposinf(t))
        assert torch.equal(torch.isneginf(a), torch.isneginf(t))
        f = torch.isfinite(a)
        assert f.any()
        scale = a[f].abs().clamp_min(1e-3)
        assert ((a[f] - t[f]).abs() / scale).max() < 1e-3


def _tile(overrides, tile, how):
    overrides.setenv("CAFFE_CONV_X3", "7")
    overrides.setenv("CAFFE_X3_FWD_TILE", str(tile))
    overrides.setenv("CAFFE_X3_DGRAD_TILE", str(tile))
    overrides.setenv("CAFFE_X3_WGRAD_TILE", str(min(tile, 2)))
    for k, v in how.items():
        overrides.setenv(f"CAFFE_X3_{k}", str(v))


SPLIT3 = {f"{k}_SPLITS": 3 for k in ("FWD", "DGRAD", "WGRAD")}
TAIL2 = {"TAIL_SPLITS": 2, "TAIL_UNITS": 3}


def _same_sign_close(got, ref, R, what):
    """Sums of terms of one sign: infinite where the 64-bit sum is past the
    largest float, else within one rounding a term (and two) of it."""
    torch.cuda.synchronize()
    got = got.double().cpu().numpy()
    over = np.abs(ref) > 2.0 ** 128
    assert np.array_equal(got[over], np.copysign(np.inf, ref[over])), what
    err = np.abs(got[~over] - ref[~over])
    bound = (R + 2) * 2.0 ** -24 * np.abs(ref[~over]) + 2.0 ** -149
    assert np.all(err <= bound), f"{what}: {(err / bound).max():.2f} of the bound"
    return over


@pytest.mark.parametrize("tile", range(4))
@pytest.mark.parametrize("how", [{}, SPLIT3, TAIL2], ids=["whole", "split", "tail"])
@pytest.mark.parametrize("relu", [False, True])
def test_terms_finite_products_overflow(overrides, tile, how, relu):
    """Finite operands of which some products (2^137 and more: the small
    products, whose signs are those of the rounding, overflow too) and some
    sums are past the largest float: infinite as in float arithmetic, and the
    sums beside them stay what they are.  All terms of a sum have one sign, so
    the order of the additions decides nothing."""
    _tile(overrides, tile, how)
    c = (3, 64, 21, 19, 140, 3, 3, 1, 1, 1, 1, 2)
    N, C, H, W, K, kh, kw, sh, sw, ph, pw, g = c
    x, w, b, gd, top = _case(c)
    rng = np.random.default_rng(137)
    sign = np.where(np.arange(K) % 3 == 0, -1, 1).astype(np.float32)[:, None, None]
    big = lambda a, n, v: np.where(rng.random(a.shape) < 1 / n, np.float32(v), np.float32(1))
    x = np.abs(x) * big(x, 50, 1e30)
    w = np.abs(w) * sign[..., None] * np.where(np.arange(K) % 5 < 2, np.float32(1e30),
                                               np.float32(1))[:, None, None, None]
    gd = np.abs(gd) * sign * big(gd, 4000, 3e25)
    assert all(np.isfinite(a).all() for a in (x, w, gd))
    y = cc.conv_forward(_t(x), _t(w), None, 1, 1, g, relu)
    over = _same_sign_close(y, oracle.conv_forward(x, w, None, 1, 1, g, relu), 32 * 9, "forward")
    assert 0.02 < over.mean() < 0.9
    dx, dw, db = cc.conv_backward(_t(x), _t(w), _t(gd), _t(top), 1, 1, g, relu,
                                  flags=cc.BACKWARD_MASK_BOTTOM_DIFF)
    rx, rw, rb = oracle.conv_backward(x, w, gd, top=top, stride=1, pad=1, group=g, relu=relu)
    for got, ref, R, what in ((dx, rx * (x > 0), 70 * 9, "data gradient"),
                              (dw, rw, N * H * W, "weight gradient"),
                              (db, rb, N * H * W, "bias gradient")):
        over = _same_sign_close(got, ref, R, what)
        assert what == "bias gradient" or 0.002 < over.mean() < 0.9, (what, over.mean())


@pytest.mark.parametrize("exp", [-112, -118, -126, -140])
def test_terms_smallest_operands(overrides, exp):
    """Operands down to the subnormals keep every bit (the other operand is
    large, so that the results are ordinary floats)."""
    overrides.setenv("CAFFE_CONV_X3", "7")
    c = (2, 40, 12, 9, 72, 3, 3, 1, 1, 1, 1, 2)
    x, w, b, gd, top = _case(c)
    up = np.float32(2.0 ** 90)
    lo = [(a * np.float32(2.0 ** (exp + 100)) * np.float32(2.0 ** -100)) for a in (x, w, gd)]
    hi = [a * up for a in (x, w, gd)]
    assert all(0 < np.abs(a).max() < 2.0 ** (exp + 4) for a in lo)
    for xs, ws in ((lo[0], hi[1]), (hi[0], lo[1])):
        y = cc.conv_forward(_t(xs), _t(ws), None, 1, 1, 2, False)
        _close(y, oracle.conv_forward(xs, ws, None, 1, 1, 2, False), 20 * 9, "forward")
    for xs, ws, gs in ((hi[0], hi[1], lo[2]), (lo[0], lo[1], hi[2])):
        dx, dw, _ = cc.conv_backward(_t(xs), _t(ws), _t(gs), _t(top), 1, 1, 2, True)
        rx, rw, _ = oracle.conv_backward(xs, ws, gs, top=top, stride=1, pad=1, group=2, relu=True)
        _close(dx, rx, 36 * 9, "data gradient")
        _close(dw, rw, gd.size // 72, "weight gradient")


def test_terms_infinity_times_subnormal_and_large_bias(overrides):
    """inf * y is infinite for the smallest y, and a bias past the scaled
    accumulators' range comes through."""
    overrides.setenv("CAFFE_CONV_X3", "7")
    c = (1, 16, 9, 9, 24, 1, 1, 1, 1, 0, 0, 1)
    x, w, b, _, _ = _case(c)
    w[5] = 2.0 ** -149
    w[6] = -2.0 ** -140
    b[9], b[10] = 1e30, -3e38
    x[0, 3, 4, 4] = np.inf
    y = cc.conv_forward(_t(x), _t(w), _t(b), 1, 0, 1, False).cpu().numpy()
    assert y[0, 5, 4, 4] == np.inf and y[0, 6, 4, 4] == -np.inf
    x[0, 3, 4, 4] = 0
    y[..., 4, 4] = 0
    ref = oracle.conv_forward(x, w, b, 1, 0, 1, False)
    ref[..., 4, 4] = 0
    assert np.array_equal(y[0, 9:11], ref[0, 9:11].astype(np.float32))
    keep = [k for k in range(24) if k not in (9, 10)]
    _close(torch.from_numpy(y[:, keep]), ref[:, keep], 16, "beside the large biases")


@pytest.mark.parametrize("mode", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("how", ["no relu", "relu", "masked"])
@pytest.mark.parametrize("side", [False, True], ids=["one stream", "weight stream"])
def test_terms_beside_float_passes(overrides, mode, how, side):
    """Backward passes of which one gradient runs on terms and the other on the
    float instructions (bits of the mode: 1 forward, 2 data, 4 weights), on a
    workspace of garbage: each set of outputs, added to earlier gradients, on
    a weight stream, with the forward's staging where it left one."""
    overrides.setenv("CAFFE_CONV_X3", str(mode))
    c = (3, 24, 13, 11, 40, 3, 3, 1, 1, 1, 1, 2)
    relu = how != "no relu"
    x, w, b, gd, top = _case(c, mode)
    if how == "masked":
        gd = gd * (top > 0)
    flags = cc.BACKWARD_TOP_DIFF_MASKED if how == "masked" else 0
    d = cc.conv_desc(x.shape, w.shape, 1, 1, 2, relu)
    assert cc.conv_uses_terms(d, cc.PASS_BACKWARD_DATA) == (mode & 2 != 0)
    assert cc.conv_uses_terms(d, cc.PASS_BACKWARD_WEIGHTS) == (mode & 4 != 0)
    refs = oracle.conv_backward(x, w, gd, top=top if relu else None, stride=1, pad=1, group=2,
                                relu=relu)
    X, W, B, G, T = (_t(a) for a in (x, w, b, gd, top))
    ws = torch.empty(max(cc.conv_workspace_preferred(d, p) for p in
                         (cc.PASS_FORWARD, cc.PASS_BACKWARD)), dtype=torch.uint8, device=DEV)
    stream = torch.cuda.Stream() if side else None
    R = (20 * 9, gd.size // 40, gd.size // 40)
    for want in ((1, 1, 1), (1, 1, 0), (1, 0, 1), (0, 1, 1), (0, 0, 1)):
        for accumulate in (0, 1):
            for kept in (0, cc.BACKWARD_BOTTOM_TERMS):
                ws.fill_(0xFF)
                if kept:
                    cc.caffe_conv_forward(d, X, W, B, torch.empty_like(G), ws)
                outs = [torch.full_like(a, 0.5 * accumulate) if on else None
                        for a, on in zip((X, W, B), want)]
                cc.caffe_conv_backward(d, G, T if relu and not flags else None,
                                       X if want[1] else None, W if want[0] else None, *outs,
                                       accumulate, flags | kept, ws, weight_stream=stream)
                torch.cuda.synchronize()
                for i, (o, ref) in enumerate(zip(outs, refs)):
                    if o is not None:
                        _close(o, ref + (0.5 * accumulate if i else 0), R[i],
                               f"{want} accumulate {accumulate} kept {kept}: output {i}")


def test_terms_weight_side_stays_on_stream_unasked(overrides):
    """A float backward with a weight stream keeps its weight side on the main
    stream, as it did before there were terms, unless the call names them
    (BACKWARD_BOTTOM_TERMS): behind a weight stream that is busy the gradients
    are there on the main stream without a join."""
    overrides.setenv("CAFFE_CONV_X3", "7")
    c = (4, 32, 14, 13, 72, 5, 5, 1, 1, 2, 2, 1)
    x, w, b, gd, top = (_t(a) for a in _case(c))
    d = cc.conv_desc(x.shape, w.shape, 1, 2, 1, True)
    ws = torch.empty(cc.conv_workspace_preferred(d, cc.PASS_BACKWARD), dtype=torch.uint8,
                     device=DEV)
    ref = [torch.empty_like(a) for a in (x, w, b)]
    cc.caffe_conv_backward(d, gd, top, x, w, *ref, 0, 0, ws)
    outs = [torch.full_like(a, float("nan")) for a in (x, w, b)]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        torch.cuda._sleep(10_000_000)
    cc.caffe_conv_backward(d, gd, top, x, w, *outs, 0, 0, ws, weight_stream=side)
    got = [a.clone() for a in outs]  # on the main stream, not joined
    torch.cuda.synchronize()
    assert all(torch.equal(a, t) for a, t in zip(ref, got))


def test_terms_kept_bottom_and_weight_stream(overrides):
    """The forward's staging read by the backward, and the weight side on a
    stream of its own, give the same bits; a workspace of the minimum size
    takes the float kernels."""
    overrides.setenv("CAFFE_CONV_X3", "7")
    c = (4, 32, 14, 13, 72, 5, 5, 1, 1, 2, 2, 1)
    x, w, b, gd, top = (_t(a) for a in _case(c))
    d = cc.conv_desc(x.shape, w.shape, 1, 2, 1, True)
    passes = (cc.PASS_FORWARD, cc.PASS_BACKWARD)
    need = max(cc.conv_workspace_preferred(d, p) for p in passes)
    assert all(cc.conv_workspace_preferred(d, p) > cc.conv_workspace_size(d, p) for p in passes)
    assert cc.conv_uses_terms(d, cc.PASS_BACKWARD)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device=DEV)
    side = torch.cuda.Stream()

    def run(buf, flags=0, stream=None, kept=False, fwd=None):
        y = torch.empty_like(gd)
        o = [torch.empty_like(x), torch.empty_like(w), torch.empty_like(b)]
        cc.caffe_conv_forward(d, x, w, b, y, buf if fwd is None else fwd)
        if not kept:
            buf.fill_(0xFF)
        cc.caffe_conv_backward(d, gd, top, x, w, *o, 0, flags, buf, weight_stream=stream)
        torch.cuda.synchronize()
        return [y] + o

    ref = run(ws)
    for got in (run(ws, cc.BACKWARD_BOTTOM_TERMS, None, True), run(ws, 0, side),
                run(ws, cc.BACKWARD_BOTTOM_TERMS, side, True)):
        assert all(torch.equal(a, t) for a, t in zip(ref, got))
    least = [torch.empty(cc.conv_workspace_size(d, p), dtype=torch.uint8, device=DEV)
             for p in (cc.PASS_BACKWARD, cc.PASS_FORWARD)]
    got = run(least[0], cc.BACKWARD_BOTTOM_TERMS, None, True, least[1])  # (no effect there)
    overrides.setenv("CAFFE_CONV_X3", "0")
    assert all(torch.equal(a, t) for a, t in zip(run(least[0], fwd=least[1]), got))


def test_terms_at_the_offsets_limit(overrides):
    """Both stagings just below 2^31 bytes (one image more and the layer stays
    on the float instructions): the first and last images' forward and data
    gradient and, from a top gradient that is zero in all images but those, the
    weight gradient."""
    overrides.setenv("CAFFE_CONV_X3", "7")
    C, H, N = 64, 56, (2 ** 31 - 1) // (58 * 58 * 64 * 6)
    desc = lambda n: cc.conv_desc((n, C, H, H), (C, C, 3, 3), 1, 1, 1, False)
    for p in (cc.PASS_FORWARD, cc.PASS_BACKWARD_DATA, cc.PASS_BACKWARD_WEIGHTS):
        assert cc.conv_uses_terms(desc(N), p) and not cc.conv_uses_terms(desc(N + 1), p)
    gen = torch.Generator(device=DEV).manual_seed(31)
    x = torch.randn((N, C, H, H), generator=gen, device=DEV)
    w = torch.randn((C, C, 3, 3), generator=gen, device=DEV) * 0.3
    ends = [0, 1, N - 2, N - 1]
    gd = torch.zeros_like(x)
    gd[ends] = torch.randn((4, C, H, H), generator=gen, device=DEV)
    y = cc.conv_forward(x, w, None, 1, 1)
    xs, gs, ws = (a.cpu().numpy() for a in (x[ends], gd[ends], w))
    _close(y[ends], oracle.conv_forward(xs, ws, None, 1, 1), C * 9, "forward")
    del y
    dx, dw, _ = cc.conv_backward(x, w, gd, None, 1, 1)
    rx, rw, _ = oracle.conv_backward(xs, ws, gs, stride=1, pad=1)
    _close(dx[ends], rx, C * 9, "data gradient")
    assert not dx[2:-2].any()
    _close(dw, rw, 4 * H * H, "weight gradient")


def test_terms_where_the_least_workspace_holds_them():
    """A layer whose float split partials need as much workspace as the staging:
    its least workspace is the preferred one, and every forward call, the one
    on the static scratch too, runs on terms."""
    N, C, H, W, K, k = 3, 54, 27, 17, 478, 3
    x, w, b, _, _ = _case((N, C, H, W, K, k, k, 1, 1, 1, 1, 1))
    d = cc.conv_desc(x.shape, w.shape, 1, 1, 1, True)
    need = cc.conv_workspace_size(d, cc.PASS_FORWARD)
    assert cc.conv_uses_terms(d, cc.PASS_FORWARD)
    assert need == cc.conv_workspace_preferred(d, cc.PASS_FORWARD) <= cc.NOALLOC_SCRATCH_BYTES
    X, Wt, B = _t(x), _t(w), _t(b)
    y = torch.empty((N, K, H, W), device=DEV)
    cc.caffe_conv_forward(d, X, Wt, B, y, torch.empty(need, dtype=torch.uint8, device=DEV))
    _close(y, oracle.conv_forward(x, w, b, 1, 1, 1, True), C * k * k, "forward")
    z = torch.empty_like(y)
    cc.check(cc.load().caffe_conv_forward_noalloc(
        ctypes.byref(d), *(ctypes.c_void_p(t.data_ptr()) for t in (X, Wt, B, z)),
        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    torch.cuda.synchronize()
    assert torch.equal(y, z)
