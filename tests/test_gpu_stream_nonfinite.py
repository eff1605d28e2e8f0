"""Values that are not finite in a streaming step.

Across columns they spread as in the line solver: from the columns whose values a
cell's faces weigh, and from no other, whatever stands in the copies for cells that
have zero weight (two away in second order, beyond a wall).  The other columns hold
the same values as the line solver's (a combination with weights of at most 1 of
right-hand sides of about 40 terms of size at most 4, in two orders: FP64 1e-13,
FP32 40 x 6e-8 x 4 = 1e-5).

Within a column the truncated look-ahead bounds it: a level whose own right-hand
side is not finite is not, nor are the levels that the walk eliminates after it in
its z segment; no column keeps only finite values that the line solver's does not.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

N = (36, 10, 300)
VARIANTS = {"plain": {}, "walls": dict(side_x="walls", side_y="walls"), "walls x": dict(side_x="walls"),
            "explicit z": dict(z_explicit=0.5), "fourth order": dict(face_order=4),
            "all": dict(side_x="walls", side_y="walls", face_order=4, z_explicit=0.5)}


def _ctx(method, prec, kw):
    from paper_1805_03426_amd.context import Context
    faces = [np.arange(N[0] + 1) / 32, np.arange(N[1] + 1) / 32, np.arange(N[2] + 1) * np.sqrt(2e-5 / 0.05)]
    return Context(*faces, (1, 1, 1), 1e6, 1.0, 1e-2, precision=prec, step_method=method, **kw)


def _field(shape, dtype, scale, offset, gen):
    buf = torch.zeros(offset + int(np.prod(shape)), dtype=dtype, device="cuda")
    v = buf[offset:].view(shape)
    v.copy_((torch.rand(shape, dtype=torch.float64, device="cuda", generator=gen) - 0.5) * scale)
    return v


@pytest.mark.parametrize("offset", [0, 1])     # 16-byte copies; 4-byte ones by the pointers' alignment
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("variant", list(VARIANTS))
def test_columns_reached(variant, prec, offset):
    gen = torch.Generator(device="cuda").manual_seed(5)
    nx, ny, nz = N
    kw = VARIANTS[variant]
    with _ctx("auto", prec, kw) as ctx, _ctx("line", prec, kw) as ref:
        assert ctx.step_form() == "stream" and ref.step_form() == "line"
        f = {"cur": _field(ctx.shape_cell, ctx.dtype, 2.0, offset, gen), "prev": _field(ctx.shape_cell, ctx.dtype, 2.0, offset, gen),
             "u": _field(ctx.shape_cell, ctx.dtype, 0.3, offset, gen), "v": _field(ctx.shape_cell, ctx.dtype, 0.3, offset, gen),
             "w": _field(ctx.shape_w, ctx.dtype, 0.1, offset, gen)}
        f["w"][0] = f["w"][-1] = 0.0
        points = [(0, 0, 5), (1, 3, 150), (2, 0, 299), (3, 5, 0), (4, 1, 40), (17, 4, 100), (31, 2, 7), (32, 8, 160),
                  (33, 9, 8), (34, 6, 290), (35, 9, 100), (35, 4, 33)]
        for field, t in f.items():
            for i, j, k in points:
                for bad in (float("nan"), float("inf")):
                    print("case non-finite", variant, prec, offset, field, i, j, k, bad, flush=True)
                    old = t[k, j, i].item()
                    t[k, j, i] = bad
                    out, want = ctx.empty(ctx.shape_cell), ref.empty(ref.shape_cell)
                    ctx.scalar_step(2, f["prev"], f["cur"], out, f["u"], f["v"], f["w"])
                    ref.scalar_step(2, f["prev"], f["cur"], want, f["u"], f["v"], f["w"])
                    t[k, j, i] = old
                    got_bad, want_bad = ~torch.isfinite(out), ~torch.isfinite(want)
                    assert torch.equal(got_bad.any(0), want_bad.any(0))
                    assert not (got_bad & ~want_bad).any()
                    clean = ~want_bad.any(0)
                    err = (out - want)[:, clean].abs().max().item()
                    assert err <= (1e-13 if prec == "fp64" else 1e-5), err
                    if field in ("cur", "prev"):
                        assert got_bad[k, j, i]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("variant", ["plain", "all"])
def test_levels_reached(variant, prec):
    """A level that is not finite takes those within the look-ahead along on both
    sides (13 levels at r = 0.05; at least 8 here), walking up and down, and in the
    reverse step."""
    gen = torch.Generator(device="cuda").manual_seed(6)
    with _ctx("auto", prec, VARIANTS[variant]) as ctx:
        assert ctx.step_form() == "stream"
        cur, prev = (_field(ctx.shape_cell, ctx.dtype, 2.0, 0, gen) for _ in range(2))
        u, v = (_field(ctx.shape_cell, ctx.dtype, 0.3, 0, gen) for _ in range(2))
        w = torch.zeros(ctx.shape_w, dtype=ctx.dtype, device="cuda")
        out = ctx.empty(ctx.shape_cell)
        for k in (0, 7, 20, 37, 38, 75, 150, 222, 299):
            cur[k, 5, 18] = float("nan")
            calls = [lambda: ctx.scalar_step(2, prev, cur, out, u, v, w), lambda: ctx.scalar_step(3, prev, cur, out, u, v, w)]
            if variant == "plain":
                calls += [lambda n=n: ctx.scalar_step_backward(n, prev, cur, None, out, u, v, w) for n in (2, 3)]
            for q, call in enumerate(calls):
                print("case levels", variant, prec, k, q, flush=True)
                call()
                assert not torch.isfinite(out[max(0, k - 8):k + 9, 5, 18]).any()
            cur[k, 5, 18] = 0.0
