"""The blocked kernels (any channel count, image size and stride) against the
undecomposed oracle, at the sizes where their blocks, chunks and staging units
end: lone channel groups, partial chunks, partial output blocks, images of a
few pixels, one and several block columns, odd sizes at stride 2.

Tolerance: an output adds n <= 3200 products in 32 bits; with random signs the
rounding errors add up to about sqrt(n) * 2^-25 of the largest sums, 2e-6,
and fp32 parts leave out less than 2^-24 of a product.  1e-5 of the largest
output is five times that.
"""
import numpy as np
import pytest
import torch

import harness as H
import oracle as orc
import paper_1903_06681_amd as dc
import workloads as wl
from workloads import Layer

pytestmark = pytest.mark.gpu
ALL, X, DY = dc.DC_ALL_TILES, dc.DC_X, dc.DC_DY


def _layer(dtype, N, C, K, Hh, W, R, stride=1, P=1, Q=1, halo=None, seed=900):
    return Layer("blocked", N, C, K, Hh, W, R, R, stride, R // 2, P, Q, R // 2 if halo is None else halo,
                 dtype, "uniform", seed + C + K)


LAYERS = [
    # 3x3: whole chunks, a lone last group, fewer than 8 channels, filters past a block of 64
    _layer("bf16", 2, 128, 128, 14, 14, 3), _layer("bf16", 1, 40, 72, 31, 25, 3), _layer("bf16", 2, 5, 33, 9, 130, 3),
    _layer("bf16", 1, 72, 40, 16, 24, 3, P=2, Q=2), _layer("bf16", 3, 96, 160, 7, 7, 3),
    _layer("f32", 2, 40, 72, 14, 14, 3), _layer("f32", 1, 36, 33, 9, 131, 3), _layer("f32", 1, 64, 40, 16, 24, 3, P=2, Q=2),
    # a margin wider than the padding: unaligned first columns
    _layer("bf16", 1, 24, 24, 26, 39, 3, P=2, Q=3, halo=2), _layer("f32", 1, 24, 24, 26, 39, 3, P=2, Q=3, halo=3),
    # stride 2: odd sizes (phases of unequal extent), tiles, 1x1 (phases without taps), 5x5
    _layer("bf16", 2, 48, 40, 25, 23, 3, 2), _layer("bf16", 1, 64, 96, 32, 32, 3, 2, 2, 2), _layer("bf16", 2, 40, 24, 15, 18, 1, 2),
    _layer("bf16", 1, 24, 20, 36, 44, 5, 2, 2, 2), _layer("f32", 2, 36, 20, 25, 23, 3, 2), _layer("f32", 1, 40, 24, 15, 18, 1, 2),
    _layer("f32", 1, 16, 24, 32, 24, 5, 2, 2, 2),
    # stride 3: one launch per phase
    _layer("bf16", 1, 24, 32, 24, 27, 3, 3), _layer("f32", 1, 9, 12, 24, 27, 3, 3),
    # 1x1, 5x5, 7x7
    _layer("bf16", 2, 72, 200, 13, 17, 1), _layer("bf16", 1, 281, 48, 9, 35, 1), _layer("f32", 2, 72, 40, 13, 17, 1),
    _layer("bf16", 1, 40, 24, 30, 30, 5), _layer("f32", 1, 20, 40, 20, 30, 5), _layer("bf16", 1, 64, 9, 20, 28, 7),
    # fp32 plans that take a workgroup's whole LDS, or 16 bytes less than would not fit
    _layer("f32", 1, 72, 72, 57, 3, 3, 2), _layer("f32", 1, 40, 72, 61, 4, 4), _layer("f32", 1, 16, 72, 66, 6, 4, 2),
]


def _run(L, x, w, dy):
    p, nt = dc.Problem.of(L), L.P * L.Q
    xt, dyt = H.alloc_tiles(p, X, nt, L.dtype), H.alloc_tiles(p, DY, nt, L.dtype)
    H.scatter_interiors(xt, H.to_device(x, L.dtype), p, X)
    H.scatter_interiors(dyt, H.to_device(dy, L.dtype), p, DY)
    H.fill_halos_all_tiles(p, X, xt, L.dtype)
    H.fill_halos_all_tiles(p, DY, dyt, L.dtype)
    wd = H.to_device(w, L.dtype)
    y = torch.full((nt, L.N, L.K, L.Hot, L.Wot), float("nan"), device="cuda")
    dx = torch.full((nt, L.N, L.C, L.Ht, L.Wt), float("nan"), device="cuda")
    dw = torch.full((L.K, L.C, L.R, L.S), float("nan"), device="cuda")
    ws = torch.empty(max(dc.bwd_filter_workspace_bytes(p, ALL), 16), dtype=torch.uint8, device="cuda")
    dc.conv_fwd(p, ALL, xt, wd, y)
    dc.conv_bwd_data(p, ALL, dyt, wd, dx)
    dc.conv_bwd_filter(p, ALL, xt, dyt, dw, 0, ws)
    torch.cuda.synchronize()
    return (H.gather_outputs(y, p, "y").cpu().numpy(), H.gather_outputs(dx, p, "dx").cpu().numpy(), dw.cpu().numpy())


def _oracle(L, x, w, dy):
    return (orc.round_f32(orc.conv_fwd(x, w, L.stride, L.pad)),
            orc.round_f32(orc.conv_bwd_data(dy, w, L.H, L.W, L.stride, L.pad)),
            orc.round_f32(orc.conv_bwd_filter(x, dy, L.R, L.S, L.stride, L.pad)))


def _id(L):
    return f"{L.dtype}-{L.N}x{L.C}-{L.K}-{L.H}x{L.W}-k{L.R}s{L.stride}-{L.P}x{L.Q}h{L.halo}"


@pytest.mark.parametrize("L", LAYERS, ids=_id)
def test_blocked_layer_matches_oracle(L):
    print(f"[blocked] {L}", flush=True)
    x, w, dy = (wl.draw(L, t) for t in ("x", "w", "dy"))
    for name, got, ref in zip(("y", "dx", "dw"), _run(L, x, w, dy), _oracle(L, x, w, dy)):
        err = float(np.max(np.abs(got.astype(np.float64) - ref)) / np.max(np.abs(ref)))
        assert np.all(np.isfinite(got)) and err <= 1e-5, (name, err)
    x, w, dy = (wl.draw(L, t, dist="int") for t in ("x", "w", "dy"))
    for name, got, ref in zip(("y", "dx", "dw"), _run(L, x, w, dy), _oracle(L, x, w, dy)):
        assert np.array_equal(got, ref), name


@pytest.mark.parametrize("L", [_layer("f32", 1, 40, 40, 12, 20, 3), _layer("f32", 1, 36, 24, 13, 10, 3, 2)], ids=_id)
def test_fp32_extremes(L):
    """Infinities and NaN reach the outputs that read them and no others; values near
    both ends of the range keep fp32's accuracy."""
    print(f"[extremes] {L}", flush=True)
    x, w, dy = (wl.draw(L, t) for t in ("x", "w", "dy"))
    xi, dyi = x.copy(), dy.copy()
    xi[0, 3, 5, 6], xi[0, 7, 2, 1], xi[0, 1, 9, 9] = np.inf, np.nan, -np.inf
    dyi[0, 3, 1, 2], dyi[0, 9, 4, 3] = np.inf, np.nan
    got, want = _run(L, xi, w, dyi), _oracle(L, x, w, dy)
    t = [torch.from_numpy(np.ascontiguousarray(a)).double() for a in (xi, w, dyi)]
    yi = torch.nn.functional.conv2d(t[0], t[1], stride=L.stride, padding=L.pad).numpy()
    dxi = torch.nn.grad.conv2d_input(t[0].shape, t[1], t[2], L.stride, L.pad).numpy()
    for name, g, ref, clean in (("y", got[0], yi, want[0]), ("dx", got[1], dxi, want[1])):
        fin = np.isfinite(ref)
        assert not fin.all() and np.array_equal(np.isnan(g), np.isnan(ref)), name
        assert np.array_equal(g[np.isinf(ref)], ref[np.isinf(ref)].astype(np.float32)), name
        assert float(np.max(np.abs(g[fin] - clean[fin])) / np.max(np.abs(clean))) <= 1e-5, name
    for sx, sw in ((2.0 ** -122, 2.0 ** 20), (2.0 ** 120, 2.0 ** -20), (2.0 ** -60, 2.0 ** -50)):
        xs, ws, ds = (np.ldexp(a.astype(np.float32), int(np.log2(s))) for a, s in ((x, sx), (w, sw), (dy, sx)))
        y, dx, _ = _run(L, xs, ws, ds)
        for name, g, clean in (("y", y, want[0]), ("dx", dx, want[1])):
            # scaling by a power of two is exact but for inputs below 2^-126
            e = np.max(np.abs(g.astype(np.float64) / (sx * sw) - clean)) / np.max(np.abs(clean))
            assert e <= (1e-5 if sx > 2.0 ** -100 else 2e-5), (name, sx, e)


# layers whose three passes all run on the blocked kernels (weight gradient: more than 256 outputs)
BOTTOM = [_layer("f32", 1, 40, 72, 24, 24, 3), _layer("f32", 1, 36, 48, 33, 30, 3, 2), _layer("f32", 2, 64, 96, 12, 20, 1)]


def _rel(g, r):
    return float(np.linalg.norm(g.astype(np.float64) - r) / np.linalg.norm(r))


@pytest.mark.parametrize("L", BOTTOM, ids=_id)
@pytest.mark.parametrize("lo,hi", [(-117, -115), (-126, -117), (-149, -134)])
@pytest.mark.parametrize("tiny", ["x", "w", "dy"])
def test_fp32_bottom_of_the_range(L, lo, hi, tiny):
    """One tensor between 2^lo and 2^hi (from the last bits that three bf16 parts hold
    down to fp32's last subnormals), the other two near 2^60: normal-sized results.

    Limit: up to 648 products are added in 32 bits, whose roundings (each at most
    2^-24 of a partial sum, of random sign) come to sqrt(648 / 3) * 2^-24 = 9e-7 of
    the result if every partial sum were as large as the last; 1e-6."""
    print(f"[bottom] {_id(L)} {tiny} 2^{lo}..2^{hi}", flush=True)
    rng = np.random.default_rng(L.seed + lo)
    t = {}
    for name in ("x", "w", "dy"):
        a = wl.draw(L, name)
        if name == tiny:
            a = np.ldexp(np.sign(a) * (1 + rng.random(a.shape)), rng.integers(lo, hi, a.shape)).astype(np.float32)
            assert np.all(a != 0)
        else:
            a = np.ldexp(a, 60)
        t[name] = a
    for name, got, ref in zip(("y", "dx", "dw"), _run(L, **t), _oracle(L, **t)):
        assert np.all(np.isfinite(got)) and _rel(got, ref) <= 1e-6, (name, _rel(got, ref))


@pytest.mark.parametrize("L", BOTTOM, ids=_id)
@pytest.mark.parametrize("value", [2.0 ** -112 * 1.2345678, 2.0 ** -140])
def test_fp32_one_tiny_value(L, value):
    """A single tiny value in x and in dy, alone in the windows that read it: the outputs
    that read it get it whole (one product, rounded once), all others keep fp32's accuracy."""
    print(f"[tiny] {_id(L)} {value}", flush=True)
    x, w, dy = (wl.draw(L, t) for t in ("x", "w", "dy"))
    w = np.ldexp(w, 40)
    x[:, :, 4:11, 6:13], dy[:, :, 3:10, 2:9] = 0, 0
    x[0, 5, 7, 9], dy[0, 7, 6, 5] = value, value
    got, ref = _run(L, x, w, dy), _oracle(L, x, w, dy)
    for name, g, r in zip(("y", "dx", "dw"), got, ref):
        assert np.all(np.isfinite(g)) and _rel(g, r) <= 1e-6, (name, _rel(g, r))
        if name != "dw":
            one = (r != 0) & (np.abs(r) < 2.0 ** -60)
            assert one.any() and np.max(np.abs(g[one] - r[one]) / np.abs(r[one])) <= 2.0 ** -23, name


def _reads(L, at, out):
    """The outputs (mask over H x W of y, or of dx) whose window holds input pixel `at`."""
    one = np.zeros((1, 1) + ((L.H, L.W) if out == "y" else (L.Ho, L.Wo)), np.float32)
    one[(0, 0) + at] = 1
    k = np.ones((1, 1, L.R, L.S), np.float32)
    f = orc.conv_fwd(one, k, L.stride, L.pad) if out == "y" else orc.conv_bwd_data(one, k, L.H, L.W, L.stride, L.pad)
    return f[0, 0] != 0


@pytest.mark.parametrize("L", BOTTOM + [_layer("f32", 1, 72, 72, 57, 3, 3, 2), _layer("f32", 1, 128, 128, 40, 44, 3)], ids=_id)
@pytest.mark.parametrize("value", [1e-40, 2.0 ** -112, 3e38, np.inf, np.nan])
def test_fp32_fallback_replaces_only_the_outputs_that_read_the_value(L, value):
    """Values that three bf16 parts do not hold change the arithmetic of the outputs that
    read them; every other output keeps its bits."""
    print(f"[fallback] {_id(L)} {value}", flush=True)
    x, w, dy = (wl.draw(L, t) for t in ("x", "w", "dy"))
    w = w * np.float32(0.1)
    clean = _run(L, x, w, dy)
    xat, dat = (7, 1), (5, 1)
    xv, dyv = x.copy(), dy.copy()
    xv[0, 3][xat], dyv[0, 9][dat] = value, value
    got = _run(L, xv, w, dyv)
    t = [torch.from_numpy(a).double() for a in (xv, w, dyv)]
    ref = (torch.nn.functional.conv2d(t[0], t[1], stride=L.stride, padding=L.pad).numpy(),
           torch.nn.grad.conv2d_input(t[0].shape, t[1], t[2], L.stride, L.pad).numpy())
    for name, g, c, r, at in (("y", got[0], clean[0], ref[0], xat), ("dx", got[1], clean[1], ref[1], dat)):
        m = _reads(L, at, name)
        assert m.any() and not m.all()
        assert np.array_equal(g[:, :, ~m], c[:, :, ~m]), name
        if L.N > 1:
            assert np.array_equal(g[1:], c[1:]), name
        g, r = g[0][:, m], r[0][:, m]
        fin = np.isfinite(r) & (np.abs(r) < 3e38)
        assert np.array_equal(np.isnan(g), np.isnan(r)) and np.array_equal(g[np.isinf(r)], r[np.isinf(r)].astype(np.float32))
        if fin.any():
            assert np.max(np.abs(g[fin] - r[fin])) <= 1e-5 * np.max(np.abs(r[fin])), name


@pytest.mark.parametrize("L", BOTTOM + [_layer("f32", 2, 20, 24, 26, 38, 5), _layer("f32", 1, 34, 40, 30, 70, 7),
                                        _layer("f32", 1, 24, 24, 26, 39, 3, P=2, Q=3, halo=3)], ids=_id)
@pytest.mark.parametrize("value", [1e-40, 2.0 ** -112, 3e38, np.inf, np.nan])
def test_fp32_weight_gradient_with_values_the_parts_do_not_hold(L, value):
    """The chunk that holds such a value is added in plain fp32: finite results keep
    fp32's accuracy, infinities and NaN appear where the sums have them."""
    print(f"[dw fallback] {_id(L)} {value}", flush=True)
    x, w, dy = (wl.draw(L, t) for t in ("x", "w", "dy"))
    x[0, 3, 7, 2], dy[0, 9, 5, 1], dy[0, 9, 5, 2] = value, value, 0.25
    dw = _run(L, x, w, dy)[2]
    t = [torch.from_numpy(np.ascontiguousarray(a)).double() for a in (x, dy)]
    ref = torch.nn.grad.conv2d_weight(t[0], w.shape, t[1], L.stride, L.pad).numpy()
    ref[np.abs(ref) > np.finfo(np.float32).max] = np.inf * np.sign(ref[np.abs(ref) > np.finfo(np.float32).max])
    assert np.array_equal(np.isnan(dw), np.isnan(ref)) and np.array_equal(dw[np.isinf(ref)], ref[np.isinf(ref)].astype(np.float32))
    fin = np.isfinite(ref)
    big = fin & (np.abs(ref) > 1e30)   # the sums that the large value is in, and those that it is not in
    for m in (big, fin & ~big):
        if m.any():
            assert np.max(np.abs(dw[m] - ref[m])) <= 1e-5 * np.max(np.abs(ref[m]))


@pytest.mark.parametrize("C,K,R", [(3, 16, 3), (4, 72, 3), (9, 48, 3), (17, 9, 3), (18, 40, 3), (3, 64, 5), (9, 33, 1), (18, 64, 1)])
def test_fp32_few_channels_keep_their_accuracy(C, K, R):
    """Channel groups that are mostly empty do not cost additions at the size of the sum:
    each k-step (16 channels of a tap, or 8 of two) rounds there once, by at most 2^-24 of a
    partial sum, 2^-24 / sqrt(3) on average, and partial sums grow as the root of the steps:
    the k-steps together sqrt(steps / 2) of that, the last addition one more."""
    L = Layer("few", 2, C, K, 90, 86, R, R, 2, R // 2, 1, 1, R // 2, "f32", "normal", 950 + C)
    print(f"[few] {_id(L)}", flush=True)
    x, w, dy = (wl.draw(L, t) for t in ("x", "w", "dy"))
    y = _run(L, x, w, dy)[0]
    groups = (C + 7) // 8
    steps = groups // 2 * R * R + groups % 2 * ((R * R + 1) // 2)
    err = _rel(y, orc.conv_fwd(x, w, L.stride, L.pad))
    assert err <= 2.0 ** -24 / 3 ** 0.5 * (steps / 2 + 1) ** 0.5, err


# One layer or more for every block shape, staging and wave grouping that the planner
# picks over the sizes programs run (4,000 layers drawn from classification, tile and
# mesh models) and that the layers above do not reach.
SHAPES = [
    _layer("f32", 16, 48, 8, 38, 131, 1), _layer("f32", 1, 8, 8, 44, 8, 1, 2), _layer("f32", 2, 8, 8, 4, 6, 1, 2),
    _layer("f32", 16, 40, 96, 141, 27, 1, 2), _layer("f32", 16, 32, 8, 25, 145, 3), _layer("f32", 2, 128, 8, 108, 146, 3),
    _layer("f32", 16, 64, 40, 12, 84, 3), _layer("f32", 4, 8, 136, 94, 66, 3, 2), _layer("f32", 1, 24, 16, 83, 5, 3, 2),
    _layer("f32", 1, 8, 40, 64, 8, 3, 2), _layer("f32", 2, 24, 16, 28, 19, 3, 2), _layer("f32", 2, 72, 64, 31, 67, 3, 2),
    _layer("f32", 4, 24, 136, 59, 115, 3, 2), _layer("f32", 4, 192, 96, 70, 71, 3, 2),
    _layer("bf16", 1, 8, 8, 5, 5, 1), _layer("bf16", 4, 8, 32, 139, 69, 1), _layer("bf16", 1, 8, 24, 4, 6, 1),
    _layer("bf16", 16, 72, 8, 19, 109, 1), _layer("bf16", 16, 8, 264, 55, 17, 1), _layer("bf16", 16, 40, 8, 62, 100, 1),
    _layer("bf16", 16, 96, 24, 18, 108, 1), _layer("bf16", 16, 320, 24, 6, 165, 1), _layer("bf16", 8, 8, 72, 75, 177, 1, 2),
    _layer("bf16", 16, 512, 24, 5, 147, 1, 2), _layer("bf16", 1, 40, 8, 67, 4, 1, 2), _layer("bf16", 1, 96, 96, 4, 7, 1, 2),
    _layer("bf16", 8, 128, 8, 17, 112, 3), _layer("bf16", 16, 8, 128, 9, 175, 3), _layer("bf16", 16, 136, 48, 105, 7, 3),
    _layer("bf16", 8, 48, 24, 72, 127, 3), _layer("bf16", 16, 96, 136, 50, 10, 3), _layer("bf16", 1, 16, 136, 6, 4, 3, 2),
    _layer("bf16", 16, 128, 8, 28, 142, 3, 2), _layer("bf16", 8, 40, 24, 87, 176, 3, 2), _layer("bf16", 1, 32, 64, 128, 4, 3, 2),
    _layer("bf16", 4, 8, 136, 85, 144, 3, 2), _layer("bf16", 8, 8, 128, 65, 179, 3, 2), _layer("bf16", 1, 8, 48, 4, 6, 5, 2),
    _layer("bf16", 1, 40, 48, 5, 4, 5, 2), _layer("bf16", 1, 16, 16, 8, 4, 7, 2), _layer("bf16", 16, 8, 320, 58, 22, 7, 2),
    # weights gathered: channel counts that are no multiples of 8
    _layer("bf16", 2, 77, 9, 4, 6, 1, 2), _layer("bf16", 16, 33, 25, 56, 139, 1, 2), _layer("bf16", 1, 13, 130, 4, 5, 1, 2),
    _layer("bf16", 1, 9, 25, 36, 13, 1, 2), _layer("bf16", 1, 9, 33, 6, 4, 3, 2), _layer("bf16", 2, 33, 13, 4, 5, 3, 2),
    _layer("bf16", 16, 33, 13, 49, 153, 3, 2), _layer("bf16", 16, 33, 33, 111, 81, 3, 2),
]


@pytest.mark.parametrize("L", SHAPES, ids=_id)
def test_every_planned_block_shape_matches_oracle(L):
    """Forward adds up to 4608 products, a weight gradient up to 330,000, in 32 bits: with
    random signs sqrt(n) * 2^-25 of the largest sums, at most 1.7e-5 of the rms sum and, over
    a maximum of four times that, 4.3e-6 of it; 1e-5."""
    print(f"[shapes] {_id(L)}", flush=True)
    x, w, dy = (wl.draw(L, t) for t in ("x", "w", "dy"))
    for name, got, ref in zip(("y", "dx", "dw"), _run(L, x, w, dy), _oracle(L, x, w, dy)):
        err = float(np.max(np.abs(got.astype(np.float64) - ref)) / np.max(np.abs(ref)))
        assert np.all(np.isfinite(got)) and err <= 1e-5, (name, err)


@pytest.mark.parametrize("dtype,C,K,Hh,W,R,S,stride,pad,halo", [
    # partials of whole channel blocks past the allocation-free array, of the row kernels not
    ("bf16", 33, 290000, 4, 3, 1, 1, 2, 0, 0), ("bf16", 33, 69000, 8, 4, 2, 2, 2, 0, 0), ("bf16", 33, 31000, 6, 4, 3, 3, 2, 1, 1),
    ("bf16", 33, 16500, 8, 6, 4, 4, 2, 1, 2), ("bf16", 33, 12000, 9, 6, 5, 5, 2, 2, 2), ("bf16", 33, 7600, 8, 8, 6, 6, 2, 2, 3),
    ("bf16", 33, 6000, 10, 8, 7, 7, 2, 3, 3), ("f32", 205, 15368, 6, 5, 4, 1, 1, 2, 3)])
def test_row_kernels_of_very_wide_layers(dtype, C, K, Hh, W, R, S, stride, pad, halo):
    """The row kernels behind dc_conv_bwd_filter_noalloc on layers whose dw nearly fills its
    array: sampled entries against 64 bits (up to 80 products each, 1e-5 of the largest)."""
    L = Layer("rows", 2, C, K, Hh, W, R, S, stride, pad, 1, 1, halo, dtype, "uniform", 990 + R)
    print(f"[rows] {_id(L)}", flush=True)
    p = dc.Problem.of(L)
    x, dy = wl.draw(L, "x"), wl.draw(L, "dy")
    xt, dyt = H.alloc_tiles(p, X, 1, dtype, fill=0.0), H.alloc_tiles(p, DY, 1, dtype)
    H.scatter_interiors(xt, H.to_device(x, dtype), p, X)
    H.scatter_interiors(dyt, H.to_device(dy, dtype), p, DY)
    dw = torch.full((K, C, R, S), float("nan"), device="cuda")
    assert dc.bwd_filter_workspace_bytes(p, 0) <= dc.BWD_FILTER_NOALLOC_MAX_BYTES
    dc.conv_bwd_filter_noalloc(p, 0, xt, dyt, dw, 0)
    torch.cuda.synchronize()
    rng = np.random.default_rng(3)
    o = np.unique(np.concatenate([rng.integers(0, K, 60), [0, 63, 64, K - 1]]))
    sub = dy[:, o]
    ref = orc.conv_bwd_filter(x, np.ascontiguousarray(sub), R, S, stride, pad)
    got = dw[torch.from_numpy(o).cuda()].cpu().numpy()
    assert bool(torch.isfinite(dw).all()) and np.max(np.abs(got - ref)) <= 1e-5 * np.max(np.abs(ref))
