"""The work that a training program has this library do, as timed cases.

A case is one layer's share on one GPU and the passes that a program runs on it:

  fwd    the forward pass
  bwd    the weight gradient and the input gradient
  train  forward, weight gradient, input gradient (tiles already bordered)
  step   the whole schedule of a decomposed layer on one stream: pack and unpack
         x, forward, pack and unpack dy, weight gradient, input gradient
  split  the same with the interior of both passes before the margins arrive
         and the boundary frame after

tile = -1 runs every tile of the grid in one launch, as on a single device;
otherwise one tile's share, with the neighbours' bands in a receive buffer.
"""
import math

import torch

import paper_1903_06681_amd as dc

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
#: limits of a drawn case, below those of the largest listed one
MOST_FLOPS = {"bf16": 4e10, "f32": 8e9}
MOST_BYTES = 3e8


def _case(name, op, dtype, N, C, K, H, W, R, stride=1, P=1, Q=1, tile=0):
    c = {"op": op, "dtype": dtype, "N": N, "C": C, "K": K, "H": H, "W": W, "R": R, "stride": stride,
         "P": P, "Q": Q, "tile": tile}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest layer with a halo, the whole 2x2 grid in each launch: latency and launches count
        _case("small_grid_step_f32", "step", "f32", 2, 8, 8, 32, 32, 3, P=2, Q=2, tile=-1),
        # the benchmark's hybrid sample and spatial tile: 256x256 of 1024x1024, four samples
        _case("tile3x3_step_bf16", "step", "bf16", 4, 64, 64, 1024, 1024, 3, P=4, Q=4, tile=5),
        # the 5x5 layer of the same model, its halo exchange overlapped by the interior
        _case("tile5x5_split_bf16", "split", "bf16", 4, 32, 32, 1024, 1024, 5, P=4, Q=4, tile=5),
        # the mesh model in single precision: its first layer on a 512x512 tile of 2048x2048 ...
        _case("mesh_first_train_f32", "train", "f32", 1, 18, 32, 2048, 2048, 3, P=4, Q=4, tile=5),
        # ... a block entry at stride 2, backward ...
        _case("mesh_entry_bwd_f32", "bwd", "f32", 1, 32, 32, 2048, 2048, 3, stride=2, P=4, Q=4, tile=5),
        # ... and a deeper block, where the tile is small and the channels many
        _case("mesh_deep_step_f32", "step", "f32", 1, 128, 128, 256, 256, 3, P=4, Q=4, tile=5),
        # ResNet-50 on one GPU's 32 samples: conv1 at stride 2 on three channels
        _case("res_conv1_train_bf16", "train", "bf16", 32, 3, 64, 224, 224, 7, stride=2),
        # the 3x3 layer of its first stage, backward
        _case("res_3x3_56_bwd_bf16", "bwd", "bf16", 32, 64, 64, 56, 56, 3),
        # the 3x3 layer of its second stage, forward
        _case("res_3x3_28_fwd_bf16", "fwd", "bf16", 32, 128, 128, 28, 28, 3),
        # the 1x1 layer into the first stage's narrow half
        _case("res_1x1_56_train_bf16", "train", "bf16", 32, 256, 64, 56, 56, 1),
        # a late stage's entry: 3x3 at stride 2, many channels on a small image
        _case("res_3x3_s2_28_train_bf16", "train", "bf16", 32, 256, 256, 28, 28, 3, stride=2),
        # odd image, channel counts that are no powers of two
        _case("ragged_3x3_train_bf16", "train", "bf16", 3, 40, 72, 93, 75, 3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """Mostly whole groups of 8 to 64 channels, now and then any count."""
    c, g = _log(rng, lo, hi), rng.choice((1, 8, 16, 32, 64))
    return max(lo, min(hi, (c + g // 2) // g * g)) if c > g else c


def _draw_one(rng):
    family = rng.choice(("res", "res", "tile", "mesh", "mesh", "small"))
    if family == "res":      # classification layers, whole images, one GPU's samples
        R, stride = rng.choice((1, 3, 3)), rng.choice((1, 1, 1, 2))
        return _case(None, rng.choice(("fwd", "bwd", "train")), "bf16", _log(rng, 1, 32), _channels(rng, 16, 512),
                     _channels(rng, 16, 512), _log(rng, 7, 112), _log(rng, 7, 112), R, stride)
    if family == "tile":     # spatially decomposed layers in bf16
        g, R, stride = rng.choice((2, 4)), rng.choice((3, 3, 5, 7)), rng.choice((1, 1, 1, 2))
        op = rng.choice(("step", "train", "split" if stride == 1 else "step"))
        ht, wt = _log(rng, 48, 256) // 2 * 2, _log(rng, 48, 256) // 2 * 2
        return _case(None, op, "bf16", rng.randint(1, 4), _channels(rng, 8, 128), _channels(rng, 8, 128),
                     g * ht, g * wt, R, stride, g, g, rng.randrange(g * g))
    if family == "mesh":     # spatially decomposed layers in single precision
        g, R, stride = rng.choice((2, 4)), rng.choice((3, 3, 3, 1)), rng.choice((1, 1, 2))
        op = rng.choice(("step", "fwd", "bwd", "split" if stride == 1 else "train"))
        ht, wt = _log(rng, 16, 512) // 2 * 2, _log(rng, 16, 512) // 2 * 2
        return _case(None, op, "f32", rng.randint(1, 2), _channels(rng, 3, 128), _channels(rng, 8, 128),
                     g * ht, g * wt, R, stride, g, g, rng.randrange(g * g))
    # the smallest layers, the whole grid in each launch
    return _case(None, "step", rng.choice(("f32", "bf16")), rng.randint(1, 2), _log(rng, 3, 16), _log(rng, 3, 16),
                 2 * _log(rng, 8, 32), 2 * _log(rng, 8, 32), 3, 1, 2, 2, -1)


def draw(rng):
    while True:
        c = _draw_one(rng)
        w = work(c)
        if w["flops"] <= MOST_FLOPS[c["dtype"]] and w["bytes"] <= MOST_BYTES:
            return c


def _problem(c):
    pad = c["R"] // 2
    dt = dc.DC_F32 if c["dtype"] == "f32" else dc.DC_BF16
    return dc.Problem(c["N"], c["C"], c["K"], c["H"], c["W"], c["R"], c["R"], c["stride"], pad, c["P"], c["Q"],
                      pad, dt)


def _tiles(c):
    return range(c["P"] * c["Q"]) if c["tile"] < 0 else (c["tile"],)


def _edges(c, t):
    """Whether tile t has a neighbour above, below, left and right."""
    i, j = divmod(t, c["Q"])
    return i > 0, i < c["P"] - 1, j > 0, j < c["Q"] - 1


def work(c):
    """Each input read once and each output written once, over the passes that run."""
    tiles, e = (c["P"] * c["Q"] if c["tile"] < 0 else 1), (2 if c["dtype"] == "bf16" else 4)
    h, s, pad, R = c["R"] // 2, c["stride"], c["R"] // 2, c["R"]
    Ht, Wt = c["H"] // c["P"], c["W"] // c["Q"]
    Hot = ((c["H"] + 2 * pad - R) // s + 1) // c["P"]
    Wot = ((c["W"] + 2 * pad - R) // s + 1) // c["Q"]
    x, dy = tiles * c["N"] * c["C"] * (Ht + 2 * h) * (Wt + 2 * h), tiles * c["N"] * c["K"] * (Hot + 2 * h) * (Wot + 2 * h)
    y, dx, w = tiles * c["N"] * c["K"] * Hot * Wot, tiles * c["N"] * c["C"] * Ht * Wt, c["K"] * c["C"] * R * R
    one = 2 * tiles * c["N"] * c["K"] * c["C"] * R * R * Hot * Wot
    fwd, bwd = (x + w) * e + 4 * y, (x + y + dy + w) * e + 4 * (dx + w)
    moved = 0
    if c["op"] in ("step", "split"):   # the bands, each read and written by pack and by unpack
        ring_x = tiles * c["N"] * c["C"] * ((Ht + 2 * h) * (Wt + 2 * h) - Ht * Wt)
        ring_dy = tiles * c["N"] * c["K"] * ((Hot + 2 * h) * (Wot + 2 * h) - Hot * Wot)
        moved = 4 * (ring_x + ring_dy) * e
    return {"fwd": {"bytes": fwd, "flops": one}, "bwd": {"bytes": bwd, "flops": 2 * one}}.get(
        c["op"], {"bytes": fwd + bwd + moved, "flops": 3 * one})


def tolerance(c):
    # inputs in the layer's type, products and sums in 32 bits in every pass and type: measured
    # against 64 bits the outputs are 4e-8 to 6e-7 off, the most where 1152 products are added
    # in one chain; a weight gradient adds up to 400,000
    return {"rel": 3e-6, "max": 1e-4}


def _global(c, seed):
    """x, dy over the domain that the tiles see (their bands with it) and w, from the seed alone.

    Activations and gradients are normal, the weights scaled by their fan-in.  Where the
    tile is one of a grid only it and its bands are drawn; what lies outside the domain is zero."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    p, dt = _problem(c), DTYPES[c["dtype"]]
    Ht, Wt, Hot, Wot = dc.tile_dims(p)
    h, R = p.halo, c["R"]
    ti, tj = (c["P"], c["Q"]) if c["tile"] < 0 else (1, 1)

    def padded(ch, rows, cols):
        a = torch.randn((c["N"], ch, ti * rows + 2 * h, tj * cols + 2 * h), generator=g, device="cuda").to(dt)
        if h:
            up, down, left, right = _edges(c, c["tile"]) if c["tile"] >= 0 else (False,) * 4
            for there, s in ((up, a[:, :, :h]), (down, a[:, :, -h:]), (left, a[..., :h]), (right, a[..., -h:])):
                if not there:
                    s.zero_()
        return a

    x, dy = padded(c["C"], Ht, Wt), padded(c["K"], Hot, Wot)
    w = (torch.randn((c["K"], c["C"], R, R), generator=g, device="cuda") * math.sqrt(2.0 / (c["C"] * R * R))).to(dt)
    return x, dy, w


def _layout(c, p, which, a, bordered):
    """The padded tiles of `a` in the library's layout, and what the neighbours send a lone tile.

    Margins hold the bands that the passes read (zeros around them) where `bordered`."""
    Ht, Wt, Hot, Wot = dc.tile_dims(p)
    rows, cols = (Ht, Wt) if which == dc.DC_X else (Hot, Wot)
    h, (bn, bs, bw, be) = p.halo, dc.halo_bands(p, which)
    tiles = torch.zeros((len(_tiles(c)),) + dc.tile_shape(p, which), dtype=a.dtype, device="cuda")
    for k, t in enumerate(_tiles(c)):
        i, j = divmod(t, c["Q"]) if c["tile"] < 0 else (0, 0)
        src = a[:, :, i * rows:i * rows + rows + 2 * h, j * cols:j * cols + cols + 2 * h]
        n, s, w, e = (bn, bs, bw, be) if bordered else (0, 0, 0, 0)
        at = (slice(None), slice(None), slice(h - n, h + rows + s), slice(h - w, h + cols + e))
        tiles[k][at] = src[at]
    if c["op"] not in ("step", "split"):
        return tiles, None, None
    size = max(1, dc.halo_elems(p, which))
    send = torch.zeros((len(_tiles(c)), size), dtype=a.dtype, device="cuda")
    if c["tile"] < 0:
        return tiles, send, send
    recv, off = torch.zeros_like(send), 0
    r = {"N": (h - bn, h), "S": (h + rows, h + rows + bs), "": (h, h + rows)}
    q = {"W": (h - bw, h), "E": (h + cols, h + cols + be), "": (h, h + cols)}
    for v, u in (("N", ""), ("S", ""), ("", "W"), ("", "E"), ("N", "W"), ("N", "E"), ("S", "W"), ("S", "E")):
        band = a[:, :, r[v][0]:r[v][1], q[u][0]:q[u][1]].reshape(-1)
        recv[0, off:off + band.numel()] = band
        off += band.numel()
    return tiles, send, recv


def prepare(c, seed):
    p = _problem(c)
    x, dy, w = _global(c, seed)
    Ht, Wt, Hot, Wot = dc.tile_dims(p)
    n, bordered = len(_tiles(c)), c["op"] not in ("step", "split")
    s = {"op": c["op"], "problem": p, "tile": c["tile"] if c["tile"] >= 0 else dc.DC_ALL_TILES, "w": w}
    s["x"], s["send_x"], s["recv_x"] = _layout(c, p, dc.DC_X, x, bordered)
    s["dy"], s["send_dy"], s["recv_dy"] = _layout(c, p, dc.DC_DY, dy, bordered)
    s["y"] = torch.empty((n, c["N"], c["K"], Hot, Wot), device="cuda")
    s["dx"] = torch.empty((n, c["N"], c["C"], Ht, Wt), device="cuda")
    s["dw"] = torch.empty((c["K"], c["C"], c["R"], c["R"]), device="cuda")
    s["workspace"] = torch.empty(max(16, dc.bwd_filter_workspace_bytes(p, s["tile"])), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    p, t, op = s["problem"], s["tile"], s["op"]
    if op == "fwd":
        dc.conv_fwd(p, t, s["x"], s["w"], s["y"])
        return {"y": s["y"]}
    if op in ("bwd", "train"):
        if op == "train":
            dc.conv_fwd(p, t, s["x"], s["w"], s["y"])
        dc.conv_bwd_filter(p, t, s["x"], s["dy"], s["dw"], 0, s["workspace"])
        dc.conv_bwd_data(p, t, s["dy"], s["w"], s["dx"])
        return {"dw": s["dw"], "dx": s["dx"], **({"y": s["y"]} if op == "train" else {})}
    split = op == "split"
    dc.halo_pack(p, t, dc.DC_X, s["x"], s["send_x"])
    if split:
        dc.conv_fwd_region(p, t, dc.DC_REGION_INTERIOR, s["x"], s["w"], s["y"])
    dc.halo_unpack(p, t, dc.DC_X, s["recv_x"], s["x"])
    dc.conv_fwd_region(p, t, dc.DC_REGION_BOUNDARY if split else dc.DC_REGION_ALL, s["x"], s["w"], s["y"])
    dc.halo_pack(p, t, dc.DC_DY, s["dy"], s["send_dy"])
    if split:
        dc.conv_bwd_data_region(p, t, dc.DC_REGION_INTERIOR, s["dy"], s["w"], s["dx"])
    dc.halo_unpack(p, t, dc.DC_DY, s["recv_dy"], s["dy"])
    dc.conv_bwd_filter(p, t, s["x"], s["dy"], s["dw"], 0, s["workspace"])
    dc.conv_bwd_data_region(p, t, dc.DC_REGION_BOUNDARY if split else dc.DC_REGION_ALL, s["dy"], s["w"], s["dx"])
    return {"y": s["y"], "dw": s["dw"], "dx": s["dx"], "x": s["x"], "dy": s["dy"], "send_x": s["send_x"],
            "send_dy": s["send_dy"]}


def exact(c, seed):
    """The three sums in 64 bits, tap by tap as matrix products per sample."""
    p = _problem(c)
    x, dy, w = (t.double() for t in _global(c, seed))
    Ht, Wt, Hot, Wot = dc.tile_dims(p)
    h, R, s, pad = p.halo, c["R"], c["stride"], c["R"] // 2
    ti, tj = (c["P"], c["Q"]) if c["tile"] < 0 else (1, 1)
    gh, gw, oh, ow = ti * Ht, tj * Wt, ti * Hot, tj * Wot
    y = torch.zeros((c["N"], c["K"], oh * ow), dtype=torch.float64, device="cuda")
    dw = torch.zeros((c["K"], c["C"], R, R), dtype=torch.float64, device="cuda")
    # output gradients reach input (i, j) from every output position within the margins
    dxf = torch.zeros((c["N"], c["C"], gh + 2 * R * (h + 1) * s, gw + 2 * R * (h + 1) * s), dtype=torch.float64, device="cuda")
    o = R * (h + 1) * s
    for n in range(c["N"]):
        own = dy[n, :, h:h + oh, h:h + ow].reshape(c["K"], -1)
        full = dy[n].reshape(c["K"], -1)
        for r in range(R):
            for q in range(R):
                xs = x[n, :, h - pad + r:, h - pad + q:][:, ::s, ::s][:, :oh, :ow].reshape(c["C"], -1)
                tap = w[:, :, r, q].contiguous()
                y[n] += tap @ xs
                dw[:, :, r, q] += own @ xs.t().contiguous()
                back = (tap.t().contiguous() @ full).view(c["C"], oh + 2 * h, ow + 2 * h)
                top, left = o - h * s - pad + r, o - h * s - pad + q
                dxf[n, :, top:top + s * (oh + 2 * h):s, left:left + s * (ow + 2 * h):s] += back
    y = y.view(c["N"], c["K"], oh, ow)
    dx = dxf[:, :, o:o + gh, o:o + gw]
    tiles = lambda a, rows, cols: torch.stack(  # noqa: E731
        [a[:, :, i * rows:(i + 1) * rows, j * cols:(j + 1) * cols] for i in range(ti) for j in range(tj)])
    got = {"y": tiles(y, Hot, Wot), "dw": dw, "dx": tiles(dx, Ht, Wt)}
    if c["op"] == "fwd":
        return {"y": got["y"]}
    if c["op"] == "bwd":
        return {"dw": got["dw"], "dx": got["dx"]}
    if c["op"] == "train":
        return got
    return {**got, "x": None, "dy": None, "send_x": None, "send_dy": None}
