"""What this library is timed on: calls of its public entry points, at the sizes
and with the options a user's program has.

Every case has a ``kind``, the calls one pass makes:

    step     path and tile lists built anew, then attention with the reordering
             fused in (a program that meets a new grid on each call)
    hilbert  the one-launch forward on 2^k x 2^k grids
    fwd      attention forward on tensors in sequence order, lists built before
    composed gather of q, k, v, attention, scatter of the output
    rpb      forward with the global relative position bias
    train    forward and backward with the reordering fused in
    train_seq  forward and backward on tensors in sequence order
    layer    QKV projection, attention, output projection

and the tensors' sizes ([B, heads, H * W, d]), type, pattern and tile. Inputs are
N(0, 1) draws (projection weights N(0, 0.02^2)), as in ``workloads``.
"""
from __future__ import annotations

import math

import torch

import paper_2511_05832_amd as hla

HILBERT = ("hilbert_window", "hilbert_slide", "hilbert_neighborhood", "hilbert_shifted_window")


def _case(kind, B, heads, H, W, d, pattern, p0, p1=0, dtype="bf16", tile_m=128, name=None):
    c = dict(kind=kind, B=B, heads=heads, H=H, W=W, d=d, pattern=pattern, p0=p0, p1=p1,
             dtype=dtype, tile_m=tile_m)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: one fp32 head on a 32x32 grid, path and lists included.
        # Launches and latency are what it costs.
        _case("step", 1, 1, 32, 32, 32, "hilbert_window", 64, dtype="f32", tile_m=64,
              name="step_f32_window_32"),
        # A small bf16 inference call: too few workgroups to fill the chip.
        _case("hilbert", 2, 4, 64, 64, 64, "hilbert_slide", 128, name="hilbert_band_64"),
        # The headline workload: Hilbert window attention on a 128x128 feature map.
        _case("hilbert", 4, 8, 128, 128, 64, "hilbert_window", 256, name="hilbert_window_128"),
        # Long sequence (65,536 tokens), wide band: bound by arithmetic.
        _case("hilbert", 1, 8, 256, 256, 64, "hilbert_slide", 512, name="hilbert_band_256"),
        # The row-major comparison pattern (33x33 slide): every tile is partial.
        # The largest call.
        _case("fwd", 1, 8, 256, 256, 64, "rowmajor_slide", 16, 16, name="rowmajor_slide_256"),
        # A grid that is no power of two, shifted windows, 32-wide heads, with the
        # reordering as separate calls (a model that keeps Hilbert order in between).
        _case("composed", 2, 8, 160, 160, 32, "hilbert_shifted_window", 256, 128,
              name="composed_shifted_160"),
        # Forward with the position bias of a hierarchical window transformer.
        _case("rpb", 4, 8, 128, 128, 64, "hilbert_window", 256, name="rpb_window_128"),
        # Training at the headline size.
        _case("train", 4, 8, 128, 128, 64, "hilbert_window", 256, name="train_window_128"),
        # Training on the 56x56 feature map of an image backbone: ragged last tiles.
        _case("train", 16, 2, 56, 56, 64, "hilbert_neighborhood", 289, name="train_neighborhood_56"),
        # Training in fp32 throughout (verification runs, small models).
        _case("train_seq", 2, 4, 64, 64, 64, "hilbert_slide", 128, dtype="f32",
              name="train_f32_band_64"),
        # A transformer layer's attention block at 192 channels, in grid order.
        _case("layer", 16, 6, 64, 64, 32, "hilbert_slide", 64, tile_m=64, name="layer_192"),
        # The same at 512 channels on a later, smaller stage's grid.
        _case("layer", 16, 8, 32, 32, 64, "hilbert_slide", 64, tile_m=64, name="layer_512"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("step", "hilbert", "fwd", "composed", "rpb", "train", "train_seq", "layer"))
    if kind == "hilbert" or (kind == "layer" and rng.random() < 0.7):
        H = W = rng.choice((16, 32, 64, 128, 256))
    elif kind == "layer":
        H, W = _log_int(rng, 14, 80), _log_int(rng, 14, 80)
    elif rng.random() < 0.3:
        H = W = rng.choice((32, 64, 128))
    else:
        H, W = _log_int(rng, 16, 160), _log_int(rng, 16, 160)
    N = H * W
    d = rng.choice((32, 64))
    dtype = "f32" if kind in ("step", "fwd", "train", "train_seq") and rng.random() < 0.4 else "bf16"
    tile_m = rng.choice((64, 128))
    names = HILBERT
    if kind in ("fwd", "train_seq", "rpb") and rng.random() < 0.5:
        names = ("rowmajor_window", "rowmajor_slide", "rowmajor_neighborhood")
    pattern = rng.choice(names)
    p1 = 0
    if pattern == "hilbert_window":
        p0 = rng.choice((49, 64, 144, 256, 1024))
    elif pattern == "hilbert_slide":
        p0 = _log_int(rng, 24, 512)
    elif pattern == "hilbert_neighborhood":
        p0 = min(N, rng.choice((49, 81, 169, 289, 529)))
    elif pattern == "hilbert_shifted_window":
        p0 = rng.choice((64, 144, 256))
        p1 = p0 // 2
    elif pattern == "rowmajor_window":
        p0 = p1 = rng.choice((7, 8, 16))
    elif pattern == "rowmajor_slide":
        p0 = p1 = rng.randint(3, 12)
    else:
        p0 = p1 = min(H, W, rng.choice((7, 13, 17)))
    # heads and batch: up to half a million rows (a sixteenth of that in fp32)
    rows = _log_int(rng, 1 << 12, 1 << (15 if dtype == "f32" else 19))
    if kind == "layer":
        heads = rng.choice((2, 4, 6, 8, 12, 16) if d == 32 else (1, 2, 3, 4, 6, 8))
        rows = min(rows, 1 << 16) * heads
    else:
        heads = rng.choice((1, 2, 3, 4, 8))
    B = max(1, min(64, rows // (heads * N)))
    return _case(kind, B, heads, H, W, d, pattern, p0, p1, dtype, tile_m)


def _torch_dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _inputs(c, seed):
    """The random tensors of a case, in the order they are drawn."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = _torch_dtype(c)
    B, h, d, N = c["B"], c["heads"], c["d"], c["H"] * c["W"]

    def normal(*shape, std=1.0, dtype=dt):
        return (torch.randn(shape, generator=g, device="cuda") * std).to(dtype)

    if c["kind"] == "layer":
        C = h * d
        return dict(x=normal(B, N, C), w_qkv=normal(3 * C, C, std=0.02), w_proj=normal(C, C, std=0.02))
    t = {n: normal(B, h, N, d) for n in ("q", "k", "v")}
    if c["kind"] in ("train", "train_seq"):
        t["dout"] = normal(B, h, N, d)
    if c["kind"] == "rpb":
        t["rpb"] = normal(h, 2 * c["H"] - 1, 2 * c["W"] - 1, dtype=torch.float32)
    return t


def _pattern(c):
    return (c["pattern"], c["H"], c["W"], c["p0"], c["p1"])


def _one_launch(c):
    """Whether a layer's attention can take the one-launch entry point."""
    return c["H"] == c["W"] and c["H"] & (c["H"] - 1) == 0


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case, pattern=_pattern(case))
    kind = case["kind"]
    if kind == "hilbert" or (kind == "layer" and _one_launch(case)):
        return s   # the order and the lists are computed in the kernel
    if kind == "step":
        n = case["H"] * case["W"]
        s["order"] = torch.empty(n, dtype=torch.int32, device="cuda")
        s["mask"] = hla.BlockMask(s["pattern"], case["tile_m"], 64, totals=False)
        return s
    if case["pattern"] in HILBERT:
        s["order"] = hla.hilbert_perm(case["H"], case["W"])[0]
    else:
        s["order"] = torch.arange(case["H"] * case["W"], dtype=torch.int32, device="cuda")
    s["mask"] = hla.build_block_mask(s["pattern"], case["tile_m"], 64,
                                     columns=kind in ("train", "train_seq"))
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "step":
        s["mask"].build_with_path(s["order"])
        out, lse = hla.attn_fwd_perm(s["q"], s["k"], s["v"], s["order"], s["mask"])
        return dict(out=out, lse=lse, order=s["order"], n_full=s["mask"].n_full, n_part=s["mask"].n_part)
    if kind == "hilbert":
        out, lse = hla.attn_fwd_hilbert(s["q"], s["k"], s["v"], s["pattern"], c["tile_m"], 64)
        return dict(out=out, lse=lse)
    if kind == "fwd":
        out, lse = hla.attn_fwd(s["q"], s["k"], s["v"], s["mask"])
        return dict(out=out, lse=lse)
    if kind == "composed":
        q, k, v = (hla.gather(s[n], s["order"]) for n in ("q", "k", "v"))
        out, lse = hla.attn_fwd(q, k, v, s["mask"])
        return dict(out=hla.scatter(out, s["order"]), lse=lse)
    if kind == "rpb":
        out, lse = hla.attn_fwd_rpb(s["q"], s["k"], s["v"], s["order"], s["rpb"], s["mask"])
        return dict(out=out, lse=lse)
    if kind == "train":
        out, lse = hla.attn_fwd_perm(s["q"], s["k"], s["v"], s["order"], s["mask"])
        dq, dk, dv = hla.attn_bwd_perm(s["q"], s["k"], s["v"], out, s["dout"], lse, s["order"], s["mask"])
        return dict(out=out, lse=lse, dq=dq, dk=dk, dv=dv)
    if kind == "train_seq":
        out, lse = hla.attn_fwd(s["q"], s["k"], s["v"], s["mask"])
        dq, dk, dv = hla.attn_bwd(s["q"], s["k"], s["v"], out, s["dout"], lse, s["mask"])
        return dict(out=out, lse=lse, dq=dq, dk=dk, dv=dv)
    if _one_launch(c):   # grid order in and out, the reordering inside the attention
        q, k, v = hla.qkv_proj(s["x"], s["w_qkv"], c["heads"])
        o, _ = hla.attn_fwd_hilbert(q, k, v, s["pattern"], c["tile_m"], 64, with_lse=False)
        return dict(y=hla.out_proj(o, s["w_proj"]))
    # other grids: the reordering fused into the projections
    q, k, v = hla.qkv_proj(s["x"], s["w_qkv"], c["heads"], order=s["order"])
    o, _ = hla.attn_fwd(q, k, v, s["mask"], with_lse=False)
    return dict(y=hla.out_proj(o, s["w_proj"], order=s["order"]))


# ---------------------------------------------------------------------------
# Costs and reference results, in plain torch.

def _axis(kind, x, y, size, extent):
    """One axis of a row-major pattern: whether row (column) x may attend y."""
    if kind == "rowmajor_window":
        return x // size == y // size
    if kind == "rowmajor_slide":
        return (x - y).abs() <= size
    start = (x - size // 2).clamp(0, extent - size)
    return (y >= start) & (y < start + size)


def _allowed(c, i, j):
    """Whether sequence position i may attend position j (broadcast index tensors)."""
    p, p0, p1, H, W = c["pattern"], c["p0"], c["p1"], c["H"], c["W"]
    if p == "hilbert_window":
        return i // p0 == j // p0
    if p == "hilbert_slide":
        return (i - j).abs() <= p0
    if p == "hilbert_neighborhood":
        return _axis(p, i, j, p0, H * W)
    if p == "hilbert_shifted_window":
        return (i + p0 - p1) // p0 == (j + p0 - p1) // p0
    return _axis(p, i // W, j // W, p0, H) & _axis(p, i % W, j % W, p1, W)


def _span(c, lo, hi):
    """A range of positions [a, b) that holds every key of the queries lo .. hi - 1."""
    p, p0, W, N = c["pattern"], c["p0"], c["W"], c["H"] * c["W"]
    reach = p0 if p in HILBERT else (p0 + 1) * W
    return max(0, lo - reach), min(N, hi + reach)


def _pairs(c):
    """Query-key pairs the pattern allows in one (b, head) slice."""
    N, total = c["H"] * c["W"], 0
    if c["pattern"] not in HILBERT:
        n = [int(_axis(c["pattern"], torch.arange(e)[:, None], torch.arange(e)[None], k, e).sum())
             for e, k in ((c["H"], c["p0"]), (c["W"], c["p1"]))]
        return n[0] * n[1]
    step = max(64, min(N, 1 << 11))
    for lo in range(0, N, step):
        hi = min(N, lo + step)
        a, b = _span(c, lo, hi)
        total += int(_allowed(c, torch.arange(lo, hi)[:, None], torch.arange(a, b)[None]).sum())
    return total


def work(case):
    c = case
    N, d, bh = c["H"] * c["W"], c["d"], c["B"] * c["heads"]
    es = 4 if c["dtype"] == "f32" else 2
    t = bh * N * d * es                # one q-shaped tensor
    pair = 2.0 * d * bh * _pairs(c)    # one product over the allowed pairs
    kind = c["kind"]
    if kind == "layer":
        C = c["heads"] * d
        return {"bytes": 2 * c["B"] * N * C * es + 4 * C * C * es,
                "flops": 2.0 * c["B"] * N * 4 * C * C + 2 * pair}
    if kind in ("train", "train_seq"):  # q, k, v, dout in; out, lse, dq, dk, dv out
        return {"bytes": 8 * t + 4 * bh * N, "flops": 7 * pair}
    table = 4 * c["heads"] * (2 * c["H"] - 1) * (2 * c["W"] - 1) if kind == "rpb" else 0
    return {"bytes": 4 * t + 4 * bh * N + table, "flops": 2 * pair}


def tolerance(case):
    # Two correct implementations at the same precision. Measured against float64:
    # fp32 outputs 2e-7 to 5e-7 off, bf16 outputs 2.2e-3 to 2.5e-3 (the layers
    # 3.3e-3: bf16 rounds weights, score gradients and every result to 2^-9).
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-4}
    return {"rel": 1e-2, "max": 0.2}


def _hilbert_order(H, W):
    """Row-major ids along the curve on the smallest 2^k square holding the grid,
    cells outside the grid left out (textbook index-to-cell loop, vectorised)."""
    side = 1
    while side < max(H, W):
        side *= 2
    t = torch.arange(side * side, dtype=torch.int64)
    x, y = torch.zeros_like(t), torch.zeros_like(t)
    s = 1
    while s < side:
        rx = 1 & (t // 2)
        ry = 1 & (t ^ rx)
        flip = (ry == 0) & (rx == 1)
        x, y = torch.where(flip, s - 1 - x, x), torch.where(flip, s - 1 - y, y)
        x, y = torch.where(ry == 0, y, x), torch.where(ry == 0, x, y)
        x, y = x + s * rx, y + s * ry
        t = t // 4
        s *= 2
    keep = (x < W) & (y < H)
    return (y[keep] * W + x[keep]).cuda()


def _attention(c, q, k, v, scale, bias=None, dout=None):
    """Masked softmax attention in float64 on tensors in sequence order, a chunk of
    query rows at a time against the keys in its reach; gradients if dout is given.
    bias(i, j): the score bias per head of positions i, j."""
    B, h, N, d = q.shape
    q, k, v = (t.double().reshape(B * h, N, d) for t in (q, k, v))
    out, lse = torch.empty_like(q), torch.empty((B * h, N), dtype=torch.float64, device=q.device)
    if dout is not None:
        dout = dout.double().reshape(B * h, N, d)
        dq, dk, dv = (torch.zeros_like(q) for _ in range(3))
    step = max(64, min(1024, (1 << 25) // (B * h * 512)))
    for lo in range(0, N, step):
        hi = min(N, lo + step)
        a, b = _span(c, lo, hi)
        i = torch.arange(lo, hi, device=q.device)[:, None]
        j = torch.arange(a, b, device=q.device)[None]
        kt, vt = k[:, a:b], v[:, a:b]
        s = torch.matmul(q[:, lo:hi], kt.transpose(1, 2).contiguous()) * scale
        if bias is not None:
            s = (s.reshape(B, h, hi - lo, b - a) + bias(i, j)).reshape(s.shape)
        s = s.masked_fill(~_allowed(c, i, j), -math.inf)
        lse[:, lo:hi] = torch.logsumexp(s, -1)
        p = torch.exp(s - lse[:, lo:hi, None])
        out[:, lo:hi] = torch.matmul(p, vt)
        if dout is not None:
            g = dout[:, lo:hi]
            dp = torch.matmul(g, vt.transpose(1, 2).contiguous())
            ds = p * (dp - (g * out[:, lo:hi]).sum(-1, keepdim=True)) * scale
            dq[:, lo:hi] = torch.matmul(ds, kt)
            dk[:, a:b] += torch.matmul(ds.transpose(1, 2).contiguous(), q[:, lo:hi])
            dv[:, a:b] += torch.matmul(p.transpose(1, 2).contiguous(), g)
    shape = (B, h, N, d)
    got = dict(out=out.reshape(shape), lse=lse.reshape(B, h, N))
    if dout is not None:
        got.update(dq=dq.reshape(shape), dk=dk.reshape(shape), dv=dv.reshape(shape))
    return got


def exact(case, seed):
    c, kind = case, case["kind"]
    t = _inputs(c, seed)
    N = c["H"] * c["W"]
    scale = 1.0 / math.sqrt(c["d"])
    order = (_hilbert_order(c["H"], c["W"]) if c["pattern"] in HILBERT
             else torch.arange(N, device="cuda"))

    def back(x):       # sequence order -> grid order
        y = torch.empty_like(x)
        y[:, :, order] = x
        return y

    if kind == "layer":
        B, h, d = c["B"], c["heads"], c["d"]
        qkv = t["x"].double()[:, order] @ t["w_qkv"].double().T
        q, k, v = qkv.reshape(B, N, 3, h, d).permute(2, 0, 3, 1, 4)
        o = _attention(c, q, k, v, scale)["out"]
        y = o.permute(0, 2, 1, 3).reshape(B, N, h * d) @ t["w_proj"].double().T
        res = torch.empty_like(y)
        res[:, order] = y
        return dict(y=res)
    if kind in ("fwd", "train_seq"):
        return _attention(c, t["q"], t["k"], t["v"], scale, dout=t.get("dout"))
    if kind == "rpb":
        H, W, table = c["H"], c["W"], t["rpb"].double()
        row, col = order // W, order % W

        def bias(i, j):
            return table[:, row[i] - row[j] + H - 1, col[i] - col[j] + W - 1]
        return _attention(c, t["q"], t["k"], t["v"], scale, bias=bias)
    # grid order in and out
    seq = {n: x[:, :, order] for n, x in t.items()}
    got = _attention(c, seq["q"], seq["k"], seq["v"], scale, dout=seq.get("dout"))
    if kind == "composed":         # lse stays in sequence order
        return dict(out=back(got["out"]), lse=got["lse"])
    got = {n: back(x) for n, x in got.items()}
    if kind == "step":
        got.update(order=None, n_full=None, n_part=None)
    return got
