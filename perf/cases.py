"""The timed cases of the per-rank tensor-parallel linear layer: what one rank's program has it do.

A case is one pass of one rank's share through the public entry points, on blocks that are already in
device memory.  `kind` says which calls the pass makes:

  forward    one forward product with bias and erf-GeLU, nothing saved (inference);
  train      forward with the pre-activation saved, then one backward call: own dA, bias gradient, dX, dW;
  second     the down-projection of an MLP: bias-only forward with fp32 output, bias gradient, and a
             backward whose dX takes GeLU' of the previous layer in its epilogue, and dW;
  partials   forward, own dA, bias gradient, and both backward products as partials for other owners;
  gathered   3D at the gathered local shape: forward partial, bias + GeLU on the rank's own chunk, dX, dW;
  mlp1d_fwd  the 1D feed-forward, forward only: column-cut layer, row-cut layer, bias on the sum;
  mlp1d      the same with backward: six products, the bias on the sum and the first layer's bias gradient.

M, H, F are the full (unpartitioned) layer; mode, q, d, p, ri, rj, rk the rank grid and this rank;
steps 0 is the exact share, a positive count a prefix of the sum; f32 asks for fp32 Y and dX where the
caller chooses the type (dW, db and every partial are fp32 by definition).
"""
from __future__ import annotations

import math

import torch

import paper_2110_14883_amd as T

_MODES = {"1d": T.MODE_1D_COL, "2d": T.MODE_2D, "2.5d": T.MODE_2P5D, "3d": T.MODE_3D, "3d_gathered": T.MODE_3D_GATHERED}
_BF, _F32 = torch.bfloat16, torch.float32


def _case(kind, mode, M, H, F, q=1, d=1, p=1, ri=0, rj=0, rk=0, steps=0, f32=False, **more):
    return dict(kind=kind, mode=mode, q=q, d=d, p=p, ri=ri, rj=rj, rk=rk, M=M, H=H, F=F, steps=steps, f32=f32, **more)


def listed():
    return [
        # the smallest calls: launches and the host path count
        # a 2 x 2 SUMMA rank's up-projection of 256 tokens, fp32 output: the smallest benchmark share
        _case("forward", "2d", 256, 1024, 4096, q=2, f32=True, name="2d_forward_small"),
        # token-by-token decoding of a batch of 16 through the 1D feed-forward of the 4096 / 16384 layer: streams the weights
        _case("mlp1d_fwd", "1d", 16, 4096, 16384, p=4, ri=1, name="1d_decode"),
        # a small training step with every extent ragged
        _case("train", "2d", 600, 272, 656, q=2, ri=1, name="2d_train_small_ragged"),
        # ordinary ones
        # odd extents and a 3 x 3 grid, fp32 outputs
        _case("train", "2d", 3 * 1111, 3 * 520, 3 * 2056, q=3, ri=2, rj=1, f32=True, name="2d_train_odd_f32"),
        # one layer of the two-linear range test (hidden 2048, batch 32 of 512 tokens, 4 GPUs)
        _case("train", "2d", 16384, 2048, 2048, q=2, ri=1, name="2d_train_h2048"),
        # the benchmark's 2D share, its second linear, and its backward in the other SUMMA form
        _case("train", "2d", 8192, 8192, 32768, q=4, ri=1, rj=2, name="2d_train_q4"),
        _case("second", "2d", 8192, 32768, 8192, q=4, ri=1, rj=2, name="2d_second_linear_q4"),
        _case("partials", "2d", 8192, 8192, 32768, q=4, ri=1, rj=2, name="2d_partials_q4"),
        # ViT-style MLP on a 2 x 2 x 2 grid: 32896 ragged token rows, narrow blocks
        _case("train", "2.5d", 131584, 1280, 5120, q=2, d=2, ri=1, rk=1, name="2.5d_train_vit"),
        # the largest
        # the 1D feed-forward of 16384 tokens, six products
        _case("mlp1d", "1d", 16384, 4096, 16384, p=4, ri=1, name="1d_train"),
        # a GPT-3-175B-shaped MLP on the 2 x 2 x 2 cube: one local product per pass, and the gathered local shape
        _case("train", "3d", 16384, 12288, 49152, p=2, ri=1, rk=1, steps=1, name="3d_train"),
        _case("gathered", "3d_gathered", 16384, 12288, 49152, p=2, ri=1, rk=1, name="3d_gathered"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["forward", "train", "train", "second", "partials", "gathered", "mlp1d_fwd", "mlp1d"])
    if kind.startswith("mlp1d"):
        mode, g = "1d", dict(p=rng.choice([1, 2, 4, 8]))
        g["ri"] = rng.randrange(g["p"])
    elif kind == "gathered":
        mode, g = "3d_gathered", dict(p=2, ri=rng.randrange(2), rj=rng.randrange(2), rk=rng.randrange(2))
    else:
        mode = rng.choice(["2d", "2.5d"] if kind == "partials" else ["2d", "2.5d", "3d"])
        if mode == "3d":
            g = dict(p=2, ri=rng.randrange(2), rj=rng.randrange(2), rk=rng.randrange(2))
        else:
            q = rng.choice([2, 3, 4])
            g = dict(q=q, ri=rng.randrange(q), rj=rng.randrange(q))
            if mode == "2.5d":
                g.update(d=2, rk=rng.randrange(2))
    # extents of the rank's own block: tokens m, input features h, output features f
    m = int(_log(rng, 1, 8192) if kind.endswith("fwd") or kind == "forward" else _log(rng, 64, 32896))
    h = 8 * int(_log(rng, 16, 768))
    f = 8 * int(min(3072, _log(rng, h / 16, h / 2)))
    if rng.random() < 0.5:                       # half of the widths are multiples of 128, as layer widths mostly are
        h, f = max(128, h // 128 * 128), max(128, f // 128 * 128)
    if kind == "second":
        h, f = f, h
    c = _case(kind, mode, 0, 0, 0, f32=rng.random() < 0.25, **g)
    rc, kc, cc = _chunks(c)
    while True:
        mm = max(1, m)
        c.update(M=mm * rc * (2 if kind == "gathered" else 1), H=h * kc, F=f * cc)
        if mm == 1 or work(c)["flops"] <= 4e12:
            return c
        m //= 2


# ------------------------------------------------------------------ which blocks a case reads and writes
def _grid(c):
    return T.Grid(_MODES[c["mode"]], q=c["q"], d=c["d"], p=c["p"], ri=c["ri"], rj=c["rj"], rk=c["rk"])


def _chunks(c):
    """Row chunks of X and Y, column chunks of X, column chunks of W and Y."""
    q, d, p = c["q"], c["d"], c["p"]
    return {"1d": (1, 1, p), "2d": (q, q, q), "2.5d": (q * d, q, q), "3d": (p * p, p, p), "3d_gathered": (p, p, p)}[c["mode"]]


def _layout(c):
    """The pass's blocks: `read` maps (tensor, row chunk, column chunk) to (rows, columns), each block once;
    `rows`, `cols` and the other lists say which of them the calls take, in step order; `out` are the
    shapes and types of what it returns."""
    kind, grid, dims = c["kind"], _grid(c), (c["M"], c["H"], c["F"])
    rc, kc, cc = _chunks(c)
    m, h, f = c["M"] // rc, c["H"] // kc, c["F"] // cc
    io = _F32 if c["f32"] else _BF
    L = dict(grid=grid, dims=dims, m=m, h=h, f=f, read={}, bias=[f])
    read = L["read"]

    def use(tensor, row, col, shape):
        read[(tensor, row, col)] = shape
        return (tensor, row, col)

    if kind.startswith("mlp1d"):
        L["x"], L["w1"], L["w2"] = use("X", 0, 0, (m, h)), use("W1", 0, grid.ri, (h, f)), use("W2", grid.ri, 0, (f, h))
        L["bias"] = [f, h]
        L["out"] = dict(sum=((m, h), _F32), y=((m, h), io))
        L["scratch"] = dict(z=((m, f), _BF))
        if kind == "mlp1d":
            L["g"] = use("G", 0, 0, (m, h))
            L["out"].update(z=((m, f), _BF), a=((m, f), _BF), da=((m, f), _BF), dw2=((f, h), _F32), dx=((m, h), _F32),
                            dw1=((h, f), _F32), db1=((f,), _F32))
            L["scratch"] = {}
        return L
    L["scratch"] = {}
    fw = T.tp_block_map(grid, dims, T.PASS_FWD)
    if kind == "gathered":
        p = c["p"]
        L["x"], L["w"] = use("X", *fw["a"][0], (m, h)), use("W", *fw["b"][0], (h, f))
        L["g"] = use("dA", *T.tp_block_map(grid, dims, T.PASS_DX)["a"][0], (m, f))
        L["out"] = dict(sum=((m, f), _F32), y=((m // p, f), io), pre=((m // p, f), _BF), dx=((m, h), _F32), dw=((h, f), _F32))
        return L
    n = c["steps"] or fw["n_steps"]
    L["n"] = n
    L["xs"] = [use("X", *fw["a"][k], (m, h)) for k in range(n)]
    L["ws"] = [use("W", *fw["b"][k], (h, f)) for k in range(n)]
    own = fw["out"]
    L["out"] = dict(y=((m, f), _F32 if kind == "second" else io))
    if kind == "forward":
        return L
    L["g"] = use("G", *own, (m, f))
    if kind != "second":
        L["out"].update(pre=((m, f), _BF), da=((m, f), _BF))
    L["out"].update(db=((f,), _F32))
    if kind == "partials":
        dx, dw = T.tp_partials_map(grid, dims, T.PASS_DX_PARTIALS), T.tp_partials_map(grid, dims, T.PASS_DW_PARTIALS)
        L["wx"] = [use("W", *b, (h, f)) for b in dx["other"]]
        L["xw"] = [use("X", *b, (m, h)) for b in dw["other"]]
        L["out"].update({"dx%d" % k: ((m, h), _F32) for k in range(len(L["wx"]))})
        L["out"].update({"dw%d" % k: ((h, f), _F32) for k in range(len(L["xw"]))})
        return L
    dx, dw = T.tp_block_map(grid, dims, T.PASS_DX), T.tp_block_map(grid, dims, T.PASS_DW)
    # a prefix of the sum keeps the rank's own term
    ox = sorted(range(dx["n_steps"]), key=lambda k: bool(c["steps"]) and dx["a"][k] != own)[:n]
    ow = sorted(range(dw["n_steps"]), key=lambda k: bool(c["steps"]) and dw["b"][k] != own)[:n]
    peer = "G" if kind == "second" else "dA"     # peers' blocks: the upstream gradient itself, or their dA
    L["rows"] = [None if dx["a"][k] == own else use(peer, *dx["a"][k], (m, f)) for k in ox]
    L["wx"] = [use("W", *dx["b"][k], (h, f)) for k in ox]
    L["xw"] = [use("X", *dw["a"][k], (m, h)) for k in ow]
    L["cols"] = [None if dw["b"][k] == own else use(peer, *dw["b"][k], (m, f)) for k in ow]
    if kind == "second":
        L["a1"] = use("A1", *dx["out"], (m, h))
    L["out"].update(dx=((m, h), _BF if kind == "second" else io), dw=((h, f), _F32))
    return L


# ------------------------------------------------------------------ inputs
def _block(gen, tensor, shape, dims):
    def normal(std):
        return torch.randn(shape, generator=gen, device="cuda", dtype=_BF).mul_(std)

    if tensor in ("X", "G"):
        return normal(1.0)
    if tensor in ("W", "W1", "W2"):
        return normal(0.02)
    a = normal(0.02 * math.sqrt(dims[1]))        # a pre-activation has the spread of X W
    if tensor == "A1":
        return a
    a = a.float()                                # a peer's dA = upstream gradient times GeLU'(pre-activation)
    slope = 0.5 * (1 + torch.erf(a * math.sqrt(0.5))) + a * torch.exp(-0.5 * a * a) / math.sqrt(2 * math.pi)
    return (normal(1.0) * slope).to(_BF)


def prepare(case, seed):
    """Blocks, outputs and workspace in device memory, as a rank's program holds them between passes."""
    L = _layout(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    blocks = {key: _block(gen, key[0], shape, L["dims"]) for key, shape in L["read"].items()}
    s = {k: v for k, v in L.items() if k not in ("read", "bias", "out", "scratch")}
    for name in ("x", "w", "w1", "w2", "g", "a1"):
        if name in s:
            s[name] = blocks[s[name]]
    for name in ("xs", "ws", "wx", "xw", "rows", "cols"):
        if name in s:
            s[name] = [None if key is None else blocks[key] for key in s[name]]
    s["bias"] = [torch.randn((n,), generator=gen, device="cuda", dtype=_BF).mul_(0.02) for n in L["bias"]]
    s["out"] = {k: torch.empty(shape, dtype=dt, device="cuda") for k, (shape, dt) in L["out"].items()}
    s["scratch"] = {k: torch.empty(shape, dtype=dt, device="cuda") for k, (shape, dt) in L["scratch"].items()}
    kind, (M, H, F), g = case["kind"], L["dims"], L["grid"]
    s["kind"] = kind
    sizes = [256]
    if kind.startswith("mlp1d"):
        s["g1"], s["g2"] = g, T.Grid(T.MODE_1D_ROW, p=g.p, ri=g.ri)
        s["d2"] = (M, F, H)
        for ps in (T.PASS_FWD, T.PASS_DX, T.PASS_DW) if kind == "mlp1d" else (T.PASS_FWD,):
            sizes += [T.tp_linear_workspace_size(s["g1"], s["dims"], ps), T.tp_linear_workspace_size(s["g2"], s["d2"], ps)]
    else:
        passes = {"forward": (T.PASS_FWD,), "partials": (T.PASS_FWD, T.PASS_DX_PARTIALS, T.PASS_DW_PARTIALS)}
        sizes += [T.tp_linear_workspace_size(g, s["dims"], ps) for ps in passes.get(kind, (T.PASS_FWD, T.PASS_DX, T.PASS_DW))]
    if kind in ("second", "partials", "mlp1d"):
        sizes.append(T.tp_bias_grad_workspace_size(L["m"], L["f"]))
    s["work"] = torch.empty(max(sizes), dtype=torch.uint8, device="cuda")
    if kind == "gathered":
        rows, at = L["m"] // case["p"], case["rk"] * (L["m"] // case["p"])
        s["chunk"] = s["out"]["sum"][at:at + rows]
    if kind in ("train", "second"):
        own = s["out"]["da"] if kind == "train" else s["g"]
        s["own_dx"] = next((i for i, b in enumerate(s["rows"]) if b is None), -1)
        s["own_dw"] = next((i for i, b in enumerate(s["cols"]) if b is None), -1)
        s["rows"] = [own if b is None else b for b in s["rows"]]
        s["cols"] = [own if b is None else b for b in s["cols"]]
    return s


def run(s):
    kind, o, ws = s["kind"], s["out"], s["work"]
    return _RUN[kind](s, o, ws)


# ------------------------------------------------------------------ the passes
def _forward(s, o, ws):
    T.tp_linear_fwd(s["grid"], s["dims"], s["n"], s["xs"], s["ws"], s["bias"][0], T.EPI_BIAS_GELU, o["y"], None, ws)
    return o


def _train(s, o, ws):
    T.tp_linear_fwd(s["grid"], s["dims"], s["n"], s["xs"], s["ws"], s["bias"][0], T.EPI_BIAS_GELU, o["y"], o["pre"], ws)
    T.tp_linear_bwd(s["grid"], s["dims"], s["n"], s["n"], dy_own=s["g"], preact_own=o["pre"], da_row_blocks=s["rows"],
                    w_blocks_dx=s["wx"], x_blocks_dw=s["xw"], da_col_blocks=s["cols"], own_slot_dx=s["own_dx"],
                    own_slot_dw=s["own_dw"], dx=o["dx"], dw=o["dw"], da_own_out=o["da"], db=o["db"], workspace=ws)
    return o


def _second(s, o, ws):
    T.tp_linear_fwd(s["grid"], s["dims"], s["n"], s["xs"], s["ws"], s["bias"][0], T.EPI_BIAS, o["y"], None, ws)
    T.tp_bias_grad(s["g"], o["db"], workspace=ws)
    T.tp_linear_bwd(s["grid"], s["dims"], s["n"], s["n"], da_row_blocks=s["rows"], w_blocks_dx=s["wx"], x_blocks_dw=s["xw"],
                    da_col_blocks=s["cols"], dgelu_preact=s["a1"], dx=o["dx"], dw=o["dw"], workspace=ws)
    return o


def _partials(s, o, ws):
    T.tp_linear_fwd(s["grid"], s["dims"], s["n"], s["xs"], s["ws"], s["bias"][0], T.EPI_BIAS_GELU, o["y"], o["pre"], ws)
    T.tp_dgelu(s["g"], o["pre"], o["da"])
    T.tp_bias_grad(o["da"], o["db"], workspace=ws)
    T.tp_linear_bwd_partials(s["grid"], s["dims"], o["da"], s["wx"], [o["dx%d" % k] for k in range(len(s["wx"]))],
                             s["xw"], [o["dw%d" % k] for k in range(len(s["xw"]))], ws)
    return o


def _gathered(s, o, ws):
    T.tp_linear_fwd(s["grid"], s["dims"], 1, [s["x"]], [s["w"]], None, T.EPI_NONE, o["sum"], None, ws)
    T.tp_bias_act(s["chunk"], s["bias"][0], T.EPI_BIAS_GELU, o["y"], o["pre"])
    T.tp_linear_bwd(s["grid"], s["dims"], 1, 1, da_row_blocks=[s["g"]], w_blocks_dx=[s["w"]], x_blocks_dw=[s["x"]],
                    da_col_blocks=[s["g"]], dx=o["dx"], dw=o["dw"], workspace=ws)
    return o


def _mlp1d_fwd(s, o, ws):
    z = o.get("z", s["scratch"].get("z"))
    T.tp_linear_fwd(s["g1"], s["dims"], 1, [s["x"]], [s["w1"]], s["bias"][0], T.EPI_BIAS_GELU, z, o.get("a"), ws)
    T.tp_linear_fwd(s["g2"], s["d2"], 1, [z], [s["w2"]], None, T.EPI_NONE, o["sum"], None, ws)
    T.tp_bias_act(o["sum"], s["bias"][1], T.EPI_BIAS, o["y"])
    return o


def _mlp1d(s, o, ws):
    _mlp1d_fwd(s, o, ws)
    T.tp_linear_bwd(s["g2"], s["d2"], 1, 1, da_row_blocks=[s["g"]], w_blocks_dx=[s["w2"]], x_blocks_dw=[o["z"]],
                    da_col_blocks=[s["g"]], dgelu_preact=o["a"], dx=o["da"], dw=o["dw2"], workspace=ws)
    T.tp_bias_grad(o["da"], o["db1"], workspace=ws)
    T.tp_linear_bwd(s["g1"], s["dims"], 1, 1, da_row_blocks=[o["da"]], w_blocks_dx=[s["w1"]], x_blocks_dw=[s["x"]],
                    da_col_blocks=[o["da"]], dx=o["dx"], dw=o["dw1"], workspace=ws)
    return o


_RUN = {"forward": _forward, "train": _train, "second": _second, "partials": _partials, "gathered": _gathered,
        "mlp1d_fwd": _mlp1d_fwd, "mlp1d": _mlp1d}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    L = _layout(case)
    size = {_BF: 2, _F32: 4}
    read = sum(2 * r * k for r, k in L["read"].values()) + sum(2 * n for n in L["bias"])
    written = sum(math.prod(shape) * size[dt] for shape, dt in L["out"].values())
    one = 2.0 * L["m"] * L["h"] * L["f"]
    products = {"forward": 1, "mlp1d_fwd": 2, "mlp1d": 6}.get(case["kind"], 3)
    return {"bytes": float(read + written), "flops": one * products * L.get("n", 1)}


def tolerance(case):
    # Measured between this path with other tiles, K splits and K orders: a forward product in fp32 moves by
    # 3e-7 (sums of up to some ten thousand terms in another order).  Where a bf16 tensor is returned or passed
    # on (the activation, dA), values near a midpoint round the other way: 2e-4 to 3e-4 over the whole tensor,
    # one bf16 step (7.8e-3) at a value, slightly more where GeLU' of a moved pre-activation is taken.
    if case["kind"] == "forward" and case["f32"]:
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-3, "max": 0.04}
