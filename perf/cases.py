"""The workloads whose speed this library is kept to, through its public calls.

Each case is one call (or one short sequence of calls) that a program built on
the library makes: the triangle update in its two storage types from a few
dozen tokens to thousands, a training step and a recomputing backward, one
device's share of the paper's 2-D ring, the outer product mean and the
triangle attention core.  listed() names twelve of them, draw() takes more
from the same ranges, exact() states the result in float64 with plain torch.
"""
import math

import torch

from paper_2603_14806_amd import synth
from paper_2603_14806_amd import trimul as tm

C = 128          # channels of the pair tensor and of the hidden operands
EPS = 1e-5
WEIGHTS = tm.WEIGHT_FIELDS


def listed():
    return [
        # float32 layer at the smallest size the benchmark table has: launch latency
        dict(name="update_f32_n64", op="update", n=64, dtype="f32", out="f32", direction="outgoing", mask="none", scaled=False),
        # float32 layer (a model run without bf16) at a usual crop, padded batch member
        dict(name="update_f32_n384", op="update", n=384, dtype="f32", out="f32", direction="incoming", mask="pad", scaled=False),
        # short chain in a serving loop that must not allocate
        dict(name="noalloc_bf16_n100", op="noalloc", n=100, dtype="bf16", out="f32", direction="incoming", mask="random", scaled=False),
        # bf16 inference at the size of one small complex, last tokens padded
        dict(name="update_bf16_n512", op="update", n=512, dtype="bf16", out="f32", direction="outgoing", mask="pad", scaled=False),
        # bf16 inference with the token count as it comes (no multiple of a tile), bf16 result
        dict(name="update_bf16_n1300", op="update", n=1300, dtype="bf16", out="bf16", direction="incoming", mask="pad", scaled=True),
        # the benchmark's own layer size
        dict(name="update_bf16_n4096", op="update", n=4096, dtype="bf16", out="f32", direction="outgoing", mask="none", scaled=False),
        # one training step of the layer on a usual crop: forward that keeps its state, then backward from it
        dict(name="train_bf16_n384", op="train", n=384, dtype="bf16", out="f32", direction="outgoing", mask="pad", scaled=False),
        # backward under activation checkpointing (recomputes the forward), long crop
        dict(name="backward_bf16_n1024", op="backward", n=1024, dtype="bf16", out="f32", direction="incoming", mask="pad", scaled=False),
        # one device's share of the update on a 4 x 4 grid: own projection, 4 ring steps, epilogue
        dict(name="ring_n6000_grid4", op="ring", n=6000, grid=4, dtype="bf16", out="f32", direction="outgoing", mask="pad", scaled=False),
        # outer product mean of a deep MSA on a token count as it comes
        dict(name="opm_s2048_n500", op="opm", s=2048, n=500, out="f32", mask="random"),
        # triangle attention in a bf16 model on a usual crop
        dict(name="attn_n384_h4", op="attn", rows=384, n=384, heads=4, out="bf16", mask="pad", chunks=1),
        # triangle attention at the benchmark's size, fp32 result
        dict(name="attn_n2048_h4", op="attn", rows=2048, n=2048, heads=4, out="f32", mask="none", chunks=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["update_bf16", "update_bf16", "update_f32", "noalloc", "train", "backward", "ring", "opm", "attn", "attn"])
    mask = rng.choice(["none", "pad", "random"])
    layer = dict(direction=rng.choice(["outgoing", "incoming"]), mask=mask, scaled=rng.random() < 0.3,
                 out=rng.choice(["f32", "f32", "bf16"]))
    if op == "update_bf16":
        return dict(op="update", n=_log_int(rng, 32, 2048), dtype="bf16", **layer)
    if op == "update_f32":
        return dict(op="update", n=_log_int(rng, 32, 512), dtype="f32", **dict(layer, out="f32"))
    if op == "noalloc":
        return dict(op="noalloc", n=_log_int(rng, 32, 512), dtype="bf16", **layer)
    if op in ("train", "backward"):
        return dict(op=op, n=_log_int(rng, 64, 1024), dtype="bf16", **layer)
    if op == "ring":
        grid = rng.choice([2, 3, 4])
        return dict(op="ring", n=_log_int(rng, 256, 1500) * grid + rng.randrange(grid), grid=grid, dtype="bf16", **layer)
    if op == "opm":
        return dict(op="opm", s=_log_int(rng, 32, 4096), n=_log_int(rng, 48, 768), out=layer["out"], mask=rng.choice(["none", "random"]))
    n = _log_int(rng, 64, 1536)
    return dict(op="attn", rows=n if rng.random() < 0.7 else _log_int(rng, 16, 1536), n=n, heads=rng.choice([2, 4, 4, 8]),
                out=layer["out"], mask=mask, chunks=rng.choice([1, 1, 2, 3]))


# ------------------------------------------------------------------ inputs

def _generator(seed, sub):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 64 + sub)
    return g


def _normal(shape, seed, sub, dtype=torch.bfloat16):
    return torch.randn(shape, generator=_generator(seed, sub), device="cuda", dtype=torch.float32).to(dtype)


def _token_mask(case, n, seed):
    if case["mask"] == "none":
        return None
    if case["mask"] == "pad":
        return synth.token_mask(n, n // 10, device="cuda")
    return synth.random_mask(n, 0.85, seed=seed).to("cuda")


def _layer_inputs(case, seed, shape=None, name="z"):
    scale = synth.channel_scale(C, seed) if case["scaled"] else None
    return synth.pair_tensor(case["n"], C, case["dtype"], seed=seed, scale=scale, device="cuda", name=name, shape=shape)


def _weights(case, seed):
    return synth.weights(C, C, dtype=case["dtype"], seed=seed, affine=True)


def _opposite(direction):
    return "incoming" if direction == "outgoing" else "outgoing"


def _tile(case):
    """First token and length of the last diagonal tile of the grid (the ragged one)."""
    size = -(-case["n"] // case["grid"])
    first = size * (case["grid"] - 1)
    return first, case["n"] - first


def _ring_blocks(case):
    """Token ranges of the k-panels, own tile's last."""
    size = -(-case["n"] // case["grid"])
    return [(p * size, min(case["n"], (p + 1) * size) - p * size) for p in range(case["grid"])]


def _ring_tile_z(case, seed, p):
    """z of the tile that holds the own tokens and block p: rows are the own
    tokens when the contraction runs over columns, columns otherwise."""
    own, block = _tile(case)[1], _ring_blocks(case)[p][1]
    shape = (own, block, C) if case["direction"] == "outgoing" else (block, own, C)
    return _layer_inputs(case, seed + 7919 * (p + 1), shape=shape, name="z_tile")


def _attention_inputs(case, seed):
    shape = (case["rows"], case["n"], case["heads"], 32)
    q, k, v = (_normal(shape, seed, s) for s in (1, 2, 3))
    ld = -(-case["n"] // 8) * 8
    bias = _normal((case["heads"], case["n"], ld), seed, 4)
    return q, k, v, bias, _token_mask(case, case["n"], seed)


def _opm_inputs(case, seed):
    a = _normal((case["s"], case["n"], 32), seed, 1)
    b = _normal((case["s"], case["n"], 32), seed, 2)
    mask = None
    if case["mask"] == "random":
        mask = (torch.rand((case["s"], case["n"]), generator=_generator(seed, 3), device="cuda") < 0.9).to(torch.uint8)
    w_o = _normal((C, 1024), seed, 4, torch.float32).mul_(1 / 32).to(torch.bfloat16)
    b_o = _normal((C,), seed, 5)
    return a, b, mask, w_o, b_o


def prepare(case, seed):
    op = case["op"]
    st = dict(case=case)
    if op in ("update", "noalloc", "train", "backward"):
        n = case["n"]
        st["layer"] = tm.TriMul(_weights(case, seed), dtype=case["dtype"], out_dtype=case["out"], eps=EPS)
        st["z"] = _layer_inputs(case, seed)
        st["mask"] = _token_mask(case, n, seed)
        if op == "update":
            st["layer"].workspace(n)
        if op == "noalloc":
            st["out"] = torch.empty((n, n, C), dtype=synth.DTYPES[case["out"]], device="cuda")
        if op in ("train", "backward"):
            st["dout"] = synth.pair_tensor(n, C, case["out"], seed=seed, device="cuda", name="dout")
    elif op == "ring":
        layer = st["layer"] = tm.TriMul(_weights(case, seed), dtype="bf16", out_dtype=case["out"], eps=EPS)
        n, (first, own), blocks = case["n"], _tile(case), _ring_blocks(case)
        st["mask"] = _token_mask(case, n, seed)
        st["panels"] = []           # the other devices' projections, as they arrive
        for p, (k0, klen) in enumerate(blocks[:-1]):
            z = _ring_tile_z(case, seed, p)
            row0, col0 = (first, k0) if case["direction"] == "outgoing" else (k0, first)
            st["panels"].append(layer.block_project(z, st["mask"], n, row0, col0, _opposite(case["direction"])))
        st["z"] = _ring_tile_z(case, seed, case["grid"] - 1)
        st["views"] = [tm.BlockView(n, first, first, own, own, k0, klen, 0, 0, p, len(blocks))
                       for p, (k0, klen) in enumerate(blocks)]
        st["acc"] = torch.empty(layer.block_accumulator_size(st["views"][0]) // 4, dtype=torch.float32, device="cuda")
        st["out"] = torch.empty((own, own, C), dtype=synth.DTYPES[case["out"]], device="cuda")
    elif op == "opm":
        st["a"], st["b"], st["mask"], w_o, b_o = _opm_inputs(case, seed)
        st["opm"] = tm.OuterProductMean(w_o, b_o, out_dtype=case["out"])
    else:
        st["q"], st["k"], st["v"], st["bias"], st["mask"] = _attention_inputs(case, seed)
        n = case["n"]
        if case["chunks"] > 1:
            step = -(-n // case["chunks"])
            step = -(-step // 8) * 8
            cuts = list(range(0, n, step)) + [n]
            st["views"] = [tm.TriAttnView(case["rows"], n, case["heads"], tm.DTYPE_CODE[case["out"]], st["bias"].stride(1),
                                          k0, k1 - k0, i, len(cuts) - 1) for i, (k0, k1) in enumerate(zip(cuts, cuts[1:]))]
            st["state"] = torch.empty(tm.tri_attn_state_size(st["views"][0]) // 4, dtype=torch.float32, device="cuda")
            st["out"] = torch.empty((case["rows"], n, case["heads"], 32), dtype=synth.DTYPES[case["out"]], device="cuda")
    return st


# ------------------------------------------------------------------ one pass

def run(st):
    case = st["case"]
    op = case["op"]
    if op == "update":
        return st["layer"](st["z"], st["mask"], case["direction"])
    if op == "noalloc":
        code = tm.TRI_MUL_INCOMING if case["direction"] == "incoming" else tm.TRI_MUL_OUTGOING
        tm.tri_mul_update_noalloc(st["layer"].h, st["z"], st["mask"], case["n"], code, st["out"])
        return st["out"]
    if op == "train":
        layer, n, z, mask = st["layer"], case["n"], st["z"], st["mask"]
        at, bt = layer.project(z, mask, _opposite(case["direction"]))
        c = layer.contract_transposed(at, bt, n)
        out = layer.epilogue(c, z, mask)
        dz, grads = layer.backward(z, st["dout"], mask, case["direction"], saved=(at, bt, c))
        return dict(out=out, dz=dz, grads=grads)
    if op == "backward":
        dz, grads = st["layer"].backward(st["z"], st["dout"], st["mask"], case["direction"])
        return dict(dz=dz, grads=grads)
    if op == "ring":
        layer, first = st["layer"], _tile(case)[0]
        own = layer.block_project(st["z"], st["mask"], case["n"], first, first, _opposite(case["direction"]))
        for view, (at, bt) in zip(st["views"], st["panels"] + [own]):
            layer.block_accumulate_transposed(view, at, bt, st["acc"], st["mask"], st["z"], st["out"])
        return st["out"]
    if op == "opm":
        return st["opm"].forward(st["a"], st["b"], st["mask"])
    if case["chunks"] == 1:
        return tm.triangle_attention(st["q"], st["k"], st["v"], st["bias"], st["mask"], case["out"])
    for view in st["views"]:
        tm.tri_attn_chunk(view, st["q"], st["k"], st["v"], st["bias"], st["mask"], st["state"], st["out"])
    return st["out"]


# ------------------------------------------------------------------ work and tolerance

def work(case):
    op = case["op"]
    ebytes = {"f32": 4, "bf16": 2}
    out = ebytes[case["out"]]
    if op in ("update", "noalloc", "train", "backward"):
        n, pairs, z = case["n"], case["n"] ** 2, ebytes[case["dtype"]]
        product, linear = 2.0 * n ** 3 * C, 2.0 * pairs * C * C
        if op in ("update", "noalloc"):
            return dict(bytes=pairs * C * (z + out), flops=product + 6 * linear)
        if op == "train":      # z, dout read; out, dz written
            return dict(bytes=pairs * C * (2 * z + 2 * out), flops=3 * product + 18 * linear)
        return dict(bytes=pairs * C * (2 * z + out), flops=3 * product + 18 * linear)
    if op == "ring":
        own, others = _tile(case)[1], [k for _, k in _ring_blocks(case)[:-1]]
        moved = own * own * C * (2 + out) + sum(2 * own * k * C * 2 for k in others)
        return dict(bytes=moved, flops=2.0 * own * own * case["n"] * C + 6 * 2.0 * own * own * C * C)
    if op == "opm":
        s, n = case["s"], case["n"]
        moved = 2 * s * n * 32 * 2 + (s * n if case["mask"] != "none" else 0) + n * n * C * out
        return dict(bytes=moved, flops=2.0 * s * (n * 32) ** 2 + 2.0 * n * n * 1024 * C)
    each = case["rows"] * case["n"] * case["heads"] * 32
    return dict(bytes=each * (6 + out) + case["heads"] * case["n"] ** 2 * 2, flops=4.0 * each * case["n"])


def tolerance(case):
    # four times the relative error against float64 that each path shows
    op = case["op"]
    if op in ("update", "noalloc", "ring"):
        return {"rel": 4e-6} if case["dtype"] == "f32" else {"rel": 1e-2}
    if op in ("train", "backward"):
        return {"rel": 1.5e-2}
    if case["out"] == "bf16":
        return {"rel": 8e-3}
    return {"rel": 8e-6} if op == "attn" else {"rel": 1e-5}


# ------------------------------------------------------------------ float64 statement

def _norm(x, w, b):
    d = x - x.mean(-1, keepdim=True)
    return d * (d.square().mean(-1, keepdim=True) + EPS).rsqrt() * w + b


def _f64_weights(case, seed):
    return {k: v.to("cuda").double() for k, v in _weights(case, seed).items()}


def _f64_mask(mask, n):
    return torch.ones(n, dtype=torch.float64, device="cuda") if mask is None else (mask != 0).double()


def _gated_pair(z, m, w):
    """a, b of a rectangle of pairs; m is its pair mask."""
    x = _norm(z.double(), w["ln_in_w"], w["ln_in_b"])
    m = m[..., None]
    return (m * torch.sigmoid(x @ w["w_ga"].T) * (x @ w["w_a"].T),
            m * torch.sigmoid(x @ w["w_gb"].T) * (x @ w["w_b"].T))


def _finish(c, z, m, w):
    """The update of a rectangle of pairs from its contraction c [...][C]."""
    x = _norm(z.double(), w["ln_in_w"], w["ln_in_b"])
    return m[..., None] * torch.sigmoid(x @ w["w_g"].T) * (_norm(c, w["ln_out_w"], w["ln_out_b"]) @ w["w_o"].T)


def _strip(z, mi, mj, w):
    """a, b channel-major [C][rows][cols] of a rectangle, in row chunks."""
    rows, cols = z.shape[0], z.shape[1]
    a = torch.empty((C, rows, cols), dtype=torch.float64, device="cuda")
    b = torch.empty_like(a)
    chunk = max(1, (1 << 20) // cols)
    for r in range(0, rows, chunk):
        s = slice(r, min(rows, r + chunk))
        x, y = _gated_pair(z[s], mi[s, None] * mj[None, :], w)
        a[:, s], b[:, s] = x.permute(2, 0, 1), y.permute(2, 0, 1)
    return a, b


def _finish_rows(c, z, mi, mj, w):
    rows, cols = z.shape[0], z.shape[1]
    out = torch.empty((rows, cols, C), dtype=torch.float64, device="cuda")
    chunk = max(1, (1 << 20) // cols)
    for r in range(0, rows, chunk):
        s = slice(r, min(rows, r + chunk))
        out[s] = _finish(c[:, s].permute(1, 2, 0), z[s], mi[s, None] * mj[None, :], w)
    return out


def _exact_update(case, seed):
    w, z = _f64_weights(case, seed), _layer_inputs(case, seed)
    m = _f64_mask(_token_mask(case, case["n"], seed), case["n"])
    a, b = _strip(z, m, m, w)
    for ch in range(C):          # the contraction replaces a channel by channel
        a[ch] = a[ch] @ b[ch].T if case["direction"] == "outgoing" else a[ch].T @ b[ch]
    return _finish_rows(a, z, m, m, w)


def _exact_ring(case, seed):
    w, (first, own) = _f64_weights(case, seed), _tile(case)
    m = _f64_mask(_token_mask(case, case["n"], seed), case["n"])
    mine = m[first:first + own]
    c = torch.zeros((C, own, own), dtype=torch.float64, device="cuda")
    for p, (k0, klen) in enumerate(_ring_blocks(case)):
        z, mk = _ring_tile_z(case, seed, p), m[k0:k0 + klen]
        if case["direction"] == "outgoing":
            a, b = _strip(z, mine, mk, w)
            for ch in range(C):
                c[ch] += a[ch] @ b[ch].T
        else:
            a, b = _strip(z, mk, mine, w)
            for ch in range(C):
                c[ch] += a[ch].T @ b[ch]
    return _finish_rows(c, z, mine, mine, w)      # z is the own tile's


def _exact_gradients(case, seed):
    n = case["n"]
    w = {k: v.requires_grad_(True) for k, v in _f64_weights(case, seed).items()}
    z = _layer_inputs(case, seed).double().requires_grad_(True)
    dout = synth.pair_tensor(n, C, case["out"], seed=seed, device="cuda", name="dout").double()
    m = _f64_mask(_token_mask(case, n, seed), n)
    pair = m[:, None] * m[None, :]
    a, b = (t.permute(2, 0, 1).contiguous() for t in _gated_pair(z, pair, w))
    c = a @ b.transpose(1, 2).contiguous() if case["direction"] == "outgoing" else a.transpose(1, 2).contiguous() @ b
    out = _finish(c.permute(1, 2, 0), z, pair, w)
    names = list(WEIGHTS)
    grads = torch.autograd.grad((out * dout).sum(), [z] + [w[k] for k in names])
    result = dict(dz=grads[0], grads=dict(zip(names, grads[1:])))
    if case["op"] == "train":
        result["out"] = out.detach()
    return result


def _exact_opm(case, seed):
    a, b, mask, w_o, b_o = _opm_inputs(case, seed)
    s, n = case["s"], case["n"]
    m = torch.ones((s, n), dtype=torch.float64, device="cuda") if mask is None else (mask != 0).double()
    a, b = a.double() * m[..., None], b.double() * m[..., None]
    count = m.T @ m
    inv = torch.where(count > 0, 1 / count.clamp(min=1), torch.zeros_like(count))
    w_o, b_o = w_o.double(), b_o.double()
    out = torch.empty((n, n, C), dtype=torch.float64, device="cuda")
    right = b.reshape(s, n * 32)
    for i in range(0, n, 16):
        left = a[:, i:i + 16].reshape(s, -1)
        o = (left.T @ right).reshape(-1, 32, n, 32).permute(0, 2, 1, 3).reshape(-1, n, 1024)
        out[i:i + 16] = (o * inv[i:i + 16, :, None]) @ w_o.T + b_o
    return out


def _exact_attention(case, seed):
    q, k, v, bias, mask = _attention_inputs(case, seed)
    n, rows = case["n"], case["rows"]
    bias = bias[:, :, :n].double()
    if mask is not None:
        bias = bias.masked_fill(mask[None, None, :] == 0, -math.inf)
    out = torch.empty((rows, n, case["heads"], 32), dtype=torch.float64, device="cuda")
    chunk = max(1, (1 << 28) // (case["heads"] * n * n))
    for r in range(0, rows, chunk):
        x, y, u = (t[r:r + chunk].double().permute(0, 2, 1, 3).contiguous() for t in (q, k, v))
        s = x @ y.transpose(2, 3).contiguous() / math.sqrt(32) + bias
        out[r:r + chunk] = (torch.softmax(s, -1) @ u).permute(0, 2, 1, 3)
    return out


def exact(case, seed):
    op = case["op"]
    with torch.set_grad_enabled(op in ("train", "backward")):
        if op in ("update", "noalloc"):
            return _exact_update(case, seed)
        if op in ("train", "backward"):
            return _exact_gradients(case, seed)
        if op == "ring":
            return _exact_ring(case, seed)
        if op == "opm":
            return _exact_opm(case, seed)
        return _exact_attention(case, seed)
