"""The work this library is used for, as cases that can be timed and compared.

Five families, each through the public calls of `paper_2605_11582_amd.binding`:

  gemv    one product for one token with buffers at hand (`sparse_gemv`, `int4_gemv`)
  smallm  one product for the 2 ... 64 candidate tokens of a verification step
  layers  a decoding or verification step through a few decoder layers, four calls a layer (q/k/v together, o,
          gate/up together, down), prepared once as a serving loop does that owns its buffers
  stack   the products of many layers planned as one table and run in one call
  codec   the offline side on host buffers: pruning + packing, dense quantisation, unpacking

Weights are FP16 normal values of standard deviation 0.02, pruned by magnitude and quantised per group; activations
are FP16 standard normal.  For the device families they are drawn, pruned and encoded with torch on the GPU (the
format is the one include/egt.h defines), so a stack of gigabytes is ready in a second or two.
"""
import math

import numpy as np
import torch

from paper_2605_11582_amd import binding as egt

KEEP = {"s24": 2, "s14": 1, "paired": 2, "fp16": 2, "fp16_14": 1}


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # one token through a small projection: latency and launch
        {"name": "gemv_1024x1024", "family": "gemv", "kind": "s24", "rows": 1024, "cols": 1024, "group": 128},
        # the ordinary decode product: gate or up projection of a 4096-wide decoder, 2:4 INT4
        {"name": "gemv_11008x4096", "family": "gemv", "kind": "s24", "rows": 11008, "cols": 4096, "group": 128},
        # sparsified but not quantised: the same projection with FP16 values
        {"name": "gemv_fp16_11008x4096", "family": "gemv", "kind": "fp16", "rows": 11008, "cols": 4096, "group": 0},
        # quantised but not sparsified, a width that fills no tile: 45 groups of 64, odd row count
        {"name": "gemv_dense_5003x2880", "family": "gemv", "kind": "dense", "rows": 5003, "cols": 2880, "group": 64},
        # N of N:4 chosen per row: a seeded half of the rows keeps one of four, the others two
        {"name": "gemv_rows_11008x4096", "family": "gemv", "kind": "rows", "rows": 11008, "cols": 4096, "group": 128},
        # sixteen candidates checked against one projection
        {"name": "smallm_16_11008x4096", "family": "smallm", "kind": "s24", "rows": 11008, "cols": 4096, "group": 128, "tokens": 16, "call": "plain"},
        # the most candidates a call takes, against the down projection, with the workspace the library asks for
        {"name": "smallm_64_4096x11008", "family": "smallm", "kind": "s24", "rows": 4096, "cols": 11008, "group": 128, "tokens": 64, "call": "ws"},
        # a decoding step through four layers of a layer-adaptive mix
        {"name": "decode_4_layers", "family": "layers", "kinds": "s24 d s24 s14", "hidden": 4096, "ffn": 11008, "group": 128, "tokens": 1},
        # a verification step of five candidates through two 2:4 layers and a 1:4 layer
        {"name": "verify_5_3_layers", "family": "layers", "kinds": "s24 s14 s24", "hidden": 4096, "ffn": 11008, "group": 128, "tokens": 5},
        # one token through a 32-layer stack, three storage forms, one call (the largest)
        {"name": "stack_decode_32", "family": "stack", "kinds": "s24 s14 d s24 s14 d s24 s14 d s24 s14 d s24 s14 d s24 s14 d s24 s14 d s24 s14 d s24 s14 d s24 s14 d s24 s14",
         "hidden": 4096, "ffn": 11008, "group": 128, "tokens": 1},
        # sixteen candidates through the sixteen 2:4 layers of a stack, one call
        {"name": "stack_verify_16", "family": "stack", "kinds": " ".join(["s24"] * 16), "hidden": 4096, "ffn": 11008, "group": 128, "tokens": 16},
        # compressing a projection before it is deployed
        {"name": "encode_4096x4096", "family": "codec", "op": "encode", "kind": "s24", "rows": 4096, "cols": 4096, "group": 128},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cols(rng, lo, hi):
    """A row length: mostly whole groups of 128, now and then only whole chunks of 64 or words of 32."""
    step = rng.choice([128, 128, 128, 64, 32])
    return max(1, round(_log(rng, lo, hi) / step)) * step


def _group(rng, cols):
    return rng.choice([g for g in (32, 64, 128, 128, 128, 256) if cols % g == 0])


def _widths(rng):
    hidden = 128 * _log(rng, 8, 48)
    return {"hidden": hidden, "ffn": 128 * int(round(hidden * rng.uniform(2.5, 4.0) / 128)), "group": rng.choice([64, 128, 128])}


def draw(rng):
    family = rng.choice(["gemv", "gemv", "smallm", "smallm", "layers", "stack", "codec"])
    if family == "gemv":
        kind = rng.choice(["s24", "s24", "s14", "fp16", "dense", "dense", "rows", "paired", "fp16_14"])
        cols = _cols(rng, 512, 16384)
        rows = _log(rng, 256, min(65536, (1 << 28) // cols))
        return {"family": family, "kind": kind, "rows": rows, "cols": cols, "group": 0 if kind.startswith("fp16") else _group(rng, cols)}
    if family == "smallm":
        kind = rng.choice(["s24", "s24", "s24", "s14", "fp16"])
        cols = _cols(rng, 512, 16384)
        rows = _log(rng, 256, min(32768, (1 << 27) // cols))
        tokens, call = _log(rng, 2, 64), rng.choice(["plain", "ws", "static"])
        # (the library's own scratch buffer holds 16 MiB of partial sums: a slice is at least 1024 columns)
        if 64 * rows * -(-cols // 1024) * 4 > 16 << 20 and call == "static":
            call = "ws"
        return {"family": family, "kind": kind, "rows": rows, "cols": cols, "group": 0 if kind == "fp16" else _group(rng, cols),
                "tokens": tokens, "call": call}
    if family == "layers":
        tokens = 1 if rng.random() < 0.5 else _log(rng, 2, 64)
        kinds = ["s24", "s14", "d"] if tokens == 1 else ["s24", "s24", "s14"]
        return {"family": family, "kinds": " ".join(rng.choice(kinds) for _ in range(rng.randint(1, 4))), "tokens": tokens, **_widths(rng)}
    if family == "stack":
        tokens = 1 if rng.random() < 0.5 else _log(rng, 2, 64)
        # what a table takes: groups of 128 with all forms; one token: widths of the row-per-wave kernels; several
        # tokens: 2:4 at any count, 1:4 up to 32
        kinds = ["s24", "s14", "d"] if tokens == 1 else ["s24", "s14"] if tokens <= 32 else ["s24"]
        widths = {"hidden": rng.choice([2048, 4096]), "ffn": rng.choice([8192, 128 * rng.randint(81, 96)])} if tokens == 1 else _widths(rng)
        return {"family": family, "kinds": " ".join(rng.choice(kinds) for _ in range(rng.randint(4, 12))), "tokens": tokens, **widths, "group": 128}
    op = rng.choice(["encode", "encode", "quant", "decode"])
    cols = _cols(rng, 1024, 8192)
    rows = _log(rng, 256, min(8192, (1 << 25) // cols))
    kind = "dense" if op == "quant" else rng.choice(["s24", "s24", "s14", "fp16"])
    return {"family": family, "op": op, "kind": kind, "rows": rows, "cols": cols, "group": 0 if kind == "fp16" else _group(rng, cols)}


# ---------------------------------------------------------------- inputs
def _weights(gen, rows, cols):
    return torch.randn((rows, cols), generator=gen, device="cuda", dtype=torch.float16) * 0.02


def _tokens(gen, tokens, cols):
    return torch.randn((tokens, cols), generator=gen, device="cuda", dtype=torch.float16)


def _bytes(t):
    return t.contiguous().view(torch.uint8).reshape(-1)


def _quantise(w, group):
    """Codes and {scale, zero} pairs of dense (or pruned: zeros) weights."""
    rows, cols = w.shape
    v = w.view(rows, cols // group, group).float()
    lo, hi = v.amin(-1).clamp(max=0.0), v.amax(-1).clamp(min=0.0)
    s = ((hi - lo) / 15).half()
    s = torch.where(s == 0, torch.ones_like(s), s)
    z = (-lo / s.float()).round().clamp(0, 15)
    q = ((v / s.float().unsqueeze(-1)).round() + z.unsqueeze(-1)).clamp(0, 15).to(torch.uint8).view(rows, cols)
    return q, torch.stack([s, z.half()], -1)


def _encode(w, kind, group):
    """(values, idx, qparams) of w pruned to n:4 and encoded, one row of bytes per matrix row."""
    rows, cols = w.shape
    n = KEEP[kind]
    w4 = w.view(rows, cols // 4, 4)
    mag = [w4[..., j].abs() for j in range(4)]
    keep = []
    for j in range(4):
        beats = sum((mag[i] >= mag[j] if i < j else mag[i] > mag[j]).to(torch.uint8) for i in range(4) if i != j)
        keep.append(beats < n)
    keep = torch.stack(keep, -1)
    first = keep.to(torch.uint8).argmax(-1, keepdim=True)
    if n == 1:
        off = first
    else:
        off = torch.cat([first, 3 - keep.flip(-1).to(torch.uint8).argmax(-1, keepdim=True)], -1)
    o8 = off.reshape(rows, -1, 8).to(torch.int32)
    idx = sum(o8[..., k] << (2 * k) for k in range(8)).to(torch.int16)
    if kind.startswith("fp16"):
        return w4.gather(-1, off).reshape(rows, -1), idx, None
    q, qparams = _quantise((w4 * keep).view(rows, cols), group)
    c8 = q.view(rows, cols // 4, 4).gather(-1, off).reshape(rows, -1, 8)
    order = (0, 2, 4, 6, 1, 3, 5, 7) if kind == "paired" else tuple(range(8))
    values = torch.stack([c8[..., order[2 * b]] | (c8[..., order[2 * b + 1]] << 4) for b in range(4)], -1)
    return values.reshape(rows, -1), idx, qparams


def _sparse(gen, rows, cols, kind, group):
    values, idx, qparams = _encode(_weights(gen, rows, cols), kind, group)
    row_ptr = (torch.arange(rows + 1, device="cuda", dtype=torch.int64) * (KEEP[kind] * cols // 4)).to(torch.int32)
    val_kind = egt.VAL_FP16 if qparams is None else egt.VAL_INT4_PAIRED if kind == "paired" else egt.VAL_INT4
    return egt.Packed(rows, cols, KEEP[kind], group, val_kind, _bytes(row_ptr), _bytes(values), _bytes(idx),
                      None if qparams is None else _bytes(qparams))


def _sparse_rows(gen, rows, cols, group):
    """Rows of different lengths: a random half keeps one of four, the rest two of four.  A row at 1:4 is one unit of
    cols / 4 slots, a row at 2:4 two of them."""
    two = torch.zeros(rows, dtype=torch.bool, device="cuda")
    two[torch.randperm(rows, generator=gen, device="cuda")[: rows // 2]] = True
    w = _weights(gen, rows, cols)
    unit = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), (1 + two.long()).cumsum(0)])
    values = torch.empty((int(unit[-1]), cols // 8), dtype=torch.uint8, device="cuda")
    idx = torch.empty((int(unit[-1]), cols // 32), dtype=torch.int16, device="cuda")
    qparams = torch.empty((rows, cols // group, 2), dtype=torch.float16, device="cuda")
    for kind, pick in (("s14", ~two), ("s24", two)):
        v, i, qp = _encode(w[pick], kind, group)
        at = unit[:-1][pick]
        for part in range(KEEP[kind]):
            values[at + part] = v.view(len(at), KEEP[kind], -1)[:, part]
            idx[at + part] = i.view(len(at), KEEP[kind], -1)[:, part]
        qparams[pick] = qp
    row_ptr = unit * (cols // 4)
    return egt.Packed(rows, cols, 0, group, egt.VAL_INT4, _bytes(row_ptr.to(torch.int32)), _bytes(values), _bytes(idx), _bytes(qparams), int(row_ptr[-1]))


def _dense(gen, rows, cols, group):
    q, qparams = _quantise(_weights(gen, rows, cols), group)
    return (q[:, 0::2] | (q[:, 1::2] << 4)).contiguous(), qparams.contiguous()


def _projections(case):
    """[(kind, [rows of the matrices that read the same tokens], cols)] of every step of the layers in order."""
    h, f = case["hidden"], case["ffn"]
    return [(kind, rows, cols) for kind in case["kinds"].split() for rows, cols in (([h, h, h], h), ([h], h), ([f, f], h), ([h], f))]


class _Outputs:
    """One buffer for all results of a state; every result starts on a 256-byte boundary."""

    def __init__(self, sizes):
        self.at, end = [], 0
        for n in sizes:
            self.at.append((end, n))
            end += -(-n // 128) * 128
        self.all = torch.zeros(end, dtype=torch.float16, device="cuda")

    def take(self, shape):
        start, n = self.at.pop(0)
        return self.all[start:start + n].view(shape)


def prepare(case, seed):
    if case["family"] == "codec":
        rng = np.random.default_rng(seed)
        w = (rng.standard_normal((case["rows"], case["cols"]), dtype=np.float32) * np.float32(0.02)).astype(np.float16)
        state = {"case": case, "w": w}
        if case["op"] == "decode":
            n, fp16 = KEEP[case["kind"]], case["kind"] == "fp16"
            state["packed"] = egt.pack_2bitcsr(w, egt.prune_n4(w, n), n, case["group"], egt.VAL_FP16 if fp16 else egt.VAL_INT4)
        return state
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["family"] in ("gemv", "smallm"):
        rows, cols, group, kind = case["rows"], case["cols"], case["group"], case["kind"]
        tokens = case.get("tokens", 1)
        x = _tokens(gen, tokens, cols)
        y = torch.zeros((tokens, rows), dtype=torch.float16, device="cuda")
        if case["family"] == "gemv":
            x, y = x.view(-1), y.view(-1)
        state = {"case": case, "x": x, "y": y}
        if kind == "dense":
            state["q"], state["qparams"] = _dense(gen, rows, cols, group)
        elif kind == "rows":
            state["w"] = _sparse_rows(gen, rows, cols, group)
        else:
            state["w"] = _sparse(gen, rows, cols, kind, group)
        if case.get("call") == "ws":
            need = egt.smallm_ws_bytes(state["w"], tokens)
            state["workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
        return state
    tokens, group = case["tokens"], case["group"]
    steps = _projections(case)
    out = _Outputs([tokens * r for _, rows, _ in steps for r in rows])
    calls, items = [], []
    for kind, rows, cols in steps:
        x = _tokens(gen, tokens, cols)
        if tokens == 1:
            x = x.view(-1)
        ys = [out.take((r,) if tokens == 1 else (tokens, r)) for r in rows]
        if kind == "d":
            ws = [_dense(gen, r, cols, group) for r in rows]
            items += [("dense", q, qp, r, cols, group, x, y) for (q, qp), r, y in zip(ws, rows, ys)]
            if case["family"] == "layers":
                if len(ws) > 1:
                    calls.append(egt.prepared_int4_gemv_batch([q for q, _ in ws], [qp for _, qp in ws], rows[0], cols, group, [x] * len(ws), ys))
                else:
                    calls.append(egt.prepared_int4_gemv(*ws[0], rows[0], cols, group, x, ys[0]))
            continue
        ws = [_sparse(gen, r, cols, kind, group) for r in rows]
        items += [("sparse", w, x, y) if tokens == 1 else (w, x, y) for w, y in zip(ws, ys)]
        if case["family"] == "layers":
            if tokens == 1:
                calls.append(egt.prepared_sparse_gemv_batch(ws, [x] * len(ws), ys) if len(ws) > 1 else egt.prepared_sparse_gemv(ws[0], x, ys[0]))
            else:
                calls.append(egt.prepared_sparse_gemm_smallm_batch(ws, [x] * len(ws), ys) if len(ws) > 1 else egt.prepared_sparse_gemm_smallm(ws[0], x, ys[0]))
    if case["family"] == "stack":
        calls = [egt.prepared_gemv_stack(items) if tokens == 1 else egt.prepared_gemm_stack(items)]
    return {"case": case, "calls": calls, "y": out.all}


# ---------------------------------------------------------------- one pass
def run(state):
    case = state["case"]
    family = case["family"]
    if family == "gemv":
        if case["kind"] == "dense":
            egt.int4_gemv(state["q"], state["qparams"], case["rows"], case["cols"], case["group"], state["x"], state["y"])
        else:
            egt.sparse_gemv(state["w"], state["x"], state["y"])
        return state["y"]
    if family == "smallm":
        if case["call"] == "ws":
            egt.sparse_gemm_smallm_ws(state["w"], state["x"], state["y"], state["workspace"])
        elif case["call"] == "static":
            egt.sparse_gemm_smallm_static(state["w"], state["x"], state["y"])
        else:
            egt.sparse_gemm_smallm(state["w"], state["x"], state["y"])
        return state["y"]
    if family == "codec":
        if case["op"] == "quant":
            return egt.quant_int4(state["w"], case["group"])
        if case["op"] == "decode":
            return egt.unpack_2bitcsr(state["packed"])
        n = KEEP[case["kind"]]
        mask = egt.prune_n4(state["w"], n)
        p = egt.pack_2bitcsr(state["w"], mask, n, case["group"], egt.VAL_FP16 if case["kind"] == "fp16" else egt.VAL_INT4)
        return [mask, p.row_ptr, p.values, p.idx] + ([] if p.qparams is None else [p.qparams])
    for call in state["calls"]:
        call()
    return state["y"]


# ---------------------------------------------------------------- what a pass cannot do without
def _matrix_work(kind, rows, cols, group, tokens, x_bytes):
    if kind in ("dense", "d"):
        data, entries = rows * cols // 2 + 4 * rows * (cols // group), rows * cols
    else:
        # (rows of two lengths: half at 1:4, half at 2:4)
        entries = (rows - rows // 2 + 2 * (rows // 2)) * cols // 4 if kind == "rows" else rows * KEEP[kind] * cols // 4
        data = entries // 4 + 4 * (rows + 1)
        data += 2 * entries if kind.startswith("fp16") else entries // 2 + 4 * rows * (cols // group)
    return data + x_bytes + 2 * tokens * rows, 2 * tokens * entries


def work(case):
    if case["family"] == "codec":
        rows, cols, group = case["rows"], case["cols"], case["group"]
        packed, _ = _matrix_work(case["kind"], rows, cols, group, 0, 0)
        return {"bytes": packed + (2 if case["op"] == "quant" else 3) * rows * cols, "flops": 0}
    if case["family"] in ("gemv", "smallm"):
        tokens = case.get("tokens", 1)
        b, f = _matrix_work(case["kind"], case["rows"], case["cols"], case["group"], tokens, 2 * tokens * case["cols"])
        return {"bytes": b, "flops": f}
    tokens, total_b, total_f = case["tokens"], 0, 0
    for kind, rows, cols in _projections(case):
        for k, r in enumerate(rows):
            b, f = _matrix_work(kind, r, cols, case["group"], tokens, 0 if k else 2 * tokens * cols)
            total_b, total_f = total_b + b, total_f + f
    return {"bytes": total_b, "flops": total_f}


def tolerance(case):
    # Device results are FP16 (half a unit in the last place: 2^-11) of FP32 sums of weights that a correct
    # kernel may round to FP16 (another 2^-11 each, averaging out over a row) or keep in FP32.  The encoder
    # is defined to the bit.
    return "exact" if case["family"] == "codec" else {"rel": 1e-3, "max": 1e-2}
