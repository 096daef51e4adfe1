"""The calls whose speed is measured, their inputs and their exact results.

A case is a dict of plain values: the entry point ("op") and its sizes and
options.  listed() names twelve of them, draw() gives more over the same
ranges, prepare() makes what a program holds before the call (inputs on the
GPU, the workspace and scratch it keeps), run() is one pass through the
public entry point, and exact() is the same result in 64 bits by torch alone.
"""
import math

import torch

from paper_2505_15112_amd import _lib, ops

DEV = "cuda"


def listed():
    return [
        # Offsets of a small batch (token counts, row starts): one short call,
        # all latency.
        dict(name="scan_i32_64k", op="scan", kind="i32", excl=False, n=1 << 16),
        # A half-precision cumulative sum of ordinary length.
        dict(name="scan_f16_16m", op="scan", kind="f16", excl=False, n=1 << 24),
        # An exclusive fp32 scan whose length fits no tile.
        dict(name="scan_f32_excl_67m", op="scan", kind="f32", excl=True, n=(1 << 26) + 17),
        # The longest array in common use: pure bandwidth.
        dict(name="scan_i32_268m", op="scan", kind="i32", excl=False, n=1 << 28),
        # Cumulative sums along the last dimension of a batch.
        dict(name="rows_f32_256x65536", op="rows", kind="f32", excl=False, rows=256, len=65536),
        # Masked select with indices over an odd length (filtering a column).
        dict(name="compact_idx_134m", op="compact", n=(1 << 27) + 5, keep=0.5, idx=True),
        # A large key sort with its permutation.
        dict(name="radix_u32_67m", op="radix", kind="u32", n=1 << 26, desc=False, perm=True),
        # A medium half-precision sort with indices (argsort of scores).
        dict(name="radix_f16_1m", op="radix", kind="f16", n=(1 << 20) + 1, desc=True, perm=True),
        # Nucleus sampling of a large serving batch over a 128K vocabulary.
        dict(name="topp_sample_128x131072", op="topp_sample", rows=128, len=131072, p=0.9),
        # The same for a few concurrent requests and a longer, odd vocabulary.
        dict(name="topp_sample_4x200003", op="topp_sample", rows=4, len=200003, p=0.9),
        # Top-k filtering of the same batch.
        dict(name="topk_128x131072_k64", op="topk", rows=128, len=131072, k=64, largest=True),
        # Multinomial sampling of unnormalised weights, an odd row length.
        dict(name="weighted_96x100003", op="weighted", rows=96, len=100003),
    ]


# ---------------------------------------------------------------- drawn cases

def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _rows_len(rng, max_rows, lo, hi, total, min_rows=1):
    length = _log_int(rng, lo, hi)
    if rng.random() < 0.5 and length >= 64:
        length = length // 64 * 64  # half of them padded lengths, half as they come
    return _log_int(rng, min_rows, max(min_rows, min(max_rows, total // length))), length


def draw(rng):
    op = rng.choice(["scan", "scan", "rows", "compact", "split", "radix", "sort_rows",
                     "topp_cutoff", "topp_sample", "weighted", "topk"])
    if op == "scan":
        return dict(op=op, kind=rng.choice(["i32", "f32", "f16", "u8"]), excl=rng.random() < 0.5,
                    n=_log_int(rng, 1 << 10, 1 << 28))
    if op == "rows":
        rows, length = _rows_len(rng, 8192, 64, 1 << 18, 1 << 26)
        return dict(op=op, kind=rng.choice(["i32", "f32"]), excl=rng.random() < 0.5, rows=rows,
                    len=length)
    if op == "compact":
        return dict(op=op, n=_log_int(rng, 1 << 12, 1 << 27), keep=round(rng.uniform(0.05, 0.95), 2),
                    idx=rng.random() < 0.5)
    if op == "split":
        return dict(op=op, n=_log_int(rng, 1 << 12, 1 << 26), keep=round(rng.uniform(0.05, 0.95), 2))
    if op == "radix":
        return dict(op=op, kind=rng.choice(["u32", "i32", "f32", "f16"]),
                    n=_log_int(rng, 1 << 10, 1 << 26), desc=rng.random() < 0.5,
                    perm=rng.random() < 0.75)
    if op == "sort_rows":
        rows, length = _rows_len(rng, 512, 256, 1 << 18, 1 << 24)
        return dict(op=op, rows=rows, len=length, desc=rng.random() < 0.5)
    rows, length = _rows_len(rng, 512, 1000, 1 << 18, 1 << 24, min_rows=2)
    if op == "topp_cutoff" or op == "topp_sample":
        return dict(op=op, rows=rows, len=length, p=rng.choice([0.5, 0.8, 0.9, 0.95]))
    if op == "weighted":
        return dict(op=op, rows=rows, len=length)
    return dict(op="topk", rows=rows, len=length, k=min(length, _log_int(rng, 1, 4096)),
                largest=rng.random() < 0.75)


# ---------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _probs(rows, length, g):
    """Softmax of N(0, 2^2) logits: what a sampler receives."""
    z = torch.randn((rows, length), device=DEV, generator=g) * 2.0
    return torch.softmax(z, dim=1)


def _inputs(case, seed):
    g = _gen(seed)
    op = case["op"]
    if op == "scan" or op == "rows":
        shape = (case["n"],) if op == "scan" else (case["rows"], case["len"])
        kind = case["kind"]
        if kind == "i32":
            return dict(x=torch.randint(0, 101, shape, dtype=torch.int32, device=DEV, generator=g))
        if kind == "u8":
            return dict(x=torch.randint(0, 256, shape, dtype=torch.uint8, device=DEV, generator=g))
        x = torch.rand(shape, device=DEV, generator=g).mul_(2.0).sub_(1.0)
        return dict(x=x.half() if kind == "f16" else x)
    if op == "compact" or op == "split":
        n = case["n"]
        mask = (torch.rand(n, device=DEV, generator=g) < case["keep"]).to(torch.uint8)
        if op == "compact":
            return dict(x=torch.randn(n, device=DEV, generator=g), mask=mask)
        return dict(x=torch.randint(-2**31, 2**31, (n,), dtype=torch.int32, device=DEV,
                                    generator=g), mask=mask)
    if op == "radix":
        n, kind = case["n"], case["kind"]
        if kind in ("u32", "i32"):
            return dict(x=torch.randint(-2**31, 2**31, (n,), dtype=torch.int32, device=DEV,
                                        generator=g))
        x = torch.randn(n, device=DEV, generator=g)
        return dict(x=x.half() if kind == "f16" else x)
    rows, length = case["rows"], case["len"]
    if op == "sort_rows":
        return dict(x=_probs(rows, length, g))
    if op == "topp_cutoff":
        return dict(x=torch.sort(_probs(rows, length, g), dim=1, descending=True)[0])
    if op == "topp_sample":
        x = _probs(rows, length, g)
        return dict(x=x, theta=torch.rand(rows, device=DEV, generator=g))
    if op == "weighted":  # exponential weights, a quarter of them zero
        w = -torch.log1p(-torch.rand((rows, length), device=DEV, generator=g))
        w = w * (torch.rand((rows, length), device=DEV, generator=g) >= 0.25)
        return dict(x=w, theta=torch.rand(rows, device=DEV, generator=g))
    return dict(x=_probs(rows, length, g) if case["largest"]
                else torch.randn((rows, length), device=DEV, generator=g))


def prepare(case, seed):
    """The inputs, and the workspace, scratch and (where a result has no fixed
    length) output buffers that a program keeps from call to call."""
    st = _inputs(case, seed)
    st["case"] = case
    dev = st["x"].device
    op = case["op"]
    if op == "scan":
        st["ws"] = ops.workspace(_lib.OP_SCAN, dev, case["n"])
    elif op in ("rows", "topp_cutoff"):
        st["ws"] = ops.workspace(_lib.OP_SCAN_ROWS, dev, rows=case["rows"], length=case["len"])
    elif op in ("compact", "split"):
        st["ws"] = ops.workspace(_lib.OP_COMPACT, dev, case["n"])
        if op == "compact":  # only the kept entries are written: the rest stays zero
            st["out"] = torch.zeros(case["n"], device=dev)
            st["idx"] = torch.zeros(case["n"], dtype=torch.int32, device=dev) if case["idx"] \
                else None
    elif op == "radix":
        st["ws"] = ops.workspace(_lib.OP_RADIX_SORT, dev, case["n"], bits=8)
    elif op == "sort_rows":
        st["ws"] = ops.workspace(_lib.OP_SORT_ROWS, dev, rows=case["rows"], length=case["len"])
    elif op == "weighted":
        st["ws"] = ops.workspace(_lib.OP_WEIGHTED_SAMPLE, dev, rows=case["rows"],
                                 length=case["len"])
    elif op == "topp_sample":
        st["ws"] = ops.workspace(_lib.OP_TOPP_SAMPLE, dev, rows=case["rows"], length=case["len"])
        st["scratch"] = ops.scratch(_lib.OP_TOPP_SAMPLE, dev, case["rows"], case["len"])
    else:
        st["ws"] = ops.workspace(_lib.OP_TOPK, dev, case["k"], rows=case["rows"],
                                 length=case["len"])
        st["scratch"] = ops.scratch(_lib.OP_TOPK, dev, case["rows"], case["len"], case["k"])
    return st


# ---------------------------------------------------------------- one pass

def run(st):
    case, x, ws = st["case"], st["x"], st["ws"]
    op = case["op"]
    if op == "scan":
        excl, kind = case["excl"], case["kind"]
        if kind == "i32":
            return (ops.scan_exclusive_i32 if excl else ops.scan_inclusive_i32)(x, ws=ws)
        if kind == "f32":
            return (ops.scan_exclusive_f32 if excl else ops.scan_inclusive_f32)(x, ws=ws)
        if kind == "f16":
            return (ops.scan_exclusive_f16f32 if excl else ops.scan_inclusive_f16f32)(x, ws=ws)
        return ops.scan_exclusive_u8i32(x, ws=ws)  # (y, total): the byte scan has one form
    if op == "rows":
        f = ops.scan_rows_i32 if case["kind"] == "i32" else ops.scan_rows_f32
        return f(x, exclusive=case["excl"], ws=ws)
    if op == "compact":
        out, idx, count = ops.compact_by_mask_f32(x, st["mask"], with_idx=case["idx"],
                                                  out=st["out"], idx_out=st["idx"], ws=ws)
        return (out, idx, count) if case["idx"] else (out, count)
    if op == "split":
        return ops.split_by_flags_u32(x, st["mask"], ws=ws)
    if op == "radix":
        kind, perm = case["kind"], case["perm"]
        if kind == "u32":
            keys, idx = ops.radix_sort_u32(x, with_perm=perm, ws=ws)
        else:
            f = {"i32": ops.radix_sort_i32, "f32": ops.radix_sort_f32,
                 "f16": ops.radix_sort_f16}[kind]
            keys, idx = f(x, descending=case["desc"], with_perm=perm, ws=ws)
        return (keys, idx) if perm else keys
    if op == "sort_rows":
        return ops.radix_sort_rows_f32(x, descending=case["desc"], ws=ws)
    if op == "topp_cutoff":
        return ops.topp_cutoff_f32(x, case["p"], ws=ws)
    if op == "topp_sample":
        return ops.topp_sample_f32(x, st["theta"], case["p"], with_cutoff=True, ws=ws,
                                   scratch_buf=st["scratch"])
    if op == "weighted":
        return ops.weighted_sample_f32(x, st["theta"], ws=ws)
    return ops.topk_rows_f32(x, case["k"], largest=case["largest"], ws=ws,
                             scratch_buf=st["scratch"])


# ---------------------------------------------------------------- what a pass cannot do without

_BYTES = {"i32": 4, "u32": 4, "f32": 4, "f16": 2, "u8": 1}


def work(case):
    op = case["op"]
    if op in ("scan", "rows"):
        n = case["n"] if op == "scan" else case["rows"] * case["len"]
        return {"bytes": n * (_BYTES[case["kind"]] + 4), "flops": n}
    if op == "compact":
        n = case["n"]
        kept = int(n * case["keep"])
        return {"bytes": n * 5 + kept * (8 if case["idx"] else 4) + 4, "flops": n}
    if op == "split":
        n = case["n"]
        return {"bytes": n * (4 + 1 + 4 + 4) + 4, "flops": n}
    if op == "radix":
        n, b = case["n"], _BYTES[case["kind"]]
        return {"bytes": n * (2 * b + (4 if case["perm"] else 0)), "flops": n}
    rows, length = case["rows"], case["len"]
    n = rows * length
    if op == "sort_rows":
        return {"bytes": n * 12, "flops": n}
    if op == "topk":
        return {"bytes": n * 4 + rows * case["k"] * 8, "flops": n}
    if op == "topp_cutoff":  # a row up to its cutoff: about a quarter of it here
        return {"bytes": n + rows * 4, "flops": n // 4}
    return {"bytes": n * 4 + rows * 12, "flops": n}


# ---------------------------------------------------------------- tolerances

def tolerance(case):
    op = case["op"]
    if op in ("scan", "rows"):
        if case["kind"] in ("i32", "u8"):
            return "exact"
        # 32-bit sums of values in [-1, 1) in any order: four times what the
        # comparison with 64-bit sums shows at 2^28 elements (rel 7.8e-7, max 1.5e-6)
        return {"rel": 3e-6, "max": 6e-6}
    if op in ("topp_sample", "topp_cutoff", "weighted"):
        # An index where a running sum crosses a threshold: 32-bit sums in
        # another order move it to a neighbour in some rows (against 64-bit
        # sums in up to 5 % of rows of 131072 at p <= 0.95, 11 % of rows of
        # 262144 in one batch of 64); two rows of a small batch.
        return {"differ": min(0.75, max(0.15, 2.0 / case["rows"]))}
    return "exact"


# ---------------------------------------------------------------- 64 bits, torch alone

def _code64(x):
    """Floating-point keys as integers in IEEE 754 totalOrder."""
    if x.dtype == torch.float16:
        b = x.view(torch.int16).long() & 0xFFFF
        return torch.where(b >= 0x8000, 0xFFFF - b, b + 0x8000)
    b = x.view(torch.int32).long() & 0xFFFFFFFF
    return torch.where(b >= 0x80000000, 0xFFFFFFFF - b, b + 0x80000000)


def _first(hit, default):
    """Index of the first true entry of every row, `default` where none."""
    idx = hit.to(torch.uint8).argmax(dim=1)
    return torch.where(hit.any(dim=1), idx, default)


def exact(case, seed):
    st = _inputs(case, seed)
    x, op = st["x"], case["op"]
    if op in ("scan", "rows"):
        whole = case["kind"] in ("i32", "u8")
        wide = x.to(torch.int64 if whole else torch.float64)
        y = torch.cumsum(wide, dim=-1)
        total = y[-1:] if op == "scan" else None
        if case["excl"] or case["kind"] == "u8":
            y = torch.cat((torch.zeros_like(y[..., :1]), y[..., :-1]), dim=-1)
        y = y.to(torch.int32) if whole else y
        return (y, total.to(torch.int32)) if case["kind"] == "u8" else y
    if op == "compact":
        keep = torch.nonzero(st["mask"]).squeeze(1)
        out = torch.zeros_like(x)
        out[: keep.numel()] = x[keep]
        count = torch.tensor([keep.numel()], dtype=torch.int32, device=x.device)
        if not case["idx"]:
            return out, count
        idx = torch.zeros(x.numel(), dtype=torch.int32, device=x.device)
        idx[: keep.numel()] = keep.to(torch.int32)
        return out, idx, count
    if op == "split":
        flagged = torch.nonzero(st["mask"]).squeeze(1)
        order = torch.cat((flagged, torch.nonzero(st["mask"] == 0).squeeze(1)))
        n_true = torch.tensor([flagged.numel()], dtype=torch.int32, device=x.device)
        return x[order], order.to(torch.int32), n_true
    if op in ("radix", "sort_rows"):
        if op == "sort_rows" or case["kind"] in ("f32", "f16"):
            code, desc = _code64(x), case["desc"]
        elif case["kind"] == "u32":
            code, desc = x.long() & 0xFFFFFFFF, False
        else:
            code, desc = x.long(), case["desc"]
        order = torch.sort(code, dim=-1, descending=desc, stable=True)[1]
        keys = torch.gather(x, -1, order)
        return (keys, order.to(torch.int32)) if op == "sort_rows" or case["perm"] else keys
    if op == "topk":
        order = torch.sort(_code64(x), dim=1, descending=case["largest"], stable=True)[1]
        order = order[:, : case["k"]]
        return torch.gather(x, 1, order).contiguous(), order.to(torch.int32).contiguous()
    length = case["len"]
    if op == "weighted":
        s = torch.cumsum(x.double(), dim=1)
        u = st["theta"].double()[:, None] * s[:, -1:]
        return _first(s > u, length - 1).to(torch.int32)
    p = float(torch.tensor(case["p"], dtype=torch.float32))
    if op == "topp_cutoff":
        return _first(torch.cumsum(x.double(), dim=1) >= p, length - 1).to(torch.int32)
    order = torch.sort(_code64(x), dim=1, descending=True, stable=True)[1]
    s = torch.cumsum(torch.gather(x, 1, order).double(), dim=1)
    cut = _first(s >= p, length - 1)
    u = st["theta"].double()[:, None] * torch.gather(s, 1, cut[:, None])
    pos = torch.arange(length, device=x.device)[None, :]
    j = _first((s > u) & (pos <= cut[:, None]), cut)
    return torch.gather(order, 1, j[:, None]).squeeze(1).to(torch.int32), cut.to(torch.int32)
