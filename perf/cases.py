"""Performance cases of the layout library: remaps, GEMMs and index maps, each
through the calls a program makes (``remap``, ``gemm``, ``apply_all_device``,
``inv_all_device``) on buffers and layouts it keeps.

The layouts of a shape are built once per process, as a program does that
feeds many tensors of one shape through them; ``prepare`` makes the tensors
and the output buffers.
"""
import functools
import math

import torch

import paper_2505_08091_amd as L

_DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "f64": torch.float64, "u8": torch.uint8}
_BYTES = {"f32": 4, "f16": 2, "bf16": 2, "f64": 8, "u8": 1}
_TILE = 64  # rows and columns of a tile of the blocked layouts


def _gemm(name, m, n, k, dtype, a="row", b="col", tile=""):
    return {"name": name, "op": "gemm", "m": m, "n": n, "k": k, "dtype": dtype, "a": a, "b": b, "tile": tile}


def _remap(name, kind, m, n, dtype):
    return {"name": name, "op": "remap", "kind": kind, "m": m, "n": n, "dtype": dtype}


def listed():
    return [
        # The smallest GEMM: 64x64 workgroup tiles of 16x16 wave tiles; the
        # time of a call.
        _gemm("gemm_f16_128", 128, 128, 128, "f16", tile="64x64x32x16x16"),
        # A GEMM whose tiles the program gives: 128x128x32, 64x64 wave tiles.
        _gemm("gemm_f16_1024", 1024, 1024, 1024, "f16", tile="128x128x32x64x64"),
        # Matrix product of two row-major matrices with the default plan, the
        # smallest of the sizes 2048, 4096, 8192 that the four Row/Col operand
        # variants are measured at.
        _gemm("gemm_f16_2048_row_row", 2048, 2048, 2048, "f16", b="row"),
        # A kept in Z order: the row-major A is stored so, then multiplied.
        _gemm("gemm_f16_4096_morton", 4096, 4096, 4096, "f16", a="morton", b="row"),
        # The largest GEMM, default plan.
        _gemm("gemm_bf16_8192", 8192, 8192, 8192, "bf16"),
        # Sizes that neither tiles nor 16-byte vectors divide.
        _gemm("gemm_bf16_odd", 1000, 777, 1001, "bf16", b="row"),
        # Row-major to 64x64 tiles in column-major tile order and back.
        _remap("blocked_f32_8192", "blocked", 8192, 8192, "f32"),
        # A transpose that the last-level cache holds, and one of odd extents.
        _remap("transpose_f32_2048", "transpose", 2048, 2048, "f32"),
        _remap("transpose_f16_odd", "transpose", 3001, 1999, "f16"),
        # Partial tiles: a compact matrix into zero-padded tiles and back.
        _remap("pad_crop_f32_odd", "pad", 3001, 1999, "f32"),
        # A whole matrix in antidiagonal (wavefront) order and back.
        _remap("antidiag_f32_4096", "antidiag", 4096, 4096, "f32"),
        # Forward and inverse index map of a tiled layout, every point.
        {"name": "index_i32_8192", "op": "index", "m": 8192, "n": 8192, "dtype": "i32"},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _extent(rng, lo, hi, step):
    return min(hi, max(step, _log_uniform(rng, lo, hi) // step * step))


def _whole_groups(m, rows):
    """One group of at most 8 tile rows, or whole groups of 8 (the default
    schedule).  The kernels of some other sizes abort the run-time compiler
    (a floating-point exception while it selects instructions)."""
    t = -(-m // rows)
    return t <= 8 or t % 8 == 0


def draw(rng):
    op = rng.choice(["gemm", "gemm", "gemm", "remap", "remap", "remap", "remap", "index"])
    if op == "gemm":
        a = rng.choice(["row", "row", "row", "col", "col", "morton"])
        # multiples of the tiles, of the 16-byte vectors, or neither
        step = rng.choice([64, 64, 8, 1])
        tile = rng.choice(["", "", "", "128x128x32x64x64"])
        m, n, k = (_extent(rng, 128, 8192, step) for _ in range(3))
        while not _whole_groups(m, 128 if tile else 256):
            m = _extent(rng, 128, 8192, step)
        if a == "morton":  # a square A of a power of two
            m = k = 1 << rng.randint(8, 12)
        c = _gemm("", m, n, k, rng.choice(["f16", "bf16"]), a=a, b=rng.choice(["row", "col"]), tile=tile)
    elif op == "remap":
        kind = rng.choice(["blocked", "transpose", "transpose", "morton", "pad", "pad", "antidiag"])
        dtype = rng.choice(["f32", "f32", "f16", "f16", "f64", "u8"])
        hi = 4096 if dtype == "f64" else 8192
        step = {"blocked": _TILE, "transpose": rng.choice([32, 1])}.get(kind, 1)
        m, n = (_extent(rng, 128, hi, step) for _ in range(2))
        if kind == "morton":
            m = n = 1 << rng.randint(7, 12)
        if kind == "antidiag":
            n = m
        c = _remap("", kind, m, n, dtype)
    else:
        m, n = (_extent(rng, 128, 8192, _TILE) for _ in range(2))
        c = {"op": "index", "m": m, "n": n, "dtype": rng.choice(["i32", "i64"])}
    c.pop("name", None)
    return c


def _up(x):
    return -(-x // _TILE) * _TILE


def _blocked(m, n):
    return L.TileOrderBy(L.Col(m // _TILE, n // _TILE), L.Row(_TILE, _TILE))


@functools.lru_cache(maxsize=None)
def _layout(kind, m, n):
    if kind == "row":
        return L.as_layout(L.Row(m, n))
    if kind == "col" or kind == "transpose":
        return L.as_layout(L.Col(m, n))
    if kind in ("morton", "antidiag"):
        return L.as_layout(L.GenP(kind, [m, n]))
    if kind == "blocked":
        return _blocked(m, n)
    if kind == "compact":  # m x n kept compact, seen in the padded extents
        return L.ExpandBy([m, n], [_up(m), _up(n)], L.as_layout(L.Row(_up(m), _up(n))))
    raise ValueError(kind)


def _values(n, dtype, g, normal=False):
    if dtype == "u8":
        return torch.randint(0, 256, (n,), generator=g, device="cuda", dtype=torch.uint8)
    if normal:
        return torch.randn(n, generator=g, device="cuda", dtype=torch.float32).to(_DT[dtype])
    return torch.rand(n, generator=g, device="cuda", dtype=torch.float32).mul_(2).sub_(1).to(_DT[dtype])


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _gemm_inputs(case, seed):
    g = _generator(seed)
    m, n, k, dtype = case["m"], case["n"], case["k"], case["dtype"]
    return _values(m * k, dtype, g, dtype == "bf16"), _values(k * n, dtype, g, dtype == "bf16")


def _remap_input(case, seed):
    return _values(case["m"] * case["n"], case["dtype"], _generator(seed))


def prepare(case, seed):
    m, n = case["m"], case["n"]
    s = {"op": case["op"]}
    if case["op"] == "gemm":
        k = case["k"]
        s["A"], s["B"] = _gemm_inputs(case, seed)
        s["C"] = torch.empty(m * n, dtype=torch.float32, device="cuda")
        s["size"] = (m, n, k, case["dtype"])
        s["kw"] = {"a": _layout(case["a"], m, k), "b": _layout(case["b"], k, n)}
        if case["tile"]:
            s["kw"].update(zip(("bm", "bn", "bk", "wm", "wn"), map(int, case["tile"].split("x"))))
        if case["a"] == "morton":
            s["row"], s["Z"] = _layout("row", m, k), torch.empty_like(s["A"])
    elif case["op"] == "remap":
        kind = case["kind"]
        s["X"] = _remap_input(case, seed)
        if kind == "pad":
            s["src"], s["dst"] = _layout("compact", m, n), _layout("blocked", _up(m), _up(n))
        else:
            s["src"], s["dst"] = _layout("row", m, n), _layout(kind, m, n)
        s["Y"] = torch.empty(s["dst"].phys_size(), dtype=s["X"].dtype, device="cuda")
        s["back"] = None if kind == "transpose" else torch.empty_like(s["X"])
    else:
        dt = torch.int32 if case["dtype"] == "i32" else torch.int64
        # the values are the layout's alone; the seed picks the tile order
        order = L.Col if seed % 2 else L.Row
        s["layout"] = _index_layout(m, n, order is L.Col)
        s["apply"] = torch.empty(m * n, dtype=dt, device="cuda")
        s["inv"] = torch.empty(m * n, 2, dtype=dt, device="cuda")
    return s


@functools.lru_cache(maxsize=None)
def _index_layout(m, n, col):
    order = L.Col if col else L.Row
    return L.TileOrderBy(order(m // _TILE, n // _TILE), L.Row(_TILE, _TILE))


def run(s):
    if s["op"] == "gemm":
        a = s["A"]
        if "Z" in s:
            a = s["Z"]
            L.remap(s["row"], s["kw"]["a"], s["A"], a)
        L.gemm(a, s["B"], s["C"], *s["size"], **s["kw"])
        return {"C": s["C"], "A": a} if "Z" in s else {"C": s["C"]}
    if s["op"] == "remap":
        L.remap(s["src"], s["dst"], s["X"], s["Y"])
        if s["back"] is None:
            return {"Y": s["Y"]}
        L.remap(s["dst"], s["src"], s["Y"], s["back"])
        return {"Y": s["Y"], "back": s["back"]}
    L.apply_all_device(s["layout"], s["apply"])
    L.inv_all_device(s["layout"], s["inv"])
    return {"apply": s["apply"], "inv": s["inv"]}


def work(case):
    m, n = case["m"], case["n"]
    if case["op"] == "gemm":
        k = case["k"]
        b = 2 * (m * k + k * n) + 4 * m * n
        if case["a"] == "morton":  # A read and stored in Z order
            b += 4 * m * k
        return {"bytes": b, "flops": 2 * m * n * k}
    if case["op"] == "remap":
        e = _BYTES[case["dtype"]]
        y = _up(m) * _up(n) if case["kind"] == "pad" else m * n
        if case["kind"] == "transpose":
            return {"bytes": 2 * m * n * e, "flops": 0}
        # there: m n read, y written; back: m n of the y read, m n written
        return {"bytes": (m * n + y + 2 * m * n) * e, "flops": 0}
    return {"bytes": 3 * m * n * (4 if case["dtype"] == "i32" else 8), "flops": 0}


def tolerance(case):
    # Remaps and index maps are exact.  GEMM: products of 16-bit values are
    # exact in 32 bits, sums of K of them are not: 6e-7 off the 64-bit result
    # (2-norm) at K = 8192.
    if case["op"] == "gemm":
        return {"rel": 2.5e-6, "max": 2e-5}
    return "exact"


def _tiled(x, m, n, col=True):
    """An m x n matrix in 64x64 tiles, column-major (or row-major) tile order."""
    t = x.reshape(m // _TILE, _TILE, n // _TILE, _TILE)
    return t.permute(2, 0, 1, 3).reshape(-1) if col else t.permute(0, 2, 1, 3).reshape(-1)


def _morton(x, n):
    """An n x n matrix in Z order, column bits at the even positions."""
    p = torch.arange(n * n, device=x.device)
    i = torch.zeros_like(p)
    j = torch.zeros_like(p)
    for b in range(n.bit_length() - 1):
        j |= ((p >> (2 * b)) & 1) << b
        i |= ((p >> (2 * b + 1)) & 1) << b
    return x.reshape(-1)[i * n + j]


def _antidiag(x, n):
    """An n x n matrix antidiagonal by antidiagonal, each with rows increasing."""
    r = torch.arange(n, device=x.device)
    order = torch.argsort(((r[:, None] + r[None, :]) * n + r[:, None]).reshape(-1))
    return x.reshape(-1)[order]


def exact(case, seed):
    m, n = case["m"], case["n"]
    if case["op"] == "gemm":
        k = case["k"]
        A, B = (t.double() for t in _gemm_inputs(case, seed))
        a = A.reshape(k, m).t().contiguous() if case["a"] == "col" else A.reshape(m, k)
        b = B.reshape(n, k).t().contiguous() if case["b"] == "col" else B.reshape(k, n)
        out = {"C": torch.mm(a, b).reshape(-1)}
        if case["a"] == "morton":
            out["A"] = _morton(A, k)
        return out
    if case["op"] == "remap":
        x = _remap_input(case, seed)
        kind = case["kind"]
        if kind == "transpose":
            return {"Y": x.reshape(m, n).t().reshape(-1).double()}
        if kind == "blocked":
            y = _tiled(x, m, n)
        elif kind == "pad":
            y = _tiled(torch.nn.functional.pad(x.reshape(m, n), (0, _up(n) - n, 0, _up(m) - m)), _up(m), _up(n))
        else:
            y = _morton(x, n) if kind == "morton" else _antidiag(x, n)
        return {"Y": y.double(), "back": x.double()}
    return None  # whole numbers
