"""Box remaps of extents without the factors that LDS tiles need, and box
grids that neither the XCDs nor bands of box rows divide: transposes and
antidiagonal orders around the box side, in grids of fewer than 8 boxes,
one band, whole bands and a band left over.  On the host every element of the
generated index code is compared with the oracle's remap; on the GPU every
byte."""
import os
import tempfile

import numpy as np
import pytest

from oracle import layout as OL
from oracle import remap as OR
from tests.gpu_util import bits, need_gpu, say
from tests.test_generated_host import HARNESS_REMAP, _compile_and_run

# (kind, rows, columns, element bytes)
CASES = [("transpose", 64, 65, 4), ("transpose", 65, 63, 8), ("transpose", 127, 129, 2), ("transpose", 449, 511, 8),
         ("transpose", 1001, 999, 1), ("transpose", 193, 2047, 4), ("transpose", 2050, 70, 2), ("transpose", 517, 1207, 8),
         ("antidiag", 65, 65, 4), ("antidiag", 127, 127, 8), ("antidiag", 500, 500, 2), ("antidiag", 643, 643, 4),
         ("antidiag", 1025, 1025, 1), ("antidiag", 832, 832, 2)]


def _layouts(L, case):
    kind, m, n, _ = case
    other, oother = ((L.as_layout(L.Col(m, n)), OL.as_layout(OL.Col(m, n))) if kind == "transpose" else
                     (L.as_layout(L.GenP("antidiag", [m, n])), OL.as_layout(OL.antidiag_genp(m))))
    return L.as_layout(L.Row(m, n)), other, OL.as_layout(OL.Row(m, n)), oother


@pytest.mark.parametrize("i", range(len(CASES)))
def test_box_sources_on_host(lego, i):
    row, other, orow, oother = _layouts(lego, CASES[i])
    m, n, elem = CASES[i][1:]
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "out.bin")
        for a, b, oa, ob in ((row, other, orow, oother), (other, row, oother, orow)):
            src = lego.plan_source("remap", a, b, param=elem)
            if (m // 64) * (n // 64) >= 64:
                # (32-bit index code, also for points past the extents)
                assert "#define LEGO_REMAP_BOX 1" in src and "#define IDX_T u32" in src
            _compile_and_run(src, HARNESS_REMAP, tmp, [out])
            perm = np.fromfile(out, dtype=np.int64)
            assert (perm == OR.remap(oa, ob, np.arange(m * n, dtype=np.int64))).all(), CASES[i]


@pytest.mark.gpu
@pytest.mark.parametrize("i", range(len(CASES)))
def test_box_remaps(lego, i):
    import torch
    dev = need_gpu()
    row, other, orow, oother = _layouts(lego, CASES[i])
    m, n, elem = CASES[i][1:]
    src = torch.from_numpy(np.random.default_rng(i).integers(0, 256, m * n * elem, dtype=np.uint8))
    src = src.view({1: torch.uint8, 2: torch.int16, 4: torch.int32, 8: torch.int64}[elem])
    d_src = src.to(dev)
    for a, b, oa, ob in ((row, other, orow, oother), (other, row, oother, orow)):
        say(f"remap {CASES[i]} plan={lego.remap_plan(a, b, elem)['info']}")
        d_dst = torch.full_like(d_src, -1 if elem > 1 else 255)
        lego.remap(a, b, d_src, d_dst)
        torch.cuda.synchronize()
        assert (bits(d_dst.cpu()) == OR.remap(oa, ob, bits(src))).all(), CASES[i]


# Maps that LDS tiles and boxes both take, on both sides of the rule that
# chooses: (rows, columns, tile rows, tile columns (0: a transpose), tile order,
# order inside a tile, element bytes, path there, path back)
ROUTES = [(2097, 2088, 9, 24, "Row", "Col", 1, "lds", "lds"), (1197, 1176, 9, 24, "Row", "Col", 1, "box", "box"),
          (2100, 2100, 10, 10, "Row", "Row", 1, "lds", "lds"), (3300, 3300, 10, 6, "Row", "Col", 2, "lds", "lds"),
          (1500, 1490, 10, 10, "Col", "Row", 4, "box", "box"), (2100, 2100, 0, 0, "", "", 1, "box", "box"),
          (15000, 15000, 12, 20, "Row", "Row", 1, "lds", "lds"), (15001, 15001, 0, 0, "", "", 1, "box", "box"),
          (7298, 7300, 0, 0, "", "", 4, "lds", "lds"), (9125, 9125, 0, 0, "", "", 4, "box", "box"),
          (10290, 10290, 14, 14, "Row", "Col", 2, "lds", "lds")]


def _route_layouts(L, case):
    m, n, t, u, outer, inner = case[:6]
    if not t:
        return L.as_layout(L.Row(m, n)), L.as_layout(L.Col(m, n))
    return L.as_layout(L.Row(m, n)), L.TileOrderBy(getattr(L, outer)(m // t, n // u), getattr(L, inner)(t, u))


def test_tiles_or_boxes(lego):
    for case in ROUTES:
        row, other = _route_layouts(lego, case)
        got = tuple(lego.remap_plan(a, b, case[6])["path"] for a, b in ((row, other), (other, row)))
        assert got == case[7:], (case, got)


@pytest.mark.parametrize("n,elem,order", [(6200, 8, "bands1-xcd"), (6300, 8, "row"), (8300, 4, "bands1-xcd"),
                                          (9001, 4, "row"), (9000, 4, "row"), (12345, 2, "bands1-xcd"), (14001, 2, "row")])
def test_order_of_boxes_reading_far_antidiagonals(lego, n, elem, order):
    plan = lego.remap_plan(lego.as_layout(lego.GenP("antidiag", [n, n])), lego.as_layout(lego.Row(n, n)), elem)
    assert plan["path"] == "box" and plan["info"].split()[2] == order, plan["info"]


@pytest.mark.parametrize("i", [i for i in range(len(ROUTES)) if ROUTES[i][0] < 5000])
def test_tile_and_box_sources_on_host(lego, i):
    row, other = _route_layouts(lego, ROUTES[i])
    orow, oother = _route_layouts(OL, ROUTES[i])
    m, n = ROUTES[i][:2]
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "out.bin")
        for a, b, oa, ob in ((row, other, orow, oother), (other, row, oother, orow)):
            _compile_and_run(lego.plan_source("remap", a, b, param=ROUTES[i][6]), HARNESS_REMAP, tmp, [out])
            perm = np.fromfile(out, dtype=np.int64)
            assert (perm == OR.remap(oa, ob, np.arange(m * n, dtype=np.int64))).all(), ROUTES[i]


@pytest.mark.gpu
@pytest.mark.parametrize("i", [i for i in range(len(ROUTES)) if ROUTES[i][0] < 5000])
def test_tiles_and_boxes(lego, i):
    import torch
    dev = need_gpu()
    row, other = _route_layouts(lego, ROUTES[i])
    orow, oother = _route_layouts(OL, ROUTES[i])
    m, n, elem = ROUTES[i][0], ROUTES[i][1], ROUTES[i][6]
    src = torch.from_numpy(np.random.default_rng(i).integers(0, 256, m * n * elem, dtype=np.uint8))
    src = src.view({1: torch.uint8, 2: torch.int16, 4: torch.int32}[elem])
    d_src = src.to(dev)
    for a, b, oa, ob in ((row, other, orow, oother), (other, row, oother, orow)):
        say(f"remap {ROUTES[i]} plan={lego.remap_plan(a, b, elem)['info']}")
        d_dst = torch.full_like(d_src, -1 if elem > 1 else 255)
        lego.remap(a, b, d_src, d_dst)
        torch.cuda.synchronize()
        assert (bits(d_dst.cpu()) == OR.remap(oa, ob, bits(src))).all(), ROUTES[i]
