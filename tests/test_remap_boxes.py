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
