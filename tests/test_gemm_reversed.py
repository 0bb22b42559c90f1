"""GEMMs whose operands or result run backwards along tiles or k-steps.

A range-checked direct copy adds a scalar offset (tile and k-step) and a lane
offset as unsigned 32-bit numbers; the hardware checks the lane's against what
the scalar one leaves of the buffer.  An order that runs backwards has negative
parts, which must not become scalar offsets: every copy is replayed on the host
with the kernel's 32-bit arithmetic.  On the GPU the products are compared with
the fp64 oracle: products are exact in fp32 and the sums have at most 512 terms.
Negative parts also put a kernel in 64-bit indices, of which some forms end the
compiler; the code-object checks compile these configurations (COMPILED).
"""
import tempfile

import numpy as np
import pytest

import synth_inputs as S
from oracle import gemm as OG
from oracle import genexpr as GX
from oracle import layout as OL
from oracle import remap as OR
from tests.gpu_util import need_gpu, say
from tests.test_generated_host import HARNESS_GEMM, _compile_and_run

# orders of a matrix: rows or columns backwards, the 16-byte vectors of a row
# or column backwards, 64 x 64 tiles backwards
EXPRS = {"rows": ("(n0-1-i)*n1+j", ["n0-1-x/n1", "x%n1"]),
         "columns": ("(n1-1-j)*n0+i", ["x%n0", "n1-1-x/n0"]),
         "vectors of a row": ("i*n1+(n1/8-1-j/8)*8+j%8", ["x/n1", "(n1/8-1-(x%n1)/8)*8+x%8"]),
         "vectors of a column": ("j*n0+(n0/8-1-i/8)*8+i%8", ["(n0/8-1-(x%n0)/8)*8+x%8", "x/n0"])}
ORDERS = ["Row", "Col", *EXPRS, "tiles"]  # and "all": every element backwards (C)


def _layouts(L, order, m, n):
    """The library's layout and the oracle's."""
    if order in EXPRS:
        return L.as_layout(L.GenPExpr([m, n], *EXPRS[order])), OL.as_layout(GX.expr_genp([m, n], *EXPRS[order]))
    if order == "all":
        return L.as_layout(L.GenP("reverse", [m, n])), OL.as_layout(OL.reverse_genp(m, n))
    if order == "tiles":
        return (L.TileOrderBy(L.GenP("reverse", [m // 64, n // 64]), L.Row(64, 64)),
                OL.TileOrderBy(OL.reverse_genp(m // 64, n // 64), OL.Row(64, 64)))
    return L.as_layout(getattr(L, order)(m, n)), OL.as_layout(getattr(OL, order)(m, n))


TILE = dict(bm=128, bn=128, bk=64, wm=64, wn=64)
# whole tiles, tiles padded along m and n, and along k; one tile and several
SIZES = [(256, 256, 256), (320, 192, 128), (200, 136, 72), (520, 264, 200)]
PAIRS = [(a, b) for a in ORDERS for b in ORDERS if not {a, b} <= {"Row", "Col"}]

HARNESS = r"""
template <class GT, class GK, class GL, class OK>
static void check(const char* what, u64 ntile, u64 nvec, u64 bytes, GT gt, GK gk, GL gl, OK ok) {
  for (u64 t = 0; t < ntile; ++t) for (u64 kt = 0; kt < KT; ++kt) for (u64 tid = 0; tid < NT; ++tid)
    for (u64 u = 0; u < nvec; ++u) {
      const unsigned soff = (unsigned)((long long)gt(t) + (long long)gk(kt)) * 2u;
      const unsigned off = (unsigned)gl(tid, u) * 2u;
      if (soff > bytes) FAIL("%s: scalar offset outside the operand", what);
      if (ok(t, kt, tid, u) && (u64)soff + off + 16 > bytes) FAIL("%s: copy outside the operand", what);
    }
}
#ifndef A_SOFF  // the scalar part of every separable offset
#define A_SOFF A_SEP
#define B_SOFF B_SEP
#endif
int main() {
#if DIRECT_LDS && A_BUF && A_SOFF
  check("A", GEMM_MT, A_NV, A_BYTES, [](u64 t) { return a_gt(t); }, [](u64 kt) { return a_gk(kt); },
    [](u64 tid, u64 u) { return a_gl(tid, u); }, [](u64 t, u64 kt, u64 tid, u64 u) {
#if A_EDGE
      return a_ok(t, kt, tid, u) != 0;
#else
      return true;
#endif
    });
#endif
#if DIRECT_LDS && B_BUF && B_SOFF
  check("B", GEMM_NT, B_NV, B_BYTES, [](u64 t) { return b_gt(t); }, [](u64 kt) { return b_gk(kt); },
    [](u64 tid, u64 u) { return b_gl(tid, u); }, [](u64 t, u64 kt, u64 tid, u64 u) {
#if B_EDGE
      return b_ok(t, kt, tid, u) != 0;
#else
      return true;
#endif
    });
#endif
  printf("ok\n");
  return 0;
}
"""


def _cases():
    return [(size, a, b) for size in SIZES for a, b in PAIRS
            if size[0] % 64 == 0 and size[1] % 64 == 0 and size[2] % 64 == 0 or "tiles" not in (a, b)]


@pytest.mark.parametrize("size", SIZES)
def test_copies_stay_inside_the_operands(lego, size):
    M, N, K = size
    direct = 0
    for s, a, b in _cases():
        if s != size:
            continue
        for tile in ({}, TILE):
            src = lego.plan_source("gemm", M=M, N=N, K=K, dtype="f16", a=_layouts(lego, a, M, K)[0],
                                   b=_layouts(lego, b, K, N)[0], **tile)
            direct += "#define DIRECT_LDS 1" in src
            with tempfile.TemporaryDirectory() as tmp:
                assert _compile_and_run(src, HARNESS, tmp).strip() == "ok", (a, b, tile)
    assert direct >= 20


def test_lane_offsets_of_large_operands(lego):
    """Operands of 2 GiB and more are copied through addresses: their lane
    offsets keep the kernel's index type, 64 bits where a tile spans 2^32
    elements; 32-bit ones stay with the range-checked copies."""
    for K, loc in ((1 << 20, "u32"), (1 << 25, "IDX_T")):
        src = lego.plan_source("gemm", M=512, N=256, K=K, dtype="f16")
        assert f"#define A_SOFF {int(loc == 'u32')}\n" in src and f"#define A_LOC_T {loc}\n" in src
        assert f"#define A_BUF {int(loc == 'u32')}\n" in src
        assert ("#define IDX_T i64\n" in src) == (loc == "IDX_T")


# orders of A, B and C and the tile of the products on the GPU
PRODUCTS = [((256, 256, 256), "rows", "columns", "Row", TILE), ((256, 256, 512), "columns", "rows", "Row", {}),
            ((320, 192, 128), "tiles", "vectors of a row", "Row", TILE),
            ((320, 192, 128), "rows", "vectors of a column", "Row", TILE),
            ((200, 136, 72), "vectors of a column", "rows", "Row", {}),
            ((520, 264, 200), "columns", "vectors of a column", "Row", TILE),
            ((520, 264, 200), "vectors of a row", "rows", "Row", TILE),
            # one operand or C alone
            ((256, 256, 256), "rows", "Col", "Row", TILE), ((320, 192, 128), "Row", "tiles", "Row", TILE),
            ((640, 64, 64), "Row", "Col", "all", {}), ((168, 768, 384), "Col", "Row", "all", {}),
            ((256, 384, 320), "Row", "Col", "rows", TILE), ((200, 136, 72), "Col", "Row", "columns", {})]
# compiled only: sizes at which the compiler ended
COMPILED = [((1024, 1024, 1024), "Row", "Col", "rows", {}), ((512, 1024, 1088), "Col", "Row", "rows", {}),
            ((1024, 1024, 384), "Row", "Col", "rows", TILE), ((2560, 2560, 320), "Row", "rows", "Row", {}),
            ((2560, 2560, 320), "vectors of a row", "Col", "Row", {})]


def _case(lego, size, a, b, c, tile):
    """Keyword arguments of the call, and the oracle's layouts of A, B and C."""
    M, N, K = size
    (la, oa), (lb, ob), (lc, oc) = (_layouts(lego, o, m, n) for o, m, n in ((a, M, K), (b, K, N), (c, M, N)))
    return dict(a=la, b=lb, c=lc, **tile), oa, ob, oc


def compiled_cases(lego):
    return [dict(zip("MNK", case[0]), dtype="f16", **_case(lego, *case)[0]) for case in PRODUCTS + COMPILED]


@pytest.mark.parametrize("i", range(len(PRODUCTS)))
def test_product_sources_on_host(lego, i):
    M, N, K = PRODUCTS[i][0]
    kw = _case(lego, *PRODUCTS[i])[0]
    src = lego.plan_source("gemm", M=M, N=N, K=K, dtype="f16", **kw)
    with tempfile.TemporaryDirectory() as tmp:
        assert _compile_and_run(src, HARNESS, tmp).strip() == "ok"
        assert _compile_and_run(src, HARNESS_GEMM, tmp).strip() == "ok"


@pytest.mark.gpu
@pytest.mark.parametrize("i", range(len(PRODUCTS)))
def test_products(lego, i):
    import torch
    dev = need_gpu()
    M, N, K = PRODUCTS[i][0]
    kw, oa, ob, oc = _case(lego, *PRODUCTS[i])
    dtype = ("f16", "bf16")[i % 2]
    say(f"gemm reversed {PRODUCTS[i]} {dtype} plan={lego.gemm_plan(M, N, K, dtype, **kw)}")
    a = S.tensor(M * K, dtype, dist="normal", seed=S.SEED_A)
    b = S.tensor(K * N, dtype, dist="normal", seed=S.SEED_B)
    a_bits = OR.remap(OL.as_layout(OL.Row(M, K)), oa, S.as_numpy_bits(a))
    b_bits = OR.remap(OL.as_layout(OL.Row(K, N)), ob, S.as_numpy_bits(b))
    d_a = torch.from_numpy(a_bits.view(np.int16).copy()).view(a.dtype).to(dev)
    d_b = torch.from_numpy(b_bits.view(np.int16).copy()).view(b.dtype).to(dev)
    c = torch.full((M * N,), float("nan"), dtype=torch.float32, device=dev)
    lego.gemm(d_a, d_b, c, M, N, K, dtype, **kw)
    torch.cuda.synchronize()
    r = OG.gemm(a_bits, b_bits, oa, ob, dtype)
    got = OR.remap(oc, OL.as_layout(OL.Row(M, N)), c.cpu().numpy()).reshape(M, N)
    assert np.isfinite(got).all()
    ok, mre, fre = OG.check_tolerance(got, r)
    # fp32 sums of at most 512 exact products: 2-norm error below 512 * 2^-24
    assert ok and fre < 512 * 2.0 ** -24, (mre, fre)
