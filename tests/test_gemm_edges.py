"""GEMM operands whose rows or extents do not fit 16-byte vectors or tiles.

Vectors at element alignment: the loads of such an operand are moved inside
the operand at its edges and cut in registers.  On the host, the generated
functions are run for every tile and k-step: every load must lie inside the
operand and deliver the elements that the plain element description gives,
and the elements of the last k-step that do not exist must become zero.  On
the GPU the same configurations, and those whose range-checked direct copies
take the last k-step first, are compared with the fp64 oracle: products are
exact in fp32 and the sums have at most 2049 terms, far inside the tolerance.
"""
import tempfile

import numpy as np
import pytest

import synth_inputs as S
from oracle import gemm as OG
from oracle import layout as OL
from tests.gpu_util import need_gpu, say
from tests.test_generated_host import HARNESS_GEMM, _compile_and_run

# the smallest extents that take vectors of 8, one more and one less, around
# the tiles of 32, 64 and 128, and K around one and two k-steps
SIZES = [(8, 8, 8), (9, 15, 9), (33, 31, 63), (65, 63, 65), (63, 130, 129), (129, 65, 191), (257, 77, 401)]
TILES = {"default": {}, "128 wide": dict(bm=128, bn=128, bk=64, wm=64, wn=32),
         "128 wide, 32 deep": dict(bm=128, bn=128, bk=32, wm=64, wn=64),
         "256 wide": dict(bm=256, bn=256, bk=64, wm=128, wn=64)}
CASES = [(size, tile, la, lb) for size in SIZES for tile in TILES for la, lb in
         (("Row", "Row"), ("Row", "Col"), ("Col", "Row"), ("Col", "Col"))
         if tile == "default" or size[2] in (9, 65, 191)]
# multiples of the 16-byte vectors that tiles do not divide (direct copies,
# the last k-step first), one k-step, several tiles of waves along K, and
# grouped schedules with a ragged last group (more than 8 tile rows)
DIRECT = [((200, 136, 72), {}), ((72, 264, 40), {}), ((264, 72, 1032), {}), ((712, 72, 136), {}),
          ((264, 136, 200), dict(bm=128, bn=128, bk=64, wm=64, wn=32)), ((1096, 256, 72), dict(bm=64, bn=64, bk=32, wm=32, wn=32)),
          ((520, 520, 2048), dict(max_workgroups=3)),
          # 256x128 and 128x256 tiles, and tile counts that 8 does not divide
          # in XCD order (18 and 15 * 9 tiles)
          ((520, 264, 200), dict(bm=256, bn=128, bk=64, wm=64, wn=64)),
          ((264, 520, 200), dict(bm=128, bn=256, bk=64, wm=64, wn=64)),
          ((712, 328, 72), dict(bm=128, bn=128, bk=64, wm=64, wn=32)),
          ((960, 576, 832), dict(bm=64, bn=64, bk=64, wm=32, wn=32)),
          # waves along K, several tiles a workgroup, each tile begun with its cut
          # last k-step: 2, 4 and 7 k-steps for the 4 waves
          ((96, 88, 72), dict(max_workgroups=3)), ((72, 72, 200), dict(max_workgroups=3)),
          ((136, 200, 200), dict(max_workgroups=7))]

HARNESS = r"""
template <class GP, class GC, class NV, class GL, class OK>
static void check(const char* what, u64 ntile, u64 nvec, u64 size, GP gp, GC gc, NV nv, GL gl, OK ok) {
  for (u64 t = 0; t < ntile; ++t) for (u64 kt = 0; kt < KT; ++kt) for (u64 tid = 0; tid < NT; ++tid)
    for (u64 u = 0; u < nvec; ++u) {
      const bool last = kt == KT - 1;
      const long long o = last ? (long long)gc(t, tid, u) : gp(t, kt, tid, u);
      if (o < 0 || o + 8 > (long long)size) FAIL("%s load outside the operand", what);
      const u64 n = last ? (u64)nv(t, tid, u) : 8;
      if (n > 8) FAIL("%s element count", what);
      for (u64 e = 0; e < 8; ++e) {
        const bool have = e < n;
        const bool want = ok(t, kt, tid, 8 * u + e);
        if (want && !have) FAIL("%s element lost", what);
        if (last && have && !want) FAIL("%s element past the end kept", what);
        // a vector of n elements was loaded 8 - n elements early
        if (want && (u64)o + (8 - n) + e != gl(t, kt, tid, 8 * u + e)) FAIL("%s wrong element", what);
      }
    }
}
int main() {
#if A_UA
  check("A", GEMM_MT, A_NV / 8, GEMM_M * GEMM_K,
    [](u64 t, u64 kt, u64 tid, u64 u) { return (long long)a_gt(t) + (long long)a_gk(kt) + ((long long)a_gp(t, tid, u) - (long long)a_gt(t)); },
    [](u64 t, u64 tid, u64 u) { return a_gc(t, tid, u); }, [](u64 t, u64 tid, u64 u) { return a_nv(t, tid, u); },
    [](u64 t, u64 kt, u64 tid, u64 u) { return (u64)a_gt(t) + (u64)a_gk(kt) + (u64)a_gl(tid, u); },
    [](u64 t, u64 kt, u64 tid, u64 u) {
#if A_EDGE
      return a_ok(t, kt, tid, u) != 0;
#else
      return true;
#endif
    });
#endif
#if B_UA
  check("B", GEMM_NT, B_NV / 8, GEMM_K * GEMM_N,
    [](u64 t, u64 kt, u64 tid, u64 u) { return (long long)b_gt(t) + (long long)b_gk(kt) + ((long long)b_gp(t, tid, u) - (long long)b_gt(t)); },
    [](u64 t, u64 tid, u64 u) { return b_gc(t, tid, u); }, [](u64 t, u64 tid, u64 u) { return b_nv(t, tid, u); },
    [](u64 t, u64 kt, u64 tid, u64 u) { return (u64)b_gt(t) + (u64)b_gk(kt) + (u64)b_gl(tid, u); },
    [](u64 t, u64 kt, u64 tid, u64 u) {
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


def _kw(L, size, tile, la, lb, dtype):
    M, N, K = size
    return dict(M=M, N=N, K=K, dtype=dtype, a=L.as_layout(getattr(L, la)(M, K)), b=L.as_layout(getattr(L, lb)(K, N)),
                **tile)


@pytest.mark.parametrize("i", range(len(CASES)))
def test_element_aligned_loads_on_host(lego, i):
    size, tile, la, lb = CASES[i]
    src = lego.plan_source("gemm", **_kw(lego, size, TILES[tile], la, lb, "f16"))
    if size[2] % 8 and (la, lb) == ("Row", "Col"):
        assert "#define A_UA 1" in src and "#define B_UA 1" in src
    with tempfile.TemporaryDirectory() as tmp:
        assert _compile_and_run(src, HARNESS, tmp).strip() == "ok", CASES[i]
        assert _compile_and_run(src, HARNESS_GEMM, tmp).strip() == "ok", CASES[i]


def test_other_row_orders_keep_element_loads(lego):
    """Rows that do not follow one another (here reversed) are not read past
    their ends: such an operand keeps the element loads."""
    rev = lego.as_layout(lego.GenP("reverse", [65, 65]))
    assert "#define A_UA 0" in lego.plan_source("gemm", M=65, N=65, K=65, dtype="f16", a=rev)


def _check(lego, size, tile, la, lb, dtype):
    import torch
    dev = need_gpu()
    kw = _kw(lego, size, tile, la, lb, dtype)
    M, N, K, _ = (kw.pop(k) for k in ("M", "N", "K", "dtype"))
    plan = lego.gemm_plan(M, N, K, dtype, **kw)
    say(f"gemm edges {size} {tile} A {la} B {lb} {dtype} plan={plan}")
    a = S.tensor(M * K, dtype, dist="normal", seed=S.SEED_A)
    b = S.tensor(K * N, dtype, dist="normal", seed=S.SEED_B)
    c = torch.full((M * N,), float("nan"), dtype=torch.float32, device=dev)
    lego.gemm(a.to(dev), b.to(dev), c, M, N, K, dtype, **kw)
    torch.cuda.synchronize()
    r = OG.gemm(S.as_numpy_bits(a), S.as_numpy_bits(b), OL.as_layout(getattr(OL, la)(M, K)),
                OL.as_layout(getattr(OL, lb)(K, N)), dtype)
    got = c.cpu().numpy().reshape(M, N)
    assert np.isfinite(got).all()
    ok, mre, fre = OG.check_tolerance(got, r)
    # fp32 sums of at most 2049 exact products: 2-norm error below 2049 * 2^-24
    assert ok and fre < 2049 * 2.0 ** -24, (mre, fre)
    return plan


@pytest.mark.gpu
@pytest.mark.parametrize("i", range(0, len(CASES), 3))
def test_element_aligned_operands(lego, i):
    size, tile, la, lb = CASES[i]
    _check(lego, size, TILES[tile], la, lb, ("f16", "bf16")[i % 2])


@pytest.mark.gpu
@pytest.mark.parametrize("la,lb", [("Row", "Col"), ("Col", "Row")])
@pytest.mark.parametrize("i", range(len(DIRECT)))
def test_padded_direct_copies(lego, i, la, lb):
    plan = _check(lego, *DIRECT[i], la, lb, ("f16", "bf16")[i % 2])
    assert " direct-lds " in plan, plan
    # waves along K, which walk padded tiles too, where the planner chose a
    # tile for these sizes, but not under a limit of 3 workgroups at 520 x 520
    along_k = "bm" not in DIRECT[i][1] and DIRECT[i][0] != (520, 520, 2048)
    assert ("x4k wave" in plan) == along_k, plan
    assert " persistent " in plan or not along_k, plan


def compiled_cases(lego):
    """The configurations that run on the GPU, for the code-object checks."""
    out = [_kw(lego, size, TILES[tile], la, lb, ("f16", "bf16")[i % 2])
           for i, (size, tile, la, lb) in list(enumerate(CASES))[::3]]
    for i, (size, tile) in enumerate(DIRECT):
        for la, lb in (("Row", "Col"), ("Col", "Row")):
            out.append(_kw(lego, size, tile, la, lb, ("f16", "bf16")[i % 2]))
    return out


N_COMPILED = len(CASES[::3]) + 2 * len(DIRECT)


@pytest.mark.parametrize("size", [(64, 128, 192), (256, 256, 256), (65, 63, 65), (600, 1000, 72)])
def test_reversed_c_keeps_the_wide_tiles(lego, size, tmp_path):
    """A reversed C puts the kernel in 64-bit indices: such plans keep the tiles
    of the larger sizes, and compile."""
    import os
    import subprocess
    from tests.test_isa_checks import HIPCC
    M, N, K = size
    src = lego.plan_source("gemm", M=M, N=N, K=K, dtype="f16", c=lego.as_layout(lego.GenP("reverse", [M, N])))
    assert "#define KWAVES 1\n" in src
    if not os.path.exists(HIPCC):
        pytest.skip("no ROCm compiler")
    (tmp_path / "k.hip").write_text(src)
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "--genco", "-Xclang", "-target-feature",
                        "-Xclang", "-packed-fp32-ops", "-include", "hip/hip_runtime.h", str(tmp_path / "k.hip"), "-o",
                        str(tmp_path / "k.co")], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]


# The default tile and the launch: (size, limit of workgroups, tile)
CHOICES = [((4096, 4096, 64), 0, "256x256x64"), ((6144, 6144, 512), 0, "256x256x64"), ((2816, 7424, 256), 0, "128x128x64"),
           ((2560, 2560, 2560), 0, "256x128x64"), ((8192, 8192, 8192), 0, "256x256x64"),
           # a limit makes the rounds of smaller tiles more
           ((1024, 4096, 64), 0, "128x128x64"), ((1024, 4096, 64), 64, "256x256x64"),
           ((2048, 2048, 2048), 0, "128x128x64"), ((2048, 2048, 2048), 64, "256x256x64"),
           ((512, 512, 512), 0, "32x32x64"), ((512, 512, 512), 256, "32x32x64")]


def test_default_tile_counts_the_rounds(lego):
    for (M, N, K), limit, tile in CHOICES:
        plan = lego.gemm_plan(M, N, K, "f16", max_workgroups=limit)
        assert f" tile {tile} " in plan, ((M, N, K), limit, plan)
