"""Host-side replay of planned launches (ks_plan_verify): every global access
of every thread stays in bounds, every LDS cell the MFMA reads was written,
and every element of Y is written exactly once (the row sets of the paper's
Section 4.1 partition the output, so no two workgroups may touch one element).
Runs on the CPU; nothing is enqueued."""
import pytest

import paper_2405_15013_amd as ks
from shapes import DMA_ROW_GROUP_SHAPES, DMA_SHAPES


def sweep_patterns():
    return [(a, b, c, d) for a in (1, 2, 4, 8) for b in (16, 32, 48, 64, 96, 128) for c in (16, 32, 48, 64, 96, 128)
            for d in (1, 2, 4, 8, 16) if a * b * d <= 8192 and a * c * d <= 8192]


CONFIGS = ([(2, 4, 4, 2)] + [(2 ** (l - 1), 2, 2, 2 ** (10 - l)) for l in range(1, 11)]
           + [(1, 32, 32, 32), (32, 32, 32, 1), (6, 64, 16, 8), (6, 16, 64, 8)])


@pytest.mark.parametrize("pattern", sweep_patterns()[::23])
@pytest.mark.parametrize("batch", [48, 1000, 4096])
@pytest.mark.parametrize("layout", ["bsf", "bsl"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_sweep_plans(pattern, batch, layout, dtype):
    st, rep = ks.ks_plan_verify(*pattern, batch, layout, dtype)
    assert st == 0, "%s B=%d %s %s: %s [%s]" % (pattern, batch, layout, dtype, rep,
                                                ks.ks_plan_describe(*pattern, batch, layout, dtype))


@pytest.mark.parametrize("pattern", CONFIGS)
@pytest.mark.parametrize("layout", ["bsf", "bsl"])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_config_plans_small_batch(pattern, layout, dtype):
    for batch in (1, 32, 104, 256):
        st, rep = ks.ks_plan_verify(*pattern, batch, layout, dtype)
        assert st == 0, "%s B=%d %s %s: %s" % (pattern, batch, layout, dtype, rep)


@pytest.mark.parametrize("pattern,batch", [((1, 32, 32, 32), 16384), ((6, 64, 16, 8), 25088),
                                           ((6, 16, 64, 8), 25088), ((1, 2, 2, 512), 4096)])
@pytest.mark.parametrize("layout", ["bsf", "bsl"])
def test_full_size_plans(pattern, batch, layout):
    st, rep = ks.ks_plan_verify(*pattern, batch, layout, "bf16")
    assert st == 0, rep


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("layout", ["bsf", "bsl"])
def test_all_sweep_plans_ragged_batch(dtype, layout):
    """Every sweep pattern, a batch that leaves a partial tile in both layouts."""
    bad = []
    for pattern in sweep_patterns():
        st, rep = ks.ks_plan_verify(*pattern, 72, layout, dtype)
        if st != 0:
            bad.append((pattern, rep))
    assert not bad, bad[:5]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("layout", ["bsf", "bsl"])
@pytest.mark.parametrize("batch,every", [(72, 1), (1000, 5)])
def test_all_sweep_plans_staged(dtype, layout, batch, every):
    """The LDS-staged kernel on every sweep pattern (forced): bounds, LDS cells
    written before they are read, every operand element the right X value,
    every output written once."""
    bad = []
    ks.ks_force_variant(4)
    try:
        for pattern in sweep_patterns()[::every]:
            st, rep = ks.ks_plan_verify(*pattern, batch, layout, dtype)
            if st != 0 and not (rep == "no plan" and layout == "bsl" and batch % (16 // (4 if dtype == "f32" else 2))):
                bad.append((pattern, rep))
    finally:
        ks.ks_force_variant(None)
    assert not bad, bad[:5]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("batch,every", [(72, 1), (1000, 7), (25088, 97)])
def test_all_sweep_plans_dma(dtype, batch, every):
    """The LDS-DMA kernel (forced) on every batch-size-first sweep pattern:
    every DMA lane fills one unit of the stage from an in-bounds address, every
    swizzled operand read holds the right X value, every output written once.
    It must accept every pattern of the sweep."""
    bad = []
    ks.ks_force_variant(6)
    try:
        for pattern in sweep_patterns()[::every]:
            st, rep = ks.ks_plan_verify(*pattern, batch, "bsf", dtype)
            if st != 0:
                bad.append((pattern, rep))
            else:
                assert "name=dma" in ks.ks_plan_describe(*pattern, batch, "bsf", dtype)
    finally:
        ks.ks_force_variant(None)
    assert not bad, bad[:5]


def test_sweep_plans_use_mfma_kernels():
    """The whole sweep runs on the MFMA kernels (aligned buffers): LDS-DMA for
    batch-size-first with d >= 4 or at least 8 MB of X and Y, and for
    batch-size-last in fp32, or in 16-bit types with b a power of two from 32
    and c of 32 or 64; register-direct otherwise."""
    for pattern in sweep_patterns()[::7]:
        for layout in ("bsf", "bsl"):
            for dtype in ("f32", "bf16", "f16"):
                desc = ks.ks_plan_describe(*pattern, 4096, layout, dtype)
                a, b, c, d = pattern
                big = 4096 * (a * c * d + a * b * d) * (4 if dtype == "f32" else 2) >= 8 << 20
                if layout == "bsf":
                    dma = d >= 4 or big
                else:
                    dma = dtype == "f32" or (b in (32, 64, 128) and c in (32, 64))
                want = "name=dma" if dma else "name=direct"
                assert want in desc, (pattern, layout, dtype, desc)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("batch,every", [(72, 3), (1000, 7), (25088, 97)])
def test_all_sweep_plans_dma_bsl(dtype, batch, every):
    """The batch-size-last LDS-DMA kernel (forced) on the batch-size-last sweep
    patterns it accepts (c a multiple of its stage: 16 for fp32, 32 for 16-bit
    types; the batch a multiple of the vector): DMA units in bounds and each
    written once per stage, every operand read the X value its products need,
    every output written once.  It must accept every such pattern."""
    bad = []
    ks.ks_force_variant(6)
    try:
        for pattern in sweep_patterns()[::every]:
            a, b, c, d = pattern
            if c % (16 if dtype == "f32" else 32) or batch % (4 if dtype == "f32" else 8):
                continue
            st, rep = ks.ks_plan_verify(*pattern, batch, "bsl", dtype)
            if st != 0:
                bad.append((pattern, rep))
            else:
                assert "kernel=ks_dma_bsl_kernel" in ks.ks_plan_describe(*pattern, batch, "bsl", dtype)
    finally:
        ks.ks_force_variant(None)
    assert not bad, bad[:5]


@pytest.mark.parametrize("variant", [0, 1, 2, 3, 4, 5, 6])
def test_forced_variants(variant):
    """Every variant that accepts a shape produces a valid launch for it."""
    ks.ks_force_variant(variant)
    try:
        for pattern, layout in [((2, 4, 4, 2), "bsl"), ((2, 4, 4, 2), "bsf"), ((1, 16, 16, 4), "bsf"),
                                ((1, 16, 16, 4), "bsl"), ((3, 32, 48, 2), "bsf")]:
            st, rep = ks.ks_plan_verify(*pattern, 64, layout, "f32")
            assert st in (0, 5), rep
            if st == 5:
                assert rep == "no plan", rep
    finally:
        ks.ks_force_variant(None)


def test_dma_row_group_plans_covered():
    """The GPU parity shapes of the DMA kernel reach every (MT, NT, stage
    length, strided) plan its planner makes on sweep-like patterns at batch
    4096, and each of those plans passes the replay."""
    def key(p, dt):
        f = dict(kv.split("=", 1) for kv in ks.ks_plan_describe(*p, 4096, "bsf", dt).split())
        return (dt, f["waves_m"], f["nt"], f["lch"], f["unroll"])
    have = {key(p, dt) for p in DMA_ROW_GROUP_SHAPES + DMA_SHAPES for dt in ("f32", "bf16")}
    want = {key(p, dt) for p in [(a, b, c, d) for a in (1, 2, 4, 8) for b in (16, 32, 64, 128) for c in (16, 32, 64)
                                  for d in (1, 2, 4, 8, 16) if a * b * d <= 8192 and a * c * d <= 8192]
            for dt in ("f32", "bf16")}
    assert want <= have, sorted(want - have)
    for p in DMA_ROW_GROUP_SHAPES:
        for dt in ("f32", "bf16"):
            for batch in (4096, 4000):
                st, rep = ks.ks_plan_verify(*p, batch, "bsf", dt)
                assert st == 0, (p, dt, batch, rep)


ODD = [(1, 24, 24, 8), (1, 17, 33, 3), (2, 48, 80, 2), (6, 64, 16, 8), (1, 64, 64, 1), (3, 20, 40, 1), (1, 100, 36, 2),
       (4, 16, 17, 2), (1, 33, 16, 5)]


@pytest.mark.parametrize("pattern", ODD)
@pytest.mark.parametrize("batch", [1, 37, 1001, 4096, 25087])
@pytest.mark.parametrize("layout", ["bsf", "bsl"])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_no_generic_plan_for_large_blocks(pattern, batch, layout, dtype):
    """Blocks with b or c above 16 always get an MFMA kernel (the masked one
    when b or c is not a multiple of 16 or the batch is not a multiple of the
    vector), whose host replay passes at every access width the planner may
    pick for less aligned buffers."""
    desc = ks.ks_plan_describe(*pattern, batch, layout, dtype)
    assert "name=generic" not in desc, desc
    if batch <= 4096:
        st, rep = ks.ks_plan_verify(*pattern, batch, layout, dtype)
        assert st == 0, (desc, rep)


@pytest.mark.parametrize("layout", ["bsf", "bsl"])
@pytest.mark.parametrize("batch", [4096, 1001])
def test_fp8_sweep_plans(layout, batch):
    """Host replay of the FP8 kernel's plan (access width up to 8 in both
    layouts) over every sweep pattern: coverage, padding, alignment."""
    for pattern in sweep_patterns()[::15] + [(6, 64, 16, 8), (6, 16, 64, 8), (1, 17, 33, 3), (4, 48, 32, 16),
                                           (1, 16, 8, 8), (3, 48, 40, 8), (2, 96, 24, 8), (1, 48, 64, 8)]:
        st, rep = ks.ks_plan_verify(*pattern, batch, layout, "fp8")
        assert st == 0, "%s B=%d %s: %s" % (pattern, batch, layout, rep)
        assert "name=fp8" in ks.ks_plan_describe(*pattern, batch, layout, "fp8")


def test_fp8_bsf_uses_full_rows_when_d_is_8():
    desc = ks.ks_plan_describe(6, 64, 16, 8, 25088, "bsf", "fp8")
    assert "vec=8" in desc, desc


@pytest.mark.parametrize("layout", ["bsf", "bsl"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("batch", [1, 7, 16, 33, 129])
def test_masked_plans_of_any_size(layout, dtype, batch):
    """Host replay of the masked kernels: b and c around multiples of the
    operand, chunk and tile, odd d, every vector width the batch leaves."""
    ks.ks_force_variant(7)
    try:
        for pattern in [(1, 1, 1, 1), (2, 3, 5, 7), (1, 16, 16, 3), (3, 17, 33, 1), (1, 130, 31, 5), (2, 63, 64, 2),
                        (1, 100, 129, 12)]:
            st, rep = ks.ks_plan_verify(*pattern, batch, layout, dtype)
            assert st == 0, (pattern, rep)
    finally:
        ks.ks_force_variant(None)


def test_long_rows_keep_the_register_kernel():
    """Batch-size-first rows that do not fit LDS: the register kernel."""
    desc = ks.ks_plan_describe(1, 33, 33, 4096, 8, "bsf", "f32")
    assert "name=masked" in desc and "kernel=ks_masked_kernel<float,0," in desc, desc
    assert "kernel=ks_masked_bsf_kernel<" in ks.ks_plan_describe(1, 33, 33, 16, 4096, "bsf", "f32")


def test_dma_forms_have_their_own_names():
    """Batch-size-first DMA: the name of the kernel with K operands in registers
    has seven arguments, the one with K operands in LDS is another kernel."""
    def kernel(*call):
        return dict(f.split("=", 1) for f in ks.ks_plan_describe(*call).split())["kernel"]
    assert kernel(2, 64, 64, 4, 4096, "bsf", "f32").startswith("ks_dma_kernel<float,4,false,")
    for call in ((6, 64, 16, 8, 25088, "bsf", "bf16"), (1, 128, 128, 16, 25088, "bsf", "f32")):
        name = kernel(*call)
        assert name.startswith("ks_dma_klds_kernel<" if call[2] == 128 else "ks_dma_kernel<"), name
        assert name.count(",") == 6


@pytest.mark.parametrize("dtype,inside,outside", [
    ("f32", [(1, 64, 64, 16), (1, 16, 96, 16), (1, 48, 128, 8), (2, 128, 96, 8), (1, 64, 160, 8), (1, 96, 128, 4)],
     [(1, 48, 112, 16), (2, 64, 96, 8), (2, 64, 128, 8), (1, 192, 128, 8), (1, 48, 144, 8), (1, 64, 128, 4),
      (1, 48, 144, 4)]),
    ("bf16", [(1, 64, 128, 16), (1, 64, 160, 16), (1, 64, 96, 8), (1, 48, 128, 8), (1, 48, 192, 4)],
     [(1, 32, 96, 16), (4, 128, 96, 16), (1, 48, 160, 16), (1, 48, 160, 8), (1, 48, 160, 4), (1, 64, 128, 4)])])
def test_k_through_lds_only_where_it_pays(dtype, inside, outside):
    """K operands move through LDS in the classes that measured faster, and stay
    in registers in those that measured the same or slower."""
    for pattern in inside + outside:
        desc = ks.ks_plan_describe(*pattern, 4096, "bsf", dtype)
        assert ("kernel=ks_dma_klds_kernel<" in desc) == (pattern in inside), desc


def test_fp8_long_rows_only_where_they_pay():
    """FP8 walks of one batch tile with 64 values of l and two row tiles measured
    slower than the general kernel, and keep it."""
    for pattern, batch, rows in [((8, 96, 64, 8), 4, False), ((4, 64, 64, 8), 197, False), ((4, 64, 56, 8), 197, True),
                                 ((4, 48, 64, 8), 197, True), ((4, 64, 64, 8), 25088, True)]:
        desc = ks.ks_plan_describe(*pattern, batch, "bsf", "fp8")
        assert ("kernel=ks_fp8_rows_kernel<" in desc) == rows, desc
        st, rep = ks.ks_plan_verify(*pattern, batch, "bsf", "fp8")
        assert st == 0, rep


@pytest.mark.parametrize("pattern,batch,layout", [
    ((17000000, 5, 1, 1), 1, "bsf"), ((15000000, 8, 16, 1), 4, "bsf"), ((17000000, 17, 1, 1), 1, "bsf"),
    ((33000000, 33, 1, 1), 1, "bsf"), ((70000000, 5, 1, 1), 1, "bsl"), ((70000000, 17, 1, 1), 1, "bsl"),
    ((1, 5, 5, 70000000), 2, "bsl"), ((1, 17, 1, 100000000), 1, "bsl"), ((1, 1, 33, 60000000), 1, "bsf")])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_plans_of_many_blocks_can_be_launched(pattern, batch, layout, dtype):
    """The runtime refuses 2^32 threads and more: a call of millions of blocks
    gets a kernel whose launch stays below that."""
    f = dict(x.split("=", 1) for x in ks.ks_plan_describe(*pattern, batch, layout, dtype).split())
    assert int(f["grid"]) * int(f["block"]) < 1 << 32, f


@pytest.mark.parametrize("pattern,batch,dtype,lds", [
    ((3, 29, 2, 228), 1, "bf16", False), ((2, 3, 34, 37), 104, "f32", False), ((1, 33, 33, 16), 8, "f32", False),
    ((21, 33, 4, 9), 6, "bf16", False), ((1, 115, 28, 37), 26, "f32", False), ((2, 40, 130, 1), 4, "f32", True),
    ((6, 30, 17, 21), 49, "bf16", False), ((7, 23, 31, 14), 41, "f32", False), ((2, 160, 3, 30), 51, "f16", False),
    ((1, 129, 12, 7), 64, "f16", False), ((16, 125, 77, 1), 100, "bf16", True),
    ((1, 33, 33, 16), 4096, "f32", True), ((6, 110, 80, 3), 5504, "bf16", True), ((4, 29, 89, 5), 3327, "bf16", True)])
def test_masked_rows_through_lds_where_there_are_enough(pattern, batch, dtype, lds):
    """Batch-size-first masked calls: rows through LDS only with the workgroups
    to hide the chain of products of each; both forms replayed."""
    desc = ks.ks_plan_describe(*pattern, batch, "bsf", dtype)
    assert ("kernel=ks_masked_bsf_kernel<" if lds else "kernel=ks_masked_kernel<") in desc, desc
    st, rep = ks.ks_plan_verify(*pattern, batch, "bsf", dtype)
    assert st == 0, rep


@pytest.mark.parametrize("pattern,batch,layout,dtype,valu", [
    ((2, 1, 15, 95), 2273, "bsf", "f32", True), ((4, 15, 1, 453), 429, "bsf", "f16", True),
    ((2, 5, 3, 139), 2261, "bsf", "f16", True), ((2, 5, 3, 128), 2261, "bsf", "f16", False),
    ((1, 4, 4, 256), 4096, "bsf", "f32", True), ((4, 4, 4, 512), 4096, "bsf", "f32", True),
    ((16, 4, 4, 16), 4096, "bsf", "f32", False), ((1, 8, 8, 128), 4096, "bsf", "f32", False),
    ((1, 8, 8, 256), 25088, "bsf", "bf16", False), ((2, 4, 4, 2), 32, "bsf", "f32", True),
    ((16, 5, 1, 32), 18240, "bsl", "bf16", True), ((16, 5, 1, 32), 18241, "bsl", "bf16", False),
    ((1, 5, 1, 32), 512, "bsl", "bf16", False), ((8, 4, 4, 16), 100, "bsl", "f32", True)])
def test_small_blocks_run_the_faster_kernel(pattern, batch, layout, dtype, valu):
    """b, c <= 16: the VALU kernels where their fetch of whole blocks is the
    cheaper one, the masked MFMA kernels elsewhere."""
    desc = ks.ks_plan_describe(*pattern, batch, layout, dtype)
    assert ("kernel=ks_valu_%s_kernel<" % layout in desc) == valu, desc
    assert valu or "name=masked" in desc, desc
    st, rep = ks.ks_plan_verify(*pattern, batch, layout, dtype)
    assert st == 0, rep


def test_masked_instances_replayed():
    """The calls at which the GPU suite runs each masked instance, those of up to
    half a million outputs: replayed on the host."""
    from test_gpu_parity import MASKED_RUNS
    ran = set()
    for (a, b, c, d), batch, layout, dtype, want in MASKED_RUNS:
        if dtype != "f16" and a * b * d * batch <= 5e5:
            st, rep = ks.ks_plan_verify(a, b, c, d, batch, layout, dtype)
            assert st == 0, rep
            ran.add((layout, want))
    assert {("bsl", "1,4"), ("bsl", "1,2"), ("bsl", "8,1"), ("bsf", "1,1"), ("bsf", "2,1"), ("bsf", "0,4")} <= ran


@pytest.mark.parametrize("pattern,batch,klds", [
    ((6, 128, 96, 8), 600, True), ((6, 128, 96, 8), 704, False), ((6, 128, 96, 8), 1500, False),
    ((6, 128, 96, 8), 4096, True), ((1, 256, 128, 8), 2571, False), ((1, 256, 128, 16), 2571, True)])
def test_k_through_lds_not_with_uneven_long_tiles(pattern, batch, klds):
    """fp32, d = 8: the long tiles of the form with K in LDS only where the CUs get
    about the same number of them."""
    desc = ks.ks_plan_describe(*pattern, batch, "bsf", "f32")
    assert ("kernel=ks_dma_klds_kernel<" in desc) == klds, desc
    st, rep = ks.ks_plan_verify(*pattern, batch, "bsf", "f32")
    assert st == 0, rep


@pytest.mark.parametrize("pattern,batch,dtype,vec", [
    ((1, 96, 16, 8), 65, "f16", 1), ((4, 32, 16, 1), 293, "f16", 1), ((6, 48, 16, 8), 515, "bf16", 8),
    ((4, 40, 24, 6), 10007, "f32", 4), ((2, 40, 24, 6), 515, "f32", 2), ((2, 40, 24, 6), 515, "bf16", 2)])
def test_masked_vectors_leave_wavefronts(pattern, batch, dtype, vec):
    """Batch-size-last masked calls: vectors of the batch no wider than leaves 512
    wavefronts."""
    f = dict(x.split("=", 1) for x in ks.ks_plan_describe(*pattern, batch, "bsl", dtype).split())
    assert f["name"] == "masked" and int(f["vec"]) == vec, f
    st, rep = ks.ks_plan_verify(*pattern, batch, "bsl", dtype)
    assert st == 0, rep
