"""Parity of the HIP path against the CPU oracle, element by element, through the C ABI.

Bar: bit-exact for the integer (Life) kernel; max relative error <= 1e-5 per application and
<= 1e-4 after iterated runs for fp32.  The heat kernel is specified as a fixed sequence of
fp32 operations, so for it the GPU is additionally required to match the fp32 oracle exactly.
"""
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import stencil as oracle
from paper_1511_02490_amd import workloads as wl

pytestmark = pytest.mark.gpu

REL_1 = 1e-5       # one application
REL_N = 1e-4       # after iterated runs


@pytest.fixture(scope="module")
def ls():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1511_02490_amd import libstencil
    return libstencil


def rel_err(got, ref):
    got = got.astype(np.float64)
    ref = ref.astype(np.float64)
    return float(np.max(np.abs(got - ref) / np.maximum(np.abs(ref), 1e-6)))


def set_mapping(st, blocking):
    """blocking = (cells_rows, cells_cols) under local-memory staging, ("direct", cr, cc), or
    ("temporal", cr, cc, depth)."""
    if len(blocking) == 4:
        st.set_mapping(*blocking[:3])
        st.set_option(1, blocking[3])          # STENCIL_OPT_TEMPORAL_DEPTH
    elif len(blocking) == 3:
        st.set_mapping(*blocking)
    else:
        st.set_mapping("local", *blocking)


def gpu_apply(ls, w, grid, wg, iters=None, blocking=(1, 1), offset=0):
    """Run workload `w` on `grid` through the library.  offset > 0 places the matrices that many
    elements into their allocations, so that rows are not 16-byte aligned."""
    st = ls.Stencil.from_workload(w)
    set_mapping(st, blocking)
    n = grid.size
    types = {"f32": torch.float32, "u8": torch.uint8, "i32": torch.int32, "f64": torch.float64}
    tdt = types[w.dtype]
    buf_in = torch.zeros(n + offset, dtype=tdt, device="cuda")
    buf_out = torch.full((n + offset,), 7, dtype=types[getattr(w, "out_dtype", w.dtype)], device="cuda")
    tin, tout = buf_in[offset:], buf_out[offset:]
    tin.copy_(torch.from_numpy(grid.reshape(-1)))
    st.run(tin, tout, w.iters if iters is None else iters, wg)
    torch.cuda.synchronize()
    assert np.array_equal(tin.cpu().numpy().reshape(grid.shape), grid, equal_nan=grid.dtype.kind == "f"), "input was modified"
    out = tout.cpu().numpy().reshape(grid.shape)
    st.close()
    return out


def check(ls, w, wg, iters=None, blocking=(1, 1), offset=0, grid=None):
    g = w.grid() if grid is None else grid
    it = w.iters if iters is None else iters
    ref = oracle.apply(g, w.kernel, w.halo, w.border, w.pad, w.weights, w.scalars, it)
    got = gpu_apply(ls, w, g, wg, it, blocking, offset)
    if w.dtype == "i32" or w.kernel in (wl.LIFE, wl.SOBEL, wl.NMS, wl.THRESHOLD):
        np.testing.assert_array_equal(got, ref)        # integer work, or fp32 operations in a fixed order
    elif w.dtype == "f64":
        assert rel_err(got, ref) <= 1e-13 * max(1, it)
    else:
        tol = REL_1 if it <= 1 else REL_N
        err = rel_err(got, ref)
        assert err <= tol, "rel err %.3g > %.1g (wg %s blocking %s)" % (err, tol, wg, blocking)
        if w.kernel == wl.HEAT:
            np.testing.assert_array_equal(got, ref)
    return got


def custom(kernel, rows, cols, halo, border, pad=0.0, seed=1, iters=1):
    """A workload of the synthetic family: any border region, any border mode."""
    n, s, e, w_ = halo
    rng = np.random.default_rng(seed)
    weights = None
    dtype = "f32"
    scalars = ()
    if kernel in (wl.WEIGHTED_SUM, wl.SINCOS):
        weights = rng.random((n + s + 1, e + w_ + 1), dtype=np.float32)
        if kernel == wl.WEIGHTED_SUM:
            weights /= weights.sum()
    if kernel == wl.HEAT:
        scalars = (0.2,)
    if kernel == wl.LIFE:
        dtype = "u8"
    return wl.Workload("custom", rows, cols, dtype, halo, border, pad, kernel, iters, seed, "pow2",
                       weights=weights, scalars=scalars)


# ---- C1: the small configuration, whole matrix, every listed size ----------------------------

def test_c1_all_listed_sizes(ls):
    w = wl.config(0)
    for wg in w.wg_sizes():
        check(ls, w, wg)
    for blocking in ((4, 4), (2, 1), (1, 4)):
        check(ls, w, (8, 8), blocking=blocking)


# ---- every kernel x border mode x blocking, ragged matrices spanning several tiles -----------

BLOCKINGS_F32 = [(1, 1), (2, 1), (8, 1), (1, 4), (4, 4), (8, 4)]
DIRECT_F32 = [("direct", 1, 4), ("direct", 2, 4), ("direct", 4, 4)]
DIRECT_U8 = [("direct", 1, 16), ("direct", 2, 16), ("direct", 4, 16), ("direct", 8, 16)]


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
@pytest.mark.parametrize("halo", [(1, 1, 1, 1), (2, 2, 2, 2), (3, 3, 3, 3), (4, 4, 4, 4), (2, 1, 2, 2), (0, 0, 0, 0), (7, 3, 9, 5)])
def test_weighted_sum_borders_and_regions(ls, border, halo):
    w = custom(wl.WEIGHTED_SUM, 131, 157, halo, border, pad=0.5, seed=sum(halo))
    direct = DIRECT_F32 if halo in [(1, 1, 1, 1), (2, 2, 2, 2), (3, 3, 3, 3), (4, 4, 4, 4)] else []
    for blocking in BLOCKINGS_F32 + direct:
        for wg in [(4, 4), (16, 16), (3, 21), (2, 64)]:
            check(ls, w, wg, blocking=blocking)
    # aligned rows (vector path), misaligned base pointer, and cols % 4 != 0
    w2 = custom(wl.WEIGHTED_SUM, 96, 128, halo, border, pad=0.5, seed=3)
    for off in (0, 1):
        for blocking in [(4, 4)] + direct[:2]:
            check(ls, w2, (8, 16), blocking=blocking, offset=off)
    if not direct:
        st = ls.Stencil.from_workload(w)
        with pytest.raises(ls.StencilError):
            st.set_mapping("direct", 1, 4)                  # no direct variant for this region


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
def test_sincos_borders(ls, border):
    for halo in [(1, 5, 3, 0), (2, 0, 1, 3)]:
        w = custom(wl.SINCOS, 93, 140, halo, border, pad=0.3, seed=5)
        for blocking in [(1, 1), (4, 1), (2, 4), (8, 4)]:
            for wg in [(4, 4), (8, 16), (6, 10)]:
                check(ls, w, wg, blocking=blocking)


def test_border_regions_at_the_papers_maximum(ls):
    """The synthetic template's largest border regions (30 cells, Section 5) in every direction, for
    both synthetic functions, under the paper's mapping and a blocked one; some sizes are then
    refused because the tile no longer fits local memory."""
    for halo in [(30, 1, 1, 30), (1, 30, 30, 1), (30, 30, 30, 30), (32, 32, 32, 32)]:
        for kernel, border in ((wl.WEIGHTED_SUM, "clamp"), (wl.SINCOS, "wrap")):
            w = custom(kernel, 150, 170, halo, border, pad=0.3, seed=sum(halo))
            check(ls, w, (8, 8), blocking=(1, 1))
            check(ls, w, (4, 16), blocking=(2, 4))
    w = custom(wl.SINCOS, 150, 170, (30, 30, 30, 30), "constant", pad=0.3, seed=1)
    st = ls.Stencil.from_workload(w)
    assert st.is_legal(32, 32) and st.tile_bytes(32, 32) == 92 * 92 * 8
    st.set_blocking(8, 4)
    assert not st.is_legal(16, 16)            # (128 + 60) x (64 + 64) x 8 bytes: beyond 160 KiB
    tin = torch.zeros(150 * 170, device="cuda")
    with pytest.raises(ls.Refused):
        st.run(tin, torch.empty_like(tin), 1, (16, 16))
    st.close()


def test_region_alignments_of_the_vector_walk(ls):
    """Run-time regions are walked four window columns at a time from the staged tile's aligned
    west edge: every residue of the west and east extents, against the oracle, and bit for bit
    against the one-cell-per-work-item mapping, which walks tap by tap."""
    for kernel in (wl.WEIGHTED_SUM, wl.SINCOS):
        for west in range(0, 6):
            for east in (0, 1, 2, 3, 4, 7):
                w = custom(kernel, 37, 83, (1, 2, east, west), "wrap", pad=0.3, seed=10 * west + east)
                one = check(ls, w, (4, 16), blocking=(1, 1))
                for blocking in [(1, 4), (2, 4)]:
                    np.testing.assert_array_equal(check(ls, w, (4, 16), blocking=blocking), one)
    for west, east in [(0, 0), (1, 3), (2, 1), (3, 2)]:
        n, s = 2, 1
        wf = np.random.default_rng(west).random((n + s + 1, east + west + 1), dtype=np.float32)
        wd = wl.Workload("f64", 41, 66, "f64", (n, s, east, west), "clamp", 0.5, wl.WEIGHTED_SUM, 1, 5, "pow2", weights=wf)
        np.testing.assert_array_equal(check(ls, wd, (4, 16), blocking=(2, 2)), check(ls, wd, (4, 16), blocking=(1, 1)))


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
def test_life_bit_exact(ls, border):
    for rows, cols in [(150, 203), (64, 256)]:
        w = wl.config(2, rows=rows, cols=cols, iters=12)
        w.border = border
        for blocking in [(1, 1), (4, 1), (1, 16), (2, 16)] + DIRECT_U8:
            for wg in [(4, 4), (16, 16), (2, 64), (5, 7)]:
                check(ls, w, wg, blocking=blocking)
    for shape in [(97, 61), (80, 96)]:
        w1 = wl.config(2, rows=shape[0], cols=shape[1], iters=2)
        w1.border, w1.pad = "constant", 1.0              # live padding
        check(ls, w1, (8, 8))
        check(ls, w1, (8, 8), blocking=("direct", 2, 16))
        check(ls, w1, (8, 8), blocking=("direct", 1, 16), offset=3)


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
def test_heat_matches_fp32_oracle_exactly(ls, border):
    w = wl.config(3, rows=160, cols=216, iters=25)
    w.border, w.pad = border, 50.0
    for blocking in [(1, 1), (4, 1), (1, 4), (8, 4)] + DIRECT_F32:
        for wg in [(4, 4), (16, 16), (4, 64), (7, 9)]:
            check(ls, w, wg, blocking=blocking)
    w2 = wl.config(3, rows=61, cols=83, iters=5)          # cols % 4 != 0: element-wise path
    w2.border, w2.pad = border, 50.0
    check(ls, w2, (4, 16), blocking=("direct", 2, 4))


def test_heat_conserves_total_and_long_run(ls):
    w = wl.config(3, rows=256, cols=256, iters=1000)
    g = w.grid()
    got = check(ls, w, (4, 64), blocking=(4, 4), grid=g)
    got2 = check(ls, w, (4, 64), blocking=("direct", 1, 4), grid=g)
    np.testing.assert_array_equal(got, got2)
    s0, s1 = g.astype(np.float64).sum(), got.astype(np.float64).sum()
    assert abs(s1 - s0) / s0 < 1e-6
    assert got.min() >= g.min() and got.max() <= g.max()


@pytest.mark.parametrize("cols", [160, 161, 162, 163, 175])
@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
def test_vectors_at_any_address(ls, border, cols):
    """Rows of every length modulo a vector, matrices that start at any element: tiles inside the matrix (staged
    without border resolution) and at its edges (the last vector of a row is partial)."""
    rng = np.random.default_rng(cols)
    for offset in (0, 1, 3):
        for halo in [(2, 2, 2, 2), (3, 1, 0, 4)]:
            w = custom(wl.WEIGHTED_SUM, 70, cols, halo, border, pad=0.5, seed=cols)
            for blocking, wg in [((2, 4), (4, 8)), ((1, 4), (8, 16)), ((4, 4), (2, 5))]:
                check(ls, w, wg, blocking=blocking, offset=offset)
            wf = rng.random((halo[0] + halo[1] + 1, halo[2] + halo[3] + 1), dtype=np.float32)
            wd = wl.Workload("f64", 70, cols, "f64", halo, border, 0.5, wl.WEIGHTED_SUM, 1, 5, "pow2", weights=wf)
            check(ls, wd, (4, 8), blocking=(2, 2), offset=offset)
            wi = wl.Workload("i32", 70, cols, "i32", halo, border, 3.0, wl.WEIGHTED_SUM, 1, 6, "pow2",
                             weights=np.rint(wf * 9).astype(np.float32))
            check(ls, wi, (4, 8), blocking=(2, 4), offset=offset)
            wu = wl.Workload("u8", 70, cols, "u8", halo, border, 9.0, wl.WEIGHTED_SUM, 1, 7, "pow2", weights=wf)
            check(ls, wu, (4, 8), blocking=(2, 4), offset=offset)
        life = wl.config(2, rows=70, cols=cols, iters=5)
        life.border = border
        heat = wl.config(3, rows=70, cols=cols, iters=5)
        heat.border, heat.pad = border, 50.0
        for w, cc in ((life, 16), (heat, 4)):
            check(ls, w, (4, 2), blocking=(2, cc), offset=offset)
            check(ls, w, (4, 2), blocking=("direct", 2, cc), offset=offset)
            check(ls, w, (4, 2), blocking=("temporal", 2, cc, 3), offset=offset)


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
@pytest.mark.parametrize("halo", [(2, 3, 0, 0), (0, 0, 0, 0), (1, 0, 0, 0)])
def test_staged_rows_of_a_single_item(ls, border, halo):
    """Workgroups one work-item wide under regions of one column: a staged row is one vector (or one cell), in tiles
    at the matrix's edge and inside it."""
    for cols in (1, 3, 24, 29):
        w = custom(wl.WEIGHTED_SUM, 157, cols, halo, border, pad=0.5, seed=cols)
        wd = wl.Workload("f64", 157, cols, "f64", halo, border, 0.5, wl.WEIGHTED_SUM, 1, 5, "pow2", weights=w.weights)
        wi = wl.Workload("i32", 157, cols, "i32", halo, border, 3.0, wl.WEIGHTED_SUM, 1, 6, "pow2",
                         weights=np.rint(w.weights * 99).astype(np.float32))
        for wg in [(1, 1), (3, 1), (8, 1), (64, 1)]:
            for blocking in [(1, 1), (8, 1), (1, 4), (2, 4), (8, 4)]:
                check(ls, w, wg, blocking=blocking)
            check(ls, wd, wg, blocking=(2, 2))
            check(ls, wi, wg, blocking=(2, 4))
        ws = custom(wl.SINCOS, 157, cols, halo, border, pad=0.5, seed=cols)
        one = gpu_apply(ls, ws, ws.grid(), (4, 4), blocking=(1, 1))
        np.testing.assert_array_equal(gpu_apply(ls, ws, ws.grid(), (8, 1), blocking=(2, 4)), one)


# ---- the other element types of the paper's template (Section 3.3) ---------------------------

@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
def test_weighted_sum_on_double_and_int32_matrices(ls, border):
    rng = np.random.default_rng(41)
    for halo in [(1, 1, 1, 1), (2, 2, 2, 2), (2, 1, 2, 2), (0, 3, 4, 1)]:
        n, s, e, w_ = halo
        compiled = halo in [(1, 1, 1, 1), (2, 2, 2, 2)]          # regions with variants of their own, direct ones too
        wf = rng.random((n + s + 1, e + w_ + 1), dtype=np.float32)
        wd = wl.Workload("f64", 77, 90, "f64", halo, border, 0.5, wl.WEIGHTED_SUM, 2, 5, "pow2", weights=wf)
        for blocking, wg in [((1, 1), (4, 16)), ((2, 2), (8, 32)), ((2, 2), (3, 5)), ((1, 2), (4, 16)), ((4, 2), (8, 8))] + (
                [(("direct", cr, 2), wg) for cr in (1, 2, 4) for wg in ((4, 16), (3, 5))] if compiled else []):
            check(ls, wd, wg, blocking=blocking)
        check(ls, wd, (4, 8), blocking=(2, 2), offset=1)
        wi = rng.integers(-5, 6, size=wf.shape).astype(np.float32)
        wi32 = wl.Workload("i32", 77, 90, "i32", halo, border, 3.0, wl.WEIGHTED_SUM, 3, 6, "pow2", weights=wi)
        for blocking, wg in [((1, 1), (4, 16)), ((2, 4), (8, 32)), ((2, 4), (3, 5)), ((1, 4), (4, 16)), ((4, 4), (8, 8))] + (
                [(("direct", cr, 4), wg) for cr in (1, 2, 4) for wg in ((4, 16), (3, 5))] if compiled else []):
            check(ls, wi32, wg, blocking=blocking)
        if compiled:
            check(ls, wd, (4, 8), blocking=("direct", 2, 2), offset=1)
            check(ls, wi32, (4, 8), blocking=("direct", 2, 4), offset=1)
    # wrap-around arithmetic
    big = np.full((40, 48), (1 << 20) + 1, np.int32)
    wb = wl.Workload("i32", 40, 48, "i32", (1, 1, 1, 1), border, 0.0, wl.WEIGHTED_SUM, 1, 7, "pow2",
                     weights=np.full((3, 3), float((1 << 20) + 1), np.float32))
    check(ls, wb, (4, 16), blocking=(2, 4), grid=big)
    st = ls.Stencil(8, 8, "i32")
    with pytest.raises(ls.StencilError):
        st.set_kernel("weighted_sum", np.full((3, 3), 0.5, np.float32))        # integer weights only
    with pytest.raises(ls.StencilError):
        ls.Stencil(8, 8, "f64").set_kernel("sincos", np.zeros((3, 3), np.float32))


# ---- the Canny detector's stencils (Table 2) ---------------------------------------------------

@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
def test_sobel_and_nms_bit_exact(ls, border):
    for kernel in (wl.SOBEL, wl.NMS):
        for rows, cols in [(131, 157), (96, 128), (1, 1), (3, 50)]:
            w = wl.canny_stage(kernel, rows, cols, border)
            w.pad = 0.7
            g = w.grid() * np.float32(50.0)
            for blocking in BLOCKINGS_F32 + DIRECT_F32:
                for wg in [(4, 4), (16, 16), (3, 21), (2, 64)]:
                    check(ls, w, wg, blocking=blocking, grid=g)
        w = wl.canny_stage(kernel, 64, 96, border)
        check(ls, w, (8, 16), blocking=(4, 4), offset=1)                  # unaligned rows
        check(ls, w, (8, 16), blocking=("direct", 2, 4), offset=3)
        check(ls, w, (8, 16), blocking=("direct", 2, 4), iters=3)         # iterated: ping-pong
        with pytest.raises(ls.StencilError):
            ls.Stencil.from_workload(w).set_mapping("stream", 16, 4)
    with pytest.raises(ls.StencilError):
        ls.Stencil(8, 8, "f32", (1, 1, 1, 0), border).set_kernel("sobel")   # region must be 1/1/1/1
    with pytest.raises(ls.StencilError):
        ls.Stencil(8, 8, "u8", (1, 1, 1, 1), border).set_kernel("nms")


def test_threshold_float_in_bytes_out(ls):
    for rows, cols in [(131, 157), (96, 128), (1, 1), (5, 1030)]:
        w = wl.canny_stage(wl.THRESHOLD, rows, cols, level=0.37)
        g = w.grid()
        g[0, 0] = np.nan
        g[rows // 2, cols // 2] = np.float32(0.37)                           # exactly the level: reached
        for blocking in [(1, 1), (2, 1), (1, 4), (2, 4), (4, 4)]:
            for wg in [(4, 4), (16, 16), (3, 21), (2, 64), (1, 1024)]:
                got = check(ls, w, wg, blocking=blocking, grid=g)
                assert got.dtype == np.uint8 and got[rows // 2, cols // 2] == 1 and (got[0, 0] == 0 or rows == 1)
        check(ls, w, (8, 16), blocking=(2, 4), offset=1, grid=g)             # unaligned rows
    st = ls.Stencil.from_workload(wl.canny_stage(wl.THRESHOLD, 32, 32))
    assert st.output_dtype() == ls.U8 and st.tile_bytes(8, 8) == 0 and st.features()[12] == 1.0 and st.features()[2] == 4.0
    a = torch.zeros(32 * 32, device="cuda")
    with pytest.raises(ValueError):
        st.run(a, torch.zeros(32 * 32, device="cuda"), 1, (8, 8))            # the output is a byte matrix
    out = torch.zeros(32 * 32, dtype=torch.uint8, device="cuda")
    with pytest.raises(ls.StencilError):
        st.run(a, out, 2, (8, 8))                                            # another type out than in: one application
    with pytest.raises(ls.StencilError):
        st.set_mapping("direct", 1, 4)
    with pytest.raises(ls.StencilError):
        ls.Stencil(8, 8, "f32", (1, 1, 1, 1), "clamp").set_kernel("threshold", scalars=(0.5,))   # has no border region
    res = st.sweep(a, out, [(8, 8), (4, 64), (64, 32)], iters=1, reps=3)
    assert res.status == [ls.OK, ls.OK, ls.E_REFUSED] and res.best in [(8, 8), (4, 64)]
    st.close()


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
def test_weighted_sum_of_a_byte_image_into_floats(ls, border):
    """Bytes in, floats out (Section 3.3: input and output types differ): every blocking the kernel
    has, regions of several alignments, ragged and aligned matrices, misaligned rows, a byte padding
    value; bit-identical across blockings."""
    for halo, shape in [((1, 1, 1, 1), (131, 157)), ((2, 2, 2, 2), (96, 128)), ((3, 0, 5, 2), (77, 200)), ((0, 0, 0, 0), (40, 64))]:
        n, s, e, w_ = halo
        wt = np.random.default_rng(sum(halo)).random((n + s + 1, e + w_ + 1), dtype=np.float32)
        w = wl.Workload("u8 image", shape[0], shape[1], "u8", halo, border, 200.0, wl.WEIGHTED_SUM, 1, 17, "pow2", weights=wt)
        assert w.out_dtype == "f32"
        first = None
        for blocking, wg in [((1, 1), (8, 8)), ((1, 1), (3, 21)), ((4, 1), (4, 16)), ((1, 4), (4, 16)), ((2, 4), (16, 16)),
                             ((4, 4), (3, 7)), ((1, 16), (4, 4)), ((1, 16), (16, 8)), ((2, 16), (2, 8)), ((2, 16), (5, 3))]:
            got = check(ls, w, wg, blocking=blocking)
            assert got.dtype == np.float32
            first = got if first is None else first
            np.testing.assert_array_equal(got, first)
        check(ls, w, (4, 8), blocking=(1, 16), offset=3)
        check(ls, w, (4, 8), blocking=(2, 4), offset=3)
        check(ls, w, (4, 8), blocking=(2, 4), offset=4)               # byte rows 4-aligned, float rows 16-aligned
    st = ls.Stencil(64, 64, "u8", (1, 1, 1, 1), border)
    st.set_kernel("weighted_sum", np.ones((3, 3), np.float32))
    assert st.output_dtype() == ls.F32 and st.features()[2] == 1.0 and st.features()[12] == 4.0
    tin = torch.zeros(64 * 64, dtype=torch.uint8, device="cuda")
    tout = torch.zeros(64 * 64, dtype=torch.float32, device="cuda")
    with pytest.raises(ls.StencilError):
        st.run(tin, tout, 2, (8, 8))                                   # one application only
    with pytest.raises(ValueError):
        st.run(tin, tin.clone(), 1, (8, 8))                            # the output must be float
    with pytest.raises(ls.StencilError):
        st.set_mapping("direct", 1, 16)                                # local-memory tile only
    with pytest.raises(ls.StencilError):
        st.set_border_value(256)
    st.close()


def test_canny_chain_stage_by_stage(ls):
    """Gaussian blur -> sobel -> nms -> threshold, the detector the paper takes three of its kernels
    from: every stage is checked against the oracle on the input the previous stage produced."""
    rows, cols = 300, 420
    blur = wl.config(1, rows=rows, cols=cols)
    g = blur.grid()
    yy, xx = np.mgrid[0:rows, 0:cols]
    g = (g * np.float32(0.2) + ((xx // 60 + yy // 50) % 2).astype(np.float32)).astype(np.float32)   # a noisy chequerboard
    x = check(ls, blur, (16, 8), blocking=(2, 4), grid=g)
    # the same chain from an 8-bit image: the blur takes bytes and hands floats to the sobel stage
    g8 = np.clip(np.rint(g * 200.0), 0, 255).astype(np.uint8)
    x8 = check(ls, wl.image_blur(rows, cols), (8, 8), blocking=(1, 16), grid=g8)
    assert x8.dtype == np.float32 and abs(float(x8.mean()) - 200.0 * float(x.mean())) < 1.0
    for stage in (wl.canny_stage(wl.SOBEL, rows, cols), wl.canny_stage(wl.NMS, rows, cols),
                  wl.canny_stage(wl.THRESHOLD, rows, cols, level=1.0)):
        x = check(ls, stage, (4, 16), blocking=("direct", 2, 4) if stage.kernel != wl.THRESHOLD else (2, 4), grid=x)
    assert x.dtype == np.uint8 and 0.005 < x.mean() < 0.3                      # edges are thin lines
    # an edge runs along column 60: cells next to it are marked, cells well inside a square are not
    assert x[25, 58:62].max() == 1 and x[25, 20:40].max() == 0


@pytest.mark.parametrize("wcols", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 13, 17])
def test_run_time_regions_by_number_of_columns(ls, wcols):
    """The fold compiled for its number of columns and the one in chunks, under every blocking of the tile: regions all
    east, all west and between, of one row and of several, and an infinite cell that only its neighbours may see."""
    kernels = [wl.WEIGHTED_SUM, wl.SINCOS]
    for k, (n, s, west) in enumerate([(0, 0, 0), (2, 3, wcols - 1), (3, 1, wcols // 2)]):
        halo = (n, s, wcols - 1 - west, west)
        for kernel in kernels:
            w = custom(kernel, 37, 61, halo, ("clamp", "wrap", "constant")[k], pad=0.3, seed=wcols + k)
            g = w.grid()
            one = gpu_apply(ls, w, g, (4, 8), blocking=(1, 1))
            # absolute error (a sum of sines and cosines passes near zero): each sine and cosine is within 2e-7, and
            # each of 2 taps additions rounds a partial sum of at most 2 taps
            taps = w.weights.size
            ref = oracle.apply(g, w.kernel, w.halo, w.border, w.pad, w.weights, w.scalars, 1)
            assert np.max(np.abs(one.astype(np.float64) - ref)) <= 4e-7 * taps + 2 * taps * 2.0 ** -24 * 2 * taps
            for cr, wg in [(1, (4, 8)), (2, (8, 4)), (4, (3, 5)), (8, (2, 16))]:
                np.testing.assert_array_equal(gpu_apply(ls, w, g, wg, blocking=(cr, 4), offset=cr % 2), one)
        w = custom(wl.WEIGHTED_SUM, 37, 61, halo, "clamp", seed=wcols)
        g = w.grid()
        g[11, 23] = np.inf
        ref = oracle.apply(g, w.kernel, w.halo, w.border, w.pad, w.weights, w.scalars, 1)
        for cr in (2, 8):
            np.testing.assert_array_equal(np.isinf(gpu_apply(ls, w, g, (4, 8), blocking=(cr, 4))), np.isinf(ref))


@pytest.mark.parametrize("shape", [(1, 1), (1, 9), (9, 1), (3, 3), (2, 5), (6, 3), (3, 6), (4, 5), (3, 9), (4, 7), (1, 10), (2, 10)])
def test_run_time_regions_at_the_line_between_two_folds(ls, shape):
    """Regions of as many taps as go tap by tap under four and eight rows of cells (9, 18, 27), of one more, and single rows
    beyond the compiled widths, for every element type: bit for bit the one-cell mapping's sums."""
    rows, cols = shape
    for k, border in enumerate(("clamp", "wrap", "constant")):
        halo = (rows // 2, rows - 1 - rows // 2, cols - 1 - (cols * k) // 3, (cols * k) // 3)
        wf = custom(wl.WEIGHTED_SUM, 75, 141, halo, border, pad=0.5, seed=rows * cols + k)
        others = {dtype: wl.Workload(dtype, 75, 141, dtype, halo, border, 2.0, wl.WEIGHTED_SUM, 1, 3, "pow2",
                                     weights=np.rint(wf.weights * 99).astype(np.float32)) for dtype in ("f64", "i32", "u8")}
        for w, blockings in [(wf, [(2, 4), (4, 4), (8, 4)]), (others["f64"], [(2, 2), (4, 2)]), (others["i32"], [(2, 4), (4, 4)]),
                             (others["u8"], [(2, 4), (4, 4)])]:
            g = w.grid()
            one = check(ls, w, (4, 8), grid=g)
            for blocking in blockings:
                for wg in [(2, 8), (8, 16)]:
                    np.testing.assert_array_equal(gpu_apply(ls, w, g, wg, blocking=blocking), one)


# ---- temporal blocking: several applications per launch ------------------------------------

@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
def test_temporal_blocking_heat_bit_exact(ls, border):
    for rows, cols, iters in [(160, 216, 13), (61, 83, 7), (128, 256, 8)]:
        w = wl.config(3, rows=rows, cols=cols, iters=iters)
        w.border, w.pad = border, 50.0
        for depth in (1, 2, 3, 4):
            for cr, wg in [(1, (4, 16)), (2, (4, 64)), (4, (2, 8)), (8, (3, 5)), (4, (16, 16))]:
                check(ls, w, wg, blocking=("temporal", cr, 4, depth))


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
def test_temporal_blocking_weighted_sum_and_tiny(ls, border):
    w = custom(wl.WEIGHTED_SUM, 90, 117, (1, 1, 1, 1), border, pad=0.4, seed=21, iters=9)
    for depth in (2, 4):
        check(ls, w, (4, 16), blocking=("temporal", 2, 4, depth))
        check(ls, w, (8, 8), blocking=("temporal", 4, 4, depth), offset=1)
    for shape in [(1, 1), (1, 9), (7, 1), (3, 4), (5, 6)]:      # smaller than the staged rim
        wt = wl.config(3, rows=shape[0], cols=shape[1], iters=6)
        wt.border, wt.pad = border, 20.0
        check(ls, wt, (2, 4), blocking=("temporal", 2, 4, 4))
        check(ls, wt, (2, 4), blocking=("temporal", 1, 4, 3))


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
def test_temporal_blocking_life_bit_exact(ls, border):
    for rows, cols, iters in [(150, 203, 13), (64, 256, 8), (97, 61, 7)]:
        w = wl.config(2, rows=rows, cols=cols, iters=iters)
        w.border = border
        for depth in (1, 2, 3, 4):
            for cr, wg in [(1, (4, 16)), (2, (4, 64)), (4, (2, 8)), (8, (3, 5))]:
                check(ls, w, wg, blocking=("temporal", cr, 16, depth))
    w1 = wl.config(2, rows=80, cols=96, iters=6)
    w1.border, w1.pad = "constant", 1.0                            # live padding
    check(ls, w1, (4, 4), blocking=("temporal", 2, 16, 4))
    check(ls, w1, (4, 4), blocking=("temporal", 2, 16, 3), offset=5)
    for shape in [(1, 1), (1, 9), (7, 1), (3, 4), (5, 40)]:
        wt = wl.config(2, rows=shape[0], cols=shape[1], iters=6)
        wt.border = border
        check(ls, wt, (2, 4), blocking=("temporal", 2, 16, 4))


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
@pytest.mark.parametrize("cols", [2, 15, 16, 17, 31, 33, 47, 49, 129])
def test_life_on_bits_at_word_and_tile_edges(ls, border, cols):
    """Rows that end anywhere in a word or a 16-cell vector, tiles of an odd number of vectors, workgroups of fewer
    work-items than a row has words, and a last tile of a single row."""
    for rows, wg, cr in [(1, (1, 1), 1), (33, (16, 2), 2), (65, (8, 3), 8)]:
        w = custom(wl.LIFE, rows, cols, (1, 1, 1, 1), border, pad=1.0, seed=rows + cols, iters=7)
        check(ls, w, wg, blocking=("temporal", cr, 16, 4), offset=cols % 3)


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
@pytest.mark.parametrize("wg", [(1, 1), (1, 64), (2, 64), (1, 256), (5, 13), (16, 64)])
def test_temporal_items_of_whole_and_ragged_workgroups(ls, border, wg):
    """Overlapping wavefronts, more than one pass over a row of vectors, and workgroups that are no whole wavefronts."""
    for rows, cols in [(wg[0] * 2 + 1, wg[1] * 4 - 1), (67, 2 * wg[1] * 4 + 2)]:
        w = custom(wl.WEIGHTED_SUM, rows, cols, (1, 1, 1, 1), border, pad=0.25, seed=7, iters=5)
        check(ls, w, wg, blocking=("temporal", 2, 4, 4))
        h = wl.config(3, rows=rows, cols=cols, iters=5)
        h.border, h.pad = border, 30.0
        check(ls, h, wg, blocking=("temporal", 2, 4, 4))


@pytest.mark.parametrize("border", ["wrap", "constant"])
def test_register_streaming_temporal_kernel_bit_exact(ls, border):
    """Runs under the streaming mapping, made by the march (time levels kept in registers, row neighbours from adjacent
    lanes; every wavefront owns a strip of 248, beyond depth 4 of 240 columns) or, of several launches, by the tiles in
    registers that take its place on matrices of this size: wider than one strip, ragged, smaller than a strip."""
    for rows, cols, iters in [(70, 600, 9), (37, 250, 5), (130, 83, 6), (64, 256, 8), (5, 3, 7), (1, 1, 4),
                              (40, 244, 17), (33, 484, 11)]:
        w = wl.config(3, rows=rows, cols=cols, iters=iters)
        w.border, w.pad = border, 50.0
        for depth in (1, 2, 3, 4, 5, 6, 7, 8):
            for h, wg in [(16, (1, 64)), (32, (2, 64)), (64, (4, 64)), (128, (8, 8)), (16, (2, 32)), (23, (1, 64))]:
                check(ls, w, wg, blocking=("stream", h, 4, depth))
    w = custom(wl.WEIGHTED_SUM, 90, 300, (1, 1, 1, 1), border, pad=0.4, seed=22, iters=7)
    check(ls, w, (1, 64), blocking=("stream", 32, 4, 4))
    check(ls, w, (2, 64), blocking=("stream", 16, 4, 3), offset=1)          # rows of whole vectors, at no multiple of 16 bytes
    w = custom(wl.WEIGHTED_SUM, 90, 301, (1, 1, 1, 1), border, pad=0.4, seed=23, iters=7)
    check(ls, w, (2, 64), blocking=("stream", 16, 4, 3), offset=1)          # ragged rows
    st = ls.Stencil.from_workload(wl.config(3, rows=64, cols=64))
    st.set_mapping("stream", 32, 4)
    assert st.max_wg_size() == 256 and st.tile_bytes(1, 64) == 0
    assert st.is_legal(1, 64) and st.is_legal(4, 64) and st.is_legal(16, 8)
    assert not st.is_legal(4, 4) and not st.is_legal(1, 96) and not st.is_legal(8, 64)   # whole wavefronts, <= 256
    st.set_option(1, 8)
    with pytest.raises(ls.StencilError):
        st.set_option(1, 9)                                        # two rim lanes cover eight applications
    st.set_mapping("temporal", 2, 4)
    assert not st.is_legal(4, 16)                                  # the local-memory kernels stop at four
    st.set_option(1, 4)
    assert st.is_legal(4, 16)
    clamp = wl.config(3, rows=64, cols=64)
    clamp.border = "clamp"
    with pytest.raises(ls.StencilError):
        ls.Stencil.from_workload(clamp).set_mapping("stream", 32, 4)


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
def test_runs_on_tiles_in_registers(ls, border):
    """Runs of several launches of heat and of the 3x3 sum under both fusing mappings: matrices smaller than a tile either
    way, of exactly a tile's rows or columns (64 and 128 of either) and one more, of several tiles whose last one begins within
    the one before, two and four rows per work-item in one and in several tiles per compute unit, odd and even numbers of
    applications per launch, rows that start at any address; and the bits of the mapping's own kernel (a workgroup that is no whole wavefronts keeps it)."""
    shapes = [(1, 1), (2, 131), (40, 3), (64, 128), (65, 129), (128, 64), (127, 257), (129, 63), (200, 341), (515, 130), (96, 1501),
              (1025, 1999), (2200, 2103)]
    for rows, cols in shapes:
        for iters, depth in [(5, 4), (9, 2), (29, 4)]:
            if rows * cols > 1000000 and iters != 29:
                continue
            h = wl.config(3, rows=rows, cols=cols, iters=iters)
            h.border, h.pad = border, 30.0
            w = custom(wl.WEIGHTED_SUM, rows, cols, (1, 1, 1, 1), border, pad=0.25, seed=rows + cols, iters=iters)
            check(ls, h, (4, 64), blocking=("temporal", 2, 4, depth), offset=cols % 3)
            got = check(ls, w, (4, 64), blocking=("temporal", 2, 4, depth), offset=rows % 3)
            own = gpu_apply(ls, w, w.grid(), (5, 13), blocking=("temporal", 2, 4, depth))
            np.testing.assert_array_equal(got, own)
            if border != "clamp":
                check(ls, h, (4, 64), blocking=("stream", 38, 4, depth))


@pytest.mark.parametrize("kernel,cols,mapping,depth,wg,iters", [
    (wl.LIFE, 1, ("stream", 64, 8), 8, (4, 64), 21), (wl.LIFE, 1, ("temporal", 8, 16), 4, (64, 1), 9),
    (wl.HEAT, 1, ("temporal", 8, 4), 4, (16, 4), 9), (wl.WEIGHTED_SUM, 4, ("stream", 64, 4), 0, (4, 64), 1)])
def test_matrices_as_long_as_a_handle_takes(ls, kernel, cols, mapping, depth, wg, iters):
    """Rows up to just below 2^31: both ends of the matrix agree with the oracle on the rows around the seam of the torus."""
    rows, ends = (2 ** 31 - 70) // cols, 4096
    halo = (2, 2, 2, 2) if kernel == wl.WEIGHTED_SUM else (1, 1, 1, 1)
    w = custom(kernel, 2 * ends, cols, halo, "wrap", seed=7, iters=iters)
    seam = w.grid()                                        # the last rows, then the first
    tin = torch.zeros((rows, cols), device="cuda", dtype=torch.uint8 if kernel == wl.LIFE else torch.float32)
    tin[-ends:], tin[:ends] = torch.from_numpy(seam[:ends]).cuda(), torch.from_numpy(seam[ends:]).cuda()
    st = ls.Stencil(rows, cols, "u8" if kernel == wl.LIFE else "f32", halo, "wrap")
    st.set_kernel(kernel, w.weights, scalars=w.scalars)
    st.set_mapping(*mapping)
    if depth:
        st.set_option(ls.OPT_TEMPORAL_DEPTH, depth)
    tout = st.run(tin, torch.full_like(tin, 1), iters, wg)
    got = torch.cat([tout[-ends:], tout[:ends]]).cpu().numpy()
    st.close()
    keep = slice(2 * iters + 2, 2 * ends - 2 * iters - 2)  # what the slice's own ends do not reach
    want = oracle.apply_workload(w, seam)
    if kernel == wl.WEIGHTED_SUM:
        assert rel_err(got[keep], want[keep]) <= REL_1
    else:
        np.testing.assert_array_equal(got[keep], want[keep])


def test_sweeps_over_a_rotation_of_matrix_pairs(ls):
    """stencil_set_sweep_rotation: a sample is `iters` independent applications on the pairs in turn; every
    pair's output is the single application of its own input, the sweep's own out argument is not written,
    refusals are recorded as ever, and clearing the rotation brings the chain on the caller's pair back."""
    w = wl.config(1, rows=300, cols=520)
    st = ls.Stencil.from_workload(w)
    st.set_mapping("local", 2, 4)
    grids = [w.grid() * np.float32(k + 1) for k in range(3)]
    pairs = [(torch.from_numpy(g).cuda(), torch.full(g.shape, 7.0, dtype=torch.float32, device="cuda")) for g in grids]
    tin = torch.from_numpy(w.grid()).cuda()
    tout = torch.full(w.grid().shape, 7.0, dtype=torch.float32, device="cuda")
    st.set_sweep_rotation(pairs)
    sizes = [(4, 16), (8, 8), (64, 32), (2, 64)]
    res = st.sweep(tin, tout, sizes, iters=4, fixed=(4, 4), reps=5)
    assert [s_ == ls.OK for s_ in res.status] == [True, True, False, True] and res.best is not None
    torch.cuda.synchronize()
    assert float(tout.min()) == 7.0 and float(tout.max()) == 7.0
    for g, (a, b) in zip(grids, pairs):
        ref = oracle.apply(g, w.kernel, w.halo, w.border, w.pad, w.weights, w.scalars, 1)
        assert rel_err(b.cpu().numpy(), ref) <= 1e-5
        np.testing.assert_array_equal(a.cpu().numpy(), g)
    mean, status, best = st.sweep_configs(tin, tout, [("local", 2, 4, 0, (4, 16)), ("direct", 2, 4, 0, (4, 16))], iters=3, reps=5)
    assert status == [ls.OK, ls.OK] and float(tout.min()) == 7.0
    st.set_sweep_rotation([])
    st.sweep(tin, tout, [(4, 16)], iters=4, reps=3)
    torch.cuda.synchronize()
    ref = oracle.apply(w.grid(), w.kernel, w.halo, w.border, w.pad, w.weights, w.scalars, 4)
    assert rel_err(tout.cpu().numpy(), ref) <= 1e-4
    st.close()


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
def test_register_marching_single_application_kernels(ls, border):
    """One application under the streaming mapping, at the sizes of this test marched down the matrix in registers where the
    region has up to five rows, two columns and more and up to 30 cells, in segments of up to six rows, and rows are whole
    vectors, and made by a tile of 2x4 cells elsewhere (the other marches: test_marches_at_any_address, test_c5_full_size_every_cell): matrices wider than
    one strip (252 / 248 / 240 columns), ragged ones, ones smaller than a strip or than the region, unaligned rows, segment
    heights that do and do not divide the rows, and the output bits of the local-memory mapping."""
    shapes = [(70, 600), (37, 252), (41, 256), (130, 83), (64, 1024), (5, 3), (1, 1), (9, 508)]
    for kernel, halo in [(wl.SINCOS, (1, 5, 3, 0)), (wl.WEIGHTED_SUM, (2, 2, 2, 2)), (wl.WEIGHTED_SUM, (3, 3, 3, 3)),
                         (wl.WEIGHTED_SUM, (4, 4, 4, 4)), (wl.WEIGHTED_SUM, (5, 5, 5, 5)),
                         # regions given at run time
                         (wl.WEIGHTED_SUM, (1, 5, 3, 0)), (wl.WEIGHTED_SUM, (2, 1, 2, 2)), (wl.WEIGHTED_SUM, (0, 0, 0, 0)),
                         (wl.WEIGHTED_SUM, (4, 0, 0, 3)), (wl.WEIGHTED_SUM, (0, 5, 4, 0)), (wl.WEIGHTED_SUM, (5, 5, 4, 4)),
                         (wl.WEIGHTED_SUM, (0, 0, 4, 4)), (wl.WEIGHTED_SUM, (2, 2, 1, 0)), (wl.WEIGHTED_SUM, (0, 3, 0, 1)),
                         (wl.WEIGHTED_SUM, (1, 0, 3, 3)), (wl.WEIGHTED_SUM, (2, 2, 4, 3)), (wl.WEIGHTED_SUM, (3, 3, 2, 0))]:
        for rows, cols in shapes + [(23, 241), (12, 484)]:
            w = custom(kernel, rows, cols, halo, border, pad=0.3, seed=rows + cols)
            ref = None
            for h, wg in [(64, (1, 64)), (8, (2, 64)), (1, (4, 64)), (5, (1, 64)), (6, (16, 16)), (29, (8, 8)), (4096, (2, 32))]:
                got = check(ls, w, wg, blocking=("stream", h, 4))
                if ref is None:
                    ref = gpu_apply(ls, w, w.grid(), (8, 8), blocking=(2, 4))
                np.testing.assert_array_equal(got, ref)
        w = custom(kernel, 50, 300, halo, border, pad=0.3, seed=77)
        check(ls, w, (1, 64), blocking=("stream", 5, 4), offset=1)
        check(ls, w, (1, 64), blocking=("stream", 16, 4), offset=1)            # rows of whole vectors, at no multiple of 16 bytes
        check(ls, custom(kernel, 50, 301, halo, border, pad=0.3, seed=78), (1, 64), blocking=("stream", 16, 4),
              offset=1)                                                          # ragged rows
        big = w.grid() * np.float32(300.0)                                       # beyond the small-argument range
        big[3, 5], big[20, 299] = 1.0e6, -3.0e7
        # sums of sines and cosines of large arguments pass near zero: absolute error here
        ref = oracle.apply(big, w.kernel, w.halo, w.border, w.pad, w.weights, w.scalars, 1)
        got = gpu_apply(ls, w, big, (2, 64), blocking=("stream", 16, 4))
        scale = 1.0 if kernel == wl.SINCOS else float(np.abs(big).max())
        assert np.max(np.abs(got.astype(np.float64) - ref)) <= 2e-5 * scale
        np.testing.assert_array_equal(got, gpu_apply(ls, w, big, (8, 8), blocking=(2, 4)))
    st = ls.Stencil.from_workload(wl.config(4, rows=64, cols=64))
    st.set_mapping("stream", 64, 4)
    assert st.max_wg_size() == 256 and st.tile_bytes(1, 64) == 0
    assert st.is_legal(1, 64) and st.is_legal(16, 16) and not st.is_legal(4, 4) and not st.is_legal(8, 64)
    with pytest.raises(ls.StencilError):
        st.set_mapping("stream", 5000, 4)                                        # segment height limit
    with pytest.raises(ls.StencilError):
        ls.Stencil.from_workload(custom(wl.SINCOS, 32, 32, (2, 0, 1, 3), border)).set_mapping("stream", 16, 4)
    with pytest.raises(ls.StencilError):             # beyond the largest region the run-time marching kernel is compiled for
        ls.Stencil.from_workload(custom(wl.WEIGHTED_SUM, 32, 32, (6, 0, 1, 3), border)).set_mapping("stream", 16, 4)


@pytest.mark.parametrize("border", ["wrap", "constant"])
@pytest.mark.parametrize("cols", [7, 8, 17, 31, 32, 33, 63, 64, 65, 447, 449])
def test_life_between_launches_in_bits(ls, border, cols):
    """Runs of one, two and several launches: rows too short for packed matrices, rows that end anywhere in a word
    (where a wrapped word is put together from three), tiles of one strip and of two, a last tile of a few rows."""
    for rows, wg in [(1, (1, 64)), (49, (4, 64)), (130, (2, 64))]:
        for depth, iters in [(8, 5), (8, 19), (3, 6)]:
            w = custom(wl.LIFE, rows, cols, (1, 1, 1, 1), border, pad=1.0, seed=rows * cols, iters=iters)
            check(ls, w, wg, blocking=("stream", 16, 8, depth), offset=cols % 3)


@pytest.mark.parametrize("border", ["wrap", "constant"])
@pytest.mark.parametrize("rows_per_item", [4, 8, 16])
@pytest.mark.parametrize("lanes", [16, 32, 64])
def test_every_tile_of_the_life_streams(ls, border, rows_per_item, lanes):
    """Every kernel of the Life streams - rows per work-item, lanes per row, bytes or bits in and out (a single launch, the
    first, one between and the last of a run) - on ragged boards of several tiles each way with live padding."""
    for wg, depth in [((4, 64), 8), ((2, 64), 3), ((1, 64), 1)]:
        tile_rows = wg[0] * wg[1] // lanes * rows_per_item - 2 * depth
        rows, cols = 2 * max(tile_rows, 1) + 5, 2 * (lanes - 2) * 32 + 45
        for iters in (depth, 2 * depth + 1, 3 * depth):
            w = custom(wl.LIFE, rows, cols, (1, 1, 1, 1), border, pad=1.0, seed=rows + lanes, iters=iters)
            st = ls.Stencil.from_workload(w)
            st.set_mapping("stream", 16, 8)
            st.set_option(ls.OPT_TEMPORAL_DEPTH, depth)
            st.set_option(ls.OPT_LIFE_TILE, (rows_per_item << 16) | lanes)
            g = w.grid()
            tin = torch.from_numpy(g).cuda()
            tout = torch.full_like(tin, 9)
            if tile_rows <= 0:
                with pytest.raises(ls.StencilError):
                    st.run(tin, tout, iters, wg)
            else:
                st.run(tin, tout, iters, wg)
                np.testing.assert_array_equal(tout.cpu().numpy(), oracle.apply_workload(w, g))
            st.close()


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
@pytest.mark.parametrize("tile", [None, (4, 16), (8, 32), (16, 64)])
def test_life_runs_of_several_launches(ls, border, tile):
    """Runs whose launches fuse more generations than asked for, and (a tile prescribed) exactly as many, under both fusing
    mappings: boards lower than a tile, of exactly its rows, of one and of a few rows more, whose last tile then begins
    within the one before; boards narrower than a word; rows that end in a word's first, last and middle cell."""
    mappings = [(("temporal", 2, 16, 4), (4, 64)), (("temporal", 1, 16, 3), (1, 64)), (("temporal", 4, 16, 2), (16, 64))]
    if border != "clamp":
        mappings.append((("stream", 16, 8, 8), (4, 64)))
    for blocking, wg in mappings:
        lanes, per_item = (tile[1], tile[0]) if tile else (16, 4)
        held = wg[0] * wg[1] // lanes * per_item
        for rows, cols in [(1, 5), (held - 1, 31), (held, 33), (held + 1, 65), (2 * held - 7, 32 * (lanes - 2) + 1)]:
            if rows < 1 or rows * cols > 300000:
                continue
            for iters in (blocking[3] + 1, 41):
                w = custom(wl.LIFE, rows, cols, (1, 1, 1, 1), border, pad=1.0, seed=rows + cols, iters=iters)
                st = ls.Stencil.from_workload(w)
                set_mapping(st, blocking)
                if tile:
                    st.set_option(ls.OPT_LIFE_TILE, (tile[0] << 16) | tile[1])
                g = w.grid()
                tin = torch.from_numpy(g).cuda()
                tout = torch.full_like(tin, 9)
                try:
                    st.run(tin, tout, iters, wg)
                except ls.StencilError:                # a prescribed tile without a row beside its rim
                    assert blocking[0] == "stream" and tile and held <= 2 * blocking[3]
                else:
                    np.testing.assert_array_equal(tout.cpu().numpy(), oracle.apply_workload(w, g))
                st.close()


def rows_where_tiles_are_added(ls, cols, border, iters, rows, count):
    """The first `count` heights from `rows` on at which the first launch of the run needs more tiles, or others."""
    found, before = [], None
    while len(found) < count:
        st = ls.Stencil.from_workload(custom(wl.LIFE, rows, cols, (1, 1, 1, 1), border, iters=iters))
        set_mapping(st, ("temporal", 2, 16, 4))
        run = st.describe_run(iters, (4, 64))
        st.close()
        tiles = run["wg"], run["workgroups"], run["launches"]
        if before is not None and tiles != before:
            found.append((rows, run["wg"][0] * run["wg"][1]))
        before, rows = tiles, rows + 1
    return found


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
@pytest.mark.parametrize("iters,items", [(5, 256), (9, 256), (17, 512), (41, 512)])
def test_life_runs_at_the_edges_of_their_tiles(ls, border, iters, items):
    """Boards of exactly the rows of a launch's tiles, whatever workgroup the library takes for them, one row less and one more,
    in one launch (bytes in and out) and in two."""
    for rows, found in rows_where_tiles_are_added(ls, 33, border, iters, 1, 3):
        assert found == items
        for near in (rows - 1, rows, rows + 1):
            for cols in (33, 64, 5):
                check(ls, custom(wl.LIFE, near, cols, (1, 1, 1, 1), border, pad=1.0, seed=near + cols, iters=iters), (4, 64),
                      blocking=("temporal", 2, 16, 4))


@pytest.mark.parametrize("border", ["clamp", "constant"])
def test_life_runs_of_large_workgroups_at_the_edges_of_their_tiles(ls, border):
    """The same where workgroups of 1024 are taken: boards of some 10 million cells, two launches."""
    ((rows, items),) = rows_where_tiles_are_added(ls, 2501, border, 41, 4400, 1)
    assert items == 1024
    for near in (rows - 1, rows):
        check(ls, custom(wl.LIFE, near, 2501, (1, 1, 1, 1), border, pad=1.0, seed=near, iters=41), (4, 64), blocking=("temporal", 2, 16, 4))


@pytest.mark.parametrize("border", ["wrap", "constant"])
def test_register_streaming_life_bit_exact(ls, border):
    """Generations kept in registers: matrices wider than one tile, ragged ones, ones smaller than a
    tile, live padding, unaligned rows, and every segment height and number of cells the mapping
    accepts (neither changes the kernel: test_every_tile_of_the_life_streams goes through those)."""
    for rows, cols, iters in [(70, 1200, 9), (37, 256, 5), (130, 83, 6), (64, 512, 8), (5, 3, 7), (1, 1, 4),
                              (40, 976, 17), (33, 2064, 11)]:
        w = wl.config(2, rows=rows, cols=cols, iters=iters)
        w.border = border
        for cells in (4, 8, 16):
            for depth, h, wg in [(1, 16, (1, 64)), (2, 32, (2, 64)), (3, 7, (4, 64)), (4, 64, (8, 8)), (5, 16, (2, 32)),
                                 (6, 23, (1, 64)), (7, 128, (1, 128)), (8, 38, (1, 64))]:
                check(ls, w, wg, blocking=("stream", h, cells, depth))
    w1 = wl.config(2, rows=80, cols=96, iters=6)
    w1.border, w1.pad = "constant", 1.0                            # live padding
    check(ls, w1, (1, 64), blocking=("stream", 16, 4, 4))
    check(ls, w1, (1, 64), blocking=("stream", 16, 16, 8))
    check(ls, w1, (1, 64), blocking=("stream", 16, 8, 3), offset=5)
    st = ls.Stencil.from_workload(wl.config(2, rows=64, cols=64))
    st.set_mapping("stream", 32, 8)
    assert st.max_wg_size() == 256 and st.tile_bytes(1, 64) == 0
    assert st.is_legal(1, 64) and not st.is_legal(4, 4) and not st.is_legal(8, 64)
    with pytest.raises(ls.StencilError):
        st.set_mapping("stream", 32, 2)                            # 4, 8 or 16 cells per lane
    clamp = wl.config(2, rows=64, cols=64)
    clamp.border = "clamp"
    with pytest.raises(ls.StencilError):
        ls.Stencil.from_workload(clamp).set_mapping("stream", 32, 16)


@pytest.mark.parametrize("wg,blocking", [((5, 7), (2, 4)), ((1, 100), (2, 4)), ((3, 64), (1, 4)),
                                         ((32, 32), (4, 4)), ((32, 32), (8, 4))])
@pytest.mark.parametrize("offset", [0, 1])
def test_tiles_staged_without_registers(ls, wg, blocking, offset):
    """Staging straight into local memory: workgroups that end in part of a wavefront, rows that start at any element, and
    tiles of 72 and 141 KiB, whose addresses need more than 16 bits."""
    rows, cols, halo = 3 * wg[0] * blocking[0] + 5, 3 * wg[1] * blocking[1] + 7, (2, 2, 2, 2)
    check(ls, custom(wl.WEIGHTED_SUM, rows, cols, halo, "clamp"), wg, blocking=blocking, offset=offset)
    rng = np.random.default_rng(3)
    table = rng.integers(-64, 65, size=(6, 6)).astype(np.float32)
    wi = wl.Workload("i32", rows, cols, "i32", (3, 2, 4, 1), "wrap", 3.0, wl.WEIGHTED_SUM, 1, 6, "pow2", weights=table)
    if blocking[0] <= 4:
        check(ls, wi, wg, blocking=blocking, offset=offset)
        wd = wl.Workload("f64", rows, cols, "f64", halo, "constant", 0.5, wl.WEIGHTED_SUM, 1, 5, "pow2",
                         weights=rng.random((5, 5), dtype=np.float32))
        check(ls, wd, wg, blocking=(max(2, blocking[0]), 2), offset=offset)


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
@pytest.mark.parametrize("radius", [3, 4])
@pytest.mark.parametrize("cells_rows", [2, 4])
def test_wide_gaussians_folded_by_rows(ls, border, radius, cells_rows):
    """Compile-time regions in the run-time fold's scheme: edges and remainders of tiles, matrices smaller than a tile, and
    workgroups of one row of work-items, which keep the unrolled fold."""
    # (the last one has several wavefronts per SIMD: folded by rows in every workgroup but the first's of one row)
    for rows, cols in [(3 * 8 * cells_rows + 3, 301), (8 * cells_rows, 128), (7, 5), (61, 133), (8 * cells_rows * 33 + 3, 1030)]:
        w = custom(wl.WEIGHTED_SUM, rows, cols, (radius,) * 4, border, pad=0.25, seed=radius)
        for wg in [(8, 32), (1, 64), (3, 5)]:
            got = check(ls, w, wg, blocking=(cells_rows, 4), offset=1)
            np.testing.assert_array_equal(got, check(ls, w, wg, blocking=(1, 1)))        # the same fold: the same bits


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
@pytest.mark.parametrize("kernel,halo", [(wl.WEIGHTED_SUM, (4, 4, 4, 3)), (wl.WEIGHTED_SUM, (5, 4, 3, 4)), (wl.WEIGHTED_SUM, (5, 5, 3, 3)),
                                         (wl.WEIGHTED_SUM, (1, 5, 3, 0)), (wl.WEIGHTED_SUM, (5, 5, 5, 5)), (wl.SINCOS, (1, 5, 3, 0))])
def test_single_applications_of_the_streaming_mapping(ls, kernel, halo, border):
    """On both sides of the line between the march and the tile (2^25 cells, rows of whole vectors) the output has the bits
    of one cell per work-item, which is compared with the oracle on small matrices."""
    for rows, cols in [(4097, 8192), (4094, 8192), (4100, 8191), (61, 133), (7, 12)]:
        w = custom(kernel, rows, cols, halo, border, pad=0.25, seed=rows)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(rows)
        tin = torch.rand((rows, cols), generator=gen, device="cuda")
        outs = []
        for mapping, wg, nt in [(("local", 1, 1), (8, 32), 0), (("stream", 37, 4), (4, 64), 0), (("stream", 16, 4), (1, 64), 1)]:
            st = ls.Stencil.from_workload(w)
            st.set_mapping(*mapping)
            st.set_option(ls.OPT_NT_STORE, nt)
            outs.append(st.run(tin, torch.full_like(tin, 7.0), 1, wg))
            torch.cuda.synchronize()
            st.close()
        assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2]), (rows, cols)
        if rows < 100:
            check(ls, w, (4, 64), blocking=("stream", 37, 4))


@pytest.mark.parametrize("border", ["wrap", "constant"])
@pytest.mark.parametrize("kernel", [wl.HEAT, wl.WEIGHTED_SUM])
def test_single_launches_of_the_fusing_march(ls, kernel, border):
    """Runs that one launch makes stay with the march whatever the size: every number of applications it is compiled for, rows of
    whole vectors and ragged ones at any address, fewer applications than the handle's depth."""
    for rows, cols in [(70, 600), (37, 250), (130, 83), (40, 244), (5, 3)]:
        for depth in range(1, 9):
            for iters in {depth, max(1, depth - 1)}:
                w = custom(kernel, rows, cols, (1, 1, 1, 1), border, pad=0.4, seed=rows + depth, iters=iters)
                st = ls.Stencil.from_workload(w)
                set_mapping(st, ("stream", 16, 4, depth))
                assert st.describe_run(iters, (2, 64))["kernel"] == "stream_kernel"
                st.close()
                check(ls, w, (2, 64), blocking=("stream", 16, 4, depth), offset=depth % 2)


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
def test_outputs_written_through(ls, border):
    """Launches of several applications with outputs of 16 MiB and a little more, which are written through the L2 caches: the
    march at every depth that does it, the temporal kernels, the register tiles, Life from and to bytes and bits; rows of whole
    vectors and ragged ones, at any address."""
    cases = [(kernel, 2049, 2051, ("temporal", 2, 4, 3), (8, 32), iters, name)
             for kernel in (wl.HEAT, wl.WEIGHTED_SUM) for iters, name in ((3, "temporal_kernel"), (7, "register_tile_kernel"))]
    cases += [(wl.LIFE, 4099, 4101, ("temporal", 2, 16, 4), (16, 32), 4, "life_temporal_kernel"),
              (wl.LIFE, 4099, 4101, ("temporal", 2, 16, 4), (16, 32), 21, "life_stream_kernel")]
    if border != "clamp":
        cases += [(kernel, 2049, 2052, ("stream", 38, 4, depth), (2, 64), depth, "stream_through_kernel")
                  for kernel in (wl.HEAT, wl.WEIGHTED_SUM) for depth in (4, 5, 6, 7, 8)]
        cases += [(wl.LIFE, 4099, 4101, ("stream", 16, 8, 8), (4, 64), iters, "life_stream_kernel") for iters in (8, 40)]
    for kernel, rows, cols, blocking, wg, iters, name in cases:
        w = custom(kernel, rows, cols, (1, 1, 1, 1), border, pad=1.0, seed=iters, iters=iters)
        st = ls.Stencil.from_workload(w)
        set_mapping(st, blocking)
        assert st.describe_run(iters, wg)["kernel"] == name, blocking
        st.close()
        check(ls, w, wg, blocking=blocking, offset=iters % 2)


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
@pytest.mark.parametrize("kernel,halo,rows,cols", [
    (wl.WEIGHTED_SUM, (3, 4, 4, 4), 4098, 8192), (wl.WEIGHTED_SUM, (5, 5, 4, 4), 4098, 8196), (wl.WEIGHTED_SUM, (5, 4, 3, 4), 4098, 8192),
    (wl.WEIGHTED_SUM, (5, 5, 3, 3), 4098, 8192), (wl.SINCOS, (1, 5, 3, 0), 2050, 8196), (wl.WEIGHTED_SUM, (2, 2, 2, 2), 1030, 2052),
    (wl.WEIGHTED_SUM, (1, 1, 4, 4), 1030, 2052), (wl.WEIGHTED_SUM, (2, 0, 0, 1), 517, 1028)])
def test_marches_at_any_address(ls, kernel, halo, rows, cols, border):
    """The marches of one application, each with seven to nine columns of eight rows and more, sin/cos and regions of up to five
    rows among them: rows that start at a multiple of 16 bytes and at none, both kinds of store, the bits of one cell per
    work-item (compared with the oracle on small matrices by other tests)."""
    w = custom(kernel, rows, cols, halo, border, pad=0.25, seed=rows)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows)
    for offset in (0, 1):
        tin = torch.rand(rows * cols + offset, generator=gen, device="cuda")[offset:]
        outs = []
        tall, low = (6, 3) if max(halo[:2]) <= 2 else (37, 16)
        for mapping, wg, nt in [(("local", 1, 1), (8, 32), 0), (("stream", tall, 4), (4, 64), 0), (("stream", low, 4), (1, 64), 1)]:
            st = ls.Stencil.from_workload(w)
            st.set_mapping(*mapping)
            st.set_option(ls.OPT_NT_STORE, nt)
            assert mapping[0] == "local" or "march" in st.describe_run(1, wg)["kernel"]
            out = torch.full((rows * cols + offset + 1,), 7.0, device="cuda")
            st.run(tin, out[offset:-1], 1, wg)
            torch.cuda.synchronize()
            assert float(out[-1]) == 7.0 and (offset == 0 or float(out[0]) == 7.0)
            outs.append(out)
            st.close()
        assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2]), offset


def test_temporal_blocking_not_offered_for_other_regions(ls):
    st = ls.Stencil.from_workload(wl.config(1))                    # 5x5 region
    with pytest.raises(ls.StencilError):
        st.set_mapping("temporal", 2, 4)
    st2 = ls.Stencil.from_workload(wl.config(3))
    st2.set_mapping("temporal", 2, 4)
    with pytest.raises(ls.StencilError):
        st2.set_option(1, 5)                                       # depth limit is 4
    st2.set_option(1, 4)
    assert st2.tile_bytes(4, 16) == 2 * (8 + 8) * (64 + 8) * 4 + 32     # two buffers, rim 4 rows / 1 vector


# ---- gold standard (Section 5): every workgroup size gives the output of the baseline size ---

@pytest.mark.parametrize("index", [1, 2, 3, 4])
def test_every_swept_size_matches_baseline_output(ls, index):
    rows, cols = (300, 260)
    w = wl.config(index, rows=rows, cols=cols, iters=3 if index in (2, 3) else 1)
    g = w.grid()
    base = gpu_apply(ls, w, g, (4, 4))
    sizes = wl.enumerate_wg("pow2") if index != 4 else wl.enumerate_wg("even")[::7]
    vec = 16 if w.dtype == "u8" else 4
    mappings = [(1, 1), (4, vec)] + ([("direct", 1, vec), ("direct", 4, vec)] if index != 4 else [])
    for blocking in mappings:
        st = ls.Stencil.from_workload(w)
        set_mapping(st, blocking)
        tdt = torch.float32 if w.dtype == "f32" else torch.uint8
        tin = torch.from_numpy(g).cuda()
        tout = torch.empty_like(tin)
        assert tin.dtype == tdt
        n_run = 0
        for wg in sizes:
            if not st.is_legal(*wg):
                with pytest.raises(ls.Refused):
                    st.run(tin, tout, w.iters, wg)
                continue
            tout.fill_(9)
            st.run(tin, tout, w.iters, wg)
            np.testing.assert_array_equal(tout.cpu().numpy(), base, err_msg="wg %s blocking %s" % (wg, blocking))
            n_run += 1
        assert n_run >= len(sizes) // 2
        st.close()


@pytest.mark.parametrize("index", [1, 2, 3, 4])
def test_gold_standard_at_full_size(ls, index):
    """The same check on the full-size workloads, for every size of the workload's own list (66
    powers of two; all 590 even sizes for C5) under the paper's mapping, the fast mappings and the
    register-streaming ones: outputs are compared on the device with the 4x4 baseline's, which
    the full-size tests below tie to the oracle."""
    w = wl.config(index, iters=2 if index in (2, 3) else None)
    tin = torch.from_numpy(w.grid()).cuda()
    base = torch.empty_like(tin)
    st = ls.Stencil.from_workload(w)
    st.run(tin, base, w.iters, (4, 4))
    st.close()
    vec = 16 if w.dtype == "u8" else 4
    mappings = {1: [(1, 1), (2, vec), ("direct", 2, vec), ("stream", 10, vec)],
                2: [(1, 1), (2, vec), ("direct", 2, vec), ("temporal", 2, vec, 2), ("stream", 40, 4, 2)],
                3: [(1, 1), (2, vec), ("direct", 2, vec), ("temporal", 2, vec, 2), ("stream", 38, vec, 2)],
                4: [(1, 1), (4, vec), ("stream", 134, vec)]}[index]
    tout = torch.empty_like(tin)
    for blocking in mappings:
        st = ls.Stencil.from_workload(w)
        set_mapping(st, blocking)
        n_run = 0
        for wg in w.wg_sizes():
            if not st.is_legal(*wg):
                continue
            tout.fill_(9)
            st.run(tin, tout, w.iters, wg)
            assert torch.equal(tout, base), "wg %s blocking %s" % (wg, blocking)
            n_run += 1
        assert n_run >= (4 if blocking[0] == "stream" else len(w.wg_sizes()) // 2), (blocking, n_run)
        st.close()


# ---- degenerate shapes and the error paths ----------------------------------------------------

@pytest.mark.parametrize("shape", [(1, 1), (1, 37), (41, 1), (2, 3), (5, 4)])
def test_tiny_matrices_smaller_than_the_region(ls, shape):
    for border in ("clamp", "wrap", "constant"):
        w = custom(wl.WEIGHTED_SUM, shape[0], shape[1], (3, 2, 4, 1), border, pad=0.25, seed=11)
        for blocking in [(1, 1), (4, 4)]:
            check(ls, w, (4, 8), blocking=blocking)
        wlife = wl.config(2, rows=shape[0], cols=shape[1], iters=3)
        wlife.border = border
        check(ls, wlife, (2, 2))
        check(ls, wlife, (4, 4), blocking=(2, 16))
        check(ls, wlife, (4, 4), blocking=("direct", 2, 16))
        wheat = wl.config(3, rows=shape[0], cols=shape[1], iters=3)
        wheat.border = border
        check(ls, wheat, (4, 4), blocking=("direct", 1, 4))
        w3 = custom(wl.WEIGHTED_SUM, shape[0], shape[1], (2, 2, 2, 2), border, pad=0.25, seed=12)
        check(ls, w3, (2, 8), blocking=("direct", 4, 4))


def test_iters_zero_copies_and_even_odd_iteration_counts(ls):
    w = wl.config(3, rows=64, cols=80)
    g = w.grid()
    np.testing.assert_array_equal(gpu_apply(ls, w, g, (4, 4), iters=0), g)
    for it in (1, 2, 3, 4):
        check(ls, w, (8, 8), iters=it)


def test_one_handle_serves_successive_weight_tables_and_kernels(ls):
    """A handle whose weight table (kept on the device for run-time regions) is replaced, and whose
    kernel is switched, between runs on a side stream: every run uses what was set last."""
    halo = (2, 1, 3, 0)
    w = custom(wl.WEIGHTED_SUM, 90, 117, halo, "wrap", seed=8)
    g = w.grid()
    st = ls.Stencil.from_workload(w)
    st.set_mapping("local", 2, 4)
    tin = torch.from_numpy(g).cuda()
    tout = torch.empty_like(tin)
    side = torch.cuda.Stream()
    rng = np.random.default_rng(12)
    tables, results = [], []
    for k in range(3):
        table = rng.random((halo[0] + halo[1] + 1, halo[2] + halo[3] + 1), dtype=np.float32)
        tables.append(table)
        st.set_kernel("weighted_sum", table)
        with torch.cuda.stream(side):
            for _ in range(4):                          # still in flight when the next table arrives
                st.run(tin, tout, 3, (8, 16), stream=side)
            results.append(tout.clone())
    side.synchronize()
    for table, res in zip(tables, results):
        ref = oracle.apply(g, wl.WEIGHTED_SUM, halo, "wrap", 0.0, table, (), 3)
        assert rel_err(res.cpu().numpy(), ref) <= REL_N
    st.set_kernel("sincos", table)
    st.run(tin, tout, 1, (8, 16))
    torch.cuda.synchronize()
    ref = oracle.apply(g, wl.SINCOS, halo, "wrap", 0.0, table, (), 1)
    assert np.max(np.abs(tout.cpu().numpy() - ref)) <= 1e-4
    st.close()


def test_error_paths_do_not_launch(ls):
    w = wl.config(1, rows=64, cols=64)
    st = ls.Stencil.from_workload(w)
    tin = torch.from_numpy(w.grid()).cuda()
    tout = torch.full_like(tin, -1.0)
    for wg in [(64, 32), (2048, 1), (0, 4), (-1, 4)]:
        with pytest.raises(ls.Refused):
            st.run(tin, tout, 1, wg)
    torch.cuda.synchronize()
    assert float(tout.max()) == -1.0                               # nothing ran
    with pytest.raises(ls.StencilError) as e:
        st.run(tin, tin, 1, (4, 4))                                # aliasing
    assert e.value.code == ls.E_INVALID
    both = torch.zeros(64 * 64 + 32, device="cuda")
    with pytest.raises(ls.StencilError):
        st.run(both[:4096], both[32:], 1, (4, 4))                  # partial overlap
    with pytest.raises(ls.StencilError):
        st.run(tin, tout, -1, (4, 4))
    st.run(tin, tout, 1, (0, 0))                                   # library's own choice
    torch.cuda.synchronize()
    ref = oracle.apply_workload(w)
    assert rel_err(tout.cpu().numpy(), ref) <= REL_1


def test_sweep_over_whole_configurations(ls):
    """Mapping, fused applications and workgroup size swept together; the scenario is left on the
    fastest configuration and still computes the oracle's result with it."""
    w = wl.config(3, rows=512, cols=768, iters=8)
    g = w.grid()
    st = ls.Stencil.from_workload(w)
    tin = torch.from_numpy(g).cuda()
    tout = torch.empty_like(tin)
    configs = [("local", 1, 1, 0, (4, 4)), ("direct", 2, 4, 0, (4, 16)), ("temporal", 2, 4, 4, (16, 16)),
               ("stream", 23, 4, 8, (1, 64)), ("stream", 23, 4, 8, (4, 4)),      # not whole wavefronts: refused
               ("temporal", 2, 4, 8, (16, 16)),                                   # depth the mapping lacks
               ("direct", 3, 4, 0, (4, 16)),                                      # no such mapping
               ("local", 2, 4, 0, (64, 32)),                                      # above W_max: refused
               ("direct", 2, 4, 0, (4, 16), 0)]                                   # plain workgroup numbering
    mean, status, best = st.sweep_configs(tin, tout, configs, iters=8, reps=5)
    assert status == [ls.OK, ls.OK, ls.OK, ls.OK, ls.E_REFUSED, ls.E_INVALID, ls.E_INVALID, ls.E_REFUSED, ls.OK]
    assert all((m > 0) == (s == ls.OK) for m, s in zip(mean, status)) and all(np.isnan(m) for m, s in zip(mean, status) if s != ls.OK)
    assert best == int(np.nanargmin(mean)) and status[best] == ls.OK
    sg, cr, cc = st.get_mapping()
    assert (sg, cr, cc) == ({"local": 0, "direct": 1, "temporal": 2, "stream": 3}[configs[best][0]],) + tuple(configs[best][1:3])
    st.run(tin, tout, w.iters, (0, 0))                               # the remembered size of that configuration
    torch.cuda.synchronize()
    np.testing.assert_array_equal(tout.cpu().numpy(), oracle.apply_workload(w, g))
    # nothing usable: the scenario keeps the configuration it had
    before = st.get_mapping()
    mean, status, best = st.sweep_configs(tin, tout, [("direct", 3, 4, 0, (4, 16))], iters=1, reps=3)
    assert best == -1 and status == [ls.E_INVALID] and st.get_mapping() == before
    st.close()


def test_device_copy_and_workgroup_numbering_option(ls):
    for n in (1, 15, 16, 17, 4096, 1000003):
        a = torch.randint(0, 255, (n,), dtype=torch.uint8, device="cuda")
        b = torch.zeros_like(a)
        ls.device_copy(a, b)
        torch.cuda.synchronize()
        assert torch.equal(a, b), n
    x = torch.zeros(64, device="cuda")
    with pytest.raises(ls.StencilError):
        ls.device_copy(x[:32], x[16:48])                             # overlap
    a = torch.randint(0, 255, (1 << 20,), dtype=torch.uint8, device="cuda")
    b = torch.zeros_like(a)
    mean_ms, min_ms = ls.time_copy(a, b, burst=4, reps=5)
    assert 0.0 < min_ms <= mean_ms < 10.0 and torch.equal(a, b)
    with pytest.raises(ls.StencilError):
        ls.time_copy(a, b, burst=0, reps=5)
    # the XCD-aware numbering of workgroups changes the schedule, never the values
    w = wl.config(4, rows=200, cols=312)
    g = w.grid()
    outs = []
    for remap in (1, 0):
        st = ls.Stencil.from_workload(w)
        st.set_mapping("local", 2, 4)
        st.set_option(ls.OPT_XCD_REMAP, remap)
        tin = torch.from_numpy(g).cuda()
        tout = torch.empty_like(tin)
        st.run(tin, tout, 1, (4, 8))                                # 25 x 10 tiles: above the remap threshold
        torch.cuda.synchronize()
        outs.append(tout.cpu().numpy())
        st.close()
    np.testing.assert_array_equal(outs[0], outs[1])
    assert rel_err(outs[0], oracle.apply_workload(w, g)) <= REL_1


def test_non_temporal_stores_change_no_value(ls):
    """STENCIL_OPT_NT_STORE only changes how output vectors are written: every kernel family gives
    the same matrix with it as without it, and the one the oracle gives."""
    heat = wl.config(3, rows=150, cols=256, iters=8)
    heat.border = "constant"
    life = wl.config(2, rows=150, cols=256, iters=8)
    cases = [(heat, ("local", 2, 4)), (heat, ("direct", 2, 4)), (heat, ("temporal", 2, 4, 4)), (heat, ("stream", 20, 4, 8)),
             (life, ("local", 2, 16)), (life, ("direct", 2, 16)), (life, ("temporal", 2, 16, 2)), (life, ("stream", 20, 16, 8)),
             (custom(wl.SINCOS, 90, 256, (1, 5, 3, 0), "clamp", seed=4), ("stream", 16, 4)),
             (custom(wl.WEIGHTED_SUM, 90, 256, (3, 0, 2, 1), "wrap", seed=4), ("local", 2, 4))]
    for w, blocking in cases:
        g = w.grid()
        ref = oracle.apply_workload(w, g)
        tin = torch.from_numpy(g).cuda()
        outs = []
        for nt in (0, 1):
            st = ls.Stencil.from_workload(w)
            set_mapping(st, blocking)
            st.set_option(ls.OPT_NT_STORE, nt)
            tout = torch.zeros_like(tin)
            st.run(tin, tout, w.iters, (2, 64))
            torch.cuda.synchronize()
            outs.append(tout.cpu().numpy())
            st.close()
        np.testing.assert_array_equal(outs[0], outs[1])
        if w.dtype == "u8" or w.kernel == wl.HEAT:
            np.testing.assert_array_equal(outs[1], ref)
        else:
            assert rel_err(outs[1], ref) <= REL_1
    # the switch is one of the things stencil_sweep_configs sweeps
    w = wl.config(3, rows=512, cols=512, iters=1)
    st = ls.Stencil.from_workload(w)
    tin = torch.from_numpy(w.grid()).cuda()
    tout = torch.empty_like(tin)
    mean, status, best = st.sweep_configs(tin, tout, [("direct", 2, 4, 0, (4, 16), 1, nt) for nt in (0, 1)], iters=2, reps=3)
    assert status == [ls.OK, ls.OK] and best in (0, 1)
    st.close()


def test_plain_cpp_example_runs(ls):
    """The C ABI from a program that is neither Python nor PyTorch: the example built by
    build() sweeps, runs 1000 heat steps at the best size and checks conservation itself."""
    import subprocess
    from paper_1511_02490_amd import build
    if not os.path.exists(build.EXAMPLE_BIN):
        build.build_example()              # normally done by __graft_entry__.build()
    for args, first in (([], "default size before any sweep: 4x64"),
                        ([ls.tuning_data_path("local,2,4")], "predicted size before any sweep: ")):
        proc = subprocess.run([build.EXAMPLE_BIN] + args, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True,
                              timeout=120)
        assert proc.returncode == 0, proc.stdout
        assert first in proc.stdout and "sizes swept; best" in proc.stdout and "after 1000 steps" in proc.stdout


def test_runs_on_a_side_stream(ls):
    w = wl.config(0)
    g = w.grid()
    st = ls.Stencil.from_workload(w)
    side = torch.cuda.Stream()
    tin = torch.from_numpy(g).cuda()
    tout = torch.empty_like(tin)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        st.run(tin, tout, 1, (8, 8))
    side.synchronize()
    assert rel_err(tout.cpu().numpy(), oracle.apply_workload(w, g)) <= REL_1


@pytest.mark.parametrize("rows,cols", [(1229, 1280), (1228, 1280), (1100, 1431), (2046, 4099), (2047, 4099), (2049, 4128)])
def test_single_applications_written_through(ls, rows, cols):
    """Outputs from 6 MiB on (ragged rows: up to 32 MiB) are written through by kernels of their own: the bits are those of the
    kernels that non-temporal stores keep, in every cell, and cells behind the output stay as they were."""
    gen = np.random.default_rng(rows * 10000 + cols)
    types = {"f32": torch.float32, "u8": torch.uint8, "i32": torch.int32, "f64": torch.float64}
    for kernel, dtype, halo, border, mapping in [
            ("weighted_sum", "f32", (1, 1, 1, 1), "clamp", ("local", 2, 4)), ("weighted_sum", "f32", (2, 2, 2, 2), "wrap", ("local", 2, 4)),
            ("weighted_sum", "f32", (3, 3, 3, 3), "constant", ("local", 2, 4)), ("weighted_sum", "f32", (1, 0, 3, 2), "clamp", ("local", 2, 4)),
            ("weighted_sum", "f32", (2, 2, 2, 2), "clamp", ("direct", 2, 4)), ("weighted_sum", "u8", (2, 2, 2, 2), "clamp", ("local", 2, 4)),
            ("weighted_sum", "i32", (3, 2, 4, 1), "wrap", ("local", 2, 4)), ("weighted_sum", "f64", (2, 2, 2, 2), "constant", ("local", 2, 2)),
            ("sincos", "f32", (1, 5, 3, 0), "constant", ("local", 2, 4)), ("sobel", "f32", (1, 1, 1, 1), "wrap", ("direct", 2, 4)),
            ("nms", "f32", (1, 1, 1, 1), "clamp", ("direct", 2, 4))]:
        n, s, e, w = halo
        shape = (n + s + 1, e + w + 1)
        grid = gen.integers(0, 200, size=(rows, cols)) if dtype in ("u8", "i32") else gen.random((rows, cols))
        tin = torch.from_numpy(grid).to(types[dtype]).cuda()
        st = ls.Stencil(rows, cols, dtype, halo, border)
        if kernel in ("weighted_sum", "sincos"):
            st.set_kernel(kernel, gen.integers(-9, 10, size=shape).astype(np.float32) if dtype == "i32" else gen.random(shape, dtype=np.float32))
        else:
            st.set_kernel(kernel)
        st.set_mapping(*mapping)
        outs = []
        for nt in (0, 1):
            st.set_option(ls.OPT_NT_STORE, nt)
            buf = torch.full((rows * cols + 64,), 77, dtype=types[{1: "f32"}.get(tin.element_size(), dtype)], device="cuda")
            st.run(tin, buf[:rows * cols], 1, (8, 32))
            torch.cuda.synchronize()
            assert bool((buf[rows * cols:] == 77).all())
            outs.append(buf)
        assert torch.equal(outs[0], outs[1]), (kernel, dtype, halo, border, mapping)
        st.close()


WRITTEN_THROUGH = [(wl.WEIGHTED_SUM, "f32", (1, 1, 1, 1), ("local", 2, 4)), (wl.WEIGHTED_SUM, "f32", (2, 2, 2, 2), ("local", 2, 4)),
                   (wl.WEIGHTED_SUM, "f32", (4, 4, 4, 4), ("local", 2, 4)), (wl.WEIGHTED_SUM, "f32", (1, 0, 3, 2), ("local", 2, 4)),
                   (wl.WEIGHTED_SUM, "f32", (3, 3, 3, 3), ("direct", 2, 4)), (wl.WEIGHTED_SUM, "u8", (2, 2, 2, 2), ("local", 2, 4)),
                   (wl.WEIGHTED_SUM, "i32", (3, 2, 4, 1), ("local", 2, 4)), (wl.WEIGHTED_SUM, "f64", (2, 2, 2, 2), ("local", 2, 2)),
                   (wl.SINCOS, "f32", (1, 5, 3, 0), ("local", 2, 4)), (wl.SOBEL, "f32", (1, 1, 1, 1), ("direct", 2, 4)),
                   (wl.NMS, "f32", (1, 1, 1, 1), ("local", 2, 4))]


@pytest.mark.parametrize("border", ["clamp", "wrap", "constant"])
@pytest.mark.parametrize("kernel,dtype,halo,blocking", WRITTEN_THROUGH)
def test_written_through_kernels_against_the_oracle(ls, kernel, dtype, halo, blocking, border):
    """The smallest output that is written through, by the kernel that the library says does it, and one row less, which is not:
    against the oracle, whole and ragged tiles below and right."""
    for rows in (1229, 1228):
        cols = 1280 if dtype != "f64" else 640
        w = custom(kernel, rows, cols, halo, border, pad=0.0 if dtype in ("u8", "i32") else 0.25, seed=rows)
        w.dtype = dtype
        if dtype == "i32":
            w.weights = np.rint(w.weights * 1000).astype(np.float32)
        st = ls.Stencil.from_workload(w)
        st.set_mapping(*blocking)
        assert st.describe_launch(1, (8, 32))["store"] == (ls.STORE_THROUGH if rows == 1229 else ls.STORE_PLAIN)
        st.close()
        check(ls, w, (8, 32), blocking=blocking)


def test_iterated_run_inside_a_hip_graph(ls):
    """An iterated stencil_run is only kernel launches once its scratch matrix exists, so it can
    be captured into a HIP graph; every replay must reproduce the eager result."""
    w = wl.config(3, rows=192, cols=256, iters=9)
    g = w.grid()
    ref = oracle.apply_workload(w, g)
    for blocking in [("direct", 2, 4), ("temporal", 2, 4, 4), ("stream", 23, 4, 8)]:
        st = ls.Stencil.from_workload(w)
        set_mapping(st, blocking)
        tin = torch.from_numpy(g).cuda()
        tout = torch.zeros_like(tin)
        st.run(tin, tout, w.iters, (4, 16))                     # eager: allocates the scratch matrix
        torch.cuda.synchronize()
        np.testing.assert_array_equal(tout.cpu().numpy(), ref)
        graph = torch.cuda.CUDAGraph()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            with torch.cuda.graph(graph, stream=side):
                st.run(tin, tout, w.iters, (4, 16), stream=side)
        torch.cuda.synchronize()
        for replay in range(3):
            tout.fill_(-1.0)                                    # eager work between the replays
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            np.testing.assert_array_equal(tout.cpu().numpy(), ref, err_msg="replay %d %s" % (replay, blocking))
        st.close()


# ---- the sweep (Section 5) ---------------------------------------------------------------------

def test_sweep_reports_times_best_and_refusals(ls):
    w = wl.config(1, rows=512, cols=512)
    st = ls.Stencil.from_workload(w)
    tin = torch.from_numpy(w.grid()).cuda()
    tout = torch.empty_like(tin)
    sizes = [(4, 4), (8, 8), (16, 16), (64, 4), (4, 64), (64, 32), (1, 1024), (1024, 1)]
    res = st.sweep(tin, tout, sizes, iters=1, fixed=(32, 4), reps=30)
    assert res.status[5] == ls.E_REFUSED and np.isnan(res.mean_ms[5])
    ok = [i for i, s in enumerate(res.status) if s == ls.OK]
    assert ok == [0, 1, 2, 3, 4, 6, 7]
    for i in ok:
        assert res.mean_ms[i] > 0 and res.min_ms[i] <= res.median_ms[i] and res.min_ms[i] <= res.mean_ms[i]
        assert res.stddev_ms[i] >= 0
    assert res.best_index == int(np.nanargmin(res.mean_ms))
    assert res.speedup_over_fixed > 0
    # the reductions agree with the oracle's definitions on the measured table
    from oracle import tuning
    assert res.best_index == tuning.oracle_size(sizes, res.mean_ms, [s == ls.OK for s in res.status])
    # the last sample's output is still the stencil's output
    torch.cuda.synchronize()
    assert rel_err(tout.cpu().numpy(), oracle.apply_workload(w)) <= REL_1
    # (0, 0) now means the sweep's best size
    st.run(tin, tout, 1, (0, 0))
    torch.cuda.synchronize()
    assert rel_err(tout.cpu().numpy(), oracle.apply_workload(w)) <= REL_1


def test_sweep_records_a_size_refused_at_launch_and_goes_on(ls):
    """One size of the list is made to fail when launched (the runtime's out-of-resources error in
    the launch's place): the sweep records it as refused, times the others and picks among them."""
    w = wl.config(1, rows=512, cols=512)
    st = ls.Stencil.from_workload(w)
    tin = torch.from_numpy(w.grid()).cuda()
    tout = torch.empty_like(tin)
    sizes = [(4, 4), (8, 8), (16, 16), (4, 64)]
    st.set_option(ls.OPT_FAIL_LAUNCH, (8 << 16) | 8)
    assert st.is_legal(8, 8)                              # nothing known against it before the launch
    res = st.sweep(tin, tout, sizes, iters=1, fixed=(8, 8), reps=5)
    assert res.status == [ls.OK, ls.E_REFUSED, ls.OK, ls.OK]
    assert np.isnan(res.mean_ms[1]) and np.isnan(res.min_ms[1]) and np.isnan(res.speedup_over_fixed)
    assert res.best in [(4, 4), (16, 16), (4, 64)] and all(res.mean_ms[i] > 0 for i in (0, 2, 3))
    with pytest.raises(ls.Refused) as e:
        st.run(tin, tout, 1, (8, 8))
    assert "refused at launch" in str(e.value)
    mean, status, best = st.sweep_configs(tin, tout, [("local", 1, 1, 0, (8, 8)), ("local", 2, 4, 0, (8, 8)),
                                                      ("local", 1, 1, 0, (16, 16))], iters=1, reps=3)
    assert status == [ls.E_REFUSED, ls.E_REFUSED, ls.OK] and best == 2
    st.set_option(ls.OPT_FAIL_LAUNCH, 0)
    st.run(tin, tout, 1, (8, 8))
    torch.cuda.synchronize()
    assert rel_err(tout.cpu().numpy(), oracle.apply_workload(w)) <= REL_1
    st.close()


def test_limits_come_from_the_device_and_the_largest_legal_tile_launches(ls):
    """Section 3.1 / 3.2: W_max(s) and the device's features are asked of the device and the compiled
    kernel.  After a first run f(s) carries the device's own figures; the largest tile any size of the
    sweep's list may stage - close to all of a compute unit's local memory - launches and is right."""
    halo = (30, 30, 30, 30)                                # Table 2's largest border region
    w = custom(wl.WEIGHTED_SUM, 300, 280, halo, "wrap", seed=17)
    st = ls.Stencil.from_workload(w)
    tin = torch.from_numpy(w.grid()).cuda()
    tout = torch.empty_like(tin)
    st.run(tin, tout, 1, (4, 4))
    torch.cuda.synchronize()
    props = torch.cuda.get_device_properties(0)
    f = st.features()
    assert f[9] == props.multi_processor_count
    limit = int(f[10])
    assert limit >= 64 * 1024 and f[11] == 1024.0 and st.max_wg_size() <= 1024
    ref = oracle.apply_workload(w)
    best = None
    for blocking in [(1, 1), (2, 4), (4, 4), (8, 4), (8, 1)]:
        st.set_mapping("local", *blocking)
        for wg in wl.enumerate_wg("pow2"):
            nbytes = st.tile_bytes(*wg) if wg[0] * wg[1] <= st.max_wg_size() else 0
            assert st.is_legal(*wg) == (0 < nbytes <= limit)
            if st.is_legal(*wg) and (best is None or nbytes > best[0]):
                best = (nbytes, blocking, wg)
    nbytes, blocking, wg = best
    assert nbytes > 0.9 * limit, best                      # within a tenth of the whole local memory
    st.set_mapping("local", *blocking)
    st.run(tin, tout, 1, wg)
    torch.cuda.synchronize()
    assert rel_err(tout.cpu().numpy(), ref) <= REL_1
    # one step larger in either direction is refused before any launch
    for bigger in ((wg[0] * 2, wg[1]), (wg[0], wg[1] * 2)):
        with pytest.raises(ls.Refused):
            st.run(tin, tout, 1, bigger)
    st.close()


def _training_pairs_without(path, dropped, tmp_path):
    """Copy of a training-pair file without the scenarios whose names contain `dropped`."""
    out, skip = [], False
    n = 0
    for line in open(path):
        if line.startswith("# ") and not line.startswith("# (") and not line.startswith("# scenario"):
            skip = dropped in line
            n += skip
        if not skip or line.startswith("features"):
            out.append(line)
    assert n >= 1
    target = tmp_path / "held_out.txt"
    target.write_text("".join(out))
    return str(target)


def test_pretrained_predictor_picks_a_good_size(ls, tmp_path):
    """The shipped training pairs, with the heat kernel at 4096^2 left out, still lead to a size for the
    4096^2 heat step that is legal and runs within reach of the sweep's best (Section 7's "performance");
    so does the classifier as shipped when the library makes the choice itself (wg = (0, 0))."""
    w = wl.config(3, iters=4)
    sizes = w.wg_sizes()
    tin = torch.from_numpy(w.grid()).cuda()
    tout = torch.empty_like(tin)
    for mapping in ("local,1,1", "local,2,4"):
        st = ls.Stencil.from_workload(w)
        m = mapping.split(",")
        st.set_mapping(m[0], int(m[1]), int(m[2]))
        pred = ls.Predictor.load(_training_pairs_without(ls.tuning_data_path(mapping), "he 4096x4096", tmp_path))
        wg = st.predict(pred, sizes)
        # what is asserted is that the prediction is a legal size of the list that was timed; its
        # quality is a measurement (printed, and reported by bench.py and the study), with only a
        # bound generous enough that timer noise cannot turn it red
        assert wg in sizes and st.is_legal(*wg)
        shipped = ls.pretrained_predictor(mapping)
        st.attach_predictor(shipped)
        ref = oracle.apply_workload(w, iters=4)
        st.run(tin, tout, 4, (0, 0))                       # the library's own choice: Algorithm 1 inside
        torch.cuda.synchronize()
        np.testing.assert_array_equal(tout.cpu().numpy(), ref)
        res = st.sweep(tin, tout, sizes, iters=4, fixed=(4, 4), reps=5)
        performance = res.best_ms / res.ms_of(wg)
        print("pretrained %s, heat at 4096^2 held out: predicted %s, performance %.2f, %.1fx over 4x4" % (
            mapping, wg, performance, res.ms_of((4, 4)) / res.ms_of(wg)))
        assert performance >= 0.25, (mapping, wg, performance)
        pred.close()
        st.close()


@pytest.mark.parametrize("cutoff", [0, 150])
def test_sweep_times_sizes_that_come_to_the_same_launches_once(ls, cutoff):
    """Runs of heat on tiles in registers take a workgroup of their own: of the sizes that lead there the figures are shared
    and the smallest is best; a size that is no whole wavefronts keeps the mapping's kernel and has its own."""
    w = wl.config(3, rows=700, cols=900, iters=24)
    st = ls.Stencil.from_workload(w)
    st.set_mapping("temporal", 2, 4)
    st.set_option(ls.OPT_TEMPORAL_DEPTH, 4)
    st.set_option(ls.OPT_SWEEP_CUTOFF, cutoff)
    tin = torch.from_numpy(w.grid()).cuda()
    res = st.sweep(tin, torch.empty_like(tin), [(16, 64), (5, 13), (4, 64), (3, 64)], iters=24, fixed=(8, 32), reps=5)
    assert [st.describe_run(24, wg)["kernel"] for wg in [(16, 64), (5, 13), (8, 32)]] == [
        "register_tile_kernel", "temporal_kernel", "register_tile_kernel"]
    for figures in (res.mean_ms, res.min_ms, res.median_ms, res.stddev_ms):
        assert figures[0] == figures[2] == figures[3] != figures[1]
    assert res.best == (3, 64) and st.default_wg() == (3, 64)
    if cutoff == 0:
        assert res.speedup_over_fixed == 1.0
    st.close()


def test_sweep_with_adaptive_sampling_finds_the_same_best(ls):
    import time
    w = wl.config(3, rows=1024, cols=1024)
    st = ls.Stencil.from_workload(w)
    tin = torch.from_numpy(w.grid()).cuda()
    tout = torch.empty_like(tin)
    sizes = wl.enumerate_wg("pow2")
    t0 = time.perf_counter()
    full = st.sweep(tin, tout, sizes, iters=4, reps=30)
    t_full = time.perf_counter() - t0
    st.set_option(ls.OPT_SWEEP_CUTOFF, 300)
    t0 = time.perf_counter()
    cut = st.sweep(tin, tout, sizes, iters=4, reps=30)
    t_cut = time.perf_counter() - t0
    assert cut.status == full.status
    # the landscape is flat at the top: the adaptive sweep's winner must be as good as the full one's
    # (launches of a few microseconds: means of 30 samples still move by a tenth between sweeps)
    assert full.ms_of(cut.best) <= 1.25 * full.best_ms
    assert cut.best_ms <= 1.25 * full.best_ms
    print("adaptive sweep: %.2f s against %.2f s" % (t_cut, t_full))     # informational: wall clock
    with pytest.raises(ls.StencilError):
        st.set_option(ls.OPT_SWEEP_CUTOFF, 50)


# ---- full-size configurations, in the launch configuration bench.py times ---------------------

def test_c2_full_size(ls):
    w = wl.config(1)
    g = w.grid()
    ref = oracle.apply_workload(w, g)
    for wg, blocking in [((16, 16), (1, 1)), ((4, 64), (4, 4)), ((4, 64), ("direct", 1, 4)), ((16, 8), (2, 4)),
                         ((1, 64), ("stream", 16, 4))]:
        got = gpu_apply(ls, w, g, wg, blocking=blocking)
        assert rel_err(got, ref) <= REL_1


def test_c3_full_size_100_generations(ls):
    w = wl.config(2)
    g = w.grid()
    ref = oracle.apply_workload(w, g)
    got = gpu_apply(ls, w, g, (4, 64), blocking=(2, 16))
    np.testing.assert_array_equal(got, ref)
    got = gpu_apply(ls, w, g, (4, 64), blocking=("direct", 1, 16))
    np.testing.assert_array_equal(got, ref)
    got = gpu_apply(ls, w, g, (8, 16), blocking=("temporal", 4, 16, 4))
    np.testing.assert_array_equal(got, ref)
    got = gpu_apply(ls, w, g, (1, 64), blocking=("stream", 40, 4, 8))         # 100 = 12 launches of 8 + one of 4
    np.testing.assert_array_equal(got, ref)
    got = gpu_apply(ls, w, g, (4, 64), blocking=("stream", 20, 8, 6))
    np.testing.assert_array_equal(got, ref)
    assert 0.02 < got.mean() < 0.2


def test_c4_full_size(ls):
    """All 1000 steps against the oracle, every element, bit for bit (the heat step is a fixed
    sequence of fp32 operations), in the launch configurations bench.py times and one of every
    other kernel family; the 1e-4 bound after iterated runs follows from equality.  The invariants
    (conservation, range) are checked on the same output."""
    w = wl.config(3)
    g = w.grid()
    ref100 = oracle.apply_workload(w, g, iters=100)
    for wg, blocking in [((4, 64), (4, 4)), ((4, 64), ("direct", 1, 4)), ((4, 64), ("temporal", 4, 4, 4)),
                         ((16, 16), ("temporal", 2, 4, 4)), ((2, 64), ("stream", 32, 4, 4)),
                         ((2, 64), ("stream", 38, 4, 8)), ((1, 64), ("stream", 40, 4, 6))]:
        got = gpu_apply(ls, w, g, wg, iters=100, blocking=blocking)
        np.testing.assert_array_equal(got, ref100, err_msg=str(blocking))
    ref = oracle.apply_workload(w, g)                  # the configured run: 1000 steps
    assert w.iters == 1000
    for wg, blocking in [((2, 64), ("stream", 38, 4, 8)), ((1, 128), ("stream", 38, 4, 8)),
                         ((8, 32), ("temporal", 2, 4, 3)), ((4, 16), ("direct", 2, 4)), ((16, 16), (1, 1))]:
        got = gpu_apply(ls, w, g, wg, iters=1000, blocking=blocking)
        np.testing.assert_array_equal(got, ref, err_msg=str(blocking))
        assert rel_err(got, ref) <= REL_N
    s0, s1 = g.astype(np.float64).sum(), got.astype(np.float64).sum()
    assert abs(s1 - s0) / s0 < 1e-6
    assert got.min() >= g.min() and got.max() <= g.max()


def test_c5_full_size_every_cell(ls):
    """8192^2: every cell of the configured run against the oracle's whole-matrix result, for the
    paper's mapping, a register-blocked tile and the marching kernel as bench.py launches it."""
    w = wl.config(4)
    g = w.grid()
    ref = oracle.apply_workload(w, g)
    assert ref.shape == (8192, 8192)
    got = gpu_apply(ls, w, g, (2, 64), blocking=(4, 4))
    err = rel_err(got, ref)
    assert err <= REL_1, err
    got1 = gpu_apply(ls, w, g, (16, 16), blocking=(1, 1))
    np.testing.assert_array_equal(got, got1)
    for h, wg in [(134, (32, 8)), (89, (4, 64)), (64, (1, 64))]:      # the marching kernel, as bench.py launches it
        np.testing.assert_array_equal(got, gpu_apply(ls, w, g, wg, blocking=("stream", h, 4)))


def test_weighted_sums_on_8192_squared_every_cell(ls):
    """The weighted sums bench.py times on 8192^2 - the 28-tap sum with a border region given at run time, the
    7x7 Gaussian - in its launch configurations: every cell against the oracle's whole-matrix result, and the
    streaming mapping bit for bit against a tile with other cells per work-item."""
    import bench
    for name, marches in (("W8192", [(133, (4, 64)), (89, (1, 64))]), ("G7", [(69, (4, 64)), (46, (4, 64))])):
        w = bench.named_workload(wl, name)
        g = w.grid()
        ref = oracle.apply_workload(w, g)
        got = gpu_apply(ls, w, g, (8, 32), blocking=(4, 4))
        err = rel_err(got, ref)
        assert err <= REL_1, (name, err)
        for h, wg in marches:
            np.testing.assert_array_equal(got, gpu_apply(ls, w, g, wg, blocking=("stream", h, 4)))


def test_bench_prints_its_json_line():
    """bench.py on the small configuration: one JSON line with the contract's fields."""
    import json
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--workload", "C1", "--no-others", "--reps", "5",
                          "--steps", "5", "--warmup", "1", "--cpu-seconds", "1", "--no-predictor"], cwd=root,
                         capture_output=True, text=True, timeout=280)
    assert out.returncode == 0, out.stderr[-2000:]
    lines = [l for l in out.stdout.splitlines() if l.strip()]
    assert len(lines) == 1
    rec = json.loads(lines[0])
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
                "vs_baseline", "dtype", "data", "config", "roofline", "cpu_baseline"):
        assert key in rec, key
    assert rec["n_gpus"] == 1 and rec["steps"] == 5 and rec["value"] > 0 and rec["config"]["workload"].startswith("C1")
    assert rec["roofline"]["bound"] == "hbm" and 0 < rec["roofline"]["frac"] < 1 and rec["roofline"]["peak"] == 8000.0
    assert rec["cpu_baseline"]["kind"] == "oracle" and rec["cpu_baseline"]["cores"] >= 1
    assert rec["config"]["matrix_pairs_in_rotation"] > 1


# ---- a matrix whose byte offsets pass 2^32 ------------------------------------------------------

def _window(t, rows, cols, r0, c0, h, w_, margin):
    """Rows r0-margin .. r0+h+margin and columns c0-margin .. c0+w_+margin of the device matrix `t`,
    taken periodically (the workloads here use the wrap border), as a host array."""
    ri = (torch.arange(r0 - margin, r0 + h + margin, device=t.device) % rows)
    ci = (torch.arange(c0 - margin, c0 + w_ + margin, device=t.device) % cols)
    return t.view(rows, cols).index_select(0, ri).index_select(1, ci).cpu().numpy()


def test_matrix_beyond_four_gibibytes(ls):
    """20000 x 60000 fp32 (4.8 GB per matrix): element offsets need more than 32 bits in bytes.  The
    input is drawn on the device from a seeded generator; the oracle recomputes windows at the
    corners, across the periodic edges, around the 2^32-byte line and in the interior, each cut with
    a margin as wide as the applications reach."""
    rows, cols = 20000, 60000
    free, _ = torch.cuda.mem_get_info()
    if free < 3 * rows * cols * 4 + (1 << 30):
        pytest.skip("not enough device memory")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(wl.BASE_SEED + 400)
    tin = torch.rand(rows * cols, generator=gen, device="cuda", dtype=torch.float32) * 100.0
    tout = torch.empty_like(tin)
    line = (1 << 32) // (cols * 4)                                   # the row in which byte offset 2^32 falls
    spots = [(0, 0), (0, cols - 40), (rows - 40, 0), (rows - 40, cols - 40), (line - 20, 30000), (line - 20, cols - 40),
             (9000, 12345), (rows - 40, 29990), (15000, 0)]
    heat = wl.config(3, rows=rows, cols=cols, iters=2)
    runs = [(heat, ("direct", 2, 4), None, (4, 16), 1), (heat, ("stream", 38, 4), 2, (1, 64), 2),
            (heat, ("local", 2, 4), None, (8, 8), 1), (heat, ("temporal", 2, 4), 2, (16, 16), 2)]
    sc = wl.config(4, rows=rows, cols=cols)
    sc.border = "wrap"
    runs.append((sc, ("stream", 134, 4), None, (4, 64), 1))
    for w, mapping, depth, wg, iters in runs:
        st = ls.Stencil.from_workload(w)
        st.set_mapping(*mapping)
        if depth:
            st.set_option(ls.OPT_TEMPORAL_DEPTH, depth)
        tout.fill_(-1.0)
        st.run(tin, tout, iters, wg)
        torch.cuda.synchronize()
        st.close()
        reach = max(w.halo) * iters
        for r0, c0 in spots:
            sub = _window(tin, rows, cols, r0, c0, 40, 40, reach)
            ref = oracle.apply(sub, w.kernel, w.halo, "wrap", w.pad, w.weights, w.scalars, iters)[reach:-reach, reach:-reach]
            got = tout.view(rows, cols)[r0:r0 + 40, c0:c0 + 40].cpu().numpy()
            if w.kernel == wl.HEAT:
                np.testing.assert_array_equal(got, ref, err_msg="%s %s at (%d, %d)" % (w.kernel, mapping, r0, c0))
            else:       # sines and cosines of arguments up to 100 sum to anything, zero included: absolute error
                assert np.max(np.abs(got.astype(np.float64) - ref)) <= 2e-5, (mapping, r0, c0)


def test_largest_matrix_the_library_accepts(ls):
    """rows*cols just under 2^31 (the limit stencil_create states): 32776 x 65520 cells of Life, 2 GiB
    per matrix; windows at the corners, across the periodic edges and in the interior against the
    oracle, for one generation per launch and for fused generations."""
    rows, cols = 32776, 65520
    assert rows * cols < 2 ** 31 <= (rows + 1) * cols                     # 128 cells short of 2^31
    with pytest.raises(ls.StencilError):
        ls.Stencil(rows + 1, cols, "u8", (1, 1, 1, 1), "wrap")            # one row beyond
    free, _ = torch.cuda.mem_get_info()
    if free < 3 * rows * cols + (1 << 30):
        pytest.skip("not enough device memory")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(wl.BASE_SEED + 401)
    tin = (torch.rand(rows * cols, generator=gen, device="cuda", dtype=torch.float32) < 0.3).to(torch.uint8)
    tout = torch.empty_like(tin)
    w = wl.config(2, rows=rows, cols=cols, iters=3)
    spots = [(0, 0), (0, cols - 48), (rows - 48, 0), (rows - 48, cols - 48), (rows - 48, 32000), (16384, 65000), (20000, 100)]
    for mapping, depth, wg in [(("direct", 2, 16), None, (2, 128)), (("stream", 40, 4), 3, (1, 64)),
                               (("stream", 20, 16), 2, (4, 64)), (("temporal", 2, 16), 3, (64, 8)), (("local", 1, 16), None, (16, 4))]:
        st = ls.Stencil.from_workload(w)
        st.set_mapping(*mapping)
        if depth:
            st.set_option(ls.OPT_TEMPORAL_DEPTH, depth)
        tout.fill_(9)
        st.run(tin, tout, w.iters, wg)
        torch.cuda.synchronize()
        st.close()
        for r0, c0 in spots:
            sub = _window(tin, rows, cols, r0, c0, 48, 48, w.iters)
            ref = oracle.apply(sub, w.kernel, w.halo, "wrap", 0.0, None, (), w.iters)[w.iters:-w.iters, w.iters:-w.iters]
            got = tout.view(rows, cols)[r0:r0 + 48, c0:c0 + 48].cpu().numpy()
            np.testing.assert_array_equal(got, ref, err_msg="%s at (%d, %d)" % (mapping, r0, c0))

