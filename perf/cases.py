"""Timed work of the stencil library: what its users have it do, through the public binding.

A case is one scenario - matrix, element type, border region, border mode, customising function -
with the mapping a user's program would set for it and the number of applications of one run.
`listed()` holds fixed cases, `draw(rng)` makes more of the same ranges, `prepare` builds what a
program has in hand before the call, `run` makes one pass, `work` states what the pass cannot do
without, `tolerance` how far another correct implementation may be off.

The mappings follow what the library advises: nothing set on the smallest matrices, the tile with a
few cells per work-item for a single application, the marching mapping (segment heights from
Stencil.stream_segment_rows) on matrices no cache holds, several applications per launch for
iterated runs, non-temporal stores where the output does not fit a cache.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1511_02490_amd import libstencil as ls
from paper_1511_02490_amd import workloads as wl

TORCH_TYPES = {"f32": torch.float32, "u8": torch.uint8, "i32": torch.int32, "f64": torch.float64}
BYTES = {"f32": 4, "u8": 1, "i32": 4, "f64": 8}
BIG_MATRIX_CELLS = 1 << 25       # 128 MiB of floats: in and out together no longer fit the last-level cache
SMALL_MATRIX_CELLS = 1 << 18     # up to 512 x 512 nobody sets a mapping
MAX_CELLS = 8192 * 8192
MAX_CELL_TAPS = MAX_CELLS * 28   # what the largest single application costs
MAX_CELL_UPDATES = 4096 * 4096 * 400


def _case(kernel, rows, cols, dtype="f32", halo=(1, 1, 1, 1), border="clamp", iters=1):
    """The scenario with the mapping a program would set for it."""
    n, s, e, w = halo
    case = {"kernel": kernel, "rows": rows, "cols": cols, "dtype": dtype, "north": n, "south": s, "east": e, "west": w,
            "border": border, "iters": iters, "staging": "", "cells_rows": 1, "cells_cols": 1, "depth": 0, "slots": 0,
            "wg_rows": 0, "wg_cols": 0, "nt_store": False}
    cells = rows * cols
    if kernel == "canny":
        pass                                     # four handles, each with a mapping of its own: see _canny
    elif iters > 1 and border == "clamp":        # several applications per launch, staged in local memory
        case.update(staging="temporal", depth=4, cells_rows=2, cells_cols=16 if kernel == "life" else 4,
                    wg_rows=64 if kernel == "life" else 32, wg_cols=8 if kernel == "life" else 32)
    elif iters > 1:                              # ... or kept in registers
        case.update(staging="stream", depth=8, cells_cols=8 if kernel == "life" else 4, slots=2, wg_rows=4, wg_cols=64)
    elif cells <= SMALL_MATRIX_CELLS:
        pass
    elif dtype == "f32" and cells >= BIG_MATRIX_CELLS and _marches(kernel, halo):
        case.update(staging="stream", cells_cols=4, slots=3, wg_rows=4, wg_cols=64, nt_store=True)
    else:
        case.update(staging="local", cells_rows=2, cells_cols=2 if dtype == "f64" else 4, wg_rows=8, wg_cols=32,
                    nt_store=cells * BYTES[dtype] >= BIG_MATRIX_CELLS * 4)
    return case


def _marches(kernel, halo):
    n, s, e, w = halo
    if kernel == "sincos":
        return halo == (1, 5, 3, 0)
    return n <= 5 and s <= 5 and e <= 4 and w <= 4 and halo != (1, 1, 1, 1)


def listed():
    return [
        # the smallest call: a 3x3 blur of a small image with nothing set, where launch and host path count
        dict(_case("weighted_sum", 256, 256), name="blur3_256"),
        # an ordinary Gaussian blur of a mid-sized image
        dict(_case("weighted_sum", 2048, 2048, halo=(2, 2, 2, 2)), name="blur5_2048"),
        # a wider blur of an image whose rows are no multiple of anything
        dict(_case("weighted_sum", 3001, 4099, halo=(3, 3, 3, 3)), name="blur7_3001x4099"),
        # Game of Life on a torus, a hundred generations
        dict(_case("life", 4096, 4096, "u8", border="wrap", iters=100), name="life_4096_x100"),
        # ... and on a ragged board with nearest-cell borders
        dict(_case("life", 1001, 1503, "u8", border="clamp", iters=50), name="life_1001x1503_x50"),
        # a simulation of the heat equation on a periodic grid
        dict(_case("heat", 4096, 4096, border="wrap", iters=400), name="heat_4096_x400"),
        # ... and on a ragged grid with insulated (nearest-cell) borders
        dict(_case("heat", 1025, 1999, border="clamp", iters=100), name="heat_1025x1999_x100"),
        # the compute-intensive synthetic stencil on the largest matrix
        dict(_case("sincos", 8192, 8192, halo=(1, 5, 3, 0), border="constant"), name="sincos_8192"),
        # the light synthetic stencil with an asymmetric region given at run time, on the largest matrix
        dict(_case("weighted_sum", 8192, 8192, halo=(1, 5, 3, 0), border="constant"), name="sum28_8192"),
        # the edge detector's four stencils one after the other on an 8-bit image
        dict(_case("canny", 4096, 4096, "u8", halo=(2, 2, 2, 2)), name="canny_4096"),
        # the template's other element types: doubles ...
        dict(_case("weighted_sum", 4096, 4096, "f64", halo=(2, 2, 2, 2)), name="blur5_f64_4096"),
        # ... and integers, with an asymmetric region on a ragged matrix
        dict(_case("weighted_sum", 2500, 3003, "i32", halo=(3, 2, 4, 1), border="wrap"), name="sum36_i32_2500x3003"),
    ]


def draw(rng):
    def side(lo=256, hi=8192):
        v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return v if rng.random() < 0.5 else max(lo, v // 16 * 16)       # half of them ragged

    def limited(cols, limit, rows):
        return max(64, min(rows, limit // cols))

    kind = rng.choice(["blur", "blur", "sum", "sum", "typed", "life", "life", "heat", "heat", "sincos", "canny"])
    border = rng.choice(["clamp", "wrap", "constant"])
    rows, cols = side(), side()
    if kind == "life" or kind == "heat":
        iters = int(round(math.exp(rng.uniform(math.log(10), math.log(400)))))
        rows = limited(cols, MAX_CELL_UPDATES // iters, limited(cols, 4096 * 4096, rows))
        return _case(kind, rows, cols, "u8" if kind == "life" else "f32", border=border, iters=iters)
    if kind == "canny":
        return _case("canny", limited(cols, 4096 * 4096, rows), cols, "u8", halo=(2, 2, 2, 2))
    if kind == "blur":
        radius = rng.choice([1, 2, 2, 3, 4])
        halo, dtype = (radius,) * 4, "f32"
    elif kind == "sincos":
        halo = (1, 5, 3, 0) if rng.random() < 0.5 else tuple(rng.randint(0, 5) for _ in range(4))
        dtype = "f32"
    else:                                        # the synthetic template: any region
        halo = tuple(rng.randint(0, 8 if rng.random() < 0.3 else 4) for _ in range(4))
        dtype = "f32" if kind == "sum" else rng.choice(["f64", "i32"])
    n, s, e, w = halo
    taps = (n + s + 1) * (e + w + 1)
    rows = limited(cols, min(MAX_CELLS * 4 // BYTES[dtype], MAX_CELL_TAPS // taps), rows)
    return _case("sincos" if kind == "sincos" else "weighted_sum", rows, cols, dtype, halo, border)


# ---- inputs --------------------------------------------------------------------------------------

def _weights(case, seed):
    n, s, e, w = case["north"], case["south"], case["east"], case["west"]
    shape = (n + s + 1, e + w + 1)
    rng = np.random.default_rng([seed, 1])
    if case["dtype"] == "i32":
        return rng.integers(-64, 65, size=shape).astype(np.float32)
    if case["kernel"] == "sincos":
        return rng.random(shape, dtype=np.float32)
    if n == s == e == w and n > 0:
        return wl.gaussian_weights(n, 1.0 + rng.random())
    t = rng.random(shape, dtype=np.float32)
    return t / t.sum()


def _matrix(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    shape = (case["rows"], case["cols"])

    def uniform():
        return torch.rand(shape, generator=gen, device="cuda", dtype=TORCH_TYPES[case["dtype"]])

    if case["kernel"] == "life":
        return (torch.rand(shape, generator=gen, device="cuda") < 0.3).to(torch.uint8)
    if case["kernel"] == "heat":                 # a warm plate with hot squares
        u = uniform().mul_(100.0)
        side = min(32, *shape)
        at = np.random.default_rng([seed, 2])
        for _ in range(16):
            r, c = at.integers(0, shape[0] - side + 1), at.integers(0, shape[1] - side + 1)
            u[r:r + side, c:c + side] = 1000.0
        return u
    if case["kernel"] == "sincos":
        return uniform().mul_(2.0).sub_(1.0)
    if case["dtype"] == "u8":                    # an image: broad bright and dark areas, and noise
        y = torch.linspace(0, 40, shape[0], device="cuda").sin_()
        x = torch.linspace(0, 60, shape[1], device="cuda").cos_()
        img = 127.0 + 90.0 * y[:, None] * x[None, :]
        img += torch.rand(shape, generator=gen, device="cuda") * 30.0
        return img.to(torch.uint8)
    if case["dtype"] == "i32":
        return torch.randint(-1000, 1001, shape, generator=gen, device="cuda", dtype=torch.int32)
    return uniform()


def _configure(st, case):
    if case["staging"]:
        rows = case["cells_rows"]
        st.set_mapping(case["staging"], rows, case["cells_cols"])
        if case["depth"]:
            st.set_option(ls.OPT_TEMPORAL_DEPTH, case["depth"])
        if case["slots"]:                        # a segment height that fills the device, but no sliver
            rows = max(16 if case["depth"] else 5, st.stream_segment_rows(case["slots"]))
            st.set_mapping(case["staging"], rows, case["cells_cols"])
    if case["nt_store"]:
        st.set_option(ls.OPT_NT_STORE, 1)
    return st


def _canny(case, img):
    """(handle, input, output, workgroup size) of the detector's stages: blur, sobel, nms, threshold."""
    rows, cols, border = case["rows"], case["cols"], case["border"]

    def empty(dtype):
        return torch.empty((rows, cols), dtype=dtype, device="cuda")

    blur = ls.Stencil(rows, cols, "u8", (2, 2, 2, 2), border)
    blur.set_kernel("weighted_sum", wl.gaussian_weights(2, 1.0))
    blur.set_mapping("local", 2, 4)
    sobel = ls.Stencil(rows, cols, "f32", (1, 1, 1, 1), border)
    sobel.set_kernel("sobel")
    sobel.set_mapping("direct", 2, 4)
    nms = ls.Stencil(rows, cols, "f32", (1, 1, 1, 1), border)
    nms.set_kernel("nms")
    nms.set_mapping("direct", 2, 4)
    threshold = ls.Stencil(rows, cols, "f32", (0, 0, 0, 0), border)
    threshold.set_kernel("threshold", scalars=(24.0,))
    threshold.set_mapping("local", 2, 4)
    smooth, slope, ridge, edges = empty(torch.float32), empty(torch.float32), empty(torch.float32), empty(torch.uint8)
    return [(blur, img, smooth, (8, 32)), (sobel, smooth, slope, (4, 64)), (nms, slope, ridge, (4, 64)),
            (threshold, ridge, edges, (4, 64))]


def prepare(case, seed):
    tin = _matrix(case, seed)
    if case["kernel"] == "canny":
        return {"stages": _canny(case, tin), "iters": 1}
    halo = (case["north"], case["south"], case["east"], case["west"])
    st = ls.Stencil(case["rows"], case["cols"], case["dtype"], halo, case["border"])
    if case["kernel"] in ("weighted_sum", "sincos"):
        st.set_kernel(case["kernel"], _weights(case, seed))
    elif case["kernel"] == "heat":
        st.set_kernel("heat", scalars=(0.2,))
    else:
        st.set_kernel(case["kernel"])
    _configure(st, case)
    return {"stages": [(st, tin, torch.empty_like(tin), (case["wg_rows"], case["wg_cols"]))], "iters": case["iters"]}


def run(state):
    return [st.run(tin, tout, state["iters"], wg) for st, tin, tout, wg in state["stages"]]


# ---- what a pass needs, and how exact it is --------------------------------------------------------

def work(case):
    cells = case["rows"] * case["cols"]
    taps = (case["north"] + case["south"] + 1) * (case["east"] + case["west"] + 1)
    if case["kernel"] == "canny":                # stage by stage: bytes in, bytes out; every stage's output is wanted
        return {"bytes": cells * ((1 + 4) + (4 + 4) + (4 + 4) + (4 + 1)), "flops": cells * (2 * taps - 1 + 17 + 8 + 1)}
    ops = {"weighted_sum": 2 * taps - 1, "sincos": 3 * taps + 1, "heat": 7, "life": 11}[case["kernel"]]
    return {"bytes": 2 * cells * BYTES[case["dtype"]], "flops": cells * ops * case["iters"]}


def tolerance(case):
    """Life and the integer sums are whole numbers; the heat step and the detector's stages are defined operation by
    operation, and where one of the latter decides by a comparison a last bit decides a whole cell.  The other sums:
    about four times the difference between a pass and the same sums in 64 bits (floats: 0.5e-7 to 1.5e-7 over these
    ranges) or in another order (doubles: 2.2e-16)."""
    if case["kernel"] in ("life", "heat", "canny") or case["dtype"] == "i32":
        return "exact"
    return {"rel": 1e-15 if case["dtype"] == "f64" else 6e-7}
