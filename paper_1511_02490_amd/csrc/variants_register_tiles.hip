// Runs of several launches of HEAT and of the 3x3 weighted sum on tiles in registers (register_tile_kernel.h): which tile,
// how many applications per launch, and when.
#include "variants.h"

#include "register_tile_kernel.h"

namespace {

// A launch's tile and workgroup, cut by what a run of launches like it is estimated to take (us; from some 900 runs of 96 and
// 100 heat steps on 256^2 to 4096^2 cells, workgroups of 256, 512 and 1024, 4 to 16 steps per launch, each tile below and ones of eight rows: 11 %
// off on average, and the tile taken 1.4 % slower than the best one; row_us taken again since from nine runs of 96 steps on 8 to 17
// million cells, which it gives within 7 %).  A launch, its loads and its stores: kLaunchUs and kCellUs a million cells.  An
// application: row_us for every row that a SIMD of the fullest compute unit goes through, kWaitUs for the barrier and what hangs on
// it, kOwnRowUs for every row of a work-item.
// (Eight rows per work-item leave room for one workgroup of 1024 on a compute unit, nothing beside its loads and stores: 96
// steps on 4096^2 549 us, by four rows 385.)
constexpr double kLaunchUs = 3.1, kCellUs = 0.8, kWaitUs = 0.25, kOwnRowUs = 0.023;
// heat 0.024 (0.0312 before the tile's cross-lane moves went together), a 3x3 sum 0.0468: by 0.037 its runs take too few of the
// launches that overlap (96 on 3000^2 461 us, 399 by this)
double row_us(const stencil *s) { return s->kernel == STENCIL_HEAT ? 0.024 : 0.0468; }

struct RegisterTile {
    int threads = 0, rows_per_item = 0, group_shift = 0;
    int tiles_r = 0, tiles_c = 0;
    bool small = false;              // the matrix is lower or narrower than the tile
    double simd_rows = 0.0;          // rows of a SIMD of the fullest compute unit
    double us = 0.0;                 // of one launch
};
RegisterTile register_tile(const stencil *s, int depth) {
    const int units = stencil_compute_units(), rows = (int)s->rows, cols = (int)s->cols, rim = sk::register_tile_rim(depth);
    const bool wrap = s->border == STENCIL_WRAP;
    RegisterTile best;
    for (int shift = 4; shift <= 6; ++shift) {
        const int held_c = 4 << shift, step_c = held_c - 8 * rim;
        if (step_c <= 0) continue;
        const int strips = wrap ? (cols - 1) / step_c + 1 : cols <= held_c ? 1 : (cols - held_c - 1) / step_c + 2;
        for (int threads = 256; threads <= sk::kRegisterTileMaxThreads; threads *= 2)
            for (int rpt = 2; rpt <= 4; rpt *= 2) {
                const int held_r = (threads >> shift) * rpt, step_r = held_r - 2 * depth;
                const bool small = !wrap && (rows < held_r || cols < held_c);
                if (step_r <= 0 || (small && rpt > 2)) continue;
                const int tiles = wrap ? (rows - 1) / step_r + 1 : rows <= held_r ? 1 : (rows - held_r - 1) / step_r + 2;
                // (a matrix so thin that a launch cannot have the tiles' work-items, or that its last tile ends beyond the
                // largest int)
                if ((int64_t)strips * tiles * threads > kMaxGridItems || rows > INT32_MAX - held_r || cols > INT32_MAX - held_c) continue;
                const double simd_rows = (double)(((int64_t)strips * tiles + units - 1) / units) * (threads / 256) * rpt;
                const double us = kLaunchUs + kCellUs * 1e-6 * rows * cols +
                                  depth * (row_us(s) * (shift == 4 ? 1.04 : 1.0) * simd_rows + kWaitUs + kOwnRowUs * rpt);
                if (best.threads == 0 || us < best.us) best = {threads, rpt, shift, tiles, strips, small, simd_rows, us};
            }
    }
    return best;
}

template <class Op, int B>
hipError_t launch_register_tile(const stencil *s, const void *in, bool, void *out, bool, int wr, int wc, int depth,
                                hipStream_t stream) {
    if (depth < 1 || depth > sk::kRegisterTileMaxDepth) return hipErrorInvalidValue;
    const RegisterTile t = register_tile(s, depth);
    if (t.threads == 0) return hipErrorInvalidValue;
    unsigned blocks;
    size_t unused;
    auto a = make_args<Op, sk::HaloC<1, 1, 1, 1>, 0, 4>(s, STENCIL_STAGING_STREAM, in, out, wr, wc, &blocks, &unused);
    a.tiles_c = t.tiles_c;
    // (here at every size: 1001 x 1503 1.21 -> 1.09 us a step, 512^2 0.57 -> 0.55, two steps a launch asked for)
    a.store = (sk::Store)register_tile_stores(s, out, wr, wc, depth);
    a.n_tiles = t.tiles_r * t.tiles_c;
    const dim3 grid((unsigned)a.n_tiles), block((unsigned)t.threads);
    const unsigned lds = sk::register_tile_lds(t.threads);
#define TILE_LAUNCH(RPT, SMALL, PAIRED)                                                                        \
    hipLaunchKernelGGL((sk::register_tile_kernel<Op, B, RPT, SMALL, PAIRED>), grid, block, lds, stream, a, depth, t.group_shift)
    if (t.rows_per_item == 4 && t.simd_rows > 16.0)       // more than one such tile per compute unit
        TILE_LAUNCH(4, false, true);
    else if (t.rows_per_item == 4)
        TILE_LAUNCH(4, false, false);
    else if (t.small)
        TILE_LAUNCH(2, B != sk::kWrap, false);
    else
        TILE_LAUNCH(2, false, false);
#undef TILE_LAUNCH
    return hipGetLastError();
}

template <class Op>
RunLaunchFn launcher_of(int border) {
    return border == STENCIL_CLAMP  ? &launch_register_tile<Op, sk::kClamp>
           : border == STENCIL_WRAP ? &launch_register_tile<Op, sk::kWrap>
                                    : &launch_register_tile<Op, sk::kConstant>;
}

}  // namespace

// What the marching kernel takes for a row and an application of a SIMD's wavefronts, us (runs of eight per launch on 4096^2 and
// 2048 x 8192): heat 0.037 under WRAP, 0.042 where padded cells are set back, a 3x3 sum 0.06.
static double march_row_us(const stencil *s) { return s->kernel != STENCIL_HEAT ? 0.06 : s->border == STENCIL_WRAP ? 0.037 : 0.042; }

// Applications per launch of a run that takes several launches: at least the number asked for, as far as it divides the run
// into the same launches.  0, the run stays with its mapping's kernel: nothing is to be fused; the workgroup is no whole
// wavefronts; or the marching kernel is faster, which fills the device on matrices of ten million cells and more.  Its time:
// every SIMD marches its wavefronts one after the other, march_row_us a row and application, half as much again element by element,
// unless a launch of few applications takes longer to move the matrix, 1.3 us a million cells
// (us a run of 96 heat steps, 8 per launch there, register tiles / march: 2048 x 4096 214 / 247, 3072^2 223 / 254, 4096 x 3072
// 292 / 337, 4096^2 385 / 418, CONSTANT 393 / 472; 4001 x 4003 368 / 560).
int register_tile_per_launch(const stencil *s, int iters, int wr, int wc) {
    const int asked = s->temporal_depth;
    if (wr * wc % 64 != 0 || asked == 1) return 0;
    int best = 0, launches_before = 0;
    double best_us = 0.0;
    for (int d = asked; d <= sk::kRegisterTileMaxDepth; ++d) {
        const int launches = (iters + d - 1) / d;
        if (launches == launches_before) continue;
        launches_before = launches;
        const int per = (iters + launches - 1) / launches;
        const RegisterTile t = register_tile(s, per);
        if (t.threads == 0) break;           // (nor has any with more applications one)
        const double us = launches * t.us;
        if (best == 0 || us < best_us) {
            best_us = us;
            best = per;
        }
    }
    if (best > 0 && s->staging == STENCIL_STAGING_STREAM) {
        const int strip_cols = sk::stream_cols(asked);
        const int64_t waves = (s->cols + strip_cols - 1) / strip_cols * ((s->rows + s->cr - 1) / s->cr), simds = 4 * stencil_compute_units();
        const double rows = (double)((waves + simds - 1) / simds) * (s->cr + 2 * asked);
        const double moved_us = 1.3e-6 * (double)s->rows * (double)s->cols;
        const double marched_us = asked * rows * march_row_us(s) * (s->cols % 4 != 0 ? 1.5 : 1.0);
        const double march_us = (double)iters / asked * (kLaunchUs + std::max(moved_us, marched_us));
        if (march_us <= best_us) return 0;
    }
    return best;
}

LaunchPlan register_tile_plan(const stencil *s, int, int, int depth) {
    const RegisterTile t = register_tile(s, depth);
    return {"register_tile_kernel", 1, t.threads, (int64_t)t.tiles_r * t.tiles_c, sk::register_tile_lds(t.threads)};
}

int register_tile_stores(const stencil *s, const void *, int, int, int) { return s->nt_store ? STENCIL_STORE_NON_TEMPORAL : STENCIL_STORE_THROUGH; }

RunLaunchFn register_tile_launcher(int kernel, int border) {
    return kernel == STENCIL_HEAT ? launcher_of<sk::OpHeat>(border) : launcher_of<sk::OpWeightedSum>(border);
}
