// Shared between the translation units of libstencil: tile geometry, kernel arguments, the launchers
// of every kernel family and the templates that register their variants (the scenario handle and
// the registry entry of a compiled kernel variant: scenario.h).  Each variants_*.hip instantiates one group of
// kernels and exports a register function; libstencil.hip assembles the registry and holds the
// C ABI.  (Everything here has internal linkage: each unit gets its own small copy.)
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>
#include <vector>

#include "direct_kernel.h"
#include "stream_kernel.h"
#include "temporal_kernel.h"
#include "life_bits.h"
#include "tile_kernel.h"
#include "march_kernel.h"
#include "march_masked_kernel.h"
#include "life_stream_kernel.h"
#include "pointwise_kernel.h"

#include "scenario.h"

// Runs of several launches on tiles in registers (variants_register_tiles.hip): the applications a launch of a run of so
// many makes, or 0 where the mapping's own kernel makes the run, and the launcher.
int register_tile_per_launch(const stencil *s, int iters, int wg_rows, int wg_cols);
RunLaunchFn register_tile_launcher(int kernel, int border);
LaunchPlan register_tile_plan(const stencil *s, int wg_rows, int wg_cols, int fused);
int register_tile_stores(const stencil *s, const void *out, int wg_rows, int wg_cols, int fused);

// The launcher of the fp32 sums' tile with 2 x 4 cells (variants_weighted_sum_tiles.hip): 5x5, or a run-time region.  And its kernel.
LaunchFn weighted_sum_tile(int border, bool five_by_five);
const void *weighted_sum_tile_kernel(const stencil *s, bool five_by_five);

// Local memory a workgroup may allocate: the device's own figure once a GPU has been used, the
// header's constant before that (defined in libstencil.hip).
int64_t stencil_local_memory_limit();
int stencil_compute_units();

namespace {

// the registry key of a scenario's kernel
int variant_kernel(const stencil *s) {
    if (s->kernel == STENCIL_WEIGHTED_SUM && s->dtype == STENCIL_F64) return STENCIL_WEIGHTED_SUM_F64;
    if (s->kernel == STENCIL_WEIGHTED_SUM && s->dtype == STENCIL_I32) return STENCIL_WEIGHTED_SUM_I32;
    if (s->kernel == STENCIL_WEIGHTED_SUM && s->dtype == STENCIL_U8) return STENCIL_WEIGHTED_SUM_U8;
    return s->kernel;
}

// Words per row of a Life matrix kept as bits.
int64_t life_words(const stencil *s) { return (s->cols + 31) / 32; }
// What the segment heights of stencil_stream_segment_rows are counted in for LIFE: 64 lanes of `cells` cells
// less a rim that covers `depth` generations.
int life_strip_cols(int depth, int cells) { return (64 - 2 * ((depth + cells - 1) / cells)) * cells; }

struct TileGeom {
    int th, tw;        // elements covered by one workgroup
    int pitch;         // LDS pitch in staged elements
    int plane;         // staged elements per LDS plane
    int64_t lds_bytes;
    int tiles_r, tiles_c;
};

TileGeom tile_geom(const stencil *s, const Variant &v, int wr, int wc) {
    TileGeom g;
    g.th = wr * v.cr;
    g.tw = wc * v.cc;
    const int hwa = v.cc == 1 ? s->hw : sk::round_up(s->hw, v.cc);
    const int hea = v.cc == 1 ? s->he : sk::round_up(s->he, v.cc);
    g.pitch = hwa + g.tw + hea;
    g.plane = (g.th + s->hn + s->hs) * g.pitch;
    g.lds_bytes = (int64_t)g.plane * v.staged_bytes;
    if (v.staging == STENCIL_STAGING_DIRECT) {
        g.plane = 0;
        g.lds_bytes = 0;
    } else if (v.staging == STENCIL_STAGING_STREAM) {
        // one wavefront per tile: s->cr rows of a strip of 62..64 vectors; no local memory
        g.th = s->cr;
        g.tw = !v.fuses ? sk::march_vectors(s->hw, s->he) * 4
               : s->kernel == STENCIL_LIFE ? life_strip_cols(s->temporal_depth, v.cc)
                                           : sk::stream_cols(s->temporal_depth);
        g.pitch = 4;
        g.plane = 0;
        g.lds_bytes = 0;
    } else if (v.staging == STENCIL_STAGING_TEMPORAL) {
        // tile + `depth` rows above and below, one vector left and right; two buffers
        g.pitch = g.tw + 2 * v.cc;
        g.plane = (g.th + 2 * s->temporal_depth) * g.pitch;
        g.lds_bytes = 2 * (int64_t)g.plane * v.staged_bytes + 32;   // + one spare vector at each end
    }
    g.tiles_r = (int)((s->rows + g.th - 1) / g.th);
    g.tiles_c = (int)((s->cols + g.tw - 1) / g.tw);
    return g;
}

// How a launch stores its output: as the handle says, but the kernels that make several applications per launch may write it
// through where non-temporal stores are not asked for (Store::kThrough), from half of what the device's L2 caches hold on.
constexpr size_t kThroughBytes = (size_t)16 << 20;
sk::Store store_of(const stencil *s) { return s->nt_store ? sk::Store::kNonTemporal : sk::Store::kPlain; }
static_assert((int)sk::Store::kPlain == STENCIL_STORE_PLAIN && (int)sk::Store::kNonTemporal == STENCIL_STORE_NON_TEMPORAL &&
              (int)sk::Store::kThrough == STENCIL_STORE_THROUGH, "one numbering");
// The temporal kernels and Life in registers (to bytes): up to twice that, where a matrix that was used before is still in the
// last-level cache; life_temporal_kernel from three generations on (its rows of a byte per cell hardly ever start at a cache line,
// and the pieces of lines that meet are written to memory one by one).  Written through / plain, geometric means over 2 to 85 drawn
// launches, matrices used before and fresh ones: temporal_kernel, 16 to 32 MiB 0.89 to 0.94 and 1.00 to 1.02, 32 to 64 MiB 0.98 to
// 1.00 and 1.02 to 1.06, more 1.01 to 1.03 and 1.02 to 1.07; life_temporal_kernel, 16 to 32 MiB, three and four generations 0.90 and
// 1.02, one and two 0.94 and 1.11; life_stream_kernel, 16 to 32 MiB 0.89 and 1.01 (its last launch of a run 0.87 to 0.99 and 0.96
// to 1.00), 32 to 64 MiB 1.01 and 1.01.
sk::Store fused_store(const stencil *s, bool may) {
    const bool through = may && s->out_bytes() >= kThroughBytes && s->out_bytes() < 2 * kThroughBytes;
    return s->nt_store || !through ? store_of(s) : sk::Store::kThrough;
}

// Tiles and direct kernels of a single application, two rows of one vector per work-item, where non-temporal stores are not
// asked for, write their output through: what plain stores leave in the L2 caches is written back when the launch ends, with
// nothing beside it.  From 6 MiB of output on.  But a row of a workgroup, 16 bytes for each of its work-items, that begins or ends
// within a cache line of 128 bytes or within one of its halves leaves pieces, and those are written to memory one by one:
// - Whole lines (by the workgroup's columns, the matrix's and the output's address) at every size.
// - Whole halves up to 32 MiB, where the workgroup has one half a row up to 16.
// - Else, workgroups of 14 columns and more up to 32 MiB, of nine and more up to 16, narrower ones not.
// Written through / plain, 3x3, 5x5 and 28 run-time taps of floats, 8 x 32 work-items where not said, matrices in turn.  Whole lines:
// 1024^2 0.97 to 1.02, 2048^2 0.83 to 0.89 (5x5 10.7 -> 9.1 us), 4096^2 0.97 to 1.01, 8192^2 0.97 to 0.99; of 32 x 8 0.85 to 0.92 up to
// 16 MiB, 0.96 to 1.00 beyond.  Halves: rows of 2032 0.86 to 0.94, 2864 0.91 to 0.98; 64 x 4 0.92 to 0.97 up to 16 MiB (a direct kernel
// 1.07), on 32 and 64 MiB 1.00 to 1.07; 21 x 12 0.87 to 1.01, on 64 MiB 1.00 to 1.02.  Else: 1400 x 1401 0.95 to 1.00, 2000 x 2001 0.86 to
// 0.93, 2900 x 2908 0.94 to 0.99, 4000 x 4001 1.09 to 1.12; on 4096^2 4 bytes further on 1.06, of 25, 27, 29 and 33 columns 1.06 to 1.12;
// 14 to 33 columns on 2048 x 4096 0.92 to 1.04; 9 to 13 on 2048^2 0.87 to 1.06, on 2048 x 4096 0.99 to 1.11; 5 and 7 0.97 to 1.12 and 1.10
// to 1.22; 1 to 3 on 2048^2 0.92 to 1.42, on 8192^2 1.34 to 1.59; 4 in ragged rows 1.10 to 1.31.
// 5x5 doubles on 1000^2 5.9 -> 5.4 us, on 2048^2 13.6 -> 12.8; integers there 12.8 -> 10.9; sin/cos there 12.9 -> 11.5; the
// edge detector's stages on 4096^2, three of which this serves, 88.7 -> 85.2; ten applications in turn on 2048^2 90.3 -> 87.3.
// Each is a kernel compiled once more, 120 of them an eighth of the library, and so only for the work-items that sums and the detector are
// best made with; heat, Life and one, four and eight rows would gain as much (2048^2 0.86 to 0.92, 4096^2 0.96 to 1.02).  9x9 by the
// direct kernel, which runs out of registers, gains nothing (0.98 to 1.02).
template <class Op, int CR, int CC>
constexpr bool may_go_through() {
    using O = typename sk::out_type_of<Op>::type;
    return !sk::goes_through<Op>::value && CR == 2 && CC * sizeof(O) == 16 &&
           (Op::kWeights || std::is_same<Op, sk::OpSobel>::value || std::is_same<Op, sk::OpNms>::value);
}
template <class Op, class Halo, int CR, int CC>
constexpr bool direct_may_go_through() { return may_go_through<Op, CR, CC>() && Halo::N + Halo::S < 8; }
bool tile_goes_through(const stencil *s, const void *out, int wc) {
    const size_t bytes = s->out_bytes(), mib = (size_t)1 << 20;
    if (s->nt_store || bytes < 6 * mib) return false;
    const uintptr_t ends = (uintptr_t)out | (uintptr_t)s->cols * s->out_elem() | (uintptr_t)wc * 16;
    if (ends % 128 == 0) return true;
    return bytes <= (ends % 64 == 0 ? (wc >= 8 ? 32 : 16) : wc >= 14 ? 32 : wc >= 9 ? 16 : 0) * mib;
}
template <bool MAY>
int stores_tile(const stencil *s, const void *out, int, int wc, int) {
    return MAY && tile_goes_through(s, out, wc) ? STENCIL_STORE_THROUGH : (int)store_of(s);
}

// A launch has at most so many work-items; more are turned down.
constexpr int64_t kMaxGridItems = ((int64_t)1 << 32) - 1;

// Blocks of a launch of so many tiles: the workgroups numbered for the eight XCDs, `chunk` to each, or (0) as they come.
int64_t numbered_blocks(const stencil *s, int64_t tiles, int *chunk) {
    *chunk = s->xcd_remap && tiles >= 64 ? (int)((tiles + 7) / 8) : 0;
    return *chunk ? (int64_t)*chunk * 8 : tiles;
}

// Kernel arguments and grid for one launch; `blocks` is the grid size.
template <class Op, class Halo, int CR, int CC>
sk::TileArgs<Op, Halo> make_args(const stencil *s, int staging, const void *in, void *out, int wr, int wc,
                                 unsigned *blocks, size_t *lds_bytes) {
    using T = typename Op::T;
    Variant v{};
    v.staging = staging;
    v.cr = CR;
    v.cc = CC;
    v.staged_bytes = (int)sizeof(typename Op::L) * Op::kPlanes;
    const TileGeom g = tile_geom(s, v, wr, wc);
    sk::TileArgs<Op, Halo> a;
    a.in = static_cast<const T *>(in);
    a.out = static_cast<typename sk::out_type_of<Op>::type *>(out);
    a.rows = (int)s->rows;
    a.cols = (int)s->cols;
    a.tiles_c = g.tiles_c;
    a.n_tiles = g.tiles_r * g.tiles_c;
    a.pitch = g.pitch;
    a.plane = g.plane;
    if (sk::folds_by_rows<Halo>::value && !Halo::kMasked) {
        // the tile kernel stages a region that it folds by rows from its west edge (never more than the geometry allows for)
        a.pitch = sk::round_up(s->hw + g.tw + s->he, CC);
        a.plane = (g.th + s->hn + s->hs) * a.pitch;
    }
    {
        // vectors (elements when CC = 1) per staged row; kernels that stage nothing have none
        const unsigned items = std::max(1u, (unsigned)(a.pitch / CC));
        a.stage_magic = sk::row_magic(items);
    }
    a.store = store_of(s);
    a.pad = (T)s->pad;
    a.scalar0 = s->scalar0;
    if constexpr (Halo::kStatic) {
        if constexpr (Op::kWeights)
            for (int k = 0; k < (int)(sizeof(a.w.v) / sizeof(a.w.v[0])); ++k) a.w.v[k] = (typename decltype(a.w)::W)s->weights[k];
        else
            a.w.v[0] = 0.0f;
    } else {
        a.halo.n_ = s->hn;
        a.halo.s_ = s->hs;
        a.halo.e_ = s->he;
        a.halo.w_ = s->hw;
        a.w.v = static_cast<decltype(a.w.v)>(s->table_in_use);
    }
    *blocks = (unsigned)numbered_blocks(s, a.n_tiles, &a.xcd_chunk);
    *lds_bytes = (size_t)g.lds_bytes;
    return a;
}

// ... and what such a launch starts.
LaunchPlan plan_tiles(const stencil *s, const char *kernel, int staging, int cr, int cc, int staged_bytes, int wr, int wc) {
    Variant v{};
    v.staging = staging;
    v.cr = cr;
    v.cc = cc;
    v.staged_bytes = staged_bytes;
    const TileGeom g = tile_geom(s, v, wr, wc);
    int chunk;
    return {kernel, wr, wc, numbered_blocks(s, (int64_t)g.tiles_r * g.tiles_c, &chunk), g.lds_bytes};
}
template <class Op, class Halo, int CR, int CC>
LaunchPlan plan_tile(const stencil *s, int wr, int wc, int) {
    const char *kernel = sk::folds_by_rows<Halo>::value && Halo::kStatic ? "tile_kernel by rows" : "tile_kernel";
    return plan_tiles(s, kernel, STENCIL_STAGING_LOCAL, CR, CC, (int)sizeof(typename Op::L) * Op::kPlanes, wr, wc);
}
template <class Op, int CR, int CC>
LaunchPlan plan_direct(const stencil *s, int wr, int wc, int) {
    return plan_tiles(s, std::is_same<Op, sk::OpLife>::value ? "life_direct_kernel" : "direct_kernel", STENCIL_STAGING_DIRECT, CR, CC, 0, wr, wc);
}
template <int CR>
LaunchPlan plan_temporal(const stencil *s, int wr, int wc, int) {
    return plan_tiles(s, "temporal_kernel", STENCIL_STAGING_TEMPORAL, CR, 4, 4, wr, wc);
}
// Marches: a wavefront to a segment, workgroups only group wavefronts (blocks before numbering).
LaunchPlan plan_segments(const stencil *s, const char *kernel, int strip_cols, int wr, int wc) {
    const int64_t segments = (s->rows + s->cr - 1) / s->cr * ((s->cols + strip_cols - 1) / strip_cols), waves = wr * wc / 64;
    return {kernel, wr, wc, (segments + waves - 1) / waves, 0};
}

// Tiles above 64 KiB need the kernel's dynamic local-memory limit raised, once per kernel and
// device; `raised_on` remembers the device it was last done on.
hipError_t allow_large_tiles(const void *kernel, size_t lds, int *raised_on) {
    if (lds <= 65536) return hipSuccess;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (*raised_on != dev) {
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)stencil_local_memory_limit());
        if (e != hipSuccess) return e;
        *raised_on = dev;
    }
    return hipSuccess;
}

int stores_temporal(const stencil *s, const void *, int, int, int) { return (int)fused_store(s, true); }
template <class Op, int B, int CR, int MAXT>
hipError_t launch_temporal(const stencil *s, const void *in, void *out, int wr, int wc, int depth,
                           hipStream_t stream) {
    using Halo = sk::HaloC<1, 1, 1, 1>;
    unsigned blocks;
    size_t lds;
    auto a = make_args<Op, Halo, CR, 4>(s, STENCIL_STAGING_TEMPORAL, in, out, wr, wc, &blocks, &lds);
    a.store = fused_store(s, true);
    const bool whole_waves = wr * wc % 64 == 0;
    const auto kernel = whole_waves ? &sk::temporal_kernel<Op, B, true, MAXT> : &sk::temporal_kernel<Op, B, false, MAXT>;
    static thread_local int raised_on[2] = {-1, -1};
    hipError_t e = allow_large_tiles(reinterpret_cast<const void *>(kernel), lds, &raised_on[whole_waves]);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(wc, wr), lds, stream, a, depth, CR);
    return hipGetLastError();
}

// Which launches of a march of several applications have their output written through.
bool stream_goes_through(const stencil *s, int depth) {
    return s->cols % 4 == 0 && depth >= sk::kStreamThroughDepth && !s->nt_store && s->out_bytes() >= kThroughBytes;
}
LaunchPlan plan_stream(const stencil *s, int wr, int wc, int depth) {
    return plan_segments(s, stream_goes_through(s, depth) ? "stream_through_kernel" : "stream_kernel", sk::stream_cols(depth), wr, wc);
}

int stores_stream(const stencil *s, const void *, int, int, int depth) {
    return stream_goes_through(s, depth) ? STENCIL_STORE_THROUGH : (int)store_of(s);
}

template <class Op, int B>
hipError_t launch_stream(const stencil *s, const void *in, void *out, int wr, int wc, int depth, hipStream_t stream) {
    using Halo = sk::HaloC<1, 1, 1, 1>;
    constexpr int kMaxT = 256;
    if (depth < 1 || depth > sk::kStreamMaxDepth) return hipErrorInvalidValue;
    const int CR = s->cr;   // rows per segment
    unsigned blocks;
    size_t lds;
    auto a = make_args<Op, Halo, 0, 4>(s, STENCIL_STAGING_STREAM, in, out, wr, wc, &blocks, &lds);
    // a tile is one wavefront's segment: CR rows of a strip whose width follows from the number of
    // applications this launch fuses (the last launch of a run may fuse fewer)
    const int strip_cols = sk::stream_cols(depth);
    a.tiles_c = (int)((s->cols + strip_cols - 1) / strip_cols);
    a.n_tiles = (int)((s->rows + CR - 1) / CR) * a.tiles_c;
    a.xcd_chunk = 0;
    const unsigned waves_per_block = (unsigned)(wr * wc) / 64u;
    blocks = ((unsigned)a.n_tiles + waves_per_block - 1) / waves_per_block;
    const dim3 grid(blocks), block(wc, wr);
    const bool whole = s->cols % 4 == 0;      // rows of whole vectors, or the element-by-element body
    if (stream_goes_through(s, depth)) {
        static_assert(sk::kStreamThroughDepth == 4 && sk::kStreamMaxDepth == 8, "a case each");
#define THROUGH_LAUNCH(D)                                                                                      \
    hipLaunchKernelGGL((&sk::stream_through_kernel<Op, B, D, kMaxT>), grid, block, 0, stream, a, CR);          \
    return hipGetLastError()
        switch (depth) {
        case 4: THROUGH_LAUNCH(4);
        case 5: THROUGH_LAUNCH(5);
        case 6: THROUGH_LAUNCH(6);
        case 7: THROUGH_LAUNCH(7);
        case 8: THROUGH_LAUNCH(8);
        }
#undef THROUGH_LAUNCH
    }
#define STREAM_LAUNCH(D)                                                                                       \
    hipLaunchKernelGGL(!whole        ? (&sk::stream_kernel<Op, B, D, false, false, kMaxT>)                     \
                       : s->nt_store ? (&sk::stream_kernel<Op, B, D, true, true, kMaxT>)                       \
                                     : (&sk::stream_kernel<Op, B, D, true, false, kMaxT>),                     \
                       grid, block, 0, stream, a, CR);                                                         \
    break
    switch (depth) {
    case 1: STREAM_LAUNCH(1);
    case 2: STREAM_LAUNCH(2);
    case 3: STREAM_LAUNCH(3);
    case 4: STREAM_LAUNCH(4);
    case 5: STREAM_LAUNCH(5);
    case 6: STREAM_LAUNCH(6);
    case 7: STREAM_LAUNCH(7);
    case 8: STREAM_LAUNCH(8);
    default: return hipErrorInvalidValue;
    }
#undef STREAM_LAUNCH
    return hipGetLastError();
}

// What Life runs take, us.  A launch kLifeLaunchUs and kLifeLaunchCellUs a million cells.  A generation kLifeOwnRowUs for every row of
// a work-item, the chain from the rows it is handed to those it hands on, and kLifeWaveUs for every wavefront of a SIMD of the fullest
// compute unit (by border and rows of a work-item, 2 to 16); with up to 256 work-items 10 % more than with 512, with 1024 under WRAP
// 11 %, in groups of 16 lanes 1.5 %.  (From 3395 runs of three and four launches on 30^2 to 80 million cells, 5 to 31 generations per
// launch, every tile and workgroup, and some 40 ways each to make 300 runs on up to 300 million cells: the way taken by these is 1.4 %
// slower than the fastest on average, 5 % for one run of ten.  By a SIMD's rows alone, in workgroups of 512: 240 runs 3.0 % and 11 %; 68
// generations of 4407 x 5557 in six launches 89 us, in three 64; 98 padded ones of 4265 x 5936 in ten 127, in five 99.)
constexpr double kLifeLaunchUs = 3.1, kLifeLaunchCellUs = 0.065, kLifeOwnRowUs = 0.027;
constexpr double kLifeWaveUs[3][4] = {{0.08, 0.088, 0.22, 0.31}, {0.063, 0.078, 0.117, 0.3}, {0.063, 0.097, 0.175, 0.24}};   // STENCIL_CLAMP, ...
constexpr double kLifeLeastUs = 2 * kLifeOwnRowUs + 0.063;        // of the least generation
double life_generation_us(const stencil *s, int64_t tiles, int threads, int rows_per_item, int group_shift) {
    const int units = stencil_compute_units(), kind = rows_per_item == 2 ? 0 : rows_per_item == 4 ? 1 : rows_per_item == 8 ? 2 : 3;
    const double waves = (double)(((tiles + units - 1) / units * (threads / 64) + 3) / 4);       // of a SIMD
    return (kLifeOwnRowUs * rows_per_item + waves * kLifeWaveUs[s->border][kind]) * (group_shift == 4 ? 1.015 : 1.0) *
           (threads <= 256 ? 1.1 : threads > 512 && s->border == STENCIL_WRAP ? 1.11 : 1.0);
}

// The tile of a Life launch (life_stream_kernel.h): rows per work-item and lanes per row.  Two rules:
// - A launch of as many generations as the handle asks for, or fewer, is as much loading and storing as computing, and its
//   tiles come and go: wavefronts are counted over the whole device, one at least, and narrow tiles, which load and store
//   shorter pieces of rows, cost up to a quarter.
//   (us per launch of 8 generations with 256 work-items, rows per item x lanes: 4096 x 4096 4x16 9.8, 8x16 10.3, 8x32 9.8,
//   8x64 11.2, 16x16 11.0, 16x32 10.4, 16x64 11.1; 256 x 256 4x16 4.6, 4x32 4.8, 8x32 6.2, 16x32 8.2.)  A launch that reads
//   bytes has 32 registers per row under way: 16 rows leave room for two wavefronts per SIMD, too few to keep the memory busy
//   (8192 x 8192, one generation: 4x32 25.5, 8x32 23.5, 16x32 27.6).  And a single generation on a matrix that is up to three
//   wavefronts of four-row items per SIMD (the rim aside) is over before eight rows' loads are in (4096 x 4096: 8.0, 9.3, 10.7).
// - A launch of more is a long stay of few tiles: the tile whose generations take least (life_generation_us).
struct LifeTile {
    int threads = 0;
    int rows_per_item = 0, group_shift = 0;
    int tiles_r = 0, tiles_c = 0;
    double us = 0.0;                 // of a generation
};
LifeTile life_tile(const stencil *s, int threads, int depth, bool from_bytes) {
    const bool as_asked = depth <= s->temporal_depth;
    const int rows = (int)s->rows, words = (int)life_words(s), wave_count = threads / 64;
    const double simds = 4.0 * stencil_compute_units();
    const bool few_rows = from_bytes && depth == 1 && (double)rows * words / (4 * 64) <= 3.0 * simds;
    LifeTile best;
    double best_cost = 0.0;
    for (int shift = 4; shift <= 6; ++shift) {
        const int strips = words / ((1 << shift) - 2) + (words % ((1 << shift) - 2) != 0);
        for (int rpt = as_asked ? 4 : 2; rpt <= 16; rpt *= 2) {
            const int held = (threads >> shift) * rpt, step = held - 2 * depth;
            if (step <= 0 || threads > sk::life_stream_max_threads(rpt)) continue;
            if (s->life_rows ? rpt != s->life_rows || 1 << shift != s->life_lanes : few_rows && rpt > 4 && best.tiles_r > 0) continue;
            const int steps = (rows - 1) / step + 1;
            const int tiles = s->border == STENCIL_WRAP ? steps : rows <= held ? 1 : (rows - held - 1) / step + 2;
            if ((int64_t)strips * tiles * threads > kMaxGridItems) continue;
            const double us = life_generation_us(s, (int64_t)strips * tiles, threads, rpt, shift);
            const double cost = !as_asked ? us
                                          : std::max(1.0, (double)strips * steps * wave_count / simds) * (rpt + 2) *
                                                (shift == 4 ? 1.25 : shift == 5 ? 1.05 : 1.0) * (from_bytes && rpt == 16 ? 1.3 : 1.0);
            if (best.tiles_r == 0 || cost < best_cost) {
                best_cost = cost;
                best = {threads, rpt, shift, tiles, strips, us};
            }
        }
    }
    return best;
}

// The tile and the workgroup of a run whose launches make `depth` generations.  If that is more than the handle asks for, and the
// tile is the library's: 256, 512 or 1024 work-items, whichever's tile takes least; the workgroup's own else, or if the matrix has no
// tile for these.  (us a run, 256 / 512 / 1024 work-items, each by its own tile: 100 generations, WRAP, 4096^2 77.3 / 65.5 / 67.0,
// 2048^2 51.0 / 42.2 / 48.9; CLAMP, 4096^2 86.7 / 81.5 / 69.7, 8192 x 2048 88.4 / 81.3 / 69.7; 200 of 512^2 68.4 / 67.8 / 86.9; where
// tiles of 256 with two rows per item do, 15 padded ones of 64 x 1033 6.0 / 7.2 / 9.6, 10 of 657 x 421 5.6 / 6.5 / 8.9.)
LifeTile life_run_tile(const stencil *s, int threads, int depth) {
    LifeTile best;
    for (int own = 256; own <= 1024 && s->life_rows == 0 && depth > s->temporal_depth; own *= 2) {
        const LifeTile t = life_tile(s, own, depth, false);
        if (t.tiles_r > 0 && (best.tiles_r == 0 || t.us < best.us)) best = t;
    }
    return best.tiles_r > 0 ? best : life_tile(s, threads, depth, false);
}

// Generations per launch of a run that takes several launches: a launch costs as much as several generations do
// (kLifeLaunchUs), but every generation fused repeats two more rows of every tile.  At least the number asked for, as far as
// it divides the run into the same launches, and exactly that where the tile is prescribed or nothing is to be fused.  0, the run
// stays with its mapping's kernel: the workgroup is no whole wavefronts, or too small for a tile; or the matrix is so thin that
// its tiles have more work-items than a launch, or that a tile's last columns are beyond the largest int.
int life_per_launch(const stencil *s, int iters, int wr, int wc) {
    const int threads = wr * wc;
    if (threads % 64 != 0 || s->cols > INT32_MAX - 64 * 32) return 0;
    if (s->life_rows != 0 || s->temporal_depth == 1)
        return s->staging == STENCIL_STAGING_STREAM || life_tile(s, threads, s->temporal_depth, false).tiles_r > 0 ? s->temporal_depth : 0;
    const int most = (iters + s->temporal_depth - 1) / s->temporal_depth;
    if (life_run_tile(s, threads, (iters + most - 1) / most).tiles_r == 0) return 0;      // (nor has any with more generations one)
    // from the fewest launches on, so that few more are worth a look
    const double launch_us = kLifeLaunchUs + kLifeLaunchCellUs * 1e-6 * (double)s->rows * (double)s->cols;
    int best = 0;
    double best_us = 0.0;
    for (int launches = std::min(most, (iters + sk::kLifeStreamMaxDepth - 1) / sk::kLifeStreamMaxDepth); launches <= most; ++launches) {
        const int per = (iters + launches - 1) / launches;
        if (best > 0 && launches * (launch_us + per * kLifeLeastUs) > best_us) break;
        if ((iters + per - 1) / per != launches) continue;
        const LifeTile t = life_run_tile(s, threads, per);
        if (t.tiles_r == 0) continue;
        const double us = launches * (launch_us + per * t.us);
        if (best == 0 || us <= best_us) {
            best_us = us;
            best = per;
        }
    }
    return best;
}

// Game of Life, `depth` generations per launch in registers, from and to a matrix of bytes or of bits.
template <int B, bool IN_BITS, bool OUT_BITS>
hipError_t launch_life_stream_formats(const stencil *s, const void *in, void *out, int wr, int wc, int depth,
                                      hipStream_t stream) {
    sk::LifeStreamArgs a;
    a.in = in;
    a.out = out;
    a.rows = (int)s->rows;
    a.cols = (int)s->cols;
    a.words = (int)life_words(s);
    const int threads = wr * wc;
    const LifeTile t = life_tile(s, threads, depth, !IN_BITS);
    if (t.tiles_r == 0) return hipErrorInvalidValue;
    a.group_shift = t.group_shift;
    a.tiles_c = t.tiles_c;
    a.n_tiles = t.tiles_r * t.tiles_c;
    a.pad = s->pad != 0.0;
    a.store = fused_store(s, true);
    const dim3 grid((unsigned)a.n_tiles), block((unsigned)threads);
    const unsigned lds = sk::life_stream_lds(threads);
    switch (t.rows_per_item) {
    case 2: hipLaunchKernelGGL((sk::life_stream_kernel<B, 2, IN_BITS, OUT_BITS>), grid, block, lds, stream, a, depth); break;
    case 4: hipLaunchKernelGGL((sk::life_stream_kernel<B, 4, IN_BITS, OUT_BITS>), grid, block, lds, stream, a, depth); break;
    case 8: hipLaunchKernelGGL((sk::life_stream_kernel<B, 8, IN_BITS, OUT_BITS>), grid, block, lds, stream, a, depth); break;
    default: hipLaunchKernelGGL((sk::life_stream_kernel<B, 16, IN_BITS, OUT_BITS>), grid, block, lds, stream, a, depth); break;
    }
    return hipGetLastError();
}
LaunchPlan plan_life_stream(const stencil *s, int wr, int wc, int depth) {
    const LifeTile t = life_tile(s, wr * wc, depth, true);
    return {"life_stream_kernel", wr, wc, (int64_t)t.tiles_r * t.tiles_c, sk::life_stream_lds(wr * wc)};
}
// (One for all launches of a run, also a last one that makes fewer generations: runs that begin alike are alike.)
void life_run_wg(const stencil *s, int per, int *wr, int *wc) {
    const LifeTile t = life_run_tile(s, *wr * *wc, per);
    if (t.tiles_r > 0 && t.threads != *wr * *wc) *wr = t.threads / 64, *wc = 64;
}
int stores_life_stream(const stencil *s, const void *, int, int, int) { return (int)fused_store(s, true); }
template <int B>
hipError_t launch_life_stream(const stencil *s, const void *in, void *out, int wr, int wc, int depth, hipStream_t stream) {
    if (depth < 1 || depth > STENCIL_MAX_STREAM_DEPTH) return hipErrorInvalidValue;
    return launch_life_stream_formats<B, false, false>(s, in, out, wr, wc, depth, stream);
}
// ... a launch of a run of several, also where the mapping is the local-memory temporal one.
template <int B>
hipError_t launch_life_stream_run(const stencil *s, const void *in, bool in_bits, void *out, bool out_bits, int wr, int wc,
                                  int depth, hipStream_t stream) {
    if (depth < 1 || depth > sk::kLifeStreamMaxDepth) return hipErrorInvalidValue;
    if (in_bits && out_bits) return launch_life_stream_formats<B, true, true>(s, in, out, wr, wc, depth, stream);
    if (in_bits) return launch_life_stream_formats<B, true, false>(s, in, out, wr, wc, depth, stream);
    if (out_bits) return launch_life_stream_formats<B, false, true>(s, in, out, wr, wc, depth, stream);
    return launch_life_stream_formats<B, false, false>(s, in, out, wr, wc, depth, stream);
}

// The threshold stencil: float in, bytes out, no border region (pointwise_kernel.h).
template <int CR, int CC>
hipError_t launch_threshold(const stencil *s, const void *in, void *out, int wr, int wc, int, hipStream_t stream) {
    sk::ThresholdArgs a;
    a.in = static_cast<const float *>(in);
    a.out = static_cast<uint8_t *>(out);
    a.rows = (int)s->rows;
    a.cols = (int)s->cols;
    const int th = wr * CR, tw = wc * CC;
    a.tiles_c = (a.cols + tw - 1) / tw;
    a.n_tiles = ((a.rows + th - 1) / th) * a.tiles_c;
    a.level = s->scalar0;
    const unsigned blocks = (unsigned)numbered_blocks(s, a.n_tiles, &a.xcd_chunk);
    hipLaunchKernelGGL((sk::threshold_kernel<CR, CC, STENCIL_MAX_WG_SIZE>), dim3(blocks), dim3(wc, wr), 0, stream, a);
    return hipGetLastError();
}

template <int CR, int CC>
LaunchPlan plan_threshold(const stencil *s, int wr, int wc, int) {
    return plan_tiles(s, "threshold_kernel", STENCIL_STAGING_DIRECT, CR, CC, 0, wr, wc);
}

template <int B, int CR, int MAXT>
hipError_t launch_life_temporal(const stencil *s, const void *in, void *out, int wr, int wc, int depth,
                                hipStream_t stream) {
    unsigned blocks;
    size_t lds;
    auto a = make_args<sk::OpLife, sk::HaloC<1, 1, 1, 1>, CR, 16>(s, STENCIL_STAGING_TEMPORAL, in, out, wr, wc,
                                                                  &blocks, &lds);
    a.store = fused_store(s, depth >= 3);
    // The kernel keeps the tile as bits, rows of whole words.  (Which sizes are legal still follows from
    // the tile counted in bytes: tile_geom.)
    const unsigned words = (unsigned)(a.pitch + 31) / 32;
    a.pitch = (int)words;
    a.plane = (wr * CR + 2 * s->temporal_depth) * a.pitch;
    a.stage_magic = (unsigned)((0x100000000ull + words - 1) / words);     // (never one word: a vector of cells and the rim)
    lds = 4 * (2 * (size_t)a.plane + 2);         // + one spare word at each end
    hipLaunchKernelGGL((sk::life_temporal_kernel<B, CR, MAXT>), dim3(blocks), dim3(wc, wr), lds, stream, a, depth);
    return hipGetLastError();
}
int stores_life_temporal(const stencil *s, const void *, int, int, int depth) { return (int)fused_store(s, depth >= 3); }
template <int CR>
LaunchPlan plan_life_temporal(const stencil *s, int wr, int wc, int) {
    LaunchPlan p = plan_tiles(s, "life_temporal_kernel", STENCIL_STAGING_TEMPORAL, CR, 16, 1, wr, wc);
    const int64_t words = (wc * 16 + 2 * 16 + 31) / 32;
    p.lds_bytes = 4 * (2 * (wr * CR + 2 * s->temporal_depth) * words + 2);
    return p;
}

// Which fold of the tile kernel serves a run-time region (work-items of several columns of cells).
// - Up to the Gaussian of radius 4 it is compiled for the region's number of columns: straight-line rows against blocks
//   of 8 columns with a shorter last one (2500 x 3000 floats, 2 x 4 cells: 7 x 8 taps 20.8 us compiled, 5 x 13 taps 31.1 in
//   blocks, where tap by tap took 38 either way).
// - Beyond, in blocks; tap by tap where work-items have four rows and more (fold_taps), and for a single row of taps under
//   two rows of cells, where a block's weights are loaded twice (300 x 500 floats, 1 x 41 taps: 6.5 us, 7.3 in blocks).
// - Four rows of cells and more under a region of few taps: tap by tap.  The compiled fold takes the window rows one after
//   the other, and up to 1.5 times the registers (2048 x 4096, tap by tap / compiled: floats, 4 x 4 cells, 1 x 5 taps
//   14.5 / 16.7 us, 3 x 9 taps 20.1 / 18.6; 8 x 4 cells, 1 x 5 taps 16.2 / 18.8, 8 x 5 taps 28.6 / 24.6; doubles on
//   2048^2, 4 x 2 cells, 3 x 5 taps 16.7 / 17.4, 7 x 4 taps 23.6 / 21.0).  Integers spend longer on each tap, bytes longer
//   on staging: there it pays up to a row of the widest regions (int32, 4 x 4 cells, 1 x 5 taps 16.5 / 17.4 us, 3 x 5 taps 21.3 / 20.6).
template <class Op, int CR>
sk::Fold region_fold(const stencil *s) {
    const int rows = s->hn + s->hs + 1, cols = s->he + s->hw + 1;
    constexpr bool kOnePlane = Op::kPlanes == 1;
    if (cols > sk::kCompiledColumns)
        return CR >= (kOnePlane ? 4 : 8) || (kOnePlane && CR == 2 && rows == 1) ? sk::Fold::taps : sk::Fold::blocks;
    constexpr int kFewTaps = !kOnePlane || CR < 4                             ? 0
                             : !std::is_floating_point<typename Op::T>::value ? 9
                             : CR >= 8                                        ? 27
                                                                              : 18;
    return rows * cols <= kFewTaps ? sk::Fold::taps : sk::Fold::columns;
}

// Which compile-time regions the tile folds row by row: the Gaussians of radius 3 and 4 with two and four rows of cells, whose
// unrolled folds are bound by the wavefronts their registers leave (7x7, 2 x 4 cells: 81 registers against 48; 9x9, 4 x 4:
// scratch memory).  (Unrolled / by rows, us: 7x7 on 8192^2 148 / 119, on 3001 x 4099 32.3 / 26.2, four rows of cells there 33.5 /
// 30.1; 9x9 on 8192^2 170 / 162, four rows 218 / 158.  5x5 on 3001 x 4099 22.4 / 22.9, on 2048^2 10.15 / 10.45: unrolled.)
template <class Op, class Halo, int CR, int CC>
constexpr bool by_rows() {
    return std::is_same<Op, sk::OpWeightedSum>::value && Halo::kStatic && Halo::N + Halo::S >= 6 && Halo::E + Halo::W >= 6 && CC > 1 &&
           (CR == 2 || CR == 4);
}
// ... and where it unrolls them after all.  A workgroup of one row of work-items stages up to five rows for each that it computes,
// from the region's west edge, which starts no vector in memory: unrolled, where that fits the registers (7x7 on 3001 x 4099,
// 1 x 64 work-items, 40.1 / 41.8 us).  And where hardly a SIMD has a second wavefront, registers cost nothing and the rows' round
// trips to local memory are all there is (unrolled / by rows, us: 7x7 on 118 x 42, 16 x 8 work-items, 5.1 / 5.5; four rows on
// 512 x 960, 8 x 8, 6.9 / 8.4; 9x9 on 160 x 950, 18 x 14, 5.4 / 6.4; four rows on 336 x 869, 4 x 64, 9.7 / 11.4; two to four
// wavefronts per SIMD, 9x9 on 752 x 1296, 8 x 32: 10.4 / 8.6).
template <class Halo>
constexpr bool may_unroll() { return Halo::kStatic && sk::folds_by_rows<Halo>::value && Halo::N + Halo::S <= 8; }
template <class Halo, int CR, int CC>
bool unrolls(const stencil *s, int wr, int wc) {
    if (wr == 1 && Halo::N + Halo::S <= (CR == 2 ? 8 : 6)) return true;
    const int64_t tiles = ((s->rows + wr * CR - 1) / (wr * CR)) * ((s->cols + wc * CC - 1) / (wc * CC));
    const int units = stencil_compute_units();
    return (tiles + units - 1) / units * ((wr * wc + 63) / 64) <= 6;
}

template <class Op, int B, class Halo, int CR, int CC, int MAXT>
hipError_t start_tile(const stencil *s, const void *in, void *out, int wr, int wc, hipStream_t stream) {
    unsigned blocks;
    size_t lds;
    const auto a = make_args<Op, Halo, CR, CC>(s, STENCIL_STAGING_LOCAL, in, out, wr, wc, &blocks, &lds);
    static thread_local int raised_on = -1;
    hipError_t e = allow_large_tiles(reinterpret_cast<const void *>(&sk::tile_kernel<Op, B, Halo, CR, CC, MAXT>),
                                     lds, &raised_on);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((sk::tile_kernel<Op, B, Halo, CR, CC, MAXT>), dim3(blocks), dim3(wc, wr), lds, stream, a);
    return hipGetLastError();
}

template <class Op, int B, class Halo, int CR, int CC, int MAXT>
hipError_t launch_tile(const stencil *s, const void *in, void *out, int wr, int wc, int, hipStream_t stream) {
    if constexpr (std::is_same<Halo, sk::HaloD>::value && CC > 1) {
        const sk::Fold fold = region_fold<Op, CR>(s);
        if (fold == sk::Fold::blocks) return launch_tile<Op, B, sk::HaloBlocks, CR, CC, MAXT>(s, in, out, wr, wc, 0, stream);
        if (fold == sk::Fold::taps) return launch_tile<Op, B, sk::HaloTaps, CR, CC, MAXT>(s, in, out, wr, wc, 0, stream);
    }
    if constexpr (may_unroll<Halo>()) {
        if (unrolls<Halo, CR, CC>(s, wr, wc))
            return launch_tile<Op, B, sk::HaloC<Halo::N, Halo::S, Halo::E, Halo::W>, CR, CC, MAXT>(s, in, out, wr, wc, 0, stream);
    }
    if constexpr (may_go_through<Op, CR, CC>()) {
        if (tile_goes_through(s, out, wc)) return start_tile<sk::WrittenThrough<Op>, B, Halo, CR, CC, MAXT>(s, in, out, wr, wc, stream);
    }
    return start_tile<Op, B, Halo, CR, CC, MAXT>(s, in, out, wr, wc, stream);
}

// ... and what it starts.  (The run-time folds are one kernel as far as a plan goes.)
template <class Op, class Halo, int CR, int CC>
LaunchPlan plan_launch_tile(const stencil *s, int wr, int wc, int) {
    if constexpr (may_unroll<Halo>()) {
        if (unrolls<Halo, CR, CC>(s, wr, wc)) return plan_tile<Op, sk::HaloC<Halo::N, Halo::S, Halo::E, Halo::W>, CR, CC>(s, wr, wc, 1);
    }
    return plan_tile<Op, Halo, CR, CC>(s, wr, wc, 1);
}

// Single applications under the streaming mapping: whether the march makes them, or a tile of 2 x 4 cells and 8 x 32 work-items
// (a march's workgroup only groups wavefronts, and its segment height has no meaning for a tile).  On rows of whole vectors -
// ragged ones it would move element by element - and with segments that suit it the march is ahead (us, march / tile, matrices
// fresh from memory and then in the caches):
// - under regions of up to five rows, two columns and more and up to 30 cells, in segments of up to six rows, up to six wavefronts per
//   SIMD (march / tile, geometric means over 6 to 240 drawn matrices of 2^10 to 2^24 cells, in the caches and fresh: one row 0.84 and
//   0.74, two and three 0.94 and 0.85, four to six 0.97 and 0.93; with ten wavefronts and more 1.06 to 1.40 and 1.15 to 1.42.  5x5 on
//   1024^2 5.1 / 5.0 and 5.3 / 6.7 us, on 2048^2 7.6 / 8.3 and 9.7 / 11.8).  A taller segment is a chain of as many rows, which fewer
//   wavefronts cover: seven to twelve rows 1.25 to 1.39 and 1.04 to 1.28 below a wavefront per SIMD, 0.95 to 1.07 and 1.00 to 1.10 with
//   more; 13 to 24 1.03 to 1.86 and 0.99 to 1.78; 25 and more up to 6.8.  Nor does it pay with more cells (5 x 9 on 2048^2 11.5 / 10.1
//   and 13.1 / 13.2) or in one column (S1 there 5.5 / 5.5 and 8.3 / 7.3).
// - with the sine and cosine of every cell, taken once, from 2^24 cells on: 4096^2 34.5 / 37.2 and 28.7 / 31.6, 5000^2 47.9 / 51.3
//   and 39.8 / 46.5, 8192^2 117 / 131; 2800^2 20.0 / 18.7 and 18.2 / 16.3.
// - under run-time regions of 72 cells and more on matrices that no cache holds, where it is as fast: N5 S4 E4 W3 on 8192^2 170 /
//   170, N4 S4 E3 W4 158 / 160, N3 S4 E4 W4 165 / 152.
// Under taller regions the tile is: N1 S5 E3 W0 on 2048^2 12.1 / 12.5 and 10.9 / 9.1, on 8192^2 111 / 101; 7x7 there 127 / 125, 9x9
// 192 / 170, 11x11 372 / 240.
constexpr int64_t kSinCosMarchCells = (int64_t)1 << 24, kMarchCells = (int64_t)1 << 25;
bool march_pays(const stencil *s) {
    if (s->cols % 4 != 0) return false;
    const int64_t cells = s->rows * s->cols;
    if (s->kernel == STENCIL_SINCOS) return cells >= kSinCosMarchCells;
    const int taps = (s->hn + s->hs + 1) * (s->he + s->hw + 1);
    if (s->hn <= 2 && s->hs <= 2) {
        const int strip_cols = sk::march_vectors(s->hw, s->he) * 4;
        const int64_t waves = (s->cols + strip_cols - 1) / strip_cols * ((s->rows + s->cr - 1) / s->cr);
        return s->he + s->hw >= 1 && taps <= 30 && s->cr <= 6 && waves <= 6 * 4 * (int64_t)stencil_compute_units();
    }
    const bool compiled = s->hn == s->hs && s->hn == s->he && s->hn == s->hw;
    return !compiled && taps >= 72 && cells >= kMarchCells;
}
// Its workgroup: 8 x 32 work-items, and 256 x 1 where a matrix is so thin that those would be more than a launch has (from
// 2^28 rows on).
struct StreamTile {
    int rows, cols;
};
StreamTile stream_tile(const stencil *s) {
    const int64_t tiles = ((s->rows + 15) / 16) * ((s->cols + 127) / 128);
    return (tiles + 8) * 256 > kMaxGridItems ? StreamTile{256, 1} : StreamTile{8, 32};
}

// The region as that tile folds it.
template <class Op, class Halo>
using StreamTileHalo = typename std::conditional<by_rows<Op, Halo, 2, 4>(), sk::HaloRows<Halo::N, Halo::S, Halo::E, Halo::W>, Halo>::type;

// The marches that the rule can choose (and so the compiled ones): of the compile-time regions sin/cos and 5x5 ...
template <class Op, class Halo>
constexpr bool marched() { return std::is_same<Op, sk::OpSinCos>::value || Halo::N == 2; }
// ... of the run-time ones, by the kernel's largest region, two to nine columns of up to five rows and seven to nine of more.
template <class Halo>
constexpr bool marched_columns(int columns) { return Halo::N == 2 ? columns >= 2 : columns * (Halo::N + Halo::S + 1) >= 72; }

// One application, marched down the matrix in registers (march_kernel.h).
template <class Op, int B, class Halo>
hipError_t launch_march(const stencil *s, const void *in, void *out, int wr, int wc, int, hipStream_t stream) {
    constexpr int kMaxT = 256;
    if constexpr (marched<Op, Halo>()) {
        if (march_pays(s)) {
            unsigned blocks;
            size_t lds;
            auto a = make_args<Op, Halo, 0, 4>(s, STENCIL_STAGING_STREAM, in, out, wr, wc, &blocks, &lds);
            // a tile is a wavefront's segment; workgroups only group wavefronts
            const unsigned waves_per_block = (unsigned)(wr * wc) / 64u;
            blocks = (unsigned)numbered_blocks(s, ((unsigned)a.n_tiles + waves_per_block - 1) / waves_per_block, &a.xcd_chunk);
            // with either kind of store
            hipLaunchKernelGGL(s->nt_store ? (&sk::march_kernel<Op, B, Halo, true, kMaxT>)
                                           : (&sk::march_kernel<Op, B, Halo, false, kMaxT>),
                               dim3(blocks), dim3(wc, wr), 0, stream, a, s->cr);
            return hipGetLastError();
        }
    }
    const StreamTile t = stream_tile(s);
    if constexpr (Halo::N == 2)
        return weighted_sum_tile(B, true)(s, in, out, t.rows, t.cols, 1, stream);
    else
        return launch_tile<Op, B, StreamTileHalo<Op, Halo>, 2, 4, STENCIL_MAX_WG_SIZE>(s, in, out, t.rows, t.cols, 1, stream);
}

template <class Op, class Halo>
LaunchPlan plan_march(const stencil *s, int wr, int wc, int) {
    if (!march_pays(s)) {
        const StreamTile t = stream_tile(s);
        if constexpr (Halo::kMasked) return plan_tile<Op, sk::HaloD, 2, 4>(s, t.rows, t.cols, 1);
        else return plan_launch_tile<Op, StreamTileHalo<Op, Halo>, 2, 4>(s, t.rows, t.cols, 1);
    }
    LaunchPlan p = plan_segments(s, Halo::kMasked ? "march_masked_kernel" : "march_kernel", sk::march_vectors(s->hw, s->he) * 4, wr, wc);
    int chunk;
    p.blocks = numbered_blocks(s, p.blocks, &chunk);
    return p;
}

template <class Op>
int stores_march(const stencil *s, const void *out, int, int, int) {
    if (march_pays(s)) return (int)store_of(s);
    const StreamTile t = stream_tile(s);
    return stores_tile<may_go_through<Op, 2, 4>()>(s, out, t.rows, t.cols, 1);
}

// The same for any region within the kernel's largest one (march_masked_kernel.h): the kernel compiled for the
// region's number of columns.
template <class Op, int B, class Halo, int WC = 1>
hipError_t launch_march_masked(const stencil *s, const void *in, void *out, int wr, int wc, int, hipStream_t stream) {
    constexpr int kMaxT = 256;
    if constexpr (WC > Halo::E + Halo::W + 1) {
        return hipErrorInvalidValue;
    } else {
        if (!march_pays(s)) {
            const StreamTile t = stream_tile(s);
            return weighted_sum_tile(B, false)(s, in, out, t.rows, t.cols, 1, stream);
        }
        if (s->he + s->hw + 1 != WC) return launch_march_masked<Op, B, Halo, WC + 1>(s, in, out, wr, wc, 0, stream);
        if (s->hn > Halo::N || s->hs > Halo::S || s->he > Halo::E || s->hw > Halo::W) return hipErrorInvalidValue;
        if constexpr (!marched_columns<Halo>(WC)) {
            return hipErrorInvalidValue;
        } else {
            unsigned blocks;
            size_t lds;
            auto a = make_args<Op, Halo, 0, 4>(s, STENCIL_STAGING_STREAM, in, out, wr, wc, &blocks, &lds);
            const unsigned waves_per_block = (unsigned)(wr * wc) / 64u;
            blocks = (unsigned)numbered_blocks(s, ((unsigned)a.n_tiles + waves_per_block - 1) / waves_per_block, &a.xcd_chunk);
            hipLaunchKernelGGL(s->nt_store ? (&sk::march_masked_kernel<Op, B, Halo, WC, true, kMaxT>)
                                           : (&sk::march_masked_kernel<Op, B, Halo, WC, false, kMaxT>),
                               dim3(blocks), dim3(wc, wr), 0, stream, a, s->cr);
            return hipGetLastError();
        }
    }
}

template <class Op, int B, class Halo, int CR, int CC, int MAXT>
hipError_t launch_direct(const stencil *s, const void *in, void *out, int wr, int wc, int, hipStream_t stream) {
    if constexpr (direct_may_go_through<Op, Halo, CR, CC>()) {
        if (tile_goes_through(s, out, wc)) return launch_direct<sk::WrittenThrough<Op>, B, Halo, CR, CC, MAXT>(s, in, out, wr, wc, 0, stream);
    }
    unsigned blocks;
    size_t lds;
    const auto a = make_args<Op, Halo, CR, CC>(s, STENCIL_STAGING_DIRECT, in, out, wr, wc, &blocks, &lds);
    hipLaunchKernelGGL((sk::direct_kernel<Op, B, Halo, CR, CC, MAXT>), dim3(blocks), dim3(wc, wr), 0, stream, a);
    return hipGetLastError();
}

template <int B, int CR, int MAXT>
hipError_t launch_life_direct(const stencil *s, const void *in, void *out, int wr, int wc, int, hipStream_t stream) {
    unsigned blocks;
    size_t lds;
    const auto a = make_args<sk::OpLife, sk::HaloC<1, 1, 1, 1>, CR, 16>(s, STENCIL_STAGING_DIRECT, in, out, wr, wc,
                                                                        &blocks, &lds);
    hipLaunchKernelGGL((sk::life_direct_kernel<B, CR, MAXT>), dim3(blocks), dim3(wc, wr), 0, stream, a);
    return hipGetLastError();
}


// The kernel behind each launcher (the variant for rows of whole vectors and plain stores where there are several).
template <class Op, int B, class Halo, int CR, int CC, int MAXT>
const void *kernel_tile(const stencil *s) {
    if constexpr (std::is_same<Halo, sk::HaloD>::value && CC > 1) {
        const sk::Fold fold = region_fold<Op, CR>(s);
        if (fold == sk::Fold::blocks) return kernel_tile<Op, B, sk::HaloBlocks, CR, CC, MAXT>(s);
        if (fold == sk::Fold::taps) return kernel_tile<Op, B, sk::HaloTaps, CR, CC, MAXT>(s);
    }
    return reinterpret_cast<const void *>(&sk::tile_kernel<Op, B, Halo, CR, CC, MAXT>);
}
template <class Op, int B, class Halo, int CR, int CC, int MAXT>
const void *kernel_direct(const stencil *) { return reinterpret_cast<const void *>(&sk::direct_kernel<Op, B, Halo, CR, CC, MAXT>); }
template <int B, int CR, int MAXT>
const void *kernel_life_direct(const stencil *) { return reinterpret_cast<const void *>(&sk::life_direct_kernel<B, CR, MAXT>); }
template <class Op, int B, int MAXT>
const void *kernel_temporal(const stencil *) { return reinterpret_cast<const void *>(&sk::temporal_kernel<Op, B, true, MAXT>); }
template <int B, int CR, int MAXT>
const void *kernel_life_temporal(const stencil *) { return reinterpret_cast<const void *>(&sk::life_temporal_kernel<B, CR, MAXT>); }
template <int CR, int CC>
const void *kernel_threshold(const stencil *) { return reinterpret_cast<const void *>(&sk::threshold_kernel<CR, CC, STENCIL_MAX_WG_SIZE>); }
template <class Op, int B, class Halo>
const void *kernel_march(const stencil *s) {
    if constexpr (marched<Op, Halo>()) {
        if (march_pays(s)) return reinterpret_cast<const void *>(&sk::march_kernel<Op, B, Halo, false, 256>);
    }
    if constexpr (Halo::N == 2) return weighted_sum_tile_kernel(s, true);
    else return kernel_tile<Op, B, StreamTileHalo<Op, Halo>, 2, 4, STENCIL_MAX_WG_SIZE>(s);
}
template <class Op, int B, class Halo, int WC = 1>
const void *kernel_march_masked(const stencil *s) {
    if (!march_pays(s)) return weighted_sum_tile_kernel(s, false);
    if constexpr (WC > Halo::E + Halo::W + 1)
        return nullptr;
    else if (s->he + s->hw + 1 != WC)
        return kernel_march_masked<Op, B, Halo, WC + 1>(s);
    else if constexpr (marched_columns<Halo>(WC))
        return reinterpret_cast<const void *>(&sk::march_masked_kernel<Op, B, Halo, WC, false, 256>);
    else
        return nullptr;
}
template <class Op, int B>
const void *kernel_stream(const stencil *s) {
    switch (s->temporal_depth) {
    case 1: return reinterpret_cast<const void *>(&sk::stream_kernel<Op, B, 1, true, false, 256>);
    case 2: return reinterpret_cast<const void *>(&sk::stream_kernel<Op, B, 2, true, false, 256>);
    case 3: return reinterpret_cast<const void *>(&sk::stream_kernel<Op, B, 3, true, false, 256>);
    case 4: return reinterpret_cast<const void *>(&sk::stream_kernel<Op, B, 4, true, false, 256>);
    case 5: return reinterpret_cast<const void *>(&sk::stream_kernel<Op, B, 5, true, false, 256>);
    case 6: return reinterpret_cast<const void *>(&sk::stream_kernel<Op, B, 6, true, false, 256>);
    case 7: return reinterpret_cast<const void *>(&sk::stream_kernel<Op, B, 7, true, false, 256>);
    case 8: return reinterpret_cast<const void *>(&sk::stream_kernel<Op, B, 8, true, false, 256>);
    default: return nullptr;
    }
}
template <int B>
const void *kernel_life_stream(const stencil *) { return reinterpret_cast<const void *>(&sk::life_stream_kernel<B, 16, false, false>); }

// Per-kernel workgroup-size limit (Section 3.1: the registers a kernel needs bound its
// maximum workgroup size).  The heavily blocked variants are compiled for 256 work-items so
// that their register windows stay out of scratch memory.
template <class Op, int CR, int CC>
constexpr int variant_max_threads() {
    if (std::is_same<Op, sk::OpSinCos>::value && CR * CC >= 32) return 256;
    if (std::is_same<Op, sk::OpLife>::value && CR * CC >= 64) return 256;
    if (std::is_same<Op, sk::OpWeightedSumU8>::value && CR * CC >= 32) return 256;
    return STENCIL_MAX_WG_SIZE;
}

template <class Op, int KID, int B, class Halo, int CR, int CC>
void reg_one(std::vector<Variant> &r) {
    Variant v;
    v.staging = STENCIL_STAGING_LOCAL;
    v.kernel = KID;
    v.border = B;
    if (Halo::kStatic) {
        v.hn = Halo::N; v.hs = Halo::S; v.he = Halo::E; v.hw = Halo::W;
    } else {
        v.hn = v.hs = v.he = v.hw = -1;
    }
    v.cr = CR;
    v.cc = CC;
    constexpr int kMaxT = variant_max_threads<Op, CR, CC>();
    v.max_threads = kMaxT;
    v.staged_bytes = (int)sizeof(typename Op::L) * Op::kPlanes;
    using Folded = typename std::conditional<by_rows<Op, Halo, CR, CC>(), sk::HaloRows<Halo::N, Halo::S, Halo::E, Halo::W>, Halo>::type;
    v.launch = &launch_tile<Op, B, Folded, CR, CC, kMaxT>;
    v.plan = &plan_launch_tile<Op, Folded, CR, CC>;
    v.stores = &stores_tile<may_go_through<Op, CR, CC>()>;
    v.kernel_of = &kernel_tile<Op, B, Folded, CR, CC, kMaxT>;
    r.push_back(v);
}

template <class Op, int KID, int B, class Halo, int CR, int CC>
void reg_direct_one(std::vector<Variant> &r) {
    Variant v;
    v.staging = STENCIL_STAGING_DIRECT;
    v.kernel = KID;
    v.border = B;
    v.hn = Halo::N; v.hs = Halo::S; v.he = Halo::E; v.hw = Halo::W;
    v.cr = CR;
    v.cc = CC;
    v.max_threads = STENCIL_MAX_WG_SIZE;
    v.staged_bytes = 0;
    v.launch = &launch_direct<Op, B, Halo, CR, CC, STENCIL_MAX_WG_SIZE>;
    v.plan = &plan_direct<Op, CR, CC>;
    v.stores = &stores_tile<direct_may_go_through<Op, Halo, CR, CC>()>;
    v.kernel_of = &kernel_direct<Op, B, Halo, CR, CC, STENCIL_MAX_WG_SIZE>;
    r.push_back(v);
}

template <class Op, int KID, class Halo, int CC>
void reg_direct(std::vector<Variant> &r) {
    reg_direct_one<Op, KID, sk::kClamp, Halo, 1, CC>(r);
    reg_direct_one<Op, KID, sk::kWrap, Halo, 1, CC>(r);
    reg_direct_one<Op, KID, sk::kConstant, Halo, 1, CC>(r);
    reg_direct_one<Op, KID, sk::kClamp, Halo, 2, CC>(r);
    reg_direct_one<Op, KID, sk::kWrap, Halo, 2, CC>(r);
    reg_direct_one<Op, KID, sk::kConstant, Halo, 2, CC>(r);
    reg_direct_one<Op, KID, sk::kClamp, Halo, 4, CC>(r);
    reg_direct_one<Op, KID, sk::kWrap, Halo, 4, CC>(r);
    reg_direct_one<Op, KID, sk::kConstant, Halo, 4, CC>(r);
}

template <class Op, int KID, int B, int CR>
void reg_temporal_one(std::vector<Variant> &r) {
    Variant v;
    v.staging = STENCIL_STAGING_TEMPORAL;
    v.kernel = KID;
    v.border = B;
    v.hn = v.hs = v.he = v.hw = 1;
    v.cr = CR;
    v.cc = 4;
    v.max_threads = STENCIL_MAX_WG_SIZE;
    v.staged_bytes = 4;
    v.fuses = true;
    v.launch = &launch_temporal<Op, B, CR, STENCIL_MAX_WG_SIZE>;
    v.plan = &plan_temporal<CR>;
    v.stores = &stores_temporal;
    v.kernel_of = &kernel_temporal<Op, B, STENCIL_MAX_WG_SIZE>;
    v.per_launch = &register_tile_per_launch;
    v.launch_run = register_tile_launcher(KID, B);
    v.plan_run = &register_tile_plan;
    v.stores_run = &register_tile_stores;
    r.push_back(v);
}

template <class Op, int KID, int CR>
void reg_temporal(std::vector<Variant> &r) {
    reg_temporal_one<Op, KID, sk::kClamp, CR>(r);
    reg_temporal_one<Op, KID, sk::kWrap, CR>(r);
    reg_temporal_one<Op, KID, sk::kConstant, CR>(r);
}

template <class Op, int KID, int B>
void reg_stream_one(std::vector<Variant> &r) {
    Variant v;
    v.staging = STENCIL_STAGING_STREAM;
    v.kernel = KID;
    v.border = B;
    v.hn = v.hs = v.he = v.hw = 1;
    v.cr = 0;
    v.cc = 4;
    v.max_threads = 256;
    v.staged_bytes = 0;
    v.fuses = true;
    v.launch = &launch_stream<Op, B>;
    v.plan = &plan_stream;
    v.stores = &stores_stream;
    v.kernel_of = &kernel_stream<Op, B>;
    v.per_launch = &register_tile_per_launch;
    v.launch_run = register_tile_launcher(KID, B);
    v.plan_run = &register_tile_plan;
    v.stores_run = &register_tile_stores;
    r.push_back(v);
}

template <class Op, int KID>
void reg_stream(std::vector<Variant> &r) {
    reg_stream_one<Op, KID, sk::kWrap>(r);
    reg_stream_one<Op, KID, sk::kConstant>(r);
}

template <int B, int CELLS>
void reg_life_stream_one(std::vector<Variant> &r) {
    Variant v;
    v.staging = STENCIL_STAGING_STREAM;
    v.kernel = STENCIL_LIFE;
    v.border = B;
    v.hn = v.hs = v.he = v.hw = 1;
    v.cr = 0;
    v.cc = CELLS;
    v.max_threads = sk::life_stream_max_threads(16);
    v.staged_bytes = 0;
    v.fuses = true;
    v.launch = &launch_life_stream<B>;
    v.plan = &plan_life_stream;
    v.stores = &stores_life_stream;
    v.per_launch = &life_per_launch;
    v.launch_run = &launch_life_stream_run<B>;
    v.run_wg = &life_run_wg;
    v.plan_run = &plan_life_stream;
    v.stores_run = &stores_life_stream;
    v.kernel_of = &kernel_life_stream<B>;
    r.push_back(v);
}

template <int CELLS>
void reg_life_stream(std::vector<Variant> &r) {
    reg_life_stream_one<sk::kWrap, CELLS>(r);
    reg_life_stream_one<sk::kConstant, CELLS>(r);
}

template <int B, int CR, int CC>
void reg_threshold_one(std::vector<Variant> &r) {
    Variant v;
    v.staging = STENCIL_STAGING_LOCAL;     // the paper's mapping; with no border region there is no tile to stage
    v.kernel = STENCIL_THRESHOLD;
    v.border = B;
    v.hn = v.hs = v.he = v.hw = 0;
    v.cr = CR;
    v.cc = CC;
    v.max_threads = STENCIL_MAX_WG_SIZE;
    v.staged_bytes = 0;
    v.launch = &launch_threshold<CR, CC>;
    v.plan = &plan_threshold<CR, CC>;
    v.kernel_of = &kernel_threshold<CR, CC>;
    r.push_back(v);
}

template <int CR, int CC>
void reg_threshold(std::vector<Variant> &r) {
    reg_threshold_one<sk::kClamp, CR, CC>(r);
    reg_threshold_one<sk::kWrap, CR, CC>(r);
    reg_threshold_one<sk::kConstant, CR, CC>(r);
}

template <class Op, int KID, int B, class Halo>
void reg_march_one(std::vector<Variant> &r) {
    Variant v;
    v.staging = STENCIL_STAGING_STREAM;
    v.kernel = KID;
    v.border = B;
    v.hn = Halo::N;
    v.hs = Halo::S;
    v.he = Halo::E;
    v.hw = Halo::W;
    v.cr = 0;
    v.cc = 4;
    v.max_threads = 256;
    v.staged_bytes = 0;
    v.fuses = false;
    v.launch = &launch_march<Op, B, Halo>;
    v.plan = &plan_march<Op, Halo>;
    v.stores = &stores_march<Op>;
    v.kernel_of = &kernel_march<Op, B, Halo>;
    r.push_back(v);
}

template <class Op, int KID, class Halo>
void reg_march(std::vector<Variant> &r) {
    reg_march_one<Op, KID, sk::kClamp, Halo>(r);
    reg_march_one<Op, KID, sk::kWrap, Halo>(r);
    reg_march_one<Op, KID, sk::kConstant, Halo>(r);
}

template <class Op, int KID, int B, class Halo>
void reg_march_masked_one(std::vector<Variant> &r) {
    Variant v;
    v.staging = STENCIL_STAGING_STREAM;
    v.kernel = KID;
    v.border = B;
    v.hn = v.hs = v.he = v.hw = -2;
    v.mn = Halo::N;
    v.ms = Halo::S;
    v.me = Halo::E;
    v.mw = Halo::W;
    v.cr = 0;
    v.cc = 4;
    v.max_threads = 256;
    v.staged_bytes = 0;
    v.fuses = false;
    v.launch = &launch_march_masked<Op, B, Halo>;
    v.plan = &plan_march<Op, Halo>;
    v.stores = &stores_march<Op>;
    v.kernel_of = &kernel_march_masked<Op, B, Halo>;
    r.push_back(v);
}

template <class Op, int KID, class Halo>
void reg_march_masked(std::vector<Variant> &r) {
    reg_march_masked_one<Op, KID, sk::kClamp, Halo>(r);
    reg_march_masked_one<Op, KID, sk::kWrap, Halo>(r);
    reg_march_masked_one<Op, KID, sk::kConstant, Halo>(r);
}

template <int B, int CR>
void reg_life_temporal_one(std::vector<Variant> &r) {
    Variant v;
    v.staging = STENCIL_STAGING_TEMPORAL;
    v.kernel = STENCIL_LIFE;
    v.border = B;
    v.hn = v.hs = v.he = v.hw = 1;
    v.cr = CR;
    v.cc = 16;
    v.max_threads = STENCIL_MAX_WG_SIZE;
    v.staged_bytes = 1;
    v.fuses = true;
    v.plan = &plan_life_temporal<CR>;
    v.stores = &stores_life_temporal;
    v.launch = &launch_life_temporal<B, CR, STENCIL_MAX_WG_SIZE>;
    v.per_launch = &life_per_launch;
    v.launch_run = &launch_life_stream_run<B>;
    v.run_wg = &life_run_wg;
    v.plan_run = &plan_life_stream;
    v.stores_run = &stores_life_stream;
    v.kernel_of = &kernel_life_temporal<B, CR, STENCIL_MAX_WG_SIZE>;
    r.push_back(v);
}

template <int CR>
void reg_life_temporal(std::vector<Variant> &r) {
    reg_life_temporal_one<sk::kClamp, CR>(r);
    reg_life_temporal_one<sk::kWrap, CR>(r);
    reg_life_temporal_one<sk::kConstant, CR>(r);
}

template <int B, int CR>
void reg_life_direct_one(std::vector<Variant> &r) {
    Variant v;
    v.staging = STENCIL_STAGING_DIRECT;
    v.kernel = STENCIL_LIFE;
    v.border = B;
    v.hn = v.hs = v.he = v.hw = 1;
    v.cr = CR;
    v.cc = 16;
    v.max_threads = STENCIL_MAX_WG_SIZE;
    v.staged_bytes = 0;
    v.plan = &plan_direct<sk::OpLife, CR, 16>;
    v.launch = &launch_life_direct<B, CR, STENCIL_MAX_WG_SIZE>;
    v.kernel_of = &kernel_life_direct<B, CR, STENCIL_MAX_WG_SIZE>;
    r.push_back(v);
}

template <int CR>
void reg_life_direct(std::vector<Variant> &r) {
    reg_life_direct_one<sk::kClamp, CR>(r);
    reg_life_direct_one<sk::kWrap, CR>(r);
    reg_life_direct_one<sk::kConstant, CR>(r);
}

template <class Op, int KID, class Halo, int CR, int CC>
void reg_borders(std::vector<Variant> &r) {
    reg_one<Op, KID, sk::kClamp, Halo, CR, CC>(r);
    reg_one<Op, KID, sk::kWrap, Halo, CR, CC>(r);
    reg_one<Op, KID, sk::kConstant, Halo, CR, CC>(r);
}

template <class Op, int KID, class Halo, int CCV>
void reg_blockings(std::vector<Variant> &r) {
    reg_borders<Op, KID, Halo, 1, 1>(r);
    reg_borders<Op, KID, Halo, 2, 1>(r);
    reg_borders<Op, KID, Halo, 4, 1>(r);
    reg_borders<Op, KID, Halo, 8, 1>(r);
    reg_borders<Op, KID, Halo, 1, CCV>(r);
    reg_borders<Op, KID, Halo, 2, CCV>(r);
    reg_borders<Op, KID, Halo, 4, CCV>(r);
    reg_borders<Op, KID, Halo, 8, CCV>(r);
}

}  // namespace

// The groups of variants, one translation unit each.
void register_weighted_sum_tiles(std::vector<Variant> &r);
void register_sincos(std::vector<Variant> &r);
void register_unit_region_tiles(std::vector<Variant> &r);
void register_direct_and_temporal(std::vector<Variant> &r);
void register_streams(std::vector<Variant> &r);
void register_life_streams(std::vector<Variant> &r);
void register_wide_regions(std::vector<Variant> &r);
void register_runtime_march(std::vector<Variant> &r);
