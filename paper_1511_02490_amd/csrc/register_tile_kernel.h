// Iterated stencils with the 1/1/1/1 border region on matrices of floats, many applications per launch on a tile in
// registers: what runs of several launches are made of where the matrix is too small for the marching kernel to fill the
// device (stream_kernel.h) and a launch in local memory (temporal_kernel.h) is mostly staging and launch.
//
// A work-item holds RPT rows of one vector of four cells.  16, 32 or 64 adjacent lanes hold adjacent vectors, the lanes'
// groups rows below each other, and the workgroup so holds a tile.  Per application a row's west and east neighbours
// come from the adjacent lanes by cross-lane moves, and only the first and the last row of every work-item pass through
// local memory, behind one barrier (two buffers in turn); the rows between them are computed before it.  What an application
// computes within k cells of the tile's rim is stale after k applications: `depth` rows above and below and as many cells,
// in whole vectors, left and right are not written.  Bound by vector-ALU issue (24 instructions per vector and application of
// heat, 22 % to 45 % of them for rim cells) where every SIMD has several wavefronts, by the barrier and the launch where it
// has one.  (100 heat steps, us before / now: 1025 x 1999, CLAMP, 4 per launch in local memory 280 / 108; 1001 x 1503, WRAP, 8
// per launch marched element by element 362 / 106; 64^2, WRAP, 2 per launch 285 / 43.)
//
// Borders.  WRAP: a periodic copy evolves like its original.  CLAMP and CONSTANT: the first tile of a row or column of tiles
// begins with the matrix and the last one ends with it, wherever that puts its vectors, so that no cell of a tile lies
// outside, and the neighbours that are missing (a cell itself, or the padding) are found by one selection per row at either
// end of a row of lanes and once per work-item and application above and below.  Only a matrix smaller than a tile has cells
// outside.  The per-cell arithmetic is the same fold as everywhere else: results are bit-identical to `depth` single launches.
#pragma once
#include "temporal_kernel.h"

namespace sk {

constexpr int kRegisterTileMaxDepth = 16;
constexpr int register_tile_rim(int depth) { return (depth + 3) / 4; }        // lanes per side
constexpr int kRegisterTileMaxThreads = 1024;
constexpr unsigned register_tile_lds(int threads) { return 4 * (unsigned)threads * 4 * (unsigned)sizeof(float); }

// SMALL: the matrix is lower or narrower than a tile (a kernel of its own: its registers would cost the others wavefronts).
// PAIRED: two applications per pass of the loop, which saves the moves between the two (a twelfth of the instructions)
// and costs a launch of few wavefronts the time to fetch the longer loop, some 1 us.
template <class Op, int B, int RPT, bool SMALL, bool PAIRED>
__global__ __launch_bounds__(kRegisterTileMaxThreads) void register_tile_kernel(
    const TileArgs<Op, HaloC<1, 1, 1, 1>> a, const int depth, const int group_shift) {
    static_assert(Op::kPlanes == 1 && sizeof(typename Op::T) == 4 && sizeof(typename Op::L) == 4, "fp32, one plane");
    constexpr int CC = 4;
    const int tid = (int)threadIdx.y * (int)blockDim.x + (int)threadIdx.x, nthreads = (int)(blockDim.x * blockDim.y);
    const int G = 1 << group_shift, groups = nthreads >> group_shift, lane = tid & (G - 1);
    const int rim = register_tile_rim(depth), rows = a.rows, cols = a.cols;
    const int tile_r = (int)blockIdx.x / a.tiles_c, tile_c = (int)blockIdx.x - tile_r * a.tiles_c;
    // rows and columns of the tile; how far it is from one tile to the next
    const int held_r = groups * RPT, step_r = held_r - 2 * depth, held_c = G * CC, step_c = held_c - 2 * rim * CC;
    // the first row and column it holds, and those that it writes
    int top, left, begin_r, end_r, begin_c, end_c;
    if (B == kWrap) {
        begin_r = tile_r * step_r, begin_c = tile_c * step_c;
        top = begin_r - depth, left = begin_c - rim * CC;
        end_r = min(rows, begin_r + step_r), end_c = min(cols, begin_c + step_c);
    } else {
        top = max(0, min(tile_r * step_r, rows - held_r));
        left = max(0, min(tile_c * step_c, cols - held_c));
        begin_r = tile_r == 0 ? 0 : tile_r * step_r + depth;
        begin_c = tile_c == 0 ? 0 : tile_c * step_c + rim * CC;
        end_r = tile_r * step_r + held_r >= rows ? rows : (tile_r + 1) * step_r + depth;
        end_c = tile_c * step_c + held_c >= cols ? cols : (tile_c + 1) * step_c + rim * CC;
    }
    const int row0 = top + (tid >> group_shift) * RPT, gc0 = left + lane * CC;     // the work-item's first row and column

    // does the tile lie at an edge of the matrix?  (the same for the whole workgroup)
    const bool edge = SMALL || top == 0 || left == 0 || top + held_r == rows || left + held_c == cols;
    extern __shared__ __align__(16) unsigned char lds_raw[];      // two buffers of the work-items' first and last rows
    float *const first_rows = reinterpret_cast<float *>(lds_raw), *const last_rows = first_rows + CC * nthreads;
    const int above_at = max(0, tid - G) * CC, below_at = min(tid + G, nthreads - 1) * CC;
    const bool no_above = row0 == 0, no_below = row0 + RPT == rows, no_west = gc0 == 0, no_east = gc0 + CC == cols;
    // (loads and stores within either branch: merged behind the two loops the tile would be kept in registers twice)
    auto applications = [&](auto EDGE) {
        constexpr bool kEdge = decltype(EDGE)::value;
        // Loads, all in flight together: vectors at any address; a lane whose cells are not all in the matrix takes them
        // one by one (any cells where there is none).
        float x[RPT][CC];
        {
            const bool whole = gc0 >= 0 && gc0 + CC <= cols;
            int gr = B == kWrap ? resolve<kWrap>(row0, rows) : min(row0, rows - 1);
            if (whole) {
#pragma unroll
                for (int i = 0; i < RPT; ++i) {
                    load_global(x[i], a.in + (size_t)gr * cols + gc0);
                    gr = gr + 1 == rows ? (B == kWrap ? 0 : gr) : gr + 1;
                }
            } else {
                int col[CC];
#pragma unroll
                for (int j = 0; j < CC; ++j) col[j] = resolve<B == kConstant ? kClamp : B>(gc0 + j, cols);
#pragma unroll
                for (int i = 0; i < RPT; ++i) {
                    const float *row = a.in + (size_t)gr * cols;
#pragma unroll
                    for (int j = 0; j < CC; ++j) x[i][j] = row[col[j]];
                    gr = gr + 1 == rows ? (B == kWrap ? 0 : gr) : gr + 1;
                }
            }
        }
        // SMALL, CONSTANT: cells that are not matrix cells hold the padding
        auto pad_outside = [&](float (&v)[CC], int i) {
#pragma unroll
            for (int j = 0; j < CC; ++j) v[j] = row0 + i >= rows || gc0 + j >= cols ? a.pad : v[j];
        };
        if (B == kConstant && SMALL) {
#pragma unroll
            for (int i = 0; i < RPT; ++i) pad_outside(x[i], i);
        }

        struct Ends { float w, e; };
        auto ends_of = [&](const float (&v)[CC]) {
            return Ends{__uint_as_float(from_lane_below(__float_as_uint(v[CC - 1]))), __uint_as_float(from_lane_above(__float_as_uint(v[0])))};
        };
        auto row_of = [&](const float (&v)[CC], const Ends &ends) {
            QuadRow r;
#pragma unroll
            for (int j = 0; j < CC; ++j) r.v[j] = v[j];
            r.w = ends.w, r.e = ends.e;
            if (SMALL && B == kClamp) {
                clamp_columns(r, gc0, cols);
            } else if (kEdge) {
                r.w = no_west ? (B == kClamp ? v[0] : a.pad) : r.w;
                r.e = no_east ? (B == kClamp ? v[CC - 1] : a.pad) : r.e;
            }
            return r;
        };
        // one application, x to y
        auto apply_once = [&](const float (&x)[RPT][CC], float (&y)[RPT][CC], int buffer) {
            store_vec(first_rows + buffer + tid * CC, x[0]);
            store_vec(last_rows + buffer + tid * CC, x[RPT - 1]);
            auto apply = [&](int i, const QuadRow &up, const QuadRow &mid, const QuadRow &dn) {
                if (B == kClamp && SMALL && row0 + i == rows - 1)
                    temporal_quad<Op>(y[i], up, mid, mid, a.w, a.scalar0);
                else
                    temporal_quad<Op>(y[i], up, mid, dn, a.w, a.scalar0);
                if (B == kConstant && SMALL) pad_outside(y[i], i);
            };
            // All rows' cross-lane moves together, nothing between them.  Two wavefronts of a SIMD issue vector instructions in
            // the same cycles; after a cross-lane move they take turns instead, until a scalar instruction parts them (a
            // microbenchmark's additions: 2.1 cycles each with two wavefronts, 4.1 with a move among 24 of them), and after many
            // moves in a row for no longer.  As parts of the additions all over the rows: 100 clamped heat steps on 1025 x 1999
            // 118 us, now 108; 96 on 3072^2 262 and 223.  (An s_nop behind the moves: 111.)
            Ends ends[RPT];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < RPT; ++i) ends[i] = ends_of(x[i]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 1; i < RPT - 1; ++i) apply(i, row_of(x[i - 1], ends[i - 1]), row_of(x[i], ends[i]), row_of(x[i + 1], ends[i + 1]));
            __syncthreads();
            float above[CC], below[CC];
            load_vec(above, last_rows + buffer + above_at);
            load_vec(below, first_rows + buffer + below_at);
            if (kEdge) {
#pragma unroll
                for (int j = 0; j < CC; ++j) {
                    above[j] = no_above ? (B == kClamp ? x[0][j] : a.pad) : above[j];
                    below[j] = no_below ? (B == kClamp ? x[RPT - 1][j] : a.pad) : below[j];
                }
            }
            apply(0, row_of(above, ends_of(above)), row_of(x[0], ends[0]), row_of(x[1], ends[1]));
            apply(RPT - 1, row_of(x[RPT - 2], ends[RPT - 2]), row_of(x[RPT - 1], ends[RPT - 1]), row_of(below, ends_of(below)));
        };
        float y[RPT][CC];
        auto move_back = [&] {
#pragma unroll
            for (int i = 0; i < RPT; ++i)
#pragma unroll
                for (int j = 0; j < CC; ++j) x[i][j] = y[i][j];
        };
        if constexpr (PAIRED) {
            for (int k = 0; k < depth; k += 2) {
                apply_once(x, y, 0);
                if (k + 1 == depth) {
                    move_back();
                    break;
                }
                apply_once(y, x, 2 * CC * nthreads);
            }
        } else {
            for (int k = 0; k < depth; ++k) {
                apply_once(x, y, (k & 1) * 2 * CC * nthreads);
                move_back();
            }
        }

        if (gc0 + CC <= begin_c || gc0 >= end_c) return;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int r = row0 + i;
            if (r < begin_r || r >= end_r) continue;
            float *out = a.out + (size_t)r * cols + gc0;
            if (gc0 >= begin_c && gc0 + CC <= end_c) {
                store_out_vec(out, x[i], a.store);
            } else {
#pragma unroll
                for (int j = 0; j < CC; ++j)
                    if (gc0 + j >= begin_c && gc0 + j < end_c) out[j] = x[i][j];
            }
        }
    };
    if constexpr (SMALL) {
        applications(std::true_type{});
    } else {
        if (B != kWrap && edge)
            applications(std::true_type{});
        else
            applications(std::false_type{});
    }
}

}  // namespace sk
