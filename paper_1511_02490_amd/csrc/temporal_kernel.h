// Temporal blocking for iterated stencils with the 1/1/1/1 border region: one launch
// advances the matrix by `depth` applications (1 <= depth <= 4).  The workgroup stages its tile
// plus a border region `depth` cells deep (rows) and one 16-byte vector wide (columns) in local
// memory, then ping-pongs between two LDS buffers: after application k the values within k
// cells of the staged rim are stale, and after `depth` applications exactly the tile itself is
// still right and is written out.  HBM traffic per application falls by the depth; the price is
// the redundant rim work and one barrier per application.
//
// Out-of-matrix positions inside the staged tile: a periodic copy evolves like its original (nothing
// to do) and a padded position is set back to the padding value after every application.  Clamped
// positions are not kept at all: rows outside the matrix are not computed, the first and last row
// inside read themselves in their place, and a cell at the west or east edge takes its own value for
// the neighbour it lacks.  (They used to be copied from the nearest cell's new value after every
// application, a search over the whole tile behind a second barrier that the launch waited for:
// four heat steps on 1025 x 1999, tiles of 64 x 128, 23.2 -> 13.1 us, and 11.1 us with the walk below.)
// The per-cell arithmetic is the same fold as in the single-application kernels, so results
// are bit-identical to `depth` separate launches.
#pragma once
#include "tile_kernel.h"

namespace sk {

// Four cells of one LDS row plus the cells west and east of them.
struct QuadRow {
    float v[4];
    float w, e;
};

// CLAMP: the row of a vector whose first cell lies in matrix column `gc`, with the cells beyond the
// matrix edge taking the nearest in-matrix cell's value.  (Vectors that lie outside altogether are
// never asked for.)
__device__ __forceinline__ void clamp_columns(QuadRow &r, int gc, int cols) {
    r.w = gc == 0 ? r.v[0] : r.w;
    const int last = cols - 1 - gc;
#pragma unroll
    for (int j = 1; j < 4; ++j) r.v[j] = last < j ? r.v[j - 1] : r.v[j];
    r.e = last <= 3 ? r.v[3] : r.e;
}

// One application for the four cells of `mid`, given the rows above and below.
template <class Op>
__device__ __forceinline__ void temporal_quad(typename Op::T (&res)[4], const QuadRow &up, const QuadRow &mid,
                                              const QuadRow &dn, const WeightStore<Op, HaloC<1, 1, 1, 1>> &w,
                                              float scalar0) {
    typename Op::State st[4];
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) Op::init(st[cc]);
#pragma unroll
    for (int dr = -1; dr <= 1; ++dr) {
        const QuadRow &q = dr < 0 ? up : (dr == 0 ? mid : dn);
        const float row[6] = {q.w, q.v[0], q.v[1], q.v[2], q.v[3], q.e};
#pragma unroll
        for (int cc = 0; cc < 4; ++cc)
            fold_row<Op>(
                st[cc], dr, dr + 1, 3, 1, 1, [&](int dc) { return w[(dr + 1) * 3 + dc + 1]; },
                [&](int dc) { return row[1 + cc + dc]; });
    }
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) res[cc] = Op::finish(st[cc], scalar0);
}

// What the applications of a launch share.
struct TemporalTile {
    int pitch, nq;                  // a staged row in cells and in vectors
    int row_first, col_first;       // the matrix cell under the staged tile's first one
    int staged_rows;                // ER
    int first_row, last_row;        // the staged rows that an application may read or compute
    int depth;
    int R;                          // rows of an item
};
// A work-item's item in one pass of the workgroup over an application: a vector column x a group of R rows.
struct TemporalItem {
    int gc;                         // matrix column of its cells
    int group_row;                  // first of its rows, counted from the first the application computes
    int group_off;                  // ... and where its cells lie in local memory
    int first_off, last_off;        // where the first and the last row lie that may be read
    bool stores;
};

// Application k of a launch: tile rows [k, ER - k), everything that can still be right; the LAST one, on the
// tile's own cells, goes straight to global memory.  EDGE: the staged tile reaches outside the matrix.
//
// An application is bound by the instructions it issues: 24 of a heat step's arithmetic per vector of four
// cells, and what finds and moves the vector beside them.  A work-item therefore walks down a group of R rows
// of one vector column, its window in registers that change roles instead of places, the next row requested
// one step ahead, and takes the cells west and east of its own from the adjacent lanes: wavefronts overlap by
// two lanes, whose values are not stored, so that no lane has to look elsewhere.  (Vectors at the two ends of
// a staged row get whatever the lanes beside them hold - values that only ever reach rim cells that are
// stale.)  In a workgroup that is not WHOLE wavefronts the two cells are read from local memory instead, and so
// they are in the last application, whose items are not the others'.
template <class Op, int B, bool WHOLE, bool EDGE, bool LAST>
__device__ __forceinline__ void temporal_application(const TileArgs<Op, HaloC<1, 1, 1, 1>> &a, const TemporalTile &s,
                                                     const TemporalItem &it, int k, const float *src, float *dst) {
    using T = typename Op::T;
    constexpr int CC = 4;
    const int pitch = s.pitch, rows = a.rows, cols = a.cols;
    const int k_begin = max(k, s.first_row), k_end = min(s.staged_rows - k, s.last_row + 1);
    // offsets walk with the rows (a product per row would cost as much as a third of its arithmetic)
    int at = k_begin * pitch + it.group_off;
    const int end_off = k_end * pitch + it.first_off - s.first_row * pitch;
    auto neighbours = [&](QuadRow &r, int off) {
        if (WHOLE) {
            r.w = __uint_as_float(from_lane_below(__float_as_uint(r.v[3])));
            r.e = __uint_as_float(from_lane_above(__float_as_uint(r.v[0])));
        } else {
            r.w = src[off - 1];
            r.e = src[off + CC];
        }
        if (B == kClamp && EDGE) clamp_columns(r, it.gc, cols);
    };
    QuadRow row[4];
    int off[4];
    off[0] = min(max(at - pitch, it.first_off), it.last_off);
    off[1] = min(at, it.last_off);
    off[2] = min(at + pitch, it.last_off);
#pragma unroll
    for (int p = 0; p < 3; ++p) load_vec(row[p].v, src + off[p]);
    neighbours(row[0], off[0]);
    neighbours(row[1], off[1]);
    int gr = s.row_first + k_begin + it.group_row;
    [[maybe_unused]] T *out = a.out + (ptrdiff_t)gr * cols + it.gc;
    const int R = min(s.R, k_end - k_begin);   // (a single group holds fewer rows from application to application)
    for (int rr = 0; rr < R; rr += 4) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            if (rr + p >= R) break;                // (the same for the whole workgroup)
            QuadRow &up = row[p], &mid = row[(p + 1) % 4], &dn = row[(p + 2) % 4], &ahead = row[(p + 3) % 4];
            off[(p + 3) % 4] = min(at + 2 * pitch, it.last_off);
            load_vec(ahead.v, src + off[(p + 3) % 4]);
            neighbours(dn, off[(p + 2) % 4]);
            T res[CC];
            temporal_quad<Op>(res, up, mid, dn, a.w, a.scalar0);
            if (B == kConstant && EDGE && !LAST) {
#pragma unroll
                for (int cc = 0; cc < CC; ++cc)
                    if ((unsigned)gr >= (unsigned)rows || (unsigned)(it.gc + cc) >= (unsigned)cols) res[cc] = a.pad;
            }
            if (it.stores && at < end_off) {
                if (!LAST) {
                    store_vec(dst + at, res);
                } else if (!EDGE || it.gc + CC <= cols) {
                    store_out_vec(out, res, a.store);
                } else {
#pragma unroll
                    for (int cc = 0; cc < CC; ++cc)
                        if (it.gc + cc < cols) out[cc] = res[cc];
                }
            }
            at += pitch;
            ++gr;
            out += cols;
        }
    }
}

// All applications of a launch.  The last one computes the tile's own cells, one for one those of the work-items: each its
// own `cells_rows` rows of its own vector, all lanes at work, the two cells beside the vector from local memory.  (Walked in
// the groups of the others it kept a third of the lanes idle and went on for as many rows as the first application has:
// four heat steps per launch on 4096^2, WRAP, us per launch before / now: 4x4 cells, 1x256 work-items 287 / 261, 2x5 214 / 191;
// 2x4 cells, 4x64 work-items 52.3 / 50.4.)
template <class Op, int B, bool WHOLE, bool EDGE>
__device__ __forceinline__ void temporal_applications(const TileArgs<Op, HaloC<1, 1, 1, 1>> &a, TemporalTile &s, int cells_rows,
                                                      int tid, int nthreads, float *src, float *dst) {
    const int lane = tid & 63;
    // as many groups of rows as one pass of the workgroup has lanes for: one pass, except where the workgroup
    // holds less than a row of vectors
    const int per_pass = WHOLE ? nthreads / 64 * 62 : nthreads;
    const int groups = max(1, (int)row_of_item(per_pass, a.stage_magic)), items = groups * s.nq;
    s.R = (s.staged_rows - 2 + groups - 1) / groups;
    auto item_of = [&](int base) {
        const int index = base + (WHOLE ? (tid >> 6) * 62 + lane - 1 : tid), item = max(0, min(index, items - 1));
        const int g = (int)row_of_item(item, a.stage_magic), q = item - g * s.nq;
        TemporalItem it;
        it.gc = s.col_first + q * 4;
        it.group_row = g * s.R;
        it.group_off = it.group_row * s.pitch + q * 4;
        it.first_off = s.first_row * s.pitch + q * 4;
        it.last_off = s.last_row * s.pitch + q * 4;
        it.stores = (!WHOLE || (lane > 0 && lane < 63)) && index < items;
        return it;
    };
    const TemporalItem first = item_of(0);
    for (int k = 1; k < s.depth; ++k) {
        temporal_application<Op, B, WHOLE, EDGE, false>(a, s, first, k, src, dst);
        for (int base = per_pass; base < items; base += per_pass)
            temporal_application<Op, B, WHOLE, EDGE, false>(a, s, item_of(base), k, src, dst);
        __syncthreads();
        float *tmp = src;
        src = dst;
        dst = tmp;
    }
    TemporalItem own;
    own.gc = s.col_first + (1 + (int)threadIdx.x) * 4;
    own.group_row = (int)threadIdx.y * cells_rows;
    own.group_off = own.group_row * s.pitch + (1 + (int)threadIdx.x) * 4;
    own.first_off = s.first_row * s.pitch + (1 + (int)threadIdx.x) * 4;
    own.last_off = s.last_row * s.pitch + (1 + (int)threadIdx.x) * 4;
    own.stores = own.gc < a.cols;
    s.R = cells_rows;
    temporal_application<Op, B, false, EDGE, true>(a, s, own, s.depth, src, dst);
}

template <class Op, int B, bool WHOLE, int MAXT>
__global__ __launch_bounds__(MAXT) void temporal_kernel(const TileArgs<Op, HaloC<1, 1, 1, 1>> a, const int depth,
                                                        const int cells_rows) {
    static_assert(Op::kPlanes == 1 && sizeof(typename Op::T) == 4 && sizeof(typename Op::L) == 4, "fp32, one plane");
    constexpr int CC = 4, HC = 4;   // cells per vector; staged columns each side of the tile
    extern __shared__ __align__(16) unsigned char lds_raw[];
    // [one spare vector][buffer][buffer][one spare vector]: the reads one word before a row's
    // first vector and one word after its last stay inside the allocation
    float *src = reinterpret_cast<float *>(lds_raw) + CC;
    float *dst = src + a.plane;

    const int wr = blockDim.y, wc = blockDim.x;
    const int tid = (int)threadIdx.y * wc + (int)threadIdx.x, nthreads = wr * wc;

    int t = blockIdx.x;
    if (a.xcd_chunk > 0) t = (t & 7) * a.xcd_chunk + (t >> 3);
    if (t >= a.n_tiles) return;
    const int tile_r = t / a.tiles_c, tile_c = t - tile_r * a.tiles_c;
    const int rows = a.rows, cols = a.cols, pitch = a.pitch;
    const int tile_rows = wr * cells_rows, r0 = tile_r * tile_rows, c0 = tile_c * wc * CC;
    TemporalTile s;
    s.pitch = pitch;
    s.nq = pitch / CC;
    s.row_first = r0 - depth;
    s.col_first = c0 - HC;
    const int ER = min(tile_rows, rows - r0) + 2 * depth;   // staged rows in use
    s.staged_rows = ER;
    s.depth = depth;

    stage_tile<Op, B, CC>(src, a.plane, pitch, a.in, rows, cols, s.row_first, s.col_first, ER, cols + HC, a.pad,
                          a.stage_magic, tid, nthreads);
    __syncthreads();

    // under CLAMP only matrix rows are read or computed
    s.first_row = B == kClamp ? max(0, -s.row_first) : 0;
    s.last_row = B == kClamp ? min(ER, rows - s.row_first) - 1 : ER - 1;
    // does the staged tile reach outside the matrix?  (same answer for the whole workgroup)
    if (s.row_first < 0 || s.row_first + ER > rows || s.col_first < 0 || s.col_first + pitch > cols)
        temporal_applications<Op, B, WHOLE, true>(a, s, cells_rows, tid, nthreads, src, dst);
    else
        temporal_applications<Op, B, WHOLE, false>(a, s, cells_rows, tid, nthreads, src, dst);
}

}  // namespace sk
