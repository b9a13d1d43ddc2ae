// Temporal blocking in registers for iterated stencils with the 1/1/1/1 border region:
// one launch advances the matrix by DEPTH applications without local memory or barriers.
//
// A wavefront owns a strip of the matrix: its 64 lanes hold 64 consecutive 4-cell vectors of a
// row (256 columns) and it walks down H + 2*DEPTH rows.  Every lane keeps, for each of the
// DEPTH time levels, the last three rows of its vector; as soon as input row t has arrived,
// level 1 can produce its row t - 1, level 2 its row t - 2, and so on (each level lags one row
// behind the one below), and level DEPTH's rows go straight to global memory.  Row neighbours
// come from the adjacent lanes by cross-lane moves.  What a level computes within k cells of the
// strip's edge is stale after k applications, so the outermost lanes are rim lanes (4 cells each:
// one lane per side up to 4 applications, two up to 8) and the strip's 62 or 60 inner vectors are
// written; strips therefore advance by 248 or 240 columns, rows by H.
//
// Borders: periodic copies evolve like their originals, so WRAP needs nothing beyond wrapped
// loads; under CONSTANT the out-of-matrix cells of every level are set back to the padding
// value.  (CLAMP would need a clamped row's new value before the marching order produces it;
// it stays with the local-memory temporal kernel.)  The per-cell arithmetic is the same fold as
// everywhere else: results are bit-identical to DEPTH single launches.
#pragma once
#include "tile_kernel.h"

namespace sk {

constexpr int kStreamLanes = 64;                    // vectors per strip row, rim included
constexpr int kStreamMaxDepth = 8;
// rim lanes per side, and the columns a strip writes, for `depth` applications per launch
__host__ __device__ constexpr int stream_rim(int depth) { return (depth + 3) / 4; }
__host__ __device__ constexpr int stream_cols(int depth) { return (kStreamLanes - 2 * stream_rim(depth)) * 4; }

// A vector at a byte offset in a row of so many bytes, written through the L2 cache (Store::kThrough): by the row's own buffer
// descriptor, which is scalar, so that a lane keeps its offset as for the other kinds of store.  (With a 64-bit address per lane,
// in a statement that the compiler cannot move, a heat march took 8 to 18 registers more and at 5, 7 and 8 applications per
// launch a wavefront per SIMD: constant border, 8 per launch, up to 7 % slower than with plain stores, now as fast or faster.)
template <class E>
__device__ __forceinline__ void store_through(char *row, unsigned row_bytes, unsigned offset, const E (&src)[4]) {
    static_assert(sizeof(src) == 16, "one 16-byte vector");
    typedef uint32_t word4 __attribute__((ext_vector_type(4)));
    word4 v;
    __builtin_memcpy(&v, src, sizeof(v));
    constexpr int kRaw32 = 0x00020000, kSc1 = 16;      // the descriptor's data format; the store's cache policy
    __builtin_amdgcn_raw_buffer_store_b128(v, __builtin_amdgcn_make_buffer_rsrc(row, 0, (int)row_bytes, kRaw32), (int)offset, 0, kSc1);
}

// FAST: rows are whole vectors (cols % 4 == 0).  A lane's four
// columns then lie either all inside the matrix or all outside it, every input row is one vector
// load at a per-lane column plus a wavefront-uniform row address, issued without a branch three
// steps ahead, and the time loop is straight-line code.  Otherwise elements are loaded one by one.
// S: how output vectors are stored (element-by-element stores are plain in any case).
// (A branch at the store, in an unrolled march: 148 instead of 133 registers for eight heat steps under WRAP, one wavefront
// per SIMD fewer at depths 5 and 7; 400 steps on 4096^2, 8 per launch, 1915 instead of 1873 us.)
template <class Op, int B, int DEPTH, bool FAST, Store S>
__device__ __forceinline__ void stream_body(const TileArgs<Op, HaloC<1, 1, 1, 1>> &a, const int H) {
    using T = typename Op::T;
    static_assert(B == kWrap || B == kConstant, "wrap and constant borders only");
    static_assert(DEPTH >= 1 && DEPTH <= kStreamMaxDepth, "a rim lane covers four applications");
    static_assert(Op::kPlanes == 1 && sizeof(T) == 4, "fp32, one value per cell");
    // only a cell's own row has neighbours in other lanes, nothing parts the levels of a step, and the moves of several are worth
    // their registers (97 instead of 95 at five levels, a wavefront per SIMD; five levels 338 / 332 us for 56 steps on 4096^2)
    constexpr bool kCross = std::is_same<Op, OpHeat>::value && B == kWrap && DEPTH >= 6;
    constexpr int CC = 4;
    constexpr int R = 3;                            // rows of a level kept
    constexpr int PF = 6;                           // input rows in flight = steps per round (a multiple of R)
    constexpr int kRim = stream_rim(DEPTH);
    constexpr int kCols = stream_cols(DEPTH);

    const int tid = (int)threadIdx.y * (int)blockDim.x + (int)threadIdx.x;
    const int lane = tid & 63;
    const int waves_per_block = ((int)blockDim.x * (int)blockDim.y) >> 6;
    // a wavefront's index is the same in all its lanes: keep it, and all that follows from it, scalar
    const int wave = __builtin_amdgcn_readfirstlane((int)blockIdx.x * waves_per_block + (tid >> 6));
    if (wave >= a.n_tiles) return;
    const int seg = wave / a.tiles_c, strip = wave - seg * a.tiles_c;
    const int rows = a.rows, cols = a.cols;
    const int r0 = seg * H;
    const int gc0 = strip * kCols - kRim * CC + lane * CC;     // first of this lane's four columns
    const bool writes = lane >= kRim && lane < kStreamLanes - kRim && gc0 < cols;

    // FAST: the column the lane's vector load starts at (wrapped, or any valid one for padding)
    const bool outside = (unsigned)gc0 >= (unsigned)cols;
    const int vcol = !outside ? gc0 : (B == kWrap ? resolve<B>(gc0, cols) : 0);
    const bool edge_wave = __any(outside) != 0;     // the same for the whole wavefront
    const unsigned in_off = (unsigned)vcol * (unsigned)sizeof(T);    // byte offsets inside a row
    const unsigned out_off = (unsigned)gc0 * (unsigned)sizeof(T);
    // otherwise: the lane's columns after border resolution (-1: padding)
    int col[CC];
#pragma unroll
    for (int j = 0; j < CC; ++j) col[j] = resolve<B>(gc0 + j, cols);
    bool outside_c[CC];   // CONSTANT: cells that are not matrix cells
#pragma unroll
    for (int j = 0; j < CC; ++j) outside_c[j] = (unsigned)(gc0 + j) >= (unsigned)cols;

    // A segment consumes kSteps input rows; the march makes whole rounds of PF steps (what the
    // steps past kSteps compute is never stored).
    const int kSteps = H + 2 * DEPTH;
    const int kRounds = (kSteps + PF - 1) / PF;

    // issue the loads of input row r0 - DEPTH + t
    auto load_row = [&](int t, T (&v)[CC]) {
        const int tt = t < kSteps ? t : kSteps - 1;
        const int gr = resolve<B>(r0 - DEPTH + tt, rows);      // the same for the whole wavefront
        if (FAST) {
            const char *rowp = reinterpret_cast<const char *>(a.in + (size_t)(gr < 0 ? 0 : gr) * cols);
            load_global(v, reinterpret_cast<const T *>(rowp + in_off));
        } else {
#pragma unroll
            for (int j = 0; j < CC; ++j)
                v[j] = (gr >= 0 && col[j] >= 0) ? a.in[(size_t)gr * cols + col[j]] : a.pad;
        }
    };
    // CONSTANT: cells of matrix row gr (any time level) that are not matrix cells hold the padding
    auto pad_outside = [&](int gr, T (&v)[CC]) {
        if (B != kConstant) return;
        const bool outside_r = (unsigned)gr >= (unsigned)rows;
        if (FAST) {
            if (outside_r || edge_wave) {
#pragma unroll
                for (int j = 0; j < CC; ++j) v[j] = (outside_r || outside) ? a.pad : v[j];
            }
        } else {
#pragma unroll
            for (int j = 0; j < CC; ++j)
                if (outside_r || outside_c[j]) v[j] = a.pad;
        }
    };

    // lv[k][s]: level k's row that was produced at a time step with t % 3 == s  (level 0 = input)
    T lv[DEPTH][R][CC];
#pragma unroll
    for (int k = 0; k < DEPTH; ++k)
#pragma unroll
        for (int s = 0; s < R; ++s)
#pragma unroll
            for (int j = 0; j < CC; ++j) lv[k][s][j] = 0;
    T pf[PF][CC];         // rows on their way from memory, PF time steps ahead
#pragma unroll
    for (int s = 0; s < PF; ++s) {
        load_row(s, pf[s]);
        // in the order the march consumes them: were the scheduler to issue the first-needed row
        // last, every round of the loop would begin by waiting for all loads in flight
        __builtin_amdgcn_sched_barrier(0);
    }

    for (int round = 0; round < kRounds; ++round) {
#pragma unroll
        for (int v = 0; v < PF; ++v) {
            const int t = round * PF + v;
            const int u = v % R;                    // = t % R
#pragma unroll
            for (int j = 0; j < CC; ++j) lv[0][u][j] = pf[v][j];
            pad_outside(r0 - DEPTH + t, lv[0][u]);
            load_row(t + PF, pf[v]);
            // The cross-lane moves of all levels together: the row in the middle of each is there since the step before.  (A
            // cross-lane move costs a SIMD's wavefronts the cycles in which two of them issue, many in a row no more than one:
            // register_tile_kernel.h.  As part of each level's additions a launch of eight heat steps on 4096^2, WRAP, took
            // 36.9 us, now 34.9: 18.7 k vector instructions per SIMD, at the 1.85 GHz that this load leaves of the clock.
            // CONSTANT, where a branch after every level parts them, gains nothing.)
            T sides[DEPTH][2];
            if constexpr (kCross) {
#pragma unroll
                for (int k = 0; k < DEPTH; ++k) {
                    const T(&mid)[CC] = lv[k][(u + 2) % R];
                    sides[k][0] = __uint_as_float(from_lane_below(__float_as_uint(mid[CC - 1])));
                    sides[k][1] = __uint_as_float(from_lane_above(__float_as_uint(mid[0])));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int k = 1; k <= DEPTH; ++k) {
                // level k's first row that anything depends on is r0 - DEPTH + k, due at step 2k:
                // before that the level has nothing to do (a wavefront-uniform test)
                if (t < 2 * k) continue;
                // level k's row r0 - DEPTH + t - k from level k-1's three newest rows
                const T(&up)[CC] = lv[k - 1][(u + 1) % R];
                const T(&mid)[CC] = lv[k - 1][(u + 2) % R];
                const T(&dn)[CC] = lv[k - 1][u];
                typename Op::State st[CC];
#pragma unroll
                for (int cc = 0; cc < CC; ++cc) Op::init(st[cc]);
#pragma unroll
                for (int dr = -1; dr <= 1; ++dr) {
                    const T(&q)[CC] = dr < 0 ? up : (dr == 0 ? mid : dn);
                    const T row[6] = {kCross ? sides[k - 1][0] : __uint_as_float(from_lane_below(__float_as_uint(q[3]))), q[0], q[1], q[2],
                                      q[3], kCross ? sides[k - 1][1] : __uint_as_float(from_lane_above(__float_as_uint(q[0])))};
#pragma unroll
                    for (int cc = 0; cc < CC; ++cc)
                        fold_row<Op>(
                            st[cc], dr, dr + 1, 3, 1, 1, [&](int dc) { return a.w[(dr + 1) * 3 + dc + 1]; },
                            [&](int dc) { return row[1 + cc + dc]; });
                }
                T res[CC];
#pragma unroll
                for (int cc = 0; cc < CC; ++cc) res[cc] = Op::finish(st[cc], a.scalar0);
                const int gr = r0 - DEPTH + t - k;      // the matrix row just produced
                if (k < DEPTH) {
                    pad_outside(gr, res);
#pragma unroll
                    for (int cc = 0; cc < CC; ++cc) lv[k][u][cc] = res[cc];
                } else if (t >= 2 * DEPTH && t < kSteps && gr < rows && writes) {
                    // gr = r0 + t - 2*DEPTH runs over this segment's rows
                    if (FAST) {
                        char *rowp = reinterpret_cast<char *>(a.out + (size_t)gr * cols);
                        if constexpr (S == Store::kThrough)
                            store_through(rowp, (unsigned)cols * (unsigned)sizeof(T), out_off, res);
                        else
                            store_out_vec<S>(reinterpret_cast<T *>(rowp + out_off), res);
                    } else {
                        T *out = a.out + (size_t)gr * cols + gc0;
#pragma unroll
                        for (int cc = 0; cc < CC; ++cc)
                            if (gc0 + cc < cols) out[cc] = res[cc];
                    }
                }
            }
        }
    }
}

template <class Op, int B, int DEPTH, bool FAST, bool NT, int MAXT>
__global__ __launch_bounds__(MAXT) void stream_kernel(const TileArgs<Op, HaloC<1, 1, 1, 1>> a, const int H) {
    stream_body<Op, B, DEPTH, FAST, NT ? Store::kNonTemporal : Store::kPlain>(a, H);
}
// ... and written through (store_through), over rows of whole vectors, from kStreamThroughDepth applications per launch on (heat, WRAP, a launch
// of eight on 4096^2, plain / through: 37.0 / 35.6 us; of two 22.6 / 23.2; of one 22.0 / 22.6).
constexpr int kStreamThroughDepth = 4;
template <class Op, int B, int DEPTH, int MAXT>
__global__ __launch_bounds__(MAXT) void stream_through_kernel(const TileArgs<Op, HaloC<1, 1, 1, 1>> a, const int H) {
    stream_body<Op, B, DEPTH, true, Store::kThrough>(a, H);
}

}  // namespace sk
