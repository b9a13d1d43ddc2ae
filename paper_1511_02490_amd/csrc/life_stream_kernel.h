// Game of Life, several generations per launch, on bits in registers (the arithmetic: life_bits.h).
//
// A work-item holds RPT rows of one word (32 cells) of the matrix.  16, 32 or 64 adjacent lanes hold adjacent
// words, the lanes' groups rows below each other, and the workgroup so holds a tile.  Per generation a row's
// west and east neighbours come from the adjacent lanes by cross-lane moves, and only the first and the last
// row of every work-item pass through local memory, behind one barrier (two buffers in turn).  What a generation
// computes within k rows or cells of the tile's rim is stale after k generations: `depth` rows above and below
// and a word left and right are not written.
//
// Borders.  WRAP: a periodic copy evolves like its original.  CLAMP and CONSTANT: the first tile of a column of
// tiles begins with the matrix's first row and the last one ends with its last, so that what a row lacks above or
// below is found once per work-item and generation (itself, or the padding) and not looked for at every row; at
// the west and east edge a cell takes itself for the neighbour it lacks, or the cells outside are set back.
//
// Between the launches of a run the matrix is kept as bits, rows of whole words: the first launch turns bytes
// into bits, the last one bits into bytes, and the launches between them move an eighth of the bytes.  They are
// bound by the generations' serial chain (a row's sums, the barrier, the rule), not by memory, and by what a launch,
// its loads and its stores cost whatever it computes: the tile is cut, and the generations of a run are dealt to
// launches, so that both are small together (life_tile, life_run_tile and life_per_launch in variants.h).
// (100 generations of 4096 x 4096, WRAP: 282 us by marching packed bytes down the matrix, 121 on bits with 8 to a
// launch, 65 with 25 in workgroups of 512.  50 generations of 1001 x 1503, CLAMP: 83 us by life_temporal_kernel, 4 to a launch from
// bytes to bytes, 23 here with 25.)
#pragma once
#include "life_bits.h"

namespace sk {

constexpr int kLifeStreamMaxDepth = 32;     // generations that the rim, a word of cells a side, is right for
// Workgroups: of 16 rows per work-item (the registers of a launch that reads bytes) up to 256 work-items.
constexpr int life_stream_max_threads(int rows_per_item) { return rows_per_item == 16 ? 256 : 1024; }
constexpr unsigned life_stream_lds(int threads) { return 4 * (unsigned)threads * (unsigned)sizeof(uint32_t); }

struct LifeStreamArgs {
    const void *in;
    void *out;
    int rows, cols, words;       // words per row of a matrix of bits
    int tiles_c, n_tiles;
    int group_shift;             // log2 of the lanes that hold a row of the tile
    int pad;                     // 0 or 1
    Store store;
};

template <int B, int RPT, bool IN_BITS, bool OUT_BITS>
__global__ __launch_bounds__(life_stream_max_threads(RPT)) void life_stream_kernel(const LifeStreamArgs a, const int depth) {
    const int tid = (int)threadIdx.y * (int)blockDim.x + (int)threadIdx.x, nthreads = (int)(blockDim.x * blockDim.y);
    const int G = 1 << a.group_shift, groups = nthreads >> a.group_shift;
    const int rows = a.rows, cols = a.cols;
    const int tile_r = (int)blockIdx.x / a.tiles_c, tile_c = (int)blockIdx.x - tile_r * a.tiles_c;
    const int word = tile_c * (G - 2) - 1 + (tid & (G - 1)), col = word * 32;
    const int held = groups * RPT, step = held - 2 * depth;            // rows of the tile; the rows from one tile to the next
    // the first row it holds, and the rows it writes
    int top, begin, end;
    // (differences from `rows`: what lies beyond the last tile may be beyond the largest int)
    if (B == kWrap) {
        top = tile_r * step - depth;
        begin = tile_r * step;
        end = begin + min(step, rows - begin);
    } else {
        top = max(0, min(tile_r * step, rows - held));
        begin = tile_r == 0 ? 0 : tile_r * step + depth;
        end = tile_r * step >= rows - held ? rows : (tile_r + 1) * step + depth;
    }
    const int below_top = (tid >> a.group_shift) * RPT, row0 = (int)((unsigned)top + (unsigned)below_top);
    const uint32_t pad = a.pad ? ~0u : 0u;
    const uint32_t inside = inside_bits(col, cols);

    // the matrix rows it loads: under WRAP row0's and, going round, those after it; else any where there is none
    int gr[RPT];
    gr[0] = B == kWrap ? resolve<kWrap>((top > INT32_MAX - held ? top - rows : top) + below_top, rows) : min(row0, rows - 1);
#pragma unroll
    for (int i = 1; i < RPT; ++i) {
        if (B == kWrap)
            gr[i] = gr[i - 1] + 1 == rows ? 0 : gr[i - 1] + 1;
        else
            gr[i] = min(row0 + i, rows - 1);
    }
    uint32_t x[RPT];
    if constexpr (IN_BITS) {
        const uint32_t *in = static_cast<const uint32_t *>(a.in);
        const int there = max(0, min(word, a.words - 1));
#pragma unroll
        for (int i = 0; i < RPT; ++i) x[i] = in[(unsigned)(gr[i] * a.words + there)];
        if (B == kWrap && inside != ~0u) {
            // a word that is not simply there: 32 cells from column `col` round the end of the row
            const int at = resolve<B>(col, cols);
            if (cols >= 32) {
                const int w = at >> 5, after = min(w + 1, a.words - 1), have = cols - at;
                const uint32_t keep = have >= 32 ? ~0u : (1u << have) - 1u;
#pragma unroll
                for (int i = 0; i < RPT; ++i) {
                    const uint32_t *row = in + (unsigned)(gr[i] * a.words);
                    x[i] = (__builtin_amdgcn_alignbit(row[after], row[w], at & 31) & keep) | (have >= 32 ? 0u : row[0] << (have & 31));
                }
            } else {        // the row is one word
                uint32_t y[RPT] = {};
                int from = at;
#pragma unroll 1
                for (int k = 0; k < 32; ++k) {
#pragma unroll
                    for (int i = 0; i < RPT; ++i) y[i] |= ((x[i] >> from) & 1u) << k;
                    from = from + 1 == cols ? 0 : from + 1;
                }
#pragma unroll
                for (int i = 0; i < RPT; ++i) x[i] = y[i];
            }
        }
    } else {
        const uint8_t *in = static_cast<const uint8_t *>(a.in);
        if (cols >= 16) {
            LifeLoad v[RPT][2];
#pragma unroll
            for (int i = 0; i < RPT; ++i) {
                v[i][0] = life_load16<B>(in, gr[i], col, cols);
                v[i][1] = life_load16<B>(in, gr[i], col + 16, cols);
            }
#pragma unroll
            for (int i = 0; i < RPT; ++i) {
                x[i] = life_bits16<B>(v[i][0], in, gr[i], cols, 0) | (life_bits16<B>(v[i][1], in, gr[i], cols, 0) << 16);
            }
        } else {
#pragma unroll
            for (int i = 0; i < RPT; ++i) {
                x[i] = life_bits16_narrow<B>(in, gr[i], col, cols, 0) | (life_bits16_narrow<B>(in, gr[i], col + 16, cols, 0) << 16);
            }
        }
    }
    // does the tile reach outside the matrix, east or west, and below (a matrix lower than a tile)?  The same for the
    // whole workgroup.
    const bool at_sides = tile_c == 0 || (tile_c + 1) * (G - 2) * 32 + 32 > cols, below_matrix = held > rows;
    // CONSTANT: cells that are not matrix cells hold the padding
    auto pad_outside = [&] {
        int below = rows - row0;
        asm volatile("" : "+v"(below));         // (or the rows' masks are kept in registers from generation to generation)
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const uint32_t keep = i < below ? inside : 0u;
            x[i] = (x[i] & keep) | (pad & ~keep);
        }
    };
    if (B == kConstant && (at_sides || below_matrix)) pad_outside();

    // CLAMP: the columns outside are not kept; a cell at the matrix's edge takes itself for the neighbour it lacks
    const uint32_t first = column_bit(col, 0), last = column_bit(col, cols - 1);
    extern __shared__ __align__(16) unsigned char lds_raw[];      // two buffers of the work-items' first and last rows
    uint32_t *first_rows = reinterpret_cast<uint32_t *>(lds_raw), *last_rows = first_rows + nthreads;
    const int above_at = max(0, tid - G), below_at = min(tid + G, nthreads - 1);
    const bool no_above = row0 == 0, no_below = row0 + RPT == rows;
    // EDGE, BELOW: the tile has an edge of the matrix (and may reach outside it east or west); below_matrix
    auto generations = [&](auto EDGE, auto BELOW) {
        constexpr bool kEdge = decltype(EDGE)::value, kBelow = decltype(BELOW)::value;
        // a row with its neighbours from the adjacent lanes; what the two ends of a group of lanes get is no
        // neighbour, and stays in the rim
        struct Beside { uint32_t w, e; };        // the words of the adjacent lanes
        auto beside = [](uint32_t v) { return Beside{from_lane_below(v), from_lane_above(v)}; };
        auto sums = [&](uint32_t v, Beside b) {
            uint32_t w = west_of(v, b.w), e = east_of(v, b.e);
            if (B == kClamp && kEdge) {
                w = (w & ~first) | (v & first);
                e = (e & ~last) | (v & last);
            }
            return life_bits(v, w, e);
        };
        auto next = [&](const LifeBits &up, const LifeBits &mid, const LifeBits &dn, int i) {
            return life_next(up, mid, B == kClamp && kBelow && row0 + i == rows - 1 ? mid : dn);
        };
        for (int k = 0; k < depth; ++k) {
            const int buffer = (k & 1) * 2 * nthreads;
            first_rows[buffer + tid] = x[0];
            last_rows[buffer + tid] = x[RPT - 1];
            LifeBits h[RPT];
            // (All rows' cross-lane moves together: after one the wavefronts of a SIMD take turns for a while where two would issue
            // at once, and after many in a row for no longer.  In workgroups of 256, 30 clamped generations of 1000^2 15.3 -> 13.1
            // us, 50 of 1001 x 1503 24.5 -> 22.8, 100 of 2048^2 52.8 -> 51.3; of 4096^2, by eight rows per item, 77.3 and 77.4.)
            Beside b[RPT];
#pragma unroll
            for (int i = 0; i < RPT; ++i) b[i] = beside(x[i]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < RPT; ++i) h[i] = sums(x[i], b[i]);
            const uint32_t x_first = x[0], x_last = x[RPT - 1];
#pragma unroll
            for (int i = 1; i < RPT - 1; ++i) x[i] = next(h[i - 1], h[i], h[i + 1], i);
            __syncthreads();
            uint32_t above = last_rows[buffer + above_at], below = first_rows[buffer + below_at];
            if (kEdge) {
                above = no_above ? (B == kClamp ? x_first : pad) : above;
                below = no_below ? (B == kClamp ? x_last : pad) : below;
            }
            const Beside above_b = beside(above), below_b = beside(below);
            x[0] = next(sums(above, above_b), h[0], h[1], 0);
            x[RPT - 1] = next(h[RPT - 2], h[RPT - 1], sums(below, below_b), RPT - 1);
            if (B == kConstant) {
                if (kBelow) {
                    pad_outside();
                } else if (kEdge) {
#pragma unroll
                    for (int i = 0; i < RPT; ++i) x[i] = (x[i] & inside) | (pad & ~inside);
                }
            }
        }
    };
    if (B != kWrap && below_matrix)
        generations(std::true_type{}, std::true_type{});
    else if (B != kWrap && (at_sides || top == 0 || top + held == rows))
        generations(std::true_type{}, std::false_type{});
    else
        generations(std::false_type{}, std::false_type{});

    const int lane = tid & (G - 1);
    if (!OUT_BITS && a.store == Store::kThrough) {
        // Adjacent lanes store adjacent 16 bytes: a row in two pieces, each lane one half of another lane's cells.  (By two stores
        // of a lane's own 32 cells each instruction writes every other 16 bytes of a line, which a cache puts together, but written
        // through the halves go to memory one by one: boards of 16 MiB and more, from bytes to bytes, 1.3 to 1.6 times as long.)
        const int shift = 16 * (lane & 1);
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int r = row0 + i;
            if (r < begin || r >= end) continue;                         // (the same for a group of lanes)
#pragma unroll
            for (int piece = 0; piece < 2; ++piece) {
                const int from = (lane >> 1) + piece * (G >> 1);         // the lane of the group whose cells they are
                const uint32_t cells = (uint32_t)__builtin_amdgcn_ds_bpermute(((tid - lane + from) & 63) << 2, (int)x[i]) >> shift;
                const int at = (word - lane + from) * 32 + shift;
                if (from == 0 || from == G - 1 || at >= cols) continue;
                uint8_t *out = static_cast<uint8_t *>(a.out) + (unsigned)(r * cols + at);
                if (at + 16 <= cols)
                    store_word4<Store::kThrough>(out, unpack_cells16(cells));
                else
                    store_first_cells(out, unpack_cells16(cells), cols - at);
            }
        }
        return;
    }
    if (lane == 0 || lane == G - 1 || word >= a.words) return;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int r = row0 + i;
        if (r < begin || r >= end) continue;
        if constexpr (OUT_BITS) {
            static_cast<uint32_t *>(a.out)[(unsigned)(r * a.words + word)] = x[i];
        } else {
            uint8_t *out = static_cast<uint8_t *>(a.out) + (unsigned)(r * cols + col);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const uint4 o = unpack_cells16(x[i] >> (16 * half));
                if (col + 16 * half + 16 <= cols) {
                    store_word4(out + 16 * half, o, a.store == Store::kNonTemporal);
                } else if (col + 16 * half < cols) {
                    store_first_cells(out + 16 * half, o, cols - (col + 16 * half));
                }
            }
        }
    }
}

}  // namespace sk
