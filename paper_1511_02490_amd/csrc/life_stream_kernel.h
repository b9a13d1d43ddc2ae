// Game of Life, several generations per launch, on bits in registers (the arithmetic: life_bits.h).
//
// A work-item holds RPT rows of one word (32 cells) of the matrix.  16, 32 or 64 adjacent lanes hold adjacent
// words, the lanes' groups rows below each other, and the workgroup so holds a tile.  Per generation a row's
// west and east neighbours come from the adjacent lanes by cross-lane moves, and only the first and the last
// row of every work-item pass through local memory, behind one barrier (two buffers in turn).  What a generation
// computes within k rows or cells of the tile's rim is stale after k generations: `depth` rows above and below
// and a word left and right are not written.  WRAP and CONSTANT borders: a periodic copy evolves like its
// original, a padded cell is set back after every generation.
//
// Between the launches of a run the matrix is kept as bits, rows of whole words: the first launch turns bytes
// into bits, the last one bits into bytes, and the launches between them move an eighth of the bytes.  They are
// bound by the generations' serial chain (a row's sums, the barrier, the rule), not by memory: the tile is cut
// so that the device's wavefronts are filled evenly and its rim repeats as little as possible (life_tile in
// variants.h).
// (100 generations of 4096 x 4096, WRAP, 8 per launch: 282 -> 121 us, before by marching packed bytes down the
// matrix; between two launches in bits one of 8 generations takes 9.3 us, 0.53 each and 5.1 for the launch, its loads and its
// stores.)
#pragma once
#include "life_bits.h"

namespace sk {

constexpr int kLifeStreamMaxDepth = 8;      // (the rim of 32 cells would allow more)
constexpr int kLifeStreamMaxThreads = 256;

struct LifeStreamArgs {
    const void *in;
    void *out;
    int rows, cols, words;       // words per row of a matrix of bits
    int tiles_c, n_tiles;
    int group_shift;             // log2 of the lanes that hold a row of the tile
    int pad;                     // 0 or 1
    int nt_store;
};

template <int B, int RPT, bool IN_BITS, bool OUT_BITS>
__global__ __launch_bounds__(kLifeStreamMaxThreads) void life_stream_kernel(const LifeStreamArgs a, const int depth) {
    static_assert(B == kWrap || B == kConstant, "wrap and constant borders only");
    const int tid = (int)threadIdx.y * (int)blockDim.x + (int)threadIdx.x, nthreads = (int)(blockDim.x * blockDim.y);
    const int G = 1 << a.group_shift, groups = nthreads >> a.group_shift;
    const int rows = a.rows, cols = a.cols;
    const int tile_r = (int)blockIdx.x / a.tiles_c, tile_c = (int)blockIdx.x - tile_r * a.tiles_c;
    const int word = tile_c * (G - 2) - 1 + (tid & (G - 1)), col = word * 32;
    const int tile_rows = groups * RPT - 2 * depth;                    // the rows it writes
    const int row0 = tile_r * tile_rows - depth + (tid >> a.group_shift) * RPT;
    const uint32_t pad = a.pad ? ~0u : 0u;
    const uint32_t inside = inside_bits(col, cols);

    // the matrix rows it loads: under WRAP row0's and, going round, those after it; under CONSTANT any where there is none
    int gr[RPT];
    gr[0] = B == kWrap ? resolve<kWrap>(row0, rows) : max(0, min(row0, rows - 1));
#pragma unroll
    for (int i = 1; i < RPT; ++i) {
        if (B == kWrap)
            gr[i] = gr[i - 1] + 1 == rows ? 0 : gr[i - 1] + 1;
        else
            gr[i] = max(0, min(row0 + i, rows - 1));
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
    // CONSTANT: cells that are not matrix cells hold the padding
    const bool at_border = B == kConstant && (tile_r * tile_rows < depth || tile_r * tile_rows + tile_rows + depth > rows ||
                                              tile_c == 0 || (tile_c + 1) * (G - 2) * 32 + 32 > cols);
    auto pad_outside = [&] {
        if (!at_border) return;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const uint32_t keep = (unsigned)(row0 + i) < (unsigned)rows ? inside : 0u;
            x[i] = (x[i] & keep) | (pad & ~keep);
        }
    };
    pad_outside();

    // a row with its neighbours from the adjacent lanes; what the two ends of a group of lanes get is no
    // neighbour, and stays in the rim
    auto sums = [](uint32_t v) { return life_bits(v, west_of(v, from_lane_below(v)), east_of(v, from_lane_above(v))); };
    __shared__ uint32_t first_rows[2][kLifeStreamMaxThreads], last_rows[2][kLifeStreamMaxThreads];
    const int above_at = max(0, tid - G), below_at = min(tid + G, nthreads - 1);
    for (int k = 0; k < depth; ++k) {
        first_rows[k & 1][tid] = x[0];
        last_rows[k & 1][tid] = x[RPT - 1];
        LifeBits h[RPT];
#pragma unroll
        for (int i = 0; i < RPT; ++i) h[i] = sums(x[i]);
        __syncthreads();
        const uint32_t above = last_rows[k & 1][above_at], below = first_rows[k & 1][below_at];
#pragma unroll
        for (int i = 1; i < RPT - 1; ++i) x[i] = life_next(h[i - 1], h[i], h[i + 1]);
        x[0] = life_next(sums(above), h[0], h[1]);
        x[RPT - 1] = life_next(h[RPT - 2], h[RPT - 1], sums(below));
        pad_outside();
    }

    const int lane = tid & (G - 1), end = min(rows, tile_r * tile_rows + tile_rows);
    if (lane == 0 || lane == G - 1 || word >= a.words) return;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int r = row0 + i;
        if (r < tile_r * tile_rows || r >= end) continue;
        if constexpr (OUT_BITS) {
            static_cast<uint32_t *>(a.out)[(unsigned)(r * a.words + word)] = x[i];
        } else {
            uint8_t *out = static_cast<uint8_t *>(a.out) + (unsigned)(r * cols + col);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const uint4 o = unpack_cells16(x[i] >> (16 * half));
                if (col + 16 * half + 16 <= cols) {
                    store_word4(out + 16 * half, o, a.nt_store != 0);
                } else {
                    const uint32_t w[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
                    for (int b = 0; b < 16; ++b)
                        if (col + 16 * half + b < cols) out[16 * half + b] = (uint8_t)(w[b >> 2] >> (8 * (b & 3)));
                }
            }
        }
    }
}

}  // namespace sk
