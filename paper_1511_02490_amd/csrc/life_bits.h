// Game of Life on one bit per cell: the arithmetic of the kernels that make several generations per
// launch.  Cells are 0 or 1 (the library's precondition), so 32 of them fit a register and a
// generation is bitwise logic on whole words: 14 operations for 32 cells (gfx950 has three-input
// bitwise operations; the sums of three below are one each), where adding packed bytes takes about
// 12 for 4.  Bytes become bits when a tile is loaded and bits become bytes when it is stored, which
// is paid once per launch and not once per generation.
#pragma once
#include "tile_kernel.h"

namespace sk {

// 16 cells in bytes (each 0 or 1) -> 16 bits, the first cell in bit 0.
__device__ __forceinline__ uint32_t pack_cells(any_word4 v) {
    const uint32_t lo = __builtin_amdgcn_udot4(v.y, 0x80402010u, __builtin_amdgcn_udot4(v.x, 0x08040201u, 0u, false), false);
    const uint32_t hi = __builtin_amdgcn_udot4(v.w, 0x80402010u, __builtin_amdgcn_udot4(v.z, 0x08040201u, 0u, false), false);
    return lo | (hi << 8);
}
// ... and back: four cells from bits 4 k .. 4 k + 3.  (The product's terms fall on distinct bits.)
__device__ __forceinline__ uint32_t unpack_cells(uint32_t bits, int k) {
    return __umul24((bits >> (4 * k)) & 0xfu, 0x00204081u) & 0x01010101u;
}
__device__ __forceinline__ uint4 unpack_cells16(uint32_t bits) {
    return make_uint4(unpack_cells(bits, 0), unpack_cells(bits, 1), unpack_cells(bits, 2), unpack_cells(bits, 3));
}

// The first n < 16 of 16 cells in bytes, a row's last ones: in pieces of 8, 4, 2 and 1.  (One by one they were a
// third of a launch: eight generations of 300 x 300, of which a row ends with 12 cells, 13.0 us, now 8.1.)
__device__ __forceinline__ void store_first_cells(uint8_t *out, uint4 cells, int n) {
    typedef uint16_t any_half __attribute__((aligned(1), may_alias));
    uint32_t lo = cells.x, hi = cells.y, next = cells.z, last = cells.w;
    if (n & 8) {
        any_word2 v;
        v.x = lo, v.y = hi;
        *reinterpret_cast<any_word2 *>(out) = v;
        out += 8;
        lo = next, hi = last;
    }
    if (n & 4) {
        *reinterpret_cast<any_word *>(out) = lo;
        out += 4;
        lo = hi;
    }
    if (n & 2) {
        *reinterpret_cast<any_half *>(out) = (uint16_t)lo;
        out += 2;
        lo >>= 16;
    }
    if (n & 1) *out = (uint8_t)lo;
}

// Every cell's west (east) neighbour, given the word before (after).
__device__ __forceinline__ uint32_t west_of(uint32_t x, uint32_t before) { return __builtin_amdgcn_alignbit(x, before, 31); }
__device__ __forceinline__ uint32_t east_of(uint32_t x, uint32_t after) { return __builtin_amdgcn_alignbit(after, x, 1); }

// Three-input functions by their truth tables: TABLE is the function of a = 0xf0, b = 0xcc, c = 0xaa.  (Written as
// ordinary logic the compiler makes two operations of a three-way xor, and 27 of a row's 14.)
template <uint32_t TABLE>
__device__ __forceinline__ uint32_t logic3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, TABLE);
}
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return logic3<0xf0 ^ 0xcc ^ 0xaa>(a, b, c); }
__device__ __forceinline__ uint32_t majority(uint32_t a, uint32_t b, uint32_t c) {
    return logic3<(0xf0 & 0xcc) | (0xaa & (0xf0 | 0xcc))>(a, b, c);
}

// One row as its neighbours above and below see it: the cells, and the sum of each cell and its west
// and east neighbours as a two-bit number.
struct LifeBits {
    uint32_t x, h0, h1;
};
__device__ __forceinline__ LifeBits life_bits(uint32_t x, uint32_t west, uint32_t east) {
    return {x, xor3(x, west, east), majority(x, west, east)};
}
// The next generation of mid's cells.  The 3x3 block's sum s (the cell included, 0 .. 9) is
// ones + 2 twos + 4 fours; B3/S23 says alive if s == 3, or s == 4 and the cell is.
__device__ __forceinline__ uint32_t life_next(const LifeBits &up, const LifeBits &mid, const LifeBits &dn) {
    const uint32_t ones = xor3(up.h0, mid.h0, dn.h0), carry = majority(up.h0, mid.h0, dn.h0);
    const uint32_t h = xor3(up.h1, mid.h1, dn.h1);
    const uint32_t twos = carry ^ h;
    const uint32_t fours = logic3<0xf0 ^ (0xcc & 0xaa)>(majority(up.h1, mid.h1, dn.h1), carry, h);
    const uint32_t three_or_four = logic3<~(0xf0 ^ 0xcc) & (0xf0 ^ 0xaa) & 0xff>(ones, twos, fours);
    return logic3<0xf0 & (0xcc | 0xaa)>(three_or_four, ones, mid.x);
}

// The bits of a word whose first cell is matrix column `col` that are matrix cells.
__device__ __forceinline__ uint32_t inside_bits(int col, int cols) {
    const int from = -col, to = cols - col;      // [from, to) are matrix cells
    const uint32_t low = from <= 0 ? ~0u : from >= 32 ? 0u : ~0u << from;
    const uint32_t high = to >= 32 ? ~0u : to <= 0 ? 0u : (1u << to) - 1u;
    return low & high;
}
// The bit of matrix column `at` in such a word, if it is there.
__device__ __forceinline__ uint32_t column_bit(int col, int at) {
    return (unsigned)(at - col) < 32u ? 1u << (at - col) : 0u;
}

// 16 cells of a row from column c0, a multiple of 16, on their way from memory: the load is issued
// without a branch, so that a work-item's loads are all in flight before the first is waited for (one
// after the other, each behind the test of where its cells lie, they were most of a small launch).
// A vector that crosses the end of the row loads the 16 cells that end it; one that lies outside, or
// in a padding row (gr = -1), loads any cells.
struct LifeLoad {
    any_word4 v;
    int skip;        // how many of the loaded cells come before column c0; 16 and more: none is in the matrix
};
template <int B>
__device__ __forceinline__ LifeLoad life_load16(const uint8_t *in, int gr, int c0, int cols) {
    const int at = B == kWrap ? resolve<B>(c0, cols) : c0;
    const int from = max(0, min(at, cols - 16));
    const uint8_t *row = in + (size_t)(gr < 0 ? 0 : gr) * cols;
    return {*reinterpret_cast<const any_word4 *>(row + from), B != kWrap && (gr < 0 || c0 < 0) ? 16 : at - from};
}
// ... and as bits.  Out-of-matrix cells follow the border mode; under CLAMP nobody looks at them.
template <int B>
__device__ __forceinline__ uint32_t life_bits16(const LifeLoad &l, const uint8_t *in, int gr, int cols, uint8_t pad) {
    const uint32_t bits = pack_cells(l.v);
    if (l.skip == 0) return bits;
    uint32_t after = B == kConstant && pad ? 0xffffu : 0u;
    if (l.skip >= 16) return after;
    if (B == kWrap) after = pack_cells(*reinterpret_cast<const any_word4 *>(in + (size_t)gr * cols));
    return (bits >> l.skip) | ((after << (16 - l.skip)) & 0xffffu);
}
// The same for matrices of fewer than 16 columns, cell by cell.
template <int B>
__device__ __forceinline__ uint32_t life_bits16_narrow(const uint8_t *in, int gr, int c0, int cols, uint8_t pad) {
    uint32_t bits = 0;
#pragma unroll 1
    for (int k = 0; k < 16; ++k) {
        const int gc = resolve<B>(c0 + k, cols);
        bits |= (uint32_t)(gr < 0 || gc < 0 ? pad : in[(size_t)gr * cols + gc]) << k;
    }
    return bits;
}

// ---- several generations per launch in local memory -------------------------------------------
// The scheme of temporal_kernel on bits: a workgroup stages its tile with `depth` more rows above and
// below and 16 more cells left and right (the tile starts at bit 16 of a row's first word), and
// ping-pongs between two buffers; what a generation computes within k cells of the rim is stale
// after k generations, and exactly the tile is written.  a.pitch counts words, and a.stage_magic is
// ceil(2^32 / words of a row).
//
// Out-of-matrix cells: WRAP copies evolve like their originals, CONSTANT ones are set back after every
// generation, CLAMP ones are not kept - the rows' sums take the edge cell itself there.
// What bounds a launch of four generations is the launch itself, its loads and its stores; a generation of
// a 128 x 128 tile is one pass of 512 work-items and 0.65 us.  (1001 x 1503 cells, tiles of 128 x 128, CLAMP:
// 30.5 us with packed bytes and a search for clamped cells after every generation, now 6.5 us.  Runs of several launches of
// workgroups of whole wavefronts are made by life_stream_kernel, which may fuse more.)
template <int B, int CR, int MAXT>
__global__ __launch_bounds__(MAXT) void life_temporal_kernel(const TileArgs<OpLife, HaloC<1, 1, 1, 1>> a,
                                                             const int depth) {
    constexpr int CC = 16, HC = 16;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    uint32_t *src = reinterpret_cast<uint32_t *>(lds_raw) + 1;   // one spare word before and after the two buffers
    uint32_t *dst = src + a.plane;

    const int wr = blockDim.y, wc = blockDim.x;
    const int tx = threadIdx.x, ty = threadIdx.y;
    const int tid = ty * wc + tx, nthreads = wr * wc;

    int t = blockIdx.x;
    if (a.xcd_chunk > 0) t = (t & 7) * a.xcd_chunk + (t >> 3);
    if (t >= a.n_tiles) return;
    const int tile_r = t / a.tiles_c, tile_c = t - tile_r * a.tiles_c;
    const int rows = a.rows, cols = a.cols, nw = a.pitch;
    const int th = wr * CR, tw = wc * CC;
    const int r0 = tile_r * th, c0 = tile_c * tw;
    const int row_first = r0 - depth, col_first = c0 - HC;
    const int ER = min(th, rows - r0) + 2 * depth;

    // a word is two vectors of 16 cells
    constexpr int kBatch = 2;
    if (cols >= 16) {
        for (int at = tid; at < ER * nw; at += kBatch * nthreads) {
            LifeLoad v[kBatch][2];
            int gr[kBatch];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const int item = min(at + b * nthreads, ER * nw - 1);      // (beyond the last: the last again)
                const int i = (int)__umulhi((unsigned)item, a.stage_magic);
                const int col = col_first + (item - i * nw) * 32;
                gr[b] = resolve<B>(row_first + i, rows);
                v[b][0] = life_load16<B>(a.in, gr[b], col, cols);
                v[b][1] = life_load16<B>(a.in, gr[b], col + 16, cols);
            }
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const uint32_t word = life_bits16<B>(v[b][0], a.in, gr[b], cols, a.pad) |
                                      (life_bits16<B>(v[b][1], a.in, gr[b], cols, a.pad) << 16);
                if (at + b * nthreads < ER * nw) src[at + b * nthreads] = word;
            }
        }
    } else {
        for (int at = tid; at < ER * nw; at += nthreads) {
            const int i = (int)__umulhi((unsigned)at, a.stage_magic);
            const int col = col_first + (at - i * nw) * 32, gr = resolve<B>(row_first + i, rows);
            src[at] = life_bits16_narrow<B>(a.in, gr, col, cols, a.pad) |
                      (life_bits16_narrow<B>(a.in, gr, col + 16, cols, a.pad) << 16);
        }
    }
    __syncthreads();

    auto load_row = [&](const uint32_t *p, uint32_t first, uint32_t last) {
        const uint32_t x = p[0];
        uint32_t w = west_of(x, p[-1]), e = east_of(x, p[1]);
        if (B == kClamp) {
            w = (w & ~first) | (x & first);
            e = (e & ~last) | (x & last);
        }
        return life_bits(x, w, e);
    };
    auto next = [&](const LifeBits &up, const LifeBits &mid, const LifeBits &dn, int gr) {
        if (B == kClamp) return life_next(gr == 0 ? mid : up, mid, gr == rows - 1 ? mid : dn);
        return life_next(up, mid, dn);
    };
    // Items of a generation: a word column x a group of R rows, as many groups as one pass of the workgroup has
    // work-items for.
    const int groups = max(1, (int)__umulhi((unsigned)nthreads, a.stage_magic));
    const int R = (ER - 2 + groups - 1) / groups;
    for (int k = 1; k < depth; ++k) {
        for (int item = tid; item < groups * nw; item += nthreads) {
            const int g = (int)__umulhi((unsigned)item, a.stage_magic);
            const int q = item - g * nw, col = col_first + q * 32;
            int i = k + g * R;
            const int end = min(i + R, ER - k);
            if (i >= end) continue;
            const uint32_t first = column_bit(col, 0), last = column_bit(col, cols - 1), keep = inside_bits(col, cols);
            int off = i * nw + q;
            LifeBits up = load_row(src + off - nw, first, last), mid = load_row(src + off, first, last);
            for (; i < end; ++i, off += nw) {
                const LifeBits dn = load_row(src + off + nw, first, last);
                uint32_t res = next(up, mid, dn, row_first + i);
                if (B == kConstant) {
                    const uint32_t in = (unsigned)(row_first + i) < (unsigned)rows ? keep : 0u;
                    res = (res & in) | (a.pad ? ~in : 0u);
                }
                dst[off] = res;
                up = mid;
                mid = dn;
            }
        }
        __syncthreads();
        uint32_t *tmp = src;
        src = dst;
        dst = tmp;
    }

    // last generation: the tile's own cells.  Work-item (ty, tx) owns rows ty*CR.. and the vector of 16
    // cells 1 + tx, half a word
    const int c = c0 + tx * CC;
    const int q = (1 + tx) >> 1, half = ((1 + tx) & 1) * 16;
    const uint32_t first = column_bit(col_first + q * 32, 0), last = column_bit(col_first + q * 32, cols - 1);
    const uint32_t *p = src + (depth + ty * CR) * nw + q;
    if (c >= cols) return;
    LifeBits up = load_row(p - nw, first, last), mid = load_row(p, first, last);
#pragma unroll
    for (int cr = 0; cr < CR; ++cr) {
        const int r = r0 + ty * CR + cr;
        if (r >= rows) break;
        const LifeBits dn = load_row(p + (cr + 1) * nw, first, last);
        const uint4 o = unpack_cells16(next(up, mid, dn, r) >> half);
        uint8_t *out = a.out + (size_t)r * cols + c;
        if (c + CC <= cols) {
            store_word4(out, o, a.store);
        } else {
            store_first_cells(out, o, cols - c);
        }
        up = mid;
        mid = dn;
    }
}

}  // namespace sk
