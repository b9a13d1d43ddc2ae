// The stencil skeleton's kernel (Section 2 and Figure 1 of the paper): the matrix is cut
// into workgroups of w_r x w_c work-items; each workgroup stages its tile plus the perimeter
// border region in local memory (LDS), waits, and every work-item folds the customising
// function over the border region of its cells.
//
// Beyond the paper's one-element-per-work-item mapping, a work-item may own a CR x CC block
// of adjacent cells (register blocking): the workgroup then covers (w_r*CR) x (w_c*CC)
// elements, rows of the window are pulled from LDS once and reused by all the cells they
// touch, and with CC*sizeof(T) = 16 bytes HBM and LDS traffic moves as 128-bit accesses.
#pragma once
#include "stencil_ops.h"

#include <type_traits>

namespace sk {

// Scalar loads of up to four words each of a table in constant memory.  (Nothing writes a table while a kernel reads it,
// which the constant address space says; scalar loads want no more than 4-byte alignment.)
template <class W, int CNT>
__device__ __forceinline__ void load_scalars(W (&dst)[CNT], const __attribute__((address_space(4))) W *p) {
    typedef W four __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
    for (int i = 0; i < CNT; i += 4) {
        if (i + 4 <= CNT) {
            const four t = *(const __attribute__((address_space(4))) four *)(p + i);
            dst[i] = t.x, dst[i + 1] = t.y, dst[i + 2] = t.z, dst[i + 3] = t.w;
        } else {
#pragma unroll
            for (int j = i; j < CNT; ++j) dst[j] = p[j];
        }
    }
}

template <class Op, class Halo, bool Static = Halo::kStatic>
struct WeightStore;
// Compile-time region: the weight table travels in the kernel arguments (scalar registers).
template <class Op, class Halo>
struct WeightStore<Op, Halo, true> {
    static constexpr int kCount = Op::kWeights ? (Halo::N + Halo::S + 1) * (Halo::E + Halo::W + 1) : 1;
    using W = typename weight_type_of<Op>::type;
    W v[kCount];
    __device__ __forceinline__ W operator[](int k) const { return Op::kWeights ? v[k] : W(0); }
    // Entries k .. k + CNT - 1, k the same in all lanes, from the kernel's arguments, which lie in constant memory.
    template <int CNT>
    __device__ __forceinline__ void load(W (&dst)[CNT], unsigned k) const;
};
// Run-time region: table in device memory (uniform index -> scalar loads).
template <class Op, class Halo>
struct WeightStore<Op, Halo, false> {
    using Wt = typename weight_type_of<Op>::type;
    using W = typename std::conditional<sizeof(Wt) == 4, Wt, float>::type;
    const W *v;
    __device__ __forceinline__ W operator[](int k) const { return Op::kWeights ? v[k] : W(0); }
    // Entry k, k the same in all lanes, by a scalar load whatever went before.  (The operator's is one only where nothing before
    // it may write memory, as loads straight into local memory and changes of priority may for all the compiler knows.  The
    // tap-by-tap fold by vector loads: 12 taps on 3209 x 2416 doubles 73 us, by scalar ones 55.)
    __device__ __forceinline__ W scalar(int k) const { return ((const __attribute__((address_space(4))) W *)v)[k]; }
    // Entries k .. k + CNT - 1, k the same in all lanes.
    template <int CNT>
    __device__ __forceinline__ void load(W (&dst)[CNT], unsigned k) const {
        load_scalars(dst, (const __attribute__((address_space(4))) W *)(v + k));
    }
};

// How vectors of output cells are stored (store_word4).
enum class Store : int { kPlain, kNonTemporal, kThrough };

template <class Op, class Halo>
struct TileArgs {
    const typename Op::T *in;
    typename out_type_of<Op>::type *out;
    int rows, cols;
    int tiles_c;     // tiles per row of tiles
    int n_tiles;
    int xcd_chunk;   // > 0: tiles are dealt to the 8 XCDs in contiguous chunks of this many
    int pitch;       // LDS tile pitch, in staged elements
    int plane;       // elements per LDS plane (tile rows x pitch)
    unsigned stage_magic;   // for the division by the items of a staged row: see row_of_item
    Store store;     // how vectors of output cells are stored
    typename Op::T pad;
    float scalar0;
    Halo halo;
    WeightStore<Op, Halo> w;
};

// (TileArgs is the kernels' first argument.  Through the member itself every entry would be a load with an address of its own.)
template <class Op, class Halo>
template <int CNT>
__device__ __forceinline__ void WeightStore<Op, Halo, true>::load(W (&dst)[CNT], unsigned k) const {
    const auto *args = (const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr();
    load_scalars(dst, (const __attribute__((address_space(4))) W *)(args + __builtin_offsetof(TileArgs<Op, Halo>, w)) + k);
}

// item / d, the items of a staged row, by a multiply: floor((item + 1) floor((2^32 - 1) / d) / 2^32), exact where
// (item + 1) d <= 2^32.  (The usual ceil(2^32 / d) needs no addition and 33 bits for d = 1: a workgroup one work-item wide
// under a region of one column.  The temporal Life kernel, whose rows have two words and more, uses that.)
constexpr unsigned row_magic(unsigned d) { return 0xffffffffu / d; }
__device__ __forceinline__ unsigned row_of_item(unsigned item, unsigned magic) { return __umulhi(item + 1u, magic); }

__host__ __device__ constexpr int round_up(int x, int m) { return (x + m - 1) / m * m; }
__host__ __device__ constexpr int round_down(int x, int m) { return x / m * m; }

// 16-byte moves between LDS and register arrays (16-byte aligned on the LDS side).
template <class E, int CNT>
__device__ __forceinline__ void load_vec(E (&dst)[CNT], const E *src) {
    static_assert(sizeof(E) * CNT % 16 == 0, "vector moves are whole 16-byte words");
    constexpr int NV = sizeof(E) * CNT / 16;
    uint4 tmp[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) tmp[k] = reinterpret_cast<const uint4 *>(src)[k];
    __builtin_memcpy(dst, tmp, sizeof(tmp));
}
template <class E, int CNT>
__device__ __forceinline__ void store_vec(E *dst, const E (&src)[CNT]) {
    static_assert(sizeof(E) * CNT % 16 == 0, "vector moves are whole 16-byte words");
    constexpr int NV = sizeof(E) * CNT / 16;
    uint4 tmp[NV];
    __builtin_memcpy(tmp, src, sizeof(tmp));
#pragma unroll
    for (int k = 0; k < NV; ++k) reinterpret_cast<uint4 *>(dst)[k] = tmp[k];
}
// The same between global memory and registers, from and to any element's address: gfx950 moves a
// vector of 4, 8 or 16 bytes that starts at any byte (the types say so, or the compiler would assume
// natural alignment), so a row of any length is moved in vectors and only its last, partial one
// element by element.  (Rows that do not start at multiples of 16 bytes were moved one element at a
// time before: a 7x7 sum on 3001 x 4099 floats 43.8 -> 38.5 us, four Life generations per launch on
// 1001 x 1503 bytes 34.3 -> 31.4 us, a 36-tap int32 sum on 2500 x 3003 35.0 -> 32.7 us.)
typedef uint32_t any_word __attribute__((aligned(1), may_alias));
typedef uint32_t any_word2 __attribute__((ext_vector_type(2), aligned(1), may_alias));
typedef uint32_t any_word4 __attribute__((ext_vector_type(4), aligned(1), may_alias));
template <class E, int CNT>
__device__ __forceinline__ void load_global(E (&dst)[CNT], const E *src) {
    if constexpr (sizeof(E) * CNT == 4) {       // four byte cells that are widened to floats afterwards
        const uint32_t tmp = *reinterpret_cast<const any_word *>(src);
        __builtin_memcpy(dst, &tmp, 4);
    } else {
        static_assert(sizeof(E) * CNT % 16 == 0, "vector moves are whole 16-byte words");
        constexpr int NV = sizeof(E) * CNT / 16;
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const any_word4 tmp = reinterpret_cast<const any_word4 *>(src)[k];
            __builtin_memcpy(reinterpret_cast<char *>(dst) + 16 * k, &tmp, 16);
        }
    }
}
// Stores of output cells are optionally non-temporal: they are not read again by the launch that
// writes them, and on matrices beyond the caches keeping them out of the way of the input pays
// (measured on a plain copy: +20 % on 256 MiB, nothing on 64 MiB).
// Or they are written through (kThrough), by the kernels that make several applications per launch and by tiles and direct kernels
// of their own (WrittenThrough): what plain stores leave dirty in the eight L2 caches, 4 MiB each, is written back when the kernel ends, with nothing beside it; written through it
// is on its way while the rest computes, and stays in the cache for the next launch.  (Plain / through: four Life
// generations on 4096^2 in local memory 11.4 / 9.5 us; a launch of four heat steps there 33.5 / 33.1.  Small outputs
// pay for it at the end of the last workgroups: a launch of two heat steps on 1024^2 9.4 / 10.0.  And what a store leaves of a
// cache line is written to memory by itself.  Each launcher in variants.h and variants_register_tiles.hip draws its line; for single
// applications tile_goes_through.)  The two wait states keep what follows off the stored registers: the compiler counts them only
// after its own stores.  Nothing reads the output in the same launch.
template <Store S>
__device__ __forceinline__ void store_word4(void *dst, uint4 v) {
    any_word4 t;
    t.x = v.x, t.y = v.y, t.z = v.z, t.w = v.w;
    if constexpr (S == Store::kNonTemporal)
        __builtin_nontemporal_store(t, reinterpret_cast<any_word4 *>(dst));
    else if constexpr (S == Store::kThrough)
        asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(dst), "v"(t));
    else
        *reinterpret_cast<any_word4 *>(dst) = t;
}
// The same, chosen at run time, for kernels that store at one place, once per cell row.  (The compiler makes one store of
// two that differ in nothing else, and a plain one: the empty statements keep the two branches apart.  28 taps on 8192^2
// floats, a pass on matrices not used before: 165 us with one plain store, 115 us with non-temporal ones.  In a march of
// many unrolled steps the statements cost registers and cross-lane moves that would be part of an addition: the marching
// kernels are compiled for either kind.)
__device__ __forceinline__ void store_word4(void *dst, uint4 v, bool nt) {
    if (nt) {
        asm volatile("");
        store_word4<Store::kNonTemporal>(dst, v);
        asm volatile("");
    } else {
        store_word4<Store::kPlain>(dst, v);
    }
}
__device__ __forceinline__ void store_word4(void *dst, uint4 v, Store how) {
    if (how == Store::kThrough)
        store_word4<Store::kThrough>(dst, v);
    else
        store_word4(dst, v, how == Store::kNonTemporal);
}
template <class E, int CNT, class Store>
__device__ __forceinline__ void store_words_of(E *dst, const E (&src)[CNT], Store store) {
    static_assert(sizeof(E) * CNT % 16 == 0, "vector moves are whole 16-byte words");
    constexpr int NV = sizeof(E) * CNT / 16;
    uint4 tmp[NV];
    __builtin_memcpy(tmp, src, sizeof(tmp));
#pragma unroll
    for (int k = 0; k < NV; ++k) store(reinterpret_cast<unsigned char *>(dst) + 16 * k, tmp[k]);
}
template <class E, int CNT, class How>
__device__ __forceinline__ void store_out_vec(E *dst, const E (&src)[CNT], How how) {
    store_words_of(dst, src, [&](void *p, uint4 v) { store_word4(p, v, how); });
}
template <Store S, class E, int CNT>
__device__ __forceinline__ void store_out_vec(E *dst, const E (&src)[CNT]) {
    store_words_of(dst, src, [](void *p, uint4 v) { store_word4<S>(p, v); });
}

// What a cell keeps while one row of its region goes by (operators that fold a row at a time).
struct NoRowState {};
template <class Op, bool = Op::kRowFold>
struct row_state_of { using type = NoRowState; };
template <class Op>
struct row_state_of<Op, true> { using type = typename Op::RowState; };

// Cross-lane moves inside a wavefront: the value the lane one below / one above holds.
// (Lane 0 has no lane below and lane 63 none above; they get 0 - the move's bound control -
// and must look elsewhere.)
__device__ __forceinline__ uint32_t from_lane_below(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138 /* wave_shr:1 */, 0xf, 0xf, true);
}
__device__ __forceinline__ uint32_t from_lane_above(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130 /* wave_shl:1 */, 0xf, 0xf, true);
}

// Columns staged left / right of the tile: the border region's extent, widened to whole
// 16-byte vectors when the work-items move vectors.
template <int CC>
__host__ __device__ constexpr int staged_halo(int h) { return CC == 1 ? h : round_up(h, CC); }

// stage_tile for a tile that needs no border resolution: `src` is the matrix cell under the tile's first one.
// Staging is bound by the latency of its loads and by the instructions that find their addresses, and the
// latter were a third of a light stencil's: the general walk resolves a row and four columns per vector and
// multiplies out both addresses; here an item is two adds, a compare and two selects.  (7x7 sum on 3001 x 4099
// floats 38.5 -> 36.3 us, 5x5 sum on 4096^2 doubles 59.5 -> 56.9 us.)
//
// Cells that are staged as they are go from memory to LDS without a stop in registers (16 bytes a lane, which land at the
// wavefront's own base and 16 times the lane, as item k does): every load of a work-item is in flight at once, and nothing
// waits to write.  Together with the priority of staging wavefronts (tile_kernel), which gets a new workgroup's loads out
// before others' folds go on, on fresh matrices, before / now: 28 run-time taps on 8192^2 floats 102 -> 98 us, 7x7 on
// 3001 x 4099 38.9 -> 37.0, 36 taps on 2500 x 3003 int32 26.1 -> 24.3; 5x5 on 4096^2 doubles 55.3 -> 54.9.
template <class Op, int CC>
constexpr bool staged_as_loaded() {
    using T = typename Op::T;
    return std::is_same<T, typename Op::L>::value && Op::kPlanes == 1 && CC * sizeof(T) == 16 && sizeof(T) >= 4;
}
typedef __attribute__((address_space(1))) const void global_bytes;
typedef __attribute__((address_space(3))) void local_bytes;

template <class Op, int CC>
__device__ __forceinline__ void stage_inside(typename Op::L *tile, int plane, int n_items, const typename Op::T *src, int cols,
                                             int total, unsigned magic, int tid, int nthreads) {
    using T = typename Op::T;
    using L = typename Op::L;
    constexpr int NP = Op::kPlanes;
    constexpr int kBatch = 4;
    const unsigned i0 = row_of_item(tid, magic), di = row_of_item(nthreads, magic);
    unsigned q = tid - i0 * n_items;
    const unsigned dq = nthreads - di * n_items;
    const unsigned row_bytes = (unsigned)cols * (unsigned)sizeof(T);
    unsigned off = i0 * row_bytes + q * (unsigned)(CC * sizeof(T));
    const unsigned step = di * row_bytes + dq * (unsigned)(CC * sizeof(T));       // one more pass of the workgroup, same row of items
    const unsigned carry = row_bytes - (unsigned)n_items * (unsigned)(CC * sizeof(T));   // ... and into the next row
    const char *base = reinterpret_cast<const char *>(src);
    if constexpr (staged_as_loaded<Op, CC>()) {
        char *to = reinterpret_cast<char *>(tile) + 16 * __builtin_amdgcn_readfirstlane(tid & ~63);
        for (int at = tid; at < total; at += nthreads) {
            __builtin_amdgcn_global_load_lds((global_bytes *)(base + off), (local_bytes *)to, 16, 0, 0);
            to += 16 * nthreads;
            off += step;
            q += dq;
            if (q >= (unsigned)n_items) {
                q -= n_items;
                off += carry;
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);      // vmcnt(0): the barrier that follows does not wait for these loads
        return;
    }
    for (int at = tid; at < total; at += kBatch * nthreads) {
        T v[kBatch][CC];
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            if (at + b * nthreads < total) load_global(v[b], reinterpret_cast<const T *>(base + off));
            off += step;
            q += dq;
            if (q >= (unsigned)n_items) {
                q -= n_items;
                off += carry;
            }
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            if (at + b * nthreads >= total) continue;
            L sv[NP][CC];
            Op::template stage_vec<CC>(v[b], sv);
#pragma unroll
            for (int p = 0; p < NP; ++p) store_vec(tile + p * plane + (at + b * nthreads) * CC, sv[p]);
        }
    }
}

// Stages `n_rows` rows of a tile into LDS with border resolution (Section 2).  Tile row i is
// matrix row row_first + i, tile column j is matrix column col_first + j; each plane of the
// staged values has `pitch` elements per row.  The rows are walked as one linear sequence of
// 16-byte vectors (single elements when CC = 1), work-item k taking items k, k + n, k + 2n, ...
// so that the halo columns cost a fraction of a pass rather than a whole extra pass with most
// lanes idle.  Vectors starting at or beyond matrix column `col_end` are not needed and skipped.
// `magic` belongs to pitch / CC items per row (row_of_item).
template <class Op, int B, int CC, bool INSIDE = true>
__device__ __forceinline__ void stage_tile(typename Op::L *tile, int plane, int pitch, const typename Op::T *in,
                                           int rows, int cols, int row_first, int col_first, int n_rows,
                                           int col_end, typename Op::T pad, unsigned magic, int tid,
                                           int nthreads) {
    using T = typename Op::T;
    using L = typename Op::L;
    constexpr int NP = Op::kPlanes;
    const int n_items = pitch / CC;   // per staged row
    // A tile that lies inside the matrix with its border region (nearly all of them on a large matrix) has nothing
    // to resolve: the items of the linear walk are loaded from a running 32-bit offset and, the tile being rows of
    // n_items vectors, land in LDS at their own index.  (INSIDE: whether the kernel has that walk.)
    const bool inside = INSIDE && CC > 1 && row_first >= 0 && row_first + n_rows <= rows && col_first >= 0 && col_first + pitch <= cols &&
                        (uint64_t)n_rows * cols * sizeof(T) < (1ull << 32);
    if constexpr (INSIDE && CC > 1) {
        if (inside) {
            stage_inside<Op, CC>(tile, plane, n_items, in + (size_t)row_first * cols + col_first, cols, n_rows * n_items, magic,
                                 tid, nthreads);
            return;
        }
    }
    int i = (int)row_of_item(tid, magic);
    int q = tid - i * n_items;
    const int di = (int)row_of_item(nthreads, magic), dq = nthreads - di * n_items;
    // Vectors are taken kBatch at a time: the loads of a batch are all issued before the first of
    // them is waited for and written to LDS, so a work-item with several items pays one memory
    // round trip per batch, not one per item.  (Single elements gain nothing from it.)
    constexpr int kBatch = CC == 1 ? 1 : 4;
    while (i < n_rows) {
        T v[kBatch][CC];
        int at_i[kBatch], at_q[kBatch];
        bool have[kBatch];
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            at_i[b] = i;
            at_q[b] = q;
            have[b] = i < n_rows;
            if (have[b]) {
                const int gr = resolve<B>(row_first + i, rows);
                if constexpr (CC == 1) {
                    const int gc = resolve<B>(col_first + q, cols);
                    v[b][0] = (gr < 0 || gc < 0) ? pad : in[(size_t)gr * cols + gc];
                } else {
                    const int gc0 = col_first + q * CC;
                    have[b] = gc0 < col_end;
                    if (have[b]) {
                        if (gr >= 0 && gc0 >= 0 && gc0 + CC <= cols) {
                            load_global(v[b], in + (size_t)gr * cols + gc0);
                        } else {
#pragma unroll
                            for (int k = 0; k < CC; ++k) {
                                const int gc = resolve<B>(gc0 + k, cols);
                                v[b][k] = (gr < 0 || gc < 0) ? pad : in[(size_t)gr * cols + gc];
                            }
                        }
                    }
                }
            }
            i += di;
            q += dq;
            if (q >= n_items) {
                q -= n_items;
                ++i;
            }
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            if (!have[b]) continue;
            if constexpr (CC == 1) {
                L sv[NP];
                Op::stage(v[b][0], sv);
#pragma unroll
                for (int p = 0; p < NP; ++p) tile[p * plane + at_i[b] * pitch + at_q[b]] = sv[p];
            } else {
                L sv[NP][CC];
                Op::template stage_vec<CC>(v[b], sv);
#pragma unroll
                for (int p = 0; p < NP; ++p) store_vec(tile + p * plane + at_i[b] * pitch + at_q[b] * CC, sv[p]);
            }
        }
    }
}

// ---- the fold over a run-time region ------------------------------------------------------------------
// A window row is read from local memory once, for all the cell rows of a work-item that it touches: window row wi
// is region row wi - cr of cell row cr.  What a row (or a chunk of one) needs is requested while the one before it is
// folded, and waited for before the next requests go out: scalar loads return out of order, so a wait for a vector
// from local memory waits for every weight under way as well, and one that was requested in between would be waited
// for at once.
__device__ __forceinline__ void wait_for_lds_and_scalars() {
    __builtin_amdgcn_s_waitcnt(0xc07f);          // lgkmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
}

// Regions of WC columns, compiled: a row is straight-line code, WC weights per region row in scalar registers.
// (Bound by arithmetic and by what of staging and storing it does not cover.  Before, every tap was a branch and waited
// for its own weight, and every cell row read its own window: 9 columns x 7 rows on 7135 x 456 floats 22.6 -> 13.1 us,
// 6 x 6 int32 on 2500 x 3003 32.0 -> 22.5 us, sin/cos over 7 x 4 on 3344 x 6704 152 -> 81 us.)
template <class Op, class Halo, int CR, int CC, int WC>
__device__ __forceinline__ void fold_columns(typename Op::State (&st)[CR][CC], const TileArgs<Op, Halo> &a,
                                             const typename Op::L *window, int hn, int hw, int wrows) {
    using L = typename Op::L;
    using Wt = typename WeightStore<Op, Halo>::W;
    constexpr int NP = Op::kPlanes;
    constexpr int kColumns = round_up(WC - 1 + CC, CC);              // window columns read, whole vectors
    constexpr bool kAhead = NP == 1;         // two planes of two rows do not fit the registers
    // weights of the last CR region rows kept, as far as scalar registers go and the moves from row to row pay
    constexpr bool kRing = CR * WC <= 40 && !(CR == 4 && WC <= 4);
    const int window_rows = CR - 1 + wrows;
    struct Row {
        L v[NP][kColumns];
        Wt w[WC];                            // of region row wi, the first cell row's
    };
    auto load_row = [&](Row &r, int wi) {
#pragma unroll
        for (int p = 0; p < NP; ++p) load_vec(r.v[p], window + p * a.plane + wi * a.pitch);
        if constexpr (kRing) a.w.load(r.w, (unsigned)(min(wi, wrows - 1) * WC));
    };
    Wt older[CR][WC];                        // ... of region row wi - cr, the cr-th's
    auto step = [&](Row &cur, Row &ahead, int wi) {
        if constexpr (kAhead) {
            wait_for_lds_and_scalars();
            if (wi + 1 < window_rows) load_row(ahead, wi + 1);
        } else {
            load_row(cur, wi);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int cr = 0; cr < CR; ++cr) {
            const int k = wi - cr;
            if ((unsigned)k >= (unsigned)wrows) continue;
            [[maybe_unused]] typename row_state_of<Op>::type rs[CC] = {};
            Wt own[WC];
            if constexpr (!kRing) a.w.load(own, (unsigned)(k * WC));
#pragma unroll
            for (int kk = 0; kk < WC; ++kk) {
                const Wt w = !kRing ? own[kk] : cr == 0 ? cur.w[kk] : older[cr][kk];
#pragma unroll
                for (int cc = 0; cc < CC; ++cc) {
                    L parts[NP];
#pragma unroll
                    for (int p = 0; p < NP; ++p) parts[p] = cur.v[p][kk + cc];
                    if constexpr (Op::kRowFold)
                        Op::row_visit(st[cr][cc], rs[cc], kk, w, Op::combine(parts));
                    else
                        Op::visit(st[cr][cc], k - hn, kk - hw, w, Op::combine(parts));
                }
            }
            if constexpr (Op::kRowFold) {
#pragma unroll
                for (int cc = 0; cc < CC; ++cc) Op::row_end(st[cr][cc], rs[cc], WC, k, wrows);
            }
        }
        if constexpr (kRing) {
#pragma unroll
            for (int cr = CR - 1; cr > 0; --cr)
#pragma unroll
                for (int kk = 0; kk < WC; ++kk) older[cr][kk] = cr == 1 ? cur.w[kk] : older[cr - 1][kk];
        }
    };
    Row even, odd;
    if constexpr (kAhead) load_row(even, 0);
#pragma unroll
    for (int cr = 0; cr < CR; ++cr)
#pragma unroll
        for (int kk = 0; kk < WC; ++kk) older[cr][kk] = Wt(0);
    for (int wi = 0; wi < window_rows; wi += kAhead ? 2 : 1) {
        step(even, odd, wi);
        if constexpr (kAhead)
            if (wi + 1 < window_rows) step(odd, even, wi + 1);
    }
}

// Any number of columns (compiling each up to the largest, 65, would not pay), BW at a time: the same for a block of
// columns of a row, the last of which may have fewer.
template <class Op, class Halo, int CR, int CC>
__device__ __forceinline__ void fold_blocks(typename Op::State (&st)[CR][CC], const TileArgs<Op, Halo> &a,
                                            const typename Op::L *window, int hn, int hw, int wrows, int wcols) {
    using L = typename Op::L;
    using Wt = typename WeightStore<Op, Halo>::W;
    constexpr int NP = Op::kPlanes;
    constexpr int BW = 8, VL = 16 / (int)sizeof(L);
    constexpr int kColumns = round_up(BW - 1 + CC, VL);
    constexpr bool kAhead = NP == 1;         // (two planes: see fold_columns)
    const int window_rows = CR - 1 + wrows;
    struct Block {
        L v[NP][kColumns];
        Wt w[CR][BW];                        // of region row wi - cr (of any row where there is none)
    };
    // (The weights beyond a row's last column are read, where the table has room, and not used; the cells beyond the
    // last one needed are not read.)
    auto load_block = [&](Block &r, int wi, int kk) {
        const int need = min(BW, wcols - kk) - 1 + CC;
#pragma unroll
        for (int i = 0; i < kColumns; i += VL) {
            if (i >= need) break;
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                L part[VL];
                load_vec(part, window + p * a.plane + wi * a.pitch + kk + i);
#pragma unroll
                for (int k = 0; k < VL; ++k) r.v[p][i + k] = part[k];
            }
        }
        if constexpr (kAhead) {
#pragma unroll
            for (int cr = 0; cr < CR; ++cr) a.w.load(r.w[cr], (unsigned)(max(0, min(wi - cr, wrows - 1)) * wcols + kk));
        }
    };
    [[maybe_unused]] typename row_state_of<Op>::type rs[CR][CC] = {};
    int wi = 0, kk0 = 0;                     // the block at hand: window row, first column
    auto step = [&](Block &cur, Block &ahead) {
        const bool in_row = kk0 + BW < wcols;
        const int wi1 = in_row ? wi : wi + 1, kk1 = in_row ? kk0 + BW : 0;
        if constexpr (kAhead) {
            wait_for_lds_and_scalars();
            if (wi1 < window_rows) load_block(ahead, wi1, kk1);
        } else {
            load_block(cur, wi, kk0);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int cr = 0; cr < CR; ++cr) {
            const int k = wi - cr;
            if ((unsigned)k >= (unsigned)wrows) continue;
            Wt own[BW];
            if constexpr (!kAhead) a.w.load(own, (unsigned)(k * wcols + kk0));
            auto taps = [&](int n_taps) {
#pragma unroll
                for (int t = 0; t < BW; ++t) {
                    if (t >= n_taps) break;
                    const Wt w = kAhead ? cur.w[cr][t] : own[t];
#pragma unroll
                    for (int cc = 0; cc < CC; ++cc) {
                        L parts[NP];
#pragma unroll
                        for (int p = 0; p < NP; ++p) parts[p] = cur.v[p][t + cc];
                        if constexpr (Op::kRowFold)
                            Op::row_visit(st[cr][cc], rs[cr][cc], kk0 + t, w, Op::combine(parts));
                        else
                            Op::visit(st[cr][cc], k - hn, kk0 + t - hw, w, Op::combine(parts));
                    }
                }
            };
            if (kk0 + BW <= wcols)
                taps(BW);
            else
                taps(wcols - kk0);
            if constexpr (Op::kRowFold) {
                if (!in_row) {
#pragma unroll
                    for (int cc = 0; cc < CC; ++cc) Op::row_end(st[cr][cc], rs[cr][cc], wcols, k, wrows);
                }
            }
        }
        wi = wi1;
        kk0 = kk1;
    };
    Block even, odd;
    if constexpr (kAhead) load_block(even, 0, 0);
    while (wi < window_rows) {
        step(even, odd);
        if constexpr (kAhead) {
            if (wi >= window_rows) break;
            step(odd, even);
        }
    }
}

// The same tap by tap, every cell row with its own window: the cells of a row need window columns kk .. kk + CC - 1 for
// tap kk, i.e. two aligned vectors per chunk of CC taps, of which one is the previous chunk's.  Work-items of four and more
// rows have the arithmetic between two weights to cover the wait for the next, and no registers for more
// (17 x 17 on 2500 x 3000 floats, four rows: 91 us, 8 columns at a time 105; eight rows: 99 and 132).  And where a region
// has few taps, the windows of all cell rows are requested at once, where the other folds wait for one after the other.
template <class Op, class Halo, int CR, int CC>
__device__ __forceinline__ void fold_taps(typename Op::State (&st)[CR][CC], const TileArgs<Op, Halo> &a,
                                          const typename Op::L *window, int hn, int hw, int wrows, int wcols) {
    using L = typename Op::L;
    constexpr int NP = Op::kPlanes;
    for (int i = 0; i < wrows; ++i) {
        [[maybe_unused]] typename row_state_of<Op>::type rs[CR][CC] = {};
        L va[CR][NP][CC], vb[CR][NP][CC];
        auto load_chunk = [&](L (&v)[CR][NP][CC], int j) {
#pragma unroll
            for (int cr = 0; cr < CR; ++cr)
#pragma unroll
                for (int p = 0; p < NP; ++p) load_vec(v[cr][p], window + p * a.plane + (i + cr) * a.pitch + CC * j);
        };
        // taps CC * j .. CC * j + CC - 1: `lo` holds window columns CC * j .., `hi` the next CC
        auto chunk = [&](const L (&lo)[CR][NP][CC], L (&hi)[CR][NP][CC], int j) {
            if (CC * j + 1 < wcols) load_chunk(hi, j + 1);
#pragma unroll
            for (int t = 0; t < CC; ++t) {
                const int kk = CC * j + t;
                if (kk >= wcols) continue;
                const auto w = a.w.scalar(i * wcols + kk);
#pragma unroll
                for (int cr = 0; cr < CR; ++cr)
#pragma unroll
                    for (int cc = 0; cc < CC; ++cc) {
                        L parts[NP];
#pragma unroll
                        for (int p = 0; p < NP; ++p)
                            parts[p] = t + cc < CC ? lo[cr][p][(t + cc) % CC] : hi[cr][p][(t + cc) % CC];
                        if constexpr (Op::kRowFold)
                            Op::row_visit(st[cr][cc], rs[cr][cc], kk, w, Op::combine(parts));
                        else
                            Op::visit(st[cr][cc], i - hn, kk - hw, w, Op::combine(parts));
                    }
            }
        };
        load_chunk(va, 0);
        for (int j = 0; CC * j < wcols; j += 2) {
            chunk(va, vb, j);
            if (CC * (j + 1) < wcols) chunk(vb, va, j + 1);
        }
        if constexpr (Op::kRowFold) {
#pragma unroll
            for (int cr = 0; cr < CR; ++cr)
#pragma unroll
                for (int cc = 0; cc < CC; ++cc) Op::row_end(st[cr][cc], rs[cr][cc], wcols, i, wrows);
        }
    }
}

template <class Op, int B, class Halo, int CR, int CC, int MAXT>
__global__ __launch_bounds__(MAXT) void tile_kernel(const TileArgs<Op, Halo> a) {
    using O = typename out_type_of<Op>::type;
    using L = typename Op::L;
    constexpr int NP = Op::kPlanes;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    L *tile = reinterpret_cast<L *>(lds_raw);   // NP planes of a.plane elements each

    const int wr = blockDim.y, wc = blockDim.x;
    const int tx = threadIdx.x, ty = threadIdx.y;

    int t = blockIdx.x;
    if (a.xcd_chunk > 0) t = (t & 7) * a.xcd_chunk + (t >> 3);
    if (t >= a.n_tiles) return;
    const int tile_r = t / a.tiles_c, tile_c = t - tile_r * a.tiles_c;

    const Halo h = a.halo;
    const int hn = h.n(), hs = h.s(), he = h.e(), hw = h.w();
    const int th = wr * CR, tw = wc * CC;
    const int r0 = tile_r * th, c0 = tile_c * tw;
    // columns staged west of the tile: under a run-time region exactly the region's (the fold wants the region's
    // west edge at a vector's start), else whole vectors
    const int hwa = folds_by_rows<Halo>::value ? hw : staged_halo<CC>(hw);
    const int pitch = a.pitch;
    const int rows = a.rows, cols = a.cols;
    // the whole tile height is staged, also where the last tile hangs over the matrix edge (those
    // rows resolve like any other out-of-matrix row): no window row ever needs a range check
    const int TH = th + hn + hs;

    // Under a run-time region, eight rows of cells per work-item: nine items and more per work-item, and no gain from
    // finding their addresses sooner (2048 x 4096 floats, 1 x 7 taps, resolved / not: 16.2 / 17.7 us; 7 x 4 taps 21.2 / 22.4).
    constexpr bool kInside = Halo::kStatic || CR < 8 || NP > 1;
    // (Not where single elements are staged: with scalar weights, WeightStore, it gained 1 % there and cost up to 9; and before
    // the fold it made the weights vector loads: 25 taps on 3280 x 4064 doubles, one cell per work-item, 393 us, without 240;
    // 49 on 2145 x 2816 floats, two cells, 62 and 47.)
    if constexpr (CC > 1) __builtin_amdgcn_s_setprio(3);
    stage_tile<Op, B, CC, kInside>(tile, a.plane, pitch, a.in, rows, cols, r0 - hn, c0 - hwa, TH, cols + he, a.pad,
                                   a.stage_magic, ty * wc + tx, wr * wc);
    if constexpr (CC > 1) __builtin_amdgcn_s_setprio(0);
    __syncthreads();

    // ---- fold the customising function over the border region ----------------------------
    const int lr0 = ty * CR, lc0 = tx * CC;
    if (r0 + lr0 >= rows || c0 + lc0 >= cols) return;

    typename Op::State st[CR][CC];
#pragma unroll
    for (int cr = 0; cr < CR; ++cr)
#pragma unroll
        for (int cc = 0; cc < CC; ++cc) Op::init(st[cr][cc]);

    if constexpr (!folds_by_rows<Halo>::value) {
        constexpr int N = Halo::N, S = Halo::S, E = Halo::E, W = Halo::W;
        constexpr int HWA = staged_halo<CC>(W);
        constexpr int VL = CC == 1 ? 1 : (16 / (int)sizeof(L) < 1 ? 1 : 16 / (int)sizeof(L));
        constexpr int LO = round_down(HWA - W, VL);
        constexpr int HI = round_up(HWA + CC + E, VL);
        constexpr int WW = HI - LO;
        constexpr int WCOLS = E + W + 1;
        // window rows stream through registers; row wi feeds cell-row cr with dr = wi - N - cr
#pragma unroll
        for (int wi = 0; wi < CR + N + S; ++wi) {
            L row[NP][WW];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const L *src = tile + p * a.plane + (lr0 + wi) * pitch + lc0 + LO;
                if constexpr (CC == 1) {
#pragma unroll
                    for (int k = 0; k < WW; ++k) row[p][k] = src[k];
                } else {
                    load_vec(row[p], src);
                }
            }
            auto value_at = [&](int i) {
                L parts[NP];
#pragma unroll
                for (int p = 0; p < NP; ++p) parts[p] = row[p][i];
                return Op::combine(parts);
            };
#pragma unroll
            for (int cr = 0; cr < CR; ++cr) {
                const int dr = wi - N - cr;
                if (dr < -N || dr > S) continue;
#pragma unroll
                for (int cc = 0; cc < CC; ++cc)
                    fold_row<Op>(
                        st[cr][cc], dr, dr + N, N + S + 1, W, E, [&](int dc) { return a.w[(dr + N) * WCOLS + dc + W]; },
                        [&](int dc) { return value_at(HWA - LO + cc + dc); });
            }
        }
    } else {
        // Run-time region: the cells of a work-item walk through the region together, so that a
        // tap's weight (a uniform, scalar load) is fetched once for all of them; every cell still
        // sees its taps in row-major order.
        const int wcols = he + hw + 1, wrows = hn + hs + 1;
        if constexpr (CC > 1) {
            // The tile is staged from the region's west edge: tap kk of cell cc is window column kk + cc, and a
            // work-item's window starts at a vector.
            const L *const window = tile + lr0 * pitch + lc0;
            // (which of the three serves a region: region_fold in variants.h)
            if constexpr (Halo::kFold == Fold::taps) {
                fold_taps<Op, Halo, CR, CC>(st, a, window, hn, hw, wrows, wcols);
            } else if constexpr (Halo::kFold == Fold::blocks) {
                fold_blocks<Op, Halo, CR, CC>(st, a, window, hn, hw, wrows, wcols);
            } else if constexpr (Halo::kStatic) {
                int n_rows = wrows;              // (a loop of two rows: unrolled further, rows are read ahead into more registers)
                asm("" : "+s"(n_rows));
                fold_columns<Op, Halo, CR, CC, Halo::E + Halo::W + 1>(st, a, window, hn, hw, n_rows);
            } else {
                static_assert(kCompiledColumns == 9, "a case each");
                switch (wcols) {
#define FOLD_COLUMNS(WC)                                                                                       \
                case WC: fold_columns<Op, Halo, CR, CC, WC>(st, a, window, hn, hw, wrows); break
                FOLD_COLUMNS(1);
                FOLD_COLUMNS(2);
                FOLD_COLUMNS(3);
                FOLD_COLUMNS(4);
                FOLD_COLUMNS(5);
                FOLD_COLUMNS(6);
                FOLD_COLUMNS(7);
                FOLD_COLUMNS(8);
                FOLD_COLUMNS(9);
#undef FOLD_COLUMNS
                }
            }
        } else {
            const L *nw[CR];      // the north-west corner of the region of cell (cr, 0)
#pragma unroll
            for (int cr = 0; cr < CR; ++cr) nw[cr] = tile + (lr0 + cr) * pitch + (hwa - hw) + lc0;
            for (int i = 0; i < wrows; ++i) {
                const int dr = i - hn;
                [[maybe_unused]] typename row_state_of<Op>::type rs[CR][CC] = {};
                for (int k = 0; k < wcols; ++k) {
                    const auto w = a.w[i * wcols + k];
#pragma unroll
                    for (int cr = 0; cr < CR; ++cr)
#pragma unroll
                        for (int cc = 0; cc < CC; ++cc) {
                            L parts[NP];
#pragma unroll
                            for (int p = 0; p < NP; ++p) parts[p] = nw[cr][p * a.plane + i * pitch + k + cc];
                            if constexpr (Op::kRowFold)
                                Op::row_visit(st[cr][cc], rs[cr][cc], k, w, Op::combine(parts));
                            else
                                Op::visit(st[cr][cc], dr, k - hw, w, Op::combine(parts));
                        }
                }
                if constexpr (Op::kRowFold) {
#pragma unroll
                    for (int cr = 0; cr < CR; ++cr)
#pragma unroll
                        for (int cc = 0; cc < CC; ++cc) Op::row_end(st[cr][cc], rs[cr][cc], wcols, i, wrows);
                }
            }
        }
    }

    // ---- store ------------------------------------------------------------------------------
#pragma unroll
    for (int cr = 0; cr < CR; ++cr) {
        const int r = r0 + lr0 + cr;
        if (r >= rows) break;
        O res[CC];
#pragma unroll
        for (int cc = 0; cc < CC; ++cc) res[cc] = Op::finish(st[cr][cc], a.scalar0);
        O *dst = a.out + (size_t)r * cols + c0 + lc0;
        if constexpr (CC > 1) {
            if (c0 + lc0 + CC <= cols) {
                if constexpr (goes_through<Op>::value)
                    store_out_vec<Store::kThrough>(dst, res);
                else
                    store_out_vec(dst, res, a.store == Store::kNonTemporal);
                continue;
            }
        }
#pragma unroll
        for (int cc = 0; cc < CC; ++cc)
            if (c0 + lc0 + cc < cols) dst[cc] = res[cc];
    }
}

}  // namespace sk
