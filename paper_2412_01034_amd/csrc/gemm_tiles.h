// Index arithmetic of the matrix-core GEMM (w4a16_gemm.hip) that has to hold for every size it accepts, apart
// from the kernel so that the host can walk through it: where the weight loads of a step read, and which block
// works on which tile.
#ifndef QAIL_GEMM_TILES_H
#define QAIL_GEMM_TILES_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qail {

__host__ __device__ constexpr int step_k(int bits) { return bits == 4 ? 128 : 64; }       // k per step: 64 bytes of codes per row
__host__ __device__ constexpr int ring_stages(int bits) { return bits == 4 ? 3 : 4; }     // steps in LDS, so many minus one ahead

// Codes.  A lane loads 16 bytes, piece 0..3 of the step's 64, of weight row n (row_words 4-byte words, at least
// 8): offset of the row's piece, plus that of the step that begins at k0.  Pieces past the end of K are
// loaded all the same, from inside the row (their scale is 0): from its first step, and where the row is
// shorter than a step (nibbles, K = 64: 32 bytes) from its last piece.
__host__ __device__ inline uint32_t code_offset(uint32_t n, uint32_t row_words, uint32_t piece) {
    const uint32_t last = row_words / 4u - 1u;
    return n * row_words * 4u + 16u * (piece < last ? piece : last);
}
__host__ __device__ inline uint32_t code_step_offset(uint32_t k0, uint32_t piece, uint32_t K, int bits) {
    return k0 + piece * 128u / (uint32_t)bits < K ? k0 * (uint32_t)bits / 8u : 0u;
}

// The aligned 4-byte word that holds group grp's scale (zero-point) of the weight row at byte offset `row`.  N G is even
// for every linear the kernel takes, so the word of the last scale ends with the tensor.
__host__ __device__ inline uint32_t scale_word_offset(uint32_t row, uint32_t grp) { return (row + grp * 2u) & ~3u; }
__host__ __device__ inline uint32_t zero_word_offset(uint32_t row, uint32_t grp) { return row + grp / 8u * 4u; }

constexpr int kPadK = 128;   // rows of the fp16 copy of x are padded to this
__host__ __device__ inline int round_up(int v, int m) { return (v + m - 1) / m * m; }

// How a linear's output tiles are dealt to its blocks.  Tiles are numbered with m running fastest.  The first
// `whole` tiles are dealt whole, P at a time (a round); the K steps of the others are dealt as units (one
// K step of one tile): block b of P owns the units [b * units / P, (b + 1) * units / P).  The linear is worked
// on by blocks [block_begin, block_begin + P) of the grid.
struct TilePlan {
    int Tm, tiles, steps, whole;   // row tiles, all tiles, K steps of a tile
    int block_begin, P;
};

// First unit of block b when `units` units are dealt to P blocks, and the block that owns unit u.
__host__ __device__ inline long long first_unit(long long b, long long units, int P) { return b * units / P; }
__host__ __device__ inline int owner_of(long long u, long long units, int P) { return (int)(((u + 1) * P - 1) / units); }

// The same for the second kernel, which starts with five of them: P is at most kMaxGemmBlocks, so below kUnits32 units every
// product fits 32 bits (only a K of a million reaches that line), and a 32-bit division is a sixth of the 64-bit one's
// 150 instructions, most of which wait for the one before.
constexpr int kMaxGemmBlocks = 512;     // upper bound of the grid (the workspace has two slots per block)
constexpr long long kUnits32 = (1ll << 32) / kMaxGemmBlocks;
__host__ __device__ inline int first_unit_quick(int b, long long units, int P) {
    return units < kUnits32 ? (int)((uint32_t)b * (uint32_t)units / (uint32_t)P) : (int)first_unit(b, units, P);
}
__host__ __device__ inline int owner_of_quick(int u, long long units, int P) {
    return units < kUnits32 ? (int)((((uint32_t)u + 1u) * (uint32_t)P - 1u) / (uint32_t)units) : owner_of(u, units, P);
}

// The segments (a tile and a range of its K steps) of one block, one after the other: its whole tiles, then
// its units.  tile_m: rows of a tile; Kpad: padded length of a row of x (fp16).
struct TileDealer {
    struct Segment {
        int tm, tn, ka, steps;   // row tile, column tile, first K step, K steps
        bool first_shared;       // the block's first unit is among them
    };
    TilePlan tp;
    int wtile, unit, unit0, unit1, whole_cols;
    bool x_fits_l2, pair_order, eight_rows;

    __host__ __device__ __forceinline__ TileDealer(const TilePlan& plan, int bid, int tile_m, int Kpad) : tp(plan) {
        const long long units = (long long)(tp.tiles - tp.whole) * tp.steps;
        unit0 = unit = (int)first_unit(bid, units, tp.P);
        unit1 = (int)first_unit(bid + 1, units, tp.P);
        // Whole tiles are numbered with m running fastest, so consecutive tiles share their weight columns.
        // Where the x of all row tiles fits an L2 beside the weights passing through (2.5 MB), the blocks of
        // an XCD take consecutive tiles: workgroup b of the launch runs on XCD b mod 8, so this block's rank
        // among its linear's blocks is counted XCD by XCD.  A weight tile is then fetched by one or two L2s
        // instead of one per row tile.  Measured on a decoder layer's four linears as one launch: 2 % faster
        // with three row tiles (M = 272, 288), 3-5 % slower with two (M = 160 .. 256), which stay as they
        // were.  (Taller linears: see the dealing of eight row tiles below.)
        x_fits_l2 = tp.Tm >= 3 && (long long)tp.Tm * tile_m * Kpad * 2 <= 2560 * 1024;
        // Taller linears with an even number of row tiles, where the x of two row tiles fits: the same
        // ranks, and the whole tiles are walked pair of row tiles by pair of row tiles (inside a pair column
        // by column), so that an XCD's consecutive tiles are two row tiles of a few columns.
        // Only where a round of the linear's blocks stays inside a pair (a share of a launch: all XCDs then
        // share the pair's x at the same time and each has weight columns of its own; a linear on the whole
        // grid has several pairs at once and is 7-15 % slower this way, see the dealing of eight row tiles).
        // Measured on a decoder layer's four linears as one launch: 0.4 / 1.1 / 1.4 % faster with 4 / 8 / 16 row
        // tiles, 1.1 % slower with 6, which keeps the launch order.
        whole_cols = tp.whole / tp.Tm;
        pair_order = !x_fits_l2 && tp.Tm >= 4 && (tp.Tm & 3) == 0 && 2ll * tile_m * Kpad * 2 <= 2560 * 1024 && tp.P <= 2 * whole_cols;
        eight_rows = tp.Tm == 8 && !x_fits_l2 && (tp.P & 15) == 0 && (tp.block_begin & 7) == 0;
        wtile = bid;
        if (x_fits_l2 || pair_order) {
            const int q = tp.block_begin & 7, mine = (q + bid) & 7;
            int before = 0;
            for (int x = 0; x < 8; ++x) {
                const int first = (x - q) & 7;   // the first of the linear's blocks on XCD x
                const int count = first < tp.P ? (tp.P - first + 7) >> 3 : 0;
                if (x < mine) before += count;
            }
            wtile = before + ((bid - ((mine - q) & 7)) >> 3);
        }
    }

    // K steps of all segments (before the first one is taken).
    __host__ __device__ __forceinline__ int total_steps() const {
        int total = unit1 - unit0;
        for (int w = wtile; w < tp.whole; w += tp.P) total += tp.steps;
        return total;
    }

    // false: there is none left
    __host__ __device__ __forceinline__ bool next(Segment& sg) {
        int tile;
        sg.first_shared = false;
        if (wtile < tp.whole) {
            tile = wtile;
            sg.ka = 0;
            sg.steps = tp.steps;
            wtile += tp.P;
        } else if (unit < unit1) {
            const int tt = unit / tp.steps;
            tile = tp.whole + tt;
            sg.ka = unit - tt * tp.steps;
            sg.steps = tp.steps - sg.ka < unit1 - unit ? tp.steps - sg.ka : unit1 - unit;
            sg.first_shared = unit == unit0;
            unit += sg.steps;
        } else {
            return false;
        }
        sg.tm = tile % tp.Tm;
        sg.tn = tile / tp.Tm;
        if (pair_order && tile < tp.whole) {
            // (a last, partial column among the whole tiles keeps its order)
            if (tile < whole_cols * tp.Tm) {
                const int pair = tile / (2 * whole_cols), rem = tile - pair * 2 * whole_cols;
                sg.tm = 2 * pair + (rem & 1);
                sg.tn = rem >> 1;
            }
        } else if (eight_rows && tile < tp.whole) {
            // Whole tiles of a linear that is eight row tiles high and has the grid to itself: in launch order
            // the eight row tiles that share a weight tile would sit on eight XCDs and every L2 would fetch
            // every weight column.  A round's P tiles (P / 8 columns) are dealt instead so that an XCD works on
            // two row tiles (their x fits its L2) and on every other column: a weight tile is then fetched by
            // four L2s, not eight.
            // Columns go in pairs: the last round may hold an odd number of them, and its last one keeps the
            // launch order.
            const int round = tile / tp.P, begin = round * tp.P, idx = tile - begin;
            const int in_round = tp.whole - begin < tp.P ? tp.whole - begin : tp.P;
            if (idx < (in_round & ~15)) {
                const int xcd = idx & 7, j = idx >> 3;
                sg.tm = 2 * (xcd & 3) + (j & 1);
                sg.tn = round * (tp.P >> 3) + 2 * (j >> 1) + (xcd >> 2);
            }
        }
        return true;
    }
};

// The plan of one linear on `cus` blocks, with tiles of rows x cols and K steps of step_k.
inline TilePlan plan_tiles(int M, int N, int K, int rows, int cols, int step_k, bool split_tail, int cus) {
    TilePlan tp{};
    tp.Tm = (M + rows - 1) / rows;
    tp.tiles = tp.Tm * ((N + cols - 1) / cols);
    tp.steps = (K + step_k - 1) / step_k;
    tp.whole = split_tail ? tp.tiles / cus * cus : tp.tiles;
    const int tail = tp.tiles - tp.whole;
    const long long units = (long long)tail * tp.steps;
    tp.P = tp.whole >= cus ? cus : tp.whole;
    if (tail > 0 && tp.P < cus) {   // here whole == 0
        // Blocks that share a tile take at least 128 k of it, and 256 k of byte codes: a block's sums cost the second
        // kernel as much however short its part is.  Bytes, one / two / four 64-k steps per block: 128 x 11008 at
        // M = 40 24.3 / 18.8 / 16.8 us, 512 x 4096 at M = 96 19.7 / 15.6 / 14.4, 1024 x 4096 at M = 128 17.7 / 17.7 / 15.5.
        long long parts = units;
        if (step_k == 64) parts = units / 4 > tail ? units / 4 : tail;
        tp.P = parts < cus ? (int)parts : cus;
    }
    return tp;
}

// Tile width and the treatment of the last, incomplete round of tiles, for a linear that has
// `cus` blocks to itself.
inline void choose_tile(int bits, int rows, int M, int N, int Kpad, int cus, bool alone, bool narrow_only, int* wn_out, bool* split_out) {
    // Measured on the four linears of a 7B decoder layer at M = 288 and 1024 (256 CUs), one launch each:
    //   * a round or more of wide tiles: wide tiles, and the incomplete last round is dealt in
    //     K steps only when it is short (a fuller one is cheaper left as it is: blocks that
    //     share tiles pay for slots and a second kernel, and a chip that is not full clocks higher);
    //   * between half a round and a round of wide tiles: wide tiles, whole;
    //   * less: narrow tiles (twice as many), dealt in K steps when K is long or the tiles are few.
    // A linear that shares the launch with others has only its share of the blocks, which it must
    // keep busy to the end because the others cannot use them: less than a round of wide tiles is
    // dealt in K steps, and as narrow tiles when M is a single tile high (measured 3-6 % faster than
    // wide ones at M = 17 .. 128, 2-9 % slower at M = 200 and 288).
    //
    // Bytes, narrow tiles: their steps are half as deep and two blocks that share a tile part with at least
    // four of them each (see plan_tiles), so sharing pays from shorter K on.  Measured on single linears of
    // N = 64 .. 22016 and K = 1024 .. 11008 at M = 34 .. 1024, whole / shared: 64 x 4096 at M = 40 30.8 / 12.6 us,
    // 128 x 4096 at M = 288 37.9 / 15.1, 4096 x 4096 at M = 288 38.5 / 29.7 and, above the line, M = 640 43.6 / 45.9;
    // 2048 x 1024 at M = 96 15.2 / 13.4 and, above the line, 4096 x 1024 at M = 96 15.0 / 16.3, M = 640 17.8 / 21.7;
    // 4096 x 11008 at M = 640 109.5 / 91.1.
    const int Tm = (M + rows - 1) / rows, t1 = Tm * ((N + 127) / 128), t2 = Tm * ((N + 255) / 256), k128 = Kpad / kPadK;
    const bool few_bytes = k128 >= 64 || (t1 * 2 <= cus && k128 >= 16) || (t1 * 16 <= cus && k128 >= 8);
    int wn = 2;
    bool split = false;
    if (N <= 128 || narrow_only) {
        wn = 1;
        if (bits == 4) split = k128 >= 64;
        else split = t1 >= cus ? (t1 % cus) * 5 <= cus * 2 : !alone || few_bytes;
    } else if (t2 >= cus) {
        split = (t2 % cus) * 5 <= cus * 2;
    } else if (!alone) {
        wn = M <= rows ? 1 : 2;
        split = true;
    } else if (t2 * 2 <= cus) {
        wn = 1;
        // in K steps when K is long, or when whole narrow tiles would leave half of the CUs idle
        // (measured on single linears at M = 48 .. 288: the out projection 27 -> 19 us at M = 64,
        // 37 -> 25 us at M = 128; with more tiles than that the shared tiles cost more than they give)
        split = bits == 8 ? few_bytes : k128 >= 64 || (t2 * 4 <= cus && k128 >= 16);
    }
    *wn_out = wn;
    *split_out = split;
}

// Tile height: the multiple of 32 rows (at most 128) that pads M least
inline int tile_rows(int M) {
    if (M <= 96) return round_up(M, 32);
    return round_up(M, 96) < round_up(M, 128) ? 96 : 128;
}


}  // namespace qail

#endif
