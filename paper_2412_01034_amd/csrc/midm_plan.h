// Division of labour of the medium-batch kernel (w4a16_midm.hip): which lists of linears it takes, how many tiles a block
// owns and how its waves share them.  Apart from the kernel, so that the host can walk through it.
#ifndef QAIL_MIDM_PLAN_H
#define QAIL_MIDM_PLAN_H

#include <algorithm>

#include "qail_internal.h"

namespace qail {

constexpr int kMdWaves = 8;
constexpr int kMdStepK = 128;
constexpr int kMdMaxItems = 16;
constexpr int kMdMaxBlocks = 2048;   // blocks of a launch
constexpr size_t kMdLds = 160 * 1024;

enum MdMode { kNib128 = 0, kNib64 = 1, kByte128 = 2 };

struct MdItem {
    const uint32_t* qw;
    const uint16_t* sc;
    const uint32_t* zr;
    const uint16_t* x;
    uint16_t* y;
    int N, K;
    int block_begin;             // first block of the grid that works on this item
    int tiles_base, tiles_rem;   // block b of the item owns tiles_base tiles, one more if b < tiles_rem
    uint8_t wkl;                 // log2 of the K parts
    uint8_t tiles_per_wave;      // column tiles of the wave that has most
    uint16_t table;              // LDS offset of the scales, in 64-byte units
};

struct MdArgs {
    MdItem it[kMdMaxItems];
    uint32_t item_of_block[kMdMaxBlocks / 8];   // 4 bits per block
    int M;
};

// Column tiles of wave `wave` in a block of nt tiles: one more in the first waves where they do not come out even.
__host__ __device__ inline int md_wave_tiles(int nt, int wkl, int wave) {
    const int wc = kMdWaves >> wkl;
    return (nt - (wave >> wkl) + wc - 1) >> (3 - wkl);
}

// Loads of x per wave and step: four per K part and row block, dealt to eight waves; p = log2 of the K parts.
constexpr int md_loads(int rb, int p) { return ((rb << p) + 1) / 2; }

// Steps fetched ahead, by what they cost in registers: each is C (bytes: 2 C) loads of codes and NL of x.  Three variants
// have a step less than that leaves room for: with it the compiler spilled four to eight registers, inside the loop (4096 x 11008
// at M = 32 24.6 -> 22.0 us without, 12288 x 4096 of bytes at M = 56 25.4 -> 22.1).
constexpr int md_depth(int mode, int rb, int c, int nl) {
    const int per_step = (c * (mode == kByte128 ? 2 : 1) + nl) * 4;
    const int room = 256 - 80 - 8 * c * rb - 8 * rb - (mode == kNib64 ? 4 * c + 28 : 0);   // beside the sums, the operands and the addresses
    const bool less = (mode == kNib128 && ((rb == 2 && c == 1 && nl == 8) || (rb == 4 && c == 1 && nl == 8))) ||
                      (mode == kByte128 && rb == 4 && c == 2 && nl == 8);
    return (room / per_step >= 6 ? 6 : room / per_step < 2 ? 2 : room / per_step) - (less ? 1 : 0);
}
constexpr int kMdMostTiles = 4 * kMdWaves;   // of a block, times its K parts
// The variants there are: what fits the registers, of that what some list makes use of.  Groups of 64 are the GEMM's above
// M = 48.  Many tiles of bytes and few rows of x wait for HBM with one K part as with several.
constexpr bool md_variant(int mode, int rb, int c, int p) {
    const int nl = md_loads(rb, p);
    return c <= 4 && c * rb <= (mode == kNib64 ? 9 : 12) && nl <= 8 && (nl <= 4 || c <= 2) && (mode != kNib64 || rb <= 3) &&
           (mode != kByte128 || p == 0 || c <= rb + 1);
}

// How an item is divided when its blocks own up to nt tiles.
struct MdPlan {
    float us;      // what such a block takes
    int wkl, c;
    size_t lds, table;
};

struct MdShape {
    int mode, rb;   // 16-row blocks of x
};

// The time of a block, fitted to 120 (shape, M) pairs: the launch with its start and end, and per step a barrier, the x that a
// wave stages and the tiles of the two waves of a SIMD.  A block that streams its codes at its share of the memory's rate
// (20 KB a microsecond) takes no less.
inline MdPlan md_plan(const MdShape& s, int K, int nt) {
    MdPlan best;
    best.us = -1.f;
    const int S = K / kMdStepK, groups = s.mode == kNib64 ? 2 : 1, G = S * groups;
    const bool bytes = s.mode == kByte128;
    const size_t tables = (size_t)nt * 16 * (G * 2 + (bytes ? 0 : (G + 7) / 8 * 4));
    const float stream = (float)nt * (float)K * (bytes ? 16.f / 20000.f : 8.f / 20000.f);
    // (more K parts have more column tiles a wave: past kMdMostTiles there is no variant)
    for (int wkl = 0; wkl <= 3 && (1 << wkl) <= S && nt << wkl <= kMdMostTiles; ++wkl) {
        const int c = ((nt << wkl) + kMdWaves - 1) / kMdWaves, nl = md_loads(s.rb, wkl);
        if (!md_variant(s.mode, s.rb, c, wkl)) continue;
        const size_t table = (((size_t)s.rb << wkl) * (2 * 4096 + 2 * groups * 64) + 63) / 64 * 64;
        const size_t lds = std::max(table + tables, (size_t)kMdWaves * c * s.rb * 1024);
        if (lds > kMdLds) continue;
        const float tiles = (float)c + (float)(nt << wkl) * (1.f / kMdWaves);   // of the wave that has most and of an average one: a SIMD has two waves
        const float step = 0.5f + 0.03f * (float)(s.rb * nl) + 0.065f * (float)s.rb * tiles * (groups == 2 ? 1.5f : 1.f);
        const float us = 6.5f + std::max((float)((S + (1 << wkl) - 1) >> wkl) * step, stream);
        if (best.us < 0.f || us < best.us) best = MdPlan{us, wkl, c, lds, table};
    }
    return best;
}

inline int md_mode(const qail_wdesc& d, bool b8) { return b8 ? kByte128 : d.group_size == 64 ? kNib64 : kNib128; }

// The division of a launch: tiles per block of each item.  Starting from one, the block that would still be the shortest
// with another tile gets it, until one block per CU is enough.  Lists that do not get there (a block has at most four column
// tiles a wave) are left to the other kernels: a second round of blocks, mostly a nearly empty one, costs as much as the first
// (152064 x 3584 in groups of 64 at M = 8 94 us there, 130 in two rounds; bytes at M = 32 155 against 191).
struct MdDivision {
    MdShape s;
    MdPlan plan[kMdMaxItems];
    int tiles[kMdMaxItems], blocks[kMdMaxItems];
    float us;
};

inline bool md_divide(const qail_w4a16_item* items, int count, int M, bool b8, MdDivision* v) {
    v->s.mode = md_mode(items[0].d, b8);
    v->s.rb = (M + 15) / 16;   // at most 4
    const int cus = std::min(device_cu_count(), kMdMaxBlocks);
    int nt[kMdMaxItems], used = 0;
    MdPlan next[kMdMaxItems];
    for (int i = 0; i < count; ++i) {
        v->tiles[i] = (items[i].d.N + 15) / 16;
        // (fewer tiles than this a block need not try: one block per CU could not serve the item alone)
        nt[i] = std::max(1, (v->tiles[i] + cus - 1) / cus);
        v->plan[i] = md_plan(v->s, items[i].d.K, nt[i]);
        if (v->plan[i].us < 0.f) return false;
        next[i] = md_plan(v->s, items[i].d.K, nt[i] + 1);
        used += (v->tiles[i] + nt[i] - 1) / nt[i];
    }
    while (used > cus) {
        int best = -1;
        for (int i = 0; i < count; ++i)
            if (next[i].us >= 0.f && nt[i] < v->tiles[i] && (best < 0 || next[i].us < next[best].us)) best = i;
        if (best < 0) return false;
        used -= (v->tiles[best] + nt[best] - 1) / nt[best];
        v->plan[best] = next[best];
        ++nt[best];
        used += (v->tiles[best] + nt[best] - 1) / nt[best];
        next[best] = md_plan(v->s, items[best].d.K, nt[best] + 1);
    }
    v->us = 0.f;
    for (int i = 0; i < count; ++i) {
        v->blocks[i] = (v->tiles[i] + nt[i] - 1) / nt[i];
        // the tiles as the blocks share them evenly
        const int most = (v->tiles[i] + v->blocks[i] - 1) / v->blocks[i];
        if (most != nt[i]) v->plan[i] = md_plan(v->s, items[i].d.K, most);
        v->us = std::max(v->us, v->plan[i].us);
    }
    return true;
}

inline double md_bytes(const qail_wdesc& d, int mode) { return (double)d.N * d.K * (mode == kByte128 ? 1.0 : 0.5); }

// Whether the kernel beats those that took these items before, by what was measured of both (layers of several
// widths in one call and single linears of 500 to 65000 rows and 256 to 28672 k, M = 5 .. 64; us, new buffers from call to call):
//   * groups of 128 and bytes up to M = 32: the small-batch kernel loses where its x takes several passes over K, so the
//     passes of an item, weighted by its bytes, decide.  Nibbles up to M = 16 from two passes on (4096 x 11008 at M = 16
//     20.9 -> 17.5; one pass, 4096 x 4096: 8.7 against 9.5), as long as there are 200 MB or less for each pass that is saved: over the
//     rest of the stream that kernel is 2 to 3 % faster (428 MB and 2.6 passes at M = 8 105 against 111; 3.4 passes at M = 16
//     116 -> 111).  Above M = 16 from 1.3 (M = 24, the 7B layer 42.8 -> 37.8; one pass, 2048 x 2048: a fifth slower), bytes from
//     1.2 (the layer at M = 8 / 32 53.0 -> 44.3 / 64.0 -> 49.3; one pass, 4096 x 4096 at M = 8: a tenth slower);
//   * otherwise the matrix-core GEMM, which takes 13.5 us, 1.3 per further item and a microsecond per 3 MB (bytes: 3.3; at 3.0
//     8192 x 28672 at M = 48 went from 80 to 83), measured on the low side: M = 48 the layer 56.2 -> 45.2, with bytes 73.9 -> 54.5;
//     one 4096 x 11008, whose K the GEMM divides among blocks, 23.3 against 31.6.  Groups of 64 stay below 49 rows (layers of
//     1024 to 2048 channels at M = 48 a third faster, most single linears at M = 49 slower) and need no comparison up to 16 (the
//     7B layer 54.5 -> 40.8; 4096 x 4096 14.5 -> 9.6; at M = 32 54.7 -> 46.7).
enum class MdAnswer { no, yes, by_time };
inline MdAnswer md_wanted(const qail_w4a16_item* items, int count, int M, int mode, double bytes) {   // what needs no division
    if (mode == kNib64) return M <= 16 ? MdAnswer::yes : M > 48 ? MdAnswer::no : MdAnswer::by_time;
    if (M > 32) return MdAnswer::by_time;
    double passes = 0;
    for (int i = 0; i < count; ++i) passes += md_bytes(items[i].d, mode) * smallm_passes(M, items[i].d.K);
    passes /= bytes;
    const bool better = mode == kByte128 ? passes >= 1.2 : M > 16 ? passes >= 1.3 : passes >= 2.0 && (passes - 1.0) * 2.0e8 >= bytes;
    return better ? MdAnswer::yes : MdAnswer::no;
}
inline bool md_beats_gemm(float us, int count, int mode, double bytes) {
    const double more = mode == kByte128 ? 0.0 : std::max(0.0, bytes - 60.0e6) / 9.0e6;   // nibbles: a larger share of it expansion
    return us <= 13.5 + 1.3 * (count - 1) + bytes / (mode == kByte128 ? 3.3e6 : 3.0e6) + more;
}

inline bool md_supports(const qail_wdesc& d, int M, bool b8) {
    if (M < 5 || M > 64 || d.K % kMdStepK != 0 || (d.group_size != 128 && (b8 || d.group_size != 64))) return false;
    if ((d.K / d.group_size) % 2 != 0) return false;   // the scales of a row are whole words
    return (unsigned long long)d.N * d.K / (b8 ? 1 : 2) <= 0x7FFFFFFFull && (unsigned long long)M * d.K * 2 <= 0x7FFFFFFFull;
}

// How many of the leading items of the list the kernel takes (0: none), and their division.
inline int md_take(const qail_w4a16_item* items, int count, int M, bool b8, MdDivision* v) {
    int n = 0;   // items of one group size share a launch
    while (n < count && n < kMdMaxItems && items[n].d.group_size == items[0].d.group_size && md_supports(items[n].d, M, b8)) ++n;
    if (n == 0) return 0;
    const int mode = md_mode(items[0].d, b8);
    double bytes = 0;
    for (int i = 0; i < n; ++i) bytes += md_bytes(items[i].d, mode);
    const MdAnswer answer = md_wanted(items, n, M, mode, bytes);   // (before the division: the search for one takes microseconds)
    if (answer == MdAnswer::no || !md_divide(items, n, M, b8, v)) return 0;
    return answer == MdAnswer::yes || md_beats_gemm(v->us, n, mode, bytes) ? n : 0;
}

}  // namespace qail

#endif
