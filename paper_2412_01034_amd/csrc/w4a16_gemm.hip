// W4A16 linear for M > 16 on the fp16 matrix cores:
//   y[m][n] = sum_k x[m][k] * (q[n][k] - z[n][k/g]) * s[n][k/g].
//
// Appendix "Analysis": prefill is the compute-heavy stage of the backbone, so this is
// the one W4A16 kernel bound by the matrix pipe rather than by HBM.  The design goal is
// to keep vector-ALU and LDS work per MFMA low:
//
//   * The weights are in LDS as packed codes only.  A wave owns 32 or 64 columns n; lane (c, kb) reads
//     the 8 packed words (64 consecutive k) of row n = c of a 128-k step back from LDS, where a
//     loading wave has put them, and expands one word into the 8 fp16 values one
//     v_mfma_f32_32x32x16_f16 needs from it as A operand:  0x6400 | q is the fp16 number
//     1024 + q and 0x6400 | (q << 4) is 1024 + 16 q, so a v_and_or_b32 yields two codes,
//     one packed add (or fma with 1/16) removes the offset together with the zero-point
//     exactly, and one packed multiply applies the scale: 13 vector operations per word,
//     used by BM / 32 MFMAs.
//   * The activations are staged in LDS once per block, ready for the MFMAs, and every wave reads the
//     whole tile: one 16-byte LDS read per two MFMAs (on 256-column tiles).
//   * fp16 holds every bf16 significand but not its range, so a small kernel first
//     rewrites x per row as fp16 scaled by a power of two (largest magnitude in
//     [2^14, 2^15)), with the k order inside each group of 8 that the expansion above
//     produces (0,4,1,5,2,6,3,7).  Group scales are divided by the power of two of the
//     row's largest scale, which keeps (q - z) * s below 32 in fp16; both powers of two
//     are multiplied back in fp32 at the end.  A weight is therefore rounded once to 11
//     significant bits (the bf16 alternative keeps 8).
//
// kBits = 8 is the 8-bit weight-only variant (Sec. 5.4 deploys the backbone with 8-bit weights
// too): signed bytes, one fp16 scale per group, no zero-point.  A byte q becomes fp16 without a
// conversion: (q ^ 0x80) is q + 128 as an unsigned byte u, and 0x6400 | u is the fp16 number
// 1024 + u, so one XOR per word, one byte permute per pair of codes, a packed add of -1152 (exact)
// and a packed multiply by the scale give (q * s): 14 vector operations per 8 codes.  The codes
// come out in their natural order, so x is stored in natural order for this variant.  A step is
// 64 k deep instead of 128, so that a lane's share of it is two 16-byte pieces as well and the ring
// (four slots of half the depth) fits LDS beside the wide tiles.  With 128-k steps only 128-column
// tiles fitted, on which every MFMA costs one 1 KB fragment read, the LDS's full bandwidth: one
// decoder layer at M = 288 took 213 us with them, 200 with this layout alone.
//
// MFMA operand layout (32x32x16, wave64): lane l supplies row (A) / column (B) l%32 and
// the 8 consecutive k starting at 8*(l/32); it receives D[8*(r/4) + 4*(l/32) + r%4][l%32]
// for r = 0..15.  A = weights (columns n), B = activations (rows m).
#include <algorithm>

#include <atomic>

#include "gemm_tiles.h"
#include "qail_internal.h"

namespace qail {

namespace {

typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_any_t __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x2_any_t __attribute__((ext_vector_type(2), aligned(2)));

constexpr int kRowPad = 128;            // workspace rows are padded to this

constexpr int kGemmBatch = kGemmGroup;  // linears that can share one launch

// ---------------------------------------------------------------------------------------
// Preparation, for up to kGemmBatch linears at once (blockIdx.y): blocks [0, rows) rewrite one
// row of x each, the rest find the power of two of each weight row's largest scale.
struct PrepItem {
    const uint16_t* x;
    const uint16_t* sc;
    uint16_t* xh;
    uint16_t* rscale;   // the powers of two of the rows of x and of the weight rows: exact as bf16
    uint16_t* wmul;
    int N, K, Kpad, G;
};
struct PrepBatch {
    PrepItem it[kGemmBatch];
    int M, rows;   // rows: M padded to whole tiles, what the GEMM reads
    int natural;   // 8-bit codes expand in their natural order, 4-bit ones as 0,4,1,5,2,6,3,7
};

__global__ __launch_bounds__(256) void gemm_prep_kernel(const PrepBatch args) {
    __shared__ uint32_t red[4];
    const int t = threadIdx.x;
    const PrepItem pi = args.it[blockIdx.y];
    const uint16_t* __restrict__ x = pi.x;
    const uint16_t* __restrict__ sc = pi.sc;
    uint16_t* __restrict__ xh = pi.xh;
    uint16_t* __restrict__ rscale = pi.rscale;
    uint16_t* __restrict__ wmul = pi.wmul;
    const int M = args.M, rows = args.rows, N = pi.N, K = pi.K, Kpad = pi.Kpad, G = pi.G;
    if ((int)blockIdx.x >= rows + (N + 31) / 32) return;   // the grid is as wide as the largest linear needs
    if ((int)blockIdx.x < rows) {
        const int m = blockIdx.x;
        uint4* dst = reinterpret_cast<uint4*>(xh + (size_t)m * Kpad);
        if (m >= M) {
            for (int i = t; i < Kpad / 8; i += 256) dst[i] = make_uint4(0, 0, 0, 0);
            if (t == 0) rscale[m] = 0;
            return;
        }
        const uint4* src = reinterpret_cast<const uint4*>(x + (size_t)m * K);
        // the row is read once: a thread keeps its pieces (up to kKeep of them: rows up to 2048 kKeep long) in
        // registers between the search for the largest magnitude and the rewrite; longer rows are read again
        constexpr int kKeep = 6;
        uint4 keep[kKeep];
        uint32_t mx = 0;  // largest magnitude bit pattern (order-preserving for bf16 magnitudes)
#pragma unroll
        for (int r = 0; r < kKeep; ++r) {
            const int i = t + 256 * r;
            keep[r] = i < K / 8 ? src[i] : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < kKeep; ++r) {
            const uint32_t w[4] = {keep[r].x, keep[r].y, keep[r].z, keep[r].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                mx = max(mx, w[j] & 0x7FFFu);
                mx = max(mx, (w[j] >> 16) & 0x7FFFu);
            }
        }
        for (int i = t + 256 * kKeep; i < K / 8; i += 256) {
            const uint4 v = src[i];
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                mx = max(mx, w[j] & 0x7FFFu);
                mx = max(mx, (w[j] >> 16) & 0x7FFFu);
            }
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, o));
        if (t % kWave == 0) red[t / kWave] = mx;
        __syncthreads();
        mx = max(max(red[0], red[1]), max(red[2], red[3]));
        // x * 2^p has its largest magnitude in [2^14, 2^15); p is kept in the normal fp32 range
        const int e = (int)(mx >> 7);  // biased exponent of the largest magnitude
        int p = mx == 0 ? 0 : 141 - e;
        p = p > 126 ? 126 : (p < -126 ? -126 : p);
        const float up = __builtin_bit_cast(float, (uint32_t)(127 + p) << 23);
        if (t == 0) rscale[m] = (uint16_t)((127 - p) << 7);
        auto rewrite = [&](const uint4 v) {
            const uint16_t b[8] = {(uint16_t)v.x, (uint16_t)(v.x >> 16), (uint16_t)v.y, (uint16_t)(v.y >> 16),
                                   (uint16_t)v.z, (uint16_t)(v.z >> 16), (uint16_t)v.w, (uint16_t)(v.w >> 16)};
            uint32_t h[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                h[j] = __builtin_bit_cast(uint16_t, (_Float16)(bf16_bits_to_f32(b[j]) * up));
            // stored order inside the 8: 0,4,1,5,2,6,3,7 (4-bit codes) or as they are (8-bit codes)
            return args.natural
                       ? make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16))
                       : make_uint4(h[0] | (h[4] << 16), h[1] | (h[5] << 16), h[2] | (h[6] << 16), h[3] | (h[7] << 16));
        };
#pragma unroll
        for (int r = 0; r < kKeep; ++r) {
            const int i = t + 256 * r;
            // (a kept piece past the end of the row is zero, and so is its rewrite: the padding up to Kpad)
            if (i < Kpad / 8) dst[i] = rewrite(keep[r]);
        }
        for (int i = t + 256 * kKeep; i < Kpad / 8; i += 256)
            dst[i] = i < K / 8 ? rewrite(src[i]) : make_uint4(0, 0, 0, 0);
        return;
    }
    // 8 lanes per weight row, 32 rows per block.  A row's scales are read as the aligned words that hold them (N G is
    // even, so the last word ends with the tensor), four words of a lane at a time before any is used: with
    // one scale per load and trip a row of 86 groups was eleven trips to memory, one after the other (decoder layer at
    // M = 288, with no rows of x past the tiles: 10.9 -> 9.9 us; at M = 1024 x itself takes the time, 21.9 -> 21.7).
    const int n = ((int)blockIdx.x - rows) * 32 + t / 8;
    const int part = t % 8;
    uint32_t mx = 0;
    if (n < N) {
        const size_t first = (size_t)n * G, last = first + G - 1;
        const uint32_t* const words = reinterpret_cast<const uint32_t*>(sc);
        const size_t w_last = last / 2;
        if (G <= 14) {   // eight words hold the row: one each (65536 x 256 at M = 72, 12.6 -> 12.1 us)
            const size_t w = min(first / 2 + part, w_last);
            const uint32_t v = words[w];
            mx = max(2 * w >= first ? v & 0xFFFFu : 0u, 2 * w + 1 <= last ? v >> 16 : 0u);
        } else {
            for (size_t w0 = first / 2 + part; w0 <= w_last; w0 += 32) {
                uint32_t v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = words[w0 + 8 * e < w_last ? w0 + 8 * e : w_last];   // past the row: its last word again
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const size_t w = w0 + 8 * e < w_last ? w0 + 8 * e : w_last;
                    mx = max(mx, 2 * w >= first ? v[e] & 0xFFFFu : 0u);   // a word at a row's end may hold a neighbour's scale
                    mx = max(mx, 2 * w + 1 <= last ? v[e] >> 16 : 0u);
                }
            }
        }
    }
#pragma unroll
    for (int o = 4; o >= 1; o >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, o));
    if (n < N && part == 0) {
        // scales are positive fp16, at least 2^-14 (a stored subnormal is treated as 2^-14)
        int e = (int)(mx >> 10) & 31;
        e = e < 1 ? 1 : e;
        wmul[n] = (uint16_t)((127 + e - 15) << 7);
    }
}

// ---------------------------------------------------------------------------------------
// 8 codes of a word -> 8 fp16 (q - z) * s in the order 0,4,1,5,2,6,3,7.
//   nz  = -(1024 + z) in both halves, nz6 = -(64 + z), s2 = scale in both halves.
__device__ __forceinline__ f16x8_t expand_word(uint32_t w, uint32_t magic, f16x2_t nz, f16x2_t nz6, f16x2_t s2) {
    const f16x2_t sixteenth = {(_Float16)0.0625f, (_Float16)0.0625f};
    const uint32_t w8 = w >> 8;
    const f16x2_t p0 = __builtin_bit_cast(f16x2_t, (w & 0x000F000Fu) | magic);
    const f16x2_t p1 = __builtin_bit_cast(f16x2_t, (w & 0x00F000F0u) | magic);
    const f16x2_t p2 = __builtin_bit_cast(f16x2_t, (w8 & 0x000F000Fu) | magic);
    const f16x2_t p3 = __builtin_bit_cast(f16x2_t, (w8 & 0x00F000F0u) | magic);
    const f16x2_t h0 = (p0 + nz) * s2;
    const f16x2_t h1 = (p1 * sixteenth + nz6) * s2;
    const f16x2_t h2 = (p2 + nz) * s2;
    const f16x2_t h3 = (p3 * sixteenth + nz6) * s2;
    return f16x8_t{h0[0], h0[1], h1[0], h1[1], h2[0], h2[1], h3[0], h3[1]};
}

// 8 signed bytes (two words) -> 8 fp16 q * s in their natural order.
//   flip = 0x80808080, sixfour = 0x64646464 (in vector registers), off = -1152 in both halves.
__device__ __forceinline__ f16x8_t expand_bytes(uint32_t w0, uint32_t w1, uint32_t flip, uint32_t sixfour, f16x2_t off,
                                                f16x2_t s2) {
    const uint32_t u0 = w0 ^ flip, u1 = w1 ^ flip;
    // v_perm_b32: bytes 0-3 of the selector pick from {second operand (bytes 0-3), first operand (bytes 4-7)}
    const f16x2_t p0 = __builtin_bit_cast(f16x2_t, __builtin_amdgcn_perm(sixfour, u0, 0x04010400u));
    const f16x2_t p1 = __builtin_bit_cast(f16x2_t, __builtin_amdgcn_perm(sixfour, u0, 0x04030402u));
    const f16x2_t p2 = __builtin_bit_cast(f16x2_t, __builtin_amdgcn_perm(sixfour, u1, 0x04010400u));
    const f16x2_t p3 = __builtin_bit_cast(f16x2_t, __builtin_amdgcn_perm(sixfour, u1, 0x04030402u));
    const f16x2_t h0 = (p0 + off) * s2, h1 = (p1 + off) * s2, h2 = (p2 + off) * s2, h3 = (p3 + off) * s2;
    return f16x8_t{h0[0], h0[1], h1[0], h1[1], h2[0], h2[1], h3[0], h3[1]};
}

// Global -> LDS copies by the load unit: lane l's 16 (or 4) bytes at base + off land at LDS
// address lds + 16 l (4 l).  Written as assembly on purpose: the compiler would otherwise
// make every later LDS read wait for all such copies in flight (it cannot see that the ring
// slots are distinct), which would drain the prefetch ring at every step.  The waits are
// explicit s_waitcnt vmcnt(n) at the points where a slot is handed over.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}
__device__ __forceinline__ void dma16(const void* base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds), "v"(off), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void dma4(const void* base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                 :: "s"(lds), "v"(off), "s"(base) : "memory", "m0");
}

// How a step is laid out in LDS, by code width.  The x tile has rows of kBK fp16, unpadded; the 16-byte
// chunk s of row r is kept at position s ^ swizzle(r), which makes the 16 lanes of a fragment read (16
// consecutive rows, same s) hit 16 different positions of a 256-byte line and 8 consecutive ones 8
// different ones of a 128-byte line: conflict-free.
// The codes of a step are 64 bytes per weight row and are fetched row by row (a load is 16 rows x 64 bytes:
// with every lane fetching its own pieces it touched 32 rows twice, and one decoder layer of 8-bit weights at
// M = 288, whose weight loads are the bottleneck, took 194 instead of 180 us); piece p (16 bytes) of row r is kept at position
// p ^ code_swizzle(r) of the row's 64 bytes: conflict-free reads as above.
__device__ __forceinline__ int code_swizzle(int r) { return ((r >> 2) & 3) ^ (r & 2); }
constexpr int kPow2Bytes = 768;   // powers of two of a tile: 256 columns, then 128 rows, bf16

template <int kBits>
struct Step {
    static constexpr int kBK = step_k(kBits);                     // k per step
    static constexpr int kSub = kBK / 16;                          // sub-steps: one MFMA per 32 x 32 block each
    static constexpr int kStages = ring_stages(kBits);            // slots of the ring
    static constexpr int kRowBytes = 2 * kBK;
    static constexpr int kChunks = kRowBytes / 16;
    static constexpr int kCodeLoads = kBK / 2 * kBits / 128;       // 16-byte pieces of a lane's codes of a step
    static constexpr int kLane = kCodeLoads * 1024 + (kBits == 4 ? 512 : 0);   // bytes per wave and column block: codes, nibbles: scale words, zero words
    __device__ static __forceinline__ int swizzle(int r) { return kBits == 4 ? r & 15 : (r & 7) ^ ((r >> 3) & 1); }
    static constexpr int kSegs = kStages + 1;                      // segments whose powers of two are in LDS
    // Bytes: a step lies inside one group, whose scale words (a tile's columns) are loaded once, with the
    // group's first step, into one of kSegs slots (a group lasts at least a step, as a segment does).  Loaded
    // with every step, for either half of the wave, they were a third of the weight loads (the layer above:
    // 180 -> 169 us; at M = 1024 476 -> 461).
    static constexpr int kScales = kBits == 4 ? 0 : 1024;          // bytes of such a slot
    static constexpr size_t lds(int rows, int col_blocks) {
        return (size_t)kStages * (rows * kRowBytes + col_blocks * kLane) + kSegs * (kPow2Bytes + kScales);
    }
};

struct GemmArgs {
    const uint32_t* qw;
    const uint16_t* sc;
    const uint32_t* zr;
    const uint16_t* xh;     // [Mpad][Kpad] fp16, scaled and permuted
    const uint16_t* pow2;   // bf16: [Mpad] of the rows of x, then [N] of the weight rows (from element wpow2 on)
    uint16_t* y;
    int M, N, K, Kpad, g, wpow2;
    TilePlan tp;
    float* partial;  // [2 P][tile] fp32: sums of tiles whose K range is shared between blocks
};

// Up to kGemmBatch linears share a launch: each gets a share of the grid and is dealt to its
// blocks exactly as if it had a launch of P blocks to itself.
struct GemmBatch {
    GemmArgs it[kGemmBatch];
    int count;
};

// A slot holds a tile's sums as the MFMA lanes have them, 16 bytes of a lane at a time: piece
// ((wave * MB + i) * WN + j) * 4 + q of lane (c, kb) is row 32 i + c, columns (WN wave + j) * 32 + 8 q + 4 kb + 0..3.

// Block tile (32 * MB) x (128 * WN): 4 waves side by side along n, each (32 * MB) x (32 * WN).
//
// The x tile of a step is written into LDS by the load unit itself (global_load_lds_dwordx4: lane l's 16
// bytes land at base + 16 l, so a wave fills four or eight rows per instruction) and costs no registers.
//
// Latency.  A step is only about a microsecond of matrix work, less than a trip to L2 or HBM under load,
// so the loads of step s + kStages - 1 are issued during step s: a ring of kStages x tiles (and sets of
// packed weights) in LDS.  Every load is unconditional (steps past the end of K reload the last tile,
// which nothing reads), so the number of loads in flight at each wait is a compile-time constant and the
// wait is an exact vmcnt, not a drain.
//
// The K loop is one continuous pipeline of sub-steps (16 k of every lane pair = one MFMA per
// 32 x 32 output block): the LDS reads and the expansion for sub-step u + 1 are issued
// among the MFMAs of sub-step u.  The tile of step s + 1 must be complete one sub-step
// before step s ends, so the wait + barrier sits in front of the step's last sub-step.
//
// The grid has at most one block per CU.  Tiles are dealt whole to the blocks as long as they
// fill complete rounds; what is left (fewer tiles than blocks) can be dealt in K steps instead:
// every block gets the same number of (tile, K step) units, a contiguous run of them, so no CU
// idles through a last, mostly empty round.  A block therefore works on a sequence of
// segments (a tile and a range of its K steps).  A segment that covers a tile's whole K is
// finished on the spot; otherwise its fp32 sums go to a slot of the workspace (two slots per
// block: one for its first shared segment, one for any later one) and a second kernel adds the
// slots of each such tile in K order, which keeps the result independent of timing.
//
// The segments of a block are one stream of steps: the loading waves go on with the next segment's steps
// while the multiplying waves finish the last one, and the results leave from the registers (weights are
// the MFMA's A operand, so a lane holds four neighbouring columns of one row), not through LDS, which is
// busy with the next tile.  Nothing in the K loop waits for those stores.  With the ring drained at every
// segment a tile of 128 x 256 paid 1.3 us of set-up, 4-6 us until its first step had landed and 4.7 us of
// epilogue around 57 us of K loop at K = 4096, M = 1024; 18 of 128 us at M = 288.
// One decoder layer: 60.0 -> 57.8 us at M = 48, 153.9 -> 149.8 at M = 288; 410 at M = 1024 either way, where
// the chip is limited by power (1.80 GHz sustained of 2.4) and idle time was buying clock.
// With one 128-row tile per block there is nothing to overlap, and it still costs a little where such tiles are
// wide: 4096 x 11008 at M = 2048 180.8 -> 183.3 us, the layer at M = 2048 773 -> 777.  Staging a block's last tile in
// LDS again did not help.
// What the end of a segment needs, the powers of two of its rows and columns, is loaded with its first
// step into one of kSegs slots: the step that is loaded first for segment q is loaded behind the barrier
// of step kStages before it, and segments are at least one step long, so everybody has left segment
// q - kSegs by then.

// s_waitcnt immediate: vmcnt(n), lgkmcnt(0), expcnt untouched.
__host__ __device__ constexpr int waitcnt_vm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4); }

// Besides the four multiplying waves a block has three that only load: two share the x tile loads of a
// step, the third issues the weight loads (for all four column groups, with the addresses the owning
// lanes would use); each waits for the step that is due and meets the MFMA waves at the step's barrier.
// The MFMA waves then issue no memory instruction in the K loop: with one wave per SIMD every load
// instruction otherwise sits in the same instruction stream as the MFMAs it delays.
// A second wave on a SIMD halves the registers a wave may have (256), which the 128 x 256 tile just
// fits.  Measured on a decoder layer's four linears with nibble weights: three loading waves (two for
// x, one for the weights) are 4-9 % faster than none at every M from 33 to 2048; two are as good on
// 96-row tiles and much slower on 128-row ones (32 x loads per step from one wave), four are slower
// than three (a loading wave on every SIMD).
constexpr int kXWaves = 2, kGemmThreads = 256 + 64 * (kXWaves + 1);
template <int MB, int WN, int kBits>
__global__ __launch_bounds__(kGemmThreads) void w4a16_gemm_f16_kernel(const GemmBatch args) {
    typedef Step<kBits> S;
    constexpr int kBK = S::kBK, kStages = S::kStages, kRowBytes = S::kRowBytes, kCodeLoads = S::kCodeLoads, kBLane = S::kLane;
    constexpr int kBM = 32 * MB;
    constexpr int kBN = 128 * WN;
    constexpr int kBufBytes = kBM * kRowBytes;    // one x tile
    constexpr int kBStage = 4 * WN * kBLane;      // one set of packed weights
    extern __shared__ __attribute__((aligned(16))) unsigned char As[];  // [kStages][kBM][kRowBytes]

    const int t = threadIdx.x;
    const int lane = t % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
    const int c = lane & 31, kb = lane >> 5;
    const int cwave = wave & 3;
    const bool loader = wave >= 4;   // wave-uniform
    int item = 0;
#pragma unroll
    for (int i = 1; i < kGemmBatch; ++i)
        if (i < args.count && (int)blockIdx.x >= args.it[i].tp.block_begin) item = i;
    const GemmArgs ga = args.it[item];
    const int bid = (int)blockIdx.x - ga.tp.block_begin;   // this block among the linear's own
    const int G = ga.K / ga.g, zwords = (G + 7) / 8, kw = ga.K / (32 / kBits);

    uint32_t magic = kBits == 4 ? 0x64006400u : 0x64646464u;
    asm volatile("" : "+v"(magic));  // in a VGPR: v_and_or_b32 takes one scalar operand only
    uint32_t flip = 0x80808080u;
    asm volatile("" : "+v"(flip));

    TileDealer dealer(ga.tp, bid, kBM, ga.Kpad);
    // the block's next segment: K steps [ka, ka + steps) of the tile at (bm, bn); false: there is none
    struct Seg {
        int bm, bn, ka, steps;
        int grp, kin;        // group of k = ka kBK, and the k of it that lie before
        bool first_shared;
    };
    auto next_segment = [&](Seg& sg) -> bool {
        TileDealer::Segment d;
        if (!dealer.next(d)) return false;
        sg.ka = d.ka;
        sg.steps = d.steps;
        sg.first_shared = d.first_shared;
        sg.grp = sg.ka * kBK / ga.g;
        sg.kin = sg.ka * kBK - sg.grp * ga.g;
        sg.bm = d.tm * kBM;
        sg.bn = d.tn * kBN;
        return true;
    };
    const int total = dealer.total_steps();

    // All tensors here are below 4 GB (checked by the host), so addresses are a uniform base plus a
    // 32-bit offset.
    const uint32_t as_lds = __builtin_amdgcn_readfirstlane(lds_addr(As));
    // fragment read offset of this lane (row c of a 32-row block): its half of the step's k is the
    // chunks kSub * kb + jj, and sub-step jj < kSub folds in by an XOR of the low bits
    const int aoff0 = c * kRowBytes + (((S::kSub * kb) ^ S::swizzle(c)) << 4);
    // The packed weights of a step and column block: 64 bytes of codes of each of its 32 rows, row by row, of which
    // a lane reads the two 16-byte pieces with its kBK / 2 k, and (nibbles) per lane the 4-byte words that hold
    // its group's scale and zero-point.  What a lane reads was fetched by other lanes of a loading wave: it is
    // complete once that wave has waited for the step and the step's barrier has been passed, and only
    // then.  No registers (and no compiler-inserted load waits) are tied up while the loads fly.  The group of a
    // lane's k is tracked without divisions (the group size is a multiple of 64, so they never straddle two groups).
    unsigned char* const Bs = As + kStages * kBufBytes;  // [kStages][4 waves][WN][kBLane]
    unsigned char* const Ps = Bs + kStages * kBStage;    // [kSegs][kPow2Bytes], then (bytes) [kSegs][kScales]
    unsigned char* const Cs = Ps + S::kSegs * kPow2Bytes;
    const int khalf = kBits == 4 ? kBK / 2 * kb : 0;     // first k of the lane's half, as far as groups are concerned

    if (loader) {
        // ---- the loading waves: one barrier after the first step has landed, then one per step, as the
        // MFMA waves have them.  The x waves take the x loads in turn; load q fills rows kRows q ..
        // (chunk lane % kChunks of a row at its swizzled position).  The last wave takes the 4 WN column
        // blocks: codes, scale words and zero words, each lane with the offsets of the lane that will
        // read them.
        constexpr int kRows = 64 / S::kChunks;           // rows per 1 KB load
        constexpr int kXLoads = kBM / kRows / kXWaves;   // per x wave and step
        constexpr int kWBlocks = 4 * WN;
        constexpr int kWLoads = kWBlocks * (kCodeLoads + (kBits == 4 ? 2 : 0));   // ... and what starts a segment or a group
        constexpr int kPeriod = 16 / (kRows * kXWaves);  // loads of a wave after which the swizzle repeats
        static_assert(kBM % (kRows * kXWaves) == 0 && 16 % (kRows * kXWaves) == 0, "loads divide evenly");
        static_assert((kStages - 2) * kXLoads < 64 && (kStages - 2) * kWLoads < 64, "the waits' counts fit the load counter");
        const bool xwave = wave < 4 + kXWaves;
        const int share = xwave ? wave - 4 : 0;
        const int lr = lane / S::kChunks, lp = lane % S::kChunks;
        const uint32_t pitchb = (uint32_t)ga.Kpad * 2u;
        uint32_t xsw[kPeriod];
#pragma unroll
        for (int qm = 0; qm < kPeriod; ++qm) xsw[qm] = (uint32_t)((lp ^ S::swizzle(kRows * (kXWaves * qm + share) + lr)) * 16);
        Seg sg;
        int left = 0, pstep = 0, seg_slot = 0;   // steps of the segment still to load, the next one
        uint32_t xrow0 = 0;
        uint32_t qo[kWBlocks][kCodeLoads], so[kWBlocks], zo[kWBlocks];
        const int crow = lane >> 2, cpiece = (lane & 3) ^ code_swizzle(crow);   // row of the 16, which 16 bytes of its 64
        int lk = 0, lgrp = 0, lkin = 0;
        int group_slot = -1;     // bytes: the current group's scales
        bool fresh = false;      // the next step is the first of a group
        auto load_step = [&](int slot) {
            if (left == 0) {
                if (next_segment(sg)) {
                    left = sg.steps;
                    pstep = sg.ka;
                    xrow0 = (uint32_t)(sg.bm + kRows * share + lr) * pitchb;
#pragma unroll
                    for (int mm = 0; mm < kWBlocks; ++mm) {
                        const int n = min(sg.bn + mm * 32 + c, ga.N - 1);
#pragma unroll
                        for (int part = 0; part < kCodeLoads; ++part)
                            qo[mm][part] = code_offset((uint32_t)min(sg.bn + mm * 32 + 16 * part + crow, ga.N - 1), (uint32_t)kw, (uint32_t)cpiece);
                        so[mm] = (uint32_t)n * (uint32_t)G * 2u;
                        zo[mm] = (uint32_t)n * (uint32_t)zwords * 4u;
                    }
                    lk = sg.ka * kBK + khalf;
                    fresh = true;
                    lkin = sg.kin + khalf;   // (less than two groups)
                    lgrp = sg.grp + (lkin >= ga.g);
                    lkin -= lkin >= ga.g ? ga.g : 0;
                    if (!xwave) {
                        // the tile's powers of two, in front of its first step (the waits below then wait a
                        // little longer than they have to, never too little): lanes 0-31 take 8 columns each,
                        // lanes 32-47 8 rows.  Columns past N are whatever the workspace holds there; nothing
                        // stored depends on them.
                        const uint32_t at = lane < 32 ? (uint32_t)(ga.wpow2 + sg.bn + 8 * lane) : (uint32_t)(sg.bm + 8 * (lane - 32));
                        if (lane < 32 + kBM / 8) dma16(ga.pow2, at * 2u, as_lds + kStages * (kBufBytes + kBStage) + (uint32_t)seg_slot * kPow2Bytes);
                    }
                    seg_slot = seg_slot == S::kSegs - 1 ? 0 : seg_slot + 1;
                } else {
                    left = 1 << 30;   // past the last segment: the last step's addresses again, which nothing reads
                }
            }
            --left;
            const uint32_t slot_x = as_lds + (uint32_t)slot * kBufBytes + (uint32_t)share * 1024u;
            const uint32_t slot_w = as_lds + kStages * kBufBytes + (uint32_t)slot * kBStage;
            if (xwave) {
                const uint32_t k0b = (uint32_t)(min(pstep, ga.tp.steps - 1) * kBK) * 2u;
#pragma unroll
                for (int qq = 0; qq < kXLoads; ++qq)
                    dma16(ga.xh, xrow0 + (uint32_t)(qq * kXWaves * kRows) * pitchb + xsw[qq % kPeriod] + k0b,
                          slot_x + qq * kXWaves * 1024);
            } else {
                const bool v = lk < ga.K;
                const uint32_t co = code_step_offset((uint32_t)(pstep * kBK), (uint32_t)cpiece, (uint32_t)ga.K, kBits);
                const uint32_t grp = v ? (uint32_t)lgrp : 0u;
                if (kBits == 8 && fresh) {
                    group_slot = group_slot == S::kSegs - 1 ? 0 : group_slot + 1;
                    fresh = false;
#pragma unroll
                    for (int q = 0; q < 2 * WN; ++q) {
                        const uint32_t so64 = (uint32_t)min(sg.bn + 64 * q + lane, ga.N - 1) * (uint32_t)G * 2u;
                        dma4(ga.sc, scale_word_offset(so64, grp), as_lds + (uint32_t)(Cs - As) + (uint32_t)group_slot * S::kScales + 256 * q);
                    }
                }
#pragma unroll
                for (int mm = 0; mm < kWBlocks; ++mm) {
                    const uint32_t dst = slot_w + mm * kBLane;
#pragma unroll
                    for (int part = 0; part < kCodeLoads; ++part)
                        dma16(ga.qw, qo[mm][part] + co, dst + 1024 * part);
                    if constexpr (kBits == 4) {
                        dma4(ga.sc, scale_word_offset(so[mm], grp), dst + kCodeLoads * 1024);
                        dma4(ga.zr, zero_word_offset(zo[mm], grp), dst + kCodeLoads * 1024 + 256);
                    }
                }
            }
            ++pstep;
            lk += kBK;
            lkin += kBK;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int over = lkin >= ga.g;
                lkin -= over * ga.g;
                lgrp += over;
                if (over) fresh = true;
            }
        };
#pragma unroll
        for (int p = 0; p < kStages - 1; ++p) load_step(p);
        // in flight: steps 0 .. kStages - 2; step 0 has to be complete
        if (xwave) __builtin_amdgcn_s_waitcnt(waitcnt_vm((kStages - 2) * kXLoads));
        else __builtin_amdgcn_s_waitcnt(waitcnt_vm((kStages - 2) * kWLoads));
        __syncthreads();
        int fill = kStages - 1;
        for (int s = 0; s < total; ++s) {
            // slot `fill` held step s - 1 and is free since the previous barrier
            load_step(fill);
            fill = fill == kStages - 1 ? 0 : fill + 1;
            // in flight: steps s + 1 .. s + kStages - 1; step s + 1 has to be complete
            if (xwave) __builtin_amdgcn_s_waitcnt(waitcnt_vm((kStages - 2) * kXLoads));
            else __builtin_amdgcn_s_waitcnt(waitcnt_vm((kStages - 2) * kWLoads));
            __syncthreads();
        }
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));  // nothing may still be writing LDS when the block ends
        return;
    }

    // operands of the step being multiplied; ck / cgrp follow the consumed steps like lk / lgrp.
    // A step's codes, scale word and zero word are read back from the ring (take_read) and
    // turned into the expansion's constants (take_convert) in two parts, so that the reads can be in
    // flight, and the conversions issue, under the MFMAs of the previous step's last sub-step.
    uint32_t wq[WN][4 * kCodeLoads];
    uint32_t tsw[WN], tzw[WN];
    f16x2_t nz[WN], nz6[WN], s2[WN];
    int ck = 0, cgrp = 0, ckin = 0, group_slot = -1;
    bool new_group = false;
    int bnext = 0, pnext = 0;   // columns of the step to be taken, and where its powers of two are
    uint32_t tpw[WN];
    auto take_segment = [&](const Seg& sg, int seg_slot) {
        ck = sg.ka * kBK + khalf;
        ckin = sg.kin + khalf;
        cgrp = sg.grp;
        const int over = ckin >= ga.g;
        ckin -= over * ga.g;
        cgrp += over;
        new_group = true;
        bnext = sg.bn;
        pnext = seg_slot * kPow2Bytes;
    };
    auto take_read = [&](uint32_t boff) {
        if (kBits == 8 && new_group) {
            group_slot = group_slot == S::kSegs - 1 ? 0 : group_slot + 1;
            new_group = false;
        }
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            const unsigned char* src = Bs + boff + (cwave * WN + j) * kBLane;
            const unsigned char* row = src + c * 64;
#pragma unroll
            for (int pc = 0; pc < kCodeLoads; ++pc) {
                const u32x4_t v = *reinterpret_cast<const u32x4_t*>(row + (((2 * kb + pc) ^ code_swizzle(c)) << 4));
                wq[j][4 * pc] = v.x; wq[j][4 * pc + 1] = v.y; wq[j][4 * pc + 2] = v.z; wq[j][4 * pc + 3] = v.w;
            }
            tsw[j] = kBits == 4 ? *reinterpret_cast<const uint32_t*>(src + kCodeLoads * 1024 + lane * 4)
                                : *reinterpret_cast<const uint32_t*>(Cs + group_slot * S::kScales + ((cwave * WN + j) * 32 + c) * 4);
            tpw[j] = *reinterpret_cast<const uint16_t*>(Ps + pnext + ((cwave * WN + j) * 32 + c) * 2);
            tzw[j] = kBits == 4 ? *reinterpret_cast<const uint32_t*>(src + kCodeLoads * 1024 + 256 + lane * 4) : 0u;
        }
    };
    auto take_convert = [&]() {
        const bool v = ck < ga.K;
        const uint32_t grp = v ? (uint32_t)cgrp : 0u;
        // past the end of K the scale becomes 0 by a factor, in a register: as a conditional value the
        // compiler turns it into a masked section, which nothing can be scheduled across
        float live = v ? 1.f : 0.f;
        asm volatile("" : "+v"(live));
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            // the scale's 2 bytes inside the aligned word that was fetched
            // (the parity of its position n G + grp)
            const uint32_t n = (uint32_t)min(bnext + (cwave * WN + j) * 32 + c, ga.N - 1);
            const uint32_t sbits = (tsw[j] >> (16u * (((n & (uint32_t)G) ^ grp) & 1u))) & 0xFFFFu;
            const float sf = (float)__builtin_bit_cast(_Float16, (uint16_t)sbits);
            const float z = kBits == 4 ? (float)((tzw[j] >> (4u * (grp & 7u))) & 0xFu) : 128.f;   // bytes: the flip's 128
            // one over the power of two of the column's largest scale
            const float winv = __builtin_bit_cast(float, 0x7F000000u - (tpw[j] << 16));
            const _Float16 srel = (_Float16)(sf * (winv * live));
            const _Float16 a = (_Float16)(-1024.f - z), b = (_Float16)(-64.f - z);
            nz[j] = f16x2_t{a, a};
            nz6[j] = f16x2_t{b, b};
            s2[j] = f16x2_t{srel, srel};
        }
        ck += kBK;
        ckin += kBK;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int over = ckin >= ga.g;
            ckin -= over * ga.g;
            cgrp += over;
            if (over) new_group = true;
        }
    };

    f32x16_t acc[MB][WN];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    };

    f16x8_t af[2][MB], bf[2][WN];
    auto fetch = [&](uint32_t aoff, int jj, int slot) {
        const unsigned char* src = As + aoff + (aoff0 ^ (jj << 4));
#pragma unroll
        for (int i = 0; i < MB; ++i) af[slot][i] = *reinterpret_cast<const f16x8_t*>(src + i * (32 * kRowBytes));
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            if constexpr (kBits == 4)
                bf[slot][j] = expand_word(wq[j][jj], magic, nz[j], nz6[j], s2[j]);
            else
                bf[slot][j] = expand_bytes(wq[j][2 * jj], wq[j][2 * jj + 1], flip, magic, nz[j], s2[j]);
        }
    };
    auto multiply = [&](int slot) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf[slot][j], af[slot][i], acc[i][j], 0, 0, 0);
        // issue order: the address of the next sub-step's fragments, then each MFMA followed by one LDS read
        // and a share of the vector operations that prepare the next sub-step.  (The address has a place of
        // its own because the reads wait for it: inside the first share it comes after the first read's place,
        // the pattern cannot be kept, and the reads gather behind the last MFMA, where the next sub-step waits
        // for them.  128-column tiles: 4096 x 4096 at M = 640 / 1024 40.2 / 47.2 -> 34.2 / 43.0 us, 4096 x 11008
        // at M = 1024 117 -> 104.7, 2048 x 1024 at M = 96 .. 1024 8-10 % less.)
        __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);
#pragma unroll
        for (int u = 0; u < MB * WN; ++u) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // LDS read
            __builtin_amdgcn_sched_group_barrier(0x002, ((kBits == 4 ? 13 : 14) * WN + MB * WN - 1) / (MB * WN), 0);  // VALU
        }
    };

    // The end of a segment: lane (c, kb) has row 32 i + c and columns 8 q + 4 kb + 0..3 of every 32-column
    // block in acc[i][j][4 q ..].
    auto finish = [&](const Seg& sg, int seg_slot) {
        if (sg.steps != ga.tp.steps) {
            // part of a tile's K: the raw sums go to this block's slot
            float* const slot = ga.partial + (size_t)(2 * bid + (sg.first_shared ? 0 : 1)) * (kBM * kBN);
            f32x4_t* const dst = reinterpret_cast<f32x4_t*>(slot) + cwave * (MB * WN * 4) * 64 + lane;
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        dst[((i * WN + j) * 4 + q) * 64] = f32x4_t{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
            return;
        }
        // y = acc * 2^-p(m) * 2^E(n), rounded once to bf16.  The halves of the wave exchange pieces, so that a
        // lane stores eight neighbouring columns of its row.
        // Row by row, so that the pieces of a line are stored one after the other.
        const unsigned char* const pw = Ps + seg_slot * kPow2Bytes;
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const float rs = bf16_bits_to_f32(*reinterpret_cast<const uint16_t*>(pw + 512 + (32 * i + c) * 2));
            const int m = sg.bm + 32 * i + c;
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int qp = 0; qp < 2; ++qp) {
                    const f32x16_t& v = acc[i][j];
                    uint32_t p[2][2];   // [which 8 columns][pair]
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint2 w2 = *reinterpret_cast<const uint2*>(pw + ((cwave * WN + j) * 32 + 16 * qp + 8 * h + 4 * kb) * 2);
                        const float wm[4] = {__builtin_bit_cast(float, w2.x << 16), __builtin_bit_cast(float, w2.x & 0xFFFF0000u),
                                             __builtin_bit_cast(float, w2.y << 16), __builtin_bit_cast(float, w2.y & 0xFFFF0000u)};
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            const int r = 4 * (2 * qp + h) + 2 * e;
                            p[h][e] = f32x2_to_bf16x2_rne(v[r] * rs * wm[2 * e], v[r + 1] * rs * wm[2 * e + 1]);
                        }
                    }
                    // lanes 32-63 of the first operand and lanes 0-31 of the second change places
                    const auto a = __builtin_amdgcn_permlane32_swap(p[0][0], p[1][0], false, false);
                    const auto b = __builtin_amdgcn_permlane32_swap(p[0][1], p[1][1], false, false);
                    const u32x4_t o = {a[0], b[0], a[1], b[1]};
                    const int n = sg.bn + (cwave * WN + j) * 32 + 16 * qp + 8 * kb;
                    if (m < ga.M && n < ga.N) {
                        uint16_t* dst = ga.y + (size_t)m * ga.N + n;
                        if (n + 8 <= ga.N) {
                            // (rows of y begin at any multiple of 2 bytes.  Stored value by value wherever N is
                            // no multiple of 8, N = 8154 took 73 us at M = 442, K = 5888, against 61 now)
                            *reinterpret_cast<u32x4_any_t*>(dst) = o;
                        } else {
                            const uint32_t w[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
                            for (int e = 0; e < 7; ++e)
                                if (n + e < ga.N) dst[e] = (uint16_t)(w[e / 2] >> (16 * (e & 1)));
                        }
                    }
                }
        }
    };

    Seg sg, ahead;
    if (!next_segment(sg)) return;   // (every block has one)
    ahead = sg;
    bool more = next_segment(ahead);
    int left = sg.steps, seg_slot = 0;
    uint32_t acur = 0, bcur = 0;     // the step's slot
    clear();
    __syncthreads();
    take_segment(sg, 0);
    take_read(0);
    take_convert();
    fetch(0, 0, 0);
    for (;;) {
#pragma unroll
        for (int jj = 0; jj < S::kSub - 1; ++jj) {
            __builtin_amdgcn_sched_barrier(0);
            fetch(acur, jj + 1, (jj + 1) & 1);
            multiply(jj & 1);
        }
#pragma unroll
        for (int j = 0; j < WN; ++j) asm volatile("" : "+v"(bf[1][j]));   // expanded here, not behind the barrier
        __builtin_amdgcn_sched_barrier(0);
        // The loading waves have seen step s + 1 land.  The wait covers this wave's LDS reads (lgkmcnt 0, not
        // its stores), so after the barrier the step's slot is dead for everyone once the last sub-step is
        // done (its operands are already in registers).
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(63));
        __syncthreads();
        acur = acur == (kStages - 1) * kBufBytes ? 0 : acur + kBufBytes;
        bcur = bcur == (kStages - 1) * kBStage ? 0 : bcur + kBStage;
        const bool last = --left == 0;
        const int next_slot = seg_slot == S::kSegs - 1 ? 0 : seg_slot + 1;
        if (last) take_segment(ahead, next_slot);   // (past the last segment: the last again, which nothing uses)
        __builtin_amdgcn_sched_barrier(0);
        // The last sub-step of this step (operands already in registers) with the next step's set-up under
        // it: all LDS reads first (codes, constants, x fragments), a few MFMAs while they are in flight, then
        // the conversions and the first expansion shared out among the remaining MFMAs.
        take_read(bcur);
        take_convert();
        fetch(acur, 0, 0);
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf[1][j], af[1][i], acc[i][j], 0, 0, 0);
        constexpr int kLead = MB * WN < 4 ? 1 : 3;                     // MFMAs issued before any conversion
        constexpr int kSetupValu = (kBits == 4 ? 13 + 20 : 14 + 16) * WN + 8;
        __builtin_amdgcn_sched_group_barrier(0x100, WN * (kCodeLoads + (kBits == 4 ? 3 : 2)) + MB, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, kLead, 0);
        if constexpr (MB * WN > kLead) {
#pragma unroll
            for (int u = 0; u < MB * WN - kLead; ++u) {
                __builtin_amdgcn_sched_group_barrier(0x002, (kSetupValu + MB * WN - kLead - 1) / (MB * WN - kLead), 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            }
        }
        // 256-column tiles: the next step's first fragments are expanded here, under the MFMAs; left alone the
        // compiler moves that behind the branch, to the start of the next step (layer at M = 1024 / 2048 396.7 / 780.1
        // -> 395.3 / 776.9 us, bytes at M = 1024 454 -> 449; 128-column tiles are 0.5-1 % slower with it).  On the
        // 128 x 256 nibble tile it costs 8 bytes of scratch per lane, stored and read back outside the K loop.
        if constexpr (WN == 2) asm volatile("" : "+v"(bf[0][0]), "+v"(bf[0][1]));
        __builtin_amdgcn_sched_barrier(0);
        if (!last) continue;
        finish(sg, seg_slot);
        if (!more) break;
        clear();
        sg = ahead;
        left = sg.steps;
        seg_slot = next_slot;
        more = next_segment(ahead);
    }
}

// Adds up the slots of every tile whose K range was shared between blocks (in K order) and
// finishes it like the main kernel does: y = sum * 2^-p(m) * 2^E(n), rounded once to bf16.
// Grid: (tiles dealt in K steps, pieces of 256 4-float groups per tile, linears); a thread owns one group.
template <int MB, int WN>
__global__ __launch_bounds__(256) void w4a16_gemm_fixup_kernel(const GemmBatch args) {
    constexpr int kBM = 32 * MB, kBN = 128 * WN;
    static_assert((kBM * kBN / 4) % 256 == 0, "tiles split into whole pieces");
    const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
    const GemmArgs ga = args.it[blockIdx.z];
    const TilePlan tp = ga.tp;
    const int P = tp.P;
    if ((int)blockIdx.x >= tp.tiles - tp.whole) return;   // the grid is as wide as the largest tail
    const int tile = tp.whole + blockIdx.x;
    const long long units = (long long)(tp.tiles - tp.whole) * tp.steps;
    const int u_first = (int)blockIdx.x * tp.steps, u_last = u_first + tp.steps - 1;   // (units are below 2^31, see TileDealer)
    const int b_lo = owner_of_quick(u_first, units, P), b_hi = owner_of_quick(u_last, units, P);
    if (b_lo == b_hi) return;  // one block had the whole tile and has finished it

    // The slots to add, in K order, worked out once per block (the divisions are slow) and
    // packed, so that the loads below can be issued several at a time.
    __shared__ int slots[kMaxGemmBlocks];
    __shared__ int wave_count[4];
    int count = 0;
    for (int b0 = b_lo; b0 <= b_hi; b0 += 256) {
        const int b = b0 + t;
        int sl = -1;  // with fewer units than blocks some blocks own none
        if (b <= b_hi) {
            const int fu = first_unit_quick(b, units, P);
            // a block's first shared segment is in its slot 0, a later one in slot 1 (fu <= u_last: the block's units reach this tile)
            if (fu != first_unit_quick(b + 1, units, P)) sl = 2 * b + (fu >= u_first ? 0 : 1);
        }
        const unsigned long long have = __ballot(sl >= 0);
        if (lane == 0) wave_count[wave] = __popcll(have);
        __syncthreads();
        int at = count + __popcll(have & ((1ull << lane) - 1ull));
        for (int w = 0; w < wave; ++w) at += wave_count[w];
        if (sl >= 0) slots[at] = sl;
        count += wave_count[0] + wave_count[1] + wave_count[2] + wave_count[3];
        __syncthreads();
    }

    const int idx = blockIdx.y * 256 + t;
    const int piece = idx / 64, ilane = idx % 64;
    const int q = piece % 4, j = piece / 4 % WN, i0 = piece / (4 * WN) % MB, w0 = piece / (4 * WN * MB);
    const int m = (tile % tp.Tm) * kBM + 32 * i0 + ilane % 32, n = (tile / tp.Tm) * kBN + (w0 * WN + j) * 32 + 8 * q + 4 * (ilane / 32);
    if (m >= ga.M || n >= ga.N) return;
    const float* src = ga.partial + idx * 4;
    const float rs = bf16_bits_to_f32(ga.pow2[m]);
    float wm[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) wm[e] = bf16_bits_to_f32(ga.pow2[ga.wpow2 + min(n + e, ga.N - 1)]);
    // Four slots at a time, all requested before any is added; most tiles have two or three, so in the last four a request
    // past the last slot reads that one again (from the cache) and is not added.  With the 32-bit divisions: decoder layer at
    // M = 288 / 1024 10.9 / 8.8 -> 9.7 / 8.2 us.  (That test in every four cost tiles of 64 slots, 500 x 11008 at M = 40,
    // 1.8 us of 20.)
    f32x4_t sum = {0.f, 0.f, 0.f, 0.f};
    int i = 0;
    for (; i + 4 <= count; i += 4) {
        f32x4_t v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = *reinterpret_cast<const f32x4_t*>(src + (size_t)slots[i + e] * (kBM * kBN));
#pragma unroll
        for (int e = 0; e < 4; ++e) sum += v[e];
    }
    if (i < count) {
        f32x4_t v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = *reinterpret_cast<const f32x4_t*>(src + (size_t)slots[min(i + e, count - 1)] * (kBM * kBN));
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (i + e < count) sum += v[e];
    }
    uint16_t* dst = ga.y + (size_t)m * ga.N + n;
    uint16_t h[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = f32_to_bf16_rne(sum[e] * rs * wm[e]);
    if (n + 4 <= ga.N) {
        *reinterpret_cast<u32x2_any_t*>(dst) = u32x2_any_t{h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16)};
    } else {
        for (int e = 0; e < 4 && n + e < ga.N; ++e) dst[e] = h[e];
    }
}

int gemm_max_blocks() { return device_cu_count() < kMaxGemmBlocks ? device_cu_count() : kMaxGemmBlocks; }

// One launch for `n` linears that use the same tile, each on its own blocks (its plan).
template <int MB, int WN, int kBits>
hipError_t launch_tile(const GemmArgs* gas, int n, hipStream_t st) {
    constexpr int kBM = 32 * MB, kBN = 128 * WN;
    constexpr size_t lds = Step<kBits>::lds(kBM, 4 * WN);
    static_assert(lds <= 160 * 1024, "the ring fits LDS");
    // more than 64 KB of LDS needs an opt-in; the call is idempotent, so two host threads that
    // both find the flag clear may both make it
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&w4a16_gemm_f16_kernel<MB, WN, kBits>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    GemmBatch gb;
    int grid = 0, max_tail = 0;
    for (int i = 0; i < kGemmBatch; ++i) {
        gb.it[i] = gas[i < n ? i : n - 1];
        if (i < n) {
            const TilePlan& tp = gas[i].tp;
            grid += tp.P;
            // the second kernel is only needed when some block boundary falls inside a tile
            const int tail = tp.tiles - tp.whole;
            const long long units = (long long)tail * tp.steps;
            bool shared = false;
            for (int b = 1; b < tp.P && tail > 0 && !shared; ++b) shared = first_unit(b, units, tp.P) % tp.steps != 0;
            if (shared && tail > max_tail) max_tail = tail;
        }
    }
    gb.count = n;
    hipLaunchKernelGGL((w4a16_gemm_f16_kernel<MB, WN, kBits>), dim3(grid), dim3(kGemmThreads), lds, st, gb);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (max_tail > 0) {
        hipLaunchKernelGGL((w4a16_gemm_fixup_kernel<MB, WN>), dim3(max_tail, kBM * kBN / 4 / 256, n), dim3(256), 0, st, gb);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace

bool gemm_f16_supports(const qail_wdesc& d, int M) {
    if (d.K % 64 != 0 || d.group_size % 64 != 0) return false;
    // A scale is fetched as the aligned 4-byte word that holds it; with an odd number of scales
    // the word of the last one would reach two bytes past the caller's buffer.
    if (((unsigned long long)d.N * (unsigned long long)(d.K / d.group_size)) % 2 != 0) return false;
    // 32-bit byte offsets inside the kernel
    const unsigned long long lim = 0xFFFFFFFFull;
    const unsigned long long Mpad = (unsigned long long)round_up(M, kRowPad), Kpad = (unsigned long long)round_up(d.K, kPadK);
    const unsigned long long code_bytes = (unsigned long long)d.N * d.K / (d.scheme == QAIL_W8_SYM_GROUP ? 1 : 2);
    return code_bytes <= lim && Mpad * Kpad * 2 <= lim && (unsigned long long)M * d.N * 2 <= lim;
}

// Workspace of one linear without the slots: x as fp16, the row scales, the weight rows' powers of two.
static size_t gemm_head_bytes(const qail_wdesc& d, int M) {
    const size_t Mpad = (size_t)round_up(M, kRowPad), Kpad = (size_t)round_up(d.K, kPadK);
    const size_t b = Mpad * Kpad * 2 + Mpad * 4 + (size_t)round_up(d.N, 64) * 4;
    return (b + 255) / 256 * 256;
}

// Two tile-shaped fp32 slots per block of the grid for tiles whose K range is shared between blocks.
static size_t gemm_slot_bytes(int M, bool wide) {   // wide: 256-column tiles (N > 128)
    return 2 * (size_t)gemm_max_blocks() * (size_t)tile_rows(M) * (wide ? 256 : 128) * 4;
}

size_t gemm_f16_workspace(const qail_wdesc& d, int M) {
    return gemm_head_bytes(d, M) + gemm_slot_bytes(M, d.N > 128);
}

size_t gemm_f16_batch_workspace(const qail_w4a16_item* items, int count, int M, bool wide_tiles) {
    // linears that share a launch (kGemmBatch at a time) need their heads side by side; the
    // slots are shared out with the blocks
    size_t need = 0;
    for (int i0 = 0; i0 < count; i0 += kGemmBatch) {
        size_t b = 0;
        bool wide = false;
        for (int i = i0; i < count && i < i0 + kGemmBatch; ++i) {
            b += gemm_head_bytes(items[i].d, M);
            wide = wide || (items[i].d.N > 128 && wide_tiles);
        }
        b += gemm_slot_bytes(M, wide);
        if (b > need) need = b;
    }
    return need;
}

template <int MB>
static hipError_t launch_chunk(const qail_w4a16_item* items, int n, int M, bool wide_tiles, void* ws, hipStream_t st) {
    const bool bytes = items[0].d.scheme == QAIL_W8_SYM_GROUP;   // all items of a call have the same code width
    const int Mpad = round_up(M, kRowPad);
    const int cus = gemm_max_blocks();
    GemmArgs ga[kGemmBatch];
    PrepBatch pb;
    pb.M = M;
    pb.rows = round_up(M, 32 * MB);
    pb.natural = bytes ? 1 : 0;
    char* at = static_cast<char*>(ws);
    int prep_blocks = 0;
    for (int i = 0; i < n; ++i) {
        const qail_wdesc& d = items[i].d;
        const int Kpad = round_up(d.K, kPadK), G = d.K / d.group_size;
        uint16_t* xh = reinterpret_cast<uint16_t*>(at);
        uint16_t* rscale = xh + (size_t)Mpad * Kpad;
        uint16_t* wmul = rscale + Mpad;
        at += gemm_head_bytes(d, M);
        pb.it[i] = PrepItem{items[i].x, items[i].scales, xh, rscale, wmul, d.N, d.K, Kpad, G};
        ga[i] = GemmArgs{items[i].qweight, items[i].scales, items[i].zeros, xh, rscale, items[i].y,
                         M, d.N, d.K, Kpad, d.group_size, Mpad, TilePlan{}, nullptr};
        prep_blocks = std::max(prep_blocks, pb.rows + (d.N + 31) / 32);
    }
    for (int i = n; i < kGemmBatch; ++i) pb.it[i] = pb.it[n - 1];
    float* slots = reinterpret_cast<float*>(at);
    hipLaunchKernelGGL(gemm_prep_kernel, dim3(prep_blocks, n), dim3(256), 0, st, pb);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;

    // every linear gets blocks in proportion to its weights (at least one), then its own tiling
    int share[kGemmBatch], wn[kGemmBatch];
    bool split[kGemmBatch];
    auto deal = [&](const int* idx, int m, int avail) {
        double sum = 0;
        for (int j = 0; j < m; ++j) sum += (double)items[idx[j]].d.N * items[idx[j]].d.K;
        int used = 0;
        for (int j = 0; j < m; ++j) {
            const int i = idx[j];
            share[i] = std::max(1, (int)((double)items[i].d.N * items[i].d.K / sum * avail));
            used += share[i];
        }
        for (int j = 0; used < avail; j = (j + 1) % m, ++used) ++share[idx[j]];
        while (used > avail) {   // the floors of one block each were too many: take from the largest
            int big = idx[0];
            for (int j = 1; j < m; ++j)
                if (share[idx[j]] > share[big]) big = idx[j];
            --share[big];
            --used;
        }
    };
    int all[kGemmBatch];
    for (int i = 0; i < n; ++i) all[i] = i;
    deal(all, n, std::max(cus, n));
    for (int i = 0; i < n; ++i) choose_tile(bytes ? 8 : 4, 32 * MB, M, ga[i].N, ga[i].Kpad, share[i], n == 1, !wide_tiles, &wn[i], &split[i]);
    // linears with the same tile width go out together, each group on the whole chip
    for (int w = 2; w >= 1; --w) {
        int idx[kGemmBatch], m = 0;
        for (int i = 0; i < n; ++i)
            if (wn[i] == w) idx[m++] = i;
        if (m == 0) continue;
        if (m < n) {
            deal(idx, m, std::max(cus, m));
            for (int j = 0; j < m; ++j) {
                int w2;
                choose_tile(bytes ? 8 : 4, 32 * MB, M, ga[idx[j]].N, ga[idx[j]].Kpad, share[idx[j]], n == 1, !wide_tiles, &w2, &split[idx[j]]);
            }
        }
        GemmArgs grp[kGemmBatch];
        int begin = 0;
        for (int j = 0; j < m; ++j) {
            GemmArgs& g = ga[idx[j]];
            g.tp = plan_tiles(M, g.N, g.K, 32 * MB, 128 * w, step_k(bytes ? 8 : 4), split[idx[j]], share[idx[j]]);
            g.tp.block_begin = begin;
            g.partial = slots + (size_t)2 * begin * (32 * MB) * (128 * w);
            begin += g.tp.P;
            grp[j] = g;
        }
        e = bytes ? (w == 2 ? launch_tile<MB, 2, 8>(grp, m, st) : launch_tile<MB, 1, 8>(grp, m, st))
                  : (w == 2 ? launch_tile<MB, 2, 4>(grp, m, st) : launch_tile<MB, 1, 4>(grp, m, st));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_w4a16_gemm_f16_batch(const qail_w4a16_item* items, int count, int M, bool wide_tiles, void* ws, hipStream_t st) {
    for (int i0 = 0; i0 < count; i0 += kGemmBatch) {
        const int n = std::min(kGemmBatch, count - i0);
        hipError_t e;
        switch (tile_rows(M)) {
            case 32: e = launch_chunk<1>(items + i0, n, M, wide_tiles, ws, st); break;
            case 64: e = launch_chunk<2>(items + i0, n, M, wide_tiles, ws, st); break;
            case 96: e = launch_chunk<3>(items + i0, n, M, wide_tiles, ws, st); break;
            default: e = launch_chunk<4>(items + i0, n, M, wide_tiles, ws, st); break;
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace qail
