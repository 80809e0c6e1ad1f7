// W4A16 / W8A16 linear for a medium batch: y[m][n] = sum_k x[m][k] (q[n][k] - z[n][k/g]) s[n][k/g].
//
// Between a handful of rows of x and a few hundred the weights are still the traffic that counts,
// but every weight has to meet several 16-row blocks of x.  The streaming kernel of small batches
// stops for a fresh pass of x, and the tiled GEMM has one multiplying wave per SIMD, whose reads,
// expansion and MFMAs follow each other, and two more launches around it.  Here:
//
//   * A block (eight waves, two per SIMD, one block per CU) owns up to a few dozen tiles of 16
//     weight rows and makes a single pass over K.  Wave (kw, cw) multiplies the K part kw of
//     the column tiles cw, cw + Wc, ...; K parts meet in LDS at the end, in order, so the result
//     does not depend on timing.
//   * Packed codes go from HBM straight into registers, D steps (of 128 k) ahead: a wave-wide
//     load is 16 rows x 64 bytes, a lane's 16 bytes are the B operands of four
//     v_mfma_f32_16x16x32_bf16 (0x3B80 | q is bf16 (128 + q) 2^-15).  A weight is expanded once and used
//     by all row blocks of the wave.
//   * x passes through the same registers, as far ahead (loads return in order: x fetched later
//     than the codes beside it would drain their ring), into a double buffer of LDS, one 128-k
//     step of every K part at a time, one barrier per step.  Its sums over each group, which the
//     offset form needs,
//         sum_k x (q - z) s = s * ( sum_k x (q + 128)  -  (128 + z) * sum_k x ),
//     come from four MFMAs against ones on the way.  Nothing is rounded before the fp32 sums.  Codes and ones carry a
//     factor of 2^-15 (bytes: 2^-24), taken back at the end (with the scale): a group's 128 products of x with
//     up to 255 stay finite for every finite x; without the factor an x beyond 2e36 (bytes: 1e34) gave NaN.
//   * The block's scales and zero-points are copied to LDS once: as loads beside the codes they
//     would cost as much as the codes.
//
// What bounds it: issue and latency inside a step (at M = 48 12 tiles a block with no loads take
// 30 us of the 38 that 100 MB of codes take; the codes alone 24), then HBM.  The layer of a 7B
// model in one call, before (smallm / GEMM) -> now, us: M = 24 / 32 / 48 / 64 43.7 / 45.2 / 56.0 /
// 56.4 -> 37.6 / 39.6 / 44.2 / 51.7; groups of 64 M = 8 / 32 / 48 53.1 / 53.9 / 61.8 -> 40.9 /
// 44.1 / 59.1; bytes M = 8 / 32 / 48 51.9 / 63.0 / 71.8 -> 44.6 / 51.4 / 56.9.  Measured and not
// kept: codes fetched with the pieces of a row in neighbouring lanes (22 instead of 66 cycles of
// the address unit per load) and turned through LDS, the offset as the MFMAs' start value and the
// zero-points as fp32 MFMAs, tile-outer order, a third buffer of x: none faster.
#include <string.h>

#include <algorithm>
#include <atomic>

#include "qail_internal.h"

namespace qail {

namespace {

constexpr int kMdWaves = 8;
constexpr int kMdThreads = kMdWaves * kWave;
constexpr int kMdStepK = 128;
constexpr int kMdMaxItems = 16;
constexpr int kMdMaxBlocks = 2048;   // blocks of a launch that serves more than one item
constexpr size_t kMdLds = 160 * 1024;
constexpr uint32_t kPastEnd = 0x80000000u;   // an offset no tensor here reaches: the load returns zeros and fetches nothing

enum MdMode { kNib128 = 0, kNib64 = 1, kByte128 = 2 };

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;

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
    uint32_t item_of_block[kMdMaxBlocks / 8];   // 4 bits per block; a lone item needs none
    int M;
};

// Everything in LDS before this point has been written, and nobody reads further back: vector-memory
// loads stay in flight, which __syncthreads() does not promise.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// C: column tiles of the wave, NL: loads of x per wave and step (each four rows of one K part), D: steps fetched ahead.
// The waves of a block may differ in C (a barrier counts waves, not where they stand): all meet once per step.
template <int kMode, int kRB, int C, int NL, int D>
__device__ __forceinline__ void md_block(const MdArgs& args, const MdItem& it, unsigned char* lds) {
    const int cmax = it.tiles_per_wave;
    constexpr bool kBytes = kMode == kByte128;
    constexpr int kLoads = kBytes ? 2 : 1;         // wave-wide loads per tile and step
    constexpr int kGroups = kMode == kNib64 ? 2 : 1;   // scale groups per step
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int li = lane & 15, kb = lane >> 4;
    const int M = args.M, wkl = it.wkl;
    const int N = it.N, K = it.K;
    const int S = K / kMdStepK, G = S * kGroups, zwords = (G + 7) / 8;
    const int rowbytes = kBytes ? K : K / 2;
    const int Wk = 1 << wkl, Wc = kMdWaves >> wkl;
    const int kw = wave & (Wk - 1), cw = wave >> wkl;
    const int b = (int)blockIdx.x - it.block_begin;
    const int tile0 = b * it.tiles_base + min(b, it.tiles_rem);
    const int nt = it.tiles_base + (b < it.tiles_rem ? 1 : 0);
    // LDS: x [2][K part][row block][16 rows][256 bytes], sums of x [2][K part][row block][group][16], scales, zero-points
    const int xbytes = (kRB << wkl) * 4096, sbytes = (kRB << wkl) * (kGroups * 64);
    unsigned char* const xl = lds;
    unsigned char* const s1 = lds + 2 * xbytes;
    unsigned char* const stab = lds + 64 * (int)it.table;
    unsigned char* const ztab = stab + nt * 16 * G * 2;

    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(it.sc), 0, N * G * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(it.zr), 0, kBytes ? 0 : N * zwords * 4, 0x00020000);

    // ---- this wave's codes
    const int k0 = (S * kw) >> wkl, n_k = ((S * (kw + 1)) >> wkl) - k0;
    const int n_max = (S + Wk - 1) >> wkl;       // steps of the block; a K part that has fewer multiplies its last one with zeros
    uint32_t qoff[C], srow[C], zrow[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int t = c * Wc + cw, row = (tile0 + t) * 16 + li;
        qoff[c] = t < nt && row < N ? (uint32_t)row * (uint32_t)rowbytes + 16u * kb : kPastEnd;
        const int tl = min(t, nt - 1) * 16 + li;
        srow[c] = (uint32_t)(tl * G * 2);
        zrow[c] = (uint32_t)(tl * zwords * 4);
    }
    // ---- the rows of x this wave stages: load l takes rows u, u + 4, u + 8, u + 12 of a row block of a K part, lane (li, kb)
    // the 16-byte piece 4 kb + li % 4 of row u + 4 (li / 4), so that four neighbouring lanes fetch 64 contiguous bytes
    int xk0[NL], xn[NL];
    uint32_t xoff[NL], xdst[NL], sdst = 0;
    const int last_load = (kRB << (wkl + 2)) - 1;   // a wave without a load of its own repeats the last one (the same bytes to the same place)
#pragma unroll
    for (int l = 0; l < NL; ++l) {
        const int e = min(wave + kMdWaves * l, last_load), part = (e >> 2) & (Wk - 1), R = e >> (2 + wkl), u = e & 3;
        const int m = 16 * R + u + (li & 12);
        xk0[l] = (S * part) >> wkl;
        xn[l] = ((S * (part + 1)) >> wkl) - xk0[l];
        xoff[l] = m < M ? (uint32_t)m * (uint32_t)(K * 2) + (uint32_t)(4 * kb + (li & 3)) * 16u : kPastEnd;
        // piece p of row r is kept at position p ^ r: eight neighbouring rows of one piece (a fragment read) and the two
        // rows x 4 pieces of eight neighbouring lanes (the writes) lie in eight different 16-byte columns of 128 bytes,
        // sixteen of them in sixteen of 256
        xdst[l] = (uint32_t)((part * kRB + R) * 4096 + (u + (li & 12)) * 256 + (((4 * kb + (li & 3)) ^ (u + (li & 12))) << 4));
        // lane l (groups of 64: lanes 2 l, 2 l + 1) of a quarter writes the load's sums
        if (li / kGroups == l) sdst = (uint32_t)((part * kRB + R) * (kGroups * 64) + (u + 4 * kb) * 4 + (kGroups == 2 ? (li & 1) * 64 : 0));
    }
    const uint32_t xrow_end = (uint32_t)M * (uint32_t)(K * 2);
    const uint32_t qend = (uint32_t)N * (uint32_t)rowbytes;

    u32x4_t q[D][C][kLoads], xr[D][NL];
    // the steps are walked from one of them on and around, another one in each block: blocks that ask for the same rows
    // of x do not all ask for the same stretch (one L2 channel) at a time
    const int rot = (int)((unsigned)b % (unsigned)n_max);
    int pq = rot;   // next step whose codes are requested, in steps of the K part
    int px = rot;   // ... whose x
    int iq = 0, ix = 0;
    auto issue_q = [&](int d) {
        const int step = k0 + min(pq, n_k - 1);
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(it.qw), 0, iq < n_max ? qend : 0u, 0x00020000);
#pragma unroll
        for (int h = 0; h < kLoads; ++h)
#pragma unroll
            for (int c = 0; c < C; ++c)
                q[d][c][h] = __builtin_amdgcn_raw_buffer_load_b128(r, qoff[c], step * (64 * kLoads) + 64 * h, 0);
        ++iq;
        if (++pq == n_max) pq = 0;
    };
    uint32_t xend = xrow_end;
    auto issue_x = [&](int d) {
        if (ix >= n_max) xend = 0;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(it.x), 0, px < xn[l] ? xend : 0u, 0x00020000);
            xr[d][l] = __builtin_amdgcn_raw_buffer_load_b128(r, xoff[l], (xk0[l] + px) * 256, 0);
        }
        ++ix;
        if (++px == n_max) px = 0;
    };
    uint32_t ones = kMode != kNib64 || (li & 1) == (kb >> 1) ? (kBytes ? 0x33803380u : 0x38003800u) : 0u;   // groups of 64: the sums of one in the even columns, of the other in the odd ones
    asm volatile("" : "+v"(ones));
    const u32x4_t ones4 = {ones, ones, ones, ones};
    auto put_x = [&](const u32x4_t (&v)[NL], int buf) {
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const u32x4_t p = v[l];
            u32x4_t o = p;
            if (!kBytes) {   // the order in which the expansion lays out the nibbles of a word: x0,x4 x1,x5 x2,x6 x3,x7
                o[0] = __builtin_amdgcn_perm(p[2], p[0], 0x05040100u);
                o[1] = __builtin_amdgcn_perm(p[2], p[0], 0x07060302u);
                o[2] = __builtin_amdgcn_perm(p[3], p[1], 0x05040100u);
                o[3] = __builtin_amdgcn_perm(p[3], p[1], 0x07060302u);
            }
            *reinterpret_cast<u32x4_t*>(xl + buf * xbytes + xdst[l]) = o;
        }
    };
    // lane (li, kb) supplies row li of the product; register i of the result is the sum over what lanes 4 kb + i (of every
    // quarter) hold, i.e. over a quarter of row u + 4 kb
    auto sum_x = [&](const u32x4_t (&v)[NL]) {
        float mine = 0.f;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const f32x4_t t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, v[l]), __builtin_bit_cast(bf16x8_t, ones4),
                                                                      f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            const float r = (t[0] + t[1]) + (t[2] + t[3]);
            mine = l == 0 || li / kGroups == l ? r : mine;
        }
        return mine;
    };
    auto put_sums = [&](float mine, int buf) {
        if (li < NL * kGroups) *reinterpret_cast<float*>(s1 + buf * sbytes + sdst) = mine;
    };

    // ---- requests: the tables and the first step of x, then the ring
    u32x4_t x0[NL];
    issue_x(0);
#pragma unroll
    for (int l = 0; l < NL; ++l) x0[l] = xr[0][l];
    constexpr int kTab = 6;   // words of the scales a thread fetches at a time
    const int swords = nt * 8 * G, zwordsall = kBytes ? 0 : nt * 16 * zwords;
    const uint32_t sbase = (uint32_t)tile0 * 32u * (uint32_t)G, zbase = (uint32_t)tile0 * 64u * (uint32_t)zwords;
    uint32_t tw[kTab], zw[2];
#pragma unroll
    for (int e = 0; e < kTab; ++e)
        tw[e] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)threadIdx.x + e * kMdThreads < swords ? sbase + 4u * (threadIdx.x + e * kMdThreads) : kPastEnd, 0, 0);
#pragma unroll
    for (int e = 0; e < 2; ++e)
        zw[e] = __builtin_amdgcn_raw_buffer_load_b32(rz, (int)threadIdx.x + e * kMdThreads < zwordsall ? zbase + 4u * (threadIdx.x + e * kMdThreads) : kPastEnd, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        issue_x(d);
        __builtin_amdgcn_sched_barrier(0);
        issue_q(d);
        __builtin_amdgcn_sched_barrier(0);
    }
    put_x(x0, 0);
    put_sums(sum_x(x0), 0);
#pragma unroll
    for (int e = 0; e < kTab; ++e)
        if ((int)threadIdx.x + e * kMdThreads < swords) reinterpret_cast<uint32_t*>(stab)[threadIdx.x + e * kMdThreads] = tw[e];
#pragma unroll
    for (int e = 0; e < 2; ++e)
        if ((int)threadIdx.x + e * kMdThreads < zwordsall) reinterpret_cast<uint32_t*>(ztab)[threadIdx.x + e * kMdThreads] = zw[e];
    for (int e = threadIdx.x + kTab * kMdThreads; e < swords; e += kMdThreads)
        reinterpret_cast<uint32_t*>(stab)[e] = __builtin_amdgcn_raw_buffer_load_b32(rs, sbase + 4u * e, 0, 0);
    for (int e = threadIdx.x + 2 * kMdThreads; e < zwordsall; e += kMdThreads)
        reinterpret_cast<uint32_t*>(ztab)[e] = __builtin_amdgcn_raw_buffer_load_b32(rz, zbase + 4u * e, 0, 0);

    // ---- fragments: lane (li, kb) reads the 16-byte piece of row li that goes with the MFMA's codes
    //   nibbles, groups of 128: word j of the lane's four is piece 4 kb + j
    //   nibbles, groups of 64: the halves of the wave exchange words first (below), so that an MFMA stays in one group
    //   bytes: words 2 j, 2 j + 1 of load h are piece 8 h + 2 kb + j
    constexpr int kPiece[4] = {0, kMode == kNib128 ? 1 : kMode == kNib64 ? 2 : 1, kMode == kNib128 ? 2 : 8,
                               kMode == kNib128 ? 3 : kMode == kNib64 ? 10 : 9};
    const int pbase = kMode == kNib128 ? 4 * kb : kMode == kNib64 ? 4 * (kb & 1) + (kb >> 1) : 2 * kb;
    uint32_t aoff[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        aoff[j] = (uint32_t)(kw * kRB * 4096 + li * 256 + ((pbase ^ li ^ kPiece[j]) << 4));
    const uint32_t soff = (uint32_t)(kw * kRB * (kGroups * 64) + kb * 16);
    uint32_t magic = 0x3B803B80u;
    asm volatile("" : "+v"(magic));

    f32x4_t acc[C][kRB];
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int rb = 0; rb < kRB; ++rb) acc[c][rb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    int pc = rot;   // the step being multiplied
    auto expand = [&](uint32_t w0, uint32_t w1) {
        if constexpr (kBytes) {   // eight signed bytes b = q + 128 -> bf16 b 2^-24: as the bits of an fp16 number, a byte is that subnormal
            const uint32_t w[2] = {w0 ^ 0x80808080u, w1 ^ 0x80808080u};
            u32x4_t o;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t f0, f1, f2, f3;   // (the compiler takes a mask and a conversion for byte 2)
                asm("v_cvt_f32_f16_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0" : "=v"(f0) : "v"(w[h]));
                asm("v_cvt_f32_f16_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1" : "=v"(f1) : "v"(w[h]));
                asm("v_cvt_f32_f16_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_2" : "=v"(f2) : "v"(w[h]));
                asm("v_cvt_f32_f16_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3" : "=v"(f3) : "v"(w[h]));
                o[2 * h] = __builtin_amdgcn_perm(f1, f0, 0x07060302u);
                o[2 * h + 1] = __builtin_amdgcn_perm(f3, f2, 0x07060302u);
            }
            return o;
        } else {
            return u32x4_t{(w0 & 0x000F000Fu) | magic, ((w0 >> 4) & 0x000F000Fu) | magic, ((w0 >> 8) & 0x000F000Fu) | magic,
                           ((w0 >> 12) & 0x000F000Fu) | magic};
        }
    };
    auto step = [&](int d, int buf) {
        float sums = 0.f;
        const unsigned char* const xb = xl + buf * xbytes;
        const unsigned char* const sb = s1 + buf * sbytes + soff;
        const int g0 = (k0 + min(pc, n_k - 1)) * kGroups;
        uint32_t w[C][4];   // groups of 64: the exchanged words
        f32x4_t dd[C][kRB];
        u32x4_t af[2][kRB];
#pragma unroll
        for (int rb = 0; rb < kRB; ++rb) af[0][rb] = *reinterpret_cast<const u32x4_t*>(xb + aoff[0] + rb * 4096);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j < 3)
#pragma unroll
                for (int rb = 0; rb < kRB; ++rb) af[(j + 1) & 1][rb] = *reinterpret_cast<const u32x4_t*>(xb + aoff[j + 1] + rb * 4096);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                u32x4_t bq;
                if constexpr (kBytes) {
                    bq = expand(q[d][c][j >> 1][2 * (j & 1)], q[d][c][j >> 1][2 * (j & 1) + 1]);
                } else if constexpr (kMode == kNib64) {
                    // lower half of the wave: k of the step's first group, upper half: of its second; after the
                    // exchange of one word's upper with the other's lower half, each belongs to one group
                    if (j == 0) {
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
                            const u32x2_t r = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_permlane32_swap(q[d][c][0][2 * p], q[d][c][0][2 * p + 1], false, false));
                            w[c][p] = r[0];
                            w[c][2 + p] = r[1];
                        }
                    }
                    bq = expand(w[c][j], 0);
                } else {
                    bq = expand(q[d][c][0][j], 0);
                }
#pragma unroll
                for (int rb = 0; rb < kRB; ++rb)
                    dd[c][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8_t, af[j & 1][rb]), __builtin_bit_cast(bf16x8_t, bq),
                        j == 0 || (kGroups == 2 && j == 2) ? f32x4_t{0.f, 0.f, 0.f, 0.f} : dd[c][rb], 0, 0, 0);
            }
            if (j == 3 || (kGroups == 2 && j == 1)) {
                const int g = g0 + (kGroups == 2 ? j >> 1 : 0);
                f32x4_t xs[kRB];
#pragma unroll
                for (int rb = 0; rb < kRB; ++rb) xs[rb] = *reinterpret_cast<const f32x4_t*>(sb + rb * (kGroups * 64) + (kGroups == 2 ? (j >> 1) * 64 : 0));
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    float s = (float)*reinterpret_cast<const _Float16*>(stab + srow[c] + (uint32_t)g * 2u);
                    if (kBytes) s *= 0x1p24f;
                    asm volatile("" : "+v"(s));   // widened once, not in every multiply-add
                    float zn = -128.f;
                    if constexpr (!kBytes) {
                        const uint32_t zword = *reinterpret_cast<const uint32_t*>(ztab + zrow[c] + (uint32_t)(g >> 3) * 4u);
                        zn = __builtin_bit_cast(float, (((zword >> (4 * (g & 7))) & 0xFu) << 16) | 0xC3000000u);   // -(128 + z)
                    }
#pragma unroll
                    for (int rb = 0; rb < kRB; ++rb)
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[c][rb][i] = fmaf(s, fmaf(zn, xs[rb][i], dd[c][rb][i]), acc[c][rb][i]);
                }
            }
            // the work for later steps, a share after each quarter's MFMAs
            if (j == 0) put_x(xr[d], buf ^ 1);
            if (j == 1) {
                sums = sum_x(xr[d]);
                issue_x(d);
            }
            if (j == 2) put_sums(sums, buf ^ 1);
        }
        if (++pc == n_max) pc = 0;
    };

    int buf = 0;
    for (int i = 0; i < n_max; i += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            if (i + u >= n_max) goto done;
            lds_barrier();   // this step's x is there, the other buffer has been read
            step(u, buf);
            __builtin_amdgcn_sched_barrier(0);
            issue_q(u);
            __builtin_amdgcn_sched_barrier(0);
            buf ^= 1;
        }
    }
done:
    // ---- the K parts meet in LDS, added in their order
    __syncthreads();
    float* const red = reinterpret_cast<float*>(lds);   // [wave][C][kRB][lane][4]
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int rb = 0; rb < kRB; ++rb) *reinterpret_cast<f32x4_t*>(red + ((wave * cmax + c) * kRB + rb) * 256 + lane * 4) = acc[c][rb];
    __syncthreads();
    for (int e = wave; e < nt * kRB; e += kMdWaves) {   // one 16 x 16 result at a time
        const int R = e / nt, t = e - R * nt;
        const int src = (t & (Wc - 1)) << wkl;
        const int c = t / Wc;
        f32x4_t v = {0.f, 0.f, 0.f, 0.f};
        for (int p = 0; p < Wk; ++p) v += *reinterpret_cast<const f32x4_t*>(red + (((src + p) * cmax + c) * kRB + R) * 256 + lane * 4);
        const int n = (tile0 + t) * 16 + li;
        if (!kBytes) v *= 0x1p15f;
        const uint32_t lo = f32x2_to_bf16x2_rne(v[0], v[1]), hi = f32x2_to_bf16x2_rne(v[2], v[3]);
        const uint16_t o[4] = {(uint16_t)lo, (uint16_t)(lo >> 16), (uint16_t)hi, (uint16_t)(hi >> 16)};
        if (n < N)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int m = 16 * R + 4 * kb + i;
                if (m < M) it.y[(size_t)m * N + n] = o[i];
            }
    }
}

// Loads of x per wave and step: four per K part and row block, dealt to eight waves; p = log2 of the K parts.
constexpr int md_loads(int rb, int p) { return ((rb << p) + 1) / 2; }

// Steps fetched ahead, by what they cost in registers: each is C (bytes: 2 C) loads of codes and NL of x.
constexpr int md_depth(int mode, int rb, int c, int nl) {
    const int per_step = (c * (mode == kByte128 ? 2 : 1) + nl) * 4;
    const int room = 256 - 80 - 8 * c * rb - 8 * rb - (mode == kNib64 ? 4 * c + 28 : 0);   // beside the sums, the operands and the addresses
    return room / per_step >= 6 ? 6 : room / per_step < 2 ? 2 : room / per_step;
}
// What fits the registers.
constexpr bool md_variant(int mode, int rb, int c, int nl) { return c <= 4 && c * rb <= (mode == kNib64 ? 9 : 12) && nl <= 8 && (nl <= 4 || c <= 2); }

template <int kMode, int kRB>
__global__ __launch_bounds__(kMdThreads, 2) void midm_kernel(const MdArgs args) {
    extern __shared__ __attribute__((aligned(16))) unsigned char md_lds[];
    int idx = 0;
    if (blockIdx.x < (unsigned)kMdMaxBlocks) idx = (args.item_of_block[blockIdx.x / 8] >> (4 * (blockIdx.x % 8))) & 15;
    idx = __builtin_amdgcn_readfirstlane(idx);
    const MdItem it = args.it[idx];
    // this wave's column tiles: one more in the first waves where they do not come out even
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), p = it.wkl, wc = kMdWaves >> p;
    const int b = (int)blockIdx.x - it.block_begin;
    const int mine = (it.tiles_base + (b < it.tiles_rem ? 1 : 0) - (wave >> p) + wc - 1) >> (3 - p);
#define MD_CASE(C, P)                                                                                                  \
    case 4 * P + C:                                                                                                     \
        if constexpr (md_variant(kMode, kRB, C, md_loads(kRB, P)))                                                       \
            md_block<kMode, kRB, C, md_loads(kRB, P), md_depth(kMode, kRB, C, md_loads(kRB, P))>(args, it, md_lds);      \
        break;
#define MD_CASES(P) MD_CASE(1, P) MD_CASE(2, P) MD_CASE(3, P) MD_CASE(4, P)
    switch (4 * p + max(mine, 1)) {
        MD_CASES(0)
        MD_CASES(1)
        MD_CASES(2)
        MD_CASES(3)
        default: break;
    }
#undef MD_CASES
#undef MD_CASE
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
MdPlan md_plan(const MdShape& s, int K, int nt) {
    MdPlan best;
    best.us = -1.f;
    const int S = K / kMdStepK, groups = s.mode == kNib64 ? 2 : 1, G = S * groups;
    const bool bytes = s.mode == kByte128;
    const size_t tables = (size_t)nt * 16 * (G * 2 + (bytes ? 0 : (G + 7) / 8 * 4));
    const float stream = (float)nt * 16.f * (float)K * (bytes ? 1.f : 0.5f) / 20000.f;
    for (int wkl = 0; (1 << wkl) <= S && wkl <= 3; ++wkl) {
        const int wc = kMdWaves >> wkl, c = (nt + wc - 1) / wc, nl = md_loads(s.rb, wkl);
        if (!md_variant(s.mode, s.rb, c, nl)) continue;
        const size_t table = (((size_t)s.rb << wkl) * (2 * 4096 + 2 * groups * 64) + 63) / 64 * 64;
        const size_t lds = std::max(table + tables, (size_t)kMdWaves * c * s.rb * 1024);
        if (lds > kMdLds) continue;
        const float tiles = c + (float)nt / wc;   // of the wave that has most and of an average one: a SIMD has two waves
        const float step = 0.5f + 0.03f * s.rb * nl + 0.065f * s.rb * tiles * (groups == 2 ? 1.5f : 1.f);
        const float us = 6.5f + std::max((float)((S + (1 << wkl) - 1) >> wkl) * step, stream);
        if (best.us < 0.f || us < best.us) {
            best.us = us;
            best.wkl = wkl;
            best.c = c;
            best.lds = lds;
            best.table = table;
        }
    }
    return best;
}

template <int kMode>
const void* md_kernel(int rb) {
    switch (rb) {
        case 1: return reinterpret_cast<const void*>(&midm_kernel<kMode, 1>);
        case 2: return reinterpret_cast<const void*>(&midm_kernel<kMode, 2>);
        case 3: return reinterpret_cast<const void*>(&midm_kernel<kMode, 3>);
        default: return reinterpret_cast<const void*>(&midm_kernel<kMode, 4>);
    }
}

int md_mode(const qail_wdesc& d, bool b8) { return b8 ? kByte128 : d.group_size == 64 ? kNib64 : kNib128; }

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

bool md_divide(const qail_w4a16_item* items, int count, int M, bool b8, MdDivision* v) {
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

hipError_t md_launch(const qail_w4a16_item* items, int count, int M, const MdDivision& v, hipStream_t st) {
    const MdShape& s = v.s;
    const void* const kernel = s.mode == kNib128 ? md_kernel<kNib128>(s.rb) : s.mode == kNib64 ? md_kernel<kNib64>(s.rb) : md_kernel<kByte128>(s.rb);
    // more than 64 KB of LDS needs an opt-in; the call is idempotent, so two host threads that
    // both find the flag clear may both make it
    static std::atomic<bool> attr_done[3][4];
    if (!attr_done[s.mode][s.rb - 1].load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMdLds);
        if (e != hipSuccess) return e;
        attr_done[s.mode][s.rb - 1].store(true, std::memory_order_release);
    }
    MdArgs a;
    memset(a.item_of_block, 0, sizeof(a.item_of_block));
    int bb = 0;
    size_t lds = 0;
    for (int i = 0; i < count; ++i) {
        const qail_w4a16_item& src = items[i];
        MdItem& t = a.it[i];
        t.qw = src.qweight; t.sc = src.scales; t.zr = src.zeros; t.x = src.x; t.y = src.y;
        t.N = src.d.N; t.K = src.d.K;
        t.block_begin = bb;
        t.tiles_base = v.tiles[i] / v.blocks[i];
        t.tiles_rem = v.tiles[i] % v.blocks[i];
        t.wkl = (uint8_t)v.plan[i].wkl;
        t.tiles_per_wave = (uint8_t)v.plan[i].c;
        t.table = (uint16_t)(v.plan[i].table / 64);
        lds = std::max(lds, v.plan[i].lds);
        for (int k = bb; k < bb + v.blocks[i] && k < kMdMaxBlocks; ++k) a.item_of_block[k / 8] |= (uint32_t)i << (4 * (k % 8));
        bb += v.blocks[i];
    }
    for (int i = count; i < kMdMaxItems; ++i) a.it[i] = a.it[count - 1];
    a.M = M;
    void* params[] = {&a};
    const hipError_t e = hipLaunchKernel(kernel, dim3(bb), dim3(kMdThreads), params, lds, st);
    return e != hipSuccess ? e : hipGetLastError();
}

// Whether the division beats the kernels that took these items before, by what was measured of both (layers of several
// widths in one call and single linears of 500 to 24000 rows and 1024 to 11008 k, M = 5 .. 64):
//   * groups of 128 and bytes up to M = 32: the small-batch kernel loses where its x takes several passes over K, so the
//     passes of an item, weighted by its bytes, decide.  Nibbles up to M = 16 from two passes on (4096 x 11008 at M = 16
//     19.4 -> 16.0 us; one pass, 4096 x 4096: 9.0 against 9.5), above from 1.3 (M = 24, the 7B layer 43.7 -> 37.6; one pass,
//     2048 x 2048: 8.0 against 9.3), bytes from 1.2 (the layer at M = 8 / 32 51.9 -> 44.6 / 63.0 -> 51.4; one pass,
//     4096 x 4096 at M = 8: 9.4 against 10.2);
//   * otherwise the matrix-core GEMM, which takes 13.5 us, 1.3 per further item and a microsecond per 3 MB, measured on the
//     low side: M = 48 the layer 56.0 -> 44.2, with bytes 71.8 -> 56.9; one 4096 x 11008, whose K the GEMM divides among
//     blocks, 22.9 against 33.7.  Groups of 64 stay below 49 rows (the layer at M = 32 / 48 53.9 -> 44.1 / 61.8 -> 59.1,
//     at M = 64 62.8 against 66.6) and need no comparison up to 16 (52.9 -> 41.5; 4096 x 4096 14.9 -> 9.9).
bool md_better(const qail_w4a16_item* items, int count, int M, const MdDivision& v) {
    if (v.s.mode == kNib64 && (M <= 16 || M > 48)) return M <= 16;
    double bytes = 0, passes = 0;
    for (int i = 0; i < count; ++i) {
        const double b = (double)items[i].d.N * items[i].d.K * (v.s.mode == kByte128 ? 1.0 : 0.5);
        bytes += b;
        if (M <= 32 && v.s.mode != kNib64) passes += b * smallm_passes(M, items[i].d.K);
    }
    if (M <= 32 && v.s.mode != kNib64) return passes >= bytes * (v.s.mode == kByte128 ? 1.2 : M <= 16 ? 2.0 : 1.3);
    const double more = v.s.mode == kByte128 ? 0.0 : std::max(0.0, bytes - 60.0e6) / 9.0e6;   // nibbles: a larger share of it expansion
    return v.us <= 13.5 + 1.3 * (count - 1) + bytes / 3.0e6 + more;
}

bool md_supports(const qail_wdesc& d, int M, bool b8) {
    if (M < 5 || M > 64 || d.K % kMdStepK != 0 || (d.group_size != 128 && (b8 || d.group_size != 64))) return false;
    if ((d.K / d.group_size) % 2 != 0) return false;   // the scales of a row are whole words
    return (unsigned long long)d.N * d.K / (b8 ? 1 : 2) <= 0x7FFFFFFFull && (unsigned long long)M * d.K * 2 <= 0x7FFFFFFFull;
}

}  // namespace

hipError_t launch_midm_if_better(const qail_w4a16_item* items, int count, int M, bool b8, hipStream_t st, int* taken) {
    *taken = 0;
    int n = 0;   // items of one group size share a launch
    while (n < count && n < kMdMaxItems && items[n].d.group_size == items[0].d.group_size && md_supports(items[n].d, M, b8)) ++n;
    MdDivision v;
    if (n == 0 || !md_divide(items, n, M, b8, &v) || !md_better(items, n, M, v)) return hipSuccess;
    *taken = n;
    return md_launch(items, n, M, v, st);
}

}  // namespace qail
