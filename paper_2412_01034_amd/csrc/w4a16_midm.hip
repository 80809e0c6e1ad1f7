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
// 30 us of the 39 that the 100 MB of codes of a 7B model's layer take from the last-level cache; the
// codes alone 24), then HBM.  That layer in one call, new buffers from call to call, before
// (smallm / GEMM) -> now, us: M = 24 / 32 / 48 44.3 / 45.9 / 56.9 -> 38.5 / 39.1 / 45.4; groups of 64
// M = 8 / 16 / 32 54.0 / 54.2 / 54.7 -> 40.2 / 40.9 / 46.7; bytes M = 8 / 32 / 48 / 64 52.3 / 64.7 / 74.6 /
// 75.4 -> 42.6 / 50.0 / 58.8 / 66.7.  (Nibbles from M = 49 on are the GEMM's there: the plan's model has 61 us for
// 54.)  The very first pass over buffers that nothing has read gains nothing: M = 48 71 to 76 us
// with either kernel, four runs.  Measured and not kept: codes fetched with the pieces of a row in neighbouring lanes (22 instead of 66 cycles of
// the address unit per load) and turned through LDS, the offset as the MFMAs' start value and the
// zero-points as fp32 MFMAs, tile-outer order, a third buffer of x: none faster.
#include <string.h>

#include <algorithm>
#include <atomic>

#include "midm_plan.h"

namespace qail {

namespace {

constexpr int kMdThreads = kMdWaves * kWave;
constexpr uint32_t kPastEnd = 0x80000000u;   // an offset no tensor here reaches: the load returns zeros and fetches nothing

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;

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

template <int kMode, int kRB>
__global__ __launch_bounds__(kMdThreads, 2) void midm_kernel(const MdArgs args) {
    extern __shared__ __attribute__((aligned(16))) unsigned char md_lds[];
    int idx = 0;
    if (blockIdx.x < (unsigned)kMdMaxBlocks) idx = (args.item_of_block[blockIdx.x / 8] >> (4 * (blockIdx.x % 8))) & 15;
    idx = __builtin_amdgcn_readfirstlane(idx);
    const MdItem it = args.it[idx];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), p = it.wkl;
    const int b = (int)blockIdx.x - it.block_begin;
    const int mine = md_wave_tiles(it.tiles_base + (b < it.tiles_rem ? 1 : 0), p, wave);
#define MD_CASE(C, P)                                                                                                  \
    case 4 * P + C:                                                                                                     \
        if constexpr (md_variant(kMode, kRB, C, P))                                                                     \
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

template <int kMode>
const void* md_kernel(int rb) {
    switch (rb) {
        case 1: return reinterpret_cast<const void*>(&midm_kernel<kMode, 1>);
        case 2: return reinterpret_cast<const void*>(&midm_kernel<kMode, 2>);
        case 3: return reinterpret_cast<const void*>(&midm_kernel<kMode, 3>);
    }
    if constexpr (kMode != kNib64) return reinterpret_cast<const void*>(&midm_kernel<kMode, 4>);
    return nullptr;   // groups of 64 have no variant for four row blocks
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

}  // namespace

hipError_t launch_midm_if_better(const qail_w4a16_item* items, int count, int M, bool b8, hipStream_t st, int* taken) {
    MdDivision v;
    *taken = md_take(items, count, M, b8, &v);
    return *taken > 0 ? md_launch(items, *taken, M, v, st) : hipSuccess;
}

}  // namespace qail
