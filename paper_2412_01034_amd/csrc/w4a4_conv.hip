// W4A4 convolution as an implicit GEMM with exact int32 accumulation.
//
//   acc[(b,oh,ow)][n] = sum_{kh,kw,c} a[b][oh*s+kh-p][ow*s+kw-p][c] * w[n][kh][kw][c]
//
// Sec. 2.1 / Sec. 5.1: the driving policy's convolutions are compute-bound, so both
// GEMM operands are 4-bit integers.  CDNA4 has no 4-bit integer matrix
// instruction, so nibbles are widened to int8 in registers and fed to
// v_mfma_i32_32x32x32_i8 (int32 accumulate):
//   * unsigned activation codes:  w & 0x0F0F0F0F  and (w >> 4) & 0x0F0F0F0F
//     give the even and the odd codes of a word as bytes;
//   * signed weight codes are moved to the HIGH nibble of each byte,
//     (w << 4) & 0xF0F0F0F0 and w & 0xF0F0F0F0, which is the int8 value 16*code,
//     so no sign extension is needed; the accumulator is 16x the result and an
//     arithmetic shift by 4 restores it exactly.
// The two operands are permuted along k in the same way (even codes, then odd
// codes of each word), which leaves the sum unchanged.
//
// MFMA operand layout (32x32x32 int8, wave64): lane l supplies row (A) / column
// (B) l%32 and the 16 consecutive k starting at 16*(l/32); register r of its 16
// results is D[8*(r/4) + 4*(l/32) + r%4][l%32].  A = weights (channels n),
// B = activations (pixels m), so that a lane has four neighbouring channels of one
// pixel at a time.  The 16x16x64 form has the same operand volume per
// multiply-add but a wave issuing nothing else reaches only 0.6 of the matrix
// rate with it (2.7 against 4.5 POP/s over the chip, measured), the 32x32x32 form all of it.
//
// Tiling: a block of 4 to 16 waves owns an output tile of 64 x 64 to 128 x 128 and walks K in
// steps of 128 codes (16 packed words per row; K is ordered (kh, kw, c), so a step
// is a run of channels of one or two filter taps).  Nibbles stay packed in LDS
// (half the LDS traffic of int8); the load unit writes the tiles of the next one or two steps
// straight into a ring of LDS slots, one barrier per step.
// Zero padding costs nothing: code 0 of the unsigned activations is the value 0.
//
// Where a launch's time goes (3x3 layers of 64 / 128 / 256 / 512 channels with a shortcut at batch 32, 5 / 9 / 18 / 36 K steps,
// launches one after the other): 10.4 / 8.9 / 8.8 / 8.8 us, of which 7.0 / 5.3 / 4.9 / 4.5 are there with a single step (launch
// cadence 2.4, operands' first trip to memory, epilogue).  The loop is bound by vector issue (widening) and, with
// 64 x 64 tiles, by what a unit takes in from L2 (300 KB a block).
#include "qail_internal.h"
#include <algorithm>
#include <cmath>

namespace qail {

namespace {

constexpr int kStepWords = 16;  // packed words per row per K step (128 codes)

struct ConvGeom {
    int B, H, W, Cin, Cout, KH, KW, stride, pad, OH, OW, M;
    // ceil(2^32 / d) for the four divisors of the tiled kernel's set-up (OH * OW, OW, words per
    // pixel, KW), valid when `fastdiv` is set: the host has checked that the high word of
    // x * magic is x / d for every x the kernel divides.
    uint32_t mg_ohow, mg_ow, mg_cw, mg_kw;
    int fastdiv;
    uint32_t row_taps;   // bit kh KW for every row kh of the filter
};

// x / d as the high word of x * ceil(2^32 / d): with e = d * magic - 2^32 (0 <= e < d) the product
// is x / d + x e / (d 2^32), and its floor is floor(x / d) as long as x e < 2^32 (then the excess
// stays below 1 / d).  `ok` tells whether that holds for every x up to xmax; d = 1 has no 32-bit
// magic and is marked by 0.
inline uint32_t div_magic(uint32_t d, uint64_t xmax, bool& ok) {
    if (d == 0) ok = false;
    if (d < 2) return 0;
    const uint64_t mg = ((1ull << 32) + d - 1) / d;
    const uint64_t e = mg * d - (1ull << 32);
    if (e * xmax >= (1ull << 32)) ok = false;
    return (uint32_t)mg;
}
__device__ __forceinline__ int div_by(int x, int d, uint32_t magic, int fast) {
    return fast ? (magic ? (int)__umulhi((uint32_t)x, magic) : x) : x / d;
}

typedef __attribute__((ext_vector_type(4))) unsigned u32x4_t;

// Raw buffer descriptor over [p, p + bytes): loads past the end return 0 and stores past the
// end are dropped by the hardware, which turns every image-border, K-tail and tile-edge test
// into the choice of an offset.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
constexpr uint32_t kOut = 0xFFFFFFF0u;  // an offset no buffer here reaches

// Where the results go.  Plain outputs: acc and / or y = fma(float(acc), scale, bias).
// Fused output (out_u4 != nullptr): the next layer's packed unsigned codes, see fused_code().
struct ConvOut {
    int32_t* acc;
    const float* scale;
    const float* bias;
    float* y;
    uint32_t* out_u4;
    const uint32_t* res_u4;
    const float* res_f32;
    float s_out, res_scale;
    float inv_s_out;  // 1 / s_out, correctly rounded (host division)
    // fused output: s_out is far from the ends of the range, the quotient may be tried as a product first;
    // plain outputs: stored past the caches (kPastCaches).  One word for both: the arguments of a batch with another
    // one in each item cost the encoder at batch 32 2 % (304 -> 310 us).
    int quick;
};

// Up to kConvBatch independent convolutions share a launch: item i is the grid's plane z = i
// (its arguments are then at an offset known when the wave starts: no load depends on another);
// the x and y axes are as large as the largest item needs, the blocks outside an item's own tile
// grid leave at once.
constexpr int kConvBatch = 4;
struct ConvItem {
    ConvGeom gm;
    const uint32_t* a;
    const uint32_t* w;
    ConvOut out;
};
struct ConvBatch {
    ConvItem it[kConvBatch];
};

// One output element of the fused epilogue (Sec. 5.1: every activation tensor of the driving
// encoder is 4-bit with one step per tensor, so the consumer's step is known here).  Each
// line is one correctly rounded fp32 operation; contraction to fma is switched off because
// the code is decided by these roundings and must equal the reference bit for bit.
__device__ __forceinline__ float fused_value(int acc, float scale, float bias, float r) {
#pragma clang fp contract(off)
    float t = (float)acc * scale;
    t = t + bias;
    return t + r;   // the ReLU is part of the clamps below
}
__device__ __forceinline__ float fused_code(float t, float s_out) {
    return fminf(__builtin_rintf(fmaxf(t, 0.f) / s_out), 15.f);
}
// The same code without the division wherever that is provably the same: u = t * fl(1 / s) is
// within 1.5 * 2^-23 (relative) of fl(t / s), so below 16 the two differ by less than 2^-18 and
// round to the same integer unless u lies within 2^-17 of a half-integer, i.e. |u - rint(u)|
// (an exact difference) exceeds 1/2 - 2^-17; `worst` keeps the largest such distance of a word and
// the caller divides when it is that large.  u is clamped to 0 .. 15 first (one median-of-three, which makes 0 of a
// NaN as the ReLU does): from 15 upwards the quotient is at least 15 - 2^-18 and the code 15, below 0 the ReLU makes it
// 0, and the clamped values are no ties, so that negative and large values do not make their waves divide.
__device__ __forceinline__ float fused_code_quick(float t, float inv_s, float& worst) {
#pragma clang fp contract(off)
    const float u = __builtin_amdgcn_fmed3f(t * inv_s, 0.f, 15.f);
    const float q = __builtin_rintf(u);
    worst = fmaxf(worst, __builtin_fabsf(u - q));
    return q;
}
// N codes (small non-negative integers held as floats) -> nibbles 0 .. N - 1 of a word: a code is
// converted into its byte of the even or the odd codes' word (11 operations per output element up to here, 14 with a
// shift and an or per code and the clamps one by one: 1 % of the body at batch 32).
template <int N>
__device__ __forceinline__ uint32_t pack_codes(const float (&q)[N]) {
    uint32_t even = 0, odd = 0;
#pragma unroll
    for (int e = 0; e < N / 2; ++e) {
        even = __builtin_amdgcn_cvt_pk_u8_f32(q[2 * e], e, even);
        odd = __builtin_amdgcn_cvt_pk_u8_f32(q[2 * e + 1], e, odd);
    }
    return even | (odd << 4);
}

// N neighbouring channels of one output pixel -> their codes; sc / bi: the channels' scales and biases, r: their
// shortcut values (0 without a shortcut: t + 0 == t).
template <int N>
__device__ __forceinline__ void fused_codes(const int (&acc)[N], const float (&sc)[N], const float (&bi)[N], const float (&r)[N],
                                            const ConvOut& o, float (&q)[N]) {
    float t[N];
#pragma unroll
    for (int e = 0; e < N; ++e) t[e] = fused_value(acc[e], sc[e], bi[e], r[e]);
    float worst = o.quick ? 0.f : 1.f;
#pragma unroll
    for (int e = 0; e < N; ++e) q[e] = fused_code_quick(t[e], o.inv_s_out, worst);
    if (__builtin_expect(!(worst <= 0.5f - 0x1p-17f), 0)) {
#pragma unroll
        for (int e = 0; e < N; ++e) q[e] = fused_code(t[e], o.s_out);
    }
}
template <int N>
__device__ __forceinline__ void load_floats(const float* p, float (&v)[N]) {   // 16-byte aligned
#pragma unroll
    for (int e = 0; e < N; e += 4) {
        const float4 a = *reinterpret_cast<const float4*>(p + e);
        v[e] = a.x; v[e + 1] = a.y; v[e + 2] = a.z; v[e + 3] = a.w;
    }
}
// Shortcut values of N channels from a word of 4-bit codes (each times its step: one rounding).
template <int N>
__device__ __forceinline__ void shortcut_from_codes(uint32_t rw, float res_scale, float (&r)[N]) {
    const uint32_t even = rw & 0x0F0F0F0Fu, odd = (rw >> 4) & 0x0F0F0F0Fu;   // a byte converts to float in one operation
#pragma unroll
    for (int e = 0; e < N; ++e) {
#pragma clang fp contract(off)
        r[e] = res_scale * (float)((((e & 1) ? odd : even) >> (8 * (e / 2))) & 0xFFu);
    }
}
__device__ __forceinline__ uint32_t fused_word(const int (&acc)[8], const ConvOut& o, size_t m, int n0, int cout) {
    float sc[8], bi[8], r[8];
    load_floats(o.scale + n0, sc);
    load_floats(o.bias + n0, bi);
    if (o.res_u4) {
        shortcut_from_codes(o.res_u4[m * (size_t)(cout / 8) + n0 / 8], o.res_scale, r);
    } else if (o.res_f32) {
        load_floats(o.res_f32 + m * (size_t)cout + n0, r);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) r[e] = 0.f;
    }
    float q[8];
    fused_codes(acc, sc, bi, r, o, q);
    return pack_codes(q);
}

// Two words of codes as MFMA operand bytes: activations as they are, weights times 16.
__device__ __forceinline__ i32x4_t widen_a(uint32_t x, uint32_t y) {
    return i32x4_t{(int)(x & 0x0F0F0F0Fu), (int)((x >> 4) & 0x0F0F0F0Fu), (int)(y & 0x0F0F0F0Fu),
                   (int)((y >> 4) & 0x0F0F0F0Fu)};
}
__device__ __forceinline__ i32x4_t widen_b(uint32_t x, uint32_t y) {
    return i32x4_t{(int)((x << 4) & 0xF0F0F0F0u), (int)(x & 0xF0F0F0F0u), (int)((y << 4) & 0xF0F0F0F0u),
                   (int)(y & 0xF0F0F0F0u)};
}

// Plain outputs of this many bytes and more (int32 and fp32 together) are stored past the caches, which the codes
// and weights need; smaller ones stay there for the operator that reads them next.  us, ordinary / past the caches,
// 3x3 layers alone and with a step search and a quantiser behind them: W8A8, 12.8 MB (32 x 28 x 28 x 128)
// 12.0 / 10.6 and 25.0 / 24.6, 6.4 MB (half the batch, below the line) 8.4 / 7.9 and 19.3 / 19.9, 0.4 MB 4.1 / 4.1 and
// 12.0 / 12.4; W4A4, 12.8 MB 10.8 / 9.8 and 23.8 / 23.0, 6.4 MB 8.1 / 7.7 and 19.3 / 19.8, 0.2 MB 3.8 / 3.9 and 9.4 / 11.0.
constexpr size_t kPastCaches = (size_t)8 << 20;

// Plain outputs of 4 consecutive channels n0.. of a pixel, o = their position; 16-byte stores when Cout allows
// (sc, bi: the channels' scales and biases, fetched by the caller in that case).
__device__ __forceinline__ void store_plain(const i32x4_t v, const ConvOut& out, size_t o, int n0, int cout, const float4 sc,
                                            const float4 bi) {
    if ((cout % 4) == 0) {
        i32x4_t* const acc = reinterpret_cast<i32x4_t*>(out.acc + o);
        f32x4_t* const y = reinterpret_cast<f32x4_t*>(out.y + o);
        const f32x4_t f = {fmaf((float)v[0], sc.x, bi.x), fmaf((float)v[1], sc.y, bi.y), fmaf((float)v[2], sc.z, bi.z),
                           fmaf((float)v[3], sc.w, bi.w)};
        // (in this shape: of two alternatives for one store the compiler makes a single ordinary one)
        if (out.quick) {
            if (out.acc) __builtin_nontemporal_store(v, acc);
            if (out.y) __builtin_nontemporal_store(f, y);
        } else {
            if (out.acc) *acc = v;
            if (out.y) *y = f;
        }
    } else {
        for (int e = 0; e < 4 && n0 + e < cout; ++e) {
            if (out.acc) out.acc[o + e] = v[e];
            if (out.y) out.y[o + e] = fmaf((float)v[e], out.scale[n0 + e], out.bias[n0 + e]);
        }
    }
}

// Global -> LDS copy by the load unit through a buffer descriptor: lane l's 16 bytes at byte
// offset `off` of the buffer land at LDS address lds + 16 l; a lane whose offset lies outside the
// buffer writes 16 zero bytes (checked on the GPU with a probe), which is exactly what image
// borders, the K tail and tile edges need.  Assembly on purpose: the compiler would make every
// later LDS read wait for all such copies in flight (it cannot tell the ring slots apart).
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x4_t make_rsrc_words(const void* p, uint32_t bytes) {
    const uint64_t b = (uint64_t)(uintptr_t)p;
    u32x4_t r = {(uint32_t)b, (uint32_t)(b >> 32) & 0xFFFFu, bytes, 0x00020000u};
    r[0] = __builtin_amdgcn_readfirstlane(r[0]);
    r[1] = __builtin_amdgcn_readfirstlane(r[1]);
    r[2] = __builtin_amdgcn_readfirstlane(r[2]);
    r[3] = __builtin_amdgcn_readfirstlane(r[3]);
    return r;
}
__device__ __forceinline__ void dma16(u32x4_t rsrc, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(lds), "v"(off), "s"(rsrc) : "memory", "m0");
}
__device__ __forceinline__ void dma4(u32x4_t rsrc, uint32_t off, uint32_t lds) {   // lane l's 4 bytes at lds + 4 l
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 :: "s"(lds), "v"(off), "s"(rsrc) : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p);
}
__host__ __device__ constexpr int waitcnt_vm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4); }  // lgkmcnt 0 too

template <int kCtrl>
__device__ __forceinline__ float dpp(float v) {   // v of another lane of the row
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), kCtrl, 0xF, 0xF, false));
}

constexpr int kMaxSteps = 128;  // rows of the step table (K steps plus the ring's look-ahead)

// Tiling: a block owns a BM x BN output tile, WM x WN waves side by side with 32 UM x 32 UN of it each, and walks K in
// steps of 128 codes (64 B per row; K is ordered (kh, kw, c) and Cin % 32 == 0, so every 16-byte chunk lies
// inside one filter tap).  Rows are unpadded in LDS; chunk c of row r is kept at position
// c ^ swz(r), swz(r) = ((r / 4) % 4) ^ (r & 2), chosen through the loading lane's address: the
// 16-byte fragment reads of 8 consecutive rows then fall into 8 different 16-byte columns of
// a 128-byte line, and those of 16 consecutive rows into 16 different ones of a 256-byte line.
//
// KS > 1: KS groups of WM x WN waves share the tile and split K between them (group g takes steps
// g, g + KS, ...), each with its own ring of ST slots; the waves with the same part of the tile then hand each other pieces of
// it through LDS, so that each finishes one KS-th (integer sums: exact in any order).
//
// What bounds it is the number of vector instructions: a lone wave on a SIMD issues one per 8 cycles, two or more
// one per 4.5 together (a loop of MFMAs and ANDs: 30 / 16 ns per 8 of them), and at batch 32 a SIMD has two to four waves for
// the whole launch.  So what a row or a step needs is worked out once per block, into tables (a row's address and taps,
// a step's offsets; by every lane for the rows it loads: 3 to 6 % slower); the weights' addresses need no test (rows past Cout load the
// last one, steps past the end the last one, and neither reaches a result); halves of a K step past the end of K are not
// multiplied (64 channels: 4.5 steps, not 5); the fused epilogue works from the registers, in units of the output step (see
// there); the ring has two slots where three would leave room for fewer blocks on a unit.  Before, every lane worked out its
// own rows, the sums went through LDS and the epilogue took 11 operations per element (now 7, with a shortcut 9 instead
// of 13).  3x3 layers with a shortcut, before / now: 64 channels, 56 x 56, batch 32 / 64 / 256 12.0 / 10.3, 18.3 / 15.7,
// 60.2 / 50.7 us; 96 to 160 channels, 17 x 40 x 43 14.3 / 10.6; 256, 14 x 14, batch 48 13.5 / 10.8.
//
// kBits = 8 is the W8A8 variant of the same kernel (Sec. 5.4): bytes are MFMA operands as they
// are, a K step is 64 codes and one MFMA deep, nothing is widened and nothing shifted back.
//
// The tile at rows bm.., columns bn.. of one convolution; the two kernels below call it.
template <int UM, int UN, int WM, int WN, int KS, int ST, int kBits>
__device__ __forceinline__ void w4a4_conv_tile(const ConvGeom& gm, const uint32_t* __restrict__ a, const uint32_t* __restrict__ w,
                                               const ConvOut& out, const int bm, const int bn) {
    constexpr int G = WM * WN;                       // waves of a K group
    constexpr int BM = 32 * UM * WM, BN = 32 * UN * WN;
    constexpr int kThreads = 64 * G * KS;
    constexpr int kLA = BM / (16 * G);   // wave-wide loads per wave and step for the activation tile
    constexpr int kLB = BN / (16 * G);   // ... for the weight tile
    constexpr int kL = kLA + kLB;
    constexpr int kStageBytes = (BM + BN) * 64;
    constexpr int kQuads = 4 * UM * UN, kOwn = kQuads / KS;   // a wave's tile in pieces of 32 pixels x 8 channels, and how many it finishes
    constexpr int kHandBytes = (KS - 1) * kQuads * 1024 * G / KS;   // handed over per group
    constexpr int kGroupBytes = ST * kStageBytes > kHandBytes ? ST * kStageBytes : kHandBytes;
    static_assert(BM % (16 * G) == 0 && BN % (16 * G) == 0 && BM <= kThreads && BN % 64 == 0, "loads and tables divide evenly");
    static_assert(kQuads % KS == 0 && (kOwn == 1 || kOwn % 2 == 0), "a wave finishes one piece or pairs of them");
    static_assert((KS - 1) * kQuads * 1024 * G <= KS * kGroupBytes && kStageBytes % 16 == 0 && kGroupBytes % 16 == 0, "pieces fit the rings");
    static_assert(ST == 2 || ST == 3, "slots of a ring");
    __shared__ __attribute__((aligned(16))) unsigned char ring[KS * kGroupBytes];
    // scales, biases; fused: the same in units of the output step (bytes keep them in registers, and their blocks of three
    // slots and 128 x 64 or 64 x 128 to 40 KB, so that four fit a unit)
    __shared__ __attribute__((aligned(16))) float chan[4][kBits == 4 ? BN : 1];
    __shared__ float limit[kBits == 4 ? BN / 8 : 1];             // fused: how far from an integer a quick quotient may be
    __shared__ uint2 steptab[kMaxSteps * 4];
    __shared__ __attribute__((aligned(16))) unsigned char resid[kBits == 4 ? BM * BN / 2 : 16];   // the tile of the shortcut's codes

    const int t = threadIdx.x;
    const int lane = t % kWave;
    const int wave_all = __builtin_amdgcn_readfirstlane(t / kWave);
    const int grp = wave_all / G, wave = wave_all % G;   // K group, wave inside the group
    unsigned char* const smem = ring + grp * kGroupBytes;
    const int wm = wave / WN, wn = wave % WN;
    const int cw = gm.Cin / (32 / kBits);      // words per pixel
    const int kwords = gm.KH * gm.KW * cw;     // words per filter (a multiple of 4)
    const int gsteps = (kwords + kStepWords - 1) / kStepWords;   // K steps of the whole problem
    const int steps = (gsteps + KS - 1) / KS;                     // ... of one group (the same for all)
    const bool fused = kBits == 4 && out.out_u4;                  // (bytes have plain outputs only)

    const u32x4_t ra = make_rsrc_words(a, (uint32_t)((size_t)gm.B * gm.H * gm.W * cw * 4));
    const u32x4_t rw = make_rsrc_words(w, (uint32_t)((size_t)gm.Cout * kwords * 4));
    const uint32_t lds0 = lds_address(smem);

    // Scales and biases first: wave c takes channels 64 c .. 64 c + 63 and, for fused outputs, works on them below.
    if (kBits == 4 && wave_all < BN / 64 && out.scale && out.bias) {
        const u32x4_t rs = make_rsrc_words(out.scale, (uint32_t)gm.Cout * 4), rb = make_rsrc_words(out.bias, (uint32_t)gm.Cout * 4);
        const uint32_t c0 = lds_address(&chan[0][0]) + wave_all * 256;
        dma4(rs, (uint32_t)(bn + t) * 4u, c0);
        dma4(rb, (uint32_t)(bn + t) * 4u, c0 + BN * 4);
    }

    // Loader geometry: load i of this wave fills rows (G i + wave) * 16 + lane / 4, position
    // lane % 4, with the chunk that belongs there.
    const int lrow = lane >> 2;
    const int chunk = (lane & 3) ^ ((lrow >> 2) & 3) ^ (lrow & 2);  // which 16 bytes of a step this lane fetches
    // Weights: rows past Cout load the last one (their results are not stored), steps past the end of K the last one
    // (not multiplied).  A chunk past the end of K inside the last step is the next row's first or lies past the tensor: the
    // activations it meets are zeros.
    uint32_t bbase[kLB];
#pragma unroll
    for (int i = 0; i < kLB; ++i)
        bbase[i] = (uint32_t)min(bn + (G * i + wave) * 16 + lrow, gm.Cout - 1) * (uint32_t)(kwords * 4) + chunk * 16;
    auto issue_w = [&](int step, int slot) {
        const uint32_t k4 = (uint32_t)min(step, gsteps - 1) * (kStepWords * 4);
#pragma unroll
        for (int i = 0; i < kLB; ++i) dma16(rw, bbase[i] + k4, lds0 + slot * kStageBytes + BM * 64 + (G * i + wave) * 1024);
    };
    issue_w(grp, 0);
    issue_w(KS + grp, 1);

    // Where a pixel is: byte offset of (b, ih0, iw0, 0), which may be negative at the border, and a bit per tap that
    // lies outside the image (all of them for rows past the end).
    auto pixel = [&](int m) {
        uint2 v = make_uint2(0u, 0xFFFFFFFFu);
        if (m < gm.M) {
            const int b = div_by(m, gm.OH * gm.OW, gm.mg_ohow, gm.fastdiv);
            const int rem = m - b * (gm.OH * gm.OW);
            const int oh = div_by(rem, gm.OW, gm.mg_ow, gm.fastdiv), ow = rem - oh * gm.OW;
            const int ih0 = oh * gm.stride - gm.pad, iw0 = ow * gm.stride - gm.pad;
            v.x = (uint32_t)(((b * gm.H + ih0) * gm.W + iw0) * cw * 4);
            // taps inside the image: kw in [kw_lo, kw_hi) for every kh in [kh_lo, kh_hi); at most 32 taps, and the product
            // copies the bits of a row (fewer than KW + 1) to every row kept
            const int kw_lo = max(0, -iw0), kw_n = min(gm.KW, gm.W - iw0) - kw_lo;
            const int kh_lo = max(0, -ih0), kh_n = min(gm.KH, gm.H - ih0) - kh_lo;
            if (kw_n > 0 && kh_n > 0)
                v.y = ~(((0xFFFFFFFFu >> (32 - kw_n)) << kw_lo) *
                        (gm.row_taps & ((0xFFFFFFFFu >> (32 - kh_n * gm.KW)) << (kh_lo * gm.KW))));
        }
        return v;
    };
    // Where a K step's chunks come from is the same for every row: for (step, chunk) the byte offset of the chunk from a
    // pixel's (ih0, iw0, 0) and its tap.  Chunks past the end of K get tap 31, which is outside the image for every row:
    // there are such chunks only where K is no whole number of steps, i.e. with fewer than 32 taps (32 of them are
    // 128 words or more).  Steps past the end repeat the last one.
    auto entry = [&](int step, int ch) {
        const int kw0 = min(step, gsteps - 1) * kStepWords + ch * 4;   // first word of the chunk
        uint2 v = make_uint2(0u, 31u);
        if (kw0 < kwords) {
            const int tap = div_by(kw0, cw, gm.mg_cw, gm.fastdiv), cword = kw0 - tap * cw;
            const int kh = div_by(tap, gm.KW, gm.mg_kw, gm.fastdiv), kwi = tap - kh * gm.KW;
            v.x = (uint32_t)(((kh * gm.W + kwi) * cw + cword) * 4);
            v.y = (uint32_t)tap;
        }
        return v;
    };
    // (the rows' table is in the third slot of a ring, which is empty until the K loop, where there is one)
    __shared__ uint2 rows_apart[ST == 3 ? 1 : BM];
    uint2* const rowtab = ST == 3 ? reinterpret_cast<uint2*>(ring + 2 * kStageBytes) : rows_apart;
    if (t < BM) rowtab[t] = pixel(bm + t);
    for (int e = kThreads - 1 - t; e < (steps + 3) * KS * 4; e += kThreads) steptab[e] = entry(e >> 2, e & 3);
    __syncthreads();
    uint32_t abase[kLA], aout[kLA];
#pragma unroll
    for (int i = 0; i < kLA; ++i) {
        const uint2 v = rowtab[(G * i + wave) * 16 + lrow];
        abase[i] = v.x;
        aout[i] = v.y;
    }
    const uint2 e0 = steptab[grp * 4 + chunk], e1 = steptab[(KS + grp) * 4 + chunk];
    auto issue_a = [&](const uint2 e, int slot) {
#pragma unroll
        for (int i = 0; i < kLA; ++i) {
            const uint32_t miss = (uint32_t)__builtin_amdgcn_sbfe((int)aout[i], e.y, 1);   // 0, or all ones: an offset past every buffer
            dma16(ra, (abase[i] + e.x) | (miss << 4), lds0 + slot * kStageBytes + (G * i + wave) * 1024);
        }
    };
    issue_a(e0, 0);
    if constexpr (kBits == 4) {
        // the shortcut's codes go into LDS behind the first step: they then cost the end, where the multiplying has stopped, no
        // trip to memory, and the loop no registers
        if (fused && out.res_u4) {
            const u32x4_t rr = make_rsrc_words(out.res_u4, (uint32_t)((size_t)gm.M * gm.Cout / 2));
            const uint32_t r0 = lds_address(resid);
            if (gm.Cout % 32 == 0) {   // 32 channels of a pixel per lane (16 bytes that are inside the tensor or not as a whole)
                constexpr int kPer = BN / 32;
                for (int c = wave_all; c < BM * kPer / 64; c += G * KS) {
                    const int m = bm + (c * 64 + lane) / kPer, n = bn + lane % kPer * 32;
                    dma16(rr, m < gm.M && n < gm.Cout ? (uint32_t)m * (uint32_t)(gm.Cout / 2) + (uint32_t)(n / 2) : kOut, r0 + c * 1024);
                }
            } else {
                constexpr int kPer = BN / 8;
                for (int c = wave_all; c < BM * kPer / 64; c += G * KS) {
                    const int m = bm + (c * 64 + lane) / kPer, n = bn + lane % kPer * 8;
                    dma4(rr, m < gm.M && n < gm.Cout ? (uint32_t)m * (uint32_t)(gm.Cout / 2) + (uint32_t)(n / 2) : kOut, r0 + c * 256);
                }
            }
        }
    }
    issue_a(e1, 1);
    // (bytes: columns fixed per thread, see the stores)
    const int nq = (t % (BN / 4)) * 4;
    float4 sc = make_float4(0.f, 0.f, 0.f, 0.f), bi = sc;
    if (kBits == 8 && out.y && gm.Cout % 4 == 0 && bn + nq < gm.Cout) {
        sc = *reinterpret_cast<const float4*>(out.scale + bn + nq);
        bi = *reinterpret_cast<const float4*>(out.bias + bn + nq);
    }

    // Fragment reads for the 32 x 32 x 32 MFMA (a wave issuing only 16 x 16 x 64 ones reaches 0.6 of
    // the matrix rate, measured): lane (r32, kh) supplies 16 codes of row r32 to each MFMA, as
    // the half kh of the MFMA's 32.  Which codes those are is free as long as both operands
    // agree, so a lane reads whole 16-byte chunks (an 8-byte read of one half of a chunk by
    // every lane leaves half of the banks idle).  4-bit: chunk 2 sub + kh of the K step, whose
    // first 8 bytes go to the first MFMA of the half-step `sub` and the rest to the second.
    // 8-bit: chunk 2 h + kh for MFMA h of the step.
    const int r32 = lane & 31, kh = lane >> 5;
    const int swz = ((r32 >> 2) & 3) ^ (r32 & 2);
    int foff[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) foff[u] = r32 * 64 + (((2 * u + kh) ^ swz) << 4);

    i32x16_t acc[UM][UN];
#pragma unroll
    for (int i = 0; i < UM; ++i)
#pragma unroll
        for (int j = 0; j < UN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    i32x4_t af[2][UM][2], bf[2][UN][2];
    auto fetch = [&](int slot, int sub, int reg) {
        const unsigned char* As = smem + slot * kStageBytes + wm * (32 * UM) * 64;
        const unsigned char* Bs = smem + slot * kStageBytes + BM * 64 + wn * (32 * UN) * 64;
        if constexpr (kBits == 4) {
#pragma unroll
            for (int i = 0; i < UM; ++i) {
                const uint4 p = *reinterpret_cast<const uint4*>(As + foff[sub] + i * 32 * 64);
                af[reg][i][0] = widen_a(p.x, p.y);
                af[reg][i][1] = widen_a(p.z, p.w);
            }
#pragma unroll
            for (int j = 0; j < UN; ++j) {
                const uint4 p = *reinterpret_cast<const uint4*>(Bs + foff[sub] + j * 32 * 64);
                bf[reg][j][0] = widen_b(p.x, p.y);
                bf[reg][j][1] = widen_b(p.z, p.w);
            }
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int i = 0; i < UM; ++i)
                    af[reg][i][h] = *reinterpret_cast<const i32x4_t*>(As + foff[h] + i * 32 * 64);
#pragma unroll
                for (int j = 0; j < UN; ++j)
                    bf[reg][j][h] = *reinterpret_cast<const i32x4_t*>(Bs + foff[h] + j * 32 * 64);
            }
        }
    };
    auto multiply = [&](int reg) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < UM; ++i)
#pragma unroll
                for (int j = 0; j < UN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(bf[reg][j][h], af[reg][i][h], acc[i][j], 0, 0, 0);
        // issue order: the LDS reads and the widening of the next fragments go between the MFMAs
        constexpr int kM = 2 * UM * UN, kF = 2 * (UM + UN);   // MFMAs, operand fragments
        constexpr int kR = kBits == 4 ? kF / 2 : kF;           // LDS reads (4-bit: one per two fragments)
        constexpr int kRead = (kR + kM - 1) / kM;
#pragma unroll
        for (int u = 0; u < kM; ++u) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (u * kRead < kR) __builtin_amdgcn_sched_group_barrier(0x100, kRead, 0);
            if (kBits == 4) __builtin_amdgcn_sched_group_barrier(0x002, (4 * kF + kM - 1) / kM, 0);
        }
    };

    // Fused output, in units of the output step: u = (16 acc) c1 + c0 + shortcut with c1 = fl(scale fl(1 / s)) / 16 and
    // c0 = fl(bias fl(1 / s)) takes two roundings where the reference (fused_value, fused_code) takes three and a division.  With e = 2^-24
    // and B, C the magnitudes of bias and shortcut over s, the two differ by less than e (3 |acc scale / s| + 2 B + 3 C + the
    // partial sums) <= 8 e (|u| + B + C), so where u (clamped to 0 .. 15) is further than 2^-21 (16 + B + C), and an eighth
    // more for the terms of second order, from a half-integer, both round to the same code; `limit` keeps one half minus that
    // for each word of eight channels.  Nothing overflows on either path as long as c1, B and C are small against 2^100 and s
    // is between 2^-100 and 2^100 (quick).  Other words are worked out as the reference does.
    if (fused && t < BN) {   // (whole waves, each with what it loaded itself: in flight behind it are two steps, and at most the shortcut)
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * kL) : "memory");
        const float inv = out.inv_s_out, c1 = chan[0][t] * inv, c0 = chan[1][t] * inv;
        chan[2][t] = c1 * 0.0625f;
        chan[3][t] = c0;
        // 2^100 stands for what may not be quick at all, a NaN among it
        float bias = __builtin_fabsf(c1) < 0x1p100f && __builtin_fabsf(c0) < 0x1p100f ? __builtin_fabsf(c0) : 0x1p100f;
        bias = fmaxf(bias, dpp<0xB1>(bias));    // the word's eight lanes: neighbours, pairs, quads
        bias = fmaxf(bias, dpp<0x4E>(bias));
        bias = fmaxf(bias, dpp<0x141>(bias));
        const float lim = 0.5f - 0x1.2p-21f * (16.f + bias + (out.res_u4 ? 15.f * __builtin_fabsf(out.res_scale * inv) : 0.f));
        if (t % 8 == 0) limit[t / 8] = out.quick && lim > 0.25f ? lim : -1.f;
    }

    // in flight: weights of steps 0 and 1, pixels of step 0, the shortcut, pixels of step 1
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(kLA));
    __syncthreads();
    int pstep = 2;
    uint2 pent = steptab[(pstep * KS + grp) * 4 + chunk];   // the next step to load, its entry read one step ahead
    fetch(0, 0, 0);

    // slot of step s + 2: with three slots step s - 1 had it, whose last reads were issued before the previous barrier; with
    // two step s itself, whose last reads every wave has issued (and waited for) at the step's barrier
    auto refill = [&](int slot) {
        const uint2 e = pent;
        issue_w(pstep * KS + grp, slot);
        ++pstep;
        pent = steptab[(pstep * KS + grp) * 4 + chunk];
        issue_a(e, slot);
    };
    // in flight at a step's wait: step s + 1 and, with three slots, step s + 2
    if constexpr (kBits == 4) {
        // One K step: slot `cur`, the next step's `nxt`, the one to refill `fill`.  Only the last step of the problem can have one half, so
        // only a group's last step asks how many halves there are (a branch in the loop keeps a half's reads and widening from
        // going between the other half's MFMAs).
        auto step = [&](int cur, int nxt, int fill, int left) {
            __builtin_amdgcn_sched_barrier(0);
            fetch(cur, 1, 1);
            if (left > 0) multiply(0);
            __builtin_amdgcn_sched_barrier(0);
            if (ST == 3) refill(fill);
            __builtin_amdgcn_s_waitcnt(waitcnt_vm(ST == 3 ? kL : 0));
            __syncthreads();
            if (ST == 2) refill(fill);
            __builtin_amdgcn_sched_barrier(0);
            fetch(nxt, 0, 0);
            if (left > 1) multiply(1);
        };
        for (int s0 = 0; s0 < steps - 1; s0 += ST) {
#pragma unroll
            for (int u = 0; u < ST; ++u) {
                if (s0 + u >= steps - 1) break;
                step(u, (u + 1) % ST, (u + 2) % ST, 2);
            }
        }
        const int last = (steps - 1) % ST, halves = (kwords + kStepWords / 2 - 1) / (kStepWords / 2);   // half-steps of the whole problem
        step(last, (last + 1) % ST, (last + 2) % ST, halves - 2 * ((steps - 1) * KS + grp));
    } else {
        // one MFMA step per K step: the operand registers alternate with the step's parity, so a ring of three is unrolled twice
        constexpr int kTurn = ST % 2 ? 2 * ST : ST;
        for (int s0 = 0; s0 < steps; s0 += kTurn) {
#pragma unroll
            for (int u = 0; u < kTurn; ++u) {
                if (s0 + u >= steps) break;
                const int nxt = (u + 1) % ST, fill = (u + 2) % ST, reg = u & 1;
                const int left = gsteps - ((s0 + u) * KS + grp);
                __builtin_amdgcn_sched_barrier(0);
                if (ST == 3) refill(fill);
                __builtin_amdgcn_s_waitcnt(waitcnt_vm(ST == 3 ? kL : 0));
                __syncthreads();
                if (ST == 2) refill(fill);
                __builtin_amdgcn_sched_barrier(0);
                fetch(nxt, 0, reg ^ 1);
                if (KS == 1 || left > 0) multiply(reg);
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));  // nothing may still be writing LDS

    // Epilogue.  Piece p of the wave's tile: block (i, j), quad q (registers 4 q ..: channels 8 q + 4 kh + 0..3 of pixel r32); two neighbouring
    // pieces are quads q and q + 2 of a block.
    auto piece = [&](int o, int& i, int& j, int& q) {   // the wave's own piece o
        const int p = KS == 1 ? o : grp * kOwn + o;
        i = p / (4 * UN);
        j = p / 4 % UN;
        q = p % 4 / 2 + 2 * (p % 2);
    };
    auto quad = [&](int p) {
        const i32x16_t& v = acc[p / (4 * UN)][p / 4 % UN];
        const int at = 4 * (p % 4 / 2 + 2 * (p % 2));
        return i32x4_t{v[at], v[at + 1], v[at + 2], v[at + 3]};
    };
    // What a lane has of own piece o once the halves of the wave have changed places (see below): its first channel and row in the tile.
    constexpr int kE = kOwn == 1 ? 4 : 8;   // channels of a lane at a time
    auto at_lane = [&](int o, int& nl, int& row) {
        int i, j, q;
        piece(o, i, j, q);
        nl = (wn * UN + j) * 32 + 8 * q + (kE == 8 ? 16 * kh : 4 * kh);
        row = (wm * UM + i) * 32 + r32;
    };
    const bool res_codes = out.res_u4 != nullptr, res_floats = out.res_f32 != nullptr;
    float r[4 * kOwn];   // a real-valued shortcut, requested before the pieces change hands where K is split
    auto request = [&](int o) {
        int nl, row;
        at_lane(o, nl, row);
        const bool in = bm + row < gm.M && bn + nl < gm.Cout;
#pragma unroll
        for (int e = 0; e < kE; e += 4) {
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (in) v = *reinterpret_cast<const float4*>(out.res_f32 + (size_t)(bm + row) * gm.Cout + bn + nl + e);
            r[4 * o + e] = v.x; r[4 * o + e + 1] = v.y; r[4 * o + e + 2] = v.z; r[4 * o + e + 3] = v.w;
        }
    };
    if (KS > 1 && fused && res_floats) {
#pragma unroll
        for (int o = 0; o < kOwn; o += kE / 4) request(o);
    }
    // Plain outputs of groups whose rings hold a whole tile each are added up on their way out instead (see there).
    constexpr int kPitch = BN + 4;
    constexpr bool kSumOut = KS > 1 && kGroupBytes >= BM * kPitch * 4;
    i32x4_t own[kOwn];
    if constexpr (KS == 1) {
#pragma unroll
        for (int o = 0; o < kOwn; ++o) own[o] = quad(o);
    } else if (fused || !kSumOut) {
        __syncthreads();   // the rings have been read
        unsigned char* const hand = ring + wave * ((KS - 1) * kQuads * 1024) + lane * 16;
#pragma unroll
        for (int p = 0; p < kQuads; ++p) {
            const int owner = p / kOwn;
            if (owner != grp)
                *reinterpret_cast<i32x4_t*>(hand + ((owner * (KS - 1) + (grp < owner ? grp : grp - 1)) * kOwn + p % kOwn) * 1024) = quad(p);
        }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < KS; ++g)
            if (grp == g) {
#pragma unroll
                for (int o = 0; o < kOwn; ++o) own[o] = quad(g * kOwn + o);
            }
#pragma unroll
        for (int s = 0; s < KS - 1; ++s)
#pragma unroll
            for (int o = 0; o < kOwn; ++o)
                own[o] += *reinterpret_cast<const i32x4_t*>(hand + ((grp * (KS - 1) + s) * kOwn + o) * 1024);
    }

    if (fused) {
        const float cr = out.res_scale * out.inv_s_out;
#pragma unroll
        for (int o = 0; o < kOwn; o += kE / 4) {
            int nl, row;
            at_lane(o, nl, row);
            int av[kE];
            // Two pieces: the halves of the wave change places, so that lanes 0-31 have the eight channels of quad q, the
            // others those of quad q + 2.  (Four channels at a time, with their packed codes changing places, was 2-3 % slower.)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (kE == 8) {
                    const auto sw = __builtin_amdgcn_permlane32_swap((unsigned)own[o][e], (unsigned)own[o + 1][e], false, false);
                    av[e] = (int)sw[0];
                    av[4 + e] = (int)sw[1];
                } else {
                    av[e] = own[o][e];
                }
            }
            const int nw = kE == 8 ? nl : nl - 4 * kh, m = bm + row, n0 = bn + nw;   // (the lane's word begins at nw)
            const bool in = m < gm.M && n0 < gm.Cout;
            float c1[kE], c0[kE], u[kE], q[kE], worst = 0.f, lim = limit[nl / 8];
            load_floats(&chan[2][nl], c1);
            load_floats(&chan[3][nl], c0);
#pragma unroll
            for (int e = 0; e < kE; ++e) u[e] = fmaf((float)av[e], c1[e], c0[e]);
            uint32_t rw8 = 0;
            if (res_codes) {
                rw8 = *reinterpret_cast<const uint32_t*>(resid + row * (BN / 2) + nw / 2);
                if (kE == 4) rw8 >>= 16 * kh;
                const uint32_t even = rw8 & 0x0F0F0F0Fu, odd = (rw8 >> 4) & 0x0F0F0F0Fu;   // a byte converts to float in one operation
#pragma unroll
                for (int e = 0; e < kE; ++e)
                    u[e] = fmaf((float)((((e & 1) ? odd : even) >> (8 * (e / 2))) & 0xFFu), cr, u[e]);
            } else if (res_floats) {
                if constexpr (KS == 1) request(o);
                float top = 0.f;
#pragma unroll
                for (int e = 0; e < kE; ++e) {
                    u[e] = fmaf(r[4 * o + e], out.inv_s_out, u[e]);
                    top = fmaxf(top, __builtin_fabsf(r[4 * o + e]));
                }
                lim -= 0x1.2p-21f * (top * out.inv_s_out);   // (C above; below zero nothing is quick)
            }
#pragma unroll
            for (int e = 0; e < kE; ++e) {
                u[e] = __builtin_amdgcn_fmed3f(u[e], 0.f, 15.f);   // (0 of a NaN, as the ReLU makes of it)
                q[e] = __builtin_rintf(u[e]);
                worst = fmaxf(worst, __builtin_fabsf(u[e] - q[e]));
            }
            if (__builtin_expect(!(worst <= lim), 0)) {
                float sc[kE], bi[kE], sh[kE];
                load_floats(&chan[0][nl], sc);
                load_floats(&chan[1][nl], bi);
                shortcut_from_codes(rw8, res_codes ? out.res_scale : 0.f, sh);
                int ex[kE];
#pragma unroll
                for (int e = 0; e < kE; ++e) {
                    ex[e] = av[e] >> 4;   // 4-bit: the accumulator is 16 * result
                    if (res_floats) sh[e] = r[4 * o + e];
                }
                fused_codes(ex, sc, bi, sh, out, q);
            }
            uint32_t word = pack_codes(q);
            if constexpr (kE == 4) {   // lanes 0-31 take the four channels of lanes 32-63 as well
                const auto sw = __builtin_amdgcn_permlane32_swap(word, word, false, false);
                word |= sw[1] << 16;
            }
            if (in && (kE == 8 || kh == 0)) out.out_u4[(uint32_t)m * (uint32_t)(gm.Cout / 8) + (uint32_t)n0 / 8u] = word;
        }
    } else if constexpr (kSumOut) {
        // Plain outputs of a tile whose K was split: every group stages its sums, the piece of a row that a thread stores is added up
        // as it is read: two barriers, where handing over and staging take four.  us, handed over / this, W8A8 of
        // 256 channels, 36 steps, 4 x 17 x 16 pixels 7.36 / 7.16, of 384, 54 steps, 9 x 14 x 16 9.75 / 9.48, W4A4 of 256, 18 steps 6.24 / 6.07.
        int32_t* const stage = reinterpret_cast<int32_t*>(smem);
        if (kBits == 4 && out.y) {
            sc = *reinterpret_cast<const float4*>(&chan[0][nq]);
            bi = *reinterpret_cast<const float4*>(&chan[1][nq]);
        }
        __syncthreads();   // the rings have been read
#pragma unroll
        for (int p = 0; p < kQuads; ++p) {
            const int i = p / (4 * UN), j = p / 4 % UN, qd = p % 4 / 2 + 2 * (p % 2);
            *reinterpret_cast<i32x4_t*>(&stage[((wm * UM + i) * 32 + r32) * kPitch + (wn * UN + j) * 32 + 8 * qd + 4 * kh]) = quad(p);
        }
        __syncthreads();
        for (int row = t / (BN / 4); row < BM; row += kThreads / (BN / 4)) {
            const int m = bm + row, n = bn + nq;
            if (m >= gm.M || n >= gm.Cout) continue;
            i32x4_t v = {0, 0, 0, 0};
#pragma unroll
            for (int g = 0; g < KS; ++g) v += *reinterpret_cast<const i32x4_t*>(ring + g * kGroupBytes + (row * kPitch + nq) * 4);
            if (kBits == 4) v >>= 4;
            store_plain(v, out, (size_t)m * gm.Cout + n, n, gm.Cout, sc, bi);
        }
    } else {
        // Plain outputs leave as whole pieces of rows, through LDS (pitch BN + 4 words: the 16-byte writes of eight neighbouring
        // pixels fall on different banks), as many blocks of 32 rows at a time as the rings hold.  Stored from the registers, 32
        // bytes of each of 32 rows at a time, 12.8 MB took 30 us instead of 11.
        constexpr int kFit = KS * kGroupBytes / (32 * kPitch * 4), kBlocks = UM * WM;
        constexpr int kAtOnce = kFit < kBlocks ? kFit : kBlocks;
        static_assert(kAtOnce >= 1 && kBlocks % kAtOnce == 0 && kThreads % (BN / 4) == 0, "whole turns; columns fixed per thread");
        int32_t* const stage = reinterpret_cast<int32_t*>(ring);
        const int n = bn + nq;
        if (kBits == 4 && out.y) {
            sc = *reinterpret_cast<const float4*>(&chan[0][nq]);
            bi = *reinterpret_cast<const float4*>(&chan[1][nq]);
        }
#pragma unroll
        for (int b0 = 0; b0 < kBlocks; b0 += kAtOnce) {
            __syncthreads();   // the rings, the pieces handed over or the rows before have been read
#pragma unroll
            for (int o = 0; o < kOwn; ++o) {
                int i, j, qd;
                piece(o, i, j, qd);
                const int rb = wm * UM + i - b0;
                if (kAtOnce == kBlocks || (rb >= 0 && rb < kAtOnce)) {
                    i32x4_t v = own[o];
                    if (kBits == 4) v >>= 4;
                    *reinterpret_cast<i32x4_t*>(&stage[(rb * 32 + r32) * kPitch + (wn * UN + j) * 32 + 8 * qd + 4 * kh]) = v;
                }
            }
            __syncthreads();
            for (int row = t / (BN / 4); row < kAtOnce * 32; row += kThreads / (BN / 4)) {
                const int m = bm + b0 * 32 + row;
                if (m >= gm.M || n >= gm.Cout) continue;
                store_plain(*reinterpret_cast<const i32x4_t*>(&stage[row * kPitch + nq]), out, (size_t)m * gm.Cout + n, n, gm.Cout, sc, bi);
            }
        }
    }
}

// Waves on a SIMD that the registers have to leave room for: as many as the blocks that fit LDS bring, at most four.
constexpr int conv_waves(int um_un, int waves, int slots) { return waves == 16 ? 4 : um_un >= 4 ? 2 : slots == 3 ? 3 : 4; }

// One convolution per launch: grid (column tiles, row tiles).
template <int UM, int UN, int WM, int WN, int KS, int ST, int kBits>
__global__ __launch_bounds__(64 * WM * WN * KS, conv_waves(UM * UN, WM * WN * KS, ST)) void w4a4_conv_kernel(
    const ConvGeom gm, const uint32_t* __restrict__ a, const uint32_t* __restrict__ w, const ConvOut out) {
    w4a4_conv_tile<UM, UN, WM, WN, KS, ST, kBits>(gm, a, w, out, blockIdx.y * (32 * UM * WM), blockIdx.x * (32 * UN * WN));
}

// Several per launch: item i is the grid's plane z = i.
template <int UM, int UN, int WM, int WN, int KS, int ST, int kBits>
__global__ __launch_bounds__(64 * WM * WN * KS, conv_waves(UM * UN, WM * WN * KS, ST)) void w4a4_conv_batch_kernel(const ConvBatch args) {
    constexpr int BM = 32 * UM * WM, BN = 32 * UN * WN;
    const ConvItem& it = args.it[blockIdx.z];
    const ConvGeom gm = it.gm;
    if ((int)blockIdx.x * BN >= gm.Cout || (int)blockIdx.y * BM >= gm.M) return;   // the grid fits the largest item
    w4a4_conv_tile<UM, UN, WM, WN, KS, ST, kBits>(gm, it.a, it.w, it.out, blockIdx.y * BM, blockIdx.x * BN);
}

// The same convolution for few output pixels (one or a few frames), where a tile grid leaves most of the
// chip idle and a launch is a chain of latencies: set-up, table, ring fill, a barrier per K step, epilogue.
// Here nothing is staged: the KS waves of a block share a (16 UM) x (16 UN) output tile and split K, a wave
// loads its MFMA operands from global memory straight into registers, D steps at a time before it
// multiplies any, and the waves' sums meet in LDS by integer adds (exact in any order).  One
// round trip to memory for the operands, none for the shortcut, scales and biases, which are requested
// together with them.
//
// v_mfma_i32_16x16x64_i8: lane l supplies row / column l % 16 and the 16 codes of quarter l / 16; it
// receives D[4 (l / 16) + r][l % 16].  A 16-byte load per lane is 16 rows x 64 B, i.e. a step of 128 codes
// (64 with bytes), and feeds two MFMAs (one).
template <int UM, int UN, int KS, int D, int kBits>
__device__ __forceinline__ void conv_direct_tile(const ConvGeom& gm, const uint32_t* __restrict__ a,
                                                 const uint32_t* __restrict__ w, const ConvOut& out, const int bm,
                                                 const int bn) {
    constexpr int TM = 16 * UM, TN = 16 * UN, kPitch = TN + 4, kThreads = 64 * KS;
    __shared__ __attribute__((aligned(16))) int32_t sums[TM * kPitch];
    const int t = threadIdx.x, lane = t % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
    const int r16 = lane & 15, chunk = lane >> 4;
    const int cw = gm.Cin / (32 / kBits);
    const int kwords = gm.KH * gm.KW * cw;
    const int steps = (kwords + kStepWords - 1) / kStepWords;
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(a, (uint32_t)((size_t)gm.B * gm.H * gm.W * cw * 4));
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(w, (uint32_t)((size_t)gm.Cout * kwords * 4));

    int abase[UM], ih0[UM], iw0[UM];   // the lane's pixel of each row block: byte offset of its first tap, image position
#pragma unroll
    for (int i = 0; i < UM; ++i) {
        const int m = min(bm + 16 * i + r16, gm.M - 1);   // a row past the end works on the last one and is not stored
        const int b = div_by(m, gm.OH * gm.OW, gm.mg_ohow, gm.fastdiv);
        const int rem = m - b * (gm.OH * gm.OW);
        const int oh = div_by(rem, gm.OW, gm.mg_ow, gm.fastdiv), ow = rem - oh * gm.OW;
        ih0[i] = oh * gm.stride - gm.pad;
        iw0[i] = ow * gm.stride - gm.pad;
        abase[i] = ((b * gm.H + ih0[i]) * gm.W + iw0[i]) * cw * 4;
    }
    u32x4_t av[D][UM], bv[D][UN];
    auto load = [&](int s, int d) {
        const int kw0 = s * kStepWords + chunk * 4;   // first word of the lane's chunk: inside one tap
        const bool kin = kw0 < kwords;
        const int tap = div_by(kw0, cw, gm.mg_cw, gm.fastdiv), cword = kw0 - tap * cw;
        const int kh = div_by(tap, gm.KW, gm.mg_kw, gm.fastdiv), kwi = tap - kh * gm.KW;
        const int at = ((kh * gm.W + kwi) * cw + cword) * 4;
#pragma unroll
        for (int i = 0; i < UM; ++i) {
            const bool in = kin && (uint32_t)(ih0[i] + kh) < (uint32_t)gm.H && (uint32_t)(iw0[i] + kwi) < (uint32_t)gm.W;
            av[d][i] = __builtin_amdgcn_raw_buffer_load_b128(ra, in ? (uint32_t)(abase[i] + at) : kOut, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < UN; ++j) {
            const int n = bn + 16 * j + r16;
            bv[d][j] = __builtin_amdgcn_raw_buffer_load_b128(
                rw, kin && n < gm.Cout ? (uint32_t)(n * kwords + kw0) * 4u : kOut, 0, 0);
        }
    };
    i32x4_t acc[UM][UN];
#pragma unroll
    for (int i = 0; i < UM; ++i)
#pragma unroll
        for (int j = 0; j < UN; ++j) acc[i][j] = i32x4_t{0, 0, 0, 0};
    auto multiply = [&](int d) {
        if constexpr (kBits == 4) {
            i32x4_t af[UM][2], bf[UN][2];
#pragma unroll
            for (int i = 0; i < UM; ++i) {
                af[i][0] = widen_a(av[d][i].x, av[d][i].y);
                af[i][1] = widen_a(av[d][i].z, av[d][i].w);
            }
#pragma unroll
            for (int j = 0; j < UN; ++j) {
                bf[j][0] = widen_b(bv[d][j].x, bv[d][j].y);
                bf[j][1] = widen_b(bv[d][j].z, bv[d][j].w);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < UM; ++i)
#pragma unroll
                    for (int j = 0; j < UN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[i][h], bf[j][h], acc[i][j], 0, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < UM; ++i)
#pragma unroll
                for (int j = 0; j < UN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4_t, av[d][i]),
                                                                      __builtin_bit_cast(i32x4_t, bv[d][j]), acc[i][j], 0, 0, 0);
        }
    };

    // the first steps' operands, then what the epilogue needs of scales, biases and shortcut
#pragma unroll
    for (int d = 0; d < D; ++d) load(wave + d * KS, d);
    constexpr int kWordsPerRow = TN / 8, kQuadsPerRow = TN / 4;
    static_assert(TM * kWordsPerRow <= kThreads && TM * kQuadsPerRow <= kThreads, "one piece of the output per thread");
    const int mf = bm + t / kWordsPerRow, nf = bn + (t % kWordsPerRow) * 8;    // fused: 8 channels of a pixel
    const bool finishf = t < TM * kWordsPerRow && mf < gm.M && nf < gm.Cout;
    const int mq = bm + t / kQuadsPerRow, nq = bn + (t % kQuadsPerRow) * 4;    // plain: 4 channels of a pixel
    const bool finishq = t < TM * kQuadsPerRow && mq < gm.M && nq < gm.Cout;
    float4 scq = make_float4(0.f, 0.f, 0.f, 0.f), biq = scq;
    float sc[8], bi[8], res[8];
    uint32_t resw = 0;
    if (out.out_u4 && finishf) {
        load_floats(out.scale + nf, sc);
        load_floats(out.bias + nf, bi);
        if (out.res_u4) resw = out.res_u4[(size_t)mf * (gm.Cout / 8) + nf / 8];
        else if (out.res_f32) load_floats(out.res_f32 + (size_t)mf * gm.Cout + nf, res);
    } else if (out.y && finishq && (gm.Cout % 4) == 0) {
        scq = *reinterpret_cast<const float4*>(out.scale + nq);
        biq = *reinterpret_cast<const float4*>(out.bias + nq);
    }
    for (int i = t; i < TM * kPitch; i += kThreads) sums[i] = 0;
    __syncthreads();
    for (int s0 = wave;;) {
#pragma unroll
        for (int d = 0; d < D; ++d) multiply(d);
        s0 += D * KS;
        if (s0 >= steps) break;
#pragma unroll
        for (int d = 0; d < D; ++d) load(s0 + d * KS, d);
    }
#pragma unroll
    for (int i = 0; i < UM; ++i)
#pragma unroll
        for (int j = 0; j < UN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                __hip_atomic_fetch_add(&sums[(16 * i + 4 * chunk + r) * kPitch + 16 * j + r16], acc[i][j][r],
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
    constexpr int kShift = kBits == 4 ? 4 : 0;   // 4-bit: the sum is 16 * result
    if (out.out_u4) {
        if (!finishf) return;
        const int32_t* sg = &sums[(t / kWordsPerRow) * kPitch + (t % kWordsPerRow) * 8];
        const i32x4_t v0 = *reinterpret_cast<const i32x4_t*>(sg), v1 = *reinterpret_cast<const i32x4_t*>(sg + 4);
        const int q[8] = {v0[0] >> kShift, v0[1] >> kShift, v0[2] >> kShift, v0[3] >> kShift,
                          v1[0] >> kShift, v1[1] >> kShift, v1[2] >> kShift, v1[3] >> kShift};
        if (out.res_u4) {
            shortcut_from_codes(resw, out.res_scale, res);
        } else if (!out.res_f32) {
#pragma unroll
            for (int e = 0; e < 8; ++e) res[e] = 0.f;
        }
        float code[8];
        fused_codes(q, sc, bi, res, out, code);
        out.out_u4[(size_t)mf * (gm.Cout / 8) + nf / 8] = pack_codes(code);
    } else {
        if (!finishq) return;
        i32x4_t v = *reinterpret_cast<const i32x4_t*>(&sums[(t / kQuadsPerRow) * kPitch + (t % kQuadsPerRow) * 4]);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] >>= kShift;
        store_plain(v, out, (size_t)mq * gm.Cout + nq, nq, gm.Cout, scq, biq);
    }
}

template <int UM, int UN, int KS, int D, int kBits>
__global__ __launch_bounds__(64 * KS) void conv_direct_kernel(const ConvGeom gm, const uint32_t* __restrict__ a,
                                                              const uint32_t* __restrict__ w, const ConvOut out) {
    conv_direct_tile<UM, UN, KS, D, kBits>(gm, a, w, out, blockIdx.y * 16 * UM, blockIdx.x * 16 * UN);
}

// Several per launch: item i is the grid's plane z = i.
template <int UM, int UN, int KS, int D, int kBits>
__global__ __launch_bounds__(64 * KS) void conv_direct_batch_kernel(const ConvBatch args) {
    const ConvItem& it = args.it[blockIdx.z];
    const ConvGeom gm = it.gm;
    if ((int)blockIdx.x * 16 * UN >= gm.Cout || (int)blockIdx.y * 16 * UM >= gm.M) return;   // the grid fits the largest item
    conv_direct_tile<UM, UN, KS, D, kBits>(gm, it.a, it.w, it.out, blockIdx.y * 16 * UM, blockIdx.x * 16 * UN);
}

// Any Cin that fills whole words: one thread per output.  Slow; for shapes whose Cin is not a
// multiple of 32, more than 32 filter taps, or tensors of 4 GB and more.
template <int kBits>
__global__ __launch_bounds__(256) void w4a4_generic_kernel(
    const ConvGeom gm, const uint32_t* __restrict__ a, const uint32_t* __restrict__ w, const ConvOut out) {
    int32_t* const acc_out = out.acc;
    const float* const scale = out.scale;
    const float* const bias = out.bias;
    float* const y_out = out.y;
    const size_t o = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (o >= (size_t)gm.M * gm.Cout) return;
    const int m = (int)(o / gm.Cout), n = (int)(o % gm.Cout);
    const int b = m / (gm.OH * gm.OW);
    const int rem = m - b * (gm.OH * gm.OW);
    const int oh = rem / gm.OW, ow = rem - oh * gm.OW;
    const int cw = gm.Cin / (32 / kBits);
    int acc = 0;
    for (int kh = 0; kh < gm.KH; ++kh)
        for (int kwi = 0; kwi < gm.KW; ++kwi) {
            const int ih = oh * gm.stride + kh - gm.pad, iw = ow * gm.stride + kwi - gm.pad;
            if (ih < 0 || ih >= gm.H || iw < 0 || iw >= gm.W) continue;
            const uint32_t* ap = a + ((size_t)(b * gm.H + ih) * gm.W + iw) * cw;
            const uint32_t* wp = w + ((size_t)(n * gm.KH + kh) * gm.KW + kwi) * cw;
            for (int c = 0; c < cw; ++c) {
                const uint32_t av = ap[c], wv = wp[c];
                if (kBits == 4) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const int qa = (av >> (4 * j)) & 0xF;
                        const int qw = (int)(((wv >> (4 * j)) & 0xFu) ^ 8u) - 8;
                        acc += qa * qw;
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc += (int)(int8_t)(av >> (8 * j)) * (int)(int8_t)(wv >> (8 * j));
                }
            }
        }
    if (acc_out) acc_out[o] = acc;
    if (y_out) y_out[o] = fmaf((float)acc, scale[n], bias[n]);
}

// Fused output for the shapes above: one thread per packed output word.
__global__ __launch_bounds__(256) void w4a4_generic_u4_kernel(
    const ConvGeom gm, const uint32_t* __restrict__ a, const uint32_t* __restrict__ w, const ConvOut out) {
    const size_t o = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int wpr = gm.Cout / 8;
    if (o >= (size_t)gm.M * wpr) return;
    const int m = (int)(o / wpr), n0 = (int)(o % wpr) * 8;
    const int b = m / (gm.OH * gm.OW);
    const int rem = m - b * (gm.OH * gm.OW);
    const int oh = rem / gm.OW, ow = rem - oh * gm.OW;
    const int cw = gm.Cin / 8;
    int acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int kh = 0; kh < gm.KH; ++kh)
        for (int kwi = 0; kwi < gm.KW; ++kwi) {
            const int ih = oh * gm.stride + kh - gm.pad, iw = ow * gm.stride + kwi - gm.pad;
            if (ih < 0 || ih >= gm.H || iw < 0 || iw >= gm.W) continue;
            const uint32_t* ap = a + ((size_t)(b * gm.H + ih) * gm.W + iw) * cw;
            for (int c = 0; c < cw; ++c) {
                const uint32_t av = ap[c];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t wv = w[((size_t)((n0 + e) * gm.KH + kh) * gm.KW + kwi) * cw + c];
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        acc[e] += (int)((av >> (4 * j)) & 0xFu) * ((int)(((wv >> (4 * j)) & 0xFu) ^ 8u) - 8);
                }
            }
        }
    out.out_u4[o] = fused_word(acc, out, (size_t)m, n0, gm.Cout);
}

// One convolution made ready for a launch.
struct ConvJob {
    ConvGeom gm;
    const uint32_t* a;
    const uint32_t* w;
    ConvOut out;
    bool tiled;   // the tiled kernel can run it
    int ksteps;   // K steps of the tiled kernel
};

// One launch of the tiled kernel for n jobs (n <= kConvBatch) that share a tile configuration.
template <int kBits, int UM, int UN, int WM, int WN, int KS, int ST>
void launch_tiled(const ConvJob* jobs, int n, hipStream_t st) {
    constexpr int BM = 32 * UM * WM, BN = 32 * UN * WN, kThreads = 64 * WM * WN * KS;
    ConvBatch cb;
    int ny = 0, nx = 0;
    for (int i = 0; i < kConvBatch; ++i) {
        const ConvJob& j = jobs[i < n ? i : 0];
        cb.it[i] = ConvItem{j.gm, j.a, j.w, j.out};
        if (i < n) {
            ny = std::max(ny, (j.gm.M + BM - 1) / BM);
            nx = std::max(nx, (j.gm.Cout + BN - 1) / BN);
        }
    }
    if (kBits == 4 && n > 1)
        hipLaunchKernelGGL((w4a4_conv_batch_kernel<UM, UN, WM, WN, KS, ST, 4>), dim3(nx, ny, n), dim3(kThreads), 0, st, cb);
    else
        hipLaunchKernelGGL((w4a4_conv_kernel<UM, UN, WM, WN, KS, ST, kBits>), dim3(nx, ny, 1), dim3(kThreads), 0, st, jobs[0].gm,
                           jobs[0].a, jobs[0].w, jobs[0].out);
}

// ... of the direct kernel.
template <int kBits, int UM, int UN, int KS, int D>
void launch_direct(const ConvJob* jobs, int n, hipStream_t st) {
    ConvBatch cb;
    int ny = 0, nx = 0;
    for (int i = 0; i < kConvBatch; ++i) {
        const ConvJob& j = jobs[i < n ? i : 0];
        cb.it[i] = ConvItem{j.gm, j.a, j.w, j.out};
        if (i < n) {
            ny = std::max(ny, (j.gm.M + 16 * UM - 1) / (16 * UM));
            nx = std::max(nx, (j.gm.Cout + 16 * UN - 1) / (16 * UN));
        }
    }
    if (kBits == 4 && n > 1)
        hipLaunchKernelGGL((conv_direct_batch_kernel<UM, UN, KS, D, 4>), dim3(nx, ny, n), dim3(64 * KS), 0, st, cb);
    else
        hipLaunchKernelGGL((conv_direct_kernel<UM, UN, KS, D, kBits>), dim3(nx, ny, 1), dim3(64 * KS), 0, st, jobs[0].gm,
                           jobs[0].a, jobs[0].w, jobs[0].out);
}

template <int kBits>
ConvJob make_job(const qail_conv_desc& d, const uint32_t* a, const uint32_t* w, const ConvOut& out) {
    constexpr int kPerWord = 32 / kBits;
    ConvJob job;
    ConvGeom& gm = job.gm;
    gm.B = d.B; gm.H = d.H; gm.W = d.W; gm.Cin = d.Cin; gm.Cout = d.Cout;
    gm.KH = d.KH; gm.KW = d.KW; gm.stride = d.stride; gm.pad = d.pad;
    gm.OH = (d.H + 2 * d.pad - d.KH) / d.stride + 1;
    gm.OW = (d.W + 2 * d.pad - d.KW) / d.stride + 1;
    gm.M = d.B * gm.OH * gm.OW;
    {
        // the tiled kernel divides m < M by OH OW, the remainder by OW, a word index below the
        // filter's words by the words per pixel and a tap below KH KW by KW
        const uint32_t cw = (uint32_t)(gm.Cin / kPerWord);
        bool ok = gm.M > 0;
        gm.mg_ohow = div_magic((uint32_t)(gm.OH * gm.OW), (uint64_t)gm.M, ok);
        gm.mg_ow = div_magic((uint32_t)gm.OW, (uint64_t)gm.OH * gm.OW, ok);
        gm.mg_cw = div_magic(cw, (uint64_t)gm.KH * gm.KW * cw, ok);
        gm.mg_kw = div_magic((uint32_t)gm.KW, (uint64_t)gm.KH * gm.KW, ok);
        gm.fastdiv = ok ? 1 : 0;
        gm.row_taps = 0;
        for (long long b = 0; b < (long long)gm.KH * gm.KW && b < 32; b += gm.KW) gm.row_taps |= 1u << b;
    }
    const size_t cwb = (size_t)gm.Cin / kPerWord * 4;  // bytes per pixel
    const bool fits32 = (size_t)gm.B * gm.H * gm.W * cwb < 0xFFFFFFF0ull &&
                        (size_t)gm.Cout * gm.KH * gm.KW * cwb < 0xFFFFFFF0ull &&
                        (size_t)gm.M * gm.Cout * 4 < 0xFFFFFFF0ull;
    job.ksteps = (gm.KH * gm.KW * (gm.Cin / kPerWord) + kStepWords - 1) / kStepWords;
    // a 16-byte chunk (32 or 16 codes) must lie inside one filter tap
    job.tiled = d.Cin % (4 * kPerWord) == 0 && d.KH * d.KW <= 32 && fits32 && job.ksteps + 16 <= kMaxSteps;
    job.a = a;
    job.w = w;
    job.out = out;
    // (two outputs of rows that end inside a 64-byte sector, which the block of the next columns completes, go through the caches
    // whatever their size: 316 channels, 75 MB 35.8 us past them, 17.9 through; 280, 24 MB 10.9 / 7.9.  One column of blocks, up to 128
    // channels, writes whole sectors: 72 channels, 20 MB 10.6 / 12.2.  One output alone is 1 % slower through them at 8 to 16 MB
    // and 10 % faster from 24 MB on.)
    if (!out.out_u4)
        job.out.quick = (size_t)gm.M * gm.Cout * ((out.acc ? 4 : 0) + (out.y ? 4 : 0)) >= kPastCaches &&
                        !(out.acc && out.y && gm.Cout > 128 && gm.Cout % 16 != 0);
    return job;
}

// Launches n jobs the tiled kernel can run (n <= kConvBatch) as one grid.  The tile is chosen for the job with the most
// work (the one that decides how long the launch takes), as if it had as many more tiles as the others are worth in its K steps.
template <int kBits>
void launch_tiled_jobs(const ConvJob* jobs, int n, hipStream_t st) {
    int lead = 0;
    for (int i = 1; i < n; ++i)
        if ((long long)jobs[i].ksteps * jobs[i].gm.M > (long long)jobs[lead].ksteps * jobs[lead].gm.M) lead = i;
    const ConvGeom& gm = jobs[lead].gm;
    const int ksteps = jobs[lead].ksteps;
    long long all64 = 0, all32 = 0, all16 = 0;   // (all64: in tiles of the lead)
    for (int i = 0; i < n; ++i) {
        all32 += (long long)((jobs[i].gm.M + 31) / 32) * ((jobs[i].gm.Cout + 31) / 32);
        all64 += (long long)((jobs[i].gm.M + 63) / 64) * ((jobs[i].gm.Cout + 63) / 64) * jobs[i].ksteps / ksteps;
        all16 += (long long)((jobs[i].gm.M + 15) / 16) * ((jobs[i].gm.Cout + 15) / 16);
    }
    // Few 16 x 16 tiles: the direct kernel, whose tile and K split grow with them.  It reads every operand
    // once per 16 or 32 rows (columns) it meets, so its time grows with tiles x K steps while the tiled
    // kernel's stays near its fixed cost.  us per launch, direct / tiled, 4-bit ResNet layers of 64 / 128 /
    // 256 / 512 channels (5 / 9 / 18 / 36 steps): one image 3.5 / 5.0, 3.3 / 4.9, 3.8 / 6.6, 4.6 / 8.3; four
    // images 4.7 / 5.3, 4.6 / 5.0, 4.9 / 6.6, 5.4 / 8.4; eight images 7.0 / 5.7 (28 k tile steps, above the
    // line), 5.4 / 5.1 (above), 6.7 / 6.8 (above), 6.5 / 8.5.  8-bit, 72 steps, four images 8.0 / 8.3, eight
    // 9.9 / 8.5 (above the line).
    // With few K steps the direct kernel is bound by its blocks, not by its steps, so their number has a limit of
    // its own: three and a half 32 x 32 blocks per CU.  3x3 layers of 3 steps, 784 / 1176 blocks 4.9 / 5.5, 6.2 / 5.7 (above);
    // 1x1 layers (plain output) of 1 step, 392 / 784 / 1568 / 3136 blocks 4.1 / 4.8, 4.9 / 5.0, 7.0 / 5.6, 10.3 / 8.0 (the last
    // two above).  The tiled kernel's set-up is shorter for one tap, and its epilogue for fused outputs: there
    // 784 blocks are 5.1 / 4.8 already, and with 8-bit codes or fused outputs 12.5 k tile steps 5.3 / 5.2, 5.8 / 5.5.
    const long long cus = device_cu_count(), work = all16 * ksteps;
    if (all16 <= cus && work <= 120 * cus) return launch_direct<kBits, 1, 1, 8, 2>(jobs, n, st);
    if (all16 <= 2 * cus && work <= 120 * cus) return launch_direct<kBits, 1, 2, 8, 2>(jobs, n, st);
    if (all16 <= 4 * cus && work <= (kBits == 4 ? 120 : 96) * cus) return launch_direct<kBits, 2, 2, 8, 1>(jobs, n, st);
    const bool one_tap = gm.KH * gm.KW == 1, fused = jobs[lead].out.out_u4 != nullptr;
    if (2 * all32 <= (one_tap && fused ? 5 : 7) * cus && work <= (one_tap && (fused || kBits == 8) ? 44 : 64) * cus)
        return launch_direct<kBits, 2, 2, 4, 1>(jobs, n, st);
    // The tiled kernel's shapes, by the number t of 64 x 64 tiles per CU and the K steps (sweeps of some hundred drawn convolutions
    // with operands that come from beyond L2, as a layer's do; us).  4-bit: up to one tile per CU K is split between groups of four
    // waves with 32 x 32 each, four groups where it is long (36 steps 8.4, two groups 9.0; 18 steps 7.0 / 6.7).  Up to three the
    // same waves without a split as long as K is short (9 steps, t = 2.3 7.6, split with 64 x 32 each 8.0; 13 steps, t = 1.1 / 2.6
    // 7.4 / 9.4 against 7.1 / 9.9), with one where it is long (14 steps, t = 1.1 / 2.5 7.9 / 11.3 against 7.3 / 10.9; 18 steps, t =
    // 1.1 / 2.3 / 2.8 9.1 / 11.8 / 12.7 against 8.2 / 11.1 / 11.7).  Above that four waves with 64 x 32 or 32 x 64 each, whichever pads
    // the channels less, a ring of three where all blocks fit a CU with it (t <= 6; t = 4.6, 5 steps 12.7 / 12.8, t = 3.8 9.0 / 9.4, t =
    // 6.1 11.7 / 10.7), and from t = 6 on 128 x 128 where that pads no more (t = 6.1, 9 steps 12.8, 128 x 64 15.0; 18 steps, t = 12.2 20.4 /
    // 22.3), unless there are only a step or two (1x1, 128 -> 512 channels 12.9, 64 x 128 10.9).
    // Bytes have nothing to widen and wait for their operands instead: three slots almost throughout.  Up to one tile per CU
    // no split (up to 4 steps; 1 step 4.0, two groups 4.2), two groups or, from 24 steps on, four.  Up to three no split up to 16
    // steps (9 steps, t = 1.3 / 2.1 6.3 / 6.3, with two slots 7.2 / 7.0), then two groups, of four waves up to t = 2 (25 steps, t = 1.5
    // 9.0, two waves and two slots 9.7; 512 channels, t = 1.5, inside the body at batch 64 7 us less), of two waves above
    // (72 steps, t = 2.3 20.1 / 23.1).  Above that 128 x 64 where tiles 128 wide would pad much (96 -> 280 channels, 14 steps 17.0, 128 x 128
    // 19.2; but 400, 14 steps 19.2 / 15.6, and 1x1, 280 12.0, 64 x 128 10.7), else 64 x 128 up to t = 6 or 4 steps and 128 x 128 above, with two
    // slots for one output (t = 6.1, 9 steps 9.9 / 10.6) and three for two (14.9 / 14.0) or many tiles (t = 12.2, 18 steps 28.5 / 24.6).
    if constexpr (kBits == 4) {
        const bool fits128 = (gm.Cout + 127) / 128 * 2 == (gm.Cout + 63) / 64;   // tiles 128 wide pad no more than tiles 64 wide
        if (all64 <= cus) return ksteps >= 24 ? launch_tiled<4, 1, 1, 2, 2, 4, 3>(jobs, n, st) : launch_tiled<4, 1, 1, 2, 2, 2, 3>(jobs, n, st);
        if (all64 < 3 * cus) {
            if (ksteps <= 12) return launch_tiled<4, 1, 1, 2, 2, 1, 2>(jobs, n, st);
            return launch_tiled<4, 2, 1, 1, 2, 2, 2>(jobs, n, st);
        }
        if (fits128 && all64 >= 6 * cus && ksteps > 2) return launch_tiled<4, 2, 2, 2, 2, 1, 2>(jobs, n, st);
        if (all64 <= 6 * cus) return fits128 ? launch_tiled<4, 1, 2, 2, 2, 1, 3>(jobs, n, st) : launch_tiled<4, 2, 1, 2, 2, 1, 3>(jobs, n, st);
        return fits128 ? launch_tiled<4, 1, 2, 2, 2, 1, 2>(jobs, n, st) : launch_tiled<4, 2, 1, 2, 2, 1, 2>(jobs, n, st);
    } else {
        const bool two = jobs[lead].out.acc && jobs[lead].out.y;
        const int n64 = (gm.Cout + 63) / 64, n128 = (gm.Cout + 127) / 128;
        if (all64 <= cus) {
            if (ksteps <= 4) return launch_tiled<8, 1, 1, 2, 2, 1, 3>(jobs, n, st);
            return ksteps >= 24 ? launch_tiled<8, 1, 1, 2, 2, 4, 3>(jobs, n, st) : launch_tiled<8, 1, 1, 2, 2, 2, 3>(jobs, n, st);
        }
        const bool pads = ksteps <= 4 ? 10 * n128 > 6 * n64 : 14 * n128 > 8 * n64;   // tiles 128 wide by more than a fifth, a seventh
        if (all64 < 3 * cus) {
            if (ksteps <= 16) return launch_tiled<8, 1, 1, 2, 2, 1, 3>(jobs, n, st);
            return all64 <= 2 * cus ? launch_tiled<8, 1, 1, 2, 2, 2, 3>(jobs, n, st) : launch_tiled<8, 2, 1, 1, 2, 2, 2>(jobs, n, st);
        }
        if (pads) return launch_tiled<8, 2, 1, 2, 2, 1, 3>(jobs, n, st);
        if (all64 < 6 * cus || ksteps <= 4) return launch_tiled<8, 1, 2, 2, 2, 1, 3>(jobs, n, st);
        return two || all64 > 12 * cus ? launch_tiled<8, 2, 2, 2, 2, 1, 3>(jobs, n, st) : launch_tiled<8, 2, 2, 2, 2, 1, 2>(jobs, n, st);
    }
}

template <int kBits>
hipError_t launch_job(const ConvJob& job, hipStream_t st) {
    if (job.tiled) {
        launch_tiled_jobs<kBits>(&job, 1, st);
    } else if (job.out.out_u4) {
        const size_t words = (size_t)job.gm.M * (job.gm.Cout / 8);
        hipLaunchKernelGGL(w4a4_generic_u4_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st, job.gm,
                           job.a, job.w, job.out);
    } else {
        const size_t outs = (size_t)job.gm.M * job.gm.Cout;
        hipLaunchKernelGGL(w4a4_generic_kernel<kBits>, dim3((unsigned)((outs + 255) / 256)), dim3(256), 0, st, job.gm,
                           job.a, job.w, job.out);
    }
    return hipGetLastError();
}

template <int kBits>
hipError_t launch_conv(const qail_conv_desc& d, const uint32_t* a, const uint32_t* w, const ConvOut& out,
                       hipStream_t st) {
    return launch_job<kBits>(make_job<kBits>(d, a, w, out), st);
}

ConvOut fused_out(const float* scale, const float* bias, float s_out, const uint32_t* res_u4, float res_scale,
                  const float* res_f32, uint32_t* out_u4) {
    const float inv = 1.0f / s_out;
    const int quick = s_out >= 0x1p-100f && s_out <= 0x1p100f;   // (a normal number, and so is its reciprocal)
    return ConvOut{nullptr, scale, bias, nullptr, out_u4, res_u4, res_f32, s_out, res_scale, inv, quick};
}
}  // namespace

// Independent W4A4 convolutions (plain or fused output each) in few launches: consecutive ones the
// tiled kernel can run share a launch, kConvBatch at a time, as long as their tile grids are of
// similar size (every plane of the launch's grid is as large as the largest); the others go one by one.
hipError_t launch_w4a4_conv_batch(const qail_conv_item* items, int count, hipStream_t st) {
    ConvJob tiled[kConvBatch];
    int n = 0;
    long long lo = 0, hi = 0;   // smallest and largest tile grid (in 64 x 64 tiles) of the pending launch
    auto flush = [&]() -> hipError_t {
        if (n > 0) launch_tiled_jobs<4>(tiled, n, st);
        n = 0;
        return hipGetLastError();
    };
    for (int i = 0; i < count; ++i) {
        const qail_conv_item& it = items[i];
        const ConvOut out = it.out_u4 ? fused_out(it.scale, it.bias, it.s_out, it.res_u4, it.res_scale, it.res_f32, it.out_u4)
                                      : ConvOut{it.acc_out, it.scale, it.bias, it.y_out, nullptr, nullptr, nullptr, 1.f, 0.f, 1.f, 0};
        const ConvJob job = make_job<4>(it.d, it.a_u4, it.w_s4, out);
        if (!job.tiled) {
            const hipError_t e = launch_job<4>(job, st);
            if (e != hipSuccess) return e;
            continue;
        }
        const long long t = (long long)((job.gm.M + 63) / 64) * ((job.gm.Cout + 63) / 64);
        if (n == kConvBatch || (n > 0 && (2 * std::min(lo, t) < std::max(hi, t)))) {
            const hipError_t e = flush();
            if (e != hipSuccess) return e;
        }
        lo = n ? std::min(lo, t) : t;
        hi = n ? std::max(hi, t) : t;
        tiled[n++] = job;
    }
    return flush();
}

hipError_t launch_w4a4_conv(const qail_conv_desc& d, const uint32_t* a, const uint32_t* w, int32_t* acc,
                            const float* scale, const float* bias, float* y, hipStream_t st) {
    const ConvOut out{acc, scale, bias, y, nullptr, nullptr, nullptr, 1.f, 0.f, 1.f, 0};
    return launch_conv<4>(d, a, w, out, st);
}

hipError_t launch_w8a8_conv(const qail_conv_desc& d, const uint32_t* a, const uint32_t* w, int32_t* acc,
                            const float* scale, const float* bias, float* y, hipStream_t st) {
    const ConvOut out{acc, scale, bias, y, nullptr, nullptr, nullptr, 1.f, 0.f, 1.f, 0};
    return launch_conv<8>(d, a, w, out, st);
}

hipError_t launch_w4a4_conv_u4(const qail_conv_desc& d, const uint32_t* a, const uint32_t* w, const float* scale,
                               const float* bias, float s_out, const uint32_t* res_u4, float res_scale,
                               const float* res_f32, uint32_t* out_u4, hipStream_t st) {
    return launch_conv<4>(d, a, w, fused_out(scale, bias, s_out, res_u4, res_scale, res_f32, out_u4), st);
}

}  // namespace qail
