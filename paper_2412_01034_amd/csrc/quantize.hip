// Round-to-nearest quantisers and (un)packers (Sec. 2.1 RTN; Sec. 5.1 4-bit formats).
//
// These are one-off, HBM-bound elementwise/reduction kernels; what matters is
// that the codes are bit-identical to the definition: fp32 arithmetic with
// correctly rounded division (compile with -fhip-fp32-correctly-rounded-divide-sqrt,
// no fast-math) and rint = ties-to-even.
#include "qail_internal.h"
#include <algorithm>

namespace qail {

namespace {

constexpr int kQuantBlock = 256;

// Smallest fp16 >= v, for finite 0 <= v <= 65504, as a bit pattern.
__device__ __forceinline__ uint16_t f32_to_f16_bits_up(float v) {
    _Float16 h = (_Float16)v;  // nearest even
    uint16_t b = __builtin_bit_cast(uint16_t, h);
    if ((float)h < v) b += 1;  // positive fp16 patterns are ordered like integers
    return b;
}

__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
    const float4 a = *reinterpret_cast<const float4*>(p);
    const float4 b = *reinterpret_cast<const float4*>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// One block per row.  A team of LPG lanes (power of two) owns one group at a
// time; lane t of the team covers 8-element words t, t+LPG, ... of the group.
template <int LPG>
__global__ __launch_bounds__(kQuantBlock) void quantize_asym_kernel(
    const float* __restrict__ w, uint32_t* __restrict__ qw, uint16_t* __restrict__ scales,
    uint32_t* __restrict__ zeros, uint32_t* __restrict__ range_errors, int K, int g) {
    extern __shared__ uint8_t zbuf[];  // one zero-point per group of this row
    constexpr int kTeams = kQuantBlock / LPG;
    const int n = blockIdx.x;
    const int team = threadIdx.x / LPG;
    const int tl = threadIdx.x % LPG;
    const int G = K / g;
    const int wpg = g / 8;
    const float* wrow = w + (size_t)n * K;
    uint32_t* qrow = qw + (size_t)n * (K / 8);

    // every team runs the same number of rounds so that the team shuffles are
    // executed by whole waves
    const int rounds = (G + kTeams - 1) / kTeams;
    for (int r = 0; r < rounds; ++r) {
        const int grp = r * kTeams + team;
        const bool live = grp < G;
        float lo = 0.f, hi = 0.f;
        if (live) {
            for (int wi = tl; wi < wpg; wi += LPG) {
                float v[8];
                load8(wrow + (size_t)grp * g + wi * 8, v);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    lo = fminf(lo, v[j]);
                    hi = fmaxf(hi, v[j]);
                }
            }
        }
#pragma unroll
        for (int off = 1; off < LPG; off <<= 1) {
            lo = fminf(lo, __shfl_xor(lo, off, kWave));
            hi = fmaxf(hi, __shfl_xor(hi, off, kWave));
        }
        if (!live) continue;
        float s32 = (hi - lo) / 15.0f;
        const bool over = s32 > 65504.0f;
        if (over) s32 = 65504.0f;
        uint16_t sb = f32_to_f16_bits_up(s32);
        if (sb < 0x0400) sb = 0x0400;   // 2^-14, the smallest normal fp16
        if (hi == lo) sb = 0x3C00;      // all-zero group: scale 1
        const float s = f16_bits_to_f32(sb);
        const float z = fminf(fmaxf(rintf(-lo / s), 0.f), 15.f);
        for (int wi = tl; wi < wpg; wi += LPG) {
            float v[8];
            load8(wrow + (size_t)grp * g + wi * 8, v);
            uint32_t word = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float q = fminf(fmaxf(rintf(v[j] / s) + z, 0.f), 15.f);
                word |= (uint32_t)(int)q << (4 * j);
            }
            qrow[(size_t)grp * wpg + wi] = word;
        }
        if (tl == 0) {
            scales[(size_t)n * G + grp] = sb;
            zbuf[grp] = (uint8_t)(int)z;
            if (over && range_errors) atomicAdd(range_errors, 1u);
        }
    }
    __syncthreads();
    const int zwords = (G + 7) / 8;
    for (int zi = threadIdx.x; zi < zwords; zi += kQuantBlock) {
        uint32_t word = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int grp = zi * 8 + j;
            if (grp < G) word |= (uint32_t)zbuf[grp] << (4 * j);
        }
        zeros[(size_t)n * zwords + zi] = word;
    }
}

// One block per row (output channel): absmax, then codes.
__global__ __launch_bounds__(kQuantBlock) void quantize_sym_kernel(
    const float* __restrict__ w, uint32_t* __restrict__ qw, float* __restrict__ scales, int K) {
    __shared__ float red[kQuantBlock / kWave];
    const int n = blockIdx.x;
    const float* wrow = w + (size_t)n * K;
    const int words = K / 8;
    float amax = 0.f;
    for (int wi = threadIdx.x; wi < words; wi += kQuantBlock) {
        float v[8];
        load8(wrow + (size_t)wi * 8, v);
#pragma unroll
        for (int j = 0; j < 8; ++j) amax = fmaxf(amax, fabsf(v[j]));
    }
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) amax = fmaxf(amax, __shfl_xor(amax, off, kWave));
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = amax;
    __syncthreads();
    amax = red[0];
#pragma unroll
    for (int i = 1; i < kQuantBlock / kWave; ++i) amax = fmaxf(amax, red[i]);
    const float s = (amax == 0.f) ? 1.0f : amax / 7.0f;
    if (threadIdx.x == 0) scales[n] = s;
    uint32_t* qrow = qw + (size_t)n * words;
    for (int wi = threadIdx.x; wi < words; wi += kQuantBlock) {
        float v[8];
        load8(wrow + (size_t)wi * 8, v);
        uint32_t word = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float q = fminf(fmaxf(rintf(v[j] / s), -8.f), 7.f);
            word |= ((uint32_t)(int)q & 0xFu) << (4 * j);
        }
        qrow[wi] = word;
    }
}

template <bool kSigned>
__global__ __launch_bounds__(256) void unpack_kernel(const uint32_t* __restrict__ qw,
                                                     uint2* __restrict__ codes, size_t words) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= words) return;
    const uint32_t w = qw[i];
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        uint32_t a = (w >> (4 * j)) & 0xFu, b = (w >> (4 * (j + 4))) & 0xFu;
        if (kSigned) {
            a = (a ^ 8u) - 8u;  // sign-extend the nibble
            b = (b ^ 8u) - 8u;
        }
        lo |= (a & 0xFFu) << (8 * j);
        hi |= (b & 0xFFu) << (8 * j);
    }
    codes[i] = make_uint2(lo, hi);
}

// ---- activations ---------------------------------------------------------

// One step for a whole tensor: max / kTop over max(a) (unsigned codes) or max|a| (signed ones), 1 where
// that is 0.  Bound by the one read of a.  Non-negative floats are ordered like their bit patterns, so
// blocks meet in *s_a through an integer atomic maximum, whatever their order.  Atomics on one address
// go one after the other (11 ns each): a block adds its maximum once, and only if it is larger than what
// it finds there (an old value is a smaller one, so nothing is lost).  One atomic per wave of 4096 small
// blocks took 188 us for 3.2 M values; one per block of 1024 threads, a block per CU, takes 6.7 us.
constexpr int kScaleBlock = 1024;

template <bool kAbs>
__device__ __forceinline__ float block_top(const float* __restrict__ a, size_t n, size_t first, size_t stride) {
    __shared__ float red[kScaleBlock / kWave];
    auto up = [](float m, float v) { return fmaxf(m, kAbs ? fabsf(v) : v); };
    const size_t n4 = n / 4;
    const float4* a4 = reinterpret_cast<const float4*>(a);
    float m[4] = {0.f, 0.f, 0.f, 0.f};
    size_t i = first;
    for (; i + 3 * stride < n4; i += 4 * stride) {   // four loads in flight per thread
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = a4[i + u * stride];
#pragma unroll
        for (int u = 0; u < 4; ++u) m[u] = up(up(up(up(m[u], v[u].x), v[u].y), v[u].z), v[u].w);
    }
    for (; i < n4; i += stride) {
        const float4 v = a4[i];
        m[0] = up(up(up(up(m[0], v.x), v.y), v.z), v.w);
    }
    for (size_t e = n4 * 4 + first; e < n; e += stride) m[1] = up(m[1], a[e]);
    float t = fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3]));
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) t = fmaxf(t, __shfl_xor(t, off, kWave));
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = t;
    __syncthreads();
    t = red[0];
#pragma unroll
    for (int w = 1; w < kScaleBlock / kWave; ++w) t = fmaxf(t, red[w]);
    return t;
}

template <bool kAbs>
__device__ __forceinline__ float step_of(float top) { return top > 0.f ? top / (kAbs ? 127.0f : 15.0f) : 1.0f; }

__global__ void act_scale_init_kernel(float* s_a) { *reinterpret_cast<uint32_t*>(s_a) = 0u; }

template <bool kAbs>
__global__ __launch_bounds__(kScaleBlock) void act_scale_reduce_kernel(const float* __restrict__ a, size_t n, float* s_a) {
    const float m = block_top<kAbs>(a, n, (size_t)blockIdx.x * kScaleBlock + threadIdx.x, (size_t)gridDim.x * kScaleBlock);
    if (threadIdx.x == 0 && m > 0.f) {
        uint32_t* const top = reinterpret_cast<uint32_t*>(s_a);
        const uint32_t bits = __builtin_bit_cast(uint32_t, m);
        if (bits > __hip_atomic_load(top, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(top, bits);
    }
}

template <bool kAbs>
__global__ void act_scale_final_kernel(float* s_a) { *s_a = step_of<kAbs>(*s_a); }

// A tensor that one block reads in the time of a launch or two: everything in one launch.
template <bool kAbs>
__global__ __launch_bounds__(kScaleBlock) void act_scale_small_kernel(const float* __restrict__ a, size_t n, float* s_a) {
    const float m = block_top<kAbs>(a, n, threadIdx.x, kScaleBlock);
    if (threadIdx.x == 0) *s_a = step_of<kAbs>(m);
}

__global__ __launch_bounds__(256) void act_quant_kernel(const float* __restrict__ a, size_t words,
                                                        const float* __restrict__ s_a,
                                                        uint32_t* __restrict__ out) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= words) return;
    const float s = *s_a;
    float v[8];
    load8(a + i * 8, v);
    uint32_t word = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float q = fminf(fmaxf(rintf(v[j] / s), 0.f), 15.f);
        word |= (uint32_t)(int)q << (4 * j);
    }
    out[i] = word;
}

int next_pow2(int v) {
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}

}  // namespace

hipError_t launch_quantize_asym(const qail_wdesc& d, const float* w, uint32_t* qw, uint16_t* scales,
                                uint32_t* zeros, uint32_t* range_errors, hipStream_t st) {
    const int G = d.K / d.group_size;
    const size_t lds = (size_t)((G + 15) / 16) * 16;
    int lpg = next_pow2(d.group_size / 8);
    if (lpg > kWave) lpg = kWave;
    dim3 grid(d.N), block(kQuantBlock);
#define QAIL_LAUNCH_ASYM(L)                                                                          \
    case L:                                                                                          \
        hipLaunchKernelGGL(quantize_asym_kernel<L>, grid, block, lds, st, w, qw, scales, zeros,      \
                           range_errors, d.K, d.group_size);                                         \
        break;
    switch (lpg) {
        QAIL_LAUNCH_ASYM(1)
        QAIL_LAUNCH_ASYM(2)
        QAIL_LAUNCH_ASYM(4)
        QAIL_LAUNCH_ASYM(8)
        QAIL_LAUNCH_ASYM(16)
        QAIL_LAUNCH_ASYM(32)
        QAIL_LAUNCH_ASYM(64)
    }
#undef QAIL_LAUNCH_ASYM
    return hipGetLastError();
}

hipError_t launch_quantize_sym(const qail_wdesc& d, const float* w, uint32_t* qw, float* scales,
                               hipStream_t st) {
    hipLaunchKernelGGL(quantize_sym_kernel, dim3(d.N), dim3(kQuantBlock), 0, st, w, qw, scales, d.K);
    return hipGetLastError();
}

hipError_t launch_unpack(const qail_wdesc& d, const uint32_t* qw, uint8_t* codes, hipStream_t st) {
    const size_t words = (size_t)d.N * (d.K / 8);
    const unsigned blocks = (unsigned)((words + 255) / 256);
    if (d.scheme == QAIL_W4_SYM_CHANNEL)
        hipLaunchKernelGGL(unpack_kernel<true>, dim3(blocks), dim3(256), 0, st, qw,
                           reinterpret_cast<uint2*>(codes), words);
    else
        hipLaunchKernelGGL(unpack_kernel<false>, dim3(blocks), dim3(256), 0, st, qw,
                           reinterpret_cast<uint2*>(codes), words);
    return hipGetLastError();
}

template <bool kAbs>
static hipError_t act_scale(const float* a, size_t n, float* s_a, hipStream_t st) {
    constexpr size_t kOneBlock = 65536;   // values: 256 KB, about what one compute unit reads in 2 us
    if (n <= kOneBlock) {
        hipLaunchKernelGGL(act_scale_small_kernel<kAbs>, dim3(1), dim3(kScaleBlock), 0, st, a, n, s_a);
        return hipGetLastError();
    }
    // at most one block per compute unit: 16 waves with four loads each keep it busy, and the
    // atomics at the end of a block stay few
    const size_t blocks = std::min<size_t>((n / 4 + 2 * kScaleBlock - 1) / (2 * kScaleBlock), (size_t)device_cu_count());
    hipLaunchKernelGGL(act_scale_init_kernel, dim3(1), dim3(1), 0, st, s_a);
    hipLaunchKernelGGL(act_scale_reduce_kernel<kAbs>, dim3((unsigned)blocks), dim3(kScaleBlock), 0, st, a, n, s_a);
    hipLaunchKernelGGL(act_scale_final_kernel<kAbs>, dim3(1), dim3(1), 0, st, s_a);
    return hipGetLastError();
}

hipError_t launch_act_scale(const float* a, size_t n, float* s_a, hipStream_t st) { return act_scale<false>(a, n, s_a, st); }
hipError_t launch_act_scale_s8(const float* a, size_t n, float* s_a, hipStream_t st) { return act_scale<true>(a, n, s_a, st); }

hipError_t launch_act_quant(const float* a, size_t n, const float* s_a, uint32_t* out, hipStream_t st) {
    const size_t words = n / 8;
    const unsigned blocks = (unsigned)((words + 255) / 256);
    hipLaunchKernelGGL(act_quant_kernel, dim3(blocks), dim3(256), 0, st, a, words, s_a, out);
    return hipGetLastError();
}

}  // namespace qail
