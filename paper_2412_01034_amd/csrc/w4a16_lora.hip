// Low-rank adapter beside the 4-bit linear (Sec. 5.1: the 4-bit policy is fine-tuned with
// rank-32 adapters on the quantised backbone, which then run next to the packed weights):
//   y[m][n] = sum_k x[m][k] w_hat[n][k] + scaling * sum_j t[m][j] B[n][j],   t[m][j] = sum_k x[m][k] A[j][k].
// Two small kernels: the down-projection t = x A^T (fp32, before the linear) and, for the
// batch sizes whose linear kernel does not take the adapter into its own epilogue, the
// up-projection added to the bf16 output afterwards.  Both are bandwidth-trivial next to the
// 4-bit stream (r (K + N) bf16 per linear).
#include "qail_internal.h"

namespace qail {

namespace {

constexpr int kMaxLoraItems = 16;

struct DownItem {
    const uint16_t* x;   // bf16 [M][K]
    const uint16_t* A;   // bf16 [r][K]
    float* t;            // fp32 [M][r]
    int K, r;
};
struct DownArgs {
    DownItem it[kMaxLoraItems];
    int M;
};

// One block per (j, ROWS rows m, item): its 1024 threads split K, 8 elements a piece.  A thread's first two
// pieces (all of K up to 16384) are requested before either is used: one round trip to memory
// instead of one per piece, which is what this kernel's time consists of while its blocks fit the chip at once (512).
// That is so up to four rows of four rank-32 adapters, which take ROWS = 1: with 4 rows a block loads five streams instead of
// two and a layer of 2 rows takes 34.5 us instead of 33.0.  With more rows a row of A is read once for 4 of them
// (16 rows: 47.2 us -> 41.5; 48 rows: 82.6 -> 62.9 together with the shorter runs of lora_up_add_kernel).
constexpr int kDownThreads = 1024;
__device__ __forceinline__ float dot8(const uint4& xv, const uint4& av, float acc) {
    const uint32_t xw[4] = {xv.x, xv.y, xv.z, xv.w}, aw[4] = {av.x, av.y, av.z, av.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        acc = fmaf(__builtin_bit_cast(float, xw[e] << 16), __builtin_bit_cast(float, aw[e] << 16), acc);
        acc = fmaf(__builtin_bit_cast(float, xw[e] & 0xFFFF0000u), __builtin_bit_cast(float, aw[e] & 0xFFFF0000u), acc);
    }
    return acc;
}
template <int ROWS>
__global__ __launch_bounds__(kDownThreads) void lora_down_kernel(const DownArgs args) {
    __shared__ float red[ROWS * kDownThreads / kWave];
    const DownItem& it = args.it[blockIdx.z];
    const int j = blockIdx.x, m0 = blockIdx.y * ROWS, rows = ROWS == 1 ? 1 : min(ROWS, args.M - m0);
    if (j >= it.r) return;  // block-uniform (items of a launch may differ in rank)
    const uint4* xr = reinterpret_cast<const uint4*>(it.x + (size_t)m0 * it.K);
    const uint4* ar = reinterpret_cast<const uint4*>(it.A + (size_t)j * it.K);
    const int n8 = it.K / 8;
    uint4 xv[ROWS][2], av[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {   // every load is issued; a piece past the end re-reads piece 0 and is not used
        const int i = (int)threadIdx.x + u * kDownThreads;
#pragma unroll
        for (int q = 0; q < ROWS; ++q) xv[q][u] = xr[(size_t)min(q, rows - 1) * n8 + (i < n8 ? i : 0)];
        av[u] = ar[i < n8 ? i : 0];
    }
    float acc[ROWS] = {};
#pragma unroll
    for (int u = 0; u < 2; ++u)
        if ((int)threadIdx.x + u * kDownThreads < n8)
#pragma unroll
            for (int q = 0; q < ROWS; ++q) acc[q] = dot8(xv[q][u], av[u], acc[q]);
    for (int i = (int)threadIdx.x + 2 * kDownThreads; i < n8; i += kDownThreads) {
        const uint4 a = ar[i];
#pragma unroll
        for (int q = 0; q < ROWS; ++q) acc[q] = dot8(xr[(size_t)min(q, rows - 1) * n8 + i], a, acc[q]);
    }
#pragma unroll
    for (int q = 0; q < ROWS; ++q)
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) acc[q] += __shfl_xor(acc[q], o);
    if (threadIdx.x % kWave == 0)
#pragma unroll
        for (int q = 0; q < ROWS; ++q) red[q * (kDownThreads / kWave) + threadIdx.x / kWave] = acc[q];
    __syncthreads();
    if ((int)threadIdx.x < rows) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < kDownThreads / kWave; ++w)   // in the order of the waves: deterministic
            sum += red[(int)threadIdx.x * (kDownThreads / kWave) + w];
        it.t[(size_t)(m0 + (int)threadIdx.x) * it.r + j] = sum;
    }
}

// The down-projection of many rows, as the contraction it is: a block takes 16 rows of x and 16 of A, its 16 waves take K
// in turn, 32 elements a step (the operands of v_mfma_f32_16x16x32_bf16 as they lie in memory: lane l holds row
// l % 16, elements 8 (l / 16) .. + 8), and their sums meet in LDS.  A block reads 32 rows for 256 sums where
// lora_down_kernel reads 5 for 4, but has the latency of its K / 512 steps, 8 of them in flight: it wins from about eight
// rounds of lora_down_kernel's blocks over the chip (decoder layer with rank 32, 48 rows: 61.9 us against 74.0
// here, 96 rows: 99.8 against 99.9, 128 rows: 119 against 113, 256 rows: 212 against 179; rank 8, 256 rows: 165 against 163).
// Error of t against 64 bits, relative, over M 64 .. 2048, rank 8 .. 64, K 4096 .. 14336: 0.7 - 0.9e-7 (root mean square);
// lora_down_kernel 0.7 - 1.1e-7.
constexpr long long kTileMinBlocks = 4096;
constexpr int kTileWaves = 16;
__global__ __launch_bounds__(kTileWaves* kWave) void lora_down_tile_kernel(const DownArgs args) {
    __shared__ float red[kTileWaves * 256];
    const DownItem& it = args.it[blockIdx.z];
    const int j0 = blockIdx.x * 16, m0 = blockIdx.y * 16, M = args.M, K = it.K, r = it.r;
    if (j0 >= r) return;  // block-uniform
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int row = lane % 16, k8 = lane / 16 * 8;
    const uint16_t* xr = it.x + (size_t)min(m0 + row, M - 1) * K;   // rows past the end repeat the last: not stored
    const uint16_t* ar = it.A + (size_t)min(j0 + row, r - 1) * K;
    constexpr int kAhead = 8, kRound = 32 * kTileWaves;
    f32x4_t part[kAhead];   // short chains and a tree above them: the sums round no worse than lora_down_kernel's
#pragma unroll
    for (int u = 0; u < kAhead; ++u) part[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int kb = wave * 32; kb < K; kb += kAhead * kRound) {
        uint4 xv[kAhead], av[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {   // every load is issued; past the end of K it re-reads element 0 and counts as 0
            const int k = kb + u * kRound + k8;
            const bool in = k < K;
            xv[u] = *reinterpret_cast<const uint4*>(xr + (in ? k : 0));
            av[u] = *reinterpret_cast<const uint4*>(ar + (in ? k : 0));
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (kb + u * kRound + k8 >= K) xv[u] = av[u] = uint4{0u, 0u, 0u, 0u};
            part[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, xv[u]),
                                                              __builtin_bit_cast(bf16x8_t, av[u]), part[u], 0, 0, 0);
        }
    }
#pragma unroll
    for (int o = kAhead / 2; o >= 1; o /= 2)
#pragma unroll
        for (int u = 0; u < o; ++u) part[u] += part[u + o];
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave * 256 + (lane / 16 * 4 + i) * 16 + row] = part[0][i];
    __syncthreads();
    if (threadIdx.x >= 256) return;
    float sums[kTileWaves];
#pragma unroll
    for (int w = 0; w < kTileWaves; ++w) sums[w] = red[w * 256 + threadIdx.x];
#pragma unroll
    for (int o = kTileWaves / 2; o >= 1; o /= 2)
#pragma unroll
        for (int w = 0; w < o; ++w) sums[w] += sums[w + o];
    const int m = m0 + (int)threadIdx.x / 16, j = j0 + (int)threadIdx.x % 16;
    if (m < M && j < r) it.t[(size_t)m * r + j] = sums[0];
}

// y[m][n] = bf16(float(y[m][n]) + scaling * sum_j t[m][j] B[n][j]); a thread keeps its column's row of B in registers and
// takes four rows m at a time, whose t are the same for the whole block: scalar loads of 8, where one read of LDS per product,
// each waited for, took 2 us a row at rank 32.  A block covers 256 columns and 8 rows, so that few rows fill the
// chip too (48 rows: 224 blocks -> 1344); from 512 rows on 32, as each block reads its part of B again (1024 rows: 534 us with
// 8, 522 with 32).  All linears of a call share a launch (plane z of the grid; a wider item's blocks past a narrower one's
// columns leave at once): with one each the four linears of a layer paid for three more.
// Decoder layer, rank 32, with lora_down_kernel's part: M = 2 55.0 us -> 33.0, M = 4 69.5 -> 34.1, M = 48 303 -> 62.9,
// M = 1024 1245 -> 522.
constexpr int kUpMaxRank = 64;
constexpr int kUpStep = 4;          // rows at a time
struct UpItem {
    const uint16_t* B;   // bf16 [N][r]
    const float* t;      // fp32 [M][r]
    uint16_t* y;         // bf16 [M][N]
    int N, r;
    float scaling;
};
struct UpArgs {
    UpItem it[kMaxLoraItems];
    int M, rows;         // rows of a block
};
__global__ __launch_bounds__(256) void lora_up_add_kernel(const UpArgs args) {
    const UpItem& it = args.it[blockIdx.z];
    const int M = args.M, N = it.N, r = it.r;
    const int n = blockIdx.x * 256 + threadIdx.x;
    if (n >= N) return;
    const int m0 = blockIdx.y * args.rows;
    const int rows = min(args.rows, M - m0);
    const float* __restrict__ t = it.t + (size_t)m0 * r;
    uint16_t* __restrict__ y = it.y + (size_t)m0 * N + n;
    uint4 b[kUpMaxRank / 8];
#pragma unroll
    for (int j = 0; j < kUpMaxRank; j += 8)
        if (j < r) b[j / 8] = *reinterpret_cast<const uint4*>(it.B + (size_t)n * r + j);
    for (int mi = 0; mi < rows; mi += kUpStep) {   // a row past the end repeats the last one and is not stored
        float dot[kUpStep] = {};
        uint16_t old[kUpStep];
#pragma unroll
        for (int q = 0; q < kUpStep; ++q) old[q] = y[(size_t)min(mi + q, rows - 1) * N];
#pragma unroll
        for (int j = 0; j < kUpMaxRank; j += 8) {
            if (j < r) {
                const uint32_t w[4] = {b[j / 8].x, b[j / 8].y, b[j / 8].z, b[j / 8].w};
#pragma unroll
                for (int q = 0; q < kUpStep; ++q) {
                    const float* tr = t + min(mi + q, rows - 1) * r + j;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        dot[q] = fmaf(tr[2 * e], __builtin_bit_cast(float, w[e] << 16), dot[q]);
                        dot[q] = fmaf(tr[2 * e + 1], __builtin_bit_cast(float, w[e] & 0xFFFF0000u), dot[q]);
                    }
                }
            }
        }
#pragma unroll
        for (int q = 0; q < kUpStep; ++q)
            if (mi + q < rows)
                y[(size_t)(mi + q) * N] = f32_to_bf16_rne(fmaf(it.scaling, dot[q], bf16_bits_to_f32(old[q])));
    }
}

}  // namespace

bool lora_supports(const qail_wdesc& d, const qail_lora& l) {
    return l.r >= 8 && l.r <= kUpMaxRank && l.r % 8 == 0 && d.K % 8 == 0;
}

// t for item i starts at t + i * M * t_stride floats, rows of r floats... laid out [M][r] with
// the item's own r; t_stride >= r is the per-item allotment per row.
hipError_t launch_lora_down(const qail_w4a16_item* items, const qail_lora* loras, float* t, int t_stride,
                            int count, int M, hipStream_t st) {
    for (int i0 = 0; i0 < count; i0 += kMaxLoraItems) {
        const int c = (count - i0 < kMaxLoraItems) ? count - i0 : kMaxLoraItems;
        DownArgs a;
        int rmax = 0;
        for (int i = 0; i < c; ++i) {
            const qail_w4a16_item& s = items[i0 + i];
            const qail_lora& l = loras[i0 + i];
            a.it[i] = DownItem{s.x, l.A, t + (size_t)(i0 + i) * M * t_stride, s.d.K, l.r};
            if (l.r > rmax) rmax = l.r;
        }
        for (int i = c; i < kMaxLoraItems; ++i) a.it[i] = a.it[c - 1];
        a.M = M;
        if (M > 4 && (long long)rmax * ((M + 3) / 4) * c >= kTileMinBlocks)
            hipLaunchKernelGGL(lora_down_tile_kernel, dim3((rmax + 15) / 16, (M + 15) / 16, c), dim3(kTileWaves * kWave), 0, st, a);
        else if (M <= 4)
            hipLaunchKernelGGL(lora_down_kernel<1>, dim3(rmax, M, c), dim3(kDownThreads), 0, st, a);
        else
            hipLaunchKernelGGL(lora_down_kernel<4>, dim3(rmax, (M + 3) / 4, c), dim3(kDownThreads), 0, st, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_lora_up_add(const qail_w4a16_item* items, const qail_lora* loras, const float* t, int t_stride,
                              int count, int M, hipStream_t st) {
    for (int i0 = 0; i0 < count; i0 += kMaxLoraItems) {
        const int c = (count - i0 < kMaxLoraItems) ? count - i0 : kMaxLoraItems;
        UpArgs a;
        int widest = 0;
        for (int i = 0; i < c; ++i) {
            const qail_w4a16_item& s = items[i0 + i];
            const qail_lora& l = loras[i0 + i];
            a.it[i] = UpItem{l.B, t + (size_t)(i0 + i) * M * t_stride, s.y, s.d.N, l.r, l.scaling};
            if (s.d.N > widest) widest = s.d.N;
        }
        for (int i = c; i < kMaxLoraItems; ++i) a.it[i] = a.it[c - 1];
        a.M = M;
        a.rows = M < 512 ? 8 : 32;
        hipLaunchKernelGGL(lora_up_add_kernel, dim3((widest + 255) / 256, (M + a.rows - 1) / a.rows, c), dim3(256), 0, st, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace qail
