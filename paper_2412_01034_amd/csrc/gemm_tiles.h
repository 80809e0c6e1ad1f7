// Index arithmetic of the matrix-core GEMM (w4a16_gemm.hip) that has to hold for every size it accepts, apart
// from the kernel so that the host can walk through it: where the weight loads of a step read.
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

}  // namespace qail

#endif
