// Walks through the index arithmetic of the matrix-core GEMM (csrc/gemm_tiles.h) on the host.
#include <cstdio>
#include <cstdlib>

#include "gemm_tiles.h"

using namespace qail;

namespace {

#define CHECK(cond, ...)                                          \
    do {                                                          \
        if (!(cond)) {                                            \
            std::printf("failed: %s: ", #cond);                   \
            std::printf(__VA_ARGS__);                             \
            std::printf("\n");                                    \
            std::exit(1);                                         \
        }                                                         \
    } while (0)

// Every weight load of every step, the ring's look-ahead past the last one among them, stays inside its
// tensor, and a piece that lies inside K is the right one.
void loads(int bits, uint32_t N, uint32_t K, uint32_t g) {
    const uint32_t G = K / g, zwords = (G + 7) / 8, row_words = K * bits / 32, bk = step_k(bits);
    if (N * G % 2 != 0) return;   // not a shape the kernel takes
    const uint32_t codes = N * K * bits / 8, scales = N * G * 2, zeros = N * zwords * 4;
    const uint32_t steps = (K + bk - 1) / bk + ring_stages(bits);
    for (uint32_t n : {0u, N / 2, N - 1}) {
        for (uint32_t s = 0; s < steps; ++s)
            for (uint32_t piece = 0; piece < 4; ++piece) {
                const uint32_t at = code_offset(n, row_words, piece) + code_step_offset(s * bk, piece, K, bits);
                CHECK(at % 16 == 0 && at + 16 <= codes, "codes: bits %d N %u K %u g %u row %u step %u piece %u at %u of %u", bits, N, K, g, n, s,
                      piece, at, codes);
                const uint32_t k = s * bk + piece * 128 / bits;
                CHECK(k >= K || at == n * row_words * 4 + k * bits / 8, "codes: bits %d N %u K %u row %u k %u at %u", bits, N, K, n, k, at);
            }
        for (uint32_t grp = 0; grp < G; ++grp) {
            const uint32_t s = scale_word_offset(n * G * 2, grp), z = zero_word_offset(n * zwords * 4, grp);
            CHECK(s % 4 == 0 && s <= n * G * 2 + grp * 2 && s + 4 > n * G * 2 + grp * 2 && s + 4 <= scales, "scales: N %u K %u g %u", N, K, g);
            CHECK(z % 4 == 0 && z + 4 <= zeros, "zeros: N %u K %u g %u", N, K, g);
        }
    }
}

}  // namespace

int main() {
    for (int bits : {4, 8})
        for (uint32_t K = 64; K <= 2048; K += 64)
            for (uint32_t g = 64; g <= K; g += 64)
                for (uint32_t N : {1u, 2u, 7u, 128u, 129u, 260u, 4096u})
                    if (K % g == 0) loads(bits, N, K, g);
    std::printf("gemm tiles: ok\n");
    return 0;
}
