// Walks through the index arithmetic of the matrix-core GEMM (csrc/gemm_tiles.h) on the host.
#include <cstdio>
#include <cstdlib>
#include <vector>

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

// Every K step of every output tile is dealt to exactly one block, and nothing else is.
void dealing(const TilePlan& tp, int tile_m, int Kpad, const char* what, int M, int N) {
    const int cols = tp.tiles / tp.Tm;
    static std::vector<unsigned char> seen;
    seen.assign((size_t)tp.tiles * tp.steps, 0);
    for (int b = 0; b < tp.P; ++b) {
        TileDealer dealer(tp, b, tile_m, Kpad);
        int total = dealer.total_steps(), shared = 0;
        CHECK(total > 0, "%s M %d N %d: block %d of %d has no work", what, M, N, b, tp.P);
        TileDealer::Segment sg;
        while (dealer.next(sg)) {
            total -= sg.steps;
            CHECK(sg.tm >= 0 && sg.tm < tp.Tm && sg.tn >= 0 && sg.tn < cols, "%s M %d N %d: block %d works on tile (%d, %d) of %d x %d", what, M, N, b,
                  sg.tm, sg.tn, tp.Tm, cols);
            CHECK(sg.ka >= 0 && sg.steps >= 1 && sg.ka + sg.steps <= tp.steps, "%s M %d N %d: steps %d + %d of %d", what, M, N, sg.ka, sg.steps, tp.steps);
            // a block has two slots for sums of parts of a tile: its first shared segment's and one more
            if (sg.steps != tp.steps && !sg.first_shared) ++shared;
            for (int s = sg.ka; s < sg.ka + sg.steps; ++s) {
                unsigned char& c = seen[((size_t)sg.tn * tp.Tm + sg.tm) * tp.steps + s];
                CHECK(c == 0, "%s M %d N %d: tile (%d, %d) step %d dealt twice", what, M, N, sg.tm, sg.tn, s);
                c = 1;
            }
        }
        CHECK(total == 0 && shared <= 1, "%s M %d N %d: block %d, %d steps left over, %d shared segments", what, M, N, b, total, shared);
    }
    for (size_t i = 0; i < seen.size(); ++i)
        CHECK(seen[i], "%s M %d N %d: tile (%d, %d) step %d dealt to nobody", what, M, N, (int)(i / tp.steps % tp.Tm), (int)(i / tp.steps / tp.Tm),
              (int)(i % tp.steps));
}

// Plans as the launcher makes them, for a linear alone and for shares of the grid that begin anywhere.
void planned(int M, int N, int K, int cus) {
    const int rows = tile_rows(M), Kpad = round_up(K, kPadK);
    const int shares[][2] = {{cus, 0}, {cus / 2, 0}, {cus / 2, cus / 2}, {cus / 4 + 3, 5}, {cus / 16, 8}, {1, 3}};
    for (int bits : {4, 8})
        for (const auto& sh : shares)
            for (bool narrow_only : {false, true}) {
                int wn;
                bool split;
                choose_tile(bits, rows, M, N, Kpad, sh[0], sh[0] == cus, narrow_only, &wn, &split);
                TilePlan tp = plan_tiles(M, N, K, rows, 128 * wn, step_k(bits), split, sh[0]);
                tp.block_begin = sh[1];
                dealing(tp, rows, Kpad, bits == 4 ? "nibbles" : "bytes", M, N);
            }
}

// Byte codes: a linear of a few tiles and a K worth sharing keeps a good part of the chip busy, also where only
// narrow tiles have room.
void byte_parts(int M, int N, int K, bool narrow_only, int least) {
    int wn;
    bool split;
    choose_tile(8, tile_rows(M), M, N, round_up(K, kPadK), 256, true, narrow_only, &wn, &split);
    const TilePlan tp = plan_tiles(M, N, K, tile_rows(M), 128 * wn, step_k(8), split, 256);
    CHECK(tp.P >= least, "M %d N %d K %d: %d blocks", M, N, K, tp.P);
}

// The second kernel's arithmetic agrees with the general one on both sides of the line between them.
void quick_units() {
    for (long long units : {1ll, 2ll, 63ll, 1376ll, 4096ll, kUnits32 - 1, kUnits32, kUnits32 + 1, (1ll << 27) - 5})
        for (int P : {1, 2, 7, 114, 255, 256, 304, kMaxGemmBlocks}) {
            for (int b = 0; b <= P; ++b)
                CHECK(first_unit_quick(b, units, P) == (int)first_unit(b, units, P), "units %lld P %d block %d", units, P, b);
            for (long long u : {0ll, 1ll, units / 3, units / 2, units - 2, units - 1})
                if (u >= 0 && u < units) CHECK(owner_of_quick((int)u, units, P) == owner_of(u, units, P), "units %lld P %d unit %lld", units, P, u);
        }
}

}  // namespace

int main() {
    quick_units();
    for (int bits : {4, 8})
        for (uint32_t K = 64; K <= 2048; K += 64)
            for (uint32_t g = 64; g <= K; g += 64)
                for (uint32_t N : {1u, 2u, 7u, 128u, 129u, 260u, 4096u})
                    if (K % g == 0) loads(bits, N, K, g);
    // every width of the linears a model may have, at every tile height and number of row tiles up to sixteen
    for (int cus : {256, 304, 64})
        for (int M : {17, 33, 96, 128, 129, 288, 320, 384, 512, 640, 768, 897, 1000, 1024, 1536, 2048})
            for (int N = cus == 256 && M > 896 && M <= 1024 ? 128 : 384; N <= 24000; N += M > 896 && M <= 1024 ? 256 : 1280) planned(M, N, 1536, cus);
    for (int N : {2, 100, 128, 130, 11008, 11520, 12544, 32000})
        for (int K : {64, 192, 1024, 4096, 11008})
            for (int M : {17, 200, 1024}) planned(M, N, K, 256);
    for (bool narrow_only : {false, true}) {
        byte_parts(288, 128, 4096, narrow_only, 48);    // three tiles of 64 steps
        byte_parts(40, 64, 4096, narrow_only, 16);
        byte_parts(40, 4096, 4096, narrow_only, 256);
        byte_parts(96, 2048, 1024, narrow_only, 64);
        byte_parts(288, 4096, 11008, narrow_only, 192);
    }
    std::printf("gemm tiles: ok\n");
    return 0;
}
