// For every kind of first decode pass, payload place and workgroup: the words that the workgroups of a run of tiles read ahead
// (touch_place in eden_hix.h) lie in lines that the tiles of the run further on read, in the same row.  Host code only.
#include <cstdio>
#include <set>

#include "eden_hix.h"

using namespace eden;

// tiles in the order of the workgroups, as xcd_local_tile deals them, rotated if the pass does so
template <uint32_t TILES>
static uint32_t tile_of(uint32_t x, const char *payload, uint32_t row_bytes, bool rotated) {
    const uint32_t q = (x % TILES) >> 3, tile = ((q / 16u) * 8u + (x & 7u)) * 16u + q % 16u;
    return rotated ? align_runs_to_lines(tile, (uint32_t)__builtin_ctz(TILES), payload, row_bytes) : tile;
}

template <int M, uint32_t TILES>
static int check(uint32_t row_bytes, bool rotated) {
    int bad = 0;
    for (uintptr_t place = 0; place < 256; place += 16) {        // messages are aligned to 16 bytes
        const char *payload = reinterpret_cast<const char *>((uintptr_t)1 << 32) + place;
        for (uint32_t first = 0; first < 256; first += 128)      // workgroups first + xcd + 8 i, i < 16: a run on every XCD
            for (uint32_t xcd = 0; xcd < 8; ++xcd) {
                std::set<uintptr_t> read, rows;                  // lines of the run
                for (uint32_t i = 0; i < 16; ++i) {
                    const uint32_t tile = tile_of<TILES>(first + xcd + 8 * i, payload, row_bytes, rotated);
                    for (uint32_t row = 0; row < (1u << M); ++row)
                        for (uint32_t b = 0; b < row_bytes; b += 4)
                            read.insert((reinterpret_cast<uintptr_t>(payload) + ((size_t)row * TILES + tile) * row_bytes + b) / 128);
                }
                for (uint32_t i = 0; i < 16; ++i)
                    for (uint32_t t = 0; t < 512; ++t) {
                        const uint32_t at = touch_place<M, TILES>(first + xcd + 8 * i, t, payload, row_bytes, rotated);
                        if (at == ~0u) continue;
                        if (at + 4 > (row_bytes * TILES) << M) { printf("outside the payload\n"); return 1; }
                        rows.insert(at / (row_bytes * TILES));
                        if (!read.count((reinterpret_cast<uintptr_t>(payload) + at) / 128)) ++bad;
                    }
                if (rows.size() != (1u << M)) { printf("rows left out\n"); return 1; }
            }
    }
    if (bad) printf("M %d row_bytes %u: %d words in lines of other runs\n", M, row_bytes, bad);
    return bad != 0;
}

int main() {
    int bad = 0;
    for (uint32_t bits = 1; bits <= 4; ++bits) {                 // 32-column tiles of D = 2^21 and 2^23
        bad += check<7, 512>(4 * bits, rotates_tiles(bits));
        bad += check<9, 512>(4 * bits, rotates_tiles(bits));
    }
    bad += check<8, 256>(8, true);                               // 64-column tiles, b = 1 and 1/2
    bad += check<8, 256>(4, true);
    if (!bad) printf("touch ok\n");
    return bad != 0;
}
