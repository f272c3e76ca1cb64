// Building blocks of the workgroup-tile strided passes (gfx950), shared by eden_kernels_wg.hip (encode) and
// eden_kernels_wg_dec.hip (decode).
//
// Two passes through memory are enough for every D up to 2^27 when a workgroup keeps 2^14 .. 2^16 coordinates on chip
// (registers + one or two exchanges through LDS):
//
//   contiguous pass (index bits 0 .. P-1, P = 14, 15, 16): eden_kernels_lo14.hip, eden_kernels_lo15.hip.
//   hiX pass  (strided, index bits P .. P+M-1, M = 7..11): a workgroup owns 2^M rows of 32 consecutive
//             coordinates (128-byte segments) at stride 2^P.  Every thread keeps 64 rows of one column in
//             registers (six butterfly stages), the remaining M-6 row bits are reached by one exchange through
//             LDS, in two halves (M = 10: 64 KiB, two workgroups per CU; M = 11: 128 KiB, 1024 threads; M <= 9: with the
//             exchange in one piece the LDS held 2 to 3 waves per SIMD; 8 senders of 2^22, 2.7 bits: first decode pass 97 -> 67 us).
//
// The strided pass is the one next to the payload: encode runs it last and fuses quantization against the
// Lloyd-Max thresholds, <R(x),Q> and packing (Sec. 2.2.1, 2.3, 3, 4.1); decode runs it first and fuses
// unpacking and dequantization with S/(p sqrt D) (Sec. 2.2.2, 4.2).  The contiguous pass is the one next to x
// and to the accumulator, where the zero padding of d up to D costs nothing.
#ifndef EDEN_HIX_H
#define EDEN_HIX_H

#include "eden_device.h"

namespace eden {

template <int M, int PIECES = 2>
struct HiX {
    static constexpr int RL = 1 << (M - 6);       // row groups: the low M-6 row bits live across thread groups
    static constexpr int THREADS = 32 * RL;
    static constexpr int PH = PIECES;               // pieces (halves) of the exchange
    static constexpr int RP = 64 / PH;            // registers exchanged per half
    static constexpr int RHL = RP / RL;           // high-row values a thread holds after the exchange
    static constexpr int LDS_FLOATS = RP * RL * 32;
};

// Workgroups are dealt to the 8 XCDs round robin and each XCD has its own L2.  Neighbouring tiles touch
// neighbouring 64..128-byte pieces of the same rows (and, in decode, the same 64-byte sectors of the payload),
// so runs of 16 consecutive tiles are kept on one XCD.
template <int RUN = 16>
__device__ inline uint32_t xcd_local_tile(uint32_t tile = blockIdx.x) {
    if (gridDim.x % (8u * RUN) == 0) {
        const uint32_t xcd = tile & 7u, q = tile >> 3;
        tile = ((q / RUN) * 8u + xcd) * RUN + (q % RUN);
    }
    return tile;
}

// The payload starts 64 bytes into a message, so its 128-byte memory lines do not start where the runs of neighbouring
// tiles start: every line would be shared by two runs (two XCDs) and fetched twice (measured: 64 MiB for a 32 MiB payload).
// Rotates the column-block index of a tile so that the runs start on line boundaries.  `row_bytes`: payload bytes of one
// tile row, a power of two below 128; `cb_bits`: log2 of the column blocks per row.
__host__ __device__ inline uint32_t align_runs_to_lines(uint32_t tile, uint32_t cb_bits, const void *payload, uint32_t row_bytes) {
    const uint32_t per_line = 128u / row_bytes;
    const uint32_t shift = (uint32_t)(reinterpret_cast<uintptr_t>(payload) / row_bytes) & (per_line - 1u);
    const uint32_t mask = (1u << cb_bits) - 1u;
    return (tile & ~mask) | ((tile - shift) & mask);
}

// whether the first decode pass in 32-column tiles does so: at one bit a run is half a line wherever the payload starts on a multiple of 64
__host__ __device__ constexpr bool rotates_tiles(uint32_t bits) { return bits == 2u || bits == 4u || bits == 8u; }

// Decode: the payload of a workgroup that starts later on this XCD, brought into its L2 while this one computes.  Every workgroup of a
// first decode pass begins with a read of 2^M short pieces of the payload and can do nothing else until they are there; messages
// that have just arrived lie in memory, and a run of 16 tiles (which share the lines) waited for them together.  The 16
// workgroups of a run each read a word of 1/16 of the lines of the run 2^18 threads further on, about as many as the chip holds at a time.
// The word is not used.  The read is a volatile one behind a branch, so that its few waves wait for it before they go on; that is the better
// way where values are looked up (hot messages, us, this / a buffer load that nothing waits for: mean of 16 senders of 11,173,962, b = 2
// 307 / 313, b = 4 341 / 348, of 8 of 2^25, b = 4 538 / 546; b = 1, on the matrix cores, 169.3 / 168.3 and 312 / 311).
// Against passes without it, the same two sets of messages in turn / single passes on messages that lie in no cache, us: mean of 16 senders of
// 11,173,962, b = 1 184 -> 169 / 228 -> 218, b = 2 305 -> 299 / 442 -> 342, b = 4 418 -> 331 / 445 -> 341; of 8 of 2^25, b = 1
// 364 -> 310 / 369 -> 319, b = 4 583 -> 539 / 607 -> 572; of 4 of 2^27, b = 4 1373 -> 1281 / 1399 -> 1303 (with what else changed between
// the two builds: the sums of the last pass at b = 2 and 4).  Where an encode has just left the messages in the memory-side cache
// nothing is gained or lost (a round of 16 of 11,173,962, b = 4 755 -> 755).
// THREADS: of a workgroup; TILES: per sender, a multiple of 128; `row_bytes`: payload bytes of one tile row; `rotated`: the pass rotates
// its tiles by align_runs_to_lines.
//
// lines of a payload row that a run of 16 tiles shares
__host__ __device__ constexpr uint32_t touch_lines_per_row(uint32_t row_bytes) { return row_bytes > 8u ? 2u : 1u; }
// Where the thread's word lies in the payload of the sender of workgroup x (counted on over the senders); ~0: it has none.  (Inside the
// payload: rows below 2^M, tiles below TILES.)
template <int M, uint32_t TILES>
__host__ __device__ inline uint32_t touch_place(uint32_t x, uint32_t thread, const void *payload, uint32_t row_bytes, bool rotated) {
    constexpr uint32_t kRows = (1u << M) / 16u;
    static_assert(TILES % 128u == 0, "runs of 16 tiles on each of 8 XCDs, see xcd_local_tile");
    const uint32_t per_row = touch_lines_per_row(row_bytes);
    if (thread >= kRows * per_row) return ~0u;
    const uint32_t q = (x % TILES) >> 3, run = (q / 16u) * 8u + (x & 7u);
    const uint32_t row = (q % 16u) * kRows + thread / per_row;
    uint32_t tile = run * 16u + thread % per_row * 8u;
    if (rotated) tile = align_runs_to_lines(tile, (uint32_t)__builtin_ctz(TILES), payload, row_bytes);
    return (row * TILES + tile) * row_bytes;
}
template <uint32_t THREADS, int M, uint32_t TILES>
__device__ inline void touch_payload_ahead(const DecBatch &B, uint32_t row_bytes, bool rotated) {
    const uint32_t x = blockIdx.x + (1u << 18) / THREADS, c = blockIdx.y + x / TILES;
    if (c >= gridDim.y || wave_in_block() * 64u >= (1u << M) / 16u * touch_lines_per_row(row_bytes)) return;
    if (B.b_q8[c] != B.b_q8[blockIdx.y]) return;                 // `row_bytes` would not be that sender's
    const char *payload = static_cast<const char *>(B.msg[c]) + EDEN_HEADER_BYTES;
    const uint32_t at = touch_place<M, TILES>(x, threadIdx.x, payload, row_bytes, rotated);
    if (at != ~0u) (void)*reinterpret_cast<const volatile uint32_t *>(payload + at);
}

template <int M>
__device__ inline uint64_t hix_base(uint32_t tile, int p) {
    const uint32_t cb_bits = (uint32_t)p - 5u;                   // 2^(p-5) blocks of 32 columns
    const uint32_t cb = tile & ((1u << cb_bits) - 1u);
    const uint32_t upper = tile >> cb_bits;
    return ((uint64_t)upper << (p + M)) | ((uint64_t)cb << 5);
}

// row held in stage-1 register r by a thread of group g
template <int M>
__device__ inline uint32_t hix_row1(uint32_t g, uint32_t r) { return g + (uint32_t)HiX<M>::RL * r; }
// row held after the exchange of half ph in register s by a thread of group g
template <int M, int PIECES = 2>
__device__ inline uint32_t hix_row2(uint32_t g, int ph, int s) {
    using X = HiX<M, PIECES>;
    const uint32_t e = (uint32_t)s / X::RL, rl = (uint32_t)s % X::RL;
    const uint32_t rh = (uint32_t)ph * X::RP + g * X::RHL + e;
    return rl + (uint32_t)X::RL * rh;
}

// Exchange of half `PHASE`: stage-1 registers -> LDS -> registers that hold all low row bits of
// RHL high-row values; then the butterflies over those low row bits.  Split in two so that a caller can
// start loading the next tile into the registers the write has just freed.
template <int M, int PHASE, int N>
__device__ inline void hix_exchange_write(const float (&v)[N], float *lds) {
    using X = HiX<M>;
    const uint32_t col = threadIdx.x & 31u, g = threadIdx.x >> 5;
    // an LDS instruction reaches 64 KiB beyond its address register: M = 11 gets one register per 64 KiB (left to itself the
    // compiler keeps sixteen, and spills)
    constexpr int PER = 512 / X::RL < X::RP ? 512 / X::RL : X::RP;
#pragma unroll
    for (int first = 0; first < X::RP; first += PER) {
        uint32_t at = (uint32_t)(first * X::RL * 32) + g * 32u + col;
        if (first > 0) asm volatile("" : "+v"(at));
#pragma unroll
        for (int i = 0; i < PER; ++i) lds[at + (uint32_t)(i * X::RL * 32)] = v[PHASE * X::RP + first + i];
    }
}
// ALL_STAGES = false leaves out the stage over bit 0 of the register index (see hix_sign_words_pairs).
template <int M, bool ALL_STAGES = true>
__device__ inline void hix_exchange_read(float *lds, float (&out)[HiX<M>::RP]) {
    using X = HiX<M>;
    const uint32_t col = threadIdx.x & 31u, g = threadIdx.x >> 5;
    __syncthreads();
#pragma unroll
    for (int s = 0; s < X::RP; ++s) {
        const int e = s / X::RL, rl = s % X::RL;
        out[s] = lds[((g * X::RHL + e) * X::RL + rl) * 32 + col];
    }
    __syncthreads();
    fwht_regs_low<X::RP, M - 6, ALL_STAGES ? 1 : 2>(out);
}
template <int M, int PHASE>
__device__ inline void hix_exchange(const float (&v)[64], float *lds, float (&out)[HiX<M>::RP]) {
    hix_exchange_write<M, PHASE>(v, lds);
    hix_exchange_read<M>(lds, out);
}

// ONLY of the kernels next to the payload, beside a budget: every sender of the launch has a coin budget k + f with this k
constexpr uint32_t kCoinOnly = 0xC000u;          // + k
static inline uint32_t coin_floor_of_all(const uint32_t *b_q8, uint32_t n) {     // 0: they differ, or some budget is of another kind
    const uint32_t k = coin_q8(b_q8[0]) >> 8;
    for (uint32_t c = 1; c < n; ++c)
        if (coin_q8(b_q8[c]) >> 8 != k) return 0u;
    return k;
}

static inline uint32_t hix_tiles(int M, int log2D) { return 1u << (log2D - M - 5); }

// the plans that exist: M bits on top of a contiguous pass over P bits (D = 2^(P+M))
#define EDEN_HIX_SWITCH(M, P, CALL)                                                           \
    switch (100 * (M) + (P)) {                                                                \
        case 714: { constexpr int MM = 7, PP = 14; CALL; } break;                             \
        case 814: { constexpr int MM = 8, PP = 14; CALL; } break;                             \
        case 914: { constexpr int MM = 9, PP = 14; CALL; } break;                             \
        case 1014: { constexpr int MM = 10, PP = 14; CALL; } break;                           \
        case 1015: { constexpr int MM = 10, PP = 15; CALL; } break;                           \
        case 1115: { constexpr int MM = 11, PP = 15; CALL; } break;                           \
        default: { constexpr int MM = 11, PP = 16; CALL; } break;                             \
    }

}  // namespace eden
#endif
