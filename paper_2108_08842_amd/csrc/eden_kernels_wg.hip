// Last encode pass in workgroup tiles (D = 2^21 .. 2^27, gfx950), and the middle pass of the one-byte budgets: see eden_hix.h
// for the tiles.
#include "eden_device.h"
#include "eden_hix.h"
#include "eden_kernels.h"

namespace eden {

// ---- packing in the strided layout.  After a tile's last butterfly a register holds, across the two halves of
// a wave, two row segments of 32 consecutive coordinates: exactly one payload word each at b = 1.  A ballot
// of one bit of the index gives both words at once; lane j of each half collects the words of register j
// (v_writelane), and after the last register every lane finishes and stores the words of "its" row.
// row of the tile whose words lane j holds for register block w after half ph of the exchange
template <int M>
__device__ inline uint32_t hix_word_row(int ph, int w) {
    using X = HiX<M>;
    const uint32_t s = 32u * (uint32_t)w + (lane_id() & 31u), g = threadIdx.x >> 5;
    return s % X::RL + (uint32_t)X::RL * ((uint32_t)ph * X::RP + g * X::RHL + s / X::RL);
}

// Quantizes and packs the RP values a thread holds after one half of the exchange (rows hix_row2(g, PH, s)).
// `word0`: payload word index of this tile's 32 columns in row 0; `base`: first coordinate of the tile.
// BITS: bits of every index in the first part of the payload.  MIX = 1 (b = BITS + 1/2, Sec. 4.1): the coordinate of
// every pair that the MIX stream selects is quantized with I_{BITS+1}; the top bit of its index goes to the
// second part of the payload, one bit per pair = 16 bits per row segment of a tile.  MIX = 2 (coin budgets, Sec. 4.1):
// the coordinates with a coin use I_{BITS+1}; their top bits go to the second part (`part_c`) in coordinate order, at the
// place the prefix sums over the coins give the row segment.
// TRANSPOSE (BITS = 2 or 4, MIX = 0): instead of the ballots, a lane collects the indices of 16 or eight registers (rows) of its
// column in one word, and the lanes of as many neighbouring columns transpose their words: each then holds one payload word of
// one row.  2 instructions per register instead of 12 (b = 4), but more code: only the kernel instances whose senders all have that
// budget use it (in the instance shared by all budgets it raised the register spills and cost b = 2 a quarter of its speed).  Encode
// at b = 2 with the instance of its own: 8 senders of 10^8 2960 -> 2399 us, 16 of 11,173,962 424 -> 408, 8 of 4,000,037 78.1 -> 74.4, one of
// 1,500,000 20.9 -> 18.8.
template <int M, int P, int BITS, int MIX, bool TRANSPOSE = false>
__device__ inline void hix_quantize_pack(const float (&out)[HiX<M>::RP], int ph, const EncScratch *sc, const float *qtab,
                                         uint32_t *payload, uint16_t *part_b, uint64_t mixkey, uint64_t base, float &ip,
                                         const CoinTables &ct, uint32_t c, int log2D, uint32_t *part_c,
                                         const RankGuess<8> *guess = nullptr, uint32_t *pieces = nullptr) {
    using X = HiX<M>;
    constexpr int p = P;
    constexpr int H = 1 << (BITS - 1);
    constexpr int NW = X::RP / 32;                               // registers come in blocks of 32 = one word lane each
    const uint32_t lane = lane_id(), col = lane & 31u;
    const uint32_t word0 = (uint32_t)(base >> 5);
    if constexpr (TRANSPOSE && MIX == 0) {
        static_assert(BITS == 2 || BITS == 4, "words of whole indices");
        constexpr int PER = 32 / BITS;
        const uint32_t g = threadIdx.x >> 5, j = col & (uint32_t)(PER - 1), q = col / (uint32_t)PER;
        const float thr1 = sc->thr[1], q0 = sc->qpos[0], q1 = sc->qpos[1];
        static_for<X::RP / PER>([&](auto K) {
            constexpr int k = decltype(K)::value;
            uint32_t items;
            if constexpr (BITS == 2) {
                items = quantize_two_bits(&out[PER * k], thr1, q0, q1, ip);
            } else {
                uint32_t at[PER];
                quantize_guess<H>(&out[PER * k], *guess, sc, at, ip);
                items = pack_guesses(at);
            }
            items = transpose_items<BITS>(items, lane);
            const uint32_t row = hix_row2<M>(g, ph, (int)(PER * k + j));
            payload[(uint32_t)BITS * (word0 + (row << (p - 5))) + q] = items;
        });
        return;
    }
    const Thresholds th = thresholds_of(sc);
    uint32_t plane[BITS][NW], top[NW], chosen[NW], coin_off[NW];   // chosen: of this lane's row segments, the coordinates with I_{BITS+1}
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        top[w] = 0;
#pragma unroll
        for (int b = 0; b < BITS; ++b) plane[b][w] = 0;
        // this lane's row for register block w; 64 pairs per hash word of the MIX stream, 16 of them in that row segment
        const uint64_t first = base + ((uint64_t)hix_word_row<M>(ph, w) << p);
        chosen[w] = MIX == 1 ? chosen_of_pairs((uint32_t)(hash_word(mixkey, first >> 7) >> (16u * (uint32_t)((first >> 5) & 3u)))) : 0u;
        coin_off[w] = 0;
        if constexpr (MIX == 2) {                                // the 32 coins of that row segment: half of a block of 64
            const uint32_t blk = (uint32_t)(first >> 6), upper = (uint32_t)(first >> 5) & 1u;
            const uint64_t m64 = coin_mask_of(ct, c, log2D, blk);
            chosen[w] = upper ? hi32(m64) : lo32(m64);
            coin_off[w] = coins_before(ct, c, log2D, blk) + (upper ? (uint32_t)__popc(lo32(m64)) : 0u);
        }
    }
    uint32_t items = 0, three = 0;                               // TRANSPOSE: the low bits of 16 and of three registers
    uint32_t at[4];                                              // where the centroids of four values lie in qtab
    static_for<X::RP>([&](auto S) {
        constexpr int s = decltype(S)::value;
        uint64_t bit[BITS];                                      // lane masks of the index's low bits
        if constexpr (MIX != 0) {
            const uint64_t up = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)chosen[s / 32], 32 + s % 32) << 32 |
                                (uint32_t)__builtin_amdgcn_readlane((int)chosen[s / 32], s % 32);
            uint64_t high;
            at[s % 4] = quantize_two_tables<BITS>(out[s], up, th, bit, high);
            top[s / 32] = put_lane<s % 32>(lo32(high), top[s / 32]);
            top[s / 32] = put_lane<32 + s % 32>(hi32(high), top[s / 32]);
        } else {
            at[s % 4] = quantize_one_table<BITS>(out[s], th, bit);
        }
        if constexpr (TRANSPOSE && MIX == 2) {
            // (three values at a time, whose places fit an instruction's inline constants: with a place of its own every value took two
            // registers)
            constexpr int i = s % 16, place = 2 * (i % 3);
            three |= (__builtin_amdgcn_inverse_ballot_w64(bit[0]) ? 1u << place : 0u) | (__builtin_amdgcn_inverse_ballot_w64(bit[1]) ? 2u << place : 0u);
            asm volatile("" : "+v"(three));                      // (not the masks of all sixteen first)
            if constexpr (i % 3 == 2 || i == 15) {
                items |= three << (2 * (i - i % 3));
                three = 0;
            }
            if constexpr (i == 15) {
                items = transpose_items<2>(items, lane);
                payload[2u * (word0 + (hix_row2<M>(threadIdx.x >> 5, ph, s - 15 + (int)(col & 15u)) << (p - 5))) + (col >> 4)] = items;
                items = 0;
            }
        } else {
#pragma unroll
            for (int b = 0; b < BITS; ++b) {
                plane[b][s / 32] = put_lane<s % 32>(lo32(bit[b]), plane[b][s / 32]);
                plane[b][s / 32] = put_lane<32 + s % 32>(hi32(bit[b]), plane[b][s / 32]);
            }
        }
        if constexpr (s % 4 == 3) add_centroids<4>(&out[s - 3], at, qtab, ip);
    });
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const uint32_t word = word0 + (hix_word_row<M>(ph, w) << (p - 5));
        if constexpr (TRANSPOSE) {                               // (stored already)
        } else if constexpr (BITS == 1) {
            payload[word] = plane[0][w];
        } else if constexpr (BITS == 2) {
            const uint32_t a = plane[0][w], b = plane[1][w];
            *reinterpret_cast<uint2 *>(payload + 2u * word) =
                make_uint2(spread2(a) | (spread2(b) << 1), spread2(a >> 16) | (spread2(b >> 16) << 1));
        } else if constexpr (BITS == 3) {
            uint32_t o[3];                                       // 32 coordinates x 3 bits = 3 words
            pack3_planes(plane[0][w], plane[1][w], plane[2][w], o);
            payload[3u * word] = o[0];
            payload[3u * word + 1u] = o[1];
            payload[3u * word + 2u] = o[2];
        } else {
            uint32_t o[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                o[k] = spread4(plane[0][w] >> (8 * k)) | (spread4(plane[1][w] >> (8 * k)) << 1) |
                       (spread4(plane[2][w] >> (8 * k)) << 2) | (spread4(plane[3][w] >> (8 * k)) << 3);
            *reinterpret_cast<uint4 *>(payload + 4u * word) = make_uint4(o[0], o[1], o[2], o[3]);
        }
        if constexpr (MIX == 1) part_b[word] = (uint16_t)even_bits(top[w] | (top[w] >> 1));    // only the chosen one can be set
        if constexpr (MIX == 2) {                                // only a coordinate with a coin can have the bit
            const uint32_t piece = compress_bits(top[w], chosen[w]);
            // either the piece goes to the staging array (word = number of the segment of 32 coordinates; k_coin_pack strings
            // the pieces together) or straight to its bits of the second part, which neighbouring tiles share: atomics
            if (pieces) pieces[word] = piece;
            else or_bits(part_c, coin_off[w], piece, (uint32_t)__popc(chosen[w]));
        }
    }
}

// b = 1 and b = 1/2: the index is the sign (I_1, Sec. 3), <R(x),Q> = q_1 sum |u| / sqrt(D).  Leaves in words[w],
// lane j of each half, the 32 index bits of the row segment held in register 32 w + j.
template <int M>
__device__ inline void hix_sign_words(const float (&out)[HiX<M>::RP], float &ip, uint32_t (&words)[HiX<M>::RP / 32]) {
    using X = HiX<M>;
    float sa = 0.0f;
#pragma unroll
    for (int s = 0; s < X::RP; ++s) sa += fabsf(out[s]);
    ip = fmaf(sa, kQ1, ip);
#pragma unroll
    for (int w = 0; w < X::RP / 32; ++w) words[w] = 0;
    static_for<X::RP>([&](auto S) {
        constexpr int s = decltype(S)::value;
        const uint64_t m = __ballot((__float_as_uint(out[s]) >> 31) == 0u);      // index 1 = non-negative
        words[s / 32] = put_lane<s % 32>(lo32(m), words[s / 32]);
        words[s / 32] = put_lane<32 + s % 32>(hi32(m), words[s / 32]);
    });
}

// The same from the values BEFORE the last butterfly stage (registers 2 i and 2 i + 1 hold a and b; the transformed values
// would be a + b and a - b).  The sign quantizer needs of them only their signs and the sum of their magnitudes:
// a + b >= 0 is "not a < -b", a - b >= 0 is "not a < b" (the same decisions: rounding never changes the sign of a sum, and
// the passes before leave no negative zeros), and |a + b| + |a - b| = 2 max(|a|, |b|), which, unlike the two sums, is exact.
// Four instructions per pair (max, add, two compares) instead of six.
template <int M>
__device__ inline void hix_sign_words_pairs(const float (&out)[HiX<M>::RP], float &ip, uint32_t (&words)[HiX<M>::RP / 32]) {
    using X = HiX<M>;
    float sa = 0.0f;
#pragma unroll
    for (int s = 0; s < X::RP; s += 2) sa += fmaxf(fabsf(out[s]), fabsf(out[s + 1]));
    ip = fmaf(2.0f * sa, kQ1, ip);
#pragma unroll
    for (int w = 0; w < X::RP / 32; ++w) words[w] = 0;
    static_for<X::RP>([&](auto S) {
        constexpr int s = decltype(S)::value;
        const float a = out[s & ~1], b = out[s | 1];
        const uint64_t m = (s & 1) ? __ballot(!(a < b)) : __ballot(!(a < -b));     // index 1 = non-negative
        words[s / 32] = put_lane<s % 32>(lo32(m), words[s / 32]);
        words[s / 32] = put_lane<32 + s % 32>(hi32(m), words[s / 32]);
    });
}

template <int N> struct WordVec;
template <> struct WordVec<1> { using type = uint32_t; };
template <> struct WordVec<2> { using type = uint2; };
template <> struct WordVec<4> { using type = uint4; };

// Encode, last pass: T -> payload.  Index bits P .. P+M-1 of H, then quantization to the Lloyd-Max intervals
// (Sec. 2.2.1, Sec. 3), sum_i u_i q_i for the scale (Sec. 2.3), sub-sampling for b = 1/2 (Sec. 4.1), packing.
// Rows of the workspace at or above ceil(d / 2^P) were not written by the first pass (they are zero padding
// transformed over bits 0..P-1, i.e. zero): the buffer bounds return 0 for them without touching memory.
// A workgroup handles TPW neighbouring column blocks; the loads of the next one are issued into the registers
// that each half of the exchange has just written to LDS.  MODE 0: every sender of the launch has b <= 1; the
// words of the TPW tiles are then kept and stored together (one row of a tile is only 4 bytes of payload).
// MODE 1: any integer budget or b = 1/2.  MODE 2: also the budgets k + 1/2 (they need more registers).
// MODE 3: every sender of the launch has b = 4 (the instance holds nothing else: no spills, and the transposing pack).
// BLK: the first pass wrote the workspace in the blocked layout (blocked_offset in eden_device.h; always for P > 14).
// ONLY != 0: every sender of the launch has this budget; the instance holds that one branch of the quantizers.
template <int M, int P, int TPW, int MODE, bool BLK, uint32_t ONLY = 0>
__global__ __launch_bounds__(HiX<M>::THREADS, TPW == 1 ? 4 : 1) void k_enc_hix_last(EncBatch B, uint64_t d, int log2D, uint64_t seed,
                                                                   const float *T, double *partials,
                                                                   uint32_t partial_stride, const EncScratch *scratch,
                                                                   CoinTables ct) {
    using X = HiX<M>;
    __shared__ float lds[X::LDS_FLOATS];
    __shared__ double red[X::THREADS / 64];
    __shared__ float qtab[16];                                   // centroids; published by the first barrier of the exchange
    __shared__ float gtab[256];                                  // one-byte budgets: centroids and thresholds
    __shared__ RankGuess<8> guess;                               // b = 4 alone: the interval search by a guess and one compare
    constexpr int p = P;
    constexpr int NW = X::RP / 32;
    constexpr bool UNIT = MODE == 0;
    constexpr uint32_t COIN = ONLY > kCoinOnly && ONLY <= kCoinOnly + 3u ? ONLY - kCoinOnly : 0u;        // its k
    constexpr bool SHARED = (ONLY == 0u || COIN) && (MODE == 1 || MODE == 2);
    const uint32_t c = blockIdx.y;
    const uint32_t tile0 = xcd_local_tile<16 / TPW>() * TPW;
    const uint32_t col = threadIdx.x & 31u, g = threadIdx.x >> 5;
    uint32_t rows_written = (uint32_t)((d + (1u << p) - 1) >> p);
    if (BLK) rows_written = (rows_written + kBlockRows - 1u) / kBlockRows * kBlockRows;      // whole blocks of rows are written
    const rsrc_t rt = make_rsrc(T + ((size_t)c << log2D), rows_written << (p + 2));
    uint32_t *payload = reinterpret_cast<uint32_t *>(static_cast<char *>(B.msg[c]) + EDEN_HEADER_BYTES);
    const uint32_t b_q8 = ONLY && !COIN ? ONLY : B.b_q8[c];
    const EncScratch *sc = &scratch[c];
    // stage-1 rows: g + RL r.  Byte offset of (row, column) inside the slot = a per-thread part + a part that is the same for
    // the whole workgroup (row_off(r)) + the tile's column block
    constexpr uint32_t RLB = X::RL >= kBlockRows ? X::RL / kBlockRows : 1u;
    const uint32_t off1 = !BLK ? ((g << p) + col) * 4u
                               : X::RL >= kBlockRows ? (((g >> kBlockRowBits) << (p + kBlockRowBits)) + ((g & (kBlockRows - 1u)) << 5) + col) * 4u
                                                     : ((g << 5) + col) * 4u;
    auto row_off = [](int r) -> uint32_t {                       // r is a compile-time constant after unrolling
        if (!BLK) return ((uint32_t)X::RL * (uint32_t)r) << (p + 2);
        if (X::RL >= kBlockRows) return (RLB * (uint32_t)r) << (p + kBlockRowBits + 2);
        const uint32_t row = (uint32_t)X::RL * (uint32_t)r;      // RL = 2: rows g + 2 r, g = 0, 1
        return ((row >> kBlockRowBits) << (p + kBlockRowBits + 2)) + ((row & (kBlockRows - 1u)) << 7);
    };
    auto tile_off = [](uint32_t tile) -> uint32_t {              // (two-pass plans: the tile index is the column block)
        return BLK ? tile << (7 + kBlockRowBits) : (uint32_t)hix_base<M>(tile, p) * 4u;
    };
    const uint64_t mixkey = stream_key(seed, kStreamMix, B.client[c]);
    if constexpr (MODE == 3) fill_rank_guess<8>(guess, sc, threadIdx.x);     // published, like qtab, by the first barrier of the exchange
    if (!UNIT) {
        if (threadIdx.x < 16u) qtab[threadIdx.x] = sc->qpos[threadIdx.x];       // qpos and qpos2 are one run
        if (!COIN && byte_budget(b_q8)) {                        // centroids, then thresholds: one run of 256 floats
            const float *byte_tab = sc->grid_c;
            for (uint32_t i = threadIdx.x; i < 256u; i += X::THREADS) gtab[i] = byte_tab[i];
        }
    }
    float ip = 0.0f;
    uint32_t held[TPW][X::PH][NW];
    float v[64];
    {
        const uint32_t b0 = tile_off(tile0);
#pragma unroll
        for (int r = 0; r < 64; ++r) v[r] = buf_load(rt, off1, b0 + row_off(r));
    }
#pragma unroll
    for (int k = 0; k < TPW; ++k) {
        const uint64_t base = hix_base<M>(tile0 + k, p);
        const uint32_t next_off = tile_off(tile0 + k + 1);
        fwht_regs<64>(v);
        float out[X::RP];
        // The instances that serve several budgets hold one copy of the code behind the exchange for both halves, fed from `cur`.  With
        // two copies (75 KB in MODE 1, more than the instruction cache) or with the halves told apart by conditions (MODE 2, 100 KB in
        // one copy) they spilled 32 to 48 registers, now 0 and 6 to 17, and were slower in halves than in one piece at M = 7..9.  (One
        // sender of 7,000,001, b = 8: 48.8 -> 40.0 us, in one piece 41.9; 8 of 4,000,037 with b = 1, 3, 1.5, 8: 121 -> 98, 106; one of
        // 10^8 at 2.7 bits: 617 -> 547, in three passes 555.)  The trip count is hidden from the compiler, which would otherwise unroll
        // by threading jumps.
        int halves = X::PH;
        float cur[SHARED ? X::RP : 1];
        if constexpr (SHARED) {
            asm volatile("" : "+s"(halves));
#pragma unroll
            for (int r = 0; r < X::RP; ++r) cur[r] = v[r];
        }
#pragma unroll SHARED ? 1 : X::PH
        for (int ph = 0; ph < halves; ++ph) {
            if constexpr (SHARED) {
                hix_exchange_write<M, 0>(cur, lds);
#pragma unroll
                for (int r = 0; r < X::RP; ++r) cur[r] = v[X::RP + r];
            } else if (ph == 0) hix_exchange_write<M, 0>(v, lds);
            else hix_exchange_write<M, X::PH - 1>(v, lds);
            if constexpr (TPW > 1) {
                if (k + 1 < TPW) {
#pragma unroll
                    for (int r = ph * X::RP; r < (ph + 1) * X::RP; ++r)
                        v[r] = buf_load(rt, off1, next_off + row_off(r));
                }
            }
            hix_exchange_read<M, !UNIT>(lds, out);               // every sender b <= 1: the last stage is fused into the signs
            if (UNIT) hix_sign_words_pairs<M>(out, ip, held[k][ph]);
            else if (MODE == 3) {
                if (sc->guess_up != 1.0f) {
#pragma unroll
                    for (int s2 = 0; s2 < X::RP; ++s2) out[s2] = scale_for_guess(out[s2], sc->guess_up);
                }
                hix_quantize_pack<M, P, 4, 0, true>(out, ph, sc, qtab, payload, reinterpret_cast<uint16_t *>(payload), mixkey, base, ip, ct,
                                                 c, log2D, payload, &guess);
            } else if (SHARED && !COIN && b_q8 <= 256u) {
                uint32_t words[NW];
                hix_sign_words<M>(out, ip, words);
#pragma unroll
                for (int w = 0; w < NW; ++w) {                   // (ph is a variable here: no index into registers)
                    held[k][0][w] = ph == 0 ? words[w] : held[k][0][w];
                    held[k][X::PH - 1][w] = words[w];
                }
            }
            else if (!COIN && byte_budget(b_q8)) {
                // uniform grid (Sec. 4.3) or b = 5..8: one byte per coordinate; a row segment of the tile is 32 bytes
                uint8_t *bytes = (B.codes[c] ? B.codes[c] : reinterpret_cast<uint8_t *>(payload)) + base + col;
                const float inv = sc->grid_inv;
                const uint32_t H = wide_half_levels(b_q8);
                if (grid_q15(b_q8)) {                            // the indices replace the values in their registers
#pragma unroll
                    for (int s2 = 0; s2 < X::RP; ++s2) out[s2] = __uint_as_float(quantize_byte<true>(out[s2], H, inv, gtab, ip));
                } else {
#pragma unroll
                    for (int s2 = 0; s2 < X::RP; ++s2) out[s2] = __uint_as_float(quantize_byte<false>(out[s2], H, inv, gtab, ip));
                }
#pragma unroll
                for (int s2 = 0; s2 < X::RP; ++s2) {             // four lanes' bytes = one dword store
                    const uint32_t quad = quad_bytes(__float_as_uint(out[s2]), col);
                    if (!(col & 3u)) *reinterpret_cast<uint32_t *>(bytes + ((uint64_t)hix_row2<M>(g, ph, s2) << p)) = quad;
                }
            } else {
                int ibits, ik;
                budget_of(b_q8, ibits, ik);
                uint32_t *part_c = payload + payload_a_bytes(1ull << log2D, ibits, 1) / 4;       // second part, if any
                uint16_t *part_b = reinterpret_cast<uint16_t *>(part_c);
                const uint32_t cq = MODE == 2 ? coin_q8(b_q8) : 0u;
                // coin budgets: a staging array for the pieces of the second part, if the host gave this sender one
                uint32_t *pieces = cq ? reinterpret_cast<uint32_t *>(B.codes[c]) : nullptr;
#define EDEN_HIX_PACK(BITS, MIX) \
    hix_quantize_pack<M, P, BITS, MIX>(out, ph, sc, qtab, payload, part_b, mixkey, base, ip, ct, c, log2D, part_c, nullptr, pieces)
                if constexpr (COIN != 0u)
                    hix_quantize_pack<M, P, (int)COIN, 2, COIN == 2u>(out, ph, sc, qtab, payload, part_b, mixkey, base, ip, ct, c, log2D, part_c, nullptr, pieces);
                else if (cq && ibits == 1) EDEN_HIX_PACK(1, 2);
                else if (cq && ibits == 2) EDEN_HIX_PACK(2, 2);
                else if (cq) EDEN_HIX_PACK(3, 2);
                else if (MODE == 2 && b_q8 == 384u) EDEN_HIX_PACK(1, 1);
                else if (MODE == 2 && b_q8 == 640u) EDEN_HIX_PACK(2, 1);
                else if (MODE == 2 && b_q8 == 896u) EDEN_HIX_PACK(3, 1);
                else if (ONLY == 512u) hix_quantize_pack<M, P, 2, 0, true>(out, ph, sc, qtab, payload, part_b, mixkey, base, ip, ct, c, log2D, part_c);
                else if (b_q8 == 512u) EDEN_HIX_PACK(2, 0);
                else if (b_q8 == 768u) EDEN_HIX_PACK(3, 0);
                else EDEN_HIX_PACK(4, 0);
#undef EDEN_HIX_PACK
            }
        }
    }
    if (UNIT || (MODE != 3 && !COIN && b_q8 <= 256u)) {
        // tile0 is a multiple of TPW: the TPW words of a row are neighbours, aligned to their common size
        const uint64_t base0 = hix_base<M>(tile0, p);
        const uint32_t word0 = (uint32_t)(base0 >> 5);
        const uint64_t subkey = stream_key(seed, kStreamSubsample, B.client[c]);
#pragma unroll
        for (int ph = 0; ph < X::PH; ++ph) {
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const uint32_t row = hix_word_row<M>(ph, w);
                const uint32_t word = word0 + (row << (p - 5));
                uint32_t o[TPW];
                if (b_q8 == 256u) {
#pragma unroll
                    for (int k = 0; k < TPW; ++k) o[k] = held[k][ph][w];
                    typename WordVec<TPW>::type pack;
                    __builtin_memcpy(&pack, o, sizeof(pack));
                    *reinterpret_cast<typename WordVec<TPW>::type *>(payload + word) = pack;
                } else {
                    // b = 1/2 (Sec. 4.1): of each pair (2k, 2k+1) send the coordinate chosen by the sub-sampling
                    // stream; 64 pairs per hash word = 128 coordinates = four neighbouring row segments
                    const uint64_t first = base0 + ((uint64_t)row << p);
                    const uint64_t hw = hash_word(subkey, first >> 7) >> (16u * (uint32_t)((first >> 5) & 3u));
                    uint16_t *half = reinterpret_cast<uint16_t *>(payload) + word;
#pragma unroll
                    for (int k = 0; k < TPW; ++k) {
                        const uint32_t off = (uint32_t)(hw >> (16 * k)) & 0xFFFFu;
                        const uint32_t ev = even_bits(held[k][ph][w]), od = even_bits(held[k][ph][w] >> 1);
                        o[k] = (ev & ~off) | (od & off);
                    }
                    if constexpr (TPW == 1) half[0] = (uint16_t)o[0];
                    else if constexpr (TPW == 2) *reinterpret_cast<uint32_t *>(half) = o[0] | (o[1] << 16);
                    else *reinterpret_cast<uint2 *>(half) = make_uint2(o[0] | (o[1] << 16), o[2] | (o[3] << 16));
                }
            }
        }
    }
    const double ip_sum = MODE == 3 ? unscale_sum(ip, sc->guess_up) : (double)ip;
    const double block_total = block_sum<X::THREADS>(ip_sum, red);
    if (threadIdx.x == 0) partials[(size_t)c * partial_stride + blockIdx.x] = block_total;
}

// Middle pass of the one-byte budgets at D >= 2^25 (bits 14 .. 14+M-1), in place on the workspace (tiles are disjoint).  Elements at or above
// `load_elems` were not written by the pass before (encode: zero padding) and read as zero; elements at or above
// `store_elems` are not read by the pass after (decode: they end in the padding) and are not written.  A tile
// that lies wholly beyond either bound has nothing to do.
// TPW neighbouring column blocks per workgroup: the loads of the next one are issued into the registers that each
// half of the exchange has just written to LDS (see k_enc_hix_last).
template <int M, int TPW>
__global__ __launch_bounds__(HiX<M>::THREADS) void k_hix_mid(float *T, int log2D, uint64_t load_elems, uint64_t store_elems) {
    using X = HiX<M>;
    __shared__ float lds[X::LDS_FLOATS];
    constexpr int p = 14;
    const uint32_t tile0 = blockIdx.x * TPW;                     // the TPW tiles lie in the same 2^(p+M) block
    const uint64_t base0 = hix_base<M>(tile0, p);
    const uint64_t block_start = base0 >> (p + M) << (p + M);
    if (block_start >= load_elems || block_start >= store_elems) return;     // same decision in the whole workgroup
    const uint32_t col = threadIdx.x & 31u, g = threadIdx.x >> 5;
    const rsrc_t rl = make_rsrc(T + ((size_t)blockIdx.y << log2D), (uint32_t)(load_elems * 4));
    const rsrc_t rs = make_rsrc(T + ((size_t)blockIdx.y << log2D), (uint32_t)(store_elems * 4));
    const uint32_t off1 = ((g << p) + col) * 4u;
    const uint32_t off2 = (((g * X::RHL * X::RL) << p) + col) * 4u;
    float v[64];
#pragma unroll
    for (int r = 0; r < 64; ++r) v[r] = buf_load(rl, off1, (uint32_t)base0 * 4u + (((uint32_t)X::RL * r) << (p + 2)));
#pragma unroll
    for (int k = 0; k < TPW; ++k) {
        const uint32_t base_off = (uint32_t)hix_base<M>(tile0 + k, p) * 4u;
        const uint32_t next_off = (uint32_t)hix_base<M>(tile0 + k + 1, p) * 4u;
        fwht_regs<64>(v);
        float out[X::RP];
#pragma unroll
        for (int ph = 0; ph < X::PH; ++ph) {
            if (ph == 0) hix_exchange_write<M, 0>(v, lds);
            else hix_exchange_write<M, X::PH - 1>(v, lds);
            if (k + 1 < TPW) {
#pragma unroll
                for (int r = ph * X::RP; r < (ph + 1) * X::RP; ++r)
                    v[r] = buf_load(rl, off1, next_off + (((uint32_t)X::RL * r) << (p + 2)));
            }
            hix_exchange_read<M>(lds, out);
#pragma unroll
            for (int s = 0; s < X::RP; ++s) buf_store(rs, off2, base_off + (hix_row2<M>(0, ph, s) << (p + 2)), out[s]);
        }
    }
}

uint32_t launch_enc_hix_last(int M, int P, int blocked, const EncBatch &B, uint32_t n, uint64_t d, int log2D, uint64_t seed, const float *T,
                             double *partials, uint32_t partial_stride, const EncScratch *scratch, const CoinTables &ct,
                             hipStream_t st) {
    const uint32_t tiles = hix_tiles(M, log2D);                  // 2^(P-5) column blocks
    bool unit = true, mixed = false, four = true;                // every sender b <= 1; some sender b = k + 1/2; every sender b = 4
    for (uint32_t c = 0; c < n; ++c) {
        unit = unit && B.b_q8[c] <= 256u;
        mixed = mixed || budget_two_tables(B.b_q8[c]);
        four = four && B.b_q8[c] == 1024u;
    }
#define EDEN_ENC_HIX_LAST(TPW, MODE)                                                                                          \
    if (blocked) {                                                                                                            \
        EDEN_HIX_SWITCH(M, P, hipLaunchKernelGGL(HIP_KERNEL_NAME(k_enc_hix_last<MM, PP, TPW, MODE, true>), grid, dim3(HiX<MM>::THREADS), \
                                              0, st, B, d, log2D, seed, T, partials, partial_stride, scratch, ct))            \
    } else {                                                                                                                  \
        EDEN_HIX_SWITCH(M, P, hipLaunchKernelGGL(HIP_KERNEL_NAME(k_enc_hix_last<MM, PP, TPW, MODE, (PP > 14)>), grid, dim3(HiX<MM>::THREADS), \
                                              0, st, B, d, log2D, seed, T, partials, partial_stride, scratch, ct))            \
    }
    if (unit && tiles % 256u == 0) {                             // two neighbouring tiles per workgroup (with the blocked
        dim3 grid(tiles / 2, n);                                 // workspace: 148 us against 158 with four and 160 with one)
        EDEN_ENC_HIX_LAST(2, 0);
        return grid.x;
    }
    // every other launch: one tile per workgroup (with the blocked workspace two tiles per workgroup are slower at every size:
    // 16 senders at D = 2^23, 0.151 -> 0.142 ms at b = 2, 0.34 -> 0.18 ms at b = 1.5, 0.255 -> 0.144 ms for the b = 4 instance)
    dim3 grid(tiles, n);
    // One budget for all senders: b = 2, 3 and the budgets k + 1/2 have instances that hold only their branch (16 senders at D = 2^24,
    // against shared instances that still spilled: 0.40 -> 0.24 ms at b = 1.5, 0.277 -> 0.253 ms at b = 3; b = 2: see hix_quantize_pack).
    uint32_t same = B.b_q8[0];
    for (uint32_t c = 1; c < n; ++c) if (B.b_q8[c] != same) same = 0;
    // Coin budgets of one floor: the halves share their code as in the shared instance (two copies spilled 42 registers, 150 us); the two
    // bits of a floor of 2 go through lane transposes, the bit of a coin through ballots.  Encode, shared instance -> this: 8 senders of
    // 4,000,037 at 2.7 bits 129 -> 125 us, of 2,000,000 at 3.3 83.4 -> 81.0; 16 of 11,173,962 at 2.7 771 -> 759.
#define EDEN_ENC_HIX_ONLY(MODE, ONLY)                                                                                         \
    if (blocked) {                                                                                                            \
        EDEN_HIX_SWITCH(M, P, hipLaunchKernelGGL(HIP_KERNEL_NAME(k_enc_hix_last<MM, PP, 1, MODE, true, ONLY>), grid, dim3(HiX<MM>::THREADS), \
                                              0, st, B, d, log2D, seed, T, partials, partial_stride, scratch, ct))            \
    } else {                                                                                                                  \
        EDEN_HIX_SWITCH(M, P, hipLaunchKernelGGL(HIP_KERNEL_NAME(k_enc_hix_last<MM, PP, 1, MODE, (PP > 14), ONLY>), grid, dim3(HiX<MM>::THREADS), \
                                              0, st, B, d, log2D, seed, T, partials, partial_stride, scratch, ct))            \
    }
    if (four) { EDEN_ENC_HIX_LAST(1, 3); }
    else if (same == 512u) { EDEN_ENC_HIX_ONLY(1, 512u); }
    else if (same == 768u) { EDEN_ENC_HIX_ONLY(1, 768u); }
    else if (same == 384u) { EDEN_ENC_HIX_ONLY(2, 384u); }
    else if (same == 640u) { EDEN_ENC_HIX_ONLY(2, 640u); }
    else if (same == 896u) { EDEN_ENC_HIX_ONLY(2, 896u); }
    else if (const uint32_t cb = coin_floor_of_all(B.b_q8, n)) {
        if (cb == 1u) { EDEN_ENC_HIX_ONLY(2, kCoinOnly + 1u); } else if (cb == 2u) { EDEN_ENC_HIX_ONLY(2, kCoinOnly + 2u); } else { EDEN_ENC_HIX_ONLY(2, kCoinOnly + 3u); }
    }
    else if (mixed) { EDEN_ENC_HIX_LAST(1, 2); } else { EDEN_ENC_HIX_LAST(1, 1); }
#undef EDEN_ENC_HIX_ONLY
#undef EDEN_ENC_HIX_LAST
    return grid.x;
}
void launch_hix_mid(int M, uint32_t n, float *T, int log2D, uint64_t load_elems, uint64_t store_elems, hipStream_t st) {
    dim3 grid(hix_tiles(M, log2D) / 2, n);                       // 2^(p-5) = 512 tiles per block of 2^(p+M): pairs never straddle
#define EDEN_HIX_MID(M) \
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_hix_mid<M, 2>), grid, dim3(HiX<M>::THREADS), 0, st, T, log2D, load_elems, store_elems)
    if (M == 8) EDEN_HIX_MID(8); else if (M == 9) EDEN_HIX_MID(9); else EDEN_HIX_MID(10);
#undef EDEN_HIX_MID
}

}  // namespace eden
