// HIP kernels of the EDEN hot path for gfx950 (MI355X): wave-tile passes, scalars and headers, helpers.  Wave64 throughout.
//
// The rotation R x = D^-1/2 H (s o x) (Sec. 2.2.1; Sec. 5: randomized Hadamard transform) is computed
// unnormalised, u = H (s o x), with the D^-1/2 folded into scalars.  The index bits of the padded
// dimension D = 2^L are split into groups; one kernel ("pass") transforms one group:
//
//   lo pass   bits 0..11   a workgroup of four waves owns 4096 consecutive coordinates, 16 values per thread (eden_lo.h); the
//                          encoder's is in eden_kernels_lo14.hip.
//   hi pass   bits p..p+M-1 (M <= 6): one wave owns 2^M rows of 64 consecutive coordinates at stride 2^p;
//                          every lane keeps one column in registers; no LDS at all.
//
// Encode runs the lo pass first (it reads x, applies the signs and sums |x|^2, and only touches the tiles
// that hold part of x) and the hi passes after it, the last one fused with quantization, <R(x),Q> and bit
// packing (Sec. 2.2.1, 2.3).  Decode runs the hi passes first, the first one fused with unpacking and centroid
// lookup (Sec. 2.2.2, 4.2), and the lo pass last: it applies the signs and sums the senders in registers before
// touching the accumulator once.  D <= 4096 is handled by eden_kernels_small.hip.
#include "eden_device.h"
#include "eden_kernels.h"
#include "eden_lo.h"

namespace eden {

// ------------------------------------------------------------------------------------------------
// hi passes
template <int M>
__device__ inline void hi_tile_origin(uint32_t tile, int p, uint64_t &base) {
    const uint32_t cb_bits = (uint32_t)p - 6u;                  // 2^(p-6) blocks of 64 columns
    const uint32_t colblock = tile & ((1u << cb_bits) - 1u);
    const uint32_t upper = tile >> cb_bits;
    base = ((uint64_t)upper << (p + M)) | ((uint64_t)colblock << 6);
}

// The K-bit indices of one row segment of 64 consecutive coordinates, given as bit planes (plane[b][0/1]: bit b of
// the indices of coordinates 0..31 / 32..63), written as the 2K payload words that start at coordinate `first`
// (a multiple of 64): index i occupies bits K i .. K i + K - 1 of the little-endian bit string.
template <int K>
__device__ inline void store_row_planes(const uint32_t (&plane)[4][2], uint32_t *payload, uint64_t first) {
    if constexpr (K == 1) {
        *reinterpret_cast<uint2 *>(payload + (first >> 5)) = make_uint2(plane[0][0], plane[0][1]);
    } else if constexpr (K == 2) {
        uint32_t o[4];                                           // word k: coordinates 16 k .. 16 k + 15
#pragma unroll
        for (int k = 0; k < 4; ++k)
            o[k] = spread2(plane[0][k >> 1] >> (16 * (k & 1))) | (spread2(plane[1][k >> 1] >> (16 * (k & 1))) << 1);
        *reinterpret_cast<uint4 *>(payload + (first >> 4)) = make_uint4(o[0], o[1], o[2], o[3]);
    } else if constexpr (K == 3) {
        uint32_t lo[3], hi[3];                                   // 64 coordinates x 3 bits = 6 words
        pack3_planes(plane[0][0], plane[1][0], plane[2][0], lo);
        pack3_planes(plane[0][1], plane[1][1], plane[2][1], hi);
        uint2 *dst = reinterpret_cast<uint2 *>(payload + (first >> 6) * 6u);
        dst[0] = make_uint2(lo[0], lo[1]);
        dst[1] = make_uint2(lo[2], hi[0]);
        dst[2] = make_uint2(hi[1], hi[2]);
    } else {
        uint32_t o[8];                                           // word k: coordinates 8 k .. 8 k + 7
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            o[k] = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) o[k] |= spread4(plane[b][k >> 2] >> (8 * (k & 3))) << b;
        }
        uint4 *dst = reinterpret_cast<uint4 *>(payload + (first >> 3));
        dst[0] = make_uint4(o[0], o[1], o[2], o[3]);
        dst[1] = make_uint4(o[4], o[5], o[6], o[7]);
    }
}

// b = 2 and 4 (R >= 32 / K rows): instead of the ballots a lane collects the indices of 32 / K rows of its column in a word, and the
// lanes of as many neighbouring columns transpose their words: each then holds one payload word of one row.  `base`: first
// coordinate of the tile.  With the ballots (four v_writelane and two compares a value at b = 2, eight and four at b = 4) the pass was half
// packing: encode of 10 senders of 2^20, b = 2 33.0 -> 31.4 us, b = 4 40.5 -> 34.7 (with the search by a guess; 38.4 without), one of them
// 19.3 -> 17.0, 32 with 1/2, 1, 2 and 4 bits 82.3 -> 77.6.  From 32 rows on: below, the launch is too short for it to show (16 of 30,000,
// b = 4 14.6 us, with the guess, which takes a barrier more, 15.5).
template <int R, int K>
__device__ inline void hi_quantize_transpose(const float (&v)[R], const EncScratch &es, const RankGuess<8> &guess, uint64_t base, int p,
                                             uint32_t *payload, float &ip) {
    constexpr int PER = 32 / K;
    static_assert((K == 2 || K == 4) && R >= PER, "whole words");
    const uint32_t lane = lane_id(), j = lane & (uint32_t)(PER - 1), q = lane / (uint32_t)PER;
    const float thr1 = uniform(es.thr[1]), q0 = uniform(es.qpos[0]), q1 = uniform(es.qpos[1]);
    static_for<R / PER>([&](auto B) {
        constexpr int first = decltype(B)::value * PER;
        uint32_t items;
        if constexpr (K == 2) {
            items = quantize_two_bits(&v[first], thr1, q0, q1, ip);
        } else {
            uint32_t at[PER];
            quantize_guess<8>(&v[first], guess, &es, at, ip);
            items = pack_guesses(at);
        }
        items = transpose_items<K>(items, lane);
        payload[((base + ((uint64_t)(first + j) << p)) >> (K == 2 ? 4 : 3)) + q] = items;
    });
}

// Quantizes the R rows of a wave tile (register r = row r, one column per lane) and packs them.  K: bits of every
// index in the first part of the payload.  MIX = 1 (b = K + 1/2, Sec. 4.1): the coordinate of every pair that the MIX
// stream selects is quantized with I_{K+1}; the top bit of its index goes to the second part, one bit per pair.
// MIX = 2 (coin budgets, Sec. 4.1): the coordinates with a coin (`my_mask`: the coins of this lane's row) are quantized
// with I_{K+1}; their top bits go to the second part in coordinate order, the row's first one at bit `my_off`.
// `my_row`: first coordinate of the row that this lane (< R) finishes.
template <int R, int K, int MIX>
__device__ inline void hi_quantize_pack(const float (&v)[R], const Thresholds &th, const float *qtab, uint64_t mixkey,
                                        uint64_t my_row, uint32_t *part_a, uint32_t *part_b, float &ip,
                                        uint64_t my_mask = 0, uint32_t my_off = 0) {
    const uint32_t lane = lane_id();
    uint32_t plane[4][2], top[2] = {0u, 0u};
#pragma unroll
    for (int b = 0; b < 4; ++b) plane[b][0] = plane[b][1] = 0;
    // the coordinates of this lane's row with I_{K+1}; 64 pairs per hash word = 128 coordinates, 32 of them in a row segment
    uint64_t chosen = my_mask;
    if constexpr (MIX == 1) {
        const uint32_t offs = (uint32_t)(hash_word(mixkey, my_row >> 7) >> (32u * (uint32_t)((my_row >> 6) & 1u)));
        chosen = (uint64_t)chosen_of_pairs(offs >> 16) << 32 | chosen_of_pairs(offs);
    }
    constexpr int NA = R < 4 ? R : 4;
    uint32_t at[NA];                                             // where the centroids of a few values lie in qtab
    static_for<R>([&](auto RR) {
        constexpr int r = decltype(RR)::value;
        uint64_t bit[K];                                         // lane masks of the index's low bits
        if constexpr (MIX != 0) {
            uint64_t high;
            at[r % NA] = quantize_two_tables<K>(v[r], wave_read64(chosen, r), th, bit, high);
            top[0] = put_lane<r>(lo32(high), top[0]);
            top[1] = put_lane<r>(hi32(high), top[1]);
        } else {
            at[r % NA] = quantize_one_table<K>(v[r], th, bit);
        }
#pragma unroll
        for (int b = 0; b < K; ++b) {
            plane[b][0] = put_lane<r>(lo32(bit[b]), plane[b][0]);
            plane[b][1] = put_lane<r>(hi32(bit[b]), plane[b][1]);
        }
        if constexpr (r % NA == NA - 1) add_centroids<NA>(&v[r - (NA - 1)], at, qtab, ip);
    });
    if (lane < R) {
        store_row_planes<K>(plane, part_a, my_row);
        if constexpr (MIX == 1)                                  // only the chosen coordinate of a pair can have the bit
            part_b[my_row >> 6] = even_bits(top[0] | (top[0] >> 1)) | (even_bits(top[1] | (top[1] >> 1)) << 16);
        if constexpr (MIX == 2) {                                // only a coordinate with a coin can have the bit
            const uint64_t top64 = (uint64_t)top[0] | ((uint64_t)top[1] << 32);
            or_bits(part_b, my_off, compress_bits(top64, my_mask), (uint32_t)__popcll(my_mask));
        }
    }
}

// Encode, last pass in wave tiles: T -> payload.  Index bits p .. p+M-1 of H, then quantization to the
// Lloyd-Max intervals (Sec. 2.2.1, Sec. 3), sum_i u_i q_i for the scale (Sec. 2.3), sub-sampling for b = 1/2
// (Sec. 4.1), packing.  Register r is row r of the tile = 64 consecutive coordinates across the lanes, so a
// ballot of one index bit is 64 payload bits of that row; lane r collects the ballots of row r and packs them.
// Workspace elements at or above `valid_elems` were not written by the earlier passes because they are
// zero (transformed zero padding): the buffer bounds return 0 for them.
// ONLY != 0: every sender of the launch has this budget (1, 2 or 4 bits); the instance then holds that one branch.
template <int M, uint32_t ONLY = 0>
__global__ __launch_bounds__(256) void k_enc_hi_last(EncBatch B, uint64_t valid_elems, int log2D, int p, uint64_t seed,
                                                     const float *T, double *partials, uint32_t partial_stride,
                                                     CoinTables ct, EncTail tail) {
    constexpr int R = 1 << M;
    __shared__ double red[4];
    __shared__ uint32_t last_flag;
    __shared__ EncScratch es;
    constexpr bool GUESS = M >= 5 && (ONLY == 0u || ONLY == 1024u);
    __shared__ RankGuess<8> guess;                               // b = 4: the interval search by a guess and one compare
    const uint32_t c = blockIdx.y;
    const uint32_t lane = lane_id();
    const uint32_t tile = blockIdx.x * 4u + wave_in_block();     // (2^(p-6) tiles: a multiple of 4)
    const uint32_t b_q8 = ONLY ? ONLY : B.b_q8[c];
    float ip = 0.0f;
    EarlyPartials early;
    early.load(tail.part_n2 + (size_t)c * tail.n2_stride, tail.n2_count);
    {
        uint64_t base;
        hi_tile_origin<M>(tile, p, base);
        const rsrc_t rt = make_rsrc(T + ((size_t)c << log2D), (uint32_t)(valid_elems * 4));
        const uint32_t lane_off = lane * 4u, base_off = (uint32_t)base * 4u;
        float v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = buf_load(rt, lane_off, base_off + ((uint32_t)r << (p + 2)));
        enc_scratch_to_lds(tail, c, b_q8, early, es, red);
        // (the butterflies stand behind the norm's branch: in front of it the compiler moves half of them into it, and holds 138 registers)
        const bool valid = enc_valid_norm(es.n2);
        if (valid) fwht_regs<R>(v);
        if constexpr (GUESS) {
            if (b_q8 == 1024u) {
                fill_rank_guess<8>(guess, &es, threadIdx.x);
                if (es.guess_up != 1.0f) {
#pragma unroll
                    for (int r = 0; r < R; ++r) v[r] = scale_for_guess(v[r], es.guess_up);
                }
                __syncthreads();
            }
        }
        uint32_t *payload = reinterpret_cast<uint32_t *>(static_cast<char *>(B.msg[c]) + EDEN_HEADER_BYTES);
        const uint64_t my_row = base + ((uint64_t)(lane & (R - 1)) << p);       // lane r < R finishes row r
        if (!valid) {
            if (lane < R) zero_payload_row(B, c, log2D, my_row);
        } else if (b_q8 <= 256u) {
            // I_1 = {(-inf,0],[0,inf)}: the index is the sign; <R(x),Q> = q_1 sum |u| / sqrt(D)
            float sa = 0.0f;
#pragma unroll
            for (int r = 0; r < R; ++r) sa += fabsf(v[r]);
            ip = sa * kQ1;
            uint32_t wlo = 0, whi = 0;
            static_for<R>([&](auto RR) {
                constexpr int r = decltype(RR)::value;
                const uint64_t m = __ballot((__float_as_uint(v[r]) >> 31) == 0u);    // index 1 = non-negative
                wlo = put_lane<r>(lo32(m), wlo);
                whi = put_lane<r>(hi32(m), whi);
            });
            if (lane < R) {
                if (b_q8 == 256u) {
                    *reinterpret_cast<uint2 *>(payload + (my_row >> 5)) = make_uint2(wlo, whi);
                } else {
                    // b = 1/2: of each pair (2g, 2g+1) send the coordinate chosen by the sub-sampling stream;
                    // 64 pairs per hash word = 128 coordinates, a row segment uses 32 of them
                    const uint64_t key = stream_key(seed, kStreamSubsample, B.client[c]);
                    const uint32_t off = (uint32_t)(hash_word(key, my_row >> 7) >> (32u * (uint32_t)((my_row >> 6) & 1u)));
                    const uint32_t ev = even_bits(wlo) | (even_bits(whi) << 16);
                    const uint32_t od = even_bits(wlo >> 1) | (even_bits(whi >> 1) << 16);
                    payload[my_row >> 6] = (ev & ~off) | (od & off);
                }
            }
        } else {
            const Thresholds sc = uniform_thresholds(es);
            const float *qtab = es.qpos;
            const uint64_t mixkey = stream_key(seed, kStreamMix, B.client[c]);
            uint32_t *part_b = payload + payload_a_bytes(1ull << log2D, (int)(b_q8 >> 8), 1) / 4;
            if (byte_budget(b_q8)) {
                // uniform grid (Sec. 4.3) or b = 5..8: one byte per coordinate; a row of the tile is 64 consecutive bytes
                const float *ctab = es.grid_c;                   // centroids, then thresholds: one run of 256 floats
                const float inv = es.grid_inv;
                uint8_t *bytes = B.codes[c] ? B.codes[c] : reinterpret_cast<uint8_t *>(payload);
                const uint32_t H = wide_half_levels(b_q8);
                if (grid_q15(b_q8)) {                            // the indices replace the values in their registers
#pragma unroll
                    for (int r = 0; r < R; ++r) v[r] = __uint_as_float(quantize_byte<true>(v[r], H, inv, ctab, ip));
                } else {
#pragma unroll
                    for (int r = 0; r < R; ++r) v[r] = __uint_as_float(quantize_byte<false>(v[r], H, inv, ctab, ip));
                }
#pragma unroll
                for (int r = 0; r < R; ++r) {                    // four lanes' bytes = one dword store
                    const uint32_t quad = quad_bytes(__float_as_uint(v[r]), lane);
                    if (!(lane & 3u)) *reinterpret_cast<uint32_t *>(bytes + base + ((uint64_t)r << p) + lane) = quad;
                }
            } else if (const uint32_t cq = coin_q8(b_q8)) {
                // the coins of this lane's row, and where the row's first extra bit goes in the second part
                const uint32_t w = (uint32_t)(my_row >> 6);
                const uint64_t my_mask = coin_mask_of(ct, c, log2D, w);
                const uint32_t my_off = coins_before(ct, c, log2D, w);
                uint32_t *part_c = payload + payload_a_bytes(1ull << log2D, (int)(cq >> 8), 1) / 4;
                if ((cq >> 8) == 1u) hi_quantize_pack<R, 1, 2>(v, sc, qtab, mixkey, my_row, payload, part_c, ip, my_mask, my_off);
                else if ((cq >> 8) == 2u) hi_quantize_pack<R, 2, 2>(v, sc, qtab, mixkey, my_row, payload, part_c, ip, my_mask, my_off);
                else hi_quantize_pack<R, 3, 2>(v, sc, qtab, mixkey, my_row, payload, part_c, ip, my_mask, my_off);
            } else
            switch (b_q8) {
                case 384u: hi_quantize_pack<R, 1, 1>(v, sc, qtab, mixkey, my_row, payload, part_b, ip); break;
                case 512u:
                    if constexpr (M >= 5) hi_quantize_transpose<R, 2>(v, es, guess, base, p, payload, ip);
                    else hi_quantize_pack<R, 2, 0>(v, sc, qtab, mixkey, my_row, payload, part_b, ip);
                    break;
                case 640u: hi_quantize_pack<R, 2, 1>(v, sc, qtab, mixkey, my_row, payload, part_b, ip); break;
                case 768u: hi_quantize_pack<R, 3, 0>(v, sc, qtab, mixkey, my_row, payload, part_b, ip); break;
                case 896u: hi_quantize_pack<R, 3, 1>(v, sc, qtab, mixkey, my_row, payload, part_b, ip); break;
                default:
                    if constexpr (GUESS) hi_quantize_transpose<R, 4>(v, es, guess, base, p, payload, ip);
                    else hi_quantize_pack<R, 4, 0>(v, sc, qtab, mixkey, my_row, payload, part_b, ip);
                    break;
            }
        }
    }
    const double ip_sum = GUESS && b_q8 == 1024u ? unscale_sum(ip, es.guess_up) : (double)ip;
    const double block_total = block_sum<256>(ip_sum, red);
    enc_last_tail<256>(tail, B, c, log2D, seed, es.n2, block_total, partials + (size_t)c * partial_stride, &last_flag);
}

// One workgroup per sender: sums the per-workgroup partials of |x|^2 in index order (deterministic)
// and scales the thresholds.  Runs between the first pass and the quantizing pass because eta
// depends on the whole vector (Sec. 2.2.1).
__device__ inline void enc_norm(const EncBatch &B, uint32_t c, const double *partials, uint32_t partial_stride, uint32_t nparts,
                                EncScratch *scratch, const DevTables *tab, double *red) {
    const double n2 = ordered_sum<256>(partials + (size_t)c * partial_stride, nparts, red);
    fill_enc_scratch(&scratch[c], n2, B.b_q8[c], tab, threadIdx.x);
    fill_byte_tables(&scratch[c], B.b_q8[c], n2, tab, threadIdx.x);
}
__global__ __launch_bounds__(256) void k_enc_norm(EncBatch B, const double *partials, uint32_t partial_stride,
                                                  uint32_t nparts, EncScratch *scratch, const DevTables *tab) {
    __shared__ double red[4];
    enc_norm(B, blockIdx.x, partials, partial_stride, nparts, scratch, tab, red);
}

// Decode, first pass in wave tiles (Sec. 2.2.2, 4.2): unpack, centroid lookup times S/(p sqrt D) (or the unit
// pattern +-1 when the workspace of a b <= 1 sender is fp16), zero for coordinates that were not sampled or
// whose packet was lost, then index bits p .. p+M-1 of H.  Every (tile, sender) pair is independent.
// Elements at or above `keep_elems` are never read by the later passes (they end in the padding): the buffer
// bounds drop their stores.
// (Five waves per SIMD are requested: the budgets with two loads per value would otherwise set the register count
// for all of them; measured 0.057 against 0.073 ms on 32 senders at D = 2^20.)
// ONLY != 0: every sender of the launch has this budget (1, 2 or 4 bits, indices in the payload); the instance then holds
// that one branch (the shared one spills at its 96 registers).  kSimple: every sender has 1/2, 1, 2 or 4 bits, in any mix; without
// the branches of the others four waves per SIMD do (32 senders of 2^20, those budgets mixed: 53.9 -> 45.6 us; the encoder's
// last pass gained nothing from such an instance).
constexpr uint32_t kSimple = 1u;
__host__ __device__ inline bool simple_budget(uint32_t b_q8) { return b_q8 == 128u || b_q8 == 256u || b_q8 == 512u || b_q8 == 1024u; }
// With either, one form of load serves all rows and budgets: the words are on their way while the header is checked and the table made
// (mean of 32 senders of 2^20, those budgets mixed, 75.6 -> 63.9 us; of 10 with b = 1 29.8 -> 29.1, with b = 2 the same).
template <int M, uint32_t ONLY = 0>
__global__ __launch_bounds__(256, ONLY == kSimple ? 4 : 5) void k_dec_hi_first(DecBatch B, uint64_t keep_elems, int log2D, int p, uint64_t seed,
                                                      DecPrepareArgs prep, int narrow, float *T, CoinTables ct) {
    constexpr int R = 1 << M;
    __shared__ DecScratch ds;
    __shared__ float table[4][32];
    __shared__ float gtabs[4][kGridMax + 1];                     // uniform grid: dequantized centres of mass
    const uint32_t c = blockIdx.y;
    const uint32_t lane = lane_id(), wv = wave_in_block();
    const uint32_t tile = blockIdx.x * 4u + wv;
    constexpr bool SIMPLE = ONLY == kSimple, EARLY = ONLY != 0u;
    const uint32_t b_q8 = ONLY > kSimple ? ONLY : B.b_q8[c];
    uint64_t base;
    hi_tile_origin<M>(tile, p, base);                            // (the grid has exactly as many waves as there are tiles)
    const uint32_t *payload = reinterpret_cast<const uint32_t *>(static_cast<const char *>(B.msg[c]) + EDEN_HEADER_BYTES);
    int bits, k;
    budget_of(b_q8, bits, k);
    const uint32_t payload_bytes = (uint32_t)(((((1ull << log2D) >> (k == 2)) * (uint32_t)bits + 63) >> 6) << 3);
    const uint32_t shift = SIMPLE && k == 2 ? lane >> 1 : (lane * (uint32_t)bits) & 31u;         // EARLY: where a lane's index sits in its word
    float v[R];
    if constexpr (EARLY) {                                       // the words of all rows, on their way while the table is made
        const uint32_t first = SIMPLE && k == 2 ? (uint32_t)(base >> 6) : (uint32_t)((base * (uint32_t)bits) >> 5);
        const uint32_t row = SIMPLE && k == 2 ? 1u << (p - 4) : (uint32_t)bits << (p - 3);       // bytes of payload per row of the strided index
        const uint32_t voff = SIMPLE && k == 2 ? 0u : ((lane * (uint32_t)bits) >> 5) * 4u;
        const rsrc_t rp = make_rsrc(payload + first, payload_bytes - first * 4u);
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rp, (int)voff, (int)((uint32_t)r * row), 0));
        __builtin_amdgcn_sched_barrier(0);
    }
    // Header checks, arrival counts and the dequantization table: every workgroup of a sender does them for itself (a launch of
    // its own took 4 us in front of passes of 5 to 15), the first one for the later passes and the status words too.  The unit
    // pattern of a b <= 1 sender needs none of it here.
    const bool first_wg = blockIdx.x == 0;
    if (wv == 0 && (first_wg || narrow == 0 || b_q8 > 256u))
        dec_prepare_wave(B.msg[c], B.bitmap[c], B.client[c], b_q8, B.hdr_b_q8[c], prep.hdr_d, log2D, prep.seed, prep.tab, &ds,
                         first_wg ? prep.dev_status : nullptr, coin_q8(b_q8) ? ct.total[c] : 0u,
                         first_wg && prep.msg_flags ? prep.msg_flags + c : nullptr);
    __syncthreads();
    if (first_wg)
        for (uint32_t i = threadIdx.x; i < sizeof(DecScratch) / 4; i += 256u)
            reinterpret_cast<uint32_t *>(&prep.scratch[c])[i] = reinterpret_cast<const uint32_t *>(&ds)[i];
    const bool unit = narrow != 0 && b_q8 <= 256u, i16 = narrow == 1 && b_q8 <= 256u;      // narrow == 2: the integers as fp32
    if (lane < 16) table[wv][lane] = (unit && lane == 1) ? 1.0f : ds.deq[lane];
    else if (lane < 32) table[wv][lane] = ds.deq2[lane - 16];
    if (!EARLY && byte_budget(b_q8)) { gtabs[wv][lane] = ds.grid_deq[lane]; gtabs[wv][64 + lane] = ds.grid_deq[64 + lane]; }
    wave_lds_sync();
    const float *tb = table[wv], *tb2 = table[wv] + 16;
    const uint64_t my_row = base + ((uint64_t)(lane & (R - 1)) << p);       // lane r looks after row r
    uint64_t recv = ~0ull;                                       // bit r: the packet of row r arrived
    if (const uint32_t *bm = B.bitmap[c]) {
        const uint32_t pk = (uint32_t)(my_row >> 10);
        recv = __ballot((bm[pk >> 5] >> (pk & 31u)) & 1u);
    }
    if constexpr (EARLY) {
        const float mag = tb[1];
        if (SIMPLE && k == 2) {
            const uint64_t key = stream_key(seed, kStreamSubsample, B.client[c]);
            const uint32_t offs_mine = (uint32_t)(hash_word(key, my_row >> 7) >> (32u * (uint32_t)((base >> 6) & 1u)));
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t offs = __builtin_amdgcn_readlane(offs_mine, r);
                const bool kept = ((offs >> (lane >> 1)) & 1u) == (lane & 1u);
                const uint32_t neg = (~(__float_as_uint(v[r]) >> shift) & 1u) << 31;         // index 0 = negative
                v[r] = kept ? __uint_as_float(__float_as_uint(mag) | neg) : 0.0f;
            }
        } else if (bits == 1) {
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = __uint_as_float(__float_as_uint(mag) | ((~(__float_as_uint(v[r]) >> shift) & 1u) << 31));
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = tb[(__float_as_uint(v[r]) >> shift) & ((1u << bits) - 1u)];
        }
    } else if (b_q8 == 128) {
        // b = 1/2: pair j = i >> 1 carries one bit; coordinate i was sent iff (i & 1) equals the pair's offset bit
        const uint64_t key = stream_key(seed, kStreamSubsample, B.client[c]);
        const uint32_t offs_mine = (uint32_t)(hash_word(key, my_row >> 7) >> (32u * (uint32_t)((base >> 6) & 1u)));
        const rsrc_t rp = make_rsrc(payload + (base >> 6), payload_bytes - (uint32_t)(base >> 6) * 4u);
        const uint32_t mag = __float_as_uint(tb[1]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t w = __builtin_amdgcn_raw_buffer_load_b32(rp, 0, (int)(((uint32_t)r << (p - 6)) * 4u), 0);
            const uint32_t offs = __builtin_amdgcn_readlane(offs_mine, r);
            const bool kept = ((offs >> (lane >> 1)) & 1u) == (lane & 1u);
            const uint32_t neg = (~(w >> (lane >> 1)) & 1u) << 31;          // index 0 = negative
            v[r] = kept ? __uint_as_float(mag | neg) : 0.0f;
        }
    } else if (byte_budget(b_q8)) {
        // one byte per coordinate: the index on the uniform grid (Sec. 4.3) or of a 32..256-level quantizer
        const uint8_t *bytes = B.codes[c] ? B.codes[c] : reinterpret_cast<const uint8_t *>(payload);
        const rsrc_t rp = make_rsrc(bytes + base, (1u << log2D) - (uint32_t)base);
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = __uint_as_float(buf_load_byte(rp, lane, (uint32_t)r << p));
        const uint32_t H = wide_half_levels(b_q8);
        if (grid_q15(b_q8)) {                                    // the values replace the bytes in their registers
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = dequantize_byte<true>(__float_as_uint(v[r]), H, gtabs[wv]);
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = dequantize_byte<false>(__float_as_uint(v[r]), H, gtabs[wv]);
        }
    } else if (budget_mixed(b_q8)) {
        // b = bits + 1/2 (Sec. 4.1): every coordinate has `bits` bits in the first part; the coordinate of each pair
        // that the MIX stream selects was quantized with the finer table and has its top bit in the second part
        const uint64_t key = stream_key(seed, kStreamMix, B.client[c]);
        const uint32_t offs_mine = (uint32_t)(hash_word(key, my_row >> 7) >> (32u * (uint32_t)((base >> 6) & 1u)));
        const uint32_t lbits = lane * (uint32_t)bits, words_row = 2u * (uint32_t)bits;      // words of one row segment
        const rsrc_t rp = make_rsrc(payload + (base >> 6) * words_row, payload_bytes - (uint32_t)(base >> 6) * words_row * 4u);
        const uint32_t *part_b = payload + payload_bytes / 4u;
        const rsrc_t rb = make_rsrc(part_b + (base >> 6), (uint32_t)payload_b_bytes(1ull << log2D, b_q8) - (uint32_t)(base >> 6) * 4u);
        const uint32_t voff = (lbits >> 5) * 4u, shift = lbits & 31u;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int soff = (int)((((uint32_t)r * words_row) << (p - 6)) * 4u);
            const uint32_t w0 = __builtin_amdgcn_raw_buffer_load_b32(rp, (int)voff, soff, 0);
            const uint32_t w1 = __builtin_amdgcn_raw_buffer_load_b32(rp, (int)voff + 4, soff, 0);    // always: no branch per value
            const uint32_t low = code_at(w0, w1, shift, bits);
            const uint32_t wb = __builtin_amdgcn_raw_buffer_load_b32(rb, 0, (int)(((uint32_t)r << (p - 6)) * 4u), 0);
            const uint32_t offs = __builtin_amdgcn_readlane(offs_mine, r);
            const bool up = ((offs >> (lane >> 1)) & 1u) == (lane & 1u);
            const uint32_t top = (wb >> (lane >> 1)) & 1u;
            v[r] = up ? tb2[(top << bits) | low] : tb[low];
        }
    } else if (coin_q8(b_q8)) {
        // coin budgets (Sec. 4.1): every coordinate has `bits` bits in the first part; a coordinate with a coin was
        // quantized with the finer table and has its top bit in the second part, at the position of its rank among the coins
        const uint32_t w = (uint32_t)(my_row >> 6);
        const uint64_t mask_mine = coin_mask_of(ct, c, log2D, w);
        const uint32_t off_mine = coins_before(ct, c, log2D, w);
        const uint32_t lbits = lane * (uint32_t)bits, words_row = 2u * (uint32_t)bits;
        const rsrc_t rp = make_rsrc(payload + (base >> 6) * words_row, payload_bytes - (uint32_t)(base >> 6) * words_row * 4u);
        const rsrc_t rb = make_rsrc(payload + payload_bytes / 4u, (uint32_t)coin_b_bytes(ct.total[c]));
        const uint32_t voff = (lbits >> 5) * 4u, shift = lbits & 31u;
        // the top bits of a row's coins are at most 64 consecutive bits of the second part, from bit off_mine on: the lane
        // that looks after the row fetches them once (beyond the part: 0), and every lane finds its bit in that window
        uint64_t window_mine;
        {
            const int at = (int)((off_mine >> 5) * 4u);
            const uint32_t b0 = __builtin_amdgcn_raw_buffer_load_b32(rb, at, 0, 0), b1 = __builtin_amdgcn_raw_buffer_load_b32(rb, at + 4, 0, 0);
            const uint32_t b2 = __builtin_amdgcn_raw_buffer_load_b32(rb, at + 8, 0, 0);
            window_mine = ((uint64_t)__builtin_amdgcn_alignbit(b2, b1, off_mine & 31u) << 32) | __builtin_amdgcn_alignbit(b1, b0, off_mine & 31u);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int soff = (int)((((uint32_t)r * words_row) << (p - 6)) * 4u);
            const uint32_t w0 = __builtin_amdgcn_raw_buffer_load_b32(rp, (int)voff, soff, 0);
            const uint32_t w1 = __builtin_amdgcn_raw_buffer_load_b32(rp, (int)voff + 4, soff, 0);    // always: no branch per value
            const uint32_t low = code_at(w0, w1, shift, bits);
            const uint64_t m = wave_read64(mask_mine, r);
            const uint32_t top = (uint32_t)(wave_read64(window_mine, r) >> lanes_below(m)) & 1u;
            v[r] = __builtin_amdgcn_inverse_ballot_w64(m) ? tb2[(top << bits) | low] : tb[low];
        }
    } else if (bits == 3) {
        // 64 columns x 3 bits = 6 words per row; an index may straddle two words
        const uint32_t lbits = lane * 3u;
        const rsrc_t rp = make_rsrc(payload + (base >> 6) * 6u, payload_bytes - (uint32_t)(base >> 6) * 24u);
        const uint32_t voff = (lbits >> 5) * 4u, shift = lbits & 31u;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int soff = (int)((((uint32_t)r * 6u) << (p - 6)) * 4u);
            const uint32_t w0 = __builtin_amdgcn_raw_buffer_load_b32(rp, (int)voff, soff, 0);
            const uint32_t w1 = __builtin_amdgcn_raw_buffer_load_b32(rp, (int)voff + 4, soff, 0);
            v[r] = tb[code_at(w0, w1, shift, 3)];
        }
    } else {
        const uint32_t lbits = lane * (uint32_t)bits;
        const rsrc_t rp = make_rsrc(payload + ((base * (uint32_t)bits) >> 5), payload_bytes - (uint32_t)((base * (uint32_t)bits) >> 5) * 4u);
        const uint32_t voff = (lbits >> 5) * 4u, shift = lbits & 31u;
        const uint32_t mag = __float_as_uint(tb[1]);
#pragma unroll
        for (int r = 0; r < R; ++r)                              // all loads first, no choice per value in between
            v[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rp, (int)voff, (int)((((uint32_t)r * (uint32_t)bits) << (p - 5)) * 4u), 0));
        if (bits == 1) {
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = __uint_as_float(mag | ((~(__float_as_uint(v[r]) >> shift) & 1u) << 31));
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = tb[(__float_as_uint(v[r]) >> shift) & ((1u << bits) - 1u)];
        }
    }
    if (B.bitmap[c]) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = ((recv >> r) & 1ull) ? v[r] : 0.0f;     // wave-uniform per row
    }
    fwht_regs<R>(v);
    if (i16) {                                                   // exact integers of magnitude <= 2^M, as fp16
        const rsrc_t rt = make_rsrc(T + ((size_t)c << log2D), (uint32_t)(keep_elems * 2));
#pragma unroll
        for (int r = 0; r < R; ++r)
            __builtin_amdgcn_raw_buffer_store_b16(narrow_bits(v[r]), rt, (int)(lane * 2u),
                                                  (int)(((uint32_t)base + ((uint32_t)r << p)) * 2u), kStream);
    } else {
        const rsrc_t rt = make_rsrc(T + ((size_t)c << log2D), (uint32_t)(keep_elems * 4));
#pragma unroll
        for (int r = 0; r < R; ++r) buf_store(rt, lane * 4u, ((uint32_t)base + ((uint32_t)r << p)) * 4u, v[r]);
    }
}

// ------------------------------------------------------------------------------------------------
// Wide strided tiles for the top three index bits of D >= 2^25 when every sender has a one-byte budget (b = 5..8, uniform grid):
// these go through three passes.  (With two, the pass next to the payload moves the bytes in pieces of 32 and holds 2^16 values
// while it searches 128 thresholds: one sender of 2^27 at b = 8 took 610 us instead of 600.)
// a wave owns 8 rows of 512 consecutive coordinates at stride 2^p (p = log2 D - 3).  A lane holds, of every row,
// the columns 4 l .. 4 l + 3 and 256 + 4 l .. 256 + 4 l + 3: each workspace access of a wave is then one dense
// kilobyte (16 bytes per lane, no gaps; with 8 adjacent columns per lane the two halves of every 128-byte line
// were written by different instructions and 1.7x the bytes reached memory), and a lane's four indices of a half row are
// four bytes, 256 dense bytes per wave.
constexpr int kWideRows = 8, kWideCols = 512;

__device__ inline void wide_fwht(float (&v)[kWideRows][8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float col[kWideRows];
#pragma unroll
        for (int r = 0; r < kWideRows; ++r) col[r] = v[r][e];
        fwht_regs<kWideRows>(col);
#pragma unroll
        for (int r = 0; r < kWideRows; ++r) v[r][e] = col[r];
    }
}
// Encode, last pass (see k_enc_hi_last): index bits p .. p+2, quantization, sum_i u_i q_i, packing.
__global__ __launch_bounds__(256) void k_enc_wide_last(EncBatch B, uint64_t valid_elems, int log2D, const float *T,
                                                       double *partials, uint32_t partial_stride,
                                                       const EncScratch *scratch) {
    __shared__ double red[4];
    const uint32_t c = blockIdx.y;
    const uint32_t lane = lane_id();
    const int p = log2D - 3;
    const uint32_t tile = blockIdx.x * 4u + wave_in_block();     // 2^(p-9) column blocks, all 8 rows
    const uint32_t base = tile * (uint32_t)kWideCols;
    const rsrc_t rt = make_rsrc(T + ((size_t)c << log2D), (uint32_t)(valid_elems * 4));
    float v[kWideRows][8];
#pragma unroll
    for (int r = 0; r < kWideRows; ++r) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const u32x4_t q = __builtin_amdgcn_raw_buffer_load_b128(rt, (int)(lane * 16u),
                                                                     (int)((base + 256u * h + ((uint32_t)r << p)) * 4u), kStream);
            v[r][4 * h] = __uint_as_float(q.x); v[r][4 * h + 1] = __uint_as_float(q.y);
            v[r][4 * h + 2] = __uint_as_float(q.z); v[r][4 * h + 3] = __uint_as_float(q.w);
        }
    }
    wide_fwht(v);
    char *payload = static_cast<char *>(B.msg[c]) + EDEN_HEADER_BYTES;
    const uint32_t b_q8 = B.b_q8[c];
    const EncScratch *sc = &scratch[c];
    __shared__ float gtabs[4][256];                              // centroids and thresholds
    float *gtab = gtabs[wave_in_block()];
    const float *byte_tab = sc->grid_c;                          // grid_c[128] and wide_thr[128] are one run of 256 floats
#pragma unroll
    for (int q = 0; q < 4; ++q) gtab[64 * q + lane] = byte_tab[64 * q + lane];
    wave_lds_sync();
    float ip = 0.0f;
    // the choice of the budget sits outside the loops over the 16 groups (group = this lane's 4 coordinates of a row half)
    auto for_groups = [&](auto &&pack) {
#pragma unroll
        for (int r = 0; r < kWideRows; ++r)
#pragma unroll
            for (int h = 0; h < 2; ++h) pack((base + 256u * h + ((uint32_t)r << p)) / 4u + lane, r, h);
    };
    if (grid_q15(b_q8)) {                                        // uniform grid: one byte per coordinate
        const float inv = sc->grid_inv;
        for_groups([&](uint32_t group, int r, int h) {
            uint32_t word = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) word |= quantize_byte<true>(v[r][4 * h + e], 0u, inv, gtab, ip) << (8 * e);
            reinterpret_cast<uint32_t *>(payload)[group] = word;
        });
    } else {                                                     // b = 5..8
        const uint32_t H = wide_half_levels(b_q8);
        uint32_t *dst = reinterpret_cast<uint32_t *>(B.codes[c] ? reinterpret_cast<char *>(B.codes[c]) : payload);
        for_groups([&](uint32_t group, int r, int h) {
            uint32_t word = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) word |= quantize_byte<false>(v[r][4 * h + e], H, 0.0f, gtab, ip) << (8 * e);
            dst[group] = word;
        });
    }
    const double block_total = block_sum<256>((double)ip, red);
    if (threadIdx.x == 0) partials[(size_t)c * partial_stride + blockIdx.x] = block_total;
}

// Decode, first pass (see k_dec_hi_first): unpack, dequantize, zero the rows whose packet was lost, index bits
// p .. p+2.  A row segment of 512 coordinates lies inside one packet of 1024.
__global__ __launch_bounds__(256) void k_dec_wide_first(DecBatch B, uint64_t keep_elems, int log2D, const DecScratch *scratch,
                                                        float *T) {
    const uint32_t c = blockIdx.y;
    const uint32_t lane = lane_id(), wv = wave_in_block();
    const int p = log2D - 3;
    const uint32_t tile = blockIdx.x * 4u + wv;
    const uint32_t base = tile * (uint32_t)kWideCols;
    __shared__ float gtabs[4][kGridMax + 1];
    const uint32_t b_q8 = B.b_q8[c];
    gtabs[wv][lane] = scratch[c].grid_deq[lane];
    gtabs[wv][64 + lane] = scratch[c].grid_deq[64 + lane];
    wave_lds_sync();
    const char *payload = static_cast<const char *>(B.msg[c]) + EDEN_HEADER_BYTES;
    const char *bytes = B.codes[c] ? reinterpret_cast<const char *>(B.codes[c]) : payload;
    const uint32_t *bm = B.bitmap[c];
    // which of the 8 rows arrived (wave-uniform), then all payload loads, then the table look-ups: the choice of the
    // budget sits outside the loops so that the loads are issued back to back
    uint32_t here = 0xFFu;
    if (bm) {
        here = 0;
#pragma unroll
        for (int r = 0; r < kWideRows; ++r) {
            const uint32_t pk = (base + ((uint32_t)r << p)) >> 10;
            here |= ((bm[pk >> 5] >> (pk & 31u)) & 1u) << r;
        }
    }
    float v[kWideRows][8];
    uint32_t word[kWideRows][2];
    auto for_groups = [&](auto &&fetch) {                        // group = this lane's 4 coordinates of (row, half)
#pragma unroll
        for (int r = 0; r < kWideRows; ++r)
#pragma unroll
            for (int h = 0; h < 2; ++h) word[r][h] = fetch((base + ((uint32_t)r << p) + 256u * h) / 4u + lane);
#pragma unroll
        for (int r = 0; r < kWideRows; ++r) asm volatile("" : "+v"(word[r][0]), "+v"(word[r][1]));      // else each is loaded where it is used
    };
    auto for_values = [&](auto &&value) {
#pragma unroll
        for (int r = 0; r < kWideRows; ++r)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[r][4 * h + e] = ((here >> r) & 1u) ? value(word[r][h], e) : 0.0f;
    };
    const float *gt = gtabs[wv];
    if (grid_q15(b_q8)) {
        for_groups([&](uint32_t g) { return reinterpret_cast<const uint32_t *>(bytes)[g]; });
        for_values([&](uint32_t w, int e) { return dequantize_byte<true>((w >> (8 * e)) & 0xFFu, 0u, gt); });
    } else {
        const uint32_t H = wide_half_levels(b_q8);
        for_groups([&](uint32_t g) { return reinterpret_cast<const uint32_t *>(bytes)[g]; });
        for_values([&](uint32_t w, int e) { return dequantize_byte<false>((w >> (8 * e)) & 0xFFu, H, gt); });
    }
    wide_fwht(v);
    const rsrc_t rt = make_rsrc(T + ((size_t)c << log2D), (uint32_t)(keep_elems * 4));
#pragma unroll
    for (int r = 0; r < kWideRows; ++r) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4_t q = {__float_as_uint(v[r][4 * h]), __float_as_uint(v[r][4 * h + 1]), __float_as_uint(v[r][4 * h + 2]),
                         __float_as_uint(v[r][4 * h + 3])};
            // (no scalar offset on a store of more than 64 bits: see the note in k_dec_hix_first_mfma)
            __builtin_amdgcn_raw_buffer_store_b128(q, rt, (int)(lane * 16u + (base + 256u * h + ((uint32_t)r << p)) * 4u), 0, kStream);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// One workgroup per sender: sums the partials of sum_i u_i q_i in index order, forms
// <R(x),Q> = D^-1/2 sum and the scale S = |x|^2 / <R(x),Q> (Sec. 2.3), writes the header.
// A zero or non-finite vector gets S = 0, a status bit and an all-zero payload.
__global__ __launch_bounds__(256) void k_enc_finish(EncBatch B, uint64_t hdr_d, int log2D, uint64_t seed,
                                                    const double *partials_n2, uint32_t nparts_n2,
                                                    const double *partials_ip, uint32_t nparts_ip,
                                                    uint32_t partial_stride, uint32_t *dev_status, const uint32_t *coin_total) {
    __shared__ double red[4];
    const uint32_t c = blockIdx.x;
    const double n2 = ordered_sum<256>(partials_n2 + (size_t)c * partial_stride, nparts_n2, red);
    const double total = ordered_sum<256>(partials_ip + (size_t)c * partial_stride, nparts_ip, red);
    if (!(enc_valid_norm(n2) && total > 0.0)) zero_payload<256>(B, c, log2D, coin_total, false);
    if (threadIdx.x == 0) write_enc_header(B, c, hdr_d, log2D, seed, n2, total, dev_status, coin_total);
}

// ------------------------------------------------------------------------------------------------
// decode side
//
__global__ __launch_bounds__(64) void k_dec_prepare(DecBatch B, uint64_t hdr_d, int log2D, uint64_t seed,
                                                    const DevTables *tab, DecScratch *scratch, uint32_t *dev_status,
                                                    const uint32_t *coin_total, uint32_t *msg_flags) {
    const uint32_t c = blockIdx.x;
    dec_prepare_wave(B.msg[c], B.bitmap[c], B.client[c], B.b_q8[c], B.hdr_b_q8[c], hdr_d, log2D, seed, tab, &scratch[c], dev_status,
                     coin_q8(B.b_q8[c]) ? coin_total[c] : 0u, msg_flags ? msg_flags + c : nullptr);
}

// ---- coin budgets (Sec. 4.1): the coins of every sender of a launch that has such a budget, as lane masks per block of 64
// coordinates, with the prefix sums that give every block its place in the second part of the payload.  Both sides run
// this from the shared seed alone.  One thread per block of 64 coordinates (8 hash words of 8 coins each).
struct CoinBatch {
    uint32_t client[kMaxBatch];
    uint32_t b_q8[kMaxBatch];
    void *part_b[kMaxBatch];             // encode: the second part of the sender's payload, cleared here; decode: null
};
__device__ inline uint32_t block_exclusive_scan_256(uint32_t mine, uint32_t *wave_totals /* shared, 4 */, uint32_t &block_total) {
    const uint32_t lane = lane_id(), wv = threadIdx.x >> 6;
    uint32_t incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = (uint32_t)__shfl_up((int)incl, o, 64);
        if (lane >= (uint32_t)o) incl += v;
    }
    if (lane == 63) wave_totals[wv] = incl;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) { before += i < wv ? wave_totals[i] : 0u; all += wave_totals[i]; }
    __syncthreads();
    block_total = all;
    return before + incl - mine;
}
// bit j of byte b to bit b of byte j (Hacker's Delight, section 7-3)
__device__ inline uint64_t transpose_8x8(uint64_t x) {
    uint64_t t = (x ^ (x >> 7)) & 0x00AA00AA00AA00AAull;
    x = x ^ t ^ (t << 7);
    t = (x ^ (x >> 14)) & 0x0000CCCC0000CCCCull;
    x = x ^ t ^ (t << 14);
    t = (x ^ (x >> 28)) & 0x00000000F0F0F0F0ull;
    return x ^ t ^ (t << 28);
}
__global__ __launch_bounds__(256) void k_coin_masks(CoinBatch B, uint64_t seed, int log2D, CoinTables ct) {
    __shared__ uint32_t wave_totals[4];
    const uint32_t c = blockIdx.y;
    const uint32_t frac = coin_q8(B.b_q8[c]) & 255u;
    if (!frac) return;                                           // not a coin budget: the whole workgroup leaves
    const uint32_t words = 1u << (log2D - 6);
    const uint32_t w = blockIdx.x * (uint32_t)kCoinGroup + threadIdx.x;
    uint64_t m = 0;
    if (w < words) {
        const uint64_t key = stream_key(seed, kStreamMix, B.client[c]);
        // Byte b of hash word j is below frac?  Four bytes at a time, the answers in their top bits: those of the low seven bits by a
        // subtraction that cannot borrow.  The answers of word j end in bit j of every byte, 8 x 8 bits to be transposed.  (A compare, a
        // select and an or per byte, with a wait for each compare's mask: encode of 8 senders of 4,000,037 at 2.7 bits 105.9 -> 103.7 us,
        // decode 89.4 -> 87.4.)
        const uint32_t f = frac * 0x01010101u, f7 = f & 0x7F7F7F7Fu;
        uint32_t rows[2] = {0u, 0u};
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j) {
            const uint64_t h = hash_word(key, 8ull * w + j);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const uint32_t x = half ? hi32(h) : lo32(h), not_below = (x | 0x80808080u) - f7;
                // (~x & f) | (~(x ^ f) & ~not_below)
                const uint32_t below = (uint32_t)__builtin_amdgcn_bitop3_b32((int)x, (int)f, (int)not_below, 0x4D);
                rows[half] = (rows[half] >> 1) | (below & 0x80808080u);
            }
        }
        m = transpose_8x8((uint64_t)rows[1] << 32 | rows[0]);
    }
    uint32_t group_total;
    const uint32_t before = block_exclusive_scan_256((uint32_t)__popcll(m), wave_totals, group_total);
    if (w < words) {
        ct.mask[((size_t)c << (log2D - 6)) + w] = m;
        ct.local[((size_t)c << (log2D - 6)) + w] = before;
        if (B.part_b[c]) static_cast<uint64_t *>(B.part_b[c])[w] = 0ull;
    }
    if (threadIdx.x == 0) ct.group[(size_t)c * ct.group_stride + blockIdx.x] = group_total;
}
// One workgroup per sender: the group totals become the number of coins before each group, and the grand total.
__device__ inline void coin_scan(uint32_t c, int log2D, const CoinTables &ct) {
    __shared__ uint32_t wave_totals[4];
    const uint32_t words = 1u << (log2D - 6);
    const uint32_t groups = (words + (uint32_t)kCoinGroup - 1) / (uint32_t)kCoinGroup;
    const uint32_t per = (groups + 255u) / 256u;
    uint32_t *g = ct.group + (size_t)c * ct.group_stride;
    const uint32_t first = threadIdx.x * per;
    uint32_t mine = 0;
    for (uint32_t i = first; i < first + per && i < groups; ++i) mine += g[i];
    uint32_t all;
    uint32_t run = block_exclusive_scan_256(mine, wave_totals, all);
    for (uint32_t i = first; i < first + per && i < groups; ++i) {
        const uint32_t v = g[i];
        g[i] = run;
        run += v;
    }
    if (threadIdx.x == 0) ct.total[c] = all;
}
__global__ __launch_bounds__(256) void k_coin_scan(CoinBatch B, int log2D, CoinTables ct) {
    if (coin_q8(B.b_q8[blockIdx.x])) coin_scan(blockIdx.x, log2D, ct);
}
// Where another launch of one workgroup per sender stands between the masks and the pass that reads the sums, it does the scan as well
// (4.7 us a launch; round of 8 senders of 4,000,037 at 2.7 bits 245 -> 243 us, of 2,000,000 at 3.3 162 -> 159; encode of one of 1,500,000
// at 1.3 33.9 -> 32.4).
__global__ __launch_bounds__(256) void k_enc_norm_scan(EncBatch B, const double *partials, uint32_t partial_stride, uint32_t nparts,
                                                       EncScratch *scratch, const DevTables *tab, int log2D, CoinTables ct) {
    __shared__ double red[4];
    const uint32_t c = blockIdx.x;
    if (coin_q8(B.b_q8[c])) coin_scan(c, log2D, ct);
    enc_norm(B, c, partials, partial_stride, nparts, scratch, tab, red);
}
__global__ __launch_bounds__(256) void k_dec_prepare_scan(DecBatch B, uint64_t hdr_d, int log2D, uint64_t seed, const DevTables *tab,
                                                          DecScratch *scratch, uint32_t *dev_status, CoinTables ct, uint32_t *msg_flags) {
    const uint32_t c = blockIdx.x;
    if (coin_q8(B.b_q8[c])) coin_scan(c, log2D, ct);
    __syncthreads();                                             // the total is in memory
    if (threadIdx.x < 64u)
        dec_prepare_wave(B.msg[c], B.bitmap[c], B.client[c], B.b_q8[c], B.hdr_b_q8[c], hdr_d, log2D, seed, tab, &scratch[c], dev_status,
                         coin_q8(B.b_q8[c]) ? ct.total[c] : 0u, msg_flags ? msg_flags + c : nullptr);
}

// Coin budgets, encoder in workgroup tiles: the last pass leaves, for every segment of 32 consecutive coordinates, the top
// bits of its coins moved together towards bit 0, one word per segment, in `pieces` (bits above the segment's number of
// coins are 0).  This kernel strings them together into the second part of the payload (Sec. 4.1: one more bit for every
// coordinate with a coin, in coordinate order).  A thread looks after one block of 64 coordinates; if one of the part's 64-bit
// words begins inside the block's run of bits, the thread assembles that word from its own pieces and those of the blocks
// after it.  Every word is written by exactly one thread: no atomics (they cost the last encode pass a third of its time).
struct CoinPackBatch {
    uint32_t b_q8[kMaxBatch];
    const uint32_t *pieces[kMaxBatch];   // null: the sender's bits were placed by the last pass itself
    uint64_t *part_b[kMaxBatch];
};
__global__ __launch_bounds__(256) void k_coin_pack(CoinPackBatch B, int log2D, CoinTables ct) {
    const uint32_t c = blockIdx.y;
    const uint32_t *pieces = B.pieces[c];
    if (!coin_q8(B.b_q8[c]) || !pieces) return;
    const uint32_t blocks = 1u << (log2D - 6);
    const uint32_t k = blockIdx.x * 256u + threadIdx.x;
    if (k >= blocks) return;
    const uint64_t mine = coin_mask_of(ct, c, log2D, k);
    const uint32_t count = (uint32_t)__popcll(mine);
    const uint32_t start = coins_before(ct, c, log2D, k);       // this block's bits are [start, start + count) of the part
    const uint32_t word = (start + 63u) >> 6;                    // the first word that begins at or after `start`
    if ((uint64_t)word * 64u >= (uint64_t)start + count) return; // none begins inside this block's run
    uint32_t skip = word * 64u - start;                          // bits of this block that belong to the word before
    uint64_t bits = 0;
    uint32_t have = 0;
    for (uint32_t kk = k; have < 64u && kk < blocks; ++kk) {
        const uint64_t m = kk == k ? mine : coin_mask_of(ct, c, log2D, kk);
        const uint32_t lo = (uint32_t)__popc(lo32(m));
        uint32_t n = lo + (uint32_t)__popc(hi32(m));
        if (n == 0u) continue;
        uint64_t run = (uint64_t)pieces[2u * kk] | ((uint64_t)pieces[2u * kk + 1u] << lo);
        run >>= skip;                                            // (only the first block has bits to skip, fewer than it holds)
        n -= skip;
        skip = 0;
        bits |= run << have;
        have += n;
    }
    B.part_b[c][word] = bits;
}

// Decode, last pass at D <= 2^18: index bits 0..11 of H of one sender's vector and its sign diagonal (R^-1 = s o D^-1/2 H,
// Sec. 2.2.2; D^-1/2 is inside the dequantization scale), in place in the sender's workspace slot (a workgroup has read its tile
// before it writes it).
// One workgroup per (tile, sender): at these sizes (D <= 2^18) there are at most 64 tiles, and a wave that summed all senders of its
// tile one after the other left the chip idle (32 senders of 60,000, b = 1: 80 of the round's 139 us).  The sum follows in
// k_dec_lo_combine.  16 values per thread (eden_lo.h): a wave per tile with 64 of them was the longer chain.
// ONE: the launch has one sender, whose values go to acc at once (mean_n > 0: written, divided by mean_n; else added).
template <bool ONE>
__global__ __launch_bounds__(256, 8) void k_dec_lo_last(DecBatch B, uint64_t d, int log2D, uint64_t seed, float *T, const DecScratch *scratch,
                                                     float *acc, float mean_n) {
    __shared__ __attribute__((aligned(16))) float lds[Lo16<kLoBits>::LDS_FLOATS];
    const uint32_t t = threadIdx.x, lane = t & 63u, wv = wave_in_block(), c = blockIdx.y;
    const uint32_t tile_base = blockIdx.x << kLoBits;
    float *slot = T + ((size_t)c << log2D);
    const rsrc_t rt = make_rsrc(slot, 4u << log2D);
    float v[16];
#pragma unroll
    for (int a = 0; a < 16; ++a) v[a] = buf_load_keep(rt, 4u * t, 4u * (tile_base + 256u * a));
    lo_forward16<kLoBits>(v, lds);
    const uint64_t word = hash_word(stream_key(seed, kStreamSign, B.client[c]), (tile_base >> 6) + (t >> 2));
    const uint32_t bits = (uint32_t)(word >> (16u * (t & 3u)));          // 16 sign bits of this thread's run
#pragma unroll
    for (int e = 0; e < 16; ++e)                                 // bit 1 -> s_i = -1
        v[e] = __uint_as_float(__float_as_uint(v[e]) ^ ((bits << (31 - e)) & 0x80000000u));
    float4 x[4];
    wave_quads(v, lds + wv * (Lo16<kLoBits>::LDS_FLOATS / 4), x);
    const float scale = ONE && B.b_q8[0] <= 256u ? fabsf(scratch[0].deq[1]) : 1.0f;
    const bool overwrite = mean_n > 0.0f;
    const float div = overwrite ? mean_n : 1.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t i = tile_base + 1024u * wv + 256u * (uint32_t)j + 4u * lane;
        if constexpr (!ONE) {
            *reinterpret_cast<float4 *>(slot + i) = x[j];
        } else {                                                 // the arithmetic of k_dec_lo_combine
            const float y[4] = {x[j].x, x[j].y, x[j].z, x[j].w};
            float z[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float old = !overwrite && i + e < d ? acc[i + e] : 0.0f;
                z[e] = (old + fmaf(y[e], scale, 0.0f)) / div;
            }
            if (i + 4 <= d) {                                    // (acc is 16-byte aligned)
                *reinterpret_cast<float4 *>(acc + i) = make_float4(z[0], z[1], z[2], z[3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (i + e < d) acc[i + e] = z[e];
            }
        }
    }
}

// The sum over the senders of what k_dec_lo_last left in their slots, one after the other; the magnitude S/(p sqrt D) q_1 of a
// b <= 1 sender (whose slot holds exact integers) is applied here.  Four values per thread.  mean_n > 0: acc is written with the
// sum divided by mean_n instead of added to.
// PRE (b = 1/2 with the sparsification first, Sec. 4.1): value g of sender c belongs at coordinate 2g + o_g of acc (o_g from c's
// SUB-SAMPLING stream), g < ceil(d/2).
template <bool PRE>
__global__ __launch_bounds__(64) void k_dec_lo_combine(DecBatch B, uint32_t n, uint64_t d, int log2D, uint64_t seed, const float *T,
                                                       const DecScratch *scratch, float *acc, float mean_n) {
    constexpr int NS = PRE ? 8 : 4;                              // outputs per thread
    const uint64_t g = 4u * ((uint64_t)blockIdx.x * 64u + threadIdx.x), out = (PRE ? 2u : 1u) * g;
    if (out >= d) return;
    float sum[NS];
#pragma unroll
    for (int e = 0; e < NS; ++e) sum[e] = 0.0f;
    const bool overwrite = mean_n > 0.0f;
    float old[NS];
#pragma unroll
    for (int e = 0; e < NS; ++e) old[e] = (!overwrite && out + e < d) ? acc[out + e] : 0.0f;
#pragma unroll 8
    for (uint32_t c = 0; c < n; ++c) {
        const float4 v = *reinterpret_cast<const float4 *>(T + ((size_t)c << log2D) + g);
        const float scale = B.b_q8[c] <= 256u ? fabsf(scratch[c].deq[1]) : 1.0f;
        const float x[4] = {v.x, v.y, v.z, v.w};
        if constexpr (PRE) {
            const uint32_t offs = (uint32_t)(hash_word(stream_key(seed, kStreamSubsample, B.client[c]), g >> 6) >> (g & 63u));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool odd = (offs >> e) & 1u;
                sum[2 * e] = odd ? sum[2 * e] : fmaf(x[e], scale, sum[2 * e]);
                sum[2 * e + 1] = odd ? fmaf(x[e], scale, sum[2 * e + 1]) : sum[2 * e + 1];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] = fmaf(x[e], scale, sum[e]);
        }
    }
    const float div = overwrite ? mean_n : 1.0f;
#pragma unroll
    for (int e = 0; e < NS; ++e) sum[e] = (old[e] + sum[e]) / div;
    if (out + NS <= d) {                                         // (acc is 16-byte aligned)
#pragma unroll
        for (int q = 0; q < NS / 4; ++q)
            *reinterpret_cast<float4 *>(acc + out + 4 * q) = make_float4(sum[4 * q], sum[4 * q + 1], sum[4 * q + 2], sum[4 * q + 3]);
    } else {
#pragma unroll
        for (int e = 0; e < NS; ++e)
            if (out + e < d) acc[out + e] = sum[e];
    }
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
// Sec. 2.2.2: the plain average.  Four coordinates per thread when both pointers are 16-byte aligned.
__global__ void k_finalize_mean(const float *acc, uint64_t d, float n, float *mean, int vec) {
    const uint64_t i = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) * (vec ? 4u : 1u);
    if (vec && i + 3 < d) {
        f32x4 a = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(acc + i));
        a.x /= n; a.y /= n; a.z /= n; a.w /= n;
        *reinterpret_cast<f32x4 *>(mean + i) = a;
    } else {
        for (uint64_t e = i; e < d && e < i + (vec ? 4u : 1u); ++e) mean[e] = acc[e] / n;
    }
}

// b = 5, 6, 7: the one-byte indices of a sender, in coordinate order, to the payload's bit string (index j in bits
// j b .. j b + b - 1, Sec. 2.2.1 message) and back.  A thread handles 32 indices = 32 bytes = b payload words.
template <int BITS>
__device__ inline void pack32(const uint8_t *codes, uint32_t *words) {
    uint32_t in[8];
    const uint4 lo = reinterpret_cast<const uint4 *>(codes)[0], hi = reinterpret_cast<const uint4 *>(codes)[1];
    in[0] = lo.x; in[1] = lo.y; in[2] = lo.z; in[3] = lo.w; in[4] = hi.x; in[5] = hi.y; in[6] = hi.z; in[7] = hi.w;
    uint32_t out[BITS];
#pragma unroll
    for (int w = 0; w < BITS; ++w) out[w] = 0;
#pragma unroll
    for (int j = 0; j < 32; ++j) {
        const uint32_t code = (in[j >> 2] >> (8 * (j & 3))) & ((1u << BITS) - 1u);
        const int pos = j * BITS;
        out[pos >> 5] |= code << (pos & 31);
        if ((pos & 31) + BITS > 32) out[(pos >> 5) + 1] |= code >> (32 - (pos & 31));
    }
#pragma unroll
    for (int w = 0; w < BITS; ++w) words[w] = out[w];
}
template <int BITS>
__device__ inline void unpack32(const uint32_t *words, uint8_t *codes) {
    uint32_t in[BITS + 1];
#pragma unroll
    for (int w = 0; w < BITS; ++w) in[w] = words[w];
    in[BITS] = 0;
    uint32_t out[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) out[q] = 0;
#pragma unroll
    for (int j = 0; j < 32; ++j) {
        const int pos = j * BITS;
        const uint32_t code = code_at(in[pos >> 5], in[(pos >> 5) + 1], (uint32_t)(pos & 31), BITS);
        out[j >> 2] |= code << (8 * (j & 3));
    }
    reinterpret_cast<uint4 *>(codes)[0] = make_uint4(out[0], out[1], out[2], out[3]);
    reinterpret_cast<uint4 *>(codes)[1] = make_uint4(out[4], out[5], out[6], out[7]);
}
__global__ __launch_bounds__(256) void k_pack_bits(EncBatch B, int log2D) {
    const uint32_t c = blockIdx.y;
    const uint8_t *codes = B.codes[c];
    const uint32_t bits = wide_bits(B.b_q8[c]);
    if (!codes || bits < 5u || bits > 7u) return;                // (a coin sender's buffer holds the pieces of its second part)
    const uint64_t g = (uint64_t)blockIdx.x * 256u + threadIdx.x;        // group of 32 indices
    if (g >= (1ull << log2D) / 32) return;
    uint32_t *payload = reinterpret_cast<uint32_t *>(static_cast<char *>(B.msg[c]) + EDEN_HEADER_BYTES) + g * bits;
    if (bits == 5) pack32<5>(codes + 32 * g, payload);
    else if (bits == 6) pack32<6>(codes + 32 * g, payload);
    else pack32<7>(codes + 32 * g, payload);
}
__global__ __launch_bounds__(256) void k_unpack_bits(DecBatch B, int log2D, uint8_t *codes_all) {
    const uint32_t c = blockIdx.y;
    if (!B.codes[c]) return;
    const uint64_t g = (uint64_t)blockIdx.x * 256u + threadIdx.x;
    if (g >= (1ull << log2D) / 32) return;
    const uint32_t bits = wide_bits(B.b_q8[c]);
    const uint32_t *payload = reinterpret_cast<const uint32_t *>(static_cast<const char *>(B.msg[c]) + EDEN_HEADER_BYTES) + g * bits;
    uint8_t *codes = codes_all + ((size_t)c << log2D) + 32 * g;
    if (bits == 5) unpack32<5>(payload, codes);
    else if (bits == 6) unpack32<6>(payload, codes);
    else unpack32<7>(payload, codes);
}
__global__ __launch_bounds__(256) void k_fill_zero(float *p, uint64_t count) {
    const uint64_t i = (uint64_t)blockIdx.x * 256u + threadIdx.x;
    if (i < count) p[i] = 0.0f;
}

// Experiment helper (Sec. 4.3): histogram of the one-byte indices of a uniform-grid message and its entropy
// -sum f log2 f in bits per coordinate, what an ideal entropy coder would spend.
__global__ __launch_bounds__(256) void k_byte_histogram(const uint8_t *bytes, uint64_t count, uint32_t *hist) {
    __shared__ uint32_t local[256];
    local[threadIdx.x] = 0;
    __syncthreads();
    for (uint64_t i = (uint64_t)blockIdx.x * 256u + threadIdx.x; i < count; i += (uint64_t)gridDim.x * 256u)
        atomicAdd(&local[bytes[i]], 1u);
    __syncthreads();
    if (local[threadIdx.x]) atomicAdd(&hist[threadIdx.x], local[threadIdx.x]);
}
__global__ __launch_bounds__(256) void k_histogram_entropy(const uint32_t *hist, uint64_t count, double *out) {
    __shared__ double red[4];
    const double f = (double)hist[threadIdx.x] / (double)count;
    const double h = block_sum<256>(f > 0.0 ? -f * log2(f) : 0.0, red);
    if (threadIdx.x == 0) out[0] = h;
}

// Experiment helper: sum_i (a_i - b_i)^2 and sum_i a_i^2 in double, the two terms of the (v)NMSE definitions
// (Sec. 2.1: NMSE; Sec. 2.3: vNMSE).  Per-workgroup partials, then one workgroup adds them in index order.
__global__ __launch_bounds__(256) void k_sq_error(const float *a, const float *b, uint64_t d, double *partials) {
    __shared__ double red[4];
    double e2 = 0.0, a2 = 0.0;
    for (uint64_t i = (uint64_t)blockIdx.x * 256u + threadIdx.x; i < d; i += (uint64_t)gridDim.x * 256u) {
        const double x = a[i], y = b[i];
        e2 += (x - y) * (x - y);
        a2 += x * x;
    }
    const double te = block_sum<256>(e2, red);
    const double ta = block_sum<256>(a2, red);
    if (threadIdx.x == 0) { partials[2 * blockIdx.x] = te; partials[2 * blockIdx.x + 1] = ta; }
}
__global__ __launch_bounds__(256) void k_sq_error_finish(const double *partials, uint32_t nparts, double *out) {
    __shared__ double red[4];
    double e2 = 0.0, a2 = 0.0;
    for (uint32_t i = threadIdx.x; i < nparts; i += 256) { e2 += partials[2 * i]; a2 += partials[2 * i + 1]; }
    const double te = block_sum<256>(e2, red);
    const double ta = block_sum<256>(a2, red);
    if (threadIdx.x == 0) { out[0] = te; out[1] = ta; }
}

// ------------------------------------------------------------------------------------------------
// Writes up to kArgDoubles doubles that travel as kernel arguments (for a caller that may neither allocate nor stage a copy).
struct ArgDoubles { double v[kArgDoubles]; };
__global__ __launch_bounds__(kArgDoubles) void k_store_doubles(ArgDoubles a, uint32_t count, double *dst) {
    if (threadIdx.x < count) dst[threadIdx.x] = a.v[threadIdx.x];
}

// ------------------------------------------------------------------------------------------------
// test helpers: the hash streams written out
__global__ void k_hash_bits(uint64_t key, uint64_t nwords, uint64_t *out) {
    const uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j < nwords) out[j] = hash_word(key, j);
}
__global__ void k_loss_bitmap(uint64_t key, uint32_t npk, uint32_t drop_q32, uint32_t *bitmap) {
    const uint32_t w = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t nw = (npk + 31u) / 32u;
    if (w >= nw) return;
    uint32_t bits = 0;
    for (uint32_t e = 0; e < 32; ++e) {
        const uint32_t j = w * 32u + e;
        if (j >= npk) break;
        const uint32_t top = (uint32_t)(hash_word(key, j) >> 32);
        if (top >= drop_q32) bits |= 1u << e;                  // received
    }
    bitmap[w] = bits;
}

// ------------------------------------------------------------------------------------------------
// host-side launchers
#define EDEN_HI_SWITCH(M, CALL)            \
    switch (M) {                           \
        case 1: { constexpr int MM = 1; CALL; } break; \
        case 2: { constexpr int MM = 2; CALL; } break; \
        case 3: { constexpr int MM = 3; CALL; } break; \
        case 4: { constexpr int MM = 4; CALL; } break; \
        case 5: { constexpr int MM = 5; CALL; } break; \
        default: { constexpr int MM = 6; CALL; } break; \
    }

uint32_t launch_enc_hi_last(int M, const EncBatch &B, uint32_t n, uint64_t valid_elems, int log2D, int p, uint64_t seed,
                            const float *T, double *partials, uint32_t partial_stride,
                            const CoinTables &ct, const EncTail &tail, hipStream_t st) {
    const uint32_t ntiles = 1u << (log2D - 6 - M);
    dim3 grid((ntiles + 3) / 4, n);
    bool all1 = M >= 5, all2 = M >= 5, all4 = M >= 5;            // one budget for all (two-pass sizes): its own instance
    for (uint32_t c = 0; c < n; ++c) {
        all1 = all1 && B.b_q8[c] == 256u;
        all2 = all2 && B.b_q8[c] == 512u;
        all4 = all4 && B.b_q8[c] == 1024u;
    }
#define EDEN_ENC_HI_LAST(MM, ONLY)                                                                                            \
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_enc_hi_last<MM, ONLY>), grid, dim3(256), 0, st, B, valid_elems, log2D, p, seed, T, partials, \
                       partial_stride, ct, tail)
    if (all1) { if (M == 5) EDEN_ENC_HI_LAST(5, 256u); else EDEN_ENC_HI_LAST(6, 256u); }
    else if (all2) { if (M == 5) EDEN_ENC_HI_LAST(5, 512u); else EDEN_ENC_HI_LAST(6, 512u); }
    else if (all4) { if (M == 5) EDEN_ENC_HI_LAST(5, 1024u); else EDEN_ENC_HI_LAST(6, 1024u); }
    else EDEN_HI_SWITCH(M, EDEN_ENC_HI_LAST(MM, 0u));
#undef EDEN_ENC_HI_LAST
    return grid.x;
}
uint32_t launch_enc_wide_last(const EncBatch &B, uint32_t n, uint64_t valid_elems, int log2D, const float *T, double *partials,
                              uint32_t partial_stride, const EncScratch *scratch, hipStream_t st) {
    dim3 grid(1u << (log2D - 3 - 9 - 2), n);                     // D / 8 rows / 512 columns / 4 waves
    hipLaunchKernelGGL(k_enc_wide_last, grid, dim3(256), 0, st, B, valid_elems, log2D, T, partials, partial_stride, scratch);
    return grid.x;
}
void launch_dec_wide_first(const DecBatch &B, uint32_t n, uint64_t keep_elems, int log2D, const DecScratch *scratch, float *T,
                           hipStream_t st) {
    dim3 grid(1u << (log2D - 3 - 9 - 2), n);
    hipLaunchKernelGGL(k_dec_wide_first, grid, dim3(256), 0, st, B, keep_elems, log2D, scratch, T);
}
void launch_enc_norm(const EncBatch &B, uint32_t n, const double *partials, uint32_t partial_stride, uint32_t nparts,
                     EncScratch *scratch, const DevTables *tab, int log2D, const CoinTables *coins, hipStream_t st) {
    if (coins) hipLaunchKernelGGL(k_enc_norm_scan, dim3(n), dim3(256), 0, st, B, partials, partial_stride, nparts, scratch, tab, log2D, *coins);
    else hipLaunchKernelGGL(k_enc_norm, dim3(n), dim3(256), 0, st, B, partials, partial_stride, nparts, scratch, tab);
}
void launch_enc_finish(const EncBatch &B, uint32_t n, uint64_t hdr_d, int log2D, uint64_t seed,
                       const double *partials_n2, uint32_t nparts_n2, const double *partials_ip, uint32_t nparts_ip,
                       uint32_t partial_stride, uint32_t *dev_status, const uint32_t *coin_total, hipStream_t st) {
    hipLaunchKernelGGL(k_enc_finish, dim3(n), dim3(256), 0, st, B, hdr_d, log2D, seed, partials_n2, nparts_n2, partials_ip,
                       nparts_ip, partial_stride, dev_status, coin_total);
}
void launch_coin_tables(const uint32_t *clients, const uint32_t *b_q8, void *const *part_b, uint32_t n, uint64_t seed, int log2D,
                        const CoinTables &ct, bool scan, hipStream_t st) {
    CoinBatch B;
    for (uint32_t i = 0; i < (uint32_t)kMaxBatch; ++i) {
        B.client[i] = i < n ? clients[i] : 0u;
        B.b_q8[i] = i < n ? b_q8[i] : 0u;
        B.part_b[i] = (i < n && part_b) ? part_b[i] : nullptr;
    }
    const uint32_t words = 1u << (log2D - 6);
    hipLaunchKernelGGL(k_coin_masks, dim3((words + kCoinGroup - 1) / kCoinGroup, n), dim3(256), 0, st, B, seed, log2D, ct);
    if (scan) hipLaunchKernelGGL(k_coin_scan, dim3(n), dim3(256), 0, st, B, log2D, ct);
}
void launch_coin_pack(const uint32_t *b_q8, const uint32_t *const *pieces, void *const *part_b, uint32_t n, int log2D,
                      const CoinTables &ct, hipStream_t st) {
    CoinPackBatch B;
    for (uint32_t i = 0; i < (uint32_t)kMaxBatch; ++i) {
        B.b_q8[i] = i < n ? b_q8[i] : 0u;
        B.pieces[i] = i < n ? pieces[i] : nullptr;
        B.part_b[i] = i < n ? static_cast<uint64_t *>(part_b[i]) : nullptr;
    }
    const uint32_t blocks = 1u << (log2D - 6);
    hipLaunchKernelGGL(k_coin_pack, dim3((blocks + 255u) / 256u, n), dim3(256), 0, st, B, log2D, ct);
}
void launch_dec_hi_first(int M, const DecBatch &B, uint32_t n, uint64_t keep_elems, int log2D, int p, uint64_t seed,
                         const DecPrepareArgs &prep, int narrow, float *T, const CoinTables &ct, hipStream_t st) {
    const uint32_t ntiles = 1u << (log2D - 6 - M);
    dim3 grid((ntiles + 3) / 4, n);
    bool all1 = M >= 5, all2 = M >= 5, all4 = M >= 5;            // one budget for all (two-pass sizes): its own instance
    bool simple = M >= 5;
    for (uint32_t c = 0; c < n; ++c) {
        all1 = all1 && B.b_q8[c] == 256u;
        all2 = all2 && B.b_q8[c] == 512u && !B.codes[c];
        all4 = all4 && B.b_q8[c] == 1024u && !B.codes[c];
        simple = simple && simple_budget(B.b_q8[c]);
    }
#define EDEN_DEC_HI_FIRST(MM, ONLY)                                                                                           \
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_dec_hi_first<MM, ONLY>), grid, dim3(256), 0, st, B, keep_elems, log2D, p, seed, prep, \
                       narrow, T, ct)
    if (all1) { if (M == 5) EDEN_DEC_HI_FIRST(5, 256u); else EDEN_DEC_HI_FIRST(6, 256u); }
    else if (all2) { if (M == 5) EDEN_DEC_HI_FIRST(5, 512u); else EDEN_DEC_HI_FIRST(6, 512u); }
    else if (all4) { if (M == 5) EDEN_DEC_HI_FIRST(5, 1024u); else EDEN_DEC_HI_FIRST(6, 1024u); }
    else if (simple) { if (M == 5) EDEN_DEC_HI_FIRST(5, kSimple); else EDEN_DEC_HI_FIRST(6, kSimple); }
    else EDEN_HI_SWITCH(M, EDEN_DEC_HI_FIRST(MM, 0u));
#undef EDEN_DEC_HI_FIRST
}
void launch_dec_prepare(const DecBatch &B, uint32_t n, uint64_t hdr_d, int log2D, uint64_t seed, const DevTables *tab,
                        DecScratch *scratch, uint32_t *dev_status, const CoinTables &ct, bool scan, uint32_t *msg_flags,
                        hipStream_t st) {
    if (scan) {
        hipLaunchKernelGGL(k_dec_prepare_scan, dim3(n), dim3(256), 0, st, B, hdr_d, log2D, seed, tab, scratch, dev_status, ct, msg_flags);
        return;
    }
    const uint32_t *coin_total = ct.total;
    hipLaunchKernelGGL(k_dec_prepare, dim3(n), dim3(64), 0, st, B, hdr_d, log2D, seed, tab, scratch, dev_status, coin_total,
                       msg_flags);
}
void launch_dec_lo_last(const DecBatch &B, uint32_t n, uint64_t d_src, int pre, int log2D, uint64_t seed, float *T,
                        const DecScratch *scratch, float *acc, float mean_n, hipStream_t st) {
    const uint64_t d = pre == 1 ? (d_src + 1) / 2 : d_src;       // dimension of the decoded vectors
    const uint32_t tiles = (uint32_t)((d + (1u << kLoBits) - 1) >> kLoBits);
    if (n == 1 && pre == 0) {
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_dec_lo_last<true>), dim3(tiles, 1), dim3(256), 0, st, B, d, log2D, seed, T, scratch, acc, mean_n);
        return;
    }
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_dec_lo_last<false>), dim3(tiles, n), dim3(256), 0, st, B, d, log2D, seed, T, scratch, acc, mean_n);
    if (pre == 2) return;
    const dim3 grid((uint32_t)((d + 255) / 256));                // four values per thread
    if (pre == 1) hipLaunchKernelGGL(HIP_KERNEL_NAME(k_dec_lo_combine<true>), grid, dim3(64), 0, st, B, n, d_src, log2D, seed, T, scratch, acc, mean_n);
    else hipLaunchKernelGGL(HIP_KERNEL_NAME(k_dec_lo_combine<false>), grid, dim3(64), 0, st, B, n, d_src, log2D, seed, T, scratch, acc, mean_n);
}
void launch_finalize_mean(const float *acc, uint64_t d, uint32_t n, float *mean, hipStream_t st) {
    const int vec = ((reinterpret_cast<uintptr_t>(acc) | reinterpret_cast<uintptr_t>(mean)) & 15u) == 0;
    const uint64_t per_block = 256u * (vec ? 4u : 1u);
    const uint32_t blocks = (uint32_t)((d + per_block - 1) / per_block);
    hipLaunchKernelGGL(k_finalize_mean, dim3(blocks), dim3(256), 0, st, acc, d, (float)n, mean, vec);
}
void launch_pack_bits(const EncBatch &B, uint32_t n, int log2D, hipStream_t st) {          // multi-pass sizes: D >= 2^13
    const uint64_t groups = (1ull << log2D) / 32;
    hipLaunchKernelGGL(k_pack_bits, dim3((uint32_t)((groups + 255) / 256), n), dim3(256), 0, st, B, log2D);
}
void launch_unpack_bits(const DecBatch &B, uint32_t n, int log2D, uint8_t *codes_all, hipStream_t st) {
    const uint64_t groups = (1ull << log2D) / 32;
    hipLaunchKernelGGL(k_unpack_bits, dim3((uint32_t)((groups + 255) / 256), n), dim3(256), 0, st, B, log2D, codes_all);
}
void launch_fill_zero(float *p, uint64_t count, hipStream_t st) {
    hipLaunchKernelGGL(k_fill_zero, dim3((uint32_t)((count + 255) / 256)), dim3(256), 0, st, p, count);
}
void launch_byte_entropy(const uint8_t *bytes, uint64_t count, uint32_t *hist, double *out, hipStream_t st) {
    launch_fill_zero(reinterpret_cast<float *>(hist), 256, st);          // 256 words of zero bits
    uint32_t blocks = (uint32_t)((count + 4095) / 4096);
    if (blocks > 2048u) blocks = 2048u;
    if (blocks < 1u) blocks = 1u;
    hipLaunchKernelGGL(k_byte_histogram, dim3(blocks), dim3(256), 0, st, bytes, count, hist);
    hipLaunchKernelGGL(k_histogram_entropy, dim3(1), dim3(256), 0, st, hist, count, out);
}
void launch_sq_error(const float *a, const float *b, uint64_t d, double *partials, uint32_t max_parts, double *out,
                     hipStream_t st) {
    uint32_t blocks = (uint32_t)((d + 1023) / 1024);
    if (blocks > 1024u) blocks = 1024u;
    if (blocks > max_parts) blocks = max_parts;
    if (blocks < 1u) blocks = 1u;
    hipLaunchKernelGGL(k_sq_error, dim3(blocks), dim3(256), 0, st, a, b, d, partials);
    hipLaunchKernelGGL(k_sq_error_finish, dim3(1), dim3(256), 0, st, partials, blocks, out);
}
void launch_store_doubles(const double *src_host, uint32_t count, double *dst, hipStream_t st) {
    ArgDoubles a;
    for (uint32_t i = 0; i < (uint32_t)kArgDoubles; ++i) a.v[i] = i < count ? src_host[i] : 0.0;
    hipLaunchKernelGGL(k_store_doubles, dim3(1), dim3(kArgDoubles), 0, st, a, count, dst);
}
void launch_hash_bits(uint64_t key, uint64_t nwords, uint64_t *out, hipStream_t st) {
    hipLaunchKernelGGL(k_hash_bits, dim3((uint32_t)((nwords + 255) / 256)), dim3(256), 0, st, key, nwords, out);
}
void launch_loss_bitmap(uint64_t key, uint32_t npk, uint32_t drop_q32, uint32_t *bitmap, hipStream_t st) {
    const uint32_t nw = (npk + 31u) / 32u;
    hipLaunchKernelGGL(k_loss_bitmap, dim3((nw + 255) / 256), dim3(256), 0, st, key, npk, drop_q32, bitmap);
}

}  // namespace eden
