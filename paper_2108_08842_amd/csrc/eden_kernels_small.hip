// D <= 4096: one sender is one workgroup (encode) or one team of waves of a workgroup (decode), the vector in registers.
//
// A round at these sizes is all latency: a few KiB per sender, so what counts is the number of launches, the length of the
// dependent chain inside a kernel and how many senders run side by side.  A sender gets max(1, D / 256) waves with four
// values per lane, value (register r, wave w, lane l) = coordinate 64 (w + W r) + l: loads are coalesced, a register of
// a wave is 64 consecutive coordinates = one word of the hash streams, and a ballot of an index bit is 64 payload bits.
// The transform runs over the lane bits by cross-lane exchanges (six stages), over the two top bits in registers, and
// over the wave bits in registers after one (W <= 4) or two (W = 8, 16) exchanges through LDS: at most two barriers, where one
// stage per barrier in LDS took ten to twelve.
#include "eden_device.h"
#include "eden_kernels.h"

namespace eden {

// block of 64 coordinates that register r of wave w holds before (in) and after (out) the transform; W waves per sender
template <int W> __device__ inline uint32_t small_block_in(uint32_t w, uint32_t r) { return w + (uint32_t)W * r; }
template <int W> __device__ inline uint32_t small_block_out(uint32_t w, uint32_t q) {
    if constexpr (W == 1) return q;
    else if constexpr (W <= 4) return q + 4u * w;
    else return (w & 3u) + 4u * q + 16u * (w >> 2);
}

// one butterfly stage over lane bit X of every register
template <int X>
__device__ inline float lane_butterfly(float v, bool upper) {
    const float sign = upper ? -1.0f : 1.0f;
    float other;
    if constexpr (X <= 8) other = __uint_as_float(lane_xor_u32<X>(__float_as_uint(v)));
    else if constexpr (X == 16) other = __uint_as_float((uint32_t)__builtin_amdgcn_ds_swizzle((int)__float_as_uint(v), 0x001F | (16 << 10)));
    else other = __shfl_xor(v, 32, 64);
    return fmaf(v, sign, other);                                 // lower lane a + b, upper lane a - b, rounded once
}
template <int X>
__device__ inline void lane_stage(float (&v)[4], uint32_t lane) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = lane_butterfly<X>(v[r], (lane & (uint32_t)X) != 0u);
}
__device__ inline void reg_stage0(float (&v)[4]) {
    const float a = v[0], b = v[1], c = v[2], e = v[3];
    v[0] = a + b; v[1] = a - b; v[2] = c + e; v[3] = c - e;
}
__device__ inline void reg_stage1(float (&v)[4]) {
    const float a = v[0], b = v[1], c = v[2], e = v[3];
    v[0] = a + c; v[2] = a - c; v[1] = b + e; v[3] = b - e;
}
// H over log2D bits (log2D = 8 + log2 W for W > 1).  `lds`: 256 W floats of this sender; every thread of the workgroup calls
// it.  A thread reads back exactly the places it wrote before a second exchange, so one barrier per exchange is enough.
template <int W>
__device__ inline void small_fwht(float (&v)[4], int log2D, float *lds, uint32_t w, uint32_t lane) {
    if constexpr (W == 1) {
        if (log2D > 0) lane_stage<1>(v, lane);
        if (log2D > 1) lane_stage<2>(v, lane);
        if (log2D > 2) lane_stage<4>(v, lane);
        if (log2D > 3) lane_stage<8>(v, lane);
        if (log2D > 4) lane_stage<16>(v, lane);
        if (log2D > 5) lane_stage<32>(v, lane);
        if (log2D > 6) reg_stage0(v);
        if (log2D > 7) reg_stage1(v);
    } else {
        lane_stage<1>(v, lane); lane_stage<2>(v, lane); lane_stage<4>(v, lane);
        lane_stage<8>(v, lane); lane_stage<16>(v, lane); lane_stage<32>(v, lane);
        reg_stage0(v); reg_stage1(v);
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) lds[64u * small_block_in<W>(w, r) + lane] = v[r];
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) v[q] = lds[64u * (q + 4u * w) + lane];
        reg_stage0(v);
        if constexpr (W >= 4) reg_stage1(v);
        if constexpr (W >= 8) {
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) lds[64u * (q + 4u * w) + lane] = v[q];
            __syncthreads();
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) v[q] = lds[64u * small_block_out<W>(w, q) + lane];
            reg_stage0(v);
            if constexpr (W == 16) reg_stage1(v);
        }
    }
}
// The hash words of the four blocks of 64 coordinates a wave holds: lane q < 4 hashes the word of register q.
template <int W, bool OUT>
__device__ inline uint64_t small_words(uint64_t key, uint32_t w, uint32_t lane) {
    const uint32_t q = lane & 3u;
    return hash_word(key, OUT ? small_block_out<W>(w, q) : small_block_in<W>(w, q));
}
template <int BITS>
__device__ inline uint32_t small_pack_word(const uint8_t *code, uint32_t w, uint32_t D) {       // payload bits 32 w .. 32 w + 31
    uint32_t word = 0;
    const uint32_t first = 32u * w / (uint32_t)BITS;
    const int shift = (int)(first * (uint32_t)BITS) - (int)(32u * w);        // <= 0: the first index may straddle the word
#pragma unroll
    for (int e = 0; e < (32 + BITS - 1) / BITS + 1; ++e) {
        const uint32_t j = first + (uint32_t)e;
        const int at = shift + e * BITS;
        if (at < 32 && j < D) {
            const uint32_t v = (uint32_t)code[j] & ((1u << BITS) - 1u);
            word |= at >= 0 ? v << at : v >> -at;
        }
    }
    return word;
}

// Encode (Sec. 2.2.1, 2.3, 4.1): pad, signs, |x|^2, transform, quantize, <R(x),Q>, pack, header, one launch.
// (n = 4, D = 1024, b = 1: 4.2 us, against 12.1 us with the vector in LDS and one barrier per stage.)
template <int W>
__global__ __launch_bounds__(64 * W) void k_enc_small(EncBatch B, uint64_t d, int pre, uint64_t hdr_d, int log2D, uint64_t seed,
                                                      const DevTables *tab, uint32_t *dev_status) {
    constexpr uint32_t T = 64u * W;
    __shared__ float buf[256 * W];
    __shared__ __attribute__((aligned(8))) uint8_t code[256 * W];
    __shared__ double red_n2[W], red_ip[W];
    __shared__ EncScratch s;
    __shared__ uint32_t coin_words[8 * W + 2];                   // coin budgets: the second part of the payload
    __shared__ uint32_t coin_count[4 * W];                       // ... and the coins of every block of 64 coordinates
    const uint32_t c = blockIdx.x, lane = lane_id(), w = wave_in_block();
    const uint32_t D = 1u << log2D;
    const uint32_t b_q8 = B.b_q8[c];
    const float *x = B.x[c];
    float v[4];
    if (pre) {                                                   // Sec. 4.1: x'[i] = 2 x[2i + o_i], sparsification before the rotation
        const uint64_t offs = small_words<W, false>(stream_key(seed, kStreamSubsample, B.client[c]), w, lane);
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const uint64_t i = 64u * small_block_in<W>(w, r) + lane, src = 2u * i + ((wave_read64(offs, (int)r) >> lane) & 1ull);
            v[r] = src < d ? 2.0f * x[src] : 0.0f;
        }
    } else {
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const uint32_t i = 64u * small_block_in<W>(w, r) + lane;
            v[r] = i < d ? x[i] : 0.0f;
        }
    }
    const uint64_t signs = small_words<W, false>(stream_key(seed, kStreamSign, B.client[c]), w, lane);
    double n2p = 0.0;
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r) {
        n2p += (double)v[r] * (double)v[r];
        v[r] = negate_where(v[r], wave_read64(signs, (int)r)) + 0.0f;        // + 0: no negative zeros
    }
    n2p = wave_sum(n2p);
    if (lane == 0) red_n2[w] = n2p;
    small_fwht<W>(v, log2D, buf, w, lane);
    if (W == 1) wave_lds_sync();
    double n2 = 0.0;
#pragma unroll
    for (int i = 0; i < W; ++i) n2 += red_n2[i];                 // in wave order, the same in every thread
    int bits, k;
    budget_of(b_q8, bits, k);
    const bool mix = budget_mixed(b_q8);                         // b = k + 1/2: one coordinate of every pair uses I_{k+1}
    const uint32_t coin_frac = coin_q8(b_q8) & 255u;             // coin budgets: a coordinate with a coin uses I_{k+1}
    const bool bytes = byte_budget(b_q8);                        // uniform grid (Sec. 4.3) or b = 5..8: one-byte indices
    const bool signs_only = b_q8 <= 256u;                        // I_1: the index is the sign
    float ip = 0.0f;
    uint64_t top[4] = {0, 0, 0, 0}, coins[4] = {0, 0, 0, 0};     // mixed and coin budgets: top bits and coins of the blocks
    if (signs_only) {
#pragma unroll
        for (int q = 0; q < 4; ++q) ip = fmaf(fabsf(v[q]), kQ1, ip);
    } else {
        fill_enc_scratch(&s, n2, b_q8, tab, threadIdx.x);
        for (uint32_t i = threadIdx.x; i <= (uint32_t)kGridMax; i += T) fill_byte_tables(&s, b_q8, n2, tab, i);
        __syncthreads();
        const int H = 1 << (bits - 1);
        const uint64_t mixkey = stream_key(seed, kStreamMix, B.client[c]);
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const uint32_t blk = small_block_out<W>(w, q), i = 64u * blk + lane;
            uint32_t idx;
            if (bytes) {                                         // grid_c and wide_thr are adjacent
                idx = grid_q15(b_q8) ? quantize_byte<true>(v[q], 0u, s.grid_inv, s.grid_c, ip)
                                     : quantize_byte<false>(v[q], wide_half_levels(b_q8), 0.0f, s.grid_c, ip);
            } else {
                const float a = fabsf(v[q]);
                bool up = false;
                if (mix) up = ((hash_word(mixkey, blk >> 1) >> ((i >> 1) & 63u)) & 1ull) == (i & 1u);
                else if (coin_frac) up = coin_of(mixkey, i, coin_frac) && i < D;
                const float *thr = up ? s.thr2 : s.thr, *qp = up ? s.qpos2 : s.qpos;
                const int Hu = up ? 2 * H : H;
                uint32_t mag = 0;
                for (int t = 1; t < Hu; ++t) mag = (a > thr[t]) ? (uint32_t)t : mag;
                ip = fmaf(a, qp[mag], ip);
                idx = (__float_as_uint(v[q]) >> 31) ? (uint32_t)(Hu - 1) - mag : (uint32_t)Hu + mag;
                if (mix || coin_frac) top[q] = __ballot(i < D && up && ((idx >> bits) & 1u));
                if (coin_frac) coins[q] = __ballot(up);
            }
            code[i] = (uint8_t)idx;
            if (coin_frac && lane == 0) coin_count[blk] = (uint32_t)__popcll(coins[q]);
        }
    }
    if (coin_frac)
        for (uint32_t i = threadIdx.x; i < 8u * W + 2u; i += T) coin_words[i] = 0u;
    const double ipw = wave_sum((double)ip);
    if (lane == 0) red_ip[w] = ipw;
    __syncthreads();                                             // also publishes the codes and the counts of the coins
    double ipt = 0.0;
#pragma unroll
    for (int i = 0; i < W; ++i) ipt += red_ip[i];
    // (a uniform grid so coarse that every coordinate falls into the interval around 0 leaves <R(x),Q> = 0)
    const bool valid = (n2 > 0.0) && (n2 < INFINITY) && (ipt > 0.0);
    uint32_t *payload = reinterpret_cast<uint32_t *>(static_cast<char *>(B.msg[c]) + EDEN_HEADER_BYTES);
    const uint32_t nsent = D / (uint32_t)k;                      // transmitted indices
    const uint32_t nwords = 2u * ((nsent * (uint32_t)bits + 63u) / 64u);
    if (signs_only) {
        // lane q takes the 64 sign bits of register q (index 1 = non-negative; bits beyond D are padding: zero)
        const uint64_t inside = D >= 64u ? ~0ull : (1ull << D) - 1ull;
        uint64_t mine = 0;
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const uint64_t m = __ballot((__float_as_uint(v[q]) >> 31) == 0u) & inside;
            if (lane == q) mine = m;
        }
        if (!valid) mine = 0;
        const uint32_t blk = small_block_out<W>(w, lane & 3u);
        if (lane < 4u && (64u * blk < D)) {
            if (k == 1) {
                *reinterpret_cast<uint2 *>(payload + 2u * blk) = make_uint2(lo32(mine), hi32(mine));
            } else {                                             // b = 1/2: of every pair the coordinate the SUBSAMPLE stream picks
                const uint32_t off = (uint32_t)(hash_word(stream_key(seed, kStreamSubsample, B.client[c]), blk >> 1) >> (32u * (blk & 1u)));
                const uint32_t ev = even_bits(lo32(mine)) | (even_bits(hi32(mine)) << 16);
                const uint32_t od = even_bits(lo32(mine) >> 1) | (even_bits(hi32(mine) >> 1) << 16);
                payload[blk] = (ev & ~off) | (od & off);
                if (D <= 64u) payload[1] = 0u;                   // the payload is a whole number of 64-bit words
            }
        }
    } else {
        for (uint32_t i = threadIdx.x; i < nwords; i += T) {
            uint32_t word;
            switch (bits) {
                case 1: word = small_pack_word<1>(code, i, D); break;
                case 2: word = small_pack_word<2>(code, i, D); break;
                case 3: word = small_pack_word<3>(code, i, D); break;
                case 4: word = small_pack_word<4>(code, i, D); break;
                case 5: word = small_pack_word<5>(code, i, D); break;
                case 6: word = small_pack_word<6>(code, i, D); break;
                case 7: word = small_pack_word<7>(code, i, D); break;
                default: word = small_pack_word<8>(code, i, D); break;
            }
            payload[i] = valid ? word : 0u;
        }
    }
    if (mix) {                                                   // second part: the top bit of every pair's finer index
        uint64_t mine = 0;
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q)
            if (lane == q) mine = top[q];                        // only the chosen coordinate of a pair can have the bit
        if (!valid) mine = 0;
        const uint32_t blk = small_block_out<W>(w, lane & 3u);
        if (lane < 4u && 64u * blk < D) {
            payload[nwords + blk] = even_bits(lo32(mine) | (lo32(mine) >> 1)) | (even_bits(hi32(mine) | (hi32(mine) >> 1)) << 16);
            if (D <= 64u) payload[nwords + 1u] = 0u;
        }
    }
    uint32_t extra_bits = 0;
    if (coin_frac) {
        // second part: the top bits of the coordinates with a coin, in coordinate order: every lane with a set bit places it.
        // Coins before a block: a scan over the (at most 64) blocks, one per lane.
        const uint32_t blocks = W == 1 ? (D + 63u) / 64u : 4u * (uint32_t)W;
        uint32_t incl = lane < blocks ? coin_count[lane] : 0u;
        const uint32_t own = incl;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t t = (uint32_t)__shfl_up((int)incl, o, 64);
            if (lane >= (uint32_t)o) incl += t;
        }
        extra_bits = __builtin_amdgcn_readlane(incl, 63);
        const uint32_t before = incl - own;
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const uint32_t blk = small_block_out<W>(w, q);
            const uint32_t at = (uint32_t)__shfl((int)before, (int)(blk & 63u), 64) + lanes_below(coins[q]);
            if ((top[q] >> lane) & 1ull) atomicOr(&coin_words[at >> 5], 1u << (at & 31u));
        }
        __syncthreads();
        const uint32_t nwords_b = 2u * ((extra_bits + 63u) / 64u);
        for (uint32_t i = threadIdx.x; i < nwords_b; i += T) payload[nwords + i] = valid ? coin_words[i] : 0u;
    }
    if (threadIdx.x == 0) {
        MsgHeader h;
        h.magic = kMagic; h.log2D = (uint32_t)log2D; h.d = hdr_d; h.b_q8 = B.hdr_b_q8[c]; h.client = B.client[c];
        h.extra_bits = extra_bits; h.seed = seed; h.N2 = n2;
        if (valid) {
            h.IP = ipt * exp2(-0.5 * (double)log2D);             // <R(x),Q> = D^-1/2 sum u_i q_i
            h.S = n2 / h.IP;                                     // Sec. 2.3
            h.status = 0;
        } else {
            h.IP = 0.0; h.S = 0.0;
            h.status = (n2 >= 0.0 && n2 < INFINITY) ? EDEN_DEV_ZERO_VECTOR : EDEN_DEV_NONFINITE;
            atomicOr(dev_status, h.status);
        }
        *static_cast<MsgHeader *>(B.msg[c]) = h;
    }
}

// Decode (Sec. 2.2.2, 4.2): a workgroup holds up to 16 / W senders, one per team of W waves; their vectors are added through
// LDS, in the order of the senders.  With more senders than one workgroup holds, every workgroup leaves its sum in `partial`
// and the last one to finish adds the sums in order and touches acc (one launch, and the result does not depend on
// which one that is).  (n = 4, D = 1024: 8.1 us, against 29.8 us when one workgroup took the senders one after the other;
// n = 16, D = 4096: 13.6 us.)  What is left is the chain header -> scale -> table -> transform, not work.
// pre == 1 (EDEN_B_HALF_PRE): value i of a sender belongs at 2 i + o_i of the output.  pre == 2: nothing is summed, sender c's
// vector goes to slots + (c << log2D).  mean_n > 0: acc is written with (0 + sum) / mean_n instead of added to.
template <int W>
__global__ __launch_bounds__(1024) void k_dec_small(DecBatch B, uint32_t n, uint64_t d, int pre, uint64_t hdr_d, int log2D,
                                                    uint64_t seed, const DevTables *tab, int any_coin, float *acc, float mean_n,
                                                    float *slots, float *partial, uint32_t *arrived, uint32_t turn, uint32_t *dev_status,
                                                    uint32_t *msg_flags) {
    constexpr uint32_t TEAMS = 16u / W, T = 64u * W;
    __shared__ float buf[8192];                                  // 256 floats per wave; the senders' results (pre == 1: twice as many)
    __shared__ DecScratch scr[TEAMS];
    __shared__ uint64_t coin_mask[64];                           // coin budgets: coins of every block of 64 coordinates, per team
    __shared__ uint32_t last_flag;
    const uint32_t lane = lane_id(), wave = wave_in_block(), team = wave / (uint32_t)W, w = wave % (uint32_t)W;
    const uint32_t teams = blockDim.x / T;                       // of this launch
    const uint32_t c = blockIdx.x * teams + team;
    const bool active = c < n;                                   // the same for a whole team
    const uint32_t cc = active ? c : 0u;
    const uint32_t D = 1u << log2D;
    const uint32_t b_q8 = B.b_q8[cc];
    const uint64_t mixkey = stream_key(seed, kStreamMix, B.client[cc]);
    const uint32_t coin_frac = active ? coin_q8(b_q8) & 255u : 0u;
    DecScratch &s = scr[team];
    uint32_t extra_bits = 0, coins_before_block = 0;
    if (any_coin) {                                              // the receiver draws the same coins and counts them
        if (coin_frac) {
#pragma unroll
            for (uint32_t r = 0; r < 4; ++r) {
                const uint32_t blk = small_block_in<W>(w, r), i = 64u * blk + lane;
                const uint64_t m = __ballot(i < D && coin_of(mixkey, i, coin_frac));
                if (lane == 0) coin_mask[team * 4u * W + blk] = m;
            }
        }
        __syncthreads();
        if (coin_frac) {
            const uint32_t own = lane < 4u * W ? (uint32_t)__popcll(coin_mask[team * 4u * W + lane]) : 0u;
            uint32_t incl = own;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t t = (uint32_t)__shfl_up((int)incl, o, 64);
                if (lane >= (uint32_t)o) incl += t;
            }
            extra_bits = __builtin_amdgcn_readlane(incl, 63);
            coins_before_block = incl - own;                     // lane b: before block b
        }
    }
    int bits, k;
    budget_of(b_q8, bits, k);
    const uint32_t *payload = reinterpret_cast<const uint32_t *>(static_cast<const char *>(B.msg[cc]) + EDEN_HEADER_BYTES);
    const uint32_t nwords = 2u * (((D / (uint32_t)k) * (uint32_t)bits + 63u) / 64u);
    const bool mix = budget_mixed(b_q8);
    // the payload words are on their way while the first wave of the team looks at the header
    uint32_t w0[4] = {0, 0, 0, 0}, w1[4] = {0, 0, 0, 0}, wb[4] = {0, 0, 0, 0};
    const uint64_t offs = k == 2 ? hash_word(stream_key(seed, kStreamSubsample, B.client[cc]), small_block_in<W>(w, lane & 3u) >> 1) : 0ull;
    const uint64_t pairs = mix ? hash_word(mixkey, small_block_in<W>(w, lane & 3u) >> 1) : 0ull;
    if (active) {
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const uint32_t i = 64u * small_block_in<W>(w, r) + lane;
            if (i < D) {
                const uint32_t at = ((k == 2 ? i >> 1 : i) * (uint32_t)bits) >> 5;
                w0[r] = payload[at];
                w1[r] = at + 1u < nwords ? payload[at + 1u] : 0u;            // an index may straddle two words
                if (mix) wb[r] = payload[nwords + (i >> 6)];
            }
        }
        if (w == 0)
            dec_prepare_wave(B.msg[cc], B.bitmap[cc], B.client[cc], b_q8, B.hdr_b_q8[cc], hdr_d, log2D, seed, tab, &s, dev_status,
                             extra_bits, msg_flags ? msg_flags + c : nullptr);
    }
    __syncthreads();
    float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (active) {
        const uint32_t *bm = B.bitmap[cc];
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const uint32_t blk = small_block_in<W>(w, r), i = 64u * blk + lane;
            if (i >= D) continue;
            bool here = true;
            if (bm) here = (bm[blk >> 9] >> ((blk >> 4) & 31u)) & 1u;        // packet i >> 10
            if (k == 2) here = here && (((wave_read64(offs, (int)r) >> ((i >> 1) & 63u)) & 1ull) == (i & 1u));
            const uint32_t idx = code_at(w0[r], w1[r], ((k == 2 ? i >> 1 : i) * (uint32_t)bits) & 31u, bits);
            float val = grid_q15(b_q8) ? dequantize_byte<true>(idx, 0u, s.grid_deq)
                      : wide_bits(b_q8) ? dequantize_byte<false>(idx, wide_half_levels(b_q8), s.grid_deq) : s.deq[idx & 15u];
            if (mix && ((wave_read64(pairs, (int)r) >> ((i >> 1) & 63u)) & 1ull) == (i & 1u))
                val = s.deq2[(((wb[r] >> ((i >> 1) & 31u)) & 1u) << bits) | idx];
            if (coin_frac) {
                const uint64_t m = coin_mask[team * 4u * W + blk];
                const uint32_t rank = (uint32_t)__shfl((int)coins_before_block, (int)blk, 64) + lanes_below(m);
                if ((m >> lane) & 1ull) val = s.deq2[(((payload[nwords + (rank >> 5)] >> (rank & 31u)) & 1u) << bits) | idx];
            }
            v[r] = here ? val : 0.0f;
        }
    }
    small_fwht<W>(v, log2D, buf + team * 256u * W, w, lane);
    const uint64_t signs = small_words<W, true>(stream_key(seed, kStreamSign, B.client[cc]), w, lane);
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = negate_where(v[q], wave_read64(signs, q));
    if (pre == 2) {
        if (active) {
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) {
                const uint32_t i = 64u * small_block_out<W>(w, q) + lane;
                if (i < D) slots[((size_t)c << log2D) + i] = v[q];
            }
        }
        return;
    }
    const uint32_t stride = pre ? 2u * D : D;                    // outputs per sender
    __syncthreads();                                             // the exchanges of the transform have been read
    if (pre) {
        const uint64_t which = small_words<W, true>(stream_key(seed, kStreamSubsample, B.client[cc]), w, lane);
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const uint32_t i = 64u * small_block_out<W>(w, q) + lane;
            const bool odd = (wave_read64(which, (int)q) >> lane) & 1ull;
            if (i < D) {
                buf[team * stride + 2u * i] = odd ? 0.0f : v[q];
                buf[team * stride + 2u * i + 1u] = odd ? v[q] : 0.0f;
            }
        }
    } else {
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const uint32_t i = 64u * small_block_out<W>(w, q) + lane;
            if (i < D) buf[team * stride + i] = v[q];
        }
    }
    __syncthreads();
    const uint32_t here = n - blockIdx.x * teams < teams ? n - blockIdx.x * teams : teams;      // senders of this workgroup
    const bool one_block = gridDim.x == 1;
    const float div = mean_n > 0.0f ? mean_n : 1.0f;
    for (uint32_t i = threadIdx.x; i < stride; i += blockDim.x) {
        float sum = 0.0f;
        for (uint32_t t = 0; t < here; ++t) sum += buf[t * stride + i];
        if (!one_block) store_through(partial + (size_t)blockIdx.x * stride + i, sum);
        else if (i < d) acc[i] = ((mean_n > 0.0f ? 0.0f : acc[i]) + sum) / div;
    }
    if (one_block) return;
    // Calls that overlapped against the rules may leave a counter non-zero, and with it this launch would add too early or never.
    // The launches of a context take the counters in turn and clear all but their own, so the calls after such an overlap
    // find theirs at 0.  (A captured launch keeps its counter: any other decode of the context clears it.)
    if (blockIdx.x == 0 && threadIdx.x < kDecCounters && threadIdx.x != turn) arrived[threadIdx.x] = 0u;
    if (!arrive_last(arrived + turn, gridDim.x, &last_flag)) return;
    for (uint32_t i = threadIdx.x; i < stride && i < d; i += blockDim.x) {
        float sum = 0.0f;
        for (uint32_t g = 0; g < gridDim.x; g += 8) {            // eight loads in flight: one after the other took 1 us each
            float part[8];
#pragma unroll
            for (uint32_t e = 0; e < 8; ++e) part[e] = g + e < gridDim.x ? load_through(partial + (size_t)(g + e) * stride + i) : 0.0f;
#pragma unroll
            for (uint32_t e = 0; e < 8; ++e) sum = g + e < gridDim.x ? sum + part[e] : sum;
        }
        acc[i] = ((mean_n > 0.0f ? 0.0f : acc[i]) + sum) / div;
    }
}

// waves per sender: four values per lane
#define EDEN_SMALL_SWITCH(CALL)                           \
    switch (log2D) {                                      \
        case 12: { constexpr int W = 16; CALL; } break;   \
        case 11: { constexpr int W = 8; CALL; } break;    \
        case 10: { constexpr int W = 4; CALL; } break;    \
        case 9: { constexpr int W = 2; CALL; } break;     \
        default: { constexpr int W = 1; CALL; } break;    \
    }

void launch_enc_small(const EncBatch &B, uint32_t n, uint64_t d, int pre, uint64_t hdr_d, int log2D, uint64_t seed,
                      const DevTables *tab, uint32_t *dev_status, hipStream_t st) {
    EDEN_SMALL_SWITCH(hipLaunchKernelGGL(HIP_KERNEL_NAME(k_enc_small<W>), dim3(n), dim3(64 * W), 0, st, B, d, pre, hdr_d, log2D, seed,
                                         tab, dev_status))
}
void launch_dec_small(const DecBatch &B, uint32_t n, uint64_t d, int pre, uint64_t hdr_d, int log2D, uint64_t seed,
                      const DevTables *tab, float *acc, float mean_n, float *slots, float *partial, uint32_t *arrived, uint32_t turn,
                      uint32_t *dev_status, uint32_t *msg_flags, hipStream_t st) {
    int any_coin = 0;
    for (uint32_t c = 0; c < n; ++c) any_coin |= coin_q8(B.b_q8[c]) != 0u;
    const uint32_t waves = log2D > 8 ? 1u << (log2D - 8) : 1u;
    const uint32_t teams = n < 16u / waves ? n : 16u / waves;    // senders per workgroup of at most 1024 threads
    dim3 grid((n + teams - 1) / teams), block(64u * waves * teams);
    EDEN_SMALL_SWITCH(hipLaunchKernelGGL(HIP_KERNEL_NAME(k_dec_small<W>), grid, block, 0, st, B, n, d, pre, hdr_d, log2D, seed, tab,
                                         any_coin, acc, mean_n, slots, partial, arrived, turn, dev_status, msg_flags))
}

}  // namespace eden
