// The contiguous passes of D = 2^25 .. 2^27 (gfx950): 15 or 16 index bits, so that two passes through memory do (the strided pass
// takes the 10 or 11 bits above, eden_hix.h).
//
// A workgroup of 16 waves transforms 2^15 coordinates, 32 per thread, in three groups of five butterfly stages:
//
//   group 1   bits 10..14  v[a] = coordinate 1024 a + t (coalesced loads)
//   exchange  through LDS between all waves (registers <-> bits 5..9), 128 KiB
//   group 2   bits 5..9
//   exchange  through LDS inside halves of a wave (registers <-> bits 0..4)
//   group 3   bits 0..4
//
// Afterwards thread t holds the 32 consecutive coordinates 32 t + e.  HALVES (D = 2^27, 16 bits): two workgroups share a tile of
// 2^16; both read all of it, one transforms the sums of its halves, the other the differences (the stage over bit 15).  2^16
// values and as many sums over the senders would be the whole register file of a CU.  The pair runs at the same time on the same
// XCD (workgroups i and i + 8), so the second read of a line is meant to find it in that XCD's L2.
// (measured: the encoder's pass fetches every line from memory once).
// It replaces a 14-bit contiguous pass and a second strided pass (one more trip through memory per direction).  8 senders of 2^27,
// b = 4: this pass 1.96 ms (encode) and 1.10 ms (decode), the strided ones 1.37 and 1.39 ms (1.22 with touch_payload_ahead); a round 8.03 -> 5.85 ms; at 2^25
// 1.94 -> 1.16 ms, with b = 1 1.91 -> 0.91 ms.  With one workgroup per CU what is left is the time in which its waves all wait
// for memory or all compute (vector instructions 48%, 31% of the time).
#include "eden_device.h"
#include "eden_kernels.h"

namespace eden {

constexpr int kLo15Row = 36;                     // 32 values + 4: rows of consecutive lanes start 4 banks apart
constexpr int kLo15Wave = 64 * kLo15Row;         // one wave's region of the second exchange
constexpr int kLo15LdsWords = 16 * kLo15Wave;    // 147456 bytes; the first exchange needs 2^15 words
static_assert(kLo15LdsWords >= (1 << 15), "LDS sizing");

// in:  v[a] = coordinate 1024 a + t;  out: v[e] = coordinate 32 t + e, fully transformed over the 15 bits
__device__ __forceinline__ void lo15_forward32(float (&v)[32], float *lds) {
    const uint32_t t = threadIdx.x, lane = t & 63u, wv = t >> 6;
    fwht_regs<32>(v);                                            // bits 10..14
    uint32_t upper = (1u << 14) + t;                             // (an LDS instruction reaches 64 KiB beyond its address register)
    asm volatile("" : "+v"(upper));
#pragma unroll
    for (int a = 0; a < 16; ++a) lds[1024 * a + t] = v[a];
#pragma unroll
    for (int a = 0; a < 16; ++a) lds[upper + 1024u * a] = v[16 + a];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 32; ++r) v[r] = lds[1024u * (t >> 5) + 32u * r + (t & 31u)];
    fwht_regs<32>(v);                                            // bits 5..9
    __syncthreads();                                             // all reads done before the regions are reused
    float *L = lds + wv * kLo15Wave;
#pragma unroll
    for (int r = 0; r < 32; ++r) L[((lane & 32u) + (uint32_t)r) * kLo15Row + (lane & 31u)] = v[r];
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const float4 x = *reinterpret_cast<const float4 *>(&L[lane * kLo15Row + 4 * q]);
        v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
    }
    fwht_regs<32>(v);                                            // bits 0..4
}

// tile and half of a workgroup: pairs are 8 workgroups apart
template <bool HALVES>
__device__ inline void lo15_tile(uint32_t &tile, uint32_t &half) {
    tile = HALVES ? ((blockIdx.x >> 4) << 3) + (blockIdx.x & 7u) : blockIdx.x;
    half = HALVES ? (blockIdx.x >> 3) & 1u : 0u;
}

// Encode, first pass: x -> T (see k_enc_lo_first), always in the blocked layout.
template <bool PRE, bool HALVES>
__global__ __launch_bounds__(1024) void k_enc_lo15_first(EncBatch B, uint64_t d_src, int log2D, uint64_t seed, float *T,
                                                         double *partials, uint32_t partial_stride) {
    static_assert(!(PRE && HALVES), "a vector sparsified by pairs has at most 2^26 coordinates");
    constexpr int P = HALVES ? 16 : 15;
    __shared__ __attribute__((aligned(16))) float lds[kLo15LdsWords];
    __shared__ double red[16];
    const uint32_t c = blockIdx.y, t = threadIdx.x, lane = t & 63u, wv = wave_in_block();
    uint32_t tile, half;
    lo15_tile<HALVES>(tile, half);
    const rsrc_t rx = make_rsrc(B.x[c], (uint32_t)(d_src * 4));           // reads past d_src give the zero padding
    float u[32], w[HALVES ? 32 : 1];
    if constexpr (PRE) {
        const uint64_t offs = hash_word(stream_key(seed, kStreamSubsample, B.client[c]), ((uint64_t)tile << (P - 6)) + 16u * (lane & 31u) + wv);
#pragma unroll
        for (int a = 0; a < 32; ++a) {
            const uint32_t odd = __builtin_amdgcn_inverse_ballot_w64(wave_read64(offs, a)) ? 4u : 0u;
            u[a] = 2.0f * buf_load(rx, 8u * t + odd, (tile << (P + 3)) + 8192u * a);
        }
    } else {
#pragma unroll
        for (int a = 0; a < 32; ++a) u[a] = buf_load(rx, 4u * t, (tile << (P + 2)) + 4096u * a);
        if constexpr (HALVES) {
#pragma unroll
            for (int a = 0; a < 32; ++a) w[a] = buf_load(rx, 4u * t, (tile << (P + 2)) + (1u << 17) + 4096u * a);
        }
    }
    // register a of this wave = 64 consecutive coordinates = one sign word: lane a hashes the word of register a (lane 32 + a
    // that of the same register of the upper half)
    const uint64_t mine = hash_word(stream_key(seed, kStreamSign, B.client[c]),
                                    ((uint64_t)tile << (P - 6)) + 16u * (lane & 31u) + wv + (HALVES ? 512u * (lane >> 5) : 0u));
    const float side = half ? -1.0f : 1.0f;
    double n2 = 0.0;
#pragma unroll
    for (int a = 0; a < 32; ++a) {
        const float mine_only = HALVES && half ? w[HALVES ? a : 0] : u[a];       // each half of the tile is counted once
        n2 += (double)mine_only * (double)mine_only;
        if ((a & 7) == 7) __builtin_amdgcn_sched_barrier(0);     // keeps the widened values of one group live at a time
    }
#pragma unroll
    for (int a = 0; a < 32; ++a) {
        u[a] = negate_where(u[a], wave_read64(mine, a)) + 0.0f;  // + 0: no negative zeros
        if constexpr (HALVES) {
            const float upper = negate_where(w[a], wave_read64(mine, 32 + a)) + 0.0f;
            u[a] = fmaf(upper, side, u[a]);                      // the stage over bit 15 (one rounding)
        }
    }
    lo15_forward32(u, lds);
    store_runs<P, true>(u, lds + wv * kLo15Wave, T + ((size_t)c << log2D), tile, 1024u * half + 64u * wv);
    const double block_total = block_sum<1024>(n2, red);
    if (t == 0) partials[(size_t)c * partial_stride + blockIdx.x] = block_total;
}

// Decode, last pass (see k_dec_lo14_last): index bits 0..P-1 of H for every sender, its signs, the sum over the senders in
// registers, one contiguous read-modify-write of acc (mean_n > 0: acc is written with the sum divided by mean_n).  These sizes
// have at least 512 (half) tiles: no split by sender.
// KIND: kWide: no sender of the launch has an fp16 slot (every b > 1), kNarrow: every sender has one, kMixed.
enum : int { kMixed = 0, kWide = 1, kNarrow = 2 };
template <bool PRE, bool HALVES, int KIND>
__global__ __launch_bounds__(1024) void k_dec_lo15_last(DecBatch B, uint32_t n, uint64_t d_src, int log2D, uint64_t seed, const float *T,
                                                        const DecScratch *scratch, float *acc, float mean_n) {
    static_assert(!(PRE && HALVES), "a vector sparsified by pairs has at most 2^26 coordinates");
    constexpr int P = HALVES ? 16 : 15;
    constexpr int NS = PRE ? 64 : 32;                            // accumulator coordinates per thread
    __shared__ __attribute__((aligned(16))) float lds[kLo15LdsWords];
    const uint32_t t = threadIdx.x, lane = t & 63u, wv = wave_in_block();
    uint32_t tile, half;
    lo15_tile<HALVES>(tile, half);
    const uint64_t row = (uint64_t)tile << P;                    // first coordinate of the tile in a slot
    if (HALVES && row >= d_src) return;                          // (the grid has whole groups of 8 tiles)
    float sum[NS];
#pragma unroll
    for (int e = 0; e < NS; ++e) sum[e] = 0.0f;
    // (through a buffer descriptor: one offset register for all loads; with flat addresses the kernel spilled 44 registers, and
    // spilled registers go through memory)
    auto is_narrow = [&](uint32_t c) { return KIND == kNarrow || (KIND == kMixed && B.b_q8[c] <= 256u); };
    auto load = [&](uint32_t c, uint32_t at, float (&v)[32]) {
        // (beyond the last sender the bounds are 0: no branch around the loads, which would cost registers, and no traffic)
        const uint32_t cc = c < n ? c : 0u;
        const rsrc_t r = make_rsrc(T + ((size_t)cc << log2D), c < n ? 4u << log2D : 0u);     // the tile lies inside the slot
        if (is_narrow(cc)) {
#pragma unroll
            for (int a = 0; a < 32; ++a)
                v[a] = __int_as_float((int)__builtin_amdgcn_raw_buffer_load_b16(r, (int)(2u * t), (int)(2u * at + 2048u * a), kStream));
        } else {
#pragma unroll
            for (int a = 0; a < 32; ++a) v[a] = buf_load(r, 4u * t, 4u * at + 4096u * a);
        }
    };
    const float side = half ? -1.0f : 1.0f;
    float ahead[32];                                             // the next sender's (lower half of the) tile
    if (!PRE) load(0, (uint32_t)row, ahead);
    for (uint32_t c = 0; c < n; ++c) {
        const bool i16 = is_narrow(c);
        float u[32];
        if constexpr (PRE) load(c, (uint32_t)row, ahead);
        if constexpr (HALVES) load(c, (uint32_t)row + (1u << 15), u);
#pragma unroll
        for (int a = 0; a < 32; ++a) {
            const float low = i16 ? narrow_value((short)__float_as_int(ahead[a])) : ahead[a];
            if constexpr (HALVES) {
                const float up = i16 ? narrow_value((short)__float_as_int(u[a])) : u[a];
                u[a] = fmaf(up, side, low);                      // the stage over bit 15 (one rounding)
            } else {
                u[a] = low;
            }
        }
        __builtin_amdgcn_sched_barrier(0);                       // the conversions stay above the next sender's loads
        if (!PRE) load(c + 1, (uint32_t)row, ahead);
        lo15_forward32(u, lds);
        const uint32_t scale = __float_as_uint(i16 ? scratch[c].deq[1] : 1.0f) & 0x7FFFFFFFu;   // > 0; x*1+s is exact
        // the wave's 2048 coordinates use 32 sign words: lane l < 32 hashes word l, every thread fetches its own
        const uint64_t word0 = (row + ((uint64_t)half << 15) + 2048u * wv) >> 6;
        const uint64_t mine = hash_word(stream_key(seed, kStreamSign, B.client[c]), word0 + (lane & 31u));
        const uint32_t wlo = (uint32_t)__shfl((int)(uint32_t)mine, (int)(lane >> 1), 64);
        const uint32_t whi = (uint32_t)__shfl((int)(uint32_t)(mine >> 32), (int)(lane >> 1), 64);
        const uint32_t bits = (t & 1u) ? whi : wlo;              // 32 sign bits of this thread's run
        if constexpr (PRE) {
            const uint64_t omine = hash_word(stream_key(seed, kStreamSubsample, B.client[c]), word0 + (lane & 31u));
            const uint32_t olo = (uint32_t)__shfl((int)(uint32_t)omine, (int)(lane >> 1), 64);
            const uint32_t ohi = (uint32_t)__shfl((int)(uint32_t)(omine >> 32), (int)(lane >> 1), 64);
            const uint32_t offs = (t & 1u) ? ohi : olo;          // which member of each of this thread's 32 pairs
#pragma unroll
            for (int e = 0; e < 32; ++e) {
                const float val = u[e] * __uint_as_float(scale | ((bits << (31 - e)) & 0x80000000u));
                const bool odd = (offs >> e) & 1u;
                sum[2 * e] += odd ? 0.0f : val;
                sum[2 * e + 1] += odd ? val : 0.0f;
            }
        } else {
#pragma unroll
            for (int e = 0; e < 32; ++e) {
                // hash bit 1 -> s_i = -1: the factor is the scale with bit e of the sign word moved to the sign position
                const uint32_t shifted = bits << (31 - e);
                sum[e] = fmaf(u[e], __uint_as_float((scale & 0x7FFFFFFFu) | (shifted & 0x80000000u)), sum[e]);
            }
        }
        __syncthreads();                                         // LDS is reused by the next sender
    }
    // The wave's 64 runs of NS coordinates go out as whole 128-byte lines, eight lanes a line, through its region of the LDS (quads
    // swizzled as in store_runs): with a run per lane every line was touched by eight instructions, and read from L2 as often
    // (whole decode: one sender of 5 * 10^7 sparsified by pairs, added to acc, 244 -> 98 us; of 10^8 466 -> 228; 4 senders of 2^27, b = 4,
    // 1483 -> 1384).
    const bool overwrite = mean_n > 0.0f;
    const float div = overwrite ? mean_n : 1.0f;
    const uint64_t out0 = (PRE ? 2u : 1u) * (row + ((uint64_t)half << 15) + 2048u * wv);     // the wave's first coordinate of acc
    float *L = lds + wv * kLo15Wave;
    const uint32_t swz = lane & 7u;
#pragma unroll
    for (int h = 0; h < NS / 32; ++h) {
        wave_lds_sync();
#pragma unroll
        for (int q = 0; q < 8; ++q)
            *reinterpret_cast<float4 *>(&L[lane * 32u + 4u * ((uint32_t)q ^ swz)]) =
                make_float4(sum[32 * h + 4 * q], sum[32 * h + 4 * q + 1], sum[32 * h + 4 * q + 2], sum[32 * h + 4 * q + 3]);
        wave_lds_sync();
        auto place = [&](int j) {                                // this lane's quad of turn j: run 8 j + lane / 8
            const uint32_t run = 8u * (uint32_t)j + (lane >> 3);
            return out0 + run * (uint32_t)NS + 32u * (uint32_t)h + 4u * (swz ^ (run & 7u));
        };
        float4 a[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            a[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            const uint64_t at = place(j);
            if (!overwrite && at + 4 <= d_src) a[j] = *reinterpret_cast<const float4 *>(acc + at);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint64_t at = place(j);
            const float4 x = *reinterpret_cast<const float4 *>(&L[(8u * (uint32_t)j + (lane >> 3)) * 32u + 4u * swz]);
            if (at + 4 <= d_src) {
                *reinterpret_cast<float4 *>(acc + at) = make_float4((a[j].x + x.x) / div, (a[j].y + x.y) / div, (a[j].z + x.z) / div,
                                                                    (a[j].w + x.w) / div);
            } else {
                const float v[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (at + e < d_src) acc[at + e] = ((overwrite ? 0.0f : acc[at + e]) + v[e]) / div;
            }
        }
    }
}

// tiles of 2^P coordinates that reach below d; for P = 16 rounded up to whole groups of 8 (see lo15_tile), for the encoder to
// whole blocks of rows of the blocked layout
static uint32_t lo15_tiles(uint64_t d, int P, uint32_t group) {
    const uint32_t tiles = (uint32_t)((d + (1ull << P) - 1) >> P);
    return (tiles + group - 1) / group * group;
}

uint32_t launch_enc_lo15_first(int P, const EncBatch &B, uint32_t n, uint64_t d_src, int pre, int log2D, uint64_t seed, float *T,
                               double *partials, uint32_t partial_stride, hipStream_t st) {
    const uint64_t d = pre ? (d_src + 1) / 2 : d_src;
    const dim3 grid(P == 16 ? 2 * lo15_tiles(d, 16, 8) : lo15_tiles(d, 15, kBlockRows), n);
    if (P == 16)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_enc_lo15_first<false, true>), grid, dim3(1024), 0, st, B, d_src, log2D, seed, T, partials, partial_stride);
    else if (pre)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_enc_lo15_first<true, false>), grid, dim3(1024), 0, st, B, d_src, log2D, seed, T, partials, partial_stride);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_enc_lo15_first<false, false>), grid, dim3(1024), 0, st, B, d_src, log2D, seed, T, partials, partial_stride);
    return grid.x;
}
void launch_dec_lo15_last(int P, const DecBatch &B, uint32_t n, uint64_t d_src, int pre, int log2D, uint64_t seed, const float *T,
                          const DecScratch *scratch, float *acc, float mean_n, hipStream_t st) {
    const uint64_t d = pre ? (d_src + 1) / 2 : d_src;
    const dim3 grid(P == 16 ? 2 * lo15_tiles(d, 16, 8) : lo15_tiles(d, 15, 1));
    bool wide = true, small = true;                              // no sender, every sender with an fp16 slot
    for (uint32_t c = 0; c < n; ++c) { wide = wide && B.b_q8[c] > 256u; small = small && B.b_q8[c] <= 256u; }
#define EDEN_DEC_LO15(PRE, HALVES, KIND) \
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_dec_lo15_last<PRE, HALVES, KIND>), grid, dim3(1024), 0, st, B, n, d_src, log2D, seed, T, scratch, acc, mean_n)
    if (P == 16) { if (wide) EDEN_DEC_LO15(false, true, kWide); else if (small) EDEN_DEC_LO15(false, true, kNarrow); else EDEN_DEC_LO15(false, true, kMixed); }
    else if (pre) EDEN_DEC_LO15(true, false, kNarrow);           // (these senders have b = 1)
    else { if (wide) EDEN_DEC_LO15(false, false, kWide); else if (small) EDEN_DEC_LO15(false, false, kNarrow); else EDEN_DEC_LO15(false, false, kMixed); }
#undef EDEN_DEC_LO15
}

}  // namespace eden
