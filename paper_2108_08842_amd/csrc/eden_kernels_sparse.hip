// b = m/64: sparsification before the rotation with p = m/64 (Sec. 4.1).  Of every block of 64 consecutive coordinates the m
// with the smallest (key, position) pairs are kept, the 16-bit key of coordinate i being bits 16 (i & 3) .. +15 of word i >> 2
// of the SPARSE stream; a kept coordinate's slot is block * m + its rank among the kept ones in position order.
//
// Both directions are the same selection (vector instructions) around a copy (memory).  A lane looks after one block: it
// hashes the block's 16 words, transposes the 64 keys into 16 bit planes (16 x 16 bits in both halves of a register at once,
// four swap steps) and walks the planes from the top bit: of the candidates that still agree with the threshold, those with a
// 0 in this plane are counted; if they are at least as many as are still to be kept, the others are out, otherwise
// they are all kept and the search goes on among the others.  About 750 issue slots per wave of 64 blocks, 320 of them the hash
// (1000 and 110 registers while the compiler chose the forms of the masks and multiplied the counter anew for every word; now 46
// registers); a bitonic sort of the keys across lanes took 3000.
// 16 senders of 11,173,962, m = 6, us (averages of kernel traces): gather 283 with the sort, 147 with masks and one load form, 126 now
// (782 MB: 6.2 TB/s); scatter 218, 109 (95% of the issue slots), 72 now (84% with two sets of vectors in turn, 84 us).
#include "eden_device.h"
#include "eden_kernels.h"

namespace eden {

constexpr uint32_t kSparseWave = 64u;            // blocks of 64 coordinates per wave of the selection
// One half (32 coordinates) of a block: which of them are kept (bit = position), and the slot of the first kept one among the
// kept coordinates of the wave's 64 blocks.
struct KeptHalf { uint32_t mask, slot; };

// any function of three bits, as its table over (x, y, z): the table of x is 0xF0, of y 0xCC, of z 0xAA.  (One instruction; left to
// itself the compiler spreads masks that two steps share over three.)
template <uint32_t TABLE>
__device__ __forceinline__ uint32_t logic3(uint32_t x, uint32_t y, uint32_t z) { return (uint32_t)__builtin_amdgcn_bitop3_b32((int)x, (int)y, (int)z, TABLE); }
constexpr uint32_t kSelect = 0xCA;               // x ? y : z
template <int S>
__device__ __forceinline__ void swap_step(uint32_t (&R)[16]) {
    constexpr uint32_t low = S == 4 ? 0x0F0F0F0Fu : S == 2 ? 0x33333333u : 0x55555555u;      // bits whose number has bit S clear
#pragma unroll
    for (int g = 0; g < 16; g += 2 * S)
#pragma unroll
        for (int i = g; i < g + S; ++i) {
            const uint32_t a = R[i], b = R[i + S];
            R[i] = logic3<kSelect>(low, a, b << S);
            R[i + S] = logic3<kSelect>(low, a >> S, b);
        }
}
// R[i] holds in each half 16 bits; afterwards bit k of a half of R[i] is bit i of that half of the former R[k].
__device__ __forceinline__ void transpose_16x16(uint32_t (&R)[16]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {                                // the bytes of the halves
        const uint32_t a = R[i], b = R[i + 8];
        R[i] = __builtin_amdgcn_perm(b, a, 0x06020400u);
        R[i + 8] = __builtin_amdgcn_perm(b, a, 0x07030501u);
    }
    swap_step<4>(R);
    swap_step<2>(R);
    swap_step<1>(R);
}
// bit k of the low half -> bit 2 k, bit k of the high half -> bit 2 k + 1
__device__ __forceinline__ uint32_t interleave_halves(uint32_t x) {
    constexpr uint32_t XorAnd = 0x28, Xor3 = 0x96;               // (x ^ y) & z, x ^ y ^ z
    uint32_t t = logic3<XorAnd>(x, x >> 8, 0x0000FF00u); x = logic3<Xor3>(x, t, t << 8);
    t = logic3<XorAnd>(x, x >> 4, 0x00F000F0u); x = logic3<Xor3>(x, t, t << 4);
    t = logic3<XorAnd>(x, x >> 2, 0x0C0C0C0Cu); x = logic3<Xor3>(x, t, t << 2);
    t = logic3<XorAnd>(x, x >> 1, 0x22222222u); return logic3<Xor3>(x, t, t << 1);
}

// The kept coordinates of this lane's block: bit i of lo (hi): coordinate i (32 + i).  Every lane of the wave calls it.  Block
// numbers and coordinates fit 32 bits (d <= 2^EDEN_MAX_LOG2_D).
__device__ __forceinline__ void sparse_select(uint64_t key, uint32_t block, uint32_t m, uint32_t &lo, uint32_t &hi) {
    const uint64_t word0 = key + kPhi * (uint64_t)(block * 16u + 1u);
    uint32_t P[2][16];                                           // halves of register (g, i): keys of coordinates 32 g + 2 i, + 1
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const uint64_t w = mix64(word0 + kPhi * (uint64_t)j);    // hash_word(key, 16 block + j)
        P[j >> 3][2 * (j & 7)] = (uint32_t)w;
        P[j >> 3][2 * (j & 7) + 1] = (uint32_t)(w >> 32);
    }
    transpose_16x16(P[0]);                                       // P[g][b]: bit b of the keys of the 32 coordinates of half g
    transpose_16x16(P[1]);
    uint32_t c0 = ~0u, c1 = ~0u, s0 = 0, s1 = 0, left = m;       // candidates, kept for certain, still to be kept (>= 1)
#pragma unroll
    for (int b = 15; b >= 0; --b) {
        constexpr uint32_t AndXor = 0x60, OrAndNot = 0xF4;       // x & (y ^ z), x | (y & ~z)
        const uint32_t z0 = c0 & ~P[0][b], z1 = c1 & ~P[1][b];
        const uint32_t zeros = (uint32_t)__popc(z0) + (uint32_t)__popc(z1);
        const uint32_t out = zeros >= left ? ~0u : 0u;           // the threshold has a 0 here: candidates with a 1 are out
        c0 = logic3<AndXor>(c0, P[0][b], out);
        c1 = logic3<AndXor>(c1, P[1][b], out);
        s0 = logic3<OrAndNot>(s0, z0, out);
        s1 = logic3<OrAndNot>(s1, z1, out);
        left -= zeros & ~out;
    }
    // what is left agrees with the threshold in every bit: its lowest `left` positions are kept, nearly always all of them
    uint32_t extra = (uint32_t)__popc(c0) + (uint32_t)__popc(c1) - left;
    if (__ballot(extra != 0u) != 0ull) {
        c0 = interleave_halves(c0);
        c1 = interleave_halves(c1);
        while (__ballot(extra != 0u) != 0ull) {                  // (each turn takes the highest candidate of every lane with one too many)
            if (extra) {
                if (c1) c1 &= ~(0x80000000u >> __builtin_clz(c1));
                else c0 &= ~(0x80000000u >> __builtin_clz(c0));
                --extra;
            }
        }
        lo = interleave_halves(s0) | c0;
        hi = interleave_halves(s1) | c1;
    } else {
        lo = interleave_halves(s0 | c0);
        hi = interleave_halves(s1 | c1);
    }
}
// ... as the two entries of a wave's table of KeptHalf
__device__ __forceinline__ void sparse_table(uint64_t key, uint32_t first_block, uint32_t m, uint32_t lane, KeptHalf *table) {
    uint32_t lo, hi;
    sparse_select(key, first_block + lane, m, lo, hi);
    table[2u * lane] = KeptHalf{lo, lane * m};
    table[2u * lane + 1u] = KeptHalf{hi, lane * m + (uint32_t)__popc(lo)};
}

// ... as the list of the kept coordinates of the wave's 64 blocks, in order: their places among the wave's 4096 coordinates.
__device__ __forceinline__ void sparse_list(uint64_t key, uint32_t first_block, uint32_t m, uint32_t lane, uint16_t *list) {
    uint32_t lo, hi;
    sparse_select(key, first_block + lane, m, lo, hi);
    uint64_t mask = (uint64_t)hi << 32 | lo;
    uint16_t *mine = list + lane * m;
    for (uint32_t r = 0; r < m; ++r) {                           // (every block has exactly m)
        const uint32_t low = (uint32_t)mask, high = (uint32_t)(mask >> 32);
        mine[r] = (uint16_t)(64u * lane + (low ? (uint32_t)__builtin_ctz(low) : 32u + (uint32_t)__builtin_ctz(high)));
        mask &= mask - 1u;
    }
}

// BYTES per lane from memory into the LDS, lane after lane from `to` (uniform) on, without a register between.  Nothing but vmcnt says when
// they are there.
template <int BYTES, int POLICY>
__device__ inline void load_to_lds(const float *from, float *to) {
    static_assert(BYTES == 4 || BYTES == 16, "a word or four");
    const auto src = (const __attribute__((address_space(1))) void *)from;
    const auto dst = (__attribute__((address_space(3))) void *)to;
    if constexpr (BYTES == 16) __builtin_amdgcn_global_load_lds(src, dst, 16, 0, POLICY);
    else __builtin_amdgcn_global_load_lds(src, dst, 4, 0, POLICY);
}

// the four coordinates of a lane: one 16-byte load when `vec` (pointer aligned) and all four are below d, else 0-padded
__device__ inline void load4_padded(const float *x, uint32_t i, uint32_t d, bool vec, float (&v)[4]) {
    if (vec && i + 3 < d) {
        const float4 q = *reinterpret_cast<const float4 *>(x + i);
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (i + e < d) ? x[i + e] : 0.0f;
    }
}

// out[c][block m + slot] = x_c[i] for the kept coordinates (0 for a kept position beyond d), out[c] = out + (c << log2_stride).
// A wave takes 64 blocks = 4096 coordinates of sender blockIdx.y.  x goes straight into the LDS, all of it on its way while the wave
// selects; the kept coordinates are then picked from there by a list, and leave in one run.  (Loads behind the selection and a test of
// every coordinate against the masks: encode, us, m = 6 188 -> 169, one sender 30.2 -> 27.3, 2 of 4,000,037 25.2 -> 22.2; m = 32, 8
// senders of 11,173,962 206 -> 184; half of each by the selection itself.)
template <int POLICY>
__global__ __launch_bounds__(64) void k_sparse_gather(EncBatch B, uint32_t d, uint32_t m, uint64_t seed, float *out, int log2_stride) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    const uint32_t lane = threadIdx.x, c = blockIdx.y, first = blockIdx.x * kSparseWave;
    const uint32_t blocks = (d + 63u) >> 6;
    float *tile = reinterpret_cast<float *>(lds);                // the wave's 4096 coordinates
    uint16_t *list = reinterpret_cast<uint16_t *>(lds + 64u * kSparseWave);
    const float *x = B.x[c] + (size_t)first * 64u;
    const bool vec = (reinterpret_cast<uintptr_t>(x) & 15u) == 0;
    if ((first + kSparseWave) * 64u > d) {                       // the last, partial one
#pragma unroll 4
        for (uint32_t it = 0; it < 16u; ++it) {
            float v[4];
            load4_padded(x, it * 256u + 4u * lane, d - first * 64u, vec, v);
            *reinterpret_cast<float4 *>(tile + it * 256u + 4u * lane) = make_float4(v[0], v[1], v[2], v[3]);
        }
    } else if (vec) {
#pragma unroll
        for (uint32_t it = 0; it < 16u; ++it) load_to_lds<16, POLICY>(x + it * 256u + 4u * lane, tile + it * 256u);
    } else {
#pragma unroll 16
        for (uint32_t it = 0; it < 64u; ++it) load_to_lds<4, POLICY>(x + it * 64u + lane, tile + it * 64u);
    }
    sparse_list(stream_key(seed, kStreamSparse, B.client[c]), first, m, lane, list);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // the loads have reached the LDS
    wave_lds_sync();
    float *dst = out + ((size_t)c << log2_stride) + (size_t)first * m;
    if (first + kSparseWave <= blocks) {                         // 64 m floats, 256 m bytes into the slot: whole 16-byte pieces
        for (uint32_t i = lane; i < 16u * m; i += 64u) {
            const uint2 at = reinterpret_cast<const uint2 *>(list)[i];
            reinterpret_cast<float4 *>(dst)[i] = make_float4(tile[at.x & 0xFFFFu], tile[at.x >> 16], tile[at.y & 0xFFFFu], tile[at.y >> 16]);
        }
    } else {
        for (uint32_t i = lane; i < (blocks - first) * m; i += 64u) dst[i] = tile[list[i]];
    }
}

// acc[i] += the values of all senders whose selection holds coordinate i, one sender after the other (the factor 64/m is already
// in the values); mean_n > 0: acc is written with the sum divided by mean_n instead of added to.
// A workgroup takes 64 blocks = 4096 coordinates: its waves select for one sender at a time, and then its threads add, NQ times four
// coordinates at a time.
// Few senders leave most of eight waves idle while the others select, and one or two have no other sender's loads to overlap with:
// four waves where the launch fills the chip all the same, and NQ = 4 (see launch_sparse_scatter).
template <int NQ>
__global__ __launch_bounds__(512) void k_sparse_scatter(DecBatch B, uint32_t n, uint32_t d, uint32_t m, uint64_t seed, const float *in,
                                                         int log2_stride, float *acc, float mean_n) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    KeptHalf *tables = reinterpret_cast<KeptHalf *>(lds);        // n tables of 128
    const uint32_t lane = lane_id(), wv = wave_in_block(), first = blockIdx.x * kSparseWave;
    for (uint32_t c = wv; c < n; c += blockDim.x >> 6)
        sparse_table(stream_key(seed, kStreamSparse, B.client[c]), first, m, lane, tables + c * 2u * kSparseWave);
    __syncthreads();
    const float div = mean_n > 0.0f ? mean_n : 1.0f;
    const bool overwrite = mean_n > 0.0f;
    for (uint32_t q0 = threadIdx.x; q0 < 1024u; q0 += NQ * blockDim.x) {
        if (first * 64u + 4u * q0 >= d) break;
        float sum[NQ][4], old[NQ][4];
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            const uint32_t i = first * 64u + 4u * (q0 + (uint32_t)j * blockDim.x);
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[j][e] = old[j][e] = 0.0f;
            if (!overwrite) load4_padded(acc, i, d, true, old[j]);               // (acc is 16-byte aligned)
        }
#pragma unroll 4 / NQ
        for (uint32_t c = 0; c < n; ++c) {
            // (a read beyond the slot can only be one whose value is not used: 0 by the buffer bounds)
            const rsrc_t r = make_rsrc(in + ((size_t)c << log2_stride), 4u << log2_stride);
#pragma unroll
            for (int j = 0; j < NQ; ++j) {
                const uint32_t q = q0 + (uint32_t)j * blockDim.x, shift = 4u * (q & 7u), below = (1u << shift) - 1u;
                const KeptHalf h = tables[c * 2u * kSparseWave + (q >> 3)];
                uint32_t at = (first * m + h.slot + (uint32_t)__popc(h.mask & below)) * 4u;
                if (NQ > 1 && first * 64u + 4u * q >= d) at = 0xFFFFFFE0u;       // blocks beyond the last one: out of bounds, 0
                const uint32_t kept = h.mask >> shift;
#pragma unroll
                for (int e = 0; e < 4; ++e) {                    // no branch per value: the loads of several senders are in flight
                    const float value = buf_load_keep(r, at, 0u);
                    sum[j][e] += ((kept >> e) & 1u) ? value : 0.0f;
                    at += ((kept >> e) & 1u) << 2;
                }
            }
        }
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            const uint32_t i = first * 64u + 4u * (q0 + (uint32_t)j * blockDim.x);
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[j][e] = (old[j][e] + sum[j][e]) / div;
            if (i + 3u < d) {
                *reinterpret_cast<float4 *>(acc + i) = make_float4(sum[j][0], sum[j][1], sum[j][2], sum[j][3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (i + e < d) acc[i + e] = sum[j][e];
            }
        }
    }
}

// The same for few kept coordinates (see launch_sparse_scatter): instead of asking for every coordinate and sender whether it was kept
// (560 issue slots per 64 blocks and sender), a wave goes through the kept values of its blocks, sender by sender, and adds them to sums
// in the LDS.  (A sender has at most one value for a coordinate, and one wave adds all of a coordinate's: the same sums in the same
// order.)
template <int NI>
__global__ __launch_bounds__(512) void k_sparse_scatter_list(DecBatch B, uint32_t n, uint32_t d, uint32_t m, uint64_t seed, const float *in,
                                                             int log2_stride, float *acc, float mean_n) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    float *sums = reinterpret_cast<float *>(lds);                // of the 4096 coordinates
    uint16_t *lists = reinterpret_cast<uint16_t *>(lds + 64u * kSparseWave);     // n lists of 64 m
    const uint32_t lane = lane_id(), wv = wave_in_block(), waves = blockDim.x >> 6, first = blockIdx.x * kSparseWave;
    for (uint32_t q = threadIdx.x; q < 1024u; q += blockDim.x) reinterpret_cast<float4 *>(sums)[q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (uint32_t c = wv; c < n; c += waves)
        sparse_list(stream_key(seed, kStreamSparse, B.client[c]), first, m, lane, lists + c * kSparseWave * m);
    __syncthreads();
    const uint32_t mine = kSparseWave / waves * m, from = wv * mine;             // this wave's values of every sender
    for (uint32_t c0 = 0; c0 < n; c0 += 4u) {                    // the values of four senders on their way at a time
        float value[4][NI];
        uint32_t at[4][NI];
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            const uint32_t c = c0 + k < n ? c0 + k : c0;
            const rsrc_t r = make_rsrc(in + ((size_t)c << log2_stride), c0 + k < n ? 4u << log2_stride : 0u);
#pragma unroll
            for (uint32_t j = 0; j < (uint32_t)NI; ++j) {        // (values of blocks beyond the last one go to coordinates beyond d)
                const uint32_t i = lane + 64u * j;
                value[k][j] = buf_load_keep(r, i < mine ? (first * m + from + i) * 4u : 0xFFFFFFFCu, 0u);
                at[k][j] = lists[c * kSparseWave * m + from + (i < mine ? i : 0u)];
            }
        }
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            if (c0 + k >= n) break;
#pragma unroll
            for (uint32_t j = 0; j < (uint32_t)NI; ++j) {
                if (lane + 64u * j < mine) sums[at[k][j]] += value[k][j];
                wave_lds_sync();                                 // the next sender's value for that sum may be another lane's
            }
        }
    }
    __syncthreads();
    const float div = mean_n > 0.0f ? mean_n : 1.0f;
    const bool overwrite = mean_n > 0.0f;
    for (uint32_t q = threadIdx.x; q < 1024u; q += blockDim.x) {
        const uint32_t i = first * 64u + 4u * q;
        if (i >= d) break;
        float old[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (!overwrite) load4_padded(acc, i, d, true, old);      // (acc is 16-byte aligned)
        const float4 s = reinterpret_cast<const float4 *>(sums)[q];
        const float v[4] = {(old[0] + s.x) / div, (old[1] + s.y) / div, (old[2] + s.z) / div, (old[3] + s.w) / div};
        if (i + 3u < d) {
            *reinterpret_cast<float4 *>(acc + i) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (i + e < d) acc[i + e] = v[e];
        }
    }
}

// The same by a workgroup of eight waves per 64 blocks (see launch_sparse_gather): one wave selects while the others wait with their 512
// coordinates in registers, then all of them test theirs against the masks, compact and store.
__global__ __launch_bounds__(512) void k_sparse_gather_team(EncBatch B, uint32_t d, uint32_t m, uint64_t seed, float *out, int log2_stride) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    const uint32_t lane = lane_id(), wv = wave_in_block(), c = blockIdx.y;
    const uint32_t blocks = (d + 63u) >> 6, first = blockIdx.x * kSparseWave;
    KeptHalf *table = reinterpret_cast<KeptHalf *>(lds);
    float *run = reinterpret_cast<float *>(lds + 4u * kSparseWave);
    const float *x = B.x[c];
    const bool vec = (reinterpret_cast<uintptr_t>(x) & 15u) == 0;
    float v[2][4];
#pragma unroll
    for (uint32_t it = 0; it < 2u; ++it) load4_padded(x, first * 64u + (2u * wv + it) * 256u + 4u * lane, d, vec, v[it]);
    if (wv == 0) sparse_table(stream_key(seed, kStreamSparse, B.client[c]), first, m, lane, table);
    __syncthreads();
    const uint32_t shift = 4u * (lane & 7u), below = (1u << shift) - 1u;
#pragma unroll
    for (uint32_t it = 0; it < 2u; ++it) {                       // 256 coordinates = 8 halves per turn
        const KeptHalf h = table[(2u * wv + it) * 8u + (lane >> 3)];
        uint32_t at = h.slot + (uint32_t)__popc(h.mask & below);
        const uint32_t kept = h.mask >> shift;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if ((kept >> e) & 1u) run[at++] = v[it][e];
    }
    __syncthreads();
    float *dst = out + ((size_t)c << log2_stride) + (size_t)first * m;
    if (first + kSparseWave <= blocks) {
        for (uint32_t i = threadIdx.x; i < 16u * m; i += 512u) reinterpret_cast<float4 *>(dst)[i] = reinterpret_cast<const float4 *>(run)[i];
    } else {
        for (uint32_t i = threadIdx.x; i < (blocks - first) * m; i += 512u) dst[i] = run[i];
    }
}

void launch_sparse_gather(const EncBatch &B, uint32_t n, uint64_t d, uint32_t m, uint64_t seed, float *out, int log2_stride, hipStream_t st) {
    const uint32_t blocks = (uint32_t)((d + 63) / 64);
    const uint32_t groups = (blocks + kSparseWave - 1) / kSparseWave;
    // Launches that would leave most of the chip idle, and those that keep so many that the serial list of k_sparse_gather (a step for
    // each of m) takes longer than the test of every coordinate: the team.  Whole encode, us, team / one wave: one sender of 2^21, m =
    // 16 (512 groups) 16.6 / 17.9, m = 63 26.9 / 29.5; 8 of 500,001, m = 6 (984) 14.6 / 15.8; beyond 1024 groups 8 of 1,000,000, m = 6
    // 19.4 / 18.2, m = 16 23.3 / 22.7; m = 24, 32 senders of 200,003 (1568) 25.3 / 27.2, 2 of 2^24 (8192) 65.9 / 66.8, 4 of 2^24 127.8
    // / 122.9; m = 32, the same 25.4 / 28.7, 74.1 / 77.5, 146.8 / 145.3; m = 48 29.4 / 33.7, 97.7 / 103.6, 16 of 11,173,962 491 / 516;
    // m = 63 31.0 / 39.6, 119 / 130, 633 / 685.
    const uint64_t waves = (uint64_t)groups * n;
    if (waves <= 1024 || m >= 48u || (m >= 24u && waves <= 8192)) {
        hipLaunchKernelGGL(k_sparse_gather_team, dim3(groups, n), dim3(512), 2u * kSparseWave * (uint32_t)sizeof(KeptHalf) + kSparseWave * m * 4u, st,
                           B, (uint32_t)d, m, seed, out, log2_stride);
        return;
    }
    const uint32_t bytes = 64u * kSparseWave * (uint32_t)sizeof(float) + kSparseWave * m * (uint32_t)sizeof(uint16_t);    // at most 22 KiB
    // x beyond the size of the memory-side cache is read with the streaming policy (the line of launch_enc_lo_first lies lower because a
    // workspace as large as x is written beside it; here it is m/64 of it).  Whole encode, us, default / streaming: one sender of
    // 50,000,001, m = 6 60.1 / 61.6, 2 of 25,000,001, m = 16 75.4 / 80.0; one of 2^27, m = 6 145 / 133, 16 of 11,173,962 184 / 166.
    if ((uint64_t)n * d * 4u <= (256u << 20))
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_sparse_gather<0>), dim3(groups, n), dim3(64), bytes, st, B, (uint32_t)d, m, seed, out, log2_stride);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_sparse_gather<kStream>), dim3(groups, n), dim3(64), bytes, st, B, (uint32_t)d, m, seed, out, log2_stride);
}
void launch_sparse_scatter(const DecBatch &B, uint32_t n, uint64_t d, uint32_t m, uint64_t seed, const float *in, int log2_stride,
                           float *acc, float mean_n, hipStream_t st) {
    const uint32_t blocks = (uint32_t)((d + 63) / 64);
    const uint32_t groups = (blocks + kSparseWave - 1) / kSparseWave;
    // Fewer than eight senders: four waves per workgroup once eight would make more than 4096, 16 for each CU; with one or two senders
    // NQ = 4 then.  (Whole decode, m = 32: one sender of 250,000 24.6 us with one wave and NQ = 1, 15.1 with eight; with 1, 2, 4 waves and
    // NQ = 4 and with 8: one of 4,000,037 37.6, 35.4, 32.9, 36.6; of 11,173,962 58.7, 56.7, 57.4, 66.0; two of 11,173,962 84.2, 80.4,
    // 78.6, 88.1; four of 2^24, NQ = 1, 154.9 with four, 160.7 with eight; six 229 and 240.)
    const uint32_t waves = n < 8u && groups * 8u > 4096u ? 4u : 8u;
    // Up to 16 kept of 64, eight senders or two of large vectors: by lists.  Whole decode, us, by masks / by lists: m = 6, 16 senders of
    // 11,173,962 124.0 / 104.5, 4 48.1 / 43.2, 2 35.0 / 32.7 (with eight waves 37.0), one 28.5 / 28.8; 32 of 4,000,037 95.8 / 82.1; 16 of
    // 300,007 21.9 / 20.7; 4 of 2^20 15.1 / 15.5; m = 16, 16 of 11,173,962 171.7 / 159.7, 32 of 4,000,037 128.0 / 119.2; m = 32, 8 of
    // 4,000,037 57.1 / 59.2.  Not for up to half of one group of blocks: the lists hold all 64 blocks' values, the masks are asked for
    // real coordinates only (32 senders of 1000, m = 16 24.0 / 28.2, of 2000 26.9 / 28.8, of 3000 31.0 / 29.8).
    if (m <= 16u && blocks > 32u && (n >= 8u || (n >= 2u && groups > 512u))) {
        const uint32_t list_waves = n >= 4u ? 8u : 4u, turns = (kSparseWave / list_waves * m + 63u) / 64u;       // at most 4
        const uint32_t bytes = 64u * kSparseWave * (uint32_t)sizeof(float) + n * kSparseWave * m * (uint32_t)sizeof(uint16_t);   // at most 80 KiB
#define EDEN_SCATTER_LIST(NI) \
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_sparse_scatter_list<NI>), dim3(groups), dim3(64u * list_waves), bytes, st, B, n, (uint32_t)d, m, seed, in, log2_stride, acc, mean_n)
        if (turns == 1u) EDEN_SCATTER_LIST(1); else if (turns == 2u) EDEN_SCATTER_LIST(2); else EDEN_SCATTER_LIST(4);
#undef EDEN_SCATTER_LIST
        return;
    }
    const uint32_t lds = n * 2u * kSparseWave * (uint32_t)sizeof(KeptHalf);
    if (n <= 2u && waves == 4u)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_sparse_scatter<4>), dim3(groups), dim3(64u * waves), lds, st, B, n, (uint32_t)d, m, seed, in, log2_stride, acc, mean_n);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_sparse_scatter<1>), dim3(groups), dim3(64u * waves), lds, st, B, n, (uint32_t)d, m, seed, in, log2_stride, acc, mean_n);
}

}  // namespace eden
