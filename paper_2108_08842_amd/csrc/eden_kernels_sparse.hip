// b = m/64: sparsification before the rotation with p = m/64 (Sec. 4.1).  Of every block of 64 consecutive coordinates the m
// with the smallest (key, position) pairs are kept, the 16-bit key of coordinate i being bits 16 (i & 3) .. +15 of word i >> 2
// of the SPARSE stream; a kept coordinate's slot is block * m + its rank among the kept ones in position order.
//
// Both directions are the same selection (vector instructions) around a copy (memory).  A lane looks after one block: it
// hashes the block's 16 words, transposes the 64 keys into 16 bit planes (16 x 16 bits in both halves of a register at once,
// four swap steps) and walks the planes from the top bit: of the candidates that still agree with the threshold, those with a
// 0 in this plane are counted; if they are at least as many as are still to be kept, the others are out, otherwise
// they are all kept and the search goes on among the others.  About 1200 issue slots per wave of 64 blocks, more than half
// of them the 64-bit multiplications of the hash; a bitonic sort of the keys across lanes took 3000.
// 16 senders, d = 11,173,962, m = 6: gather 283 -> 150 us (782 MB: the rate of a copy), scatter 218 -> 121 us (the selection; 112
// us of it by instruction count).
#include "eden_device.h"
#include "eden_kernels.h"

namespace eden {

constexpr uint32_t kSparseWave = 64u;            // blocks of 64 coordinates per wave of the selection
// One half (32 coordinates) of a block: which of them are kept (bit = position), and the slot of the first kept one among the
// kept coordinates of the wave's 64 blocks.
struct KeptHalf { uint32_t mask, slot; };

template <int S>
__device__ __forceinline__ void swap_step(uint32_t (&R)[16]) {
    constexpr uint32_t low = S == 4 ? 0x0F0F0F0Fu : S == 2 ? 0x33333333u : 0x55555555u;      // bits whose number has bit S clear
#pragma unroll
    for (int g = 0; g < 16; g += 2 * S)
#pragma unroll
        for (int i = g; i < g + S; ++i) {
            const uint32_t a = R[i], b = R[i + S];
            R[i] = (a & low) | ((b << S) & ~low);
            R[i + S] = ((a >> S) & low) | (b & ~low);
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
    uint32_t t = (x ^ (x >> 8)) & 0x0000FF00u; x ^= t ^ (t << 8);
    t = (x ^ (x >> 4)) & 0x00F000F0u; x ^= t ^ (t << 4);
    t = (x ^ (x >> 2)) & 0x0C0C0C0Cu; x ^= t ^ (t << 2);
    t = (x ^ (x >> 1)) & 0x22222222u; return x ^ t ^ (t << 1);
}

// The kept coordinates of this lane's block: bit i of lo (hi): coordinate i (32 + i).  Every lane of the wave calls it.  Block
// numbers and coordinates fit 32 bits (d <= 2^EDEN_MAX_LOG2_D).
__device__ __forceinline__ void sparse_select(uint64_t key, uint32_t block, uint32_t m, uint32_t &lo, uint32_t &hi) {
    uint32_t P[2][16];                                           // halves of register (g, i): keys of coordinates 32 g + 2 i, + 1
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const uint64_t w = hash_word(key, (uint64_t)(block * 16u + (uint32_t)j));
        P[j >> 3][2 * (j & 7)] = (uint32_t)w;
        P[j >> 3][2 * (j & 7) + 1] = (uint32_t)(w >> 32);
    }
    transpose_16x16(P[0]);                                       // P[g][b]: bit b of the keys of the 32 coordinates of half g
    transpose_16x16(P[1]);
    uint32_t c0 = ~0u, c1 = ~0u, s0 = 0, s1 = 0, left = m;       // candidates, kept for certain, still to be kept (>= 1)
#pragma unroll
    for (int b = 15; b >= 0; --b) {
        const uint32_t z0 = c0 & ~P[0][b], z1 = c1 & ~P[1][b];
        const uint32_t zeros = (uint32_t)__popc(z0) + (uint32_t)__popc(z1);
        const uint32_t out = zeros >= left ? ~0u : 0u;           // the threshold has a 0 here: candidates with a 1 are out
        c0 &= P[0][b] ^ out;
        c1 &= P[1][b] ^ out;
        s0 |= z0 & ~out;
        s1 |= z1 & ~out;
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
// A wave takes 64 blocks = 4096 coordinates of sender blockIdx.y: the selection, then x in coalesced 16-byte loads, the
// kept values moved together in LDS, and the run of 64 m values stored in one piece.
__global__ __launch_bounds__(128) void k_sparse_gather(EncBatch B, uint32_t d, uint32_t m, uint64_t seed, float *out, int log2_stride) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    const uint32_t lane = lane_id(), wv = wave_in_block(), c = blockIdx.y;
    const uint32_t blocks = (d + 63u) >> 6, first = (blockIdx.x * 2u + wv) * kSparseWave;
    if (first >= blocks) return;                                 // wave-uniform; no workgroup barrier below
    KeptHalf *table = reinterpret_cast<KeptHalf *>(lds) + wv * 2u * kSparseWave;
    float *run = reinterpret_cast<float *>(lds + 2u * 4u * kSparseWave) + wv * kSparseWave * m;
    sparse_table(stream_key(seed, kStreamSparse, B.client[c]), first, m, lane, table);
    wave_lds_sync();
    const float *x = B.x[c];
    const bool vec = (reinterpret_cast<uintptr_t>(x) & 15u) == 0;
    const uint32_t shift = 4u * (lane & 7u), below = (1u << shift) - 1u;
#pragma unroll 8
    for (uint32_t it = 0; it < 16u; ++it) {                      // 256 coordinates = 8 halves per turn
        float v[4];
        load4_padded(x, first * 64u + it * 256u + 4u * lane, d, vec, v);
        const KeptHalf h = table[it * 8u + (lane >> 3)];
        uint32_t at = h.slot + (uint32_t)__popc(h.mask & below);
        const uint32_t kept = h.mask >> shift;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if ((kept >> e) & 1u) run[at++] = v[e];
    }
    wave_lds_sync();
    float *dst = out + ((size_t)c << log2_stride) + (size_t)first * m;
    if (first + kSparseWave <= blocks) {                         // 64 m floats, 256 m bytes into the slot: whole 16-byte pieces
        for (uint32_t i = lane; i < 16u * m; i += 64u) reinterpret_cast<float4 *>(dst)[i] = reinterpret_cast<const float4 *>(run)[i];
    } else {
        for (uint32_t i = lane; i < (blocks - first) * m; i += 64u) dst[i] = run[i];
    }
}

// acc[i] += the values of all senders whose selection holds coordinate i, one sender after the other (the factor 64/m is already
// in the values); mean_n > 0: acc is written with the sum divided by mean_n instead of added to.
// A workgroup takes 64 blocks = 4096 coordinates: its waves select for one sender at a time, and then its threads add, NQ times four
// coordinates at a time.  Two workgroups of eight waves share a CU, one selecting while the other adds: 121 us at the size
// above; sixteen waves, alone on a CU, 147 us; four waves 126 us; 64 or 80 registers instead of 109 spill: 210 and 162 us.
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

// The same by a workgroup of eight waves per 64 blocks, for launches that would leave most of the chip idle: one wave selects while the
// others wait with their 512 coordinates in registers, then all of them compact and store.  (Up to 1024 groups of 64 blocks; whole
// encode, against two waves on their own: one sender of 2^20, m = 32, 23.7 -> 21.1 us; 8 of 300,007 29.4 -> 27.2; one of 4,000,037
// 32.1 -> 29.3; beyond, 2048 groups of 8 senders of 2^20 28.7 -> 30.4 and one sender of 7,000,001 34.3 -> 34.8.)
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
    if ((uint64_t)groups * n <= 1024) {
        hipLaunchKernelGGL(k_sparse_gather_team, dim3(groups, n), dim3(512), 2u * kSparseWave * (uint32_t)sizeof(KeptHalf) + kSparseWave * m * 4u, st,
                           B, (uint32_t)d, m, seed, out, log2_stride);
        return;
    }
    const uint32_t bytes = 2u * (2u * kSparseWave * (uint32_t)sizeof(KeptHalf) + kSparseWave * m * 4u);        // at most 34 KiB
    hipLaunchKernelGGL(k_sparse_gather, dim3((blocks + 2u * kSparseWave - 1) / (2u * kSparseWave), n), dim3(128), bytes, st, B, (uint32_t)d, m,
                       seed, out, log2_stride);
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
    const uint32_t lds = n * 2u * kSparseWave * (uint32_t)sizeof(KeptHalf);
    if (n <= 2u && waves == 4u)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_sparse_scatter<4>), dim3(groups), dim3(64u * waves), lds, st, B, n, (uint32_t)d, m, seed, in, log2_stride, acc, mean_n);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_sparse_scatter<1>), dim3(groups), dim3(64u * waves), lds, st, B, n, (uint32_t)d, m, seed, in, log2_stride, acc, mean_n);
}

}  // namespace eden
