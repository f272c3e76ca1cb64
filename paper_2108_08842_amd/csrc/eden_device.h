// Device-side building blocks shared by the EDEN kernels (gfx950, wave64).
#ifndef EDEN_DEVICE_H
#define EDEN_DEVICE_H

#include <hip/hip_runtime.h>

#include <utility>
#include <stddef.h>
#include <stdint.h>

#include "eden.h"                    // status bits, packet size

namespace eden {

constexpr int kMaxBatch = 32;            // senders handled by one launch; larger batches are chunked
constexpr uint32_t kEncCounterStride = 32;  // words between the arrival counters of two senders: a memory line each (see enc_last_tail)
constexpr uint32_t kDecCounters = 8;     // arrival counters of the small decode launches, used in turn (see k_dec_small)
constexpr int kLoBits = 12;              // index bits transformed by the contiguous pass up to D = 2^18

// ---- shared randomness (Sec. 2.1): counter hash = splitmix64 stream started at a per-(seed,stream,client) key
constexpr uint64_t kPhi = 0x9E3779B97F4A7C15ull;
enum : uint32_t { kStreamSign = 0, kStreamSubsample = 1, kStreamLoss = 2, kStreamMix = 3, kStreamSparse = 4 };

__host__ __device__ inline uint64_t mix64(uint64_t z) {
    z ^= z >> 30; z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27; z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z;
}
__host__ __device__ inline uint64_t stream_key(uint64_t seed, uint32_t stream, uint32_t client) {
    const uint64_t tag = ((uint64_t)stream << 32) | (uint64_t)client;
    return mix64(mix64(seed + kPhi) + kPhi * tag + kPhi);
}
__host__ __device__ inline uint64_t hash_word(uint64_t key, uint64_t j) { return mix64(key + kPhi * (j + 1)); }

// ---- bit budgets (Sec. 4.1): b_q8 = 256 b -> bits per transmitted index, keep one coordinate in k.
// b = 1.5, 2.5, 3.5 ("mixed"): every coordinate has floor(b) bits in the first part of the payload and one
// coordinate of every pair, chosen by the MIX stream, one more bit in a second part (it is quantized with the
// next finer table).
// b = 1/2 with the sparsification before the rotation (Sec. 4.1, the paper's default for b < 1): the vector
// x'[g] = 2 x[2g + offset_g] of dimension ceil(d/2) is encoded with b = 1; the kernels then see b_q8 = 256 and
// only the gather (first encode pass), the scatter (last decode pass) and the header know about it.
constexpr uint32_t kPreHalf = 0x10000u | 128u;
// b = m/64, 1 <= m <= 63 (Sec. 4.1 sub-bit compression with p = m/64, sparsification before the rotation): of every
// 64 consecutive coordinates the m with the smallest 16-bit keys of the SPARSE stream are kept (ties by position)
// and the vector of kept coordinates is encoded with b = 1; the receiver multiplies by 64/m.  Only a gather kernel
// before the encoder, a scatter kernel after the decoder and the header know about it.
constexpr uint32_t kSparseFlag = 0x20000u;
__host__ __device__ inline uint32_t sparse_m(uint32_t b_q8) {
    const uint32_t m = b_q8 & 0xFFFFu;
    return ((b_q8 & ~0xFFFFu) == kSparseFlag && m >= 1 && m <= 63) ? m : 0;
}
// Uniform-grid quantizer of Sec. 4.3: the intervals [Delta (n - 1/2), Delta (n + 1/2)], Delta = (b_q8 & 0xFFFF) / 32768;
// the index n of the interval that holds z (endpoints: closer to zero), clipped to +-127, travels as one signed byte (what an entropy
// coder would shrink to about H(Delta) bits); the value of an interval is its centre of mass under N(0,1).
constexpr uint32_t kGridFlag = 0x30000u;
constexpr int kGridMax = 127;
__host__ __device__ inline uint32_t grid_q15(uint32_t b_q8) {
    return ((b_q8 & ~0xFFFFu) == kGridFlag && (b_q8 & 0xFFFFu) >= 1u) ? (b_q8 & 0xFFFFu) : 0u;
}
// b = 5..8: the Lloyd-Max quantizers with 32..256 levels.  Like the uniform grid they are handled one byte per
// coordinate inside the kernels (index = rank of the interval); for b = 5, 6, 7 a separate kernel packs the bytes to
// b bits (and unpacks them before decoding), for b = 8 the bytes are the payload.
__host__ __device__ inline uint32_t wide_bits(uint32_t b_q8) {
    return (b_q8 == 1280u || b_q8 == 1536u || b_q8 == 1792u || b_q8 == 2048u) ? (b_q8 >> 8) : 0u;
}
__host__ __device__ inline bool byte_budget(uint32_t b_q8) { return grid_q15(b_q8) != 0u || wide_bits(b_q8) != 0u; }
__host__ __device__ inline bool budget_mixed(uint32_t b_q8) { return b_q8 == 384 || b_q8 == 640 || b_q8 == 896; }
// General non-integer b > 1 in the paper's own form (Sec. 4.1): every coordinate is quantized with I_{floor(b)+1} with
// probability b - floor(b), by an independent coin from the shared randomness: coordinate i gets the extra bit iff byte
// (i & 7) of word (i >> 3) of the MIX stream is below 256 (b - floor(b)).  b = (b_q8 & 0xFFFF) / 256, 1 < b < 4, not an
// integer.  The message length then depends on the coins (never on the data); positions in the second part of the payload
// come from a prefix sum over the coins that a small kernel computes for sender and receiver alike.
constexpr uint32_t kCoinFlag = 0x40000u;
__host__ __device__ inline uint32_t coin_q8(uint32_t b_q8) {
    const uint32_t low = b_q8 & 0xFFFFu;
    return ((b_q8 & ~0xFFFFu) == kCoinFlag && low > 256u && low < 1024u && (low & 255u) != 0u) ? low : 0u;
}
// some coordinates carry one bit more than the others: the stratified k + 1/2 budgets and the coin budgets
__host__ __device__ inline bool budget_two_tables(uint32_t b_q8) { return budget_mixed(b_q8) || coin_q8(b_q8) != 0u; }
__host__ __device__ inline bool budget_of(uint32_t b_q8, int &bits, int &k) {
    if (coin_q8(b_q8)) { bits = (int)(coin_q8(b_q8) >> 8); k = 1; return true; }
    if (b_q8 == 128) { bits = 1; k = 2; return true; }
    if (b_q8 == 256 || b_q8 == 512 || b_q8 == 768 || b_q8 == 1024 || budget_mixed(b_q8)) {
        bits = (int)(b_q8 >> 8); k = 1; return true;
    }
    if (grid_q15(b_q8)) { bits = 8; k = 1; return true; }
    if (wide_bits(b_q8)) { bits = (int)wide_bits(b_q8); k = 1; return true; }
    return false;
}
// bytes of the first part of the payload (the floor(b)-bit indices), a multiple of 8
__host__ __device__ inline uint64_t payload_a_bytes(uint64_t D, int bits, int k) {
    return ((((D / (uint64_t)k) * (uint64_t)bits) + 63) / 64) * 8;
}
// bytes of the second part (one bit per pair of coordinates) of a mixed budget; for a coin budget the room that fits
// any outcome of the coins (one bit per coordinate)
__host__ __device__ inline uint64_t payload_b_bytes(uint64_t D, uint32_t b_q8) {
    if (coin_q8(b_q8)) return ((D + 63) / 64) * 8;
    return budget_mixed(b_q8) ? ((D / 2 + 63) / 64) * 8 : 0;
}
// bytes of the second part of a coin budget whose coins gave `extra_bits` coordinates the extra bit
__host__ __device__ inline uint64_t coin_b_bytes(uint64_t extra_bits) { return ((extra_bits + 63) / 64) * 8; }

// Coins of one sender, written by k_coin_masks / k_coin_scan: a lane mask per 64 consecutive coordinates, the number of
// coins before each such block inside its group of 256 blocks, the number of coins before each group, and the total.
constexpr int kCoinGroup = 256;          // blocks of 64 coordinates per group (one workgroup of k_coin_masks)
struct CoinTables {
    uint64_t *mask;                      // slot c: mask + (c << (log2D - 6)); bit j of word w: coordinate 64 w + j has a coin
    uint32_t *local;                     // slot c: local + (c << (log2D - 6)); coins before block w inside its group
    uint32_t *group;                     // slot c: group + c * group_stride; coins before group g
    uint32_t *total;                     // total[c]: all coins of sender c = bits of the second part of its payload
    uint32_t group_stride;
};
__device__ inline bool coin_of(uint64_t mixkey, uint64_t i, uint32_t frac) {
    return ((uint32_t)(hash_word(mixkey, i >> 3) >> (8u * (uint32_t)(i & 7u))) & 0xFFu) < frac;
}

// ---- message header (64 bytes, little endian)
struct MsgHeader {
    uint32_t magic, log2D;
    uint64_t d;
    uint32_t b_q8, client, status, extra_bits;   // extra_bits: coin budgets only (bits of the second part), else 0
    double S, N2, IP;
    uint64_t seed;
};
static_assert(sizeof(MsgHeader) == 64, "header layout");
constexpr uint32_t kMagic = 0x4E454445u;

// the positive centroid of I_1, sqrt(2/pi) (Sec. 3: Q_{I_1} = {+-sqrt(2/pi)}); b = 1 and b = 1/2 need no other table
constexpr float kQ1 = 0.7978845608028654f;

// ---- device copies of the Lloyd-Max tables (positive halves, Sec. 3), index [bits][k]
struct DevTables {
    double t[5][8];
    double q[5][8];
    double t_big[4][128];   // b = 5..8 at index b - 5
    double q_big[4][128];
};

// per-sender scalars that travel between the passes of one encode
struct EncScratch {
    double n2;              // |x|^2 (Sec. 2.2.1: equals |R(x)|^2)
    float thr[8];           // positive thresholds of I_b times |x|: compared against |H(s o x)|
    float thr2[8];          // mixed budgets: the same for I_{floor(b)+1}
    float qpos[8];          // positive centroids
    float qpos2[8];         // (the kernels look centroids up in qpos .. qpos2 as one run of 16 floats)
    float grid_inv;         // uniform grid: 1 / (Delta |x|), so that round(u * grid_inv) is the index
    float guess_c1, guess_c3, guess_cap, guess_up;      // b = 4: see quantize_guess
    unsigned pad;
    float grid_c[kGridMax + 1];     // uniform grid: centre of mass of the interval of index n >= 0; b = 5..8: positive centroids
    float wide_thr[128];            // b = 5..8: positive thresholds times |x|
};

static_assert(offsetof(EncScratch, wide_thr) == offsetof(EncScratch, grid_c) + 128 * sizeof(float) &&
                  offsetof(EncScratch, qpos2) == offsetof(EncScratch, qpos) + 8 * sizeof(float),
              "the kernels use centroids and thresholds of the one-byte budgets as one run of 256 floats, qpos and qpos2 as one of 16");

// per-message scalars of one decode
struct DecScratch {
    float deq[16];          // (S / (p sqrt(D))) * q_l for every index l (all zero if the message contributes nothing)
    float deq2[16];         // mixed budgets: the same for the indices of I_{floor(b)+1}
    uint32_t flags;
    uint32_t pad[3];
    float grid_deq[kGridMax + 1];   // uniform grid and b = 5..8: (S / (p sqrt(D))) * positive centroid
};

struct EncBatch {
    const float *x[kMaxBatch];
    void *msg[kMaxBatch];
    uint32_t client[kMaxBatch];
    uint32_t b_q8[kMaxBatch];       // what the kernels quantize with
    uint32_t hdr_b_q8[kMaxBatch];   // what the header says (differs for the budgets that sparsify before the rotation)
    uint8_t *codes[kMaxBatch];      // b = 5, 6, 7: where the one-byte indices go before they are packed (else null)
};
struct DecBatch {
    const void *msg[kMaxBatch];
    const uint32_t *bitmap[kMaxBatch];
    uint32_t client[kMaxBatch];
    uint32_t b_q8[kMaxBatch];
    uint32_t hdr_b_q8[kMaxBatch];
    const uint8_t *codes[kMaxBatch];    // b = 5, 6, 7: the unpacked one-byte indices (else null)
};

// ---- wave-level helpers
__device__ inline uint32_t lane_id() { return threadIdx.x & 63u; }
__device__ inline uint32_t wave_in_block() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// LDS traffic of one wave is processed in issue order; this only stops the compiler from moving
// the reads of a transpose above the writes of other lanes.
__device__ inline void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// v or -v per lane, chosen by bit `lane` of a wave-uniform 64-bit mask (one VALU op: the mask is
// used directly as the lane-select operand).  Written with the builtin, not inline assembly: an SGPR
// written by a vector instruction (v_readlane, v_cmp) needs wait states before a vector instruction
// reads it, and the compiler only inserts them for instructions it can see.
__device__ inline float negate_where(float v, uint64_t mask) {
    return __builtin_amdgcn_inverse_ballot_w64(mask) ? -v : v;
}

// v or 0 per lane, chosen by bit `lane` of a wave-uniform mask
__device__ inline float keep_where(float v, uint64_t mask) {
    return __builtin_amdgcn_inverse_ballot_w64(mask) ? v : 0.0f;
}

// a float that is the same in every lane, in a scalar register
__device__ inline float uniform(float v) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v))); }

// The 64-bit value held by lane `src` (compile-time constant), as a wave-uniform scalar.
__device__ inline uint64_t wave_read64(uint64_t v, int src) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, src);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), src);
    return ((uint64_t)hi << 32) | lo;
}

// ---- buffer addressing: one resource descriptor per sender buffer, a per-lane byte offset in a VGPR and
// a wave-uniform byte offset in an SGPR per access.  Strided passes issue 64 loads back to back; with flat
// 64-bit addresses each of them would pin two VGPRs.  Reads beyond `bytes` return 0 and writes beyond it
// are dropped, which is exactly the zero padding of d up to D.
using rsrc_t = __amdgpu_buffer_rsrc_t;
__device__ inline rsrc_t make_rsrc(const void *base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}
constexpr int kStream = 2;   // cache-policy bit "nt": the data is touched once per pass (measured +5..9% on copies)
__device__ inline float buf_load(rsrc_t r, uint32_t lane_off, uint32_t wave_off) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)lane_off, (int)wave_off, kStream));
}
__device__ inline void buf_store(rsrc_t r, uint32_t lane_off, uint32_t wave_off, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, (int)lane_off, (int)wave_off, kStream);
}
// read-modify-write data that another kernel reads soon (the accumulator): default cache policy
__device__ inline float buf_load_keep(rsrc_t r, uint32_t lane_off, uint32_t wave_off) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)lane_off, (int)wave_off, 0));
}

// Sub-word accesses of neighbouring lanes go through whole dwords (a byte or half-word load per lane is not merged
// with its neighbours': measured 3x slower on the first decode pass of the one-byte budgets).
// The byte at `byte_off` (lane part) + `wave_off` of the buffer; descriptor base and wave_off are multiples of 4.
__device__ inline uint32_t buf_load_byte(rsrc_t r, uint32_t byte_off, uint32_t wave_off) {
    const uint32_t w = __builtin_amdgcn_raw_buffer_load_b32(r, (int)(byte_off & ~3u), (int)wave_off, 0);
    return (w >> (8u * (byte_off & 3u))) & 0xFFu;
}
__device__ inline uint32_t buf_load_half(rsrc_t r, uint32_t byte_off, uint32_t wave_off) {     // byte_off even
    const uint32_t w = __builtin_amdgcn_raw_buffer_load_b32(r, (int)(byte_off & ~3u), (int)wave_off, 0);
    return (w >> (8u * (byte_off & 2u))) & 0xFFFFu;
}
// The bytes of lanes 4k .. 4k+3 as one dword (byte of lane 4k + i in bits 8i..), in all four lanes.
__device__ inline uint32_t quad_bytes(uint32_t byte, uint32_t lane) {
    uint32_t x = (byte & 0xFFu) << (8u * (lane & 3u));
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true);     // quad_perm [1,0,3,2]: lane ^ 1
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true);     // quad_perm [2,3,0,1]: lane ^ 2
    return x;
}

// In-register Walsh-Hadamard butterflies over the register index: (a,b) -> (a+b, a-b) at spans 1..N/2.
template <int N>
__device__ inline void fwht_regs(float (&v)[N]) {
#pragma unroll
    for (int h = 1; h < N; h <<= 1) {
#pragma unroll
        for (int i = 0; i < N; i += 2 * h) {
#pragma unroll
            for (int j = i; j < i + h; ++j) {
                const float a = v[j], b = v[j + h];
                v[j] = a + b;
                v[j + h] = a - b;
            }
        }
    }
}

// The value of another lane, by data-parallel primitives instead of the cross-lane path through the LDS (a sum over the wave took 0.3 us
// that way): lane ^ 1, lane ^ 2 inside a quad; then, since every lane of a quad (8, 16 lanes) already holds the same sum, the mirrored
// lane of 8 and of 16 stand for lane ^ 4 and lane ^ 8.
template <int CTRL>
__device__ inline uint32_t dpp_u32(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true); }
template <int CTRL>
__device__ inline double dpp_f64(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(double, (uint64_t)dpp_u32<CTRL>((uint32_t)b) | ((uint64_t)dpp_u32<CTRL>((uint32_t)(b >> 32)) << 32));
}
enum : int { kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppMirror8 = 0x141, kDppMirror16 = 0x140 };
// the values of both lanes of a pair (lane, lane ^ 16) or (lane, lane ^ 32), the lower one's first
template <int X>
__device__ inline void lane_pair(uint32_t v, uint32_t &lower, uint32_t &upper) {
    static_assert(X == 16 || X == 32, "rows of 16 lanes");
    const auto r = X == 16 ? __builtin_amdgcn_permlane16_swap(v, v, false, false) : __builtin_amdgcn_permlane32_swap(v, v, false, false);
    lower = r[0]; upper = r[1];
}
// One butterfly stage between the halves of a wave: register pairs 2 i, 2 i + 1 swap, so that afterwards bit 0 of the register index
// stands for what lane bit 5 stood for, and lane bit 5 for what bit 0 of the register index did.
template <int N>
__device__ inline void swap_stage32(float (&v)[N]) {
#pragma unroll
    for (int i = 0; i < N; i += 2) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 1]), false, false);
        const float a = __uint_as_float(r[0]), b = __uint_as_float(r[1]);
        v[i] = a + b;
        v[i + 1] = a - b;
    }
}
template <int X>
__device__ inline double pair_sum(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    uint32_t lo0, lo1, hi0, hi1;
    lane_pair<X>((uint32_t)b, lo0, lo1);
    lane_pair<X>((uint32_t)(b >> 32), hi0, hi1);
    return __builtin_bit_cast(double, (uint64_t)lo0 | ((uint64_t)hi0 << 32)) + __builtin_bit_cast(double, (uint64_t)lo1 | ((uint64_t)hi1 << 32));
}
__device__ inline double wave_sum(double v) {          // fixed order: deterministic
    v += dpp_f64<kDppXor1>(v);
    v += dpp_f64<kDppXor2>(v);
    v += dpp_f64<kDppMirror8>(v);
    v += dpp_f64<kDppMirror16>(v);
    return pair_sum<32>(pair_sum<16>(v));
}
__device__ inline uint32_t wave_sum_u32(uint32_t v) {
    v += dpp_u32<kDppXor1>(v);
    v += dpp_u32<kDppXor2>(v);
    v += dpp_u32<kDppMirror8>(v);
    v += dpp_u32<kDppMirror16>(v);
    uint32_t a, b;
    lane_pair<16>(v, a, b);
    lane_pair<32>(a + b, a, b);
    return a + b;
}

// block-level deterministic sum of one double per thread; result valid in thread 0
template <int THREADS>
__device__ inline double block_sum(double v, double *red /* shared, THREADS/64 */) {
    v = wave_sum(v);
    const uint32_t w = threadIdx.x >> 6;
    if (lane_id() == 0) red[w] = v;
    __syncthreads();
    double total = 0.0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < THREADS / 64; ++i) total += red[i];
    }
    __syncthreads();
    return total;
}

// ---- values that one workgroup of a launch leaves for another of the same launch.  The eight XCDs have an L2 each, so such a
// value is written through to memory and read past the caches (relaxed atomics of device scope: no cache is written back or
// invalidated as a whole, which a release fence of device scope would do), and the counter is bumped when the writes have
// been acknowledged.
__device__ inline void store_through(float *p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline float load_through(const float *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// True, in every thread, in the workgroup that arrives last of `total`; it finds what the others stored before they
// arrived.  The last one puts the counter back to 0 for the next launch.  No workgroup waits for another.
__device__ inline bool arrive_last(uint32_t *counter, uint32_t total, uint32_t *flag /* shared */) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // this thread's stores have reached memory
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t before = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t last = before + 1u == total ? 1u : 0u;
        if (last) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *flag = last;
    }
    __syncthreads();
    return *flag != 0u;
}

// Interval rank of one coordinate of the unnormalised transform against the scaled thresholds of I_b
// (Sec. 2.2.1, Sec. 3), and its contribution |u| q to sum_i u_i Q_i (Sec. 2.3).  H = 2^(b-1) levels per sign.
// A value exactly on a threshold stays in the interval closer to zero (strict compare); u = +0 is
// non-negative.  thr[0] is unused (it is the threshold 0, decided by the sign).
// The thresholds are wave-uniform (Thresholds); the centroid is looked up in `qtab`, the workgroup's copy of qpos
// (entries 0..7) and qpos2 (8..15) in LDS.
struct Thresholds {
    float thr[8], thr2[8];
};
__device__ inline Thresholds thresholds_of(const EncScratch *s) {
    Thresholds t;
#pragma unroll
    for (int i = 0; i < 8; ++i) { t.thr[i] = s->thr[i]; t.thr2[i] = s->thr2[i]; }
    return t;
}
__device__ inline Thresholds uniform_thresholds(const EncScratch &s /* shared */) {
    Thresholds t;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        t.thr[i] = uniform(s.thr[i]);
        t.thr2[i] = uniform(s.thr2[i]);
    }
    return t;
}
// b = 2: the indices of 16 values side by side in one word, value i in bits 2 i, 2 i + 1.  Index = (2 | magnitude) with both bits turned
// over where the value is negative: 7 instructions a value, no read of the table.
__device__ inline uint32_t quantize_two_bits(const float *u, float thr1, float q0, float q1, float &ip) {
    uint32_t mags = 0xAAAAAAAAu, signs = 0u;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const bool outer = fabsf(u[i]) > thr1;
        ip = fmaf(fabsf(u[i]), outer ? q1 : q0, ip);
        mags |= outer ? 1u << (2 * i) : 0u;
        const uint32_t mask = 3u << (2 * i);
        signs = (signs & ~mask) | ((uint32_t)(__float_as_int(u[i]) >> 31) & mask);
    }
    return mags ^ signs;
}

// The search in one guess and one compare, for kernels that hold b = 4 alone (quantize_one_table, which leaves lane masks, takes 21
// instructions with the packing by ballots; this 12 with the packing by lane transposes).
// The number of a Lloyd-Max threshold is nearly a quadratic function of its value: with r(u) = u (c1 + c3 |u|) through
// thresholds H / 2 and H - 1, r differs from the number of every other threshold of I_4 by less than 0.07.  The threshold with the
// number nearest to r is therefore the one above or the one below u, and comparing u with it alone gives the index.  The
// result is the one of quantize_one_table for every input: the margin (0.43 of a number) is far beyond the rounding of r, u is capped
// above the outermost threshold where r still rises, and the compare is exact: a value on a positive threshold stays below
// it, one on a negative threshold (or on 0) stays above it, which "u > the float just below the threshold" says with
// the same compare.  c3 goes with 1 / |x|^2: where the outermost threshold is below 2^-60 or above 2^60, values and thresholds are
// multiplied by a power of two first (guess_up, scale_for_guess).  Where |x| is so large that outer thresholds are +inf (beyond 1.4e38),
// no value exceeds one of those: the cap then is the u at which r is 0.4 above the last finite threshold's number, so that this one
// decides about everything beyond.
// |x| = 0 or not finite, u = NaN: any index in range will do, the payload is cleared afterwards (the cap keeps it in range).
// kGuessRound added to r + H leaves the nearest whole number in the low bits of the float.
// Measured against a guess through u / |x|, a conversion and shifts of the indices (26 vector instructions a value with the butterflies,
// now 20): strided pass of 16 x 11,173,962 222.6 -> 211.3 us, of 8 x 4,000,037 33.9 -> 32.5; encode of 16 x 250,000 23.6 -> 23.1.
// Two four-byte reads of tables of 18 entries (lanes that hit one bank read one address: no conflicts); a table of 64 cells
// with the threshold, both centroids and the count in 16 bytes cost three times their LDS time.
template <int H>
struct RankGuess {
    float thr[2 * H + 2];   // [s], s = 1 .. 2 H - 1: the signed thresholds in order, as what u has to exceed
    float q[2 * H + 2];     // [index + 1]: signed centroids
};
template <int H>
__device__ inline void fill_rank_guess(RankGuess<H> &g, const EncScratch *sc, uint32_t thread) {
    if (thread >= 2u * H + 2u) return;
    // the float just below -thr (or 0) has the next larger magnitude (next to an infinite one is a NaN, which the cap keeps out of use)
    const int j = (int)thread - H;
    const float mag = (j > -H && j < H && j != 0) ? sc->thr[j < 0 ? -j : j] * sc->guess_up : 0.0f;
    g.thr[thread] = j <= -H || j >= H ? __builtin_inff() : j > 0 ? mag : __uint_as_float(0x80000000u | (__float_as_uint(mag) + 1u));
    const int index = (int)thread - 1;
    g.q[thread] = index < 0 || index >= 2 * H ? 0.0f : index >= H ? sc->qpos[index - H] : -sc->qpos[H - 1 - index];
}
typedef const __attribute__((address_space(3))) float *LdsFloats;
__device__ inline uint32_t lds_address(const float *shared) { return (uint32_t)(uintptr_t)(LdsFloats)shared; }
__device__ inline float lds_read(uint32_t address, int i) { return ((LdsFloats)(uintptr_t)address)[i]; }
// u[i] * sc->guess_up, never 0 where u[i] is not (far below every threshold but that one, so that its sign alone decides)
__device__ inline float scale_for_guess(float u, float up) {
    const float v = u * up;
    return v == 0.0f && u != 0.0f ? copysignf(__uint_as_float(1u), u) : v;
}
// sum |u| q of values that were multiplied by guess_up, in the units of the values: it overflows where it would have without the factor
__device__ inline double unscale_sum(float ip, float up) { return up < 1.0f ? (double)(ip * (1.0f / up)) : (double)ip / (double)up; }
constexpr float kGuessRound = 0x1.8p23f;
constexpr uint32_t kGuessBits = 0x4B400000u;                     // its bit pattern
// at[i] = kGuessBits + index + 1 of u[i], which is sc->guess_up times the value.  The table reads of N values are issued together: one value
// after the other, as the compiler would schedule it, every value waits for the LDS twice.
template <int H, int N>
__device__ inline void quantize_guess(const float *u, const RankGuess<H> &g, const EncScratch *sc, uint32_t (&at)[N], float &ip) {
    const float c1 = sc->guess_c1, c3 = sc->guess_c3, cap = sc->guess_cap;
    // an entry's address from the bits as they are and one scalar register (left to add up the constants by itself the compiler takes
    // three instructions)
    uint32_t zero = lds_address(g.thr) - 4u * kGuessBits;
    asm("" : "+s"(zero));
    float t[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float v = __builtin_amdgcn_fmed3f(u[i], -cap, cap);
        at[i] = __float_as_uint(fmaf(v, fmaf(fabsf(v), c3, c1), (float)H + kGuessRound));
        asm("" : "+v"(at[i]));
        t[i] = lds_read((at[i] << 2) + zero, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        at[i] += u[i] > t[i] ? 1u : 0u;
        asm("" : "+v"(at[i]));
        t[i] = lds_read((at[i] << 2) + zero, 2 * H + 2);         // g.q
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) ip = fmaf(u[i], t[i], ip);       // (|u| |q|: u and its centroid have the same sign)
}

// eight indices side by side in one word, index i in bits 4 i .. 4 i + 3 (a sum, so that index + 1 = 16 may carry in between)
__device__ inline uint32_t pack_guesses(const uint32_t (&at)[8]) {
    uint32_t items = 0u - 0x11111111u * (kGuessBits + 1u);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        items += at[i] << (4 * i);
        asm("" : "+v"(items));
    }
    return items;
}

// ---- collecting ballots in lanes, and bit interleaving for the packed payload
__device__ inline uint32_t lo32(uint64_t x) { return (uint32_t)x; }
__device__ inline uint32_t hi32(uint64_t x) { return (uint32_t)(x >> 32); }
// v_writelane_b32 through its compiler intrinsic (this compiler has no builtin of that name): the compiler then
// also places the wait states an SGPR written by v_cmp needs before a vector instruction may read it.
extern "C" __device__ int eden_writelane_i32(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");
template <int LANE>
__device__ inline uint32_t put_lane(uint32_t value, uint32_t old) {      // old with lane LANE replaced by a wave-uniform value
    return (uint32_t)eden_writelane_i32((int)value, LANE, (int)old);
}
template <class F, int... I>
__device__ inline void static_for_impl(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ inline void static_for(F &&f) {                       // f(integral_constant<int, 0>) ... f(<N-1>)
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}
// The value of lane (l ^ X) of the same row of 16 lanes: data-parallel primitives where one exists for the pattern, the
// cross-lane swizzle of the LDS unit (no memory access) for X = 4.
template <int X>
__device__ inline uint32_t lane_xor_u32(uint32_t v) {
    static_assert(X == 1 || X == 2 || X == 4 || X == 8, "one lane bit");
    if constexpr (X == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);         // quad_perm [1,0,3,2]
    else if constexpr (X == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);    // quad_perm [2,3,0,1]
    else if constexpr (X == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, true);   // row_ror:8
    else return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x001F | (4 << 10));
}
// A word holds N = 32 / BITS items of BITS bits; the N lanes that differ only in their low log2 N lane bits transpose
// them: item i of lane j becomes item j of lane i.  One step per lane bit b: the two lanes of a pair swap the items
// whose index differs from their own side in bit b (a rotation by the width of 2^b items brings them into place; what it
// wraps around falls outside the mask).
template <int BITS, int B = 0>
__device__ inline uint32_t transpose_items(uint32_t x, uint32_t lane) {
    constexpr int N = 32 / BITS;
    if constexpr ((1 << B) >= N) {
        return x;
    } else {
        constexpr uint32_t width = (uint32_t)BITS << B;
        constexpr uint32_t unit = (1u << width) - 1u;
        uint32_t keep_low = 0;                               // items whose index has bit B clear
#pragma unroll
        for (uint32_t pos = 0; pos < 32u; pos += 2u * width) keep_low |= unit << pos;
        const uint32_t t = lane_xor_u32<(1 << B)>(x);
        const bool up = (lane >> B) & 1u;
        const uint32_t other = __builtin_amdgcn_alignbit(t, t, up ? width : 32u - width);
        const uint32_t mask = up ? ~keep_low : keep_low;
        return transpose_items<BITS, B + 1>((uint32_t)__builtin_amdgcn_bitop3_b32((int)mask, (int)x, (int)other, 0xCA), lane);   // mask ? x : other
    }
}
__device__ inline uint32_t even_bits(uint32_t x) {               // bits 0,2,4,..,30 -> bits 0..15
    x &= 0x55555555u;
    x = (x | (x >> 1)) & 0x33333333u;
    x = (x | (x >> 2)) & 0x0F0F0F0Fu;
    x = (x | (x >> 4)) & 0x00FF00FFu;
    return (x | (x >> 8)) & 0x0000FFFFu;
}
__device__ inline uint32_t spread2(uint32_t x) {                 // bit j of the low 16 -> bit 2j
    x &= 0xFFFFu;
    x = (x | (x << 8)) & 0x00FF00FFu;
    x = (x | (x << 4)) & 0x0F0F0F0Fu;
    x = (x | (x << 2)) & 0x33333333u;
    return (x | (x << 1)) & 0x55555555u;
}
__device__ inline uint32_t spread4(uint32_t x) {                 // bit j of the low 8 -> bit 4j
    x &= 0xFFu;
    x = (x | (x << 12)) & 0x000F000Fu;
    x = (x | (x << 6)) & 0x03030303u;
    return (x | (x << 3)) & 0x11111111u;
}

__device__ inline uint32_t spread3(uint32_t x) {                 // bit j of the low 11 -> bit 3j
    const uint32_t top = ((x >> 10) & 1u) << 30;
    x &= 0x3FFu;
    x = (x | (x << 16)) & 0x030000FFu;
    x = (x | (x << 8)) & 0x0300F00Fu;
    x = (x | (x << 4)) & 0x030C30C3u;
    x = (x | (x << 2)) & 0x09249249u;
    return x | top;
}
// 3-bit codes of 32 consecutive coordinates, given as three bit planes (bit i of plane k = bit k of code i),
// as the 96-bit little-endian string in which code i occupies bits 3i .. 3i+2
__device__ inline void pack3_planes(uint32_t p0, uint32_t p1, uint32_t p2, uint32_t (&out)[3]) {
    const uint32_t plane[3] = {p0, p1, p2};
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {                            // coordinates 11c .. 11c+10 start at bit 33c + k
            const uint64_t v = (uint64_t)spread3((plane[k] >> (11 * c)) & 0x7FFu) << ((33 * c + k) & 31);
            w[(33 * c + k) >> 5] |= (uint32_t)v;
            w[((33 * c + k) >> 5) + 1] |= (uint32_t)(v >> 32);
        }
    }
    out[0] = w[0]; out[1] = w[1]; out[2] = w[2];
}
// the `bits`-wide code that starts `shift` bits into the 64-bit little-endian window w1:w0
__device__ inline uint32_t code_at(uint32_t w0, uint32_t w1, uint32_t shift, int bits) {
    return __builtin_amdgcn_alignbit(w1, w0, shift) & ((1u << bits) - 1u);
}

// Centre of mass of N(0,1) on [delta (n - 1/2), delta (n + 1/2)], n >= 1; the interval of n = 127 runs to infinity
// (Sec. 3: the optimal value of an interval; Sec. 4.3: the uniform grid).
__device__ inline double grid_centroid(double delta, int n) {
    const double a = delta * (n - 0.5), b = delta * (n + 0.5);
    const bool open = n >= kGridMax;
    const double mass = 0.5 * (erfc(a * 0.7071067811865476) - (open ? 0.0 : erfc(b * 0.7071067811865476)));
    const double num = 0.3989422804014327 * (exp(-0.5 * a * a) - (open ? 0.0 : exp(-0.5 * b * b)));
    return mass > 0.0 ? num / mass : a;
}
// index of one coordinate on the uniform grid (as a signed byte in the low 8 bits) and its contribution |u| c to
// sum_i u_i Q_i; `ctab`: the centres of mass in LDS
// (a value on an interval endpoint goes to the interval closer to zero, Sec. 2.2.1 footnote: |n| = ceil(|z| / Delta - 1/2);
// the subtraction is exact for every quotient that matters, so the rounding of the quotient is the only error)
__device__ inline uint32_t quantize_grid(float u, float grid_inv, const float *ctab, float &ip) {
    const float m = fminf(ceilf(fabsf(u * grid_inv) - 0.5f), (float)kGridMax);
    const int mag = (int)m;                                      // -0.0 below half a step: 0
    ip = fmaf(fabsf(u), ctab[mag], ip);
    return (uint32_t)((__float_as_uint(u) >> 31) ? -mag : mag) & 0xFFu;
}
// value of a received byte: sign(n) * table[|n|]
__device__ inline float dequantize_grid(uint32_t byte, const float *dtab) {
    const int n = (int)(int8_t)byte;
    const int a = n < 0 ? -n : n;
    const float m = dtab[a > kGridMax ? kGridMax : a];           // (a sender never writes -128)
    return n < 0 ? -m : m;
}

// One-byte budgets.  `tab` in LDS: [0..127] the positive centroids (centres of mass), [128..255] the positive
// thresholds times |x| (b = 5..8 only; entries from H on are +inf).  b = 5..8: rank of |u| among the H - 1 positive
// thresholds by bisection over all 128 entries (seven reads, no branch: the padding never moves the rank), index =
// H + rank or H - 1 - rank (Sec. 2.2.1, Sec. 3).  GRID is a compile-time choice so that loops over many values
// stay free of branches (with a branch per value the compiler waits for every load before it issues the next).
template <bool GRID>
__device__ inline uint32_t quantize_byte(float u, uint32_t H, float grid_inv, const float *tab, float &ip) {
    if constexpr (GRID) {
        return quantize_grid(u, grid_inv, tab, ip);
    } else {
        const float a = fabsf(u);
        uint32_t mag = 0;
#pragma unroll
        for (uint32_t step = 64; step; step >>= 1) mag += (a > tab[128u + mag + step]) ? step : 0u;    // strict: ties stay closer to zero
        ip = fmaf(a, tab[mag], ip);
        return (__float_as_uint(u) >> 31) ? H - 1u - mag : H + mag;
    }
}
template <bool GRID>
__device__ inline float dequantize_byte(uint32_t byte, uint32_t H, const float *dtab) {
    if constexpr (GRID) {
        return dequantize_grid(byte, dtab);
    } else {
        const uint32_t code = byte & (2u * H - 1u);
        const float m = dtab[code >= H ? code - H : H - 1u - code];
        return code >= H ? m : -m;
    }
}
__device__ inline uint32_t wide_half_levels(uint32_t b_q8) { return wide_bits(b_q8) ? 1u << (wide_bits(b_q8) - 1u) : 0u; }

// b = K + 1/2 and the coin budgets (Sec. 4.1): one coordinate per lane, quantized with I_{K+1} in the lanes of `up` (the index has K+1
// bits there), else with I_K.  low[]: the low K bits of the index as lane masks, top: the bit above them (clear outside `up`).  Masks
// stand in scalar registers and are combined there; a value costs a select and a compare per step of a search in which both quantizers
// share their steps, and the sums.  (Counting the thresholds of both below |u| and putting both indices together took 36 vector
// instructions a value at K = 2, with the packing; this 17.)
// Measured (strided encode pass): 16 x 11,173,962 at b = 2.7 460 -> 372 us, b = 2.5 343 -> 251, b = 1.5 241 -> 217; 8 x 4,000,037 at b =
// 2.7 60.9 -> 50.3.
//   magnitude rank: in the lanes of `up` c0 c1 .. (K bits: 2^K - 1 thresholds), else c0 .. (K - 1 bits)
//   index before the sign: up 1, rank; else 1, rank; the sign turns all of its bits over
// Returns 4 times the entry of the centroid in a table that holds I_K's from entry 0 and I_{K+1}'s from entry 8 (qtab).
__device__ inline float select_where(uint64_t mask, float x, float y) { return __builtin_amdgcn_inverse_ballot_w64(mask) ? x : y; }
template <int K>
__device__ inline uint32_t quantize_two_tables(float u, uint64_t up, const Thresholds &th, uint64_t (&low)[K], uint64_t &top) {
    const float a = fabsf(u);
    uint64_t v[K];                                               // the low bits before the sign, v[0] the lowest
    if constexpr (K == 1) {
        v[0] = ~up | __ballot(a > th.thr2[1]);
    } else if constexpr (K == 2) {
        const uint64_t c0 = __ballot(a > select_where(up, th.thr2[2], th.thr[1]));
        const uint64_t c1 = __ballot(a > select_where(c0, th.thr2[3], th.thr2[1]));
        v[1] = ~up | c0;
        v[0] = (up & c1) | (~up & c0);
    } else {
        static_assert(K == 3, "budgets that exist");
        const uint64_t c0 = __ballot(a > select_where(up, th.thr2[4], th.thr[2]));
        const float above = select_where(up, th.thr2[6], th.thr[3]), below = select_where(up, th.thr2[2], th.thr[1]);
        const uint64_t c1 = __ballot(a > select_where(c0, above, below));
        const float upper = select_where(c1, th.thr2[7], th.thr2[5]), lower = select_where(c1, th.thr2[3], th.thr2[1]);
        const uint64_t c2 = __ballot(a > select_where(c0, upper, lower));
        v[2] = ~up | c0;
        v[1] = (up & c1) | (~up & c0);
        v[0] = (up & c2) | (~up & c1);
    }
    // entry 8 + rank, or rank = v without its leading 1
    uint32_t at = __builtin_amdgcn_inverse_ballot_w64(up) ? 32u : 0u - (4u << (K - 1));
#pragma unroll
    for (int b = 0; b < K; ++b) at += __builtin_amdgcn_inverse_ballot_w64(v[b]) ? 4u << b : 0u;
    const uint64_t neg = __ballot(__float_as_int(u) < 0);
#pragma unroll
    for (int b = 0; b < K; ++b) low[b] = v[b] ^ neg;
    top = up & ~neg;
    return at;
}
// The same for b = 2, 3, 4 alone (low: the whole index; entries 0 .. of qtab).  K = 3: 14 vector instructions a value with the packing,
// 23 while the thresholds below |u| were counted.  Encode of 4 x 100,000,001 at b = 3 1388 -> 1191 us, of 10 x 2^20 39.8 -> 35.6; of a
// launch of b = 1, 2, 3, 4 and 1.5 (16 x 11,173,962) 496 -> 457.
template <int K>
__device__ inline uint32_t quantize_one_table(float u, const Thresholds &th, uint64_t (&low)[K]) {
    static_assert(K >= 2 && K <= 4, "budgets that exist");
    const float a = fabsf(u);
    uint64_t v[K];
    v[K - 1] = ~0ull;
    if constexpr (K == 2) {
        v[0] = __ballot(a > th.thr[1]);
    } else if constexpr (K == 3) {
        v[1] = __ballot(a > th.thr[2]);
        v[0] = __ballot(a > select_where(v[1], th.thr[3], th.thr[1]));
    } else {
        v[2] = __ballot(a > th.thr[4]);
        v[1] = __ballot(a > select_where(v[2], th.thr[6], th.thr[2]));
        const float upper = select_where(v[1], th.thr[7], th.thr[5]), lower = select_where(v[1], th.thr[3], th.thr[1]);
        v[0] = __ballot(a > select_where(v[2], upper, lower));
    }
    uint32_t at = 0;
#pragma unroll
    for (int b = 0; b + 1 < K; ++b) at += __builtin_amdgcn_inverse_ballot_w64(v[b]) ? 4u << b : 0u;
    const uint64_t neg = __ballot(__float_as_int(u) < 0);
#pragma unroll
    for (int b = 0; b < K; ++b) low[b] = v[b] ^ neg;
    return at;
}
// adds |u| times the centroids of N values to ip: their reads go out together, one after the other every value would wait for the LDS
template <int N>
__device__ inline void add_centroids(const float *u, const uint32_t (&at)[N], const float *qtab, float &ip) {
    float q[N];
#pragma unroll
    for (int i = 0; i < N; ++i) q[i] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(qtab) + at[i]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) ip = fmaf(fabsf(u[i]), q[i], ip);
    asm volatile("" : "+v"(ip));                                 // (left to itself the compiler adds up at the end and keeps the values)
}
// the 32 coordinates of 16 pairs whose offset bits are `offs`: a mask of the chosen ones
__device__ inline uint32_t chosen_of_pairs(uint32_t offs) {
    const uint32_t second = spread2(offs);
    return (second << 1) | (second ^ 0x55555555u);
}

// ---- encode: what the quantizers derive from |x|^2
// After |x|^2 is known: the thresholds of I_b scaled to the unnormalised transform.
// z = eta R(x) = u / |x| (Sec. 2.2.1 with d -> D), so z > t  <=>  u > t |x|.  Threads 0..7 fill one table entry each.
__device__ inline void fill_enc_scratch(EncScratch *s, double n2, uint32_t b_q8, const DevTables *tab, uint32_t tid) {
    if (tid > 7u) return;
    int bits, k;
    budget_of(b_q8, bits, k);
    const double norm = sqrt(n2);
    if (tid == 0u) s->n2 = n2;
    if (grid_q15(b_q8)) {                                        // uniform grid: no table of thresholds, only the step
        if (tid == 0u) s->grid_inv = (float)(32768.0 / ((double)grid_q15(b_q8) * norm));
        return;
    }
    if (wide_bits(b_q8)) return;                                 // b = 5..8: the long tables are filled by fill_byte_tables
    const int finer = budget_two_tables(b_q8) ? bits + 1 : bits;
    s->thr[tid] = (float)(tab->t[bits][tid] * norm);
    s->qpos[tid] = (float)tab->q[bits][tid];
    s->thr2[tid] = (float)(tab->t[finer][tid] * norm);
    s->qpos2[tid] = (float)tab->q[finer][tid];
    if (bits == 4 && tid == 0u) {                                // r = a x + b x |x|, x = u / (the last threshold): r = 4, 7 at thresholds 4, 7
        const double t7 = tab->t[4][7], m = tab->t[4][4] / t7, b = (7.0 - 4.0 / m) / (1.0 - m), a = 7.0 - b;
        const double last = t7 * norm, up = last < 0x1p-60 ? 0x1p100 : last > 0x1p60 ? 0x1p-90 : 1.0;
        const bool usable = last > 0.0 && last < (double)INFINITY;
        const double per_u = usable ? 1.0 / (last * up) : 0.0;
        int top = 7;                                             // the last threshold that is a finite float
        while (top > 0 && !((float)(tab->t[4][top] * norm) < INFINITY)) --top;
        const double cap = top == 7 ? 1.1 : (sqrt(a * a + 4.0 * b * (top + 0.4)) - a) / (2.0 * b);
        s->guess_c1 = (float)(a * per_u);
        s->guess_c3 = (float)(b * per_u * per_u);
        s->guess_cap = usable ? (float)(cap * last * up) : 0.0f;
        s->guess_up = (float)up;
    }
}
__device__ inline void fill_grid_table(EncScratch *s, uint32_t q15, uint32_t tid) {
    s->grid_c[tid] = tid ? (float)grid_centroid((double)q15 / 32768.0, (int)tid) : 0.0f;
}
// b = wb = 5..8
__device__ inline void fill_wide_tables(EncScratch *s, uint32_t wb, double n2, const DevTables *tab, uint32_t tid) {
    const uint32_t H = 1u << (wb - 1u);
    s->grid_c[tid] = tid < H ? (float)tab->q_big[wb - 5u][tid] : 0.0f;
    s->wide_thr[tid] = tid < H ? (float)(tab->t_big[wb - 5u][tid] * sqrt(n2)) : INFINITY;       // padding for the bisection
}
// The tables of the one-byte budgets, one entry per thread (tid < 128): the centres of mass of the uniform grid's
// intervals, or the positive centroids and scaled thresholds of the 32..256-level quantizers.
__device__ inline void fill_byte_tables(EncScratch *s, uint32_t b_q8, double n2, const DevTables *tab, uint32_t tid) {
    if (tid > (uint32_t)kGridMax) return;
    if (const uint32_t q15 = grid_q15(b_q8)) fill_grid_table(s, q15, tid);
    else if (const uint32_t wb = wide_bits(b_q8)) fill_wide_tables(s, wb, n2, tab, tid);
}

// The sum of `count` partials in the order of 256 threads that take every 256th of them, whatever the workgroup's size: the same bits
// in every kernel that needs it.  `red`: 4 doubles in LDS; the result in every thread.
template <int THREADS>
__device__ inline double ordered_sum(const double *part, uint32_t count, double *red) {
    const uint32_t lane = lane_id();
    for (uint32_t w = threadIdx.x >> 6; w < 4u; w += THREADS / 64) {
        double s = 0.0;
        for (uint32_t i = 64u * w + lane; i < count; i += 256u) s += part[i];
        s = wave_sum(s);
        if (lane == 0) red[w] = s;
    }
    __syncthreads();
    const double total = ((0.0 + red[0]) + red[1]) + red[2] + red[3];
    __syncthreads();
    return total;
}
// The same by one wave alone, from partials that workgroups of this launch have stored.
__device__ inline double ordered_sum_through(const double *part, uint32_t count) {
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (uint32_t i = lane_id(); i < count; i += 256u)
#pragma unroll
        for (uint32_t w = 0; w < 4u; ++w)
            if (i + 64u * w < count) s[w] += __hip_atomic_load(part + i + 64u * w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int w = 0; w < 4; ++w) s[w] = wave_sum(s[w]);
    return ((0.0 + s[0]) + s[1]) + s[2] + s[3];
}
// The same in two steps, for a workgroup of 256 threads that issues the loads in front of those of its tile and adds while these are on
// their way (loads come back in order).
struct EarlyPartials {
    double x;
    __device__ inline void load(const double *part, uint32_t count /* <= 256 */) { x = threadIdx.x < count ? part[threadIdx.x] : 0.0; }
    // in every thread; `red`: 4 doubles in LDS
    __device__ inline double sum(double *red) const {
        const double s = wave_sum(x);
        if (lane_id() == 0) red[threadIdx.x >> 6] = s;
        __syncthreads();
        return ((0.0 + red[0]) + red[1]) + red[2] + red[3];
    }
};

// ---- encode: the header of a message (one thread).  `total`: sum_i u_i q_i.  A zero or non-finite vector gets S = 0 and a status bit.
// (<R(x),Q> = 0 can only happen on a uniform grid so coarse that every coordinate falls into the interval around 0.)
__device__ inline bool enc_valid_norm(double n2) { return n2 > 0.0 && n2 < INFINITY; }
__device__ inline void write_enc_header(const EncBatch &B, uint32_t c, uint64_t hdr_d, int log2D, uint64_t seed, double n2, double total,
                                        uint32_t *dev_status, const uint32_t *coin_total) {
    MsgHeader h;
    h.magic = kMagic; h.log2D = (uint32_t)log2D; h.d = hdr_d; h.b_q8 = B.hdr_b_q8[c]; h.client = B.client[c];
    h.extra_bits = coin_q8(B.b_q8[c]) ? coin_total[c] : 0u; h.seed = seed; h.N2 = n2;
    if (enc_valid_norm(n2) && total > 0.0) {
        h.IP = total * exp2(-0.5 * (double)log2D);               // <R(x),Q> = D^-1/2 sum u_i q_i
        h.S = n2 / h.IP;                                         // Sec. 2.3
        h.status = 0;
    } else {
        h.IP = 0.0; h.S = 0.0;
        h.status = (n2 >= 0.0 && n2 < INFINITY) ? EDEN_DEV_ZERO_VECTOR : EDEN_DEV_NONFINITE;
        atomicOr(dev_status, h.status);
    }
    *static_cast<MsgHeader *>(B.msg[c]) = h;
}

// ---- encode in two launches (D <= 2^20: the plans whose strided pass runs in wave tiles).  The thresholds need |x|^2, the sum over all
// workgroups of the first pass, and the header needs the sum over all workgroups of the last one; launches of their own for these sums
// cost 4 to 6 us each.  Instead
// - every workgroup of the last pass adds the partial sums of |x|^2 up again: the loads go out in front of those of its tile, and the
//   sum and the thresholds are ready about when the tile is there (the centres of mass of a uniform grid, which do not depend on
//   |x|, are left in `scratch` by the first pass);
// - the workgroup of a sender that finishes last writes the header.  Only the first wave of a workgroup waits for its partial sum
//   to reach memory, and every sender's counter has a memory line of its own (512 arrivals on neighbouring words took 36 us, on a
//   line per sender 10).
// Encode, us, launches of their own -> this: 10 senders of 2^20, b = 2 38.9 -> 34.3; 32 of 2^17, b = 2 25.2 -> 20.9; 24 of 300,007, b = 2
// 35.4 -> 30.8; 32 of 250,000, b = 1 23.8 -> 22.5; one of 20,000, b = 2 (where the workgroup that arrived last filled the thresholds,
// too) 14.1 -> 12.9.  The workgroup-tile passes (D >= 2^21) keep the separate launches: with 512 workgroups per sender the arrivals
// alone take longer, and adding up 684 partial sums per workgroup costs 16 senders of 2^24 at b = 4 9 us.
struct EncTail {
    uint32_t *arrived;      // kEncCounterStride words apart, a counter per sender, 0 between calls; null: launches of their own
    const double *part_n2;  // the partial sums of |x|^2, n2_stride apart per sender, n2_count <= 256 of them
    uint32_t n2_stride, n2_count;
    EncScratch *scratch;
    const DevTables *tab;
    uint64_t hdr_d;
    uint32_t *dev_status;
    const uint32_t *coin_total;
};
// first pass, one workgroup per sender: the counter of the last pass is cleared (it is 0 already unless calls overlapped against
// the rules), and a uniform grid gets its table.
template <int THREADS>
__device__ inline void enc_first_side(const EncTail &f, uint32_t c, uint32_t b_q8) {
    if (!f.arrived || blockIdx.x != 0) return;
    if (threadIdx.x == 0) f.arrived[c * kEncCounterStride] = 0u;
    if (grid_q15(b_q8))
        for (uint32_t i = threadIdx.x; i <= (uint32_t)kGridMax; i += THREADS) fill_grid_table(&f.scratch[c], grid_q15(b_q8), i);
}
// last pass, 256 threads: |x|^2 of the sender and what the quantizers derive from it, in LDS.  Barriers inside.
__device__ inline void enc_scratch_to_lds(const EncTail &f, uint32_t c, uint32_t b_q8, const EarlyPartials &early, EncScratch &s, double *red4) {
    const double n2 = early.sum(red4);
    if (b_q8 <= 256u) {
        if (threadIdx.x == 0) s.n2 = n2;
    } else {
        fill_enc_scratch(&s, n2, b_q8, f.tab, threadIdx.x);
        if (threadIdx.x <= (uint32_t)kGridMax) {
            if (wide_bits(b_q8)) fill_wide_tables(&s, wide_bits(b_q8), n2, f.tab, threadIdx.x);
            else if (grid_q15(b_q8)) s.grid_c[threadIdx.x] = f.scratch[c].grid_c[threadIdx.x];
        }
    }
    __syncthreads();
}
// What a message whose sums are unusable owes beside its header: a payload of zeros, `codes` the one-byte indices that it is packed
// from later.
template <int THREADS>
__device__ inline void zero_payload(const EncBatch &B, uint32_t c, int log2D, const uint32_t *coin_total, bool codes) {
    const uint32_t b_q8 = B.b_q8[c];
    int bits, k;
    budget_of(b_q8, bits, k);
    const uint64_t D = 1ull << log2D;
    uint32_t *dst = codes ? reinterpret_cast<uint32_t *>(B.codes[c])
                          : reinterpret_cast<uint32_t *>(static_cast<char *>(B.msg[c]) + EDEN_HEADER_BYTES);
    const uint64_t words = (codes ? D : payload_a_bytes(D, bits, k) + (coin_q8(b_q8) ? coin_b_bytes(coin_total[c]) : payload_b_bytes(D, b_q8))) / 4;
    for (uint64_t i = threadIdx.x; i < words; i += THREADS) dst[i] = 0u;
}
// Whether sum_i u_i q_i may turn out unusable (not positive, or NaN) although |x|^2 is usable.  Every value of the transform and
// of its stages is at most sqrt(D) |x|, so with D |x|^2 <= 2^254 nothing overflows in fp32 and no inf - inf arises; with |x| >= 2^-100
// no product of a value in an interval that does not touch 0 underflows.  (A grid so coarse that every index is 0 has a zero payload anyway.)
__device__ inline bool enc_sum_in_doubt(double n2, int log2D) {
    return enc_valid_norm(n2) && !(n2 >= 0x1p-200 && n2 * (double)(1ull << log2D) <= 0x1p254);
}
// last pass: the header; and the zero payload of a sender whose sum is unusable.  Other workgroups have stored pieces of that
// payload, some of them from other XCDs: where the sum is in doubt every workgroup therefore writes its L2 back before it arrives
// (no other sender pays for that), and the last one clears after it has seen them all.
template <int THREADS>
__device__ inline void enc_last_tail(const EncTail &f, const EncBatch &B, uint32_t c, int log2D, uint64_t seed, double n2,
                                     double block_total, double *part, uint32_t *flag) {
    double total;
    if (!enc_sum_in_doubt(n2, log2D)) {
        if (threadIdx.x >= 64u) return;                          // (no barrier from here on)
        uint32_t before = 0;
        if (threadIdx.x == 0) {
            __hip_atomic_store(part + blockIdx.x, block_total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the store has reached memory
            before = __hip_atomic_fetch_add(f.arrived + c * kEncCounterStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (__builtin_amdgcn_readfirstlane(before) + 1u != gridDim.x) return;
        if (threadIdx.x == 0) __hip_atomic_store(f.arrived + c * kEncCounterStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        total = ordered_sum_through(part, gridDim.x);
    } else {
        if (threadIdx.x == 0) __hip_atomic_store(part + blockIdx.x, block_total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        if (!arrive_last(f.arrived + c * kEncCounterStride, gridDim.x, flag)) return;
        total = ordered_sum_through(part, gridDim.x);            // (every wave the same)
        if (!(total > 0.0)) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            zero_payload<THREADS>(B, c, log2D, f.coin_total, wide_bits(B.b_q8[c]) != 0u && B.codes[c] != nullptr);
        }
    }
    if (threadIdx.x == 0) write_enc_header(B, c, f.hdr_d, log2D, seed, n2, total, f.dev_status, f.coin_total);
}
// The payload of a vector without a usable norm is all zero: what a row of a wave tile owes of it, the 64 coordinates from `first`
// on.  (The second part of a coin budget is cleared by a kernel of its own.)
__device__ inline void zero_payload_row(const EncBatch &B, uint32_t c, int log2D, uint64_t first) {
    const uint32_t b_q8 = B.b_q8[c];
    int bits, k;
    budget_of(b_q8, bits, k);
    char *payload = static_cast<char *>(B.msg[c]) + EDEN_HEADER_BYTES;
    const bool codes = wide_bits(b_q8) != 0u && B.codes[c] != nullptr;           // b = 5, 6, 7: one-byte indices, packed later
    uint32_t *dst = codes ? reinterpret_cast<uint32_t *>(B.codes[c] + first)
                          : reinterpret_cast<uint32_t *>(payload + first * (uint32_t)bits / 8u / (uint32_t)k);
    const uint32_t words = codes ? 16u : 2u * (uint32_t)bits / (uint32_t)k;
    for (uint32_t i = 0; i < words; ++i) dst[i] = 0;
    if (budget_mixed(b_q8)) reinterpret_cast<uint32_t *>(payload + payload_a_bytes(1ull << log2D, bits, 1))[first >> 6] = 0u;
}

// ---- operands of the matrix instructions (v_mfma_f32_32x32x16_f16 / _fp8_fp8).  Lane l = 32 h + m holds, of A (32 x 16), row m
// and k = 8 h .. 8 h + 7; of B (16 x 32), column m and the same k; of the 32 x 32 result, column m and rows
// 8 (r / 4) + 4 h + r % 4 in registers r = 0 .. 15 (checked on the device with random integer matrices).
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
// entry (a, b) of the Sylvester Hadamard matrix
__device__ inline _Float16 hadamard_entry(uint32_t a, uint32_t b) {
    return (__builtin_popcount(a & b) & 1) ? (_Float16)-1.0f : (_Float16)1.0f;
}
// the second operand of the second of two chained transforms: the 16 result registers of the first product (rows of D1 in
// the order above) are, packed to fp16 in pairs, the B operands of two instructions (registers 0..7 and 8..15); entry e of
// instruction q on lane (h, m) of the Hadamard A operand must then stand for row 16 q + 8 (e / 4) + 4 h + e % 4
__device__ inline half8_t hadamard_rows_of_result(uint32_t q, uint32_t h, uint32_t m) {
    half8_t r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = hadamard_entry(16u * q + 8u * ((uint32_t)e >> 2) + 4u * h + ((uint32_t)e & 3u), m);
    return r;
}

// ---- narrow decode workspace.  After the strided pass of a two-pass size the values of a b <= 1 sender are integers of
// magnitude at most 2^10 (+-1 or 0 through at most ten butterfly stages): the workspace holds them as fp16, which is exact
// (11 significant bits) and is the operand type of the matrix-core pass that reads them back.
__device__ inline short narrow_bits(float v) { return __builtin_bit_cast(short, (_Float16)v); }
__device__ inline float narrow_value(short bits) { return (float)__builtin_bit_cast(_Float16, bits); }
// two int16 in one register -> two fp16, in place (written out: the compiler converts into two registers and packs them)
__device__ inline uint32_t narrow_pair_from_int16(uint32_t w) {
    asm("v_cvt_f16_i16_sdwa %0, %0 dst_sel:WORD_0 dst_unused:UNUSED_PRESERVE src0_sel:WORD_0\n\t"
        "v_cvt_f16_i16_sdwa %0, %0 dst_sel:WORD_1 dst_unused:UNUSED_PRESERVE src0_sel:WORD_1"
        : "+v"(w));
    return w;
}

// ---- blocked layout of the encoder's workspace between the contiguous pass over P bits and a workgroup-tile strided pass that
// covers all the bits above it.  Element (row r, column block cb of 32 coordinates, column) of a sender's slot sits, in
// floats, at ((r / R) * 512 + cb) * (R * 32) + (r % R) * 32 + column with R = kBlockRows: the 128-byte segments of R
// consecutive rows are interleaved.  Row-major would be r * 2^14 + cb * 32 + column.  (P = 14; rows of 2^P coordinates have 2^(P-5)
// column blocks.)  (At 16 senders of 2^24: R = 4 took the strided pass from 170 to 156 us and left the contiguous pass where it was; R =
// 8 slowed both passes by 10 us.)
constexpr uint32_t kBlockRows = 4;
constexpr uint32_t kBlockRowBits = 2;
template <int P>
__host__ __device__ inline size_t blocked_offset(uint32_t row, uint32_t cb) {
    return ((size_t)(row >> kBlockRowBits) << (P + kBlockRowBits)) + ((size_t)cb << (5 + kBlockRowBits)) +
           ((size_t)(row & (kBlockRows - 1u)) << 5);
}

// ---- coin budgets: positions in the second part of the payload
// coins before the block of 64 coordinates number w of sender slot c
__device__ inline uint32_t coins_before(const CoinTables &ct, uint32_t c, int log2D, uint32_t w) {
    return ct.group[(size_t)c * ct.group_stride + w / (uint32_t)kCoinGroup] + ct.local[((size_t)c << (log2D - 6)) + w];
}
__device__ inline uint64_t coin_mask_of(const CoinTables &ct, uint32_t c, int log2D, uint32_t w) {
    return ct.mask[((size_t)c << (log2D - 6)) + w];
}
// set bits of `mask` below this lane's position
__device__ inline uint32_t lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi(hi32(mask), __builtin_amdgcn_mbcnt_lo(lo32(mask), 0u));
}
// Bits of a word to and from the set positions of `mask`, in order, by moves of 1, 2, 4, 8 and 16 places (the parallel suffix method of
// Warren's Hacker's Delight, chapter 7): step i moves what has an odd number of multiples of 2^i clear positions below it.  About 85
// instructions whatever the mask; a loop over the set bits took ten for each of the most that a lane of the wave had (strided encode pass
// of 8 senders of 4,000,037 at 2.7 bits 47.5 -> 41.5 us).
struct BitMoves {
    uint32_t step[5];                                            // in step i these move by 2^i
    __device__ inline explicit BitMoves(uint32_t mask) {
        uint32_t below = ~mask << 1;                             // clear positions below: those that still count
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            uint32_t odd = below;
#pragma unroll
            for (int s = 1; s < 32; s <<= 1) odd ^= odd << s;
            step[i] = odd & mask;
            mask = (mask ^ step[i]) | (step[i] >> (1 << i));
            below &= ~odd;
        }
    }
};
// the bits of `value` at the set positions of `mask`, moved together towards bit 0 in the same order
__device__ inline uint32_t compress_bits(uint32_t value, uint32_t mask) {
    const BitMoves moves(mask);
    value &= mask;
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const uint32_t moved = value & moves.step[i];
        value = (value ^ moved) | (moved >> (1 << i));
    }
    return value;
}
__device__ inline uint64_t compress_bits(uint64_t value, uint64_t mask) {
    return compress_bits(lo32(value), lo32(mask)) | (uint64_t)compress_bits(hi32(value), hi32(mask)) << __popc(lo32(mask));
}
// the other way round: bit k of `value` at the set position number k of `mask`
__device__ inline uint32_t expand_bits(uint32_t value, uint32_t mask) {
    const BitMoves moves(mask);
#pragma unroll
    for (int i = 4; i >= 0; --i)
        value = (uint32_t)__builtin_amdgcn_bitop3_b32((int)moves.step[i], (int)(value << (1 << i)), (int)value, 0xCA);      // step ? moved : value
    return value & mask;
}
// ORs the low `count` bits of `value` (the others are zero) into a zeroed little-endian bit string at bit `off`.  The string
// starts on an 8-byte boundary (the second part of a payload does) and is a whole number of 8-byte words long: 64-bit atomics,
// one per piece unless the piece straddles a word (about a third fewer than with 32-bit ones; they are what this costs).
__device__ inline void or_bits(uint32_t *words, uint32_t off, uint64_t value, uint32_t count) {
    if (!count) return;
    unsigned long long *q = reinterpret_cast<unsigned long long *>(words) + (off >> 6);
    const uint32_t sh = off & 63u;
    const unsigned long long lo = value << sh, hi = sh ? value >> (64u - sh) : 0ull;
    if (lo) atomicOr(q, lo);
    if (hi) atomicOr(q + 1, hi);
}

// Butterflies over the low LOGB bits of the register index only (FIRST = 2: all but the stage over bit 0).
template <int N, int LOGB, int FIRST = 1>
__device__ inline void fwht_regs_low(float (&v)[N]) {
#pragma unroll
    for (int h = FIRST; h < (1 << LOGB); h <<= 1) {
#pragma unroll
        for (int i = 0; i < N; i += 2 * h) {
#pragma unroll
            for (int j = i; j < i + h; ++j) {
                const float a = v[j], b = v[j + h];
                v[j] = a + b;
                v[j + h] = a - b;
            }
        }
    }
}

// ---- decode: what the receiver derives from a message's header and its packet bitmap
//
// One wave per message: check the header against what the receiver agreed on, count the coordinates
// that arrived (Sec. 4.2: the receiver finds p by counting), and build the dequantization table
// (S / (p sqrt(D))) * q_l  -- S/p from Sec. 4.2, D^-1/2 from the inverse rotation.
// `hdr_d`, `hdr_b_q8`: what the header must say; `b_q8`: the budget the kernels dequantize with.
// `extra_bits`: coin budgets only, the number of coins the receiver counted itself; the header must agree.
__device__ inline void dec_prepare_wave(const void *msg, const uint32_t *bitmap, uint32_t client, uint32_t b_q8,
                                        uint32_t hdr_b_q8, uint64_t hdr_d, int log2D, uint64_t seed, const DevTables *tab,
                                        DecScratch *out, uint32_t *dev_status, uint32_t extra_bits = 0,
                                        uint32_t *msg_flag = nullptr) {
    const uint32_t lane = lane_id();
    const MsgHeader h = *static_cast<const MsgHeader *>(msg);
    uint32_t flags = 0;
    if (h.magic != kMagic || h.log2D != (uint32_t)log2D || h.d != hdr_d || h.b_q8 != hdr_b_q8 ||
        h.client != client || h.seed != seed || (coin_q8(b_q8) && h.extra_bits != extra_bits))
        flags |= EDEN_DEV_HEADER_MISMATCH;
    else
        flags |= h.status & (EDEN_DEV_ZERO_VECTOR | EDEN_DEV_NONFINITE);
    const uint64_t D = 1ull << log2D;
    const uint32_t npk = D >= EDEN_PACKET_COORDS ? (uint32_t)(D / EDEN_PACKET_COORDS) : 1u;
    uint32_t got = 0;
    if (bitmap) {
        const uint32_t nw = (npk + 31u) / 32u;
        for (uint32_t w = lane; w < nw; w += 64) {
            uint32_t bits = bitmap[w];
            if (w == nw - 1 && (npk & 31u)) bits &= (1u << (npk & 31u)) - 1u;
            got += __popc(bits);
        }
        got = wave_sum_u32(got);
    } else {
        got = npk;
    }
    int bits, k;
    budget_of(b_q8, bits, k);
    const uint64_t per_packet = D >= EDEN_PACKET_COORDS ? EDEN_PACKET_COORDS : D;
    const uint64_t arrived = (uint64_t)got * per_packet / (uint64_t)k;
    if (flags == 0 && arrived == 0) flags |= EDEN_DEV_NOTHING_ARRIVED;
    double coef = 0.0;
    if (flags == 0) coef = h.S * exp2(0.5 * (double)log2D) / (double)arrived;     // S / (p sqrt(D)), p = arrived / D
    if (sparse_m(hdr_b_q8)) coef *= 64.0 / (double)sparse_m(hdr_b_q8);             // the 1/p of the sparsification (Sec. 4.1)
    if (lane < 32) {                                             // lanes 16..31: the finer table of a mixed budget
        const int tb = (lane < 16 || !budget_two_tables(b_q8)) ? bits : bits + 1;
        const int H = 1 << (tb - 1), l = (int)(lane & 15u);
        double q = 0.0;
        if (l < 2 * H) q = (l >= H) ? tab->q[tb][l - H] : -tab->q[tb][H - 1 - l];
        if (lane < 16) out->deq[l] = (float)(coef * q);
        else out->deq2[l] = (float)(coef * q);
    }
    if (grid_q15(b_q8)) {                                        // uniform grid: the centres of mass, two per lane
        const double delta = (double)grid_q15(b_q8) / 32768.0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int n = (int)lane + 64 * h;
            out->grid_deq[n] = n ? (float)(coef * grid_centroid(delta, n)) : 0.0f;
        }
    } else if (const uint32_t wb = wide_bits(b_q8)) {            // b = 5..8: the positive centroids, two per lane
#pragma unroll
        for (int h = 0; h < 2; ++h) out->grid_deq[lane + 64 * h] = (float)(coef * tab->q_big[wb - 5u][lane + 64 * h]);
    }
    if (lane == 0) {
        out->flags = flags;
        if (msg_flag) *msg_flag = flags;                         // per message, for eden_last_decode_flags
        if (dev_status && (flags & (EDEN_DEV_HEADER_MISMATCH | EDEN_DEV_NOTHING_ARRIVED))) atomicOr(dev_status, flags);
    }
}

// What dec_prepare_wave needs besides the batch, for a first decode pass that does the work of launch_dec_prepare itself.
struct DecPrepareArgs {
    uint64_t hdr_d, seed;
    const DevTables *tab;
    DecScratch *scratch;
    uint32_t *dev_status;
    uint32_t *msg_flags;                 // null or one word per sender of the batch
};

}  // namespace eden
#endif
