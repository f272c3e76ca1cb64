// The contiguous passes for D <= 2^24 (gfx950): the encoder's over 12 or 14 bits, the decoder's over 14.
//
// A workgroup owns 2^12 or 2^14 consecutive coordinates.  The encoder's transform is EncLo here, the decoder's lo_forward16 of eden_lo.h;
// where all values of a decode launch are small integers, ten of the 14 bits run on the matrix cores.  The encode pass is bound by memory
// where a launch fills the chip (16 senders of 11,173,962: 1.43 GB at 6.2 TB/s) and by the length of a wave's chain and the waves to be
// started where it does not: encode of one sender of 20,000, b = 2 12.9 -> 10.5 us, 8 of 131,072 15.2 -> 13.0 with four waves of 16 values
// per lane for 4096 coordinates instead of one of 64.
#include "eden_device.h"
#include "eden_kernels.h"
#include "eden_lo.h"

namespace eden {

constexpr int kLo14Bits = 14;

// The encoder's transform of a tile of 2^P coordinates, VALUES of them per thread: three groups of stages in registers,
// exchanges through LDS between them, the first between all waves, the others inside a wave, in the place this wave alone has just read.
// The order of the stages is part of the results: sums round differently in another one, and an index next to a threshold moves
// (8e-6 of the bytes at b = 8).  It is 6 .. 11, 0 .. 5 for P = 12 and 9 .. 13, 4 .. 8, 0 .. 3 for P = 14, and the groups are cut so
// that the bits a group needs are the ones the exchange before it can bring into registers.  Against passes that went from the top
// bit down (encode, us): one sender of 20,000, b = 2 9.9 and 9.8; 32 of 250,000, b = 1 23.4 and 23.3; one of 300,007, b = 1 12.4 and 12.2; 10 of
// 2^20, b = 2 32.6 -> 31.1; 2 of 4,000,037, b = 2 31.9 -> 28.7; 8 of them, b = 8 114.5 -> 110.3; one of 8,000,000, b = 1 29.3 -> 25.9; 16 of
// 11,173,962, b = 1 373 and 372, one of them 37.2 -> 35.9, 16 with pairs before the rotation 234 -> 240.
//   wave_at(wv) + lane + STEP a   coordinate in the tile of v[a] on entry: a register of a wave is 64 consecutive coordinates
//   quad(wv, lane, j)             first coordinate of x[j] on return
template <int P, int WAVES> struct EncLo;

//   P = 12  4 waves, 16 values: registers 6..9 | 10, 11, 0, 1 | 2..5; the waves are bits 10 and 11 before and bits 8 and 9 after the first exchange.
//   A row of 64 coordinates keeps its place in LDS; its 16 quads are swizzled by bits 6, 7, 10, 11, so that both directions of the other
//   exchanges, quads of bits 0 and 1 on one side and registers of bits 2..5 on the other, are free of bank conflicts.
template <> struct EncLo<12, 4> {
    static constexpr uint32_t VALUES = 16, STEP = 64;
    static __device__ inline uint32_t wave_at(uint32_t wv) { return 1024u * wv; }
    static __device__ inline uint32_t quad(uint32_t wv, uint32_t lane, uint32_t j) { return 1024u * j + 256u * wv + 4u * lane; }
    static __device__ inline void forward(float (&v)[16], float *lds, float4 (&x)[4]) {
        const uint32_t lane = lane_id(), wv = wave_in_block();
        fwht_regs<16>(v);                                        // bits 6..9
#pragma unroll
        for (uint32_t a = 0; a < 16; ++a) lds[wave_at(wv) + STEP * a + lane] = v[a];
        __syncthreads();
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {                       // j: bits 10, 11
            const float4 y = *reinterpret_cast<const float4 *>(&lds[quad(wv, lane, j)]);
            v[j] = y.x; v[j + 4] = y.y; v[j + 8] = y.z; v[j + 12] = y.w;
        }
        fwht_regs<16>(v);                                        // bits 10, 11, 0, 1
        // quad lane & 15 of row 16 j + 4 wv + (lane >> 4), swizzled by bits 6, 7 (lane >> 4) and 10, 11 (j)
        const uint32_t mine = 256u * wv + 64u * (lane >> 4) + 4u * ((lane & 15u) ^ (lane >> 4));
        wave_lds_sync();
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j)
            *reinterpret_cast<float4 *>(&lds[1024u * j + (mine ^ (16u * j))]) = make_float4(v[j], v[j + 4], v[j + 8], v[j + 12]);
        wave_lds_sync();
        // lane: bits 0, 1, 6, 7, 10, 11; register r: bits 2..5
        const uint32_t one = 1024u * (lane >> 4) + 256u * wv + 64u * ((lane >> 2) & 3u) + (lane & 3u) + 4u * (lane >> 2);
#pragma unroll
        for (uint32_t r = 0; r < 16; ++r) v[r] = lds[one ^ (4u * r)];
        fwht_regs<16>(v);                                        // bits 2..5
        wave_lds_sync();
#pragma unroll
        for (uint32_t r = 0; r < 16; ++r) lds[one ^ (4u * r)] = v[r];
        wave_lds_sync();
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) x[j] = *reinterpret_cast<const float4 *>(&lds[1024u * j + (mine ^ (16u * j))]);
    }
};

//   P = 14  8 waves, 32 values: registers 9..13 | 4..8 | 0 and 1, then 2 and 3 between the lanes of a quad; the waves are bits 6..8 before and
//   11..13 after the first exchange.  Bits 4 and 5 of the place in LDS are swizzled by bits 9 and 10 (no bank conflicts in any direction).
//   The values leave as quads of bits 0 and 1 without a further exchange.
template <> struct EncLo<14, 8> {
    static constexpr uint32_t VALUES = 32, STEP = 512;
    static __device__ inline uint32_t wave_at(uint32_t wv) { return 64u * wv; }
    static __device__ inline uint32_t quad(uint32_t wv, uint32_t lane, uint32_t j) { return 2048u * wv + 256u * j + 4u * lane; }
    static __device__ inline void forward(float (&v)[32], float *lds, float4 (&x)[8]) {
        const uint32_t lane = lane_id(), wv = wave_in_block();
        fwht_regs<32>(v);                                        // bits 9..13
#pragma unroll
        for (uint32_t a = 0; a < 32; ++a) lds[wave_at(wv) + STEP * a + (lane ^ (16u * (a & 3u)))] = v[a];
        __syncthreads();
        // lane: bits 0..3, 9, 10; register r: bits 4..8
        const uint32_t one = 2048u * wv + 512u * (lane >> 4) + (lane & 15u) + 16u * (lane >> 4);
#pragma unroll
        for (uint32_t r = 0; r < 32; ++r) v[r] = lds[(one ^ (16u * (r & 3u))) + 64u * (r >> 2)];
        fwht_regs<32>(v);                                        // bits 4..8
        wave_lds_sync();
#pragma unroll
        for (uint32_t r = 0; r < 32; ++r) lds[(one ^ (16u * (r & 3u))) + 64u * (r >> 2)] = v[r];
        wave_lds_sync();
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j) {                       // j: bits 8..10; lane: bits 2..7
            const float4 y = *reinterpret_cast<const float4 *>(&lds[quad(wv, lane, j) ^ (16u * (j >> 1))]);
            const float p = y.x + y.y, q = y.x - y.y, r = y.z + y.w, s = y.z - y.w;              // bit 0
            x[j] = make_float4(p + r, q + s, p - r, q - s);                                      // bit 1
        }
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j) { quad_stage<1>(x[j]); quad_stage<2>(x[j]); }           // bits 2, 3
    }
};

//   P = 14  16 waves, 16 values: registers 9..12 | 13, 4, 5, 6 | 7, 8, 0, 1, then 2 and 3 between the lanes of a quad; the waves are bits
//   6, 7, 8, 13 before and 9..12 after the first exchange.  Bits 4 and 5 of the place in LDS are swizzled by bits 7 and 8.
template <> struct EncLo<14, 16> {
    static constexpr uint32_t VALUES = 16, STEP = 512;
    static __device__ inline uint32_t wave_at(uint32_t wv) { return 8192u * (wv >> 3) + 64u * (wv & 7u); }
    static __device__ inline uint32_t quad(uint32_t wv, uint32_t lane, uint32_t j) {
        return 8192u * (lane >> 5) + 512u * wv + 128u * j + 4u * (lane & 31u);
    }
    static __device__ inline void forward(float (&v)[16], float *lds, float4 (&x)[4]) {
        const uint32_t lane = lane_id(), wv = wave_in_block();
        fwht_regs<16>(v);                                        // bits 9..12
        const uint32_t from = wave_at(wv) + (lane ^ (16u * ((wv >> 1) & 3u)));
#pragma unroll
        for (uint32_t a = 0; a < 16; ++a) lds[from + STEP * a] = v[a];
        __syncthreads();
        // lane: bits 0..3, 7, 8; register r: bits 13, 4, 5, 6
        const uint32_t one = 512u * wv + 128u * (lane >> 4) + (lane & 15u) + 16u * (lane >> 4);
#pragma unroll
        for (uint32_t r = 0; r < 16; ++r) v[r] = lds[(one ^ (16u * ((r >> 1) & 3u))) + 8192u * (r & 1u) + 64u * (r >> 3)];
        fwht_regs<16>(v);                                        // bits 13, 4, 5, 6
        wave_lds_sync();
#pragma unroll
        for (uint32_t r = 0; r < 16; ++r) lds[(one ^ (16u * ((r >> 1) & 3u))) + 8192u * (r & 1u) + 64u * (r >> 3)] = v[r];
        wave_lds_sync();
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {                       // j: bits 7, 8; lane: bits 2..6, 13
            const float4 y = *reinterpret_cast<const float4 *>(&lds[quad(wv, lane, j) ^ (16u * j)]);
            v[j] = y.x; v[j + 4] = y.y; v[j + 8] = y.z; v[j + 12] = y.w;
        }
        fwht_regs<16>(v);                                        // bits 7, 8, 0, 1
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
            x[j] = make_float4(v[j], v[j + 4], v[j + 8], v[j + 12]);
            quad_stage<1>(x[j]);                                 // bit 2
            quad_stage<2>(x[j]);                                 // bit 3
        }
    }
};

// Encode, first pass: x -> T.  Zero padding (Sec. 5: the transform needs a power of two), the sign diagonal of
// the rotation from the shared seed (Sec. 2.1), |x|^2 for eta and S (Sec. 2.2.1, 2.3), index bits 0 .. P-1 of H, P = 12 or 14.
// Only the ceil(d / 2^P) tiles that hold part of x (rounded up to whole blocks of rows in the blocked layout) are
// transformed and written: a tile of padding stays zero under these bits, and the strided pass that follows reads it
// as zero through its buffer bounds.
// PRE (b = 1/2 with the sparsification first, Sec. 4.1): the vector that is transformed is x'[g] = 2 x[2g + o_g],
// g < ceil(d_src/2), o_g from the SUB-SAMPLING stream; x is read as 0 beyond d_src.
// KEEP: x and the workspace of the launch fit the memory-side cache together: the loads of x leave it there, see launch_enc_lo_first.
// WAVES: of a workgroup.  |x|^2 is the same to the last bit for both numbers at P = 14: eight waves keep the sums of the two values of
// bit 13, which tell sixteen waves apart, to themselves.
template <int P, int WAVES, bool PRE, bool BLOCKED, bool KEEP>
__global__ __launch_bounds__(64 * WAVES, WAVES == 8 ? 4 : 8) void k_enc_lo_first(EncBatch B, uint64_t d_src, int log2D, uint64_t seed, float *T,
                                                            double *partials, uint32_t partial_stride, EncTail tail) {
    using L = EncLo<P, WAVES>;
    constexpr int N = (int)L::VALUES;
    __shared__ __attribute__((aligned(16))) float lds[1 << P];
    __shared__ double red[WAVES * N / 16];
    const uint32_t c = blockIdx.y, lane = lane_id();
    const uint32_t wv = wave_in_block();
    const rsrc_t rx = make_rsrc(B.x[c], (uint32_t)(d_src * 4));           // reads past d_src give the zero padding
    float *Tc = T + ((size_t)c << log2D);
    const uint32_t tile = blockIdx.x;                            // one tile per workgroup: the phases of two workgroups on a CU
                                                                 // interleave better than two tiles in one workgroup with the
                                                                 // second one's loads issued early
    // register a of this wave is 64 consecutive coordinates = one sign word; lane l hashes the word of register l % N.  With PRE an
    // element comes from x[2 i + o_i], and the register is 64 pairs = one word of offsets
    const uint32_t first = (tile << P) + L::wave_at(wv);
    const uint64_t word = (first >> 6) + (L::STEP / 64u) * (lane & (uint32_t)(N - 1));
    float u[N];
    if constexpr (PRE) {
        const uint64_t offs = hash_word(stream_key(seed, kStreamSubsample, B.client[c]), word);
#pragma unroll
        for (int a = 0; a < N; ++a) {
            const uint32_t odd = __builtin_amdgcn_inverse_ballot_w64(wave_read64(offs, a)) ? 4u : 0u;
            u[a] = 2.0f * buf_load(rx, 8u * lane + odd, 8u * (first + L::STEP * a));
        }
    } else {
#pragma unroll
        for (int a = 0; a < N; ++a) {
            const uint32_t at = 4u * (first + L::STEP * a);
            u[a] = KEEP ? buf_load_keep(rx, 4u * lane, at) : buf_load(rx, 4u * lane, at);
        }
    }
    const uint64_t mine = hash_word(stream_key(seed, kStreamSign, B.client[c]), word);
    double n2[N / 16] = {};
#pragma unroll
    for (int a = 0; a < N; ++a) {
        n2[a / 16] += (double)u[a] * (double)u[a];
        if ((a & 7) == 7) __builtin_amdgcn_sched_barrier(0);     // keeps the widened values of one group live at a time
    }
#pragma unroll
    for (int a = 0; a < N; ++a) u[a] = negate_where(u[a], wave_read64(mine, a)) + 0.0f;   // + 0: no negative zeros
    // whole lines leave: the lanes of a wave hold consecutive quads.  BLOCKED: the 128-byte segments of kBlockRows
    // consecutive rows are interleaved (see blocked_offset).  (Write-back stores: with the streaming hint this pass ran 13% slower; the pass
    // that reads the tiles back does better with the hint on its loads.)
    float4 x[N / 4];
    L::forward(u, lds, x);
#pragma unroll
    for (uint32_t j = 0; j < (uint32_t)N / 4u; ++j) {
        const uint32_t at = L::quad(wv, lane, j);
        *reinterpret_cast<float4 *>(Tc + (BLOCKED ? blocked_offset<P>(tile, at >> 5) + (at & 31u) : ((size_t)tile << P) + at)) = x[j];
    }
#pragma unroll
    for (int i = 0; i < N / 16; ++i) {
        const double sum = wave_sum(n2[i]);
        if (lane == 0) red[i * WAVES + wv] = sum;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double total = 0.0;
#pragma unroll
        for (int i = 0; i < WAVES * N / 16; ++i) total += red[i];
        partials[(size_t)c * partial_stride + blockIdx.x] = total;
    }
    enc_first_side<64 * WAVES>(tail, c, B.b_q8[c]);
}

// Decode, last pass: index bits 0..13 of H for every sender, that sender's sign diagonal (R^-1 = s o D^-1/2 H,
// Sec. 2.2.2), sum over senders in registers, one contiguous read-modify-write of acc.
// `narrow`: senders with b <= 1 have an fp16 workspace holding exact integers; their magnitude S/(p sqrt D) q_1
// is applied together with the sign.
//
// Work split.  A workgroup's time is proportional to the senders it sums and the chip holds `2 x CUs` of these
// workgroups at once, so a tile count far below that would leave most of the chip idle.  The first `full_tiles`
// tiles get one workgroup each that sums all n senders into acc.  Each of the remaining tiles gets K workgroups: group 0 sums its share
// of the senders into acc, group k > 0 stores its sum in partial[k-1][tile - full_tiles][2^14]; k_dec_lo14_combine then adds those to acc
// in the order k = 1, 2, ... (fixed, so the result does not depend on scheduling).
//
// `separate`: K = n, one sender per workgroup, nothing is summed: every sender's decoded tile goes to its slot of `partial`, for a
// caller that puts the values elsewhere afterwards (fp32 slots: possibly the workspace itself, in place; the workgroup has
// read the tile before it writes it).
// WIDE_ONLY: no sender of the launch has an fp16 slot (every b > 1): the instance without that branch in the sender loop.
// AHEAD: the values of sender c + 1 are on their way while those of sender c are transformed, for the launches that do not split
// tiles (whole decode at b = 4, us, with / without: 4 senders of 11,173,962 92 / 95, 16 298 / 305; with split tiles the other workgroup
// of the CU fills that time: 10 of 2^20, b = 2 36.9 / 34.9).
//
// 16 values per thread, 64 registers, two workgroups of 16 waves per CU.  With 32 values in 8 waves (116 registers, half as many
// waves), whole decode: 8 senders of 300,007, b = 2 26.9 -> 23.5 us; one of 11,173,962, b = 4 65 -> 43, 16 of them 314 -> 299; 32 of 2^20 with
// 1/2, 1, 2 and 4 bits 83 -> 77.
template <bool WIDE_ONLY, bool AHEAD>
__global__ __launch_bounds__(1024, 8) void k_dec_lo14_last(DecBatch B, uint32_t n, uint64_t d, int log2D, uint64_t seed,
                                                       const float *T, const DecScratch *scratch, int narrow_arg, float *acc,
                                                       uint32_t full_tiles, uint32_t K, uint32_t split_tiles,
                                                       float *partial, int separate, float mean_n) {
    __shared__ __attribute__((aligned(16))) float lds[Lo16<14>::LDS_FLOATS];
    // Four threads share a word of the SIGN stream.  Where four waves hash all of them by turns, for the others, the launches that do not
    // split tiles are faster (16 of 11,173,962, b = 4 297 against 291 us, 32 of 2^20 with 1/2, 1, 2 and 4 bits 66.0 / 64.5), those that
    // do slower (8 of 4,000,037, b = 3 74.9 / 76.5): there every thread hashes its own.
    constexpr bool BY_TURNS = AHEAD || !WIDE_ONLY;
    __shared__ uint32_t words[2][BY_TURNS ? 1 << (kLo14Bits - 5) : 1];           // in halves
    const int narrow = WIDE_ONLY ? 0 : narrow_arg;
    const uint32_t t = threadIdx.x, lane = t & 63u, wv = wave_in_block();
    uint32_t tile = blockIdx.x, c_begin = 0, c_end = n;
    float *part_tile = nullptr;                                  // this tile in the partial buffer
    if (blockIdx.x >= full_tiles) {
        const uint32_t idx = blockIdx.x - full_tiles, k = idx % K;
        tile = full_tiles + idx / K;
        c_begin = __builtin_amdgcn_readfirstlane(n * k / K);
        c_end = __builtin_amdgcn_readfirstlane(n * (k + 1u) / K);
        if (separate) part_tile = partial + ((size_t)k << log2D) + ((size_t)tile << kLo14Bits);
        else if (k > 0) part_tile = partial + (((size_t)(k - 1) * split_tiles + (tile - full_tiles)) << kLo14Bits);
    }
    const uint32_t tile_base = tile << kLo14Bits;
    float sum[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) sum[e] = 0.0f;

    auto load = [&](uint32_t c, float (&dst)[16]) {
        if (narrow && B.b_q8[c] <= 256u) {
            const rsrc_t r16 = make_rsrc(T + ((size_t)c << log2D), 2u << log2D);
#pragma unroll
            for (int a = 0; a < 16; ++a)
                dst[a] = __uint_as_float((uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r16, (int)(t * 2u), (int)((tile_base + 1024u * a) * 2u), kStream));
        } else {
            const rsrc_t r32 = make_rsrc(T + ((size_t)c << log2D), 4u << log2D);
#pragma unroll
            for (int a = 0; a < 16; ++a) dst[a] = buf_load(r32, t * 4u, (tile_base + 1024u * a) * 4u);
        }
    };
    float next[16];
    if (AHEAD && c_begin < c_end) load(c_begin, next);
    for (uint32_t c = c_begin; c < c_end; ++c) {
        const bool i16 = narrow && B.b_q8[c] <= 256u;
        if (!AHEAD) load(c, next);
        if (BY_TURNS && (wv >> 2) == (c & 3u)) {
            const uint64_t word = hash_word(stream_key(seed, kStreamSign, B.client[c]), (tile_base >> 6) + (t & 255u));
            words[c & 1u][2u * (t & 255u)] = lo32(word);
            words[c & 1u][2u * (t & 255u) + 1u] = hi32(word);
        }
        __builtin_amdgcn_sched_barrier(0);                       // (while the values are on their way)
        float u[16];
#pragma unroll
        for (int a = 0; a < 16; ++a) u[a] = i16 ? narrow_value((short)__float_as_int(next[a])) : next[a];
        __builtin_amdgcn_sched_barrier(0);                       // the conversions stay above the next sender's loads
        if (AHEAD && c + 1 < c_end) load(c + 1, next);
        if (c > c_begin) __syncthreads();                        // LDS is free again
        lo_forward16<kLo14Bits>(u, lds);                         // (with a barrier)
        const uint32_t scale = __float_as_uint(i16 ? scratch[c].deq[1] : 1.0f) & 0x7FFFFFFFu;   // > 0; x*1+s is exact
        // 16 sign bits of this thread's run, turned over where the stages between lanes left the values so
        uint32_t bits = 0u - ((t ^ t >> 1) & 1u);
        if constexpr (BY_TURNS) bits ^= words[c & 1u][t >> 1] >> (16u * (t & 1u));
        else bits ^= (uint32_t)(hash_word(stream_key(seed, kStreamSign, B.client[c]), (tile_base >> 6) + (t >> 2)) >> (16u * (t & 3u)));
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            // hash bit 1 -> s_i = -1: the factor is the scale with bit e of the sign word moved to the sign position
            // (one shift, one bit-field insert)
            const uint32_t factor = (scale & 0x7FFFFFFFu) | ((bits << (31 - e)) & 0x80000000u);
            sum[e] = fmaf(u[e], __uint_as_float(factor), sum[e]);
        }
    }
    float4 x[4];
    wave_quads(sum, lds + wv * Lo16<14>::ROW, x);
    const uint32_t at = 1024u * wv + 4u * lane;                  // quad j: coordinates at + 256 j .. + 3 of the tile
    if (part_tile) {
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<float4 *>(part_tile + at + 256 * j) = x[j];
        return;
    }
    // mean_n > 0: acc is written, not added to; the division happens here when no other workgroup adds to this tile
    const bool overwrite = mean_n > 0.0f;
    const float div = (overwrite && blockIdx.x < full_tiles) ? mean_n : 1.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint64_t i = tile_base + at + 256 * j;
        if (i + 4 <= d) {
            float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (!overwrite) a = *reinterpret_cast<const float4 *>(acc + i);
            a.x = (a.x + x[j].x) / div; a.y = (a.y + x[j].y) / div; a.z = (a.z + x[j].z) / div; a.w = (a.w + x[j].w) / div;
            *reinterpret_cast<float4 *>(acc + i) = a;
        } else {                                                 // the quad that straddles d, and those beyond
            const float v[4] = {x[j].x, x[j].y, x[j].z, x[j].w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (i + e < d) acc[i + e] = ((overwrite ? 0.0f : acc[i + e]) + v[e]) / div;
        }
    }
}

// ---- the same pass (index bits 0..13 of H, the sign diagonal and the sum over the senders, Sec. 2.2.2) for launches whose
// senders all have an fp16 workspace of small exact integers (b <= 1, D <= 2^24:
// |value| <= 2^10 after at most ten strided bits), with ten of the fourteen bits on the matrix cores.
//
// The tile is a 16 x 32 x 32 array (u, n, k) = index bits 10..13, 5..9, 0..4.  A wave owns two values of u.  For one u:
//   step 1  bits 0..4   D1[n][k'] = sum_k X[n][k] H[k][k']: v_mfma_f32_32x32x16_f16 twice, X as the A operand straight from
//           memory (a lane holds 16 consecutive fp16 of its row n: exact integers, |x| <= 2^10 < 2^11).
//   step 2  bits 5..9   D2[n'][k'] = sum_n H[n'][n] D1[n][k']: the registers that hold D1 ARE a B operand (lane = column k',
//           registers = 8 values of n per lane half), the Hadamard A operand is built with its columns in that order, so
//           nothing moves between the steps.  |D1| <= 2^15 does not fit fp16's 11 bits: every value is split into its fp16
//           truncation and the remainder (<= 5 bits, exact), and both go through the matrix cores into the same fp32
//           accumulators (four instructions).  All sums are integers below 2^24: exact in fp32 in any order.
//   exchange through LDS: lds[u][r][lane] = register r of the wave that owns u; wave w reads r = 2w, 2w + 1 of all 16 u
//           (same lane: the exchange swaps the register index with the wave index, conflict free in both directions).
//   step 3  bits 10..13 four butterfly stages over the 16 values of u in registers (fp32, exact).
// Register (u, j) of thread (wave w, lane l = 32 h + m) then holds coordinate 1024 u + 32 n' + m of the tile with
// n' = 8 (w / 2) + 4 h + 2 (w % 2) + j: 32 lanes cover one 128-byte line of acc, and the 32 sign bits of those lanes are one
// half (j) of one 64-bit word of the sender's SIGN stream.
// Per coordinate and sender this leaves 9 vector instructions (split 2, butterflies 4, sign and accumulate 3)
// where the all-vector version spends 19, and one exchange instead of two.  The loads of the next sender go out into the registers that the
// products of step 1 have just read (issued in front of them they cost 32 moves), their descriptors come from scalar registers (out of vector
// registers every load went through a loop), the sign words from the LDS: 16 senders of 11,173,962, us, 103.8 -> 91.3 (averages of a kernel
// trace; decode 169.6 -> 160.3), one of them 19.3 -> 18.6, 20 of 600,000 23.3 -> 22.3.
// x - (float)h for the fp16 in the low (HIGH = 0) or high half of `packed`: one mixed-precision fused multiply-add
// (-1 * h + x, exact: h is x truncated to 11 bits)
template <int HIGH>
__device__ inline float minus_half(float x, uint32_t packed) {
    float r;
    if (HIGH) asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(packed), "v"(-1.0f), "v"(x));
    else asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(packed), "v"(-1.0f), "v"(x));
    return r;
}

__global__ __launch_bounds__(512, 4) void k_dec_lo14_last_mfma(DecBatch B, uint32_t n, uint64_t d, int log2D, uint64_t seed,
                                                               const float *T, const DecScratch *scratch, float *acc,
                                                               uint32_t full_tiles, uint32_t K, uint32_t split_tiles,
                                                               float *partial, int separate, float mean_n) {
    __shared__ __attribute__((aligned(16))) float lds[1 << kLo14Bits];
    __shared__ uint64_t words[1 << (kLo14Bits - 6)];             // the tile's words of the sender's SIGN stream
    const uint32_t t = threadIdx.x, lane = t & 63u, wv = wave_in_block(), h = lane >> 5, m = lane & 31u;
    uint32_t tile = blockIdx.x, c_begin = 0, c_end = n;
    float *part = nullptr;                                       // this tile in the partial buffer
    if (blockIdx.x >= full_tiles) {
        const uint32_t idx = blockIdx.x - full_tiles, k = idx % K;
        tile = full_tiles + idx / K;
        // (in scalar registers, which the compiler does not see behind the divisions: a buffer descriptor made from them would go through
        // a loop)
        c_begin = __builtin_amdgcn_readfirstlane(n * k / K);
        c_end = __builtin_amdgcn_readfirstlane(n * (k + 1u) / K);
        if (separate) part = partial + ((size_t)k << log2D) + ((size_t)tile << kLo14Bits);
        else if (k > 0) part = partial + (((size_t)(k - 1) * split_tiles + (tile - full_tiles)) << kLo14Bits);
    }
    const uint64_t tile_base = (uint64_t)tile << kLo14Bits;

    // the two Hadamard operands: entry e of instruction q on lane (h, m)
    //   step 1, B[k][k']: k' = m, k = 16 h + 8 q + e    (the 16 consecutive fp16 a lane loads are k = 16 h .. 16 h + 15)
    //   step 2, A[n'][n]: n' = m, n = row of D1 that register 8 q + e of lane half h holds = 16 q + 8 (e / 4) + 4 h + e % 4
    half8_t Hk[2], Hn[2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            Hk[q][e] = hadamard_entry(16u * h + 8u * q + e, m);
        }
    Hn[0] = hadamard_rows_of_result(0, h, m);
    Hn[1] = hadamard_rows_of_result(1, h, m);

    float sum[32];                                               // sum[16 j + u]
#pragma unroll
    for (int e = 0; e < 32; ++e) sum[e] = 0.0f;

    // raw[2 s + q]: fp16 k = 16 h + 8 q .. + 7 of row n = m of unit u = wv + 8 s
    const uint32_t lane_off = (m * 32u + 16u * h) * 2u;
    u32x4_t raw[4];
    auto load = [&](uint32_t c, int s) {                         // (beyond the last sender: bounds of 0, no traffic)
        const rsrc_t r16 = make_rsrc(T + ((size_t)(c < c_end ? c : c_begin) << log2D), c < c_end ? 2u << log2D : 0u);     // the tile lies inside the slot
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            // (default cache policy: the two instructions q take the two 16-byte halves of every 32 bytes, and with the
            // streaming hint the second one fetched some lines again: 106 against 103 us)
            const auto x = __builtin_amdgcn_raw_buffer_load_b128(
                r16, (int)lane_off, (int)(((uint32_t)tile_base + (wv + 8u * s) * 1024u + 8u * q) * 2u), 0);
            raw[2 * s + q] = u32x4_t{x[0], x[1], x[2], x[3]};
        }
    };
    // sign bits of this thread's coordinates: bit m of the halves (j) of words 16 u + my_word of the tile
    const uint32_t my_word = 4u * (wv >> 1) + (wv & 1u) + 2u * h;

    load(c_begin, 0);
    load(c_begin, 1);
    for (uint32_t c = c_begin; c < c_end; ++c) {
        if (c > c_begin) __syncthreads();                        // every wave has read the previous sender's values and words
        // four waves in turn hash the tile's words for all of them (per lane and register pair, for itself, every wave hashed twice as many, and
        // took two lane reads a value to bring the bits into scalar registers)
        if ((wv >> 2) == (c & 1u)) words[t & 255u] = hash_word(stream_key(seed, kStreamSign, B.client[c]), (tile_base >> 6) + (t & 255u));
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            float16_t d1 = {0};
            d1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8_t, raw[2 * s]), Hk[0], d1, 0, 0, 0);
            d1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8_t, raw[2 * s + 1]), Hk[1], d1, 0, 0, 0);
            load(c + 1, s);                                      // into the registers the products have just read
            u32x4_t hi[2], lo[2];                                  // fp16 pairs: registers 2 i, 2 i + 1 of d1
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const uint32_t top = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(d1[r], d1[r + 1]));   // truncated to 11 bits
                hi[r >> 3][(r & 7) >> 1] = top;
                lo[r >> 3][(r & 7) >> 1] = __builtin_bit_cast(                                  // what is left: at most 5 bits
                    uint32_t, __builtin_amdgcn_cvt_pkrtz(minus_half<0>(d1[r], top), minus_half<1>(d1[r + 1], top)));
            }
            float16_t d2 = {0};
            d2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(Hn[0], __builtin_bit_cast(half8_t, hi[0]), d2, 0, 0, 0);
            d2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(Hn[1], __builtin_bit_cast(half8_t, hi[1]), d2, 0, 0, 0);
            d2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(Hn[0], __builtin_bit_cast(half8_t, lo[0]), d2, 0, 0, 0);
            d2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(Hn[1], __builtin_bit_cast(half8_t, lo[1]), d2, 0, 0, 0);
            float *L = lds + (wv + 8u * s) * 1024u + lane;
#pragma unroll
            for (int r = 0; r < 16; ++r) L[64 * r] = d2[r];
        }
        __syncthreads();
        float v0[16], v1[16];                                    // j = 0, 1
        const float *R = lds + 128u * wv + lane;
#pragma unroll
        for (int u = 0; u < 16; ++u) { v0[u] = R[1024 * u]; v1[u] = R[1024 * u + 64]; }
        fwht_regs<16>(v0);
        fwht_regs<16>(v1);
        const uint32_t scale = __float_as_uint(scratch[c].deq[1]) & 0x7FFFFFFFu;     // > 0
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            // hash bit 1 -> s_i = -1: the factor is the scale with the bit moved to the sign position
            const uint64_t w = words[my_word + 16u * (uint32_t)u];
            const uint32_t f0 = (scale & 0x7FFFFFFFu) | ((lo32(w) << (31u - m)) & 0x80000000u);
            const uint32_t f1 = (scale & 0x7FFFFFFFu) | ((hi32(w) << (31u - m)) & 0x80000000u);
            sum[u] = fmaf(v0[u], __uint_as_float(f0), sum[u]);
            sum[16 + u] = fmaf(v1[u], __uint_as_float(f1), sum[16 + u]);
        }
    }
    // register (u, j): coordinate 1024 u + 32 n' + m of the tile
    const uint32_t nrow = 8u * (wv >> 1) + 4u * h + 2u * (wv & 1u);
    const uint32_t mine_off = 32u * nrow + m;
    if (part) {
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            part[1024 * u + mine_off] = sum[u];
            part[1024 * u + mine_off + 32] = sum[16 + u];
        }
        return;
    }
    // mean_n > 0: acc is written, not added to; the division happens here when no other workgroup adds to this tile
    const bool overwrite = mean_n > 0.0f;
    const float div = (overwrite && blockIdx.x < full_tiles) ? mean_n : 1.0f;
    if (tile_base + (1u << kLo14Bits) <= d) {
        float *A = acc + tile_base + mine_off;
        float old[32];
#pragma unroll
        for (int e = 0; e < 32; ++e) old[e] = 0.0f;
        if (!overwrite) {
#pragma unroll
            for (int u = 0; u < 16; ++u) { old[u] = A[1024 * u]; old[16 + u] = A[1024 * u + 32]; }
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) { A[1024 * u] = (old[u] + sum[u]) / div; A[1024 * u + 32] = (old[16 + u] + sum[16 + u]) / div; }
    } else {                                                     // the one tile that straddles d
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const uint64_t i = tile_base + 1024u * u + mine_off;
            if (i < d) acc[i] = ((overwrite ? 0.0f : acc[i]) + sum[u]) / div;
            if (i + 32 < d) acc[i + 32] = ((overwrite ? 0.0f : acc[i + 32]) + sum[16 + u]) / div;
        }
    }
}

// ---- the same matrix-core pass for senders that sparsified by pairs before the rotation (EDEN_B_HALF_PRE, Sec. 4.1): the
// decoded vector has ceil(d / 2) coordinates, and coordinate g of sender c belongs to position 2 g + o_c(g) of the output
// (o from the sender's SUBSAMPLE stream), the other position of the pair getting nothing from this sender.  Every
// coordinate therefore needs two sums, and a thread of the kernel above has no registers for 64: here a workgroup has 16
// waves, wave w owns the one unit u = w in steps 1 and 2, and reads register w of all 16 units back from the exchange,
// so that a thread holds 16 coordinates (two sums each).  Register u of thread (wave w, lane 32 h + m) is coordinate
// 1024 u + 32 n' + m of the tile with n' = 8 (w / 4) + 4 h + w % 4: its bit of the SIGN and SUBSAMPLE streams is bit
// 32 (w % 2) + m of word 16 u + 4 (w / 4) + 2 h + (w / 2) % 2 of the tile, and the 32 lanes m write 64 consecutive floats.
// mean_n > 0: the output is written ((0 + sum) / mean_n) instead of added to.
__global__ __launch_bounds__(1024) void k_dec_lo14_last_pairs(DecBatch B, uint32_t n, uint64_t d_src, int log2D, uint64_t seed,
                                                              const float *T, const DecScratch *scratch, float *acc, float mean_n) {
    __shared__ __attribute__((aligned(16))) float lds[1 << kLo14Bits];
    const uint32_t t = threadIdx.x, lane = t & 63u, wv = wave_in_block(), h = lane >> 5, m = lane & 31u;
    const uint64_t tile_base = (uint64_t)blockIdx.x << kLo14Bits;

    half8_t Hk[2], Hn[2];                                        // as in k_dec_lo14_last_mfma
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int e = 0; e < 8; ++e) Hk[q][e] = hadamard_entry(16u * h + 8u * q + e, m);
    Hn[0] = hadamard_rows_of_result(0, h, m);
    Hn[1] = hadamard_rows_of_result(1, h, m);

    float even[16], odd[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) even[u] = odd[u] = 0.0f;

    // raw[q]: fp16 k = 16 h + 8 q .. + 7 of row n = m of unit u = wv
    const uint32_t lane_off = (m * 32u + 16u * h) * 2u;
    auto load = [&](uint32_t c, uint32_t (&raw)[2][4]) {
        const rsrc_t r16 = make_rsrc(T + ((size_t)c << log2D), 2u << log2D);       // the tile lies inside the slot
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const auto x = __builtin_amdgcn_raw_buffer_load_b128(r16, (int)lane_off,
                                                                 (int)(((uint32_t)tile_base + wv * 1024u + 8u * q) * 2u), 0);
            raw[q][0] = x[0]; raw[q][1] = x[1]; raw[q][2] = x[2]; raw[q][3] = x[3];
        }
    };
    // lane 16 hh + uu of either half of the wave hashes word (uu, hh)
    const uint32_t my_word = 16u * (lane & 15u) + 4u * (wv >> 2) + 2u * ((lane >> 4) & 1u) + ((wv >> 1) & 1u);

    uint32_t raw[2][4];
    load(0, raw);
    for (uint32_t c = 0; c < n; ++c) {
        half8_t x[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const u32x4_t v = {raw[q][0], raw[q][1], raw[q][2], raw[q][3]};
            x[q] = __builtin_bit_cast(half8_t, v);
        }
        if (c + 1 < n) load(c + 1, raw);
        if (c > 0) __syncthreads();                              // every wave has read the previous sender's values
        {
            float16_t d1 = {0};
            d1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[0], Hk[0], d1, 0, 0, 0);
            d1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[1], Hk[1], d1, 0, 0, 0);
            u32x4_t hi[2], lo[2];                                // fp16 pairs: the truncation to 11 bits and what is left
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const uint32_t top = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(d1[r], d1[r + 1]));
                hi[r >> 3][(r & 7) >> 1] = top;
                lo[r >> 3][(r & 7) >> 1] = __builtin_bit_cast(
                    uint32_t, __builtin_amdgcn_cvt_pkrtz(minus_half<0>(d1[r], top), minus_half<1>(d1[r + 1], top)));
            }
            float16_t d2 = {0};
            d2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(Hn[0], __builtin_bit_cast(half8_t, hi[0]), d2, 0, 0, 0);
            d2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(Hn[1], __builtin_bit_cast(half8_t, hi[1]), d2, 0, 0, 0);
            d2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(Hn[0], __builtin_bit_cast(half8_t, lo[0]), d2, 0, 0, 0);
            d2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(Hn[1], __builtin_bit_cast(half8_t, lo[1]), d2, 0, 0, 0);
            float *L = lds + wv * 1024u + lane;
#pragma unroll
            for (int r = 0; r < 16; ++r) L[64 * r] = d2[r];
        }
        __syncthreads();
        float v[16];
        const float *R = lds + 64u * wv + lane;
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = R[1024 * u];
        fwht_regs<16>(v);
        const uint32_t scale = __float_as_uint(scratch[c].deq[1]) & 0x7FFFFFFFu;     // > 0
        // one hash per lane serves both streams: lanes 0..31 take the words of the SIGN stream, lanes 32..63 the same words of
        // the SUBSAMPLE stream
        const uint64_t sign_key = stream_key(seed, kStreamSign, B.client[c]), pick_key = stream_key(seed, kStreamSubsample, B.client[c]);
        const uint64_t word = hash_word(h ? pick_key : sign_key, (tile_base >> 6) + my_word);
        const uint32_t half = (wv & 1u) ? (uint32_t)(word >> 32) : (uint32_t)word;
        const float pos = __uint_as_float(scale);
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            // Lanes u and 16 + u hold the SIGN words of the two halves of the wave, lanes 32 + u and 48 + u the SUBSAMPLE words:
            // side by side in a scalar register pair they are the 64 bits of the wave's lanes, and selects driven by such a
            // pair need no lane to fetch or shift anything.  Hash bit 1 -> s_i = -1; offset bit 1 -> the pair's second position.
            const uint64_t neg = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)half, 16 + u) << 32) |
                                 (uint32_t)__builtin_amdgcn_readlane((int)half, u);
            const uint64_t second = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)half, 48 + u) << 32) |
                                    (uint32_t)__builtin_amdgcn_readlane((int)half, 32 + u);
            const float factor = __builtin_amdgcn_inverse_ballot_w64(neg) ? -pos : pos;
            const bool to_second = __builtin_amdgcn_inverse_ballot_w64(second);
            even[u] = fmaf(v[u], to_second ? 0.0f : factor, even[u]);
            odd[u] = fmaf(v[u], to_second ? factor : 0.0f, odd[u]);
        }
    }
    const bool overwrite = mean_n > 0.0f;
    const float div = overwrite ? mean_n : 1.0f;
    const uint32_t nrow = 8u * (wv >> 2) + 4u * h + (wv & 3u);
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const uint64_t out = 2u * (tile_base + 1024u * (uint32_t)u + 32u * nrow + m);
        if (out + 1 < d_src) {
            float2 a = make_float2(0.0f, 0.0f);
            if (!overwrite) a = *reinterpret_cast<const float2 *>(acc + out);
            a.x = (a.x + even[u]) / div; a.y = (a.y + odd[u]) / div;
            *reinterpret_cast<float2 *>(acc + out) = a;
        } else if (out < d_src) {
            acc[out] = ((overwrite ? 0.0f : acc[out]) + even[u]) / div;
        }
    }
}

// acc[i] += partial[0][i'] + partial[1][i'] + ... for the tiles that k_dec_lo14_last split over K workgroups
// (added one after the other, in this order); with mean_n > 0 the total is divided by it.  One thread per four coordinates.
__global__ __launch_bounds__(256) void k_dec_lo14_combine(float *acc, uint64_t d, uint32_t full_tiles, uint32_t K,
                                                          uint32_t split_tiles, const float *partial, float mean_n) {
    const uint64_t local = ((uint64_t)blockIdx.x * 256u + threadIdx.x) * 4u;         // inside the split tiles
    const uint64_t i = ((uint64_t)full_tiles << kLo14Bits) + local;
    if (local >= ((uint64_t)split_tiles << kLo14Bits) || i >= d) return;
    float s[4];
    const bool whole = i + 4 <= d;                               // (acc is 16-byte aligned)
    if (whole) {
        const float4 a = *reinterpret_cast<const float4 *>(acc + i);
        s[0] = a.x; s[1] = a.y; s[2] = a.z; s[3] = a.w;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = (i + e < d) ? acc[i + e] : 0.0f;
    }
    // eight groups' loads on their way at a time: one after the other they took most of the kernel (whole decode, 8 senders of 300,007,
    // b = 2, 23.7 -> 22.9 us; of 4,000,037 at 2.7 bits 120.6 -> 118.3)
    for (uint32_t k0 = 1; k0 < K; k0 += 8) {
        float4 p[8];
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j)
            if (k0 + j < K) p[j] = *reinterpret_cast<const float4 *>(partial + (((size_t)(k0 + j - 1) * split_tiles) << kLo14Bits) + local);
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j)
            if (k0 + j < K) { s[0] += p[j].x; s[1] += p[j].y; s[2] += p[j].z; s[3] += p[j].w; }
    }
    const float div = mean_n > 0.0f ? mean_n : 1.0f;
    if (whole) {
        *reinterpret_cast<float4 *>(acc + i) = make_float4(s[0] / div, s[1] / div, s[2] / div, s[3] / div);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (i + e < d) acc[i + e] = s[e] / div;
    }
}

uint32_t launch_enc_lo_first(int P, const EncBatch &B, uint32_t n, uint64_t d_src, int pre, int blocked, int log2D, uint64_t seed, float *T,
                             double *partials, uint32_t partial_stride, const EncTail &tail, uint32_t compute_units, hipStream_t st) {
    const uint64_t d = pre ? (d_src + 1) / 2 : d_src;
    uint32_t tiles = (uint32_t)((d + (1u << P) - 1) >> P);
    // blocked layout: whole blocks of rows are written (a tile beyond d reads zeros and stores zeros), so that the strided
    // pass finds no unwritten row inside a block
    if (blocked) tiles = (tiles + kBlockRows - 1) / kBlockRows * kBlockRows;
    dim3 grid(tiles, n);
    // Up to 128 MiB of x and workspace x is read with the default policy, so that vectors that are encoded again are found in the
    // memory-side cache; beyond, with the streaming one (a pure read 7.2 against 6.4 TB/s). Encode, us, streaming / default, of the
    // same vectors over and over: one sender of 11,173,962, b = 1 36.9 / 35.1, of 15,000,000 45.5 / 40.4; 10 of 2^20, b = 2 33.0 /
    // 31.0; 24 of 300,007 30.9 / 26.2; of vectors that another kernel has just written: 36.8 / 36.9, 41.7 / 42.1, 40.2 / 39.6, 40.6 /
    // 40.5; of vectors that lie in no cache, whose lines then take the workspace's place: 36.6 / 37.8, 45.2 / 45.5, 32.5 / 33.4, 31.0
    // / 26.5. 32 of 2^20 (256 MiB), 1/2 to 4 bits, a round 147 / 150; 8 of 11,173,962, b = 1 178 / 192, 16 of them 373 / 399.
    const bool keep = !pre && (d_src + ((uint64_t)tiles << P)) * n * 4u <= (128u << 20);
#define EDEN_ENC_LO_LAUNCH(P, WAVES, PRE, BLK, KEEP) \
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_enc_lo_first<P, WAVES, PRE, BLK, KEEP>), grid, dim3(64 * WAVES), 0, st, B, d_src, log2D, seed, T, \
                       partials, partial_stride, tail)
#define EDEN_ENC_LO(P, WAVES, PRE, BLK) \
    do { if (keep) EDEN_ENC_LO_LAUNCH(P, WAVES, PRE, BLK, !(PRE)); else EDEN_ENC_LO_LAUNCH(P, WAVES, PRE, BLK, false); } while (0)
#define EDEN_ENC_LO14(WAVES) \
    do { \
        if (pre) { if (blocked) EDEN_ENC_LO(14, WAVES, true, true); else EDEN_ENC_LO(14, WAVES, true, false); } \
        else { if (blocked) EDEN_ENC_LO(14, WAVES, false, true); else EDEN_ENC_LO(14, WAVES, false, false); } \
    } while (0)
    // Sixteen waves while every workgroup has a CU to itself, eight beyond.  Encode, us, sixteen / eight: one sender of 300,007, b = 1 (19
    // workgroups) 12.2 / 12.8, of 2^20, b = 2 (64) 14.8 / 15.3, of 1,500,000, b = 1 (92) 15.9 / 16.3, 4 of 2^20, b = 2 (256) 17.8 /
    // 18.5.  Beyond, cards of one kind differ: 10 of 2^20, b = 2 (640) 29.6 / 30.6 and one of 7,500,000, b = 1 (460) 23.9 / 24.9 on one,
    // 34.8 / 31.1 and, of 8,000,000 (492), 30.9 / 25.9 on another, where a launch of 16 waves a workgroup takes 17 or 23 us from one call
    // to the next.
    if (P == 12) { if (pre) EDEN_ENC_LO(12, 4, true, false); else EDEN_ENC_LO(12, 4, false, false); }
    else if (tiles * n <= compute_units) EDEN_ENC_LO14(16);
    else EDEN_ENC_LO14(8);
#undef EDEN_ENC_LO14
#undef EDEN_ENC_LO_LAUNCH
#undef EDEN_ENC_LO
    return grid.x;
}
void launch_dec_lo14_last(const DecBatch &B, uint32_t n, uint64_t d_src, int pre, int log2D, uint64_t seed, const float *T,
                          const DecScratch *scratch, int narrow, float *acc, float *out, uint32_t resident, float *partial,
                          uint32_t partial_tiles, float mean_n, hipStream_t st) {
    const uint64_t d = pre == 1 ? (d_src + 1) / 2 : d_src;       // dimension of the decoded vectors
    const uint32_t tiles = (uint32_t)((d + (1u << kLo14Bits) - 1) >> kLo14Bits);     // tiles that reach below d
    if (pre == 1) {                                              // (fp16 workspace of small integers: on the matrix cores)
        hipLaunchKernelGGL(k_dec_lo14_last_pairs, dim3(tiles), dim3(1024), 0, st, B, n, d_src, log2D, seed, T, scratch, acc, mean_n);
        return;
    }
    if (pre == 2) {                                              // every sender on its own, into its slot of `out`
        if (narrow)
            hipLaunchKernelGGL(k_dec_lo14_last_mfma, dim3(tiles * n), dim3(512), 0, st, B, n, d_src, log2D, seed, T, scratch, acc, 0u, n, tiles,
                               out, 1, 0.0f);
        else
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_dec_lo14_last<true, false>), dim3(tiles * n), dim3(1024), 0, st, B, n, d_src, log2D, seed,
                               T, scratch, 0, acc, 0u, n, tiles, out, 1, 0.0f);
        return;
    }
    bool all16 = narrow != 0;                                    // every sender's workspace slot holds fp16
    for (uint32_t c = 0; c < n; ++c) all16 = all16 && B.b_q8[c] <= 256u;
    // Fewer tiles than half the resident workgroups: split every tile K ways by sender so that the chip is filled
    // (measured 2.2x on 64 tiles x 32 senders).  With more tiles than resident workgroups, splitting only the
    // last, partly filled wave of workgroups was measured 3..10% slower than leaving it: a CU with one workgroup runs it faster.
    uint32_t full = 0, rest = tiles, K = 1;
    if (2 * tiles <= resident) {
        K = resident / tiles;
        if (K > n) K = n;
        while (K > 1 && (uint64_t)(K - 1) * rest > partial_tiles) --K;    // what the partial buffer holds
        // No more groups than it takes for the longest one, where that spares a third of them or where the workgroups would take up
        // nearly every slot of the chip (a CU with one workgroup runs it faster).  Whole decode, us, all groups / fewer: 10 senders of
        // 2^20, b = 2 (512 -> 320 workgroups) 40.3 / 32.4; 20 of 2^20 (512 -> 448) 56.4 / 51.2, b = 1 40.4 / 37.0; 9 of 2,000,000 (492 -> 369)
        // 57.5 / 49.3, b = 1 41.3 / 37.8; 14 of 600,000 (481 -> 259) 37.7 / 30.4, b = 1 30.8 / 28.5; 12 of 800,000, b = 3 44.2 / 36.6.  At b = 1
        // the others do better with all of them or the same: 8 of 1,500,000 33.0 / 34.1, 31 of 600,000 (481 -> 407) 41.6 / 41.7.  The kernel for
        // values would do better with fewer there too (b = 2: 12 of 1,500,000, 460 -> 368, 55.0 / 49.6; 31 of 600,000 51.5 / 47.0); the rule
        // keeps them all at every budget.
        const uint32_t most = (n + K - 1) / K, fewer = (n + most - 1) / most;
        if (3 * fewer <= 2 * K || 20 * K * tiles >= 19 * resident) K = fewer;
    }
    if (K == 1) { full = tiles; rest = 0; }
    dim3 grid(full + rest * K);
    if (all16)                                                   // |values| <= 2^10: ten of the bits on the matrix cores
        hipLaunchKernelGGL(k_dec_lo14_last_mfma, grid, dim3(512), 0, st, B, n, d_src, log2D, seed, T, scratch, acc, full, K, rest,
                           partial, 0, mean_n);
    else {
        bool none16 = true;                                      // no sender with an fp16 slot
        for (uint32_t c = 0; c < n; ++c) none16 = none16 && !(narrow && B.b_q8[c] <= 256u);
#define EDEN_DEC_LO14_LAST(WIDE_ONLY, AHEAD)                                                                                          \
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_dec_lo14_last<WIDE_ONLY, AHEAD>), grid, dim3(1024), 0, st, B, n, d_src, log2D, seed, T, scratch, \
                       narrow, acc, full, K, rest, partial, 0, mean_n)
        if (!none16) EDEN_DEC_LO14_LAST(false, false);
        else if (K > 1) EDEN_DEC_LO14_LAST(true, false);
        else EDEN_DEC_LO14_LAST(true, true);
#undef EDEN_DEC_LO14_LAST
    }
    if (K > 1) {
        dim3 cgrid((uint32_t)((((uint64_t)rest << kLo14Bits) / 4 + 255) / 256));
        hipLaunchKernelGGL(k_dec_lo14_combine, cgrid, dim3(256), 0, st, acc, d, full, K, rest, partial, mean_n);
    }
}

}  // namespace eden
