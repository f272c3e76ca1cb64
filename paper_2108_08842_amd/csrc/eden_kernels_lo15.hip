// The contiguous passes of D = 2^25 .. 2^27 (gfx950): 15 or 16 index bits, so that two passes through memory do (the strided pass
// takes the 10 or 11 bits above, eden_hix.h).
//
// The decoder: a workgroup of 16 waves transforms 2^15 coordinates, 32 per thread, as the encoder does (see below), and adds them up over the
// senders in registers.  HALVES (D = 2^27, 16 bits): two workgroups share a tile of 2^16; both read all of it, one transforms the
// sums of its halves, the other the differences (the stage over bit 15).  2^16 values and as many sums over the senders would be the
// whole register file of a CU.  The pair runs at the same time on the same XCD (workgroups i and i + 8), so the second read of a
// line is meant to find it in that XCD's L2.
//
// The encoder has no sums to keep: see k_enc_lo15_first, k_enc_lo16_first.
//
// The two replace a 14-bit contiguous pass and a second strided pass (one more trip through memory per direction): a round of 8 senders of 2^27,
// b = 4 8.03 -> 5.85 ms; at 2^25 1.94 -> 1.16 ms, with b = 1 1.91 -> 0.91 ms.
#include "eden_device.h"
#include "eden_kernels.h"
#include "eden_lo.h"

namespace eden {

// tile and half of a workgroup: pairs are 8 workgroups apart
template <bool HALVES>
__device__ inline void lo15_tile(uint32_t i, uint32_t &tile, uint32_t &half) {
    tile = HALVES ? ((i >> 4) << 3) + (i & 7u) : i;
    half = HALVES ? (i >> 3) & 1u : 0u;
}

// Encode, first pass: x -> T (see k_enc_lo_first), always in the blocked layout.
//
// The stages run over bits (15,) 10 .. 14, 5 .. 9, 0 .. 4 in this order (sums round differently in another one, and an index next to a
// threshold moves).  Behind those over bits 10..14 the 1024 coordinates of a register are a transform of their own, so the tile goes through the
// LDS in pieces of 16 registers, a wave taking one of them, 16 values per lane, through all ten stages left.  An exchange of the whole tile
// took 144 KiB and one workgroup per CU; a piece takes 64 KiB, so that
// - at P = 15 a second workgroup on the CU (64 registers) computes while the waves of the first wait for memory: encode of 4 senders of
//   60,000,001 sparsified by pairs 363 -> 347 us, of 8 of 2^25, b = 1 617 -> 612 (this pass: 5.5 TB/s, a copy's rate);
// - at P = 16 one workgroup holds the whole tile and loads the next one meanwhile, where two workgroups read it twice (k_enc_lo16_first).
//   v[a] = coordinate 1024 a + t; piece q: a = 16 q + wave
//   registers 5..8, lanes 0..4 and 9 | bit 9 against bit 5 between the halves of the wave | exchange inside the wave: quads of bits 0 and 1,
//   then 2, 3, 4 between lanes 1, 2 and 8 apart
constexpr uint64_t kFlipped = 0xF00F0FF0F00F0FF0ull;             // of 64 consecutive coordinates those with an odd number of ones in bits 2, 3, 4
// `mine`: the 1024 floats of LDS with this wave's coordinates; x[j] on return: the quad at lo15_quad(j), transformed
__device__ inline uint32_t lo15_quad(uint32_t lane, uint32_t j) {
    return 256u * j + 64u * (lane >> 4) + 32u * ((lane >> 2) & 1u) + 16u * ((lane >> 3) & 1u) + 4u * (lane & 3u);
}
// The stages between lanes leave (BEFORE: expect) the values with the signs of kFlipped turned over: flip_stages.
template <bool BEFORE>
__device__ inline void lo15_piece_forward(float *mine, uint32_t lane, float4 (&x)[4]) {
    const float *from = mine + 512u * (lane >> 5) + (lane & 31u);
    float y[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) y[r] = from[32 * r];
    fwht_regs<16>(y);                                            // bits 5..8
    swap_stage32(y);                                             // bit 9: register bit 0 now is bit 9, lane bit 5 is bit 5
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 16; ++r) mine[512 * (r & 1) + 64 * (r >> 1) + lane] = y[r];
    wave_lds_sync();
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
        const float4 z = *reinterpret_cast<const float4 *>(&mine[lo15_quad(lane, j)]);
        const float p = z.x + z.y, q = z.x - z.y, r = z.z + z.w, s = z.z - z.w;                  // bit 0
        x[j] = make_float4(p + r, q + s, p - r, q - s);                                          // bit 1
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) flip_stages<BEFORE, true>(x[j].x, x[j].y, x[j].z, x[j].w);       // bits 2, 3, 4
}

// stores them; `rt`: the sender's slot.  (Write-back stores: with the streaming hint the pass over 14 bits ran 13% slower.  Offsets in
// one vector register: 64-bit addresses of all pieces were kept in registers, and spilled; none in a scalar one, see
// wide_stores_with_scalar_offset in build.py.)
template <int P>
__device__ inline void lo15_store_piece(const float4 (&x)[4], rsrc_t rt, uint32_t tile, uint32_t block, uint32_t lane) {
    static_assert(kBlockRows == 4, "rows of the blocked layout");
    uint32_t at = ((tile >> kBlockRowBits) << (P + kBlockRowBits + 2)) + ((tile & (kBlockRows - 1u)) << 7) + (block << 14) +
                  (lane >> 4 << 10) + (lane >> 2 & 1u) * 512u + (lane >> 3 & 1u) * 64u + 16u * (lane & 3u);
    asm volatile("" : "+v"(at));
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
        const u32x4_t v = {__float_as_uint(x[j].x), __float_as_uint(x[j].y), __float_as_uint(x[j].z), __float_as_uint(x[j].w)};
        __builtin_amdgcn_raw_buffer_store_b128(v, rt, (int)(at + 4096u * j), 0, 0);
    }
}

template <bool PRE>
__global__ __launch_bounds__(1024, 8) void k_enc_lo15_first(EncBatch B, uint64_t d_src, int log2D, uint64_t seed, float *T,
                                                            double *partials, uint32_t partial_stride) {
    constexpr int P = 15;
    __shared__ __attribute__((aligned(16))) float lds[1 << 14];
    __shared__ double red[16];
    const uint32_t c = blockIdx.y, t = threadIdx.x, lane = t & 63u, wv = wave_in_block(), tile = blockIdx.x;
    const rsrc_t rx = make_rsrc(B.x[c], (uint32_t)(d_src * 4));           // reads past d_src give the zero padding
    // register a of this wave = 64 consecutive coordinates = one sign word: lane a hashes the word of register a
    const uint64_t word = ((uint64_t)tile << (P - 6)) + 16u * (lane & 31u) + wv;
    float u[32];
    if constexpr (PRE) {
        const uint64_t offs = hash_word(stream_key(seed, kStreamSubsample, B.client[c]), word);
#pragma unroll
        for (int a = 0; a < 32; ++a) {
            const uint32_t odd = __builtin_amdgcn_inverse_ballot_w64(wave_read64(offs, a)) ? 4u : 0u;
            u[a] = 2.0f * buf_load(rx, 8u * t + odd, (tile << (P + 3)) + 8192u * a);
        }
    } else {
#pragma unroll
        for (int a = 0; a < 32; ++a) u[a] = buf_load(rx, 4u * t, (tile << (P + 2)) + 4096u * a);
    }
    const uint64_t mine = hash_word(stream_key(seed, kStreamSign, B.client[c]), word) ^ kFlipped;
    double n2 = 0.0;
#pragma unroll
    for (int a = 0; a < 32; ++a) {
        n2 += (double)u[a] * (double)u[a];
        if ((a & 3) == 3) __builtin_amdgcn_sched_barrier(0);     // keeps the widened values of one group live at a time
    }
#pragma unroll
    for (int a = 0; a < 32; ++a) u[a] = negate_where(u[a], wave_read64(mine, a)) + 0.0f;     // + 0: no negative zeros
    fwht_regs<32>(u);                                            // bits 10..14
    const rsrc_t rt = make_rsrc(T + ((size_t)c << log2D), 4u << log2D);
    static_for<2>([&](auto H) {
        constexpr int h = decltype(H)::value;
        if (h) __syncthreads();                                  // the first half's regions have been read
#pragma unroll
        for (int i = 0; i < 16; ++i) lds[1024 * i + t] = u[16 * h + i];
        __syncthreads();
        float4 x[4];
        lo15_piece_forward<true>(lds + 1024u * wv, lane, x);
        lo15_store_piece<P>(x, rt, tile, 16u * h + wv, lane);
    });
    const double block_total = block_sum<1024>(n2, red);
    if (t == 0) partials[(size_t)c * partial_stride + blockIdx.x] = block_total;
}

// The same at D = 2^27: 2^16 coordinates per tile, 64 per thread, in four pieces.  One workgroup per CU, which takes one tile after the
// other: the registers of a piece are free once it lies in the LDS, and the loads of the next tile go out into them.  Bound by memory (the
// copy of a vector of 4 GiB reaches 5.3 to 5.8 TB/s here).  Two workgroups per tile, one for the sums of its halves and one for the
// differences, -> this, us: 8 senders of 2^27 1987 -> 1640 (4.3 -> 5.2 TB/s), of 80,000,001 1160 -> 992, one of 2^27 237 -> 190.  With a
// workgroup per tile, or two or four of them per CU: 1630 .. 1650 and 202 .. 219.  (83 scalar registers are spilled, to lanes of vector
// registers; none to memory.)
__global__ __launch_bounds__(1024) void k_enc_lo16_first(EncBatch B, uint32_t n, uint32_t tiles, uint64_t d_src, int log2D, uint64_t seed, float *T,
                                                         double *partials, uint32_t partial_stride) {
    constexpr int P = 16;
    __shared__ __attribute__((aligned(16))) float lds[2][1 << 14];
    __shared__ double red[2][16];
    const uint32_t wv = wave_in_block(), total = n * tiles;
    uint32_t t = threadIdx.x;
    uint32_t c = blockIdx.x / tiles, tile = blockIdx.x % tiles;
    rsrc_t rx = make_rsrc(B.x[c], (uint32_t)(d_src * 4));        // reads past d_src give the zero padding
    float u[64];
#pragma unroll
    for (int a = 0; a < 64; ++a) u[a] = buf_load(rx, 4u * t, (tile << (P + 2)) + 4096u * a);
#pragma unroll 1
    for (uint32_t i = blockIdx.x; i < total; ) {
        asm volatile("" : "+v"(t));                              // (what follows from it is not worth a register across the loop)
        const uint32_t lane = t & 63u;
        // register a of this wave = 64 consecutive coordinates = one sign word: lane a hashes the word of register a
        const uint64_t mine = hash_word(stream_key(seed, kStreamSign, B.client[c]), ((uint64_t)tile << (P - 6)) + 16u * lane + wv) ^ kFlipped;
        double n2[2] = {0.0, 0.0};
#pragma unroll
        for (int a = 0; a < 64; ++a) {
            n2[a >> 5] += (double)u[a] * (double)u[a];
            u[a] = negate_where(u[a], wave_read64(mine, a)) + 0.0f;      // + 0: no negative zeros
            if ((a & 7) == 7) __builtin_amdgcn_sched_barrier(0); // keeps the widened values of one group live at a time
        }
        asm volatile("" : "+v"(n2[0]), "+v"(n2[1]));             // (left to itself the compiler adds one half up at the end and keeps its values)
#pragma unroll
        for (int a = 0; a < 32; ++a) {                           // bit 15
            const float lo = u[a], hi = u[32 + a];
            u[a] = lo + hi;
            u[32 + a] = lo - hi;
        }
        fwht_regs_low<64, 5>(u);                                 // bits 10..14
        // the next tile (none after the last one: bounds of 0, no traffic)
        i += gridDim.x;
        const bool more = i < total;
        const uint32_t c_next = more ? i / tiles : 0u, tile_next = more ? i % tiles : 0u;
        rx = make_rsrc(B.x[c_next], more ? (uint32_t)(d_src * 4) : 0u);
        const rsrc_t rt = make_rsrc(T + ((size_t)c << log2D), 4u << log2D);
        static_for<4>([&](auto Q) {
            constexpr int q = decltype(Q)::value;
            float *buf = lds[q & 1];                             // (two pieces later every wave has passed the barrier behind its reads)
#pragma unroll
            for (int r = 0; r < 16; ++r) buf[1024 * r + t] = u[16 * q + r];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < 16; ++r) u[16 * q + r] = buf_load(rx, 4u * t, (tile_next << (P + 2)) + 4096u * (16 * q + r));
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            float4 x[4];
            lo15_piece_forward<true>(buf + 1024u * wv, lane, x);
            lo15_store_piece<P>(x, rt, tile, 16u * q + wv, lane);
            __builtin_amdgcn_sched_barrier(0);
        });
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const double sum = wave_sum(n2[h]);
            if (lane == 0) red[h][wv] = sum;
        }
        __syncthreads();
        if (t < 2u) {                                            // a partial sum per half of a tile
            double sum = 0.0;
#pragma unroll
            for (int w = 0; w < 16; ++w) sum += red[t][w];
            partials[(size_t)c * partial_stride + ((tile >> 3) << 4) + (t << 3) + (tile & 7u)] = sum;
        }
        c = c_next;
        tile = tile_next;
    }
}

// Decode, last pass (see k_dec_lo14_last): index bits 0..P-1 of H for every sender, its signs, the sum over the senders in
// registers, one contiguous read-modify-write of acc (mean_n > 0: acc is written with the sum divided by mean_n).  These sizes
// have at least 512 (half) tiles: no split by sender.
// Neither memory nor the vector units were busy half of the time while a workgroup, alone on its CU, waited for all of a sender's tile and then
// computed.  So a workgroup goes through the senders of a tile and on to its next tile with the loads of what comes next on their way: the upper
// half's registers are free after the stage over bit 15, those of a piece once it lies in the LDS.  Mean, last pass, us: 8 senders of
// 2^27, b = 4 1110 -> 1000 (4.8 TB/s; with a workgroup per tile 1062), b = 1 949 -> 875, one of 2^27 285 -> 212, 8 of 2^25, b = 4 239 ->
// 211, 4 of 10^8, b = 1 and 4 680 -> 400, b = 2 497 -> 417.
// KIND: kWide: no sender of the launch has an fp16 slot (every b > 1), kNarrow: every sender has one, kMixed.
enum : int { kMixed = 0, kWide = 1, kNarrow = 2 };
template <bool HALVES, int KIND>
__global__ __launch_bounds__(1024) void k_dec_lo15_last(DecBatch B, uint32_t n, uint32_t tiles, uint64_t d_src, int log2D, uint64_t seed, const float *T,
                                                        const DecScratch *scratch, float *acc, float mean_n) {
    constexpr int P = HALVES ? 16 : 15;
    // (both kinds of loads for 64 registers spilled: 692 us against 403, 4 senders of 10^8, b = 1 and 4)
    constexpr bool UP_AHEAD = KIND != kMixed;
    __shared__ __attribute__((aligned(16))) float lds[2][1 << 14];
    __shared__ uint32_t words[16][64];                           // halves of each wave's sign words
    uint32_t t = threadIdx.x;
    const uint32_t wv = wave_in_block();
    float sum[32];
#pragma unroll
    for (int e = 0; e < 32; ++e) sum[e] = 0.0f;
    auto is_narrow = [&](uint32_t c) { return KIND == kNarrow || (KIND == kMixed && B.b_q8[c] <= 256u); };
    // (through a buffer descriptor: one offset register for all loads.  After the last sender of the last tile the bounds are 0: no
    // branch around the loads, and no traffic)
    auto load = [&](rsrc_t r, bool i16, uint32_t first, float (&v)[32], auto A0, auto COUNT) {
        constexpr int a0 = decltype(A0)::value, count = decltype(COUNT)::value;
        if (i16) {
#pragma unroll
            for (int a = a0; a < a0 + count; ++a)
                v[a] = __int_as_float((int)__builtin_amdgcn_raw_buffer_load_b16(r, (int)(2u * t), (int)(2u * first + 2048u * a), kStream));
        } else {
#pragma unroll
            for (int a = a0; a < a0 + count; ++a) v[a] = buf_load(r, 4u * t, 4u * first + 4096u * a);
        }
    };
    auto value = [](float v, bool i16) { return i16 ? narrow_value((short)__float_as_int(v)) : v; };
    auto slot = [&](uint32_t c, bool some) { return make_rsrc(T + ((size_t)c << log2D), some ? 4u << log2D : 0u); };
    using std::integral_constant;
    uint32_t i = blockIdx.x, c = 0u, tile, half;
    lo15_tile<HALVES>(i, tile, half);
    float u[32], up[HALVES ? 32 : 1];
    {
        const rsrc_t r = slot(0u, ((uint64_t)tile << P) < d_src);
        load(r, is_narrow(0u), tile << P, u, integral_constant<int, 0>{}, integral_constant<int, 32>{});
        if constexpr (HALVES && UP_AHEAD) load(r, is_narrow(0u), (tile << P) + (1u << 15), up, integral_constant<int, 0>{}, integral_constant<int, 32>{});
    }
#pragma unroll 1
    for (;;) {
        asm volatile("" : "+v"(t));                              // (what follows from it is not worth a register across the loop)
        const uint32_t lane = t & 63u;
        const bool i16 = is_narrow(c);
        // what comes next
        const bool last = c + 1u == n;
        const uint32_t c_next = last ? 0u : c + 1u, i_next = last ? i + gridDim.x : i;
        uint32_t tile_next, half_next;
        lo15_tile<HALVES>(i_next, tile_next, half_next);
        const rsrc_t next = slot(c_next, i_next < tiles && ((uint64_t)tile_next << P) < d_src);
        const bool next16 = is_narrow(c_next);
        // 32 sign words for the wave's 2048 coordinates: lane l < 32 hashes the word l & 15 of its block in piece l / 16
        const uint64_t row = ((uint64_t)tile << P) + ((uint64_t)half << 15);     // first coordinate
        const uint64_t word = (row >> 6) + ((lane & 16u) << 4) + 16u * wv + (lane & 15u);
        wave_lds_sync();                                         // the last sender's have been read
        if (lane < 32u) {
            const uint64_t signs = hash_word(stream_key(seed, kStreamSign, B.client[c]), word) ^ kFlipped;
            words[wv][2u * lane] = lo32(signs);
            words[wv][2u * lane + 1u] = hi32(signs);
        }
        if constexpr (HALVES) {
            const float side = half ? -1.0f : 1.0f;
            if constexpr (!UP_AHEAD)
                load(slot(c, ((uint64_t)tile << P) < d_src), i16, (tile << P) + (1u << 15), up, integral_constant<int, 0>{},
                     integral_constant<int, 32>{});
#pragma unroll
            for (int a = 0; a < 32; ++a) {                       // the stage over bit 15 (one rounding)
                u[a] = fmaf(value(up[a], i16), side, value(u[a], i16));
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (UP_AHEAD) load(next, next16, (tile_next << P) + (1u << 15), up, integral_constant<int, 0>{}, integral_constant<int, 32>{});
            __builtin_amdgcn_sched_barrier(0);
        } else {
#pragma unroll
            for (int a = 0; a < 32; ++a) u[a] = value(u[a], i16);
        }
        fwht_regs<32>(u);                                        // bits 10..14
        const uint32_t scale = __float_as_uint(i16 ? scratch[c].deq[1] : 1.0f) & 0x7FFFFFFFu;    // > 0; x*1+s is exact
        static_for<2>([&](auto Q) {
            constexpr int q = decltype(Q)::value;
            asm volatile("" : "+v"(t));
            const uint32_t lane = t & 63u;
            float *buf = lds[q];                                 // (two pieces later every wave has passed the barrier behind its reads)
#pragma unroll
            for (int r = 0; r < 16; ++r) buf[1024 * r + t] = u[16 * q + r];
            __builtin_amdgcn_sched_barrier(0);
            load(next, next16, tile_next << P, u, integral_constant<int, 16 * q>{}, integral_constant<int, 16>{});
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            float4 x[4];
            lo15_piece_forward<false>(buf + 1024u * wv, lane, x);
            // the quad's four bits lie in one half of a word
            const uint32_t *my_words = words[wv] + 2u * (lane >> 4) + ((lane >> 2) & 1u);
            const uint32_t place = 16u * ((lane >> 3) & 1u) + 4u * (lane & 3u);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t bits = my_words[32 * q + 8 * j] >> place;
                const float y[4] = {x[j].x, x[j].y, x[j].z, x[j].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // hash bit 1 -> s_i = -1: the factor is the scale with the sign bit moved to the sign position
                    const float factor = __uint_as_float(scale | ((bits << (31 - e)) & 0x80000000u));
                    sum[16 * q + 4 * j + e] = fmaf(y[e], factor, sum[16 * q + 4 * j + e]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if (last) {
            const bool overwrite = mean_n > 0.0f;
            const float div = overwrite ? mean_n : 1.0f;
            const uint64_t out0 = row + 1024u * wv;
            const uint32_t left = out0 < d_src ? (uint32_t)(d_src - out0) : 0u;
            const rsrc_t ra = make_rsrc(acc + out0, left * 4u);
            uint32_t at = 4u * lo15_quad(lane, 0u);              // the wave's quads of a turn lie side by side
            asm volatile("" : "+v"(at));
            if (left >= 16384u + 1024u) {
#pragma unroll
                for (int k = 0; k < 2; ++k) {                    // four quads at a time, 256 coordinates apart
                    u32x4_t a[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) a[j] = u32x4_t{0u, 0u, 0u, 0u};
                    if (!overwrite) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) a[j] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)(at + 1024u * j), 65536 * k, 0);
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        u32x4_t v;
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = __float_as_uint((__uint_as_float(a[j][e]) + sum[16 * k + 4 * j + e]) / div);
                        __builtin_amdgcn_raw_buffer_store_b128(v, ra, (int)(at + 65536u * k + 1024u * j), 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {                                             // one by one: the bounds drop what lies beyond d_src
#pragma unroll
                for (int e = 0; e < 32; ++e) {
                    const uint32_t offset = at + 65536u * (e / 16) + 1024u * (e / 4 % 4) + 4u * (e % 4);
                    const float a = overwrite ? 0.0f : __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ra, (int)offset, 0, 0));
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint((a + sum[e]) / div), ra, (int)offset, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int e = 0; e < 32; ++e) sum[e] = 0.0f;
            if (i_next >= tiles) break;
        }
        i = i_next;
        c = c_next;
        tile = tile_next;
        half = half_next;
    }
}

// The same for launches of fp16 slots at P = 15, the tile through the LDS as a whole: a thread then has 32 coordinates in a row, after
// 628 vector instructions a sender where the pieces take 676 and 17 waits.  A CU that goes through many senders is bound by those; with
// few of them it is the loads ahead that count (see launch_dec_lo15_last).
// PAIRS: senders sparsified by pairs (one output coordinate of each pair): 64 sums a thread.  With the pieces, which tie the pair's
// choice to the quads, 4 senders of 60,000,001 took 149 us, this 137.
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

template <bool PAIRS>
__global__ __launch_bounds__(1024) void k_dec_lo15_last_rows(DecBatch B, uint32_t n, uint64_t d_src, int log2D, uint64_t seed, const float *T,
                                                             const DecScratch *scratch, float *acc, float mean_n) {
    constexpr int NS = PAIRS ? 64 : 32;                          // accumulator coordinates per thread
    __shared__ __attribute__((aligned(16))) float lds[kLo15LdsWords];
    const uint32_t t = threadIdx.x, lane = t & 63u, wv = wave_in_block();
    const uint64_t row = (uint64_t)blockIdx.x << 15;             // first coordinate of the tile in a slot
    float sum[NS];
#pragma unroll
    for (int e = 0; e < NS; ++e) sum[e] = 0.0f;
    // (through a buffer descriptor: one offset register for all loads; with flat addresses the kernel spilled 44 registers)
    auto load = [&](uint32_t c, float (&v)[32]) {                // (beyond the last sender: bounds of 0, no traffic)
        const rsrc_t r = make_rsrc(T + ((size_t)(c < n ? c : 0u) << log2D), c < n ? 4u << log2D : 0u);
#pragma unroll
        for (int a = 0; a < 32; ++a)
            v[a] = __int_as_float((int)__builtin_amdgcn_raw_buffer_load_b16(r, (int)(2u * t), (int)(2u * (uint32_t)row + 2048u * a), kStream));
    };
    float ahead[32];
    if (!PAIRS) load(0, ahead);
    for (uint32_t c = 0; c < n; ++c) {
        if (PAIRS) load(c, ahead);
        float u[32];
#pragma unroll
        for (int a = 0; a < 32; ++a) u[a] = narrow_value((short)__float_as_int(ahead[a]));
        __builtin_amdgcn_sched_barrier(0);                       // the conversions stay above the next sender's loads
        if (!PAIRS) load(c + 1, ahead);
        lo15_forward32(u, lds);
        const uint32_t scale = __float_as_uint(scratch[c].deq[1]) & 0x7FFFFFFFu;         // > 0
        // the wave's 2048 coordinates use 32 sign words: lane l < 32 hashes word l, every thread fetches its own
        const uint64_t word0 = (row + 2048u * wv) >> 6;
        const uint64_t mine = hash_word(stream_key(seed, kStreamSign, B.client[c]), word0 + (lane & 31u));
        const uint32_t wlo = (uint32_t)__shfl((int)(uint32_t)mine, (int)(lane >> 1), 64);
        const uint32_t whi = (uint32_t)__shfl((int)(uint32_t)(mine >> 32), (int)(lane >> 1), 64);
        const uint32_t bits = (t & 1u) ? whi : wlo;              // 32 sign bits of this thread's run
        if constexpr (PAIRS) {
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
    // swizzled by the low three bits of the run): with a run per lane every line was touched by eight instructions, and read from L2 as often
    // (whole decode: one sender of 5 * 10^7, added to acc, 244 -> 98 us; of 10^8 466 -> 228).
    const bool overwrite = mean_n > 0.0f;
    const float div = overwrite ? mean_n : 1.0f;
    const uint64_t out0 = (PAIRS ? 2u : 1u) * (row + 2048u * wv);        // the wave's first coordinate of acc
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
                               double *partials, uint32_t partial_stride, uint32_t compute_units, hipStream_t st) {
    const uint64_t d = pre ? (d_src + 1) / 2 : d_src;
    if (P == 16) {
        const uint32_t tiles = lo15_tiles(d, 16, 8), total = tiles * n;
        hipLaunchKernelGGL(k_enc_lo16_first, dim3(total < compute_units ? total : compute_units), dim3(1024), 0, st, B, n, tiles, d_src, log2D, seed, T,
                           partials, partial_stride);
        return 2 * tiles;
    }
    const dim3 grid(lo15_tiles(d, 15, kBlockRows), n);
    if (pre)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_enc_lo15_first<true>), grid, dim3(1024), 0, st, B, d_src, log2D, seed, T, partials, partial_stride);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_enc_lo15_first<false>), grid, dim3(1024), 0, st, B, d_src, log2D, seed, T, partials, partial_stride);
    return grid.x;
}
void launch_dec_lo15_last(int P, const DecBatch &B, uint32_t n, uint64_t d_src, int pre, int log2D, uint64_t seed, const float *T,
                          const DecScratch *scratch, float *acc, float mean_n, uint32_t compute_units, hipStream_t st) {
    const uint64_t d = pre ? (d_src + 1) / 2 : d_src;
    const uint32_t tiles = P == 16 ? 2 * lo15_tiles(d, 16, 8) : lo15_tiles(d, 15, 1);
    if (pre) {                                                   // (these senders have b = 1: fp16 slots)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_dec_lo15_last_rows<true>), dim3(tiles), dim3(1024), 0, st, B, n, d_src, log2D, seed, T, scratch, acc, mean_n);
        return;
    }
    // a workgroup per CU, which goes from tile to tile with the next one's loads on their way (whole groups of pairs)
    const uint32_t resident = compute_units < 16u ? 16u : compute_units / 16u * 16u;
    const dim3 grid(tiles < resident ? tiles : resident);
    bool wide = true, small = true;                              // no sender, every sender with an fp16 slot
    for (uint32_t c = 0; c < n; ++c) { wide = wide && B.b_q8[c] > 256u; small = small && B.b_q8[c] <= 256u; }
    // Nine senders or more as a whole.  Whole decode at b = 1, us, in pieces / as a whole: one sender of 2^26 128 / 148, 4 355 / 372, 8
    // 644 / 646, 12 937 / 923, 16 1227 / 1193, 32 2392 / 2293; 8 of 2^24 + 1 236 / 233, of 2^25 298 / 305, 16 571 / 547, 32 1080 / 1031.
    if (small && P == 15 && n > 8u) {
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_dec_lo15_last_rows<false>), dim3(tiles), dim3(1024), 0, st, B, n, d_src, log2D, seed, T, scratch, acc, mean_n);
        return;
    }
#define EDEN_DEC_LO15(HALVES, KIND) \
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_dec_lo15_last<HALVES, KIND>), grid, dim3(1024), 0, st, B, n, tiles, d_src, log2D, seed, T, scratch, acc, mean_n)
    if (P == 16) { if (wide) EDEN_DEC_LO15(true, kWide); else if (small) EDEN_DEC_LO15(true, kNarrow); else EDEN_DEC_LO15(true, kMixed); }
    else { if (wide) EDEN_DEC_LO15(false, kWide); else if (small) EDEN_DEC_LO15(false, kNarrow); else EDEN_DEC_LO15(false, kMixed); }
#undef EDEN_DEC_LO15
}

}  // namespace eden
