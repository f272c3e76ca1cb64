// The decoder's contiguous transform with 16 values per thread (gfx950): 2^B consecutive coordinates by 2^B / 16 threads, B = 12 or 14.
// (The encoder's, whose order of the stages is part of a message, is EncLo in eden_kernels_lo14.hip.)
//
//   group 1    bits B-4 .. B-1   v[a] = coordinate a T + t, T = 2^(B-4) threads (coalesced loads)
//   exchange 1 through LDS between the waves: registers <-> bits B-8 .. B-5
//   group 2    bits B-8 .. B-5
//   exchange 2 through LDS inside the wave, in the place this wave alone has just read: registers <-> bits 0 .. 3
//   group 3    bits 0 .. 3, and (B = 14) bits 4 and 5 between the four lanes of a quad
//
// Thread t then holds the 16 coordinates 16 t .. 16 t + 15: a quarter of a 64-bit sign word of the rotation.
// With 16 values (and sums, and values on their way) a thread fits 64 registers: 32 waves per CU, twice as many as with 32 values, and in a
// launch of few tiles half the instructions in a row per wave.
#ifndef EDEN_LO_H
#define EDEN_LO_H

#include "eden_device.h"

namespace eden {

template <int B>
struct Lo16 {
    static_assert(B == 12 || B == 14, "tiles that exist");
    static constexpr int T = 1 << (B - 4);                       // threads
    // floats between the LDS rows of two values of a.  B = 14: a row becomes one wave's 16 rows of 64 + 4 in exchange 2.  B = 12: four rows
    // become its 4 x 16 rows of 16 (quads swizzled by the row instead of padding, so that eight workgroups fit a CU), and 272 = 16
    // (mod 64) keeps the four apart in the banks.
    static constexpr int ROW = B == 14 ? 16 * 68 : 272;
    static constexpr int LDS_FLOATS = 16 * ROW;
};

// one butterfly stage between lanes that differ in lane bit X = 1 or 2
template <int X>
__device__ inline void quad_stage(float &v) {
    const float sign = (threadIdx.x & (uint32_t)X) ? -1.0f : 1.0f;
    v = fmaf(v, sign, __uint_as_float(lane_xor_u32<X>(__float_as_uint(v))));
}
template <int X>
__device__ inline void quad_stage(float4 &v) { quad_stage<X>(v.x); quad_stage<X>(v.y); quad_stage<X>(v.z); quad_stage<X>(v.w); }
// The stages over lane bits 1, 2 (and 8) of four values, one instruction a stage and value, where signs can be turned over before or after: the
// other lane's value times 1 or -1 is added.  (Nothing gained in the encoder's pass over 14 bits, which waits for memory.)
//   AFTER:  in every stage the lane with bit X gets (own) - (other), the stage's difference with its sign turned over
//   BEFORE: that lane's input has its sign turned over; the results are the stage's
// Signs that depend on the lane pass through the stages over other bits as they are, so that the stages leave (expect) them turned over
// where the coordinate has an odd number of ones in their bits: the caller turns them over with those of the rotation.
// Written out, because the compiler leaves the exchange and the multiply-add two instructions.  What an instruction has written may be
// read from another lane two wait states later: the s_nop at the front keeps that distance to the instructions before the block, the one
// at the end to those behind it (the compiler does not look inside), and the three other values stand between two stages of one.
// build.py checks the built code.
template <bool BEFORE, bool BIT8>
__device__ inline void flip_stages(float &a, float &b, float &c, float &d) {
    const float sign1 = ((threadIdx.x & 1u) != 0u) == BEFORE ? 1.0f : -1.0f;
    const float sign2 = ((threadIdx.x & 2u) != 0u) == BEFORE ? 1.0f : -1.0f;
#define EDEN_FLIP(SIGN, PATTERN)                                                                                            \
    "v_fmac_f32_dpp %0, %0, " SIGN " " PATTERN " row_mask:0xf bank_mask:0xf\n\tv_fmac_f32_dpp %1, %1, " SIGN " " PATTERN   \
    " row_mask:0xf bank_mask:0xf\n\tv_fmac_f32_dpp %2, %2, " SIGN " " PATTERN " row_mask:0xf bank_mask:0xf\n\t"           \
    "v_fmac_f32_dpp %3, %3, " SIGN " " PATTERN " row_mask:0xf bank_mask:0xf\n\t"
    if constexpr (BIT8) {
        const float sign8 = ((threadIdx.x & 8u) != 0u) == BEFORE ? 1.0f : -1.0f;
        asm("s_nop 1\n\t" EDEN_FLIP("%4", "quad_perm:[1,0,3,2]") EDEN_FLIP("%5", "quad_perm:[2,3,0,1]") EDEN_FLIP("%6", "row_ror:8") "s_nop 1"
            : "+v"(a), "+v"(b), "+v"(c), "+v"(d) : "v"(sign1), "v"(sign2), "v"(sign8));
    } else {
        asm("s_nop 1\n\t" EDEN_FLIP("%4", "quad_perm:[1,0,3,2]") EDEN_FLIP("%5", "quad_perm:[2,3,0,1]") "s_nop 1"
            : "+v"(a), "+v"(b), "+v"(c), "+v"(d) : "v"(sign1), "v"(sign2));
    }
#undef EDEN_FLIP
}

// in: v[a] = coordinate a T + t of the tile; out: v[e] = coordinate 16 t + e, fully transformed (B = 14: with the sign turned over where
// t has an odd number of ones in bits 0 and 1, see flip_stages).  The caller puts a barrier between a use of `lds` and the next one.
template <int B>
__device__ inline void lo_forward16(float (&v)[16], float *lds) {
    using L = Lo16<B>;
    const uint32_t t = threadIdx.x, lane = t & 63u;
    fwht_regs<16>(v);
#pragma unroll
    for (int a = 0; a < 16; ++a) lds[a * L::ROW + t] = v[a];
    __syncthreads();
    if constexpr (B == 14) {
        float *mine = lds + (t >> 6) * L::ROW;                   // wave = a
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = mine[64 * r + lane];
        fwht_regs<16>(v);
        wave_lds_sync();
#pragma unroll
        for (int r = 0; r < 16; ++r) mine[68 * r + lane] = v[r];
        wave_lds_sync();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 x = *reinterpret_cast<const float4 *>(&mine[(lane >> 2) * 68u + (lane & 3u) * 16u + 4 * q]);
            v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
        }
        fwht_regs<16>(v);
#pragma unroll
        for (int q = 0; q < 4; ++q) flip_stages<false, false>(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    } else {
        const uint32_t a = t >> 4, low = t & 15u, a2 = a & 3u;
        float *mine = lds + (a >> 2) * (4 * L::ROW);             // the four rows of this wave
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = mine[a2 * L::ROW + 16 * r + low];
        fwht_regs<16>(v);
        wave_lds_sync();
#pragma unroll
        for (int r = 0; r < 16; ++r) mine[a2 * L::ROW + 16 * r + (low ^ (uint32_t)(4 * (r >> 2)))] = v[r];
        wave_lds_sync();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 x = *reinterpret_cast<const float4 *>(&mine[a2 * L::ROW + 16u * low + 4u * ((uint32_t)q ^ (low >> 2))]);
            v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
        }
        fwht_regs<16>(v);
    }
}

// Turns the wave's values round in its own LDS (1024 floats of its rows): in v[e] = coordinate 16 lane + e of the wave's 1024, out x[j] =
// coordinates 4 (64 j + lane) .. + 3: an access then covers whole lines.  (Quads swizzled by the lane: no bank conflicts either way.)
__device__ inline void wave_quads(const float (&v)[16], float *mine, float4 (&x)[4]) {
    const uint32_t lane = threadIdx.x & 63u;
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4 *>(&mine[16u * lane + 4u * ((uint32_t)q ^ ((lane >> 2) & 3u))]) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    wave_lds_sync();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t from = 16u * (uint32_t)j + (lane >> 2);
        x[j] = *reinterpret_cast<const float4 *>(&mine[16u * from + 4u * ((lane & 3u) ^ ((from >> 2) & 3u))]);
    }
}

}  // namespace eden
#endif
