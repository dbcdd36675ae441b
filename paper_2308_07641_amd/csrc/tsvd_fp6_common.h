// What the kernels on fp4 codes x fp6 (E2M3) planes share (tsvd_fp6.hip, tsvd_fp6_split.hip): the plane records and how
// they are made, and the matrix instruction.  Everything device-side sits in an unnamed namespace.
#ifndef TSVD_FP6_COMMON_H
#define TSVD_FP6_COMMON_H
#include "tsvd_gemm_common.h"

namespace {

// Record of one (16-token tile, 128-index block): planes' first 16 bytes per lane [3][64][16], last
// 8 bytes per lane [3][64][8], scale words [64][4] = 4864 bytes; lane (i, g) holds, for token i of
// the tile, the indices that meet elements 0..31 of lane group g of the A operand built from the
// tile format (tsvd_step_column).  Records are stored [128-token group][block][tile in group].
#define FP6_REC_BYTES 4864
#ifndef FP6_LDS_DEPTH
#define FP6_LDS_DEPTH 2                            // operand reads ahead of the MFMAs, in steps of eight MFMAs
#endif
#define FP6_PAIR_BYTES (8 * FP6_REC_BYTES)      // one block of one 128-token group: 38 KiB exactly
typedef int i32x8 __attribute__((ext_vector_type(8)));

// One lane's 32 values -> COUNT (three) E2M3 planes (the value, the residual of its rounding, the residual of that, ...), each
// with its own power-of-two scale.  put(plane, first 16 bytes, last 8 bytes) receives the lane's 24 bytes of each
// plane; the return value holds the scale bytes (COUNT <= 4).  KEEP: v is left holding what the planes do not resolve
// (for a second set of planes); else it is used up.  RISE: what is left from the second plane on is multiplied by 2^4 at each, so that the scales of
// the last planes reach below 2^-126 (mfma_fp6 takes that back: the third plane is 2^4 times what it stands for, the fourth 2^8, the fifth 2^12).
// TOP: the caller knows the largest magnitude.
template <bool KEEP = false, int COUNT = 3, bool RISE = false, bool TOP = false, typename Put>
__device__ __forceinline__ uint32_t tsvd_planes_of_32(float (&v)[32], Put put, float top = 0.f) {
    typedef float f32x16 __attribute__((ext_vector_type(16)));
    typedef float f32x32 __attribute__((ext_vector_type(32)));
    typedef unsigned u32x6 __attribute__((ext_vector_type(6)));
    uint32_t scales = 0;
#pragma unroll
    for (int pl = 0; pl < COUNT; ++pl) {
        float m = top;
        if (!TOP || pl > 0) {
            m = 0.f;
#pragma unroll
            for (int e = 0; e < 32; ++e) m = fmaxf(m, fabsf(v[e]));
        }
        // exponent ex with m 2^-ex <= 7.5, the largest E2M3 magnitude (m = f 2^x, 0.5 <= f < 1)
        int x = 0;
        const float f = frexpf(m, &x);
        int ex = m > 0.f ? (f <= 0.9375f ? x - 3 : x - 2) : 0;
        ex = max(-126, min(126, ex));
        scales |= (uint32_t)(127 + ex) << (8 * pl);
        const float unit = ldexpf(1.0f, ex);
        // v_cvt_scalef32_2xpk16_fp6_f32: element 2 j of the result is src0[j] / scale, element 2 j + 1 is
        // src1[j] / scale, rounded to nearest even on the E2M3 grid (saturating); the reverse conversion
        // returns the elements in the same order, times the scale (measured on gfx950)
        f32x16 s0, s1;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            s0[j] = v[2 * j];
            s1[j] = v[2 * j + 1];
        }
        // The conversions take several passes over their registers, and the register allocator lets the result of the
        // builtins share registers with operands that die at the instruction.  Measured on gfx950: a result tuple that
        // started in the scale's register left elements 2..31 converted with a wrong scale.  Hence the instructions are
        // written out with results that may not overlap any operand.
        u32x6 w;
        asm("v_cvt_scalef32_2xpk16_fp6_f32 %0, %1, %2, %3" : "=&v"(w) : "v"(s0), "v"(s1), "v"(unit));
        if (pl < COUNT - 1 || KEEP) {
            f32x32 back;
            constexpr float STEP = 16.f;
            const bool rise = RISE && pl > 0;
            asm("v_cvt_scalef32_pk32_f32_fp6 %0, %1, %2" : "=&v"(back) : "v"(w), "v"(rise ? STEP * unit : unit));
            // exact: the next plane codes this residual (v is at most 2^-4 of the first plane's here, so that 2^4 times it is in range)
#pragma unroll
            for (int e = 0; e < 32; ++e) v[e] = rise ? fmaf(STEP, v[e], -back[e]) : v[e] - back[e];
        }
        put(pl, u32x4{w[0], w[1], w[2], w[3]}, u32x2{w[4], w[5]});
    }
    return scales;
}
// ... written to the lane's places in the record at `rec`
template <bool KEEP = false>
__device__ __forceinline__ void tsvd_planes_of_32(float (&v)[32], unsigned char* rec, int lane) {
    const uint32_t scales = tsvd_planes_of_32<KEEP>(v, [&](int pl, u32x4 lo, u32x2 hi) {
        *reinterpret_cast<u32x4*>(rec + pl * 1024 + lane * 16) = lo;
        *reinterpret_cast<u32x2*>(rec + 3072 + pl * 512 + lane * 8) = hi;
    });
    *reinterpret_cast<uint32_t*>(rec + 4608 + lane * 4) = scales;
}
// Six planes for fp32 values: a record of three, and a second record for what those leave (2^-14 of a block's largest
// magnitude times 2^-14 again: below the last bit of an fp32 value of that magnitude).
__device__ __forceinline__ void tsvd_planes_of_32_twice(float (&v)[32], unsigned char* rec, unsigned char* rec2, int lane) {
    tsvd_planes_of_32<true>(v, rec, lane);
    tsvd_planes_of_32<false>(v, rec2, lane);
}

// The 32 values of one operand lane from a token's row of N activations (T: uint16_t, the bits of bf16, or uint32_t, those of fp32): indices
// k0 + 32 (e >> 4) + (e & 15), two runs of 16 consecutive elements, 16 bytes at a time at whatever address the row has (vector
// memory takes any; a load per element costs 32 instructions that the address unit takes a lane group at a time).  A chunk that
// would pass the row's end is read to end there and shifted; indices beyond N are zero.  (313 x 1049 x 384 at 5299 tokens 26.1 -> 18.2 us.)  inside (uniform): all of this lane's
// block lies below N.
template <typename T>
__device__ __forceinline__ void tsvd_gather_row(const T* row, int k0, int N, bool inside, float (&v)[32]) {
    typedef u32x4 chunk_at __attribute__((aligned(2)));
    constexpr int PER = 16 / sizeof(T), CHUNKS = 32 / PER;
    u32x4 q[CHUNKS];
    auto first = [&](int c) { return k0 + (c < CHUNKS / 2 ? 0 : 32 - 16) + PER * c; };
    if (inside) {
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) q[c] = *reinterpret_cast<const chunk_at*>(row + first(c));
    } else if (N >= PER) {
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) q[c] = *reinterpret_cast<const chunk_at*>(row + min(first(c), N - PER));
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            const int bits = 8 * (int)sizeof(T) * max(0, first(c) - (N - PER));
            const unsigned __int128 w = __builtin_bit_cast(unsigned __int128, q[c]);
            q[c] = __builtin_bit_cast(u32x4, bits < 128 ? w >> (bits & 127) : (unsigned __int128)0);
        }
    } else {
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            unsigned __int128 w = 0;
#pragma unroll
            for (int e = 0; e < PER; ++e)
                if (first(c) + e < N) w |= (unsigned __int128)row[first(c) + e] << (8 * (int)sizeof(T) * e);
            q[c] = __builtin_bit_cast(u32x4, w);
        }
    }
#pragma unroll
    for (int e = 0; e < 32; ++e) {
        if constexpr (sizeof(T) == 4) {
            v[e] = __uint_as_float(q[e >> 2][e & 3]);
        } else {
            const uint32_t w = q[e >> 3][(e & 7) >> 1];
            v[e] = __uint_as_float((e & 1) ? (w & 0xFFFF0000u) : (w << 16));
        }
    }
}

// RISEN: the plane's number among those that tsvd_planes_of_32 left with RISE
template <int PL, int RISEN = -1>
__device__ __forceinline__ f32x4 mfma_fp6(const u32x4& a, const u32x4& lo, const u32x2& hi, uint32_t scale, f32x4 acc) {
    const i32x8 av = {(int)a.x, (int)a.y, (int)a.z, (int)a.w, 0, 0, 0, 0};
    const i32x8 bv = {(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, 0, 0};
    // cbsz = 4: A is fp4 (E2M1); blgp = 2: B is fp6 (E2M3); A scale 2^0 (2^-4, 2^-8, 2^-12: bytes 1 to 3); B scale = byte PL of `scale`
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(av, bv, acc, 4, 2, RISEN < 2 ? 0 : RISEN - 1, RISEN < 0 ? 0x7F7F7F7F : 0x73777B7F,
                                                            PL, (int)scale);
}

}  // namespace
#endif  // TSVD_FP6_COMMON_H
