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

// The 32 values of one operand lane from feature-major bf16 x (N rows of B tokens, ld apart; eight values at least): features 128 block .., tokens tok0 .. + 15 of
// a wavefront.  Its 128 rows of 32 bytes come as four chunks of eight tokens a lane, at any alignment, and are transposed in 4 KiB of LDS of its own (a load per value
// costs 32 requests, which keep the address unit busy, and an address each).  Row r of the 64 of two runs lies at position r ^ 2 ((r >> 4 ^ r >> 5) & 1), so that the lane groups
// served in a cycle hit different banks.  A chunk that would pass the end of x is read to end there and shifted; features beyond N
// are zero; tokens beyond B hold what stands there, and nobody stores what becomes of them.
// block, tok0: uniform.
__device__ __forceinline__ bool tsvd_columns_end(long long ld, int N, int block) {       // (a chunk ends at most 63 tokens beyond B: four more rows of 17 are more)
    return 128 * block + 132 > N || ld < 17 || ld >= 1 << 23;
}
__device__ __forceinline__ int tsvd_column_row(int j, int lane) {                        // row of the block that a lane's chunk j comes from
    const int pos = (lane >> 1) + 32 * (j & 1), r = pos ^ ((((pos >> 4) ^ (pos >> 5)) & 1) << 1);
    return 32 * (j >> 1) + 64 * (r >> 5) + (r & 31);
}
__device__ __forceinline__ void tsvd_request_columns(const uint16_t* x, long long ld, int N, int B, int block, int tok0, int lane, u32x4 (&raw)[4]) {
    typedef u32x4 chunk_at __attribute__((aligned(2)));
    if (tsvd_columns_end(ld, N, block)) {
        const long long last = (long long)(N - 1) * ld + B - 8;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            raw[j] = *reinterpret_cast<const chunk_at*>(x + min(min(128 * block + tsvd_column_row(j, lane), N) * ld + (tok0 + 8 * (lane & 1)), last));
    } else {
        const uint16_t* base = x + 128 * block * ld + tok0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            raw[j] = *reinterpret_cast<const chunk_at*>(base + 32 * (j >> 1) * ld + (unsigned)(tsvd_column_row(j & 1, lane) * (int)ld + 8 * (lane & 1)));
    }
}
__device__ __forceinline__ void tsvd_columns_of(u32x4 (&raw)[4], long long ld, int N, int B, int block, int tok0, int lane, unsigned char* slot, float (&v)[32]) {
    if (tsvd_columns_end(ld, N, block)) {
        const long long last = (long long)(N - 1) * ld + B - 8;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int by = (int)min(max(min(128 * block + tsvd_column_row(j, lane), N) * ld + (tok0 + 8 * (lane & 1)) - last, 0ll), 8ll);       // values read too early
            if (__any((by & 7) != 0)) {
                const unsigned __int128 w = __builtin_bit_cast(unsigned __int128, raw[j]);
                raw[j] = __builtin_bit_cast(u32x4, w >> (16 * by & 127));
            }
            if (by == 8) raw[j] = u32x4{0u, 0u, 0u, 0u};
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) *reinterpret_cast<u32x4*>(slot + j * 1024 + lane * 16) = raw[j];
    __builtin_amdgcn_wave_barrier();
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr_t;
    auto transposed = [](const unsigned char* at) { return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)at)); };
    const int i = lane & 15, g = lane >> 4, row = 32 * (g & 1) + 16 * (g >> 1) + (i >> 3) + 4 * ((i >> 2) & 1), turned = (g & 1) ^ (g >> 1);
    const int at_lo = (row + 2 * turned) * 32 + (i & 3) * 8, at_hi = (row + 2 * (1 - turned)) * 32 + (i & 3) * 8;
#pragma unroll
    for (int j = 0; j < 4; ++j) {                            // values 8 j .. + 7: word m holds m and m + 4 of them
        const u32x2 lo = transposed(slot + (j >> 1) * 2048 + at_lo + (j & 1) * 256), hi = transposed(slot + (j >> 1) * 2048 + at_hi + (j & 1) * 256);
        const uint32_t w[4] = {lo.x, lo.y, hi.x, hi.y};
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            v[8 * j + m] = __uint_as_float(w[m] << 16);
            v[8 * j + m + 4] = __uint_as_float(w[m] & 0xFFFF0000u);
        }
    }
    __builtin_amdgcn_wave_barrier();
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
