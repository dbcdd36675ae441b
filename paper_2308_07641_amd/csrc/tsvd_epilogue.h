// Internal: the last step of stage U shared by every kernel family: optional bias (the paper's
// layer listing in the supplement shows its linear layers with bias=True: y = U(S*(Vx)) + b) and
// the choice of the output type (fp32, or bf16 rounded to nearest even from the fp32 result).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// The scalar offset of an access to a buffer of `bytes` bytes.  The range check compares the vector offset with what the scalar offset leaves of the buffer, so
// it holds for scalar offsets up to the end: rows behind that (of x beyond N, of y beyond M) are put at the end, where every vector offset is outside.
__device__ __forceinline__ int tsvd_buffer_offset(int offset, uint32_t bytes) { return (int)min((uint32_t)offset, bytes); }

// fp32 -> bf16 bit pattern, round to nearest even (NaN stays NaN).
__device__ __forceinline__ uint16_t tsvd_bf16_rne(float v) {
    const uint32_t u = __float_as_uint(v);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x0040u);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// y[idx] = v as fp32 or bf16 (out_bf16 is uniform over the launch).
__device__ __forceinline__ void tsvd_store_y(void* y, size_t idx, float v, int out_bf16) {
    if (out_bf16) static_cast<uint16_t*>(y)[idx] = tsvd_bf16_rne(v);
    else static_cast<float*>(y)[idx] = v;
}

// bf16 store of two rows of a 16 x 16 result block in the layout of the MFMA result: lane (i, g)
// holds token col16 + i (col16 a multiple of 16) of rows r and r + 1 (values v0, v1).
// Neighbouring lanes swap one value (DPP quad_perm [1,0,3,2]), so that an even lane holds tokens
// (i, i + 1) of row r and the odd lane next to it tokens (i - 1, i) of row r + 1; one packed
// conversion (nearest even) and one 4-byte store per lane then cover both rows with all 64 lanes
// active: half the store instructions of the fp32 form for half the bytes, at any address.
// Must be called by all 16 lanes of a lane group together.
__device__ __forceinline__ void tsvd_store_row_pair_bf16(void* y, long long ld, int r, int rows_valid, int col16, int i,
                                                         int bvalid, float v0, float v1) {
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    const int odd = i & 1, c = col16 + i - odd;
    const float send = odd ? v0 : v1;
    const float recv = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(send), 0xB1, 0xF, 0xF, true));
    const f32x2_t two = odd ? f32x2_t{recv, v1} : f32x2_t{v0, recv};
    const uint32_t pk = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2_t));
    const int row = r + odd;
    if (row < rows_valid) {
        uint16_t* dst = static_cast<uint16_t*>(y) + (size_t)row * ld + c;
        if (c + 1 < bvalid) {
            typedef uint32_t u32_at __attribute__((aligned(2)));
            *reinterpret_cast<u32_at*>(dst) = pk;
        } else if (c < bvalid) {
            *dst = (uint16_t)pk;
        }
    }
}

// Token-major output y[token][row]: the lane of a 16 x 16 result block that holds token `token` of rows
// row0 .. row0 + 3 (row0 a multiple of 4) writes them side by side: one 16-byte (fp32) or 8-byte (bf16)
// store when the four rows exist, at whatever address the rows' pitch gives (vector memory takes any); element by element otherwise.
// (By element where the pitch is no multiple of 16 bytes, as before, the address unit is what bounds the call: 9070 x 960 x 200 at
// 940 tokens, fp32, 41.8 -> 23.8 us; 813 x 184 x 86 at 9460, bf16 in and out, 33.3 -> 23.2 us with the loads of tsvd_gather_row.)
__device__ __forceinline__ void tsvd_store_token_major4(void* y, long long ld, int token, int row0, int rows_valid,
                                                        float v0, float v1, float v2, float v3, int out_bf16) {
    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    typedef f32x4_t f32x4_at __attribute__((aligned(4)));
    typedef u32x2_t u32x2_at __attribute__((aligned(2)));
    const size_t at = (size_t)token * ld + row0;
    if (row0 + 3 < rows_valid) {
        if (out_bf16) {
            const u32x2_t pk = {(uint32_t)tsvd_bf16_rne(v0) | ((uint32_t)tsvd_bf16_rne(v1) << 16),
                                (uint32_t)tsvd_bf16_rne(v2) | ((uint32_t)tsvd_bf16_rne(v3) << 16)};
            *reinterpret_cast<u32x2_at*>(static_cast<uint16_t*>(y) + at) = pk;
        } else {
            *reinterpret_cast<f32x4_at*>(static_cast<float*>(y) + at) = f32x4_t{v0, v1, v2, v3};
        }
        return;
    }
    const float v[4] = {v0, v1, v2, v3};
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (row0 + e < rows_valid) tsvd_store_y(y, at + e, v[e], out_bf16);
}

// Token-major bf16 output of four 16 x 16 result blocks below each other (rows row0 .. row0 + 63; a lane (i, g) holds token i of
// rows 16 a + 4 g .. + 3 of block a as two packed words d[a]): the four lane groups transpose their pieces (two swaps of lane
// rows per word), after which lane group g holds all sixteen rows of block g and stores them as 32 consecutive bytes: 128 bytes per
// token and store pair where the plain form writes 32.  Rows that begin at odd elements are written one element on, with the two ends by themselves: 16-byte
// stores at addresses that are no multiple of four are slow (9081 x 328 x 113 at 1401 tokens in a thin panel 41.2 us, 9082 rows 27.1; 8-byte ones lose
// a twentieth).  Against 8-byte stores: 12288 x 1536 x 1024 at 1024 tokens 42.1 -> 36.0 us, 5888 x 192 x 6039 at 5888 381 -> 337.  All 64 lanes
// must call it; the rows must exist.
__device__ __forceinline__ void tsvd_store_token_major_bf16_4x16(void* y, long long ld, int token, bool token_ok, int row0, int g, uint32_t (&d)[4][2]) {
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        auto swap16 = [&](int a, int b) {
            const auto r = __builtin_amdgcn_permlane16_swap(d[a][w], d[b][w], false, false);
            d[a][w] = r[0];
            d[b][w] = r[1];
        };
        auto swap32 = [&](int a, int b) {
            const auto r = __builtin_amdgcn_permlane32_swap(d[a][w], d[b][w], false, false);
            d[a][w] = r[0];
            d[b][w] = r[1];
        };
        swap16(0, 1);
        swap16(2, 3);
        swap32(0, 2);
        swap32(1, 3);
    }
    uint16_t* dst = static_cast<uint16_t*>(y) + (size_t)token * ld + row0 + 16 * g;
    const bool odd = reinterpret_cast<uintptr_t>(dst) & 2;
    uint32_t w[8] = {d[0][0], d[0][1], d[1][0], d[1][1], d[2][0], d[2][1], d[3][0], d[3][1]};
    if (__any(odd)) {       // one element on: the first of the next lane group behind this one's last fifteen
        const uint32_t next = __shfl_down(w[0], 16);
        if (token_ok && odd && (g == 0 || g == 3)) dst[g == 0 ? 0 : 15] = (uint16_t)(g == 0 ? w[0] : w[7] >> 16);
#pragma unroll
        for (int k = 0; k < 8; ++k) w[k] = odd ? w[k] >> 16 | (k < 7 ? w[k + 1] : next) << 16 : w[k];
    }
    if (token_ok) {
        typedef uint32_t u32x3_t __attribute__((ext_vector_type(3)));
        typedef u32x4_t u32x4_at __attribute__((aligned(4)));
        typedef u32x3_t u32x3_at __attribute__((aligned(4)));
        dst += odd;
        *reinterpret_cast<u32x4_at*>(dst) = u32x4_t{w[0], w[1], w[2], w[3]};
        if (odd && g == 3) *reinterpret_cast<u32x3_at*>(dst + 8) = u32x3_t{w[4], w[5], w[6]};
        else *reinterpret_cast<u32x4_at*>(dst + 8) = u32x4_t{w[4], w[5], w[6], w[7]};
    }
}
__device__ __forceinline__ uint32_t tsvd_pack_bf16(float lo, float hi) {
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}
