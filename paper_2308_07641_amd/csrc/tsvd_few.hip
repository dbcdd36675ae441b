// Few tokens (bf16 activations, groups of up to 16): the two stages of Y = U (diag(S) (V X)) (paper, section "Truncated SVD in
// Network Compression"; supplement Table S1), one launch each, a group of 16 tokens filling the columns of the matrix instruction.
//
// Such a call is bound by the chain of latencies of its two launches and, on large factors, by what a compute unit can take in: the codes
// once (HBM), and all activations for every workgroup (L2: 20 to 25 bytes a cycle and compute unit, as the 0.54 MB for each in the 10 us of stage U below).  So no
// barrier stands between the launch and the products, and activations are read in whole lines: a wavefront owns columns of tiles (256 indices of the
// contraction, kw wavefronts side by side), holds their activations in registers in operand order, and multiplies the tiles of SW strips
// by them, each tile requested one column ahead; the partial sums of the kw wavefronts meet in LDS once, at the end.
//
// Stage V multiplies bf16 x as it is (codes expanded to 0 / +2 / -2 in 16 bits: 64 operations and 8 MFMAs a tile) and leaves z as
// four or five E2M3 planes (tsvd_fp6_common.h), which stage U multiplies by the codes as fp4 numbers: 12 operations and 8 (10) MFMAs a tile
// (a tile is two blocks of 128 rank positions, 6 operations each).
//
// Measured on MI355X against the kernels that take x and fp16 z through LDS in slabs (tsvd_mid.hip): 16384 x 4096 x 8192, 16 tokens, token-major
// (a transposition pass before) 21.4 -> 18.0 us a call, in a kernel trace stage V 7.9 -> 6.5, stage U 12.0 -> 11.0 (33.5 MB of codes and 105 MB of z
// from L2).  Four planes rather than three: three cost 1.2 us less there and 0.7 us on small calls, but leave 2^-14 of the largest of 32
// neighbours, so rows of y made of ranks beside such that see a feature 2000 times the rest were off by 1.1e-3 (fp16 z 2.1e-4, four planes 3e-5).  A
// record of seven whole pieces cost 1.5 us more than six and the scales apart.  Loading operand lanes of x straight from rows of tokens cost stage V 1.5 us more (16-byte pieces of 32 lines per request), and requests
// of 8 and 4 bytes for the ends of the planes cost stage U 1 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <initializer_list>
#include <type_traits>

#include "tsvd_epilogue.h"
#include "tsvd_few.h"
#include "tsvd_fp6_common.h"

namespace {

// LDS of a wavefront for its column of x: the rows of 16 tokens, 256 values each, padded by 16 bytes against bank conflicts (256 rows of 32 bytes otherwise)
constexpr int ROW_PITCH = 528, WAVE_X = 16 * ROW_PITCH;
constexpr int RED_PITCH = 17, RED_BLOCK = 16 * RED_PITCH;      // floats: a 16 x 16 result block, rows padded against bank conflicts

__device__ __forceinline__ u32x2 lds_tr(const unsigned char* lds_byte_ptr) {
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr_t;
    s16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(lds_byte_ptr));
    return __builtin_bit_cast(u32x2, r);
}

// Record of z of (16 tokens, 128 rank positions): a lane's planes, 24 bytes each, in pieces of 16 bytes [pieces][64][16], and a scale byte for each.
// Four planes: six pieces, then the scales [64][4]; five planes: eight pieces, the scales in words 2 and 3 of the last.
constexpr int record_bytes(int planes) { return planes == 4 ? 6 * 1024 + 256 : 8 * 1024; }

// Operand of stage U: the pieces of a lane (four planes: six of them, word 0 of the seventh the scales).  (Variables of their own: from a structure or an array the compiler reads
// a plane's first words as part of a longer vector, and then keeps everything in scratch memory.)
#define FEW_OPERAND(n) u32x4 n##0, n##1, n##2, n##3, n##4, n##5, n##6, n##7
#define FEW_OPERAND_OF(n) n##0, n##1, n##2, n##3, n##4, n##5, n##6, n##7

// Strip `local` of workgroup b.  Two strips: s and s + 2, whose 32 rows are the two runs of one operand lane of stage U.
__device__ __forceinline__ int strip_of(int b, int strips_wg, int local) {
    return strips_wg == 2 ? 8 * (b >> 2) + 4 * ((b >> 1) & 1) + (b & 1) + 2 * local : b * strips_wg + local;
}

// Results that a thread finishes: SW strips of 256 for kw wavefronts.
template <int KWL, int SW>
constexpr int outputs_of = 4 * SW >> KWL > 1 ? 4 * SW >> KWL : 1;

// Sum over the kw wavefronts of element (row, token) of the workgroup's result.
template <int KWL, int SW>
__device__ __forceinline__ float sum_parts(const float* red, int row, int tok) {
    const int strip = row >> 4, rw = strip / SW, s = strip % SW;
    const float* src = red + (size_t)((rw << KWL) * SW + s) * RED_BLOCK + (row & 15) * RED_PITCH + tok;
    float a = 0.f;
#pragma unroll
    for (int c = 0; c < 1 << KWL; ++c) a += src[c * SW * RED_BLOCK];
    return a;
}

template <int KWL, int SW>
__device__ __forceinline__ void leave_parts(float* red, const f32x4 (&acc)[SW], int wave, int i, int g) {
    // result block of the MFMA: lane (i, g) holds token i, rows 4 g + v
#pragma unroll
    for (int s = 0; s < SW; ++s)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[(size_t)(wave * SW + s) * RED_BLOCK + (4 * g + v) * RED_PITCH + i] = acc[s][v];
}

// x[values] times row `row` of a strip's tiles, by a wavefront, in 64 bits: for the sums of doubled values that leave fp32 (|x| of 1e37 and more).
__device__ __forceinline__ double row_sum(const unsigned char* strip, int row, int nkt, const uint16_t* x, int step, int N, int lane) {
    double sum = 0.0;
    for (int n = lane; n < 16 * nkt; n += 64) {              // word d of lane (row, g) of tile T
        const int T = n >> 4, g = n >> 2 & 3, d = n & 3, at = 256 * T + 128 * (d >> 1) + 32 * (d & 1) + 64 * (g & 1) + 16 * (g >> 1);
        const uint32_t w = *reinterpret_cast<const uint32_t*>(strip + T * 1024 + (16 * g + row) * 16 + 4 * d);
        uint16_t v[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = x[(size_t)min(at + e, N - 1) * step];
#pragma unroll
        for (int e = 0; e < 16; ++e) {                       // value e: half e >> 3, of it register m = e & 3 in 16 bits e >> 2 & 1
            const uint32_t code = w >> (16 * (e >> 2 & 1) + 4 * (e & 3) + 2 * (e >> 3));      // (0 beyond N)
            const double value = (double)__uint_as_float((uint32_t)v[e] << 16);
            sum += code & 1 ? code & 2 ? -value : value : 0.0;
        }
    }
    for (int m = 1; m < 64; m *= 2) sum += __shfl_xor(sum, m);
    return sum;
}
__device__ __forceinline__ bool in_fp32(float z) { return fabsf(z) <= 3.402823466e38f; }        // (false for NaN)

// The arguments of either kernel.  They are passed one by one, and the first fourteen words come preloaded in registers: a load from the others takes 0.3 us, and
// everything waited for it in either launch (16384 x 4096 x 8192 at 16 tokens 16.7 -> 16.2 us, 428 x 949 x 320 at 7 6.85 -> 6.3, 10543 x 726 x 138 at 12
// 8.55 -> 8.0; of 50 drawn calls of 2 to 16 tokens the 18 that come here take 0.93 to 0.98 of the time).
struct tsvd_few_v_args {
    const unsigned char* tiles;
    const uint16_t* x;
    const float* S;
    unsigned char* planes;
    int nkt, ld, N, B, blocks, z_planes;
};
struct tsvd_few_u_args {
    const unsigned char *tiles, *planes;
    void* y;
    const float* bias;
    long long ld;
    int nkt, blocks, strips, B, M;
    int strips_wg, rows_log2, token_major, out_bf16;         // one word: tsvd_few_u_form
};
unsigned tsvd_few_u_form(const tsvd_few_args& a, int waves) { return (unsigned)a.strips_wg | (unsigned)a.rows_log2 << 8 | (a.token_major ? 1u << 16 : 0u) | (a.out_bf16 ? 1u << 17 : 0u) | (unsigned)waves << 20; }

}  // namespace

// Stage V.  Workgroup (b, t) of kw wavefronts: SW strips, tokens 16 t ...; wavefront q: tile columns q, q + kw, ...
//
// x is read in chunks of eight values, of any alignment, through LDS of the wavefront's own: TOKENS (rows of tokens): 16 rows of 256
// values, read back 16 bytes a lane, their halves regrouped; else (rows of features): 256 rows of 16 tokens, read back transposed, placed so
// that position r' of a 64-row stage holds row r' ^ 2 ((r' >> 4 ^ r' >> 5) & 1) and the lane groups served in a cycle hit different banks.
// A chunk that would pass the end of what may be read (of a row of tokens, of the whole array) is read that much earlier and shifted.
// NARROW: eight tokens at most: half of the chunks (the other columns of the products hold what stands there, and nobody reads them).
template <bool TOKENS, bool NARROW, int KWL, int SW>
__global__ void __launch_bounds__(64 << KWL)
tsvd_few_v_kernel(const unsigned char* p_tiles, const uint16_t* p_x, const float* p_S, unsigned char* p_planes, int p_nkt, int p_ld, int p_N, int p_B, int p_blocks, int p_z_planes) {
    const tsvd_few_v_args p = {p_tiles, p_x, p_S, p_planes, p_nkt, p_ld, p_N, p_B, p_blocks, p_z_planes};
    constexpr int kw = 1 << KWL;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4, q = wave;
    const int tok0 = blockIdx.y * 16;
    constexpr int threads = 64 * kw, outputs = SW * 256, CHUNKS = NARROW ? 4 : 8;
    float S[outputs_of<KWL, SW>];                            // of this thread's outputs
#pragma unroll
    for (int n = 0; n < outputs_of<KWL, SW>; ++n) {
        const int row = min(tid + n * threads, outputs - 1) >> 4;
        S[n] = p.S[strip_of(blockIdx.x, SW, row >> 4) * 16 + (row & 15)];
    }
    // (two strips of a workgroup are s and s + 2)
    const int strip_step = (SW == 2 ? 2 : 1) * p.nkt * 1024;
    const unsigned char* tiles = p.tiles + (size_t)strip_of(blockIdx.x, SW, 0) * (p.nkt * 1024);
    auto load_w = [&](int s, int T) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(tiles + s * strip_step + T * 1024) + lane); };
    const int ld = (int)p.ld, total = (p.N - 1) * ld + p.B;  // (rows of features: values from the first to the last)
    // the chunks of a lane: TOKENS: values 8 (lane & 31) .. of tokens 2 j and 2 j + 1; else: half `lane & 1` of the row at position
    // (lane >> 1) + 32 (j & 1) of stage j >> 1 (NARROW: the row at position `lane` of stage j)
    auto chunk_at = [&](int j, int T) {
        if constexpr (TOKENS) return T * 256 + 8 * (lane & 31);
        const int stage = NARROW ? j : j >> 1, pos = NARROW ? lane : (lane >> 1) + 32 * (j & 1), r = pos ^ ((((pos >> 4) ^ (pos >> 5)) & 1) << 1);
        return (T * 256 + 128 * (stage >> 1) + 32 * (stage & 1) + 64 * (r >> 5) + (r & 31)) * ld + tok0 + (NARROW ? 0 : 8 * (lane & 1));
    };
    const int chunk_end = (TOKENS ? p.N : total) - 8;        // the last place a chunk is read from
    u32x4 raw[CHUNKS];
    auto load_x = [&](int T) {
#pragma unroll
        for (int j = 0; j < CHUNKS; ++j) {
            const unsigned row = TOKENS ? (unsigned)min(tok0 + 2 * j + (lane >> 5), p.B - 1) * (unsigned)ld : 0u;
            __builtin_memcpy(&raw[j], p.x + (row + (unsigned)min(chunk_at(j, T), chunk_end)), 16);
        }
    };
    unsigned char* mine = smem + wave * WAVE_X;
    const int k_lane = 64 * (g & 1) + 16 * (g >> 1);
    const int rsel = i >> 2, tr_row = 32 * (g & 1) + 16 * (g >> 1) + (rsel >> 1) + 4 * (rsel & 1), sw2 = (g & 1) ^ (g >> 1);
    const int rd_lo = (tr_row + 2 * sw2) * 32 + (i & 3) * 8, rd_hi = (tr_row + 2 * (1 - sw2)) * 32 + (i & 3) * 8;
    // operand registers: register m of half hh of word d = values m and m + 4 of the eight from 128 (d >> 1) + 32 (d & 1) + 8 hh
    u32x4 fx[8];
    auto operand = [&](int T) {
        if (TOKENS ? (T + 1) * 256 > p.N : (long long)(T + 1) * 256 * ld + tok0 + 16 > (long long)chunk_end) {
#pragma unroll
            for (int j = 0; j < CHUNKS; ++j) {
                const int by = max(chunk_at(j, T) - chunk_end, 0);   // values that the chunk was read too early; eight and more: nothing of it exists
                if (by & 1) raw[j] = u32x4{raw[j].x >> 16 | raw[j].y << 16, raw[j].y >> 16 | raw[j].z << 16, raw[j].z >> 16 | raw[j].w << 16, raw[j].w >> 16};
                if (by & 2) raw[j] = u32x4{raw[j].y, raw[j].z, raw[j].w, 0u};
                if (by & 4) raw[j] = u32x4{raw[j].z, raw[j].w, 0u, 0u};
                if (by >= 8) raw[j] = u32x4{0u, 0u, 0u, 0u};
            }
        }
        if constexpr (TOKENS) {
#pragma unroll
            for (int j = 0; j < CHUNKS; ++j) *reinterpret_cast<u32x4*>(mine + (2 * j + (lane >> 5)) * ROW_PITCH + (lane & 31) * 16) = raw[j];
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const u32x4 r = *reinterpret_cast<const u32x4*>(mine + i * ROW_PITCH + (k_lane + 128 * (j >> 2) + 32 * ((j >> 1) & 1) + 8 * (j & 1)) * 2);
                fx[j] = u32x4{__builtin_amdgcn_perm(r.z, r.x, 0x05040100u), __builtin_amdgcn_perm(r.z, r.x, 0x07060302u),
                              __builtin_amdgcn_perm(r.w, r.y, 0x05040100u), __builtin_amdgcn_perm(r.w, r.y, 0x07060302u)};
            }
        } else {
#pragma unroll
            for (int j = 0; j < CHUNKS; ++j) *reinterpret_cast<u32x4*>(mine + j * (NARROW ? 2048 : 1024) + lane * (NARROW ? 32 : 16)) = raw[j];
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const u32x2 lo = lds_tr(mine + (j >> 1) * 2048 + rd_lo + (j & 1) * 256), hi = lds_tr(mine + (j >> 1) * 2048 + rd_hi + (j & 1) * 256);
                fx[j] = u32x4{lo.x, lo.y, hi.x, hi.y};
            }
        }
        __builtin_amdgcn_wave_barrier();
    };
    f32x4 acc[SW];
#pragma unroll
    for (int s = 0; s < SW; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 w[SW];
    // (the last column of a wavefront requests nothing more)
    auto column = [&](int T, auto last) {
        operand(T);
        if constexpr (!last) load_x(T + kw);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < SW; ++s) {
            const u32x4 now = w[s];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const uint32_t ww = now[d];
                const u32x4 av0 = {TSVD_DEC(ww, 0), TSVD_DEC(ww, 2), TSVD_DEC(ww, 4), TSVD_DEC(ww, 6)};
                const u32x4 av1 = {TSVD_DEC(ww, 1), TSVD_DEC(ww, 3), TSVD_DEC(ww, 5), ww & 0xC000C000u};
                acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av0), __builtin_bit_cast(bf16x8, fx[2 * d]), acc[s], 0, 0, 0);
                acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av1), __builtin_bit_cast(bf16x8, fx[2 * d + 1]), acc[s], 0, 0, 0);
            }
            if constexpr (!last) w[s] = load_w(s, T + kw);
        }
    };
    load_x(q);
    __builtin_amdgcn_sched_barrier(0);                       // activations first: results return in the order of the requests
#pragma unroll
    for (int s = 0; s < SW; ++s) w[s] = load_w(s, q);        // (q < nkt: there are no more wavefronts side by side than columns)
    int T = q;
    for (; T + kw < p.nkt; T += kw) column(T, std::false_type{});
    column(T, std::true_type{});
    // ---- sum of the parts, times S / 4 (the codes of either stage multiply as +-2)
    float* red = reinterpret_cast<float*>(smem);
    float* zl = reinterpret_cast<float*>(smem) + (size_t)kw * SW * RED_BLOCK;    // [16 strips_wg][17]
    __syncthreads();                                         // (the wavefronts' own columns are overwritten)
    leave_parts<KWL, SW>(red, acc, wave, i, g);
    __syncthreads();
#pragma unroll
    for (int n = 0; n < outputs_of<KWL, SW>; ++n) {
        const int e = tid + n * threads;
        if (e < outputs) {
            const float z = sum_parts<KWL, SW>(red, e >> 4, e & 15) * (0.25f * S[n]);
            zl[(e >> 4) * RED_PITCH + (e & 15)] = in_fp32(z) ? z : INFINITY;     // (no NaN: maxima do not show it)
        }
    }
    __syncthreads();
    if (wave) return;
    // ---- planes: thread (pair of strips m, token): the 32 values of one operand lane of stage U
    const bool busy = lane < SW * 8 && tok0 + (lane & 15) < p.B;
    const int m = (lane >> 4) & (SW / 2 - 1), t = lane & 15;
    const int l0 = SW == 2 ? 0 : m, l1 = SW == 2 ? 1 : l0 + 2;
    const int sg = strip_of(blockIdx.x, SW, l0), gr = ((sg >> 2) & 1) | ((sg & 1) << 1);
    float v[32], top;
    auto values = [&] {
        top = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            v[e] = zl[(16 * l0 + e) * RED_PITCH + t];
            v[16 + e] = zl[(16 * l1 + e) * RED_PITCH + t];
        }
#pragma unroll
        for (int e = 0; e < 32; ++e) top = fmaxf(top, fabsf(v[e]));
    };
    // Sums of doubled values leave fp32 from |x| of 1e37 on, though z may not: those are taken again by this wavefront alone.  (It costs others nothing but a
    // look at a maximum that is needed anyway: 0.05 us of 8 to 18.  A flag in LDS that all wavefronts look at: 0.3.)
    values();
    if (__builtin_expect(__any(busy && !in_fp32(top)), 0)) {
        for (int e = 0; e < outputs; ++e) {
            const int row = e >> 4, strip = strip_of(blockIdx.x, SW, row >> 4), token = tok0 + (e & 15);
            float& z = zl[row * RED_PITCH + (e & 15)];
            if (token >= p.B || in_fp32(z)) continue;
            const double sum = row_sum(p.tiles + (size_t)strip * p.nkt * 1024, row & 15, p.nkt, p.x + (TOKENS ? (size_t)token * ld : token), TOKENS ? 1 : ld, p.N, lane);
            const float exact = (float)(sum * (0.5 * (double)p.S[strip * 16 + (row & 15)]));
            z = in_fp32(exact) ? exact : INFINITY;
        }
        values();
    }
    if (busy) {
        const uint32_t lost = in_fp32(top) ? 0u : ~0u;       // scales of z that is beyond fp32 itself: no numbers in y
        u32x4 lo[5];
        u32x2 hi[5];
        const uint32_t scales = lost | tsvd_planes_of_32<true, 4, true, true>(v, [&](int pl, u32x4 l, u32x2 h) {
            lo[pl] = l;
            hi[pl] = h;
        }, top);
        unsigned char* rec_bytes = p.planes + ((size_t)blockIdx.y * p.blocks + (sg >> 3)) * record_bytes(p.z_planes);
        u32x4* rec = reinterpret_cast<u32x4*>(rec_bytes) + 16 * gr + t;
        rec[0] = lo[0];
        rec[64] = u32x4{hi[0].x, hi[0].y, lo[1].x, lo[1].y};
        rec[128] = u32x4{lo[1].z, lo[1].w, hi[1].x, hi[1].y};
        rec[192] = lo[2];
        rec[256] = u32x4{hi[2].x, hi[2].y, lo[3].x, lo[3].y};
        rec[320] = u32x4{lo[3].z, lo[3].w, hi[3].x, hi[3].y};
        if (p.z_planes == 4) {
            reinterpret_cast<uint32_t*>(rec_bytes + 6 * 1024)[16 * gr + t] = scales;
        } else {
            // v holds what four planes do not resolve
            const uint32_t fifth = lost | tsvd_planes_of_32<false, 1>(v, [&](int, u32x4 l, u32x2 h) {
                lo[4] = l;
                hi[4] = h;
            });
            rec[384] = lo[4];
            rec[448] = u32x4{hi[4].x, hi[4].y, scales, fifth};
        }
    }
}

// Stage U.  The records of two blocks (256 rank positions) in registers, 25 or 32 each; a block's next record is requested when its products are issued.
template <int PLANES, int KWL, int SW>
__global__ void __launch_bounds__(1024)
tsvd_few_u_kernel(const unsigned char* p_tiles, const unsigned char* p_planes, const float* p_bias, int p_nkt, int p_blocks, int p_strips, int p_B, int p_M, unsigned p_form, void* p_y, long long p_ld) {
    tsvd_few_u_args p = {p_tiles, p_planes, nullptr, p_bias, 0, p_nkt, p_blocks, p_strips, p_B, p_M, (int)(p_form & 31), (int)(p_form >> 8 & 31), (int)(p_form >> 16 & 1), (int)(p_form >> 17 & 1)};
    constexpr int kw = 1 << KWL;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4, q = wave & (kw - 1), rw = wave >> KWL;
    const int tok0 = blockIdx.y * 16, threads = (int)(p_form >> 20) * 64, rows = p.strips_wg * 16, row0 = blockIdx.x * rows;
    const int strip0 = blockIdx.x * p.strips_wg + rw * SW, strip_bytes = p.nkt * 1024;
    const unsigned char* z = p.planes + (size_t)blockIdx.y * p.blocks * record_bytes(PLANES) + (16 * g + min(i, p.B - 1 - tok0)) * 16;
    const unsigned char* z_scales = z + 6 * 1024 - (16 * g + min(i, p.B - 1 - tok0)) * 12;       // (four planes)
    // (tokens that do not exist: the last one's operands again: with one token a sixteenth of the bytes, and no uninitialised columns)
    // thread t finishes outputs t, t + threads, ...: the index that runs along a row of y first
    auto output = [&](int n, int& row, int& tok) {
        const int e = tid + n * threads;
        row = p.token_major ? e & (rows - 1) : e >> 4;       // (rows is a power of two)
        tok = p.token_major ? e >> p.rows_log2 : e & 15;
        return e < rows * 16 && row0 + row < p.M && tok0 + tok < p.B;
    };
    float bias[outputs_of<KWL, SW>];
#pragma unroll
    for (int n = 0; n < outputs_of<KWL, SW>; ++n) {
        int row, tok;
        (void)output(n, row, tok);
        bias[n] = p.bias ? p.bias[min(row0 + row, p.M - 1)] : 0.f;
    }
    // (a strip beyond the matrix: the last one again, its result is dropped)
    const unsigned char* tiles[SW];
#pragma unroll
    for (int s = 0; s < SW; ++s) tiles[s] = p.tiles + (size_t)min(strip0 + s, p.strips - 1) * strip_bytes;
    auto load_w = [&](int s, int T) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(tiles[s] + T * 1024) + lane); };
    auto load_z = [&](int block, u32x4& p0, u32x4& p1, u32x4& p2, u32x4& p3, u32x4& p4, u32x4& p5, u32x4& p6, u32x4& p7) {
        auto piece = [&](int c) { return *reinterpret_cast<const u32x4*>(z + (size_t)block * record_bytes(PLANES) + c * 1024); };
        p0 = piece(0), p1 = piece(1), p2 = piece(2), p3 = piece(3), p4 = piece(4), p5 = piece(5);
        if constexpr (PLANES == 5) p6 = piece(6), p7 = piece(7);
        else p6.x = *reinterpret_cast<const uint32_t*>(z_scales + (size_t)block * record_bytes(PLANES));
    };
    f32x4 acc[SW];
#pragma unroll
    for (int s = 0; s < SW; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 w[SW];
    // (the smallest planes first)
    auto multiply = [&](uint32_t w0, uint32_t w1, f32x4& a, const u32x4& p0, const u32x4& p1, const u32x4& p2, const u32x4& p3, const u32x4& p4,
                        const u32x4& p5, const u32x4& p6, const u32x4& p7) {
        const u32x4 av = {(w0 << 2) & 0xCCCCCCCCu, w0 & 0xCCCCCCCCu, (w1 << 2) & 0xCCCCCCCCu, w1 & 0xCCCCCCCCu};
        const uint32_t scales = PLANES == 5 ? p7.z : p6.x;
        if constexpr (PLANES == 5) a = mfma_fp6<0, 4>(av, p6, u32x2{p7.x, p7.y}, p7.w, a);
        a = mfma_fp6<3, 3>(av, u32x4{p4.z, p4.w, p5.x, p5.y}, u32x2{p5.z, p5.w}, scales, a);
        a = mfma_fp6<2, 2>(av, p3, u32x2{p4.x, p4.y}, scales, a);
        a = mfma_fp6<1, 1>(av, u32x4{p1.z, p1.w, p2.x, p2.y}, u32x2{p2.z, p2.w}, scales, a);
        a = mfma_fp6<0, 0>(av, p0, u32x2{p1.x, p1.y}, scales, a);
    };
    FEW_OPERAND(z0);
    FEW_OPERAND(z1);
    load_z(2 * q, FEW_OPERAND_OF(z0));
    load_z(2 * q + 1, FEW_OPERAND_OF(z1));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < SW; ++s) w[s] = load_w(s, q);        // (q < nkt: there are no more wavefronts side by side than columns)
    p.y = p_y;
    p.ld = p_ld;
    asm volatile("" : "+s"(p.y), "+s"(p.ld));               // (the pitch is not preloaded: read behind the first requests)
    auto column = [&](int T, auto last) {
        uint32_t second[SW][2];
#pragma unroll
        for (int s = 0; s < SW; ++s) {
            multiply(w[s].x, w[s].y, acc[s], FEW_OPERAND_OF(z0));
            second[s][0] = w[s].z;
            second[s][1] = w[s].w;
            if constexpr (!last) w[s] = load_w(s, T + kw);
        }
        if constexpr (!last) load_z(2 * (T + kw), FEW_OPERAND_OF(z0));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < SW; ++s) multiply(second[s][0], second[s][1], acc[s], FEW_OPERAND_OF(z1));
        if constexpr (!last) load_z(2 * (T + kw) + 1, FEW_OPERAND_OF(z1));
        __builtin_amdgcn_sched_barrier(0);
    };
    int T = q;
    for (; T + kw < p.nkt; T += kw) column(T, std::false_type{});
    column(T, std::true_type{});
    float* red = reinterpret_cast<float*>(smem);
    leave_parts<KWL, SW>(red, acc, wave, i, g);
    __syncthreads();
#pragma unroll
    for (int n = 0; n < outputs_of<KWL, SW>; ++n) {
        int row, tok;
        if (output(n, row, tok))
            tsvd_store_y(p.y, p.token_major ? (size_t)(tok0 + tok) * p.ld + row0 + row : (size_t)(row0 + row) * p.ld + tok0 + tok,
                         sum_parts<KWL, SW>(red, row, tok) + bias[n], p.out_bf16);
    }
}

namespace {

constexpr int lds_parts(int waves, int sw) { return waves * sw * RED_BLOCK * 4; }
int lds_v(int waves, int sw, int strips_wg) { return waves * WAVE_X > lds_parts(waves, sw) + strips_wg * RED_BLOCK * 4 ? waves * WAVE_X : lds_parts(waves, sw) + strips_wg * RED_BLOCK * 4; }
enum stage { STAGE_V, STAGE_U };

template <int KWL, int SW>
hipError_t init_one() {
    constexpr int most = 16 * WAVE_X;
    constexpr int S2 = SW < 2 ? 2 : SW;
    hipError_t e;
    for (const void* k : {(const void*)tsvd_few_u_kernel<4, KWL, SW>, (const void*)tsvd_few_u_kernel<5, KWL, SW>})
        if ((e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, most)) != hipSuccess) return e;
    for (const void* k : {(const void*)tsvd_few_v_kernel<true, true, KWL, S2>, (const void*)tsvd_few_v_kernel<true, false, KWL, S2>,
                          (const void*)tsvd_few_v_kernel<false, true, KWL, S2>, (const void*)tsvd_few_v_kernel<false, false, KWL, S2>})
        if ((e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, most)) != hipSuccess) return e;
    return hipSuccess;
}
template <int KWL>
hipError_t init_kw() {
    hipError_t e;
    if ((e = init_one<KWL, 1>()) != hipSuccess) return e;
    if ((e = init_one<KWL, 2>()) != hipSuccess) return e;
    return init_one<KWL, 4>();
}
template <int KWL, int SW>
hipError_t launch(const tsvd_few_args& a, stage st, dim3 grid, int waves, hipStream_t stream) {
    constexpr int S2 = SW < 2 ? 2 : SW;
    const dim3 block((unsigned)waves * 64);
    const unsigned lds = (unsigned)(st == STAGE_U ? lds_parts(waves, SW) : lds_v(waves, SW, a.strips_wg));
    if (st == STAGE_U) (a.z_planes == 4 ? tsvd_few_u_kernel<4, KWL, SW> : tsvd_few_u_kernel<5, KWL, SW>)<<<grid, block, lds, stream>>>(a.tiles, a.planes, a.bias, a.nkt, a.blocks, a.strips, a.B, a.M, tsvd_few_u_form(a, waves), a.y, a.ld);
    else if (SW == 1) return hipErrorInvalidValue;          // (planes are made of pairs of strips)
    else (a.token_major ? a.B <= 8 ? tsvd_few_v_kernel<true, true, KWL, S2> : tsvd_few_v_kernel<true, false, KWL, S2>
                        : a.B <= 8 ? tsvd_few_v_kernel<false, true, KWL, S2> : tsvd_few_v_kernel<false, false, KWL, S2>)<<<grid, block, lds, stream>>>(a.tiles, a.x, a.S, a.planes, a.nkt, (int)a.ld, a.N, a.B, a.blocks, a.z_planes);
    return hipGetLastError();
}
template <int KWL>
hipError_t launch_kw(const tsvd_few_args& a, stage x, dim3 grid, int waves, int sw, hipStream_t stream) {
    switch (sw) {
        case 1: return launch<KWL, 1>(a, x, grid, waves, stream);
        case 2: return launch<KWL, 2>(a, x, grid, waves, stream);
        default: return launch<KWL, 4>(a, x, grid, waves, stream);
    }
}

// The shape of a launch.  kw wavefronts side by side as the columns allow.  Stage V: two strips each, four where two would be more wavefronts than
// the compute units hold.  Stage U: strips until a workgroup per compute unit is left, first more for each wavefront (its operands serve them
// all), then more wavefronts.  (Against the best of all shapes on 190 calls of random sizes: 3 and 4 % slower on the average.)
struct shape {
    int kwl, sw, rw;
    long long workgroups;
};
shape shape_of(stage st, long long strips, long long nkt, long long groups, long long cus) {
    int kwl = 0, sw = 2, rw = 1;
    while (kwl < 4 && (2 << kwl) <= nkt) ++kwl;
    kwl = std::max(0, std::min(kwl, tsvd_tune("TSVD_FEW_KWLOG2", kwl)));
    auto workgroups = [&] { return (strips + sw * rw - 1) / (sw * rw) * groups; };
    if (st == STAGE_V) {
        if (workgroups() << kwl > 16 * cus) sw = 4;
        sw = tsvd_tune("TSVD_FEW_SW_V", sw) == 4 ? 4 : 2;
    } else {
        sw = 1, rw = 2;
        while (sw * rw < 16 && workgroups() > cus) sw < 4 ? sw *= 2 : rw *= 2;
        sw = tsvd_tune("TSVD_FEW_SW_U", sw);
        rw = tsvd_tune("TSVD_FEW_RW_U", rw);
        while (rw << kwl > 16) {                             // (16 wavefronts at most: the same strips on fewer of them, else fewer side by side)
            if (rw > 1 && sw < 4) rw /= 2, sw *= 2;
            else --kwl;
        }
    }
    return {kwl, sw, rw, workgroups()};
}

hipError_t launch_stage(tsvd_few_args a, stage st, int groups, int cus, hipStream_t stream) {
    const shape f = shape_of(st, a.strips, a.nkt, groups, cus);
    if ((f.sw != 1 && f.sw != 2 && f.sw != 4) || f.rw < 1 || (f.rw & (f.rw - 1)) || f.sw * f.rw > 16) return hipErrorInvalidValue;
    a.strips_wg = f.sw * f.rw;
    a.rows_log2 = __builtin_ctz((unsigned)a.strips_wg * 16);
    const int waves = f.rw << f.kwl;
    const dim3 grid((unsigned)(f.workgroups / groups), (unsigned)groups);
    switch (f.kwl) {
        case 0: return launch_kw<0>(a, st, grid, waves, f.sw, stream);
        case 1: return launch_kw<1>(a, st, grid, waves, f.sw, stream);
        case 2: return launch_kw<2>(a, st, grid, waves, f.sw, stream);
        case 3: return launch_kw<3>(a, st, grid, waves, f.sw, stream);
        default: return launch_kw<4>(a, st, grid, waves, f.sw, stream);
    }
}

}  // namespace

hipError_t tsvd_few_init() {
    hipError_t e;
    if ((e = init_kw<0>()) != hipSuccess) return e;
    if ((e = init_kw<1>()) != hipSuccess) return e;
    if ((e = init_kw<2>()) != hipSuccess) return e;
    if ((e = init_kw<3>()) != hipSuccess) return e;
    return init_kw<4>();
}

size_t tsvd_few_bytes(long long Kp, long long B, int planes) { return (size_t)((B + 15) / 16) * (size_t)(Kp / 128) * record_bytes(planes); }

// A call in microseconds: launches, columns of a wavefront in turn, columns that the wavefronts of a compute unit share (activations, then
// strips), rounds of workgroups, results.  Non-negative least squares on relative errors over 500 calls of random sizes (2 to 600 tokens): 11 % rms.
double tsvd_few_cost(const tsvd_few_call& c) {
    const long long groups = (c.B + 15) / 16, nkt_v = (c.N + 255) / 256, nkt_u = (c.K + 255) / 256;
    struct stage_terms { double turn, share, rounds; int sw; };
    auto terms = [&](stage st, long long strips, long long nkt) {
        const shape f = shape_of(st, strips, nkt, groups, c.cus);
        const double columns = (double)((nkt + (1 << f.kwl) - 1) >> f.kwl);
        const long long slots = c.cus * std::max(1, 16 / (f.rw << f.kwl));
        const double rounds = (double)((f.workgroups + slots - 1) / slots);
        return stage_terms{columns * rounds, (double)((f.workgroups * f.rw) << f.kwl) * columns / (double)c.cus, rounds - 1, f.sw};
    };
    const stage_terms v = terms(STAGE_V, nkt_u * 16, nkt_v), u = terms(STAGE_U, (c.M + 15) / 16, nkt_u);
    const double results = (double)c.M * (double)c.B * (c.out_bf16 ? 0.5 : 1.0) / (1e3 * (double)c.cus);
    return 6.24 + 0.38 * u.turn + 0.056 * u.sw * u.share + 0.13 * u.rounds + 0.45 * results + 0.56 * v.turn +
           ((c.x_token_major ? 0 : c.x_aligned ? 0.069 : 0.182) + 0.077 * v.sw) * v.share + 0.96 * v.rounds;
}

bool tsvd_few_fits(const tsvd_blob_header& hd, long long B, long long ldx, bool x_token_major) {
    // (32-bit places of values, of the column behind the last too; 16 strips of a workgroup; a chunk of eight values to read)
    const long long limit = 1ll << 30, N = x_token_major ? hd.N : (hd.N - 1) * ldx + B;
    return ldx <= limit && ldx * (x_token_major ? B : hd.Np) < limit && N >= 8 && 2 * (hd.Np > hd.Kp ? hd.Np : hd.Kp) * 4 * 16 < limit && B <= 16 * 65535;
}

hipError_t tsvd_few_launch(const tsvd_few_problem& f, hipStream_t stream) {
    const tsvd_blob_header& hd = *f.hd;
    const int groups = (int)((f.B + 15) / 16);
    tsvd_few_args a = {};
    a.B = (int)f.B;
    a.planes = f.planes;
    a.blocks = (int)(hd.Kp / 128);
    a.z_planes = f.z_planes;
    hipError_t e;
    if (f.stages & 2) {
        a.tiles = f.blob + hd.off_V;
        a.strips = (int)(hd.Kp / 16);
        a.nkt = (int)(hd.Np / 256);
        a.x = f.x;
        a.ld = f.ldx;
        a.token_major = f.x_token_major;
        a.N = (int)hd.N;
        a.S = reinterpret_cast<const float*>(f.blob + hd.off_S);
        if ((e = launch_stage(a, STAGE_V, groups, f.cu_count, stream)) != hipSuccess) return e;
    }
    if (f.stages & 4) {
        a.tiles = f.blob + hd.off_U;
        a.strips = (int)((hd.M + 15) / 16);
        a.nkt = (int)(hd.Kp / 256);
        a.y = f.y;
        a.ld = f.ldy;
        a.token_major = f.y_token_major;
        a.M = (int)hd.M;
        a.bias = f.bias;
        a.out_bf16 = f.out_bf16;
        if ((e = launch_stage(a, STAGE_U, groups, f.cu_count, stream)) != hipSuccess) return e;
    }
    return hipSuccess;
}
