// Batched stages on fp4 codes x fp6 planes for launches with few tiles: the contraction of a tile is split over the
// wavefronts of its workgroup.  With it the operand pass that serves any layout of the activations.
//
// The kernels of tsvd_fp6.hip give every wavefront its own rows of a tile and let all of them walk the contraction
// together.  With fewer than two such tiles per compute unit a SIMD holds a single wavefront, which issues a matrix
// instruction every 24.5 cycles (16 is the pipe), and a contraction of a dozen blocks is a dozen barriers.  Here eight
// wavefronts share a tile of RW x 128 rows and 16 TN tokens: KG = 8 / RW groups of them take blocks of the contraction of their own, so a SIMD always has
// two wavefronts, and each wavefront still multiplies 128 rows (eight row blocks) by every operand that it reads.  At the end the partial sums of
// the groups meet in LDS, each group finishing its share of the tile.  Nobody waits for wavefronts that it shares nothing with: tiles of 256 rows
// (tsvd_fp6_pair_kernel) tie two of them to each other, those of 128 rows (tsvd_fp6_own_kernel) none; where stage V makes the records of x itself, all
// wavefronts do that first and meet once (tsvd_fp6_panel_kernel).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "tsvd_fp6_common.h"

namespace {

// ---- the operand lanes of x ----------------------------------------------------------------------
// The 32 values of one lane of the record of (16-token tile, 128-index block), from activations in any layout: indices k0 + 32 (e >> 4) +
// (e & 15); indices beyond N read as zero, tokens beyond B as anything.  slot: 4 KiB of LDS of this wavefront, for bf16.  (Feature-major bf16 with a load per
// value before: 5541 x 729 x 4962 at 50 tokens 17.2 -> 15.5 us, 704 x 5696 x 767 at 378 21.4 -> 19.4, 256 x 8183 x 2961 at 92 24.0 -> 22.6.)
template <bool F32>
__device__ __forceinline__ void gather_x(const void* x, long long ld, bool token_major, int N, int B, int block, int tile, int lane, float (&v)[32], unsigned char* slot) {
    using T = std::conditional_t<F32, uint32_t, uint16_t>;
    const int i = lane & 15, g = lane >> 4, tok = tile * 16 + i, k0 = block * 128 + 64 * (g & 1) + 16 * (g >> 1), tc = min(tok, B - 1);
    const T* p = static_cast<const T*>(x);
    if (token_major) {
        tsvd_gather_row(p + (size_t)tc * ld, k0, N, block * 128 + 128 <= N, v);
#pragma unroll
        for (int e = 0; e < 32; ++e)
            if (tok >= B) v[e] = 0.f;
        return;
    }
    if constexpr (!F32) {
        u32x4 chunks[4];
        tsvd_request_columns(p, ld, N, B, block, 16 * tile, lane, chunks);
        tsvd_columns_of(chunks, ld, N, B, block, 16 * tile, lane, slot, v);
    } else {
        T r[32];
#pragma unroll
        for (int e = 0; e < 32; ++e) r[e] = p[(size_t)min(k0 + 32 * (e >> 4) + (e & 15), N - 1) * ld + tc];
#pragma unroll
        for (int e = 0; e < 32; ++e) v[e] = tok < B && k0 + 32 * (e >> 4) + (e & 15) < N ? __uint_as_float(r[e]) : 0.f;
    }
}

// The operand pass: a wavefront makes one record (fp32: two, six planes), token tile blockIdx.x * 4 + wave, block blockIdx.y
// (four neighbouring tiles per workgroup: feature-major rows are then read in runs of 64 tokens).
template <bool F32>
__global__ void __launch_bounds__(256)
tsvd_planes_kernel(const void* __restrict__ x, long long ld, int token_major, int N, int B, int nblocks, unsigned char* __restrict__ planes) {
    const int tile = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    __shared__ __align__(16) unsigned char slots[F32 ? 16 : 4 * 4096];
    if (tile * 16 >= B) return;
    float v[32];
    gather_x<F32>(x, ld, token_major != 0, N, B, blockIdx.y, tile, lane, v, slots + (F32 ? 0 : (tile & 3) * 4096));
    unsigned char* rec = planes + ((size_t)((tile >> 3) * (F32 ? 2 * nblocks : nblocks) + blockIdx.y) * 8 + (tile & 7)) * FP6_REC_BYTES;
    if constexpr (F32) tsvd_planes_of_32_twice(v, rec, rec + (size_t)nblocks * 8 * FP6_REC_BYTES, lane);   // a second set behind the first
    else tsvd_planes_of_32(v, rec, lane);
}

// ---- a stage ------------------------------------------------------------------------------------
// X (stage V): the workgroup makes the records of x itself, all of them at the start, where two steps hold them: every row tile
// makes them again, and a launch with its ramp and the gap before it (4 us) is saved for about 1.5 us.  1: bf16, 2: fp32.
struct split_x {
    const void* x;
    long long ld;
    int token_major, N;
};
// Which tiles an XCD works on (workgroups go to the eight of them in turn: a grid of 8 x tiles x rows): 1 << row_log2 groups of group_rows row tiles, times
// 8 >> row_log2 groups of group_tiles token tiles, one pair of groups for each, so that its L2 fetches a part of the codes and a part of the
// planes.  (Launches without such groups, a grid of token tiles x row tiles, are kernels of their own: the choice by an argument cost each of them 0.15 us.)
struct split_place {
    int row_log2, row_tiles, token_tiles, group_tiles, group_rows;          // group_tiles, group_rows: gridDim.y, gridDim.z
};
// Workgroups without a tile get the last one and end behind their first requests, which stay inside the codes and records with it.  (Where they ended before those, the
// compiler read half of the arguments behind that branch: 3072 x 768 x 1536 fp32 at 197 tokens 16.95 -> 17.15 us.)
struct split_tile {
    int token, row;
    bool exists;
};
template <bool PLACED, typename Extra>
__device__ __forceinline__ split_tile tile_of(const Extra& p) {
    if constexpr (PLACED) {
        const int row = (blockIdx.x & ((1 << p.row_log2) - 1)) * p.group_rows + blockIdx.z, token = (blockIdx.x >> p.row_log2) * p.group_tiles + blockIdx.y;
        return {min(token, p.token_tiles - 1), min(row, p.row_tiles - 1), row < p.row_tiles && token < p.token_tiles};
    } else {
        return {(int)blockIdx.x, (int)blockIdx.y, true};
    }
}

// The arguments of a stage.  Its first requests need fourteen words, which come preloaded in registers; a load from the others takes 0.3 us, and everything waits for it
// (3072 x 768 x 1536 fp32 at 197 tokens 17.1 -> 16.6 us, 741 x 1024 x 413 fp32 at 102 11.75 -> 11.3, 1051 x 2539 x 559 at 256 13.7 -> 13.2; none of 50 drawn calls longer).  extra: words of split_x (its x stands at `act` then, N at act_bytes) or of split_place.
#define SPLIT_ARGUMENTS const uint32_t *p_tiles, const void *p_act, unsigned p_tile_bytes, unsigned p_act_bytes, int p_nkt, int p_npairs, int p_code_blocks, int p_plane_blocks, int p_bvalid, \
                        unsigned p_extra0, unsigned p_extra1, unsigned p_extra2, gemm_args p_rest
#define SPLIT_STRUCT split_stage(p_tiles, p_act, p_tile_bytes, p_act_bytes, p_nkt, p_npairs, p_code_blocks, p_plane_blocks, p_bvalid, p_rest)
__device__ __forceinline__ gemm_args split_stage(const uint32_t* tiles, const void* act, unsigned tile_bytes, unsigned act_bytes, int nkt, int npairs, int code_blocks, int plane_blocks, int bvalid,
                                                 const gemm_args& rest) {
    gemm_args p = rest;
    p.tiles = tiles, p.act = static_cast<const uint16_t*>(act), p.tile_bytes = tile_bytes, p.act_bytes = act_bytes;
    p.nkt = nkt, p.npairs = npairs, p.code_blocks = code_blocks, p.plane_blocks = plane_blocks, p.bvalid = bvalid;
    return p;
}
__device__ __forceinline__ split_x split_x_of(const void* x, unsigned N, unsigned ld_low, unsigned ld_high, unsigned token_major) {
    return {x, (long long)((unsigned long long)ld_high << 32 | ld_low), (int)token_major, (int)N};
}
__device__ __forceinline__ split_place split_place_of(unsigned e0, unsigned e1) { return {(int)(e1 & 3), (int)(e0 & 0xFFFF), (int)(e0 >> 16), (int)(e1 >> 2 & 0x7FFF), (int)(e1 >> 17)}; }
// (what the ends of a stage need, read behind its first requests: its lines are near when they are wanted)
__device__ __forceinline__ void split_touch(const gemm_args& p) { asm volatile("" ::"s"(p.S), "s"(p.out), "s"(p.rows_valid), "s"(p.rows_need)); }

// z = S (V x) / 4 (the codes of either stage multiply as +-2) of rank block kb and the token tile from tok on, whose result blocks are sum -> its record.
__device__ __forceinline__ void finish_z(const gemm_args& p, f32x4 (&sum)[8], int kb, int tok, int lane) {
    const int g = lane >> 4;
    if (kb >= p.rows_need / 128) return;
    float v[32];
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        const f32x4 sv = *reinterpret_cast<const f32x4*>(p.S + 128 * kb + 64 * (g & 1) + 16 * (g >> 1) + 32 * (a >> 2) + 4 * (a & 3));
        sum[a] *= 0.25f * sv;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * a + e] = sum[a][e];
    }
    unsigned char* rec = static_cast<unsigned char*>(p.out) + ((size_t)((tok >> 7) * (int)p.ld_out + kb) * 8 + ((tok & 127) >> 4)) * FP6_REC_BYTES;
    if (p.two_sets) tsvd_planes_of_32_twice(v, rec, rec + (size_t)p.two_sets * 8 * FP6_REC_BYTES, lane);
    else tsvd_planes_of_32(v, rec, lane);
}

// ---- stage V that makes the records of x itself, in tiles that several wavefronts read them in -------
// Step s of wavefront (rw, kg): blocks (s KG + kg) BPS .. + BPS - 1, so 16 records (76 KiB) a step, and two steps hold all of x of a token tile: made at the
// start, by all wavefronts, and multiplied behind a single barrier.
// Measured on MI355X without the barrier and the turn of buffers that each step had: 2099 x 500 x 5441 fp32 at 657 tokens 56.7 -> 50.6 us, 5854 x 256 x 1383 fp32 at
// 328 23.3 -> 21.6, 13446 x 128 x 8569 fp32 at 781 296 -> 272 (each with a stage U of pairs where that has 256 rows).
template <int RW, int TN, int X>
__global__ void __launch_bounds__(512, 1)
tsvd_fp6_panel_kernel(SPLIT_ARGUMENTS) {
    const gemm_args p = SPLIT_STRUCT;
    const split_x xs = split_x_of(p_act, p_act_bytes, p_extra0, p_extra1, p_extra2);
    constexpr int KG = 8 / RW, BPS = 16 / (KG * TN), TM = 8, RECS = KG * BPS * TN;
    static_assert(RECS == 16 && BPS >= 1, "16 records per step");
    constexpr int CHUNK = TN * FP6_REC_BYTES, STEP_BYTES = RECS * FP6_REC_BYTES;   // a chunk: a block's TN records
    constexpr int NFR = TN == 4 ? 4 : 8;                    // result blocks that meet in LDS at a time
    static_assert((size_t)TN * (KG - 1) * RW * NFR * 1024 <= 2 * STEP_BYTES, "the partial sums fit the records");
    extern __shared__ __align__(16) unsigned char smem[];   // 2 x STEP_BYTES
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rw = wave % RW, kg = wave / RW, i = lane & 15, g = lane >> 4;
    const int b0 = blockIdx.x * 16 * TN, strip0 = (blockIdx.y * RW + rw) * TM;
    const int nrun = p.npairs;
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(p.tiles), 0, p.tile_bytes, 0x00020000);

    // row 4 gg + vv of result block a comes from row 64 (gg & 1) + 16 (gg >> 1) + 32 (a >> 2) + 4 (a & 3) + vv of the
    // wavefront's 128, so that result lane (g, token) holds the 32 rank positions of stage U's operand lane (see fp6_tile)
    const int gg = i >> 2, vv = i & 3;
    const int w_voff = (4 * (gg & 1) + (gg >> 1)) * p.nkt * 1024 + (g * 16 + vv) * 16;
    u32x2 w[2][BPS][TM];
#pragma unroll
    for (int step = 0; step < 2; ++step)
#pragma unroll
        for (int j = 0; j < BPS; ++j) {
            int blk = min((step * KG + kg) * BPS + j, nrun - 1);
            if (p.code_blocks && blk >= p.code_blocks) blk -= p.code_blocks;      // (second set of planes: the same codes again)
            const int soff = (strip0 * p.nkt + (blk >> 1)) * 1024 + (blk & 1) * 8;
#pragma unroll
            for (int a = 0; a < TM; ++a)
                w[step][j][a] = __builtin_amdgcn_raw_buffer_load_b64(w_rsrc, w_voff, soff + 2 * (a >> 2) * p.nkt * 1024 + 4 * (a & 3) * 16, 0);
        }
    const int blocks = X == 2 ? nrun / 2 : nrun;             // (fp32: the second set of planes are further blocks)
    auto record = [&](int blk, int tile) {
        const int step = blk / (KG * BPS);
        return smem + step * STEP_BYTES + (blk - step * KG * BPS) * CHUNK + tile * FP6_REC_BYTES;
    };
    for (int q = wave; q < blocks * TN; q += 8) {
        const int blk = q / TN, tile = q - blk * TN;
        float v[32];
        gather_x<X == 2>(xs.x, xs.ld, xs.token_major != 0, xs.N, p.bvalid, blk, (b0 >> 4) + tile, lane, v, record(blk, tile));
        if constexpr (X == 2) tsvd_planes_of_32_twice(v, record(blk, tile), record(blk + blocks, tile), lane);
        else tsvd_planes_of_32(v, record(blk, tile), lane);
    }
    __syncthreads();

    f32x4 acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the operands of an MFMA step (one plane of one record, eight row blocks) are read two steps ahead
#pragma unroll
    for (int step = 0; step < 2; ++step) {
        const unsigned char* mine = smem + step * STEP_BYTES + kg * BPS * CHUNK;
        const int valid = nrun - (step * KG + kg) * BPS;     // blocks of this step that exist
        if (valid <= 0) break;
        constexpr int STEPS = 3 * BPS * TN;
        u32x4 lo[3];
        u32x2 hi[3];
        uint32_t sc[2];
        auto read_step = [&](int st) {
            const unsigned char* rec = mine + (st / 3) * FP6_REC_BYTES;
            const int pl = st % 3;
            lo[pl] = *reinterpret_cast<const u32x4*>(rec + pl * 1024 + lane * 16);
            hi[pl] = *reinterpret_cast<const u32x2*>(rec + 3072 + pl * 512 + lane * 8);
            if (pl == 0) sc[(st / 3) & 1] = *reinterpret_cast<const uint32_t*>(rec + 4608 + lane * 4);
        };
        read_step(0);
        read_step(1);
#pragma unroll
        for (int j = 0; j < BPS; ++j) {
            if (j >= valid) break;
            u32x4 av[TM];
#pragma unroll
            for (int a = 0; a < TM; ++a) {
                const u32x2 c = w[step][j][a];
                av[a] = u32x4{(c.x << 2) & 0xCCCCCCCCu, c.x & 0xCCCCCCCCu, (c.y << 2) & 0xCCCCCCCCu, c.y & 0xCCCCCCCCu};
            }
#pragma unroll
            for (int t = 0; t < 3 * TN; ++t) {
                const int st = j * 3 * TN + t;
                if (st + 2 < STEPS) read_step(st + 2);
                __builtin_amdgcn_sched_barrier(0);
                const int b = t / 3;
#pragma unroll
                for (int a = 0; a < TM; ++a) {
                    switch (t % 3) {
                        case 0: acc[a][b] = mfma_fp6<0>(av[a], lo[0], hi[0], sc[(st / 3) & 1], acc[a][b]); break;
                        case 1: acc[a][b] = mfma_fp6<1>(av[a], lo[1], hi[1], sc[(st / 3) & 1], acc[a][b]); break;
                        default: acc[a][b] = mfma_fp6<2>(av[a], lo[2], hi[2], sc[(st / 3) & 1], acc[a][b]); break;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    __syncthreads();

    // ---- the groups' partial sums: result block f = 8 tile + row block; group q finishes token tile q
    f32x4 fin[8];
#pragma unroll
    for (int q = 0; q < TN; ++q)
        if (q == kg) {
#pragma unroll
            for (int f = 0; f < 8; ++f) fin[f] = acc[f][q];
        }
#pragma unroll
    for (int f0 = 0; f0 < 8; f0 += NFR) {
        auto slot = [&](int q, int other, int f) { return smem + ((((q * (KG - 1) + other) * RW + rw) * NFR + f) * 64 + lane) * 16; };
        if (f0 > 0) __syncthreads();
#pragma unroll
        for (int q = 0; q < TN; ++q)
            if (q != kg) {
                const int other = kg < q ? kg : kg - 1;
#pragma unroll
                for (int f = 0; f < NFR; ++f) *reinterpret_cast<f32x4*>(slot(q, other, f)) = acc[f0 + f][q];
            }
        __syncthreads();
        if (kg < TN) {
#pragma unroll
            for (int other = 0; other < KG - 1; ++other)
#pragma unroll
                for (int f = 0; f < NFR; ++f) fin[f0 + f] += *reinterpret_cast<const f32x4*>(slot(kg, other, f));
        }
    }
    if (kg < TN) finish_z(p, fin, strip0 >> 3, b0 + 16 * kg, lane);
}

// ---- tiles of 256 rows: a pair of wavefronts goes its own way -----------------------------------------
// Two wavefronts (rw = 0, 1), on two SIMDs, share the records of their blocks; the other three pairs of the workgroup have blocks of their own.  So only the two
// wait for each other, through words in LDS: a SIMD's older wavefront, which issues first, is then a step or two ahead of its younger
// one instead of idle in front of a barrier.  A step is four records, two steps in LDS for each pair, copied by its two wavefronts
// (buffer_load ... lds) while the other one is multiplied.
// Measured on MI355X against one barrier for all eight wavefronts before each step of 16 records: 16384 x 4096 x 8192 bf16 at 256 tokens 68.3 -> 65.2 us,
// 773 x 7298 x 1424 at 981 41.9 -> 37.2, 12534 x 640 x 8950 at 92 41.5 -> 35.5, 13876 x 640 x 6211 at 256 49.0 -> 46.5; on 45 drawn calls that take these tiles 0.85 to
// 1.0 of the time.  What bounds it is the issue of a SIMD's two wavefronts: 24 to 27 cycles a matrix instruction where the pipe takes 16 to 18, the codes'
// decoding and the operand reads between them.
template <int TN, bool STAGE2, int EX, bool PLACED>
__global__ void __launch_bounds__(512, 1)
tsvd_fp6_pair_kernel(SPLIT_ARGUMENTS) {
    const gemm_args p = SPLIT_STRUCT;
    constexpr int RW = 2, KG = 4, TM = 8, BPS = 4 / TN;
    constexpr bool DIRECT = !STAGE2;
    constexpr int CHUNK = TN * FP6_REC_BYTES, PIECES = (CHUNK + 1023) / 1024, STEP_BYTES = BPS * CHUNK;
    constexpr int NQ = DIRECT ? TN : KG, NF = 8 * TN / NQ, NFR = TN == 4 ? 4 : NF;
    static_assert((size_t)NQ * (KG - 1) * RW * NFR * 1024 <= 8 * STEP_BYTES, "the partial sums fit the buffers");
    extern __shared__ __align__(16) unsigned char smem[];    // [pair][2] steps, then 16 TN ones, then a word for each wavefront
    float* ones = reinterpret_cast<float*>(smem + 8 * STEP_BYTES);
    int* ready = reinterpret_cast<int*>(ones + 16 * TN);
    const split_tile tile = tile_of<PLACED>(split_place_of(p_extra0, p_extra1));
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rw = wave % RW, kg = wave / RW, i = lane & 15, g = lane >> 4;
    const int b0 = tile.token * 16 * TN, strip0 = (tile.row * RW + rw) * TM;
    const int nrun = p.npairs, nsteps = (nrun + BPS - 1) / BPS, nblocks = p.plane_blocks;
    // steps of this pair
    const int from = nsteps * kg / KG, count = nsteps * (kg + 1) / KG - from;
    if (threadIdx.x < 16 * TN) ones[threadIdx.x] = 1.0f;
    if (threadIdx.x < 8) ready[threadIdx.x] = 0;

    const i32x4 act_rsrc = raw_rsrc(p.act, p.act_bytes);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(p.tiles), 0, p.tile_bytes, 0x00020000);
    typedef __attribute__((address_space(3))) unsigned char* lds_byte_ptr;
    unsigned char* const mine = smem + kg * 2 * STEP_BYTES;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_byte_ptr)mine;

    f32x4 acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto issue = [&](int step, int buf) {                    // step of the launch; this wavefront's half of its pieces
#pragma unroll
        for (int c = 0; c < (BPS * PIECES + 1) / 2; ++c) {
            const int idx = 2 * c + rw, chunk = idx / PIECES, piece = idx - chunk * PIECES, blk = step * BPS + chunk;
            if (idx < BPS * PIECES && blk < nrun) {
                const int at = piece * 1024 + lane * 16;
                if (CHUNK % 1024 == 0 || at < CHUNK)         // (lanes beyond the chunk would write into the next one)
                    buf_load128_to_lds(act_rsrc, lds_base + buf * STEP_BYTES + chunk * CHUNK + piece * 1024, lane * 16,
                                       ((b0 >> 7) * nblocks + blk) * FP6_PAIR_BYTES + ((b0 & 127) >> 4) * FP6_REC_BYTES + piece * 1024);
            }
        }
    };
    // (rows of stage V as in tsvd_fp6_panel_kernel)
    const int gg = i >> 2, vv = i & 3;
    const int w_voff = DIRECT ? (4 * (gg & 1) + (gg >> 1)) * p.nkt * 1024 + (g * 16 + vv) * 16 : lane * 16;
    auto load_w = [&](int step, u32x2 (&w)[BPS][TM]) {
#pragma unroll
        for (int j = 0; j < BPS; ++j) {
            int blk = min(step * BPS + j, nrun - 1);
            if (p.code_blocks && blk >= p.code_blocks) blk -= p.code_blocks;      // (second set of planes: the same codes again)
            const int soff = (strip0 * p.nkt + (blk >> 1)) * 1024 + (blk & 1) * 8;
#pragma unroll
            for (int a = 0; a < TM; ++a)
                w[j][a] = __builtin_amdgcn_raw_buffer_load_b64(
                    w_rsrc, w_voff, soff + (DIRECT ? 2 * (a >> 2) * p.nkt * 1024 + 4 * (a & 3) * 16 : a * p.nkt * 1024), 0);
        }
    };
    auto touch = [&](const u32x2 (&w)[BPS][TM]) {
#pragma unroll
        for (int j = 0; j < BPS; ++j)
#pragma unroll
            for (int a = 0; a < TM; ++a) asm volatile("" :: "v"(w[j][a].x), "v"(w[j][a].y));
    };
    // What both wavefronts of the pair requested for their step `s` has arrived, and both are done with the step before it.
    auto meet = [&](int s) {
        __hip_atomic_store(ready + wave, s + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        while (__hip_atomic_load(ready + (wave ^ 1), __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) <= s) {}
    };
    auto compute = [&](int step, int buf, const u32x2 (&w)[BPS][TM]) {
        const unsigned char* recs = mine + buf * STEP_BYTES;
        const int valid = nrun - step * BPS;                 // blocks of this step that exist
        constexpr int STEPS = 3 * BPS * TN;
        u32x4 lo[3];
        u32x2 hi[3];
        uint32_t sc[2];
        auto read_step = [&](int st) {
            const unsigned char* rec = recs + (st / 3) * FP6_REC_BYTES;
            const int pl = st % 3;
            lo[pl] = *reinterpret_cast<const u32x4*>(rec + pl * 1024 + lane * 16);
            hi[pl] = *reinterpret_cast<const u32x2*>(rec + 3072 + pl * 512 + lane * 8);
            if (pl == 0) sc[(st / 3) & 1] = *reinterpret_cast<const uint32_t*>(rec + 4608 + lane * 4);
        };
        read_step(0);
        read_step(1);
#pragma unroll
        for (int j = 0; j < BPS; ++j) {
            if (j >= valid) break;
            u32x4 av[TM];
#pragma unroll
            for (int a = 0; a < TM; ++a)
                av[a] = u32x4{(w[j][a].x << 2) & 0xCCCCCCCCu, w[j][a].x & 0xCCCCCCCCu, (w[j][a].y << 2) & 0xCCCCCCCCu, w[j][a].y & 0xCCCCCCCCu};
#pragma unroll
            for (int t = 0; t < 3 * TN; ++t) {
                const int st = j * 3 * TN + t;
                if (st + 2 < STEPS) read_step(st + 2);
                __builtin_amdgcn_sched_barrier(0);
                const int b = t / 3;
#pragma unroll
                for (int a = 0; a < TM; ++a) {
                    switch (t % 3) {
                        case 0: acc[a][b] = mfma_fp6<0>(av[a], lo[0], hi[0], sc[(st / 3) & 1], acc[a][b]); break;
                        case 1: acc[a][b] = mfma_fp6<1>(av[a], lo[1], hi[1], sc[(st / 3) & 1], acc[a][b]); break;
                        default: acc[a][b] = mfma_fp6<2>(av[a], lo[2], hi[2], sc[(st / 3) & 1], acc[a][b]); break;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    u32x2 wa[BPS][TM], wb[BPS][TM];
    load_w(min(from, nsteps - 1), wa);
    if (PLACED && !tile.exists) return;
    if (count > 0) issue(from, 0);
    split_touch(p);
    __syncthreads();                                         // (the words are zero)
    for (int s = 0; s < count; s += 2) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        touch(wa);
        meet(s);
        if (s + 1 < count) {
            load_w(from + s + 1, wb);
            issue(from + s + 1, 1);
        }
        compute(from + s, 0, wa);
        if (s + 1 < count) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            touch(wb);
            meet(s + 1);
            if (s + 2 < count) {
                load_w(from + s + 2, wa);
                issue(from + s + 2, 0);
            }
            compute(from + s + 1, 1, wb);
        }
    }
    __syncthreads();

    // ---- the pairs' partial sums: result block f = 8 tile + row block; pair q finishes blocks q NF .. + NF - 1
    f32x4 fin[NF];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
        if (q == kg) {
#pragma unroll
            for (int f = 0; f < NF; ++f) fin[f] = acc[(q * NF + f) & 7][(q * NF + f) >> 3];
        }
#pragma unroll
    for (int f0 = 0; f0 < NF; f0 += NFR) {
        auto slot = [&](int q, int other, int f) { return smem + ((((q * (KG - 1) + other) * RW + rw) * NFR + f) * 64 + lane) * 16; };
        if (f0 > 0) __syncthreads();
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            if (q != kg) {
                const int other = kg < q ? kg : kg - 1;
#pragma unroll
                for (int f = 0; f < NFR; ++f)
                    *reinterpret_cast<f32x4*>(slot(q, other, f)) = acc[(q * NF + f0 + f) & 7][(q * NF + f0 + f) >> 3];
            }
        __syncthreads();
        if (kg < NQ) {
#pragma unroll
            for (int other = 0; other < KG - 1; ++other)
#pragma unroll
                for (int f = 0; f < NFR; ++f) fin[f0 + f] += *reinterpret_cast<const f32x4*>(slot(kg, other, f));
        }
    }
    if (kg >= NQ) return;
    if constexpr (DIRECT) {
        finish_z(p, fin, strip0 >> 3, b0 + 16 * kg, lane);
    } else {
        f32x4 out[NF][1];
#pragma unroll
        for (int f = 0; f < NF; ++f) out[f][0] = fin[f];
        gemm_epilogue<NF, 1, true, EX>(p, out, strip0 + ((kg * NF) & 7), b0, 16 * ((kg * NF) >> 3), ones, i, g);
    }
}

// ---- tiles of 128 rows: a block of the contraction for a wavefront ----------------------------------
// With one group of rows no wavefront reads what another one uses, so nothing is staged and no barrier stands in the loop: wavefront w takes the blocks
// w, w + 8, ..., its operands (planes of a record, 24 bytes a lane and plane, in the order of the record) go from the L2s to registers, DEPTH blocks
// ahead, and stage V makes the planes of x in registers where it makes them itself (X; every row tile makes them again.  Feature-major bf16 passes through 4 KiB
// of LDS of the wavefront there, where the sums meet later: a barrier behind the loop).  The partial sums of the eight wavefronts meet in LDS.
// Measured on MI355X against the same tiles on records staged in LDS (a step of 16 records for every barrier; in a launch of two or three steps each one
// waited a round trip of about 1 us for the next): 3072 x 768 x 1536 fp32 at 197 tokens 20.4 -> 18.1 us, 256 x 489 x 256 fp32 at 256 13.2 -> 9.6,
// 7415 x 4199 x 4465 bf16 at 125 32.3 -> 27.5; 40 drawn fp32 and 60 bf16 calls of 30 to 2500 tokens that take these tiles 0.73 to 1.0 of the time.
template <int TN, bool STAGE2, int EX, int X, bool PLACED>
__global__ void __launch_bounds__(512, 1)
tsvd_fp6_own_kernel(SPLIT_ARGUMENTS) {
    const gemm_args p = SPLIT_STRUCT;
    const split_x xs = split_x_of(p_act, p_act_bytes, p_extra0, p_extra1, p_extra2);
    const split_tile tile = tile_of<PLACED>(split_place_of(p_extra0, p_extra1));
    constexpr int KG = 8, TM = 8, DEPTH = TN == 1 ? 3 : 2;
    constexpr bool DIRECT = !STAGE2;
    constexpr int NQ = DIRECT ? TN : KG, NF = 8 * TN / NQ;
    extern __shared__ __align__(16) unsigned char smem[];    // the partial sums, 16 TN ones behind them
    float* ones = reinterpret_cast<float*>(smem + NQ * (KG - 1) * NF * 1024);
    const int lane = threadIdx.x & 63, kg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = lane & 15, g = lane >> 4;
    const int b0 = tile.token * 16 * TN, strip0 = tile.row * TM, nrun = X == 2 ? p.npairs / 2 : p.npairs;      // (X: both sets of planes at a block)
    if (threadIdx.x < 16 * TN) ones[threadIdx.x] = 1.0f;
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(p.tiles), 0, p.tile_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t act_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(static_cast<const void*>(p.act)), 0, p.act_bytes, 0x00020000);

    f32x4 acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    // (rows of stage V as in tsvd_fp6_panel_kernel)
    const int gg = i >> 2, vv = i & 3;
    const int w_voff = DIRECT ? (4 * (gg & 1) + (gg >> 1)) * p.nkt * 1024 + (g * 16 + vv) * 16 : lane * 16;
    // (arrays of their own: the planes of a structure would be read as parts of longer vectors, and kept in scratch memory)
    constexpr int SLOTS = X ? 1 : DEPTH * TN;
    u32x4 lo[SLOTS][3];
    u32x2 hi[SLOTS][3];
    uint32_t sc[SLOTS];
    auto load_w = [&](int blk, u32x2 (&w)[TM]) {
        if (p.code_blocks && blk >= p.code_blocks) blk -= p.code_blocks;          // (second set of planes: the same codes again)
        const int soff = (strip0 * p.nkt + (blk >> 1)) * 1024 + (blk & 1) * 8;
#pragma unroll
        for (int a = 0; a < TM; ++a)
            w[a] = __builtin_amdgcn_raw_buffer_load_b64(w_rsrc, w_voff, soff + (DIRECT ? 2 * (a >> 2) * p.nkt * 1024 + 4 * (a & 3) * 16 : a * p.nkt * 1024), 0);
    };
    auto load_b = [&](int blk, auto d_c) {
        const int soff = ((b0 >> 7) * p.plane_blocks + blk) * FP6_PAIR_BYTES + ((b0 & 127) >> 4) * FP6_REC_BYTES;
#pragma unroll
        for (int b = 0; b < TN; ++b) {
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) {
                lo[decltype(d_c)::value * TN + b][pl] = buf_load128(act_rsrc, lane * 16, soff + b * FP6_REC_BYTES + pl * 1024);
                hi[decltype(d_c)::value * TN + b][pl] = __builtin_amdgcn_raw_buffer_load_b64(act_rsrc, lane * 8, soff + b * FP6_REC_BYTES + 3072 + pl * 512, 0);
            }
            sc[decltype(d_c)::value * TN + b] = __builtin_amdgcn_raw_buffer_load_b32(act_rsrc, lane * 4, soff + b * FP6_REC_BYTES + 4608, 0);
        }
    };
    auto operand_a = [&](const u32x2 (&w)[TM], u32x4 (&av)[TM]) {
#pragma unroll
        for (int a = 0; a < TM; ++a) av[a] = u32x4{(w[a].x << 2) & 0xCCCCCCCCu, w[a].x & 0xCCCCCCCCu, (w[a].y << 2) & 0xCCCCCCCCu, w[a].y & 0xCCCCCCCCu};
    };
    auto multiply = [&](const u32x4 (&av)[TM], int b, auto slot_c) {
        constexpr int n = decltype(slot_c)::value;
#pragma unroll
        for (int a = 0; a < TM; ++a) acc[a][b] = mfma_fp6<0>(av[a], lo[n][0], hi[n][0], sc[n], acc[a][b]);
#pragma unroll
        for (int a = 0; a < TM; ++a) acc[a][b] = mfma_fp6<1>(av[a], lo[n][1], hi[n][1], sc[n], acc[a][b]);
#pragma unroll
        for (int a = 0; a < TM; ++a) acc[a][b] = mfma_fp6<2>(av[a], lo[n][2], hi[n][2], sc[n], acc[a][b]);
    };
    if constexpr (X != 0) {
        for (int blk = kg; blk < nrun; blk += KG) {
            u32x2 w[TM];
            load_w(blk, w);
#pragma unroll
            for (int b = 0; b < TN; ++b) {
                float v[32];
                gather_x<X == 2>(xs.x, xs.ld, xs.token_major != 0, xs.N, p.bvalid, blk, (b0 >> 4) + b, lane, v, smem + kg * 4096);
                auto put = [&](int pl, u32x4 l, u32x2 h) { lo[0][pl] = l, hi[0][pl] = h; };
                const std::integral_constant<int, 0> slot{};
                sc[0] = tsvd_planes_of_32<X == 2>(v, put);
                {
                    u32x4 av[TM];
                    operand_a(w, av);
                    multiply(av, b, slot);
                }
                if constexpr (X == 2) {
                    sc[0] = tsvd_planes_of_32<false>(v, put);
                    u32x4 av[TM];
                    operand_a(w, av);
                    multiply(av, b, slot);
                }
            }
        }
    } else {
        u32x2 w[DEPTH][TM];
        auto ask = [&](int blk, auto d_c) {
            if (blk < nrun) {
                load_b(blk, d_c);
                load_w(blk, w[decltype(d_c)::value]);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto block = [&](int blk, auto d_c) {
            constexpr int d = decltype(d_c)::value;
            if (blk < nrun) {
                u32x4 av[TM];
                operand_a(w[d], av);
                multiply(av, 0, std::integral_constant<int, d * TN>{});
                if constexpr (TN == 2) multiply(av, 1, std::integral_constant<int, d * TN + 1>{});
                __builtin_amdgcn_sched_barrier(0);
                ask(blk + KG * DEPTH, d_c);
            }
        };
        const std::integral_constant<int, 0> d0{};
        const std::integral_constant<int, 1> d1{};
        const std::integral_constant<int, DEPTH - 1> d2{};
        ask(kg, d0);
        ask(kg + KG, d1);
        if constexpr (DEPTH == 3) ask(kg + 2 * KG, d2);
        split_touch(p);
        if (PLACED && !tile.exists) return;
        for (int blk = kg; blk < nrun; blk += KG * DEPTH) {
            block(blk, d0);
            block(blk + KG, d1);
            if constexpr (DEPTH == 3) block(blk + 2 * KG, d2);
        }
    }

    if (X == 1 && !xs.token_major) __syncthreads();           // (x passed through where the sums meet)

    // ---- the partial sums: result block f = 8 tile + row block; wavefront q finishes blocks q NF .. + NF - 1
    f32x4 fin[NF];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
        if (q == kg) {
#pragma unroll
            for (int f = 0; f < NF; ++f) fin[f] = acc[(q * NF + f) & 7][(q * NF + f) >> 3];
        }
    auto slot = [&](int q, int from, int f) { return smem + (((q * (KG - 1) + from) * NF + f) * 64 + lane) * 16; };
#pragma unroll
    for (int q = 0; q < NQ; ++q)
        if (q != kg) {
            const int from = kg < q ? kg : kg - 1;
#pragma unroll
            for (int f = 0; f < NF; ++f) *reinterpret_cast<f32x4*>(slot(q, from, f)) = acc[(q * NF + f) & 7][(q * NF + f) >> 3];
        }
    __syncthreads();
    if (kg >= NQ) return;
#pragma unroll
    for (int from = 0; from < KG - 1; ++from)
#pragma unroll
        for (int f = 0; f < NF; ++f) fin[f] += *reinterpret_cast<const f32x4*>(slot(kg, from, f));
    if constexpr (DIRECT) {
        finish_z(p, fin, strip0 >> 3, b0 + 16 * kg, lane);
    } else {
        f32x4 out[NF][1];
#pragma unroll
        for (int f = 0; f < NF; ++f) out[f][0] = fin[f];
        gemm_epilogue<NF, 1, true, EX>(p, out, strip0 + ((kg * NF) & 7), b0, 16 * ((kg * NF) >> 3), ones, i, g);
    }
}

// One group of rows leaves each wavefront its own records, two share them in LDS, and so do the wavefronts that make those of two token tiles (both in
// turn in registers: 9664 x 941 x 611 at 861 tokens 31.6 -> 34.4 us).
template <int RW, int TN, int X>
constexpr bool own = RW == 1 && (TN == 1 || X == 0);
template <int RW, int TN, bool STAGE2, int EX, int X = 0, bool PLACED = false>
auto kernel() {
    if constexpr (own<RW, TN, X>) return tsvd_fp6_own_kernel<TN, STAGE2, EX, X, PLACED>;
    else if constexpr (X == 0) return tsvd_fp6_pair_kernel<TN, STAGE2, EX, PLACED>;
    else return tsvd_fp6_panel_kernel<RW, TN, X>;
}
template <int RW, int TN, int X>
constexpr int split_lds = (own<RW, TN, X> ? 7 * 8 * TN * 1024 : 2 * 16 * FP6_REC_BYTES + (X == 0 ? 32 : 0)) + 16 * TN * 4;

template <int RW, int TN, bool STAGE2, int EX, int X = 0>
hipError_t init_one() {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel<RW, TN, STAGE2, EX, X>()), hipFuncAttributeMaxDynamicSharedMemorySize, split_lds<RW, TN, X>);
    if (e != hipSuccess || X != 0) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel<RW, TN, STAGE2, EX, 0, true>()), hipFuncAttributeMaxDynamicSharedMemorySize, split_lds<RW, TN, 0>);
}
template <int RW, int TN>
hipError_t init_shape() {
    hipError_t e;
    if ((e = init_one<RW, TN, false, 0>()) != hipSuccess) return e;
    if ((e = init_one<RW, TN, false, 0, 1>()) != hipSuccess) return e;
    if ((e = init_one<RW, TN, false, 0, 2>()) != hipSuccess) return e;
    if ((e = init_one<RW, TN, true, 0>()) != hipSuccess) return e;
    if ((e = init_one<RW, TN, true, 1>()) != hipSuccess) return e;
    if ((e = init_one<RW, TN, true, 2>()) != hipSuccess) return e;
    return init_one<RW, TN, true, 3>();
}
// The groups that leave an XCD the fewest bytes, for launches of one round of workgroups.  Tiles in turn where they are about as good: an XCD then sees one in
// gcd(token tiles, 8) of the token tiles, and (token tiles) / 8 of the row tiles.  16384 x 4096 x 8192 at 256 tokens (an XCD's codes of stage U 16.8 -> 4.2 MB, planes
// 1.3 -> 5; of stage V 8.4 -> 2.1 MB, planes 0.3 -> 1.2) 73.5 -> 68.7 us, 3072 x 768 x 1536 fp32 at 197 18.1 -> 17.1, 275 x 1257 x 597 fp32 at 418 19.7 -> 17.3;
// on 66 drawn calls 0.88 to 1.0 of the time (one 1.03).  Launches of several rounds: 0.97 to 1.04, 1.01 on the average.  A saving below half a megabyte: nothing.
bool place_of(int shape, const split_sizes& s, split_place* p, dim3* grid) {
    const long long rows_tile = shape / 8 * 128, tokens_tile = (shape & 7) * 16;
    const long long row_tiles = (s.rows + rows_tile - 1) / rows_tile, token_tiles = (s.B + tokens_tile - 1) / tokens_tile;
    // (bytes of what the launch reads: 2 bits a code, a record of 4864 bytes for 16 tokens and 128 indices)
    const double code_bytes = (double)s.rows * 32.0 * s.code_blocks, act_bytes = (double)s.blocks * ((s.B + 15) / 16) * FP6_REC_BYTES;
    *grid = dim3((unsigned)token_tiles, (unsigned)row_tiles);
    if (row_tiles * token_tiles > s.cus) return false;
    int d = 8;
    while (token_tiles % d) d /= 2;
    const double plain = code_bytes * std::min(1.0, (double)token_tiles / 8) + act_bytes / d;
    double best = std::min(0.9 * plain, plain - 512e3);
    bool found = false;
    for (int log2 = 0; log2 <= 3; ++log2) {
        const long long rows = (row_tiles + (1 << log2) - 1) >> log2, groups = 8 >> log2, tiles = (token_tiles + groups - 1) / groups;
        const double bytes = code_bytes / (1 << log2) + act_bytes / (double)groups;
        if (rows * tiles > s.cus / 8 || bytes >= best) continue;
        best = bytes;
        found = true;
        *p = {log2, (int)row_tiles, (int)token_tiles, (int)tiles, (int)rows};
        *grid = dim3(8, (unsigned)tiles, (unsigned)rows);
    }
    return found;
}
template <int RW, int TN>
hipError_t launch_shape(bool stage2, const gemm_args& a, int ex, const split_x* x, bool f32, long long cus, hipStream_t stream) {
    dim3 grid((unsigned)((a.bvalid + 16 * TN - 1) / (16 * TN)), (unsigned)((a.rows_need + RW * 128 - 1) / (RW * 128)));
    const dim3 block(512);
#define SPLIT_LAUNCH(STAGE2, EX, X, PLACED)                                                                                                                                                  \
    hipLaunchKernelGGL((kernel<RW, TN, STAGE2, EX, X, PLACED>()), grid, block, (split_lds<RW, TN, X>), stream, a.tiles, X ? x->x : static_cast<const void*>(a.act), a.tile_bytes, \
                       X ? (unsigned)x->N : a.act_bytes, a.nkt, a.npairs, a.code_blocks, a.plane_blocks, a.bvalid, extra[0], extra[1], extra[2], a)
#define SPLIT_STAGE(PLACED)                                  \
    do {                                                     \
        if (!stage2) SPLIT_LAUNCH(false, 0, 0, PLACED);      \
        else if (ex == 3) SPLIT_LAUNCH(true, 3, 0, PLACED);  \
        else if (ex == 2) SPLIT_LAUNCH(true, 2, 0, PLACED);  \
        else if (ex == 1) SPLIT_LAUNCH(true, 1, 0, PLACED);  \
        else SPLIT_LAUNCH(true, 0, 0, PLACED);               \
    } while (0)
    split_place place;
    unsigned extra[3] = {0, 0, 0};
    if (!stage2 && x) {
        extra[0] = (unsigned)x->ld, extra[1] = (unsigned)((unsigned long long)x->ld >> 32), extra[2] = (unsigned)x->token_major;
        if (f32) SPLIT_LAUNCH(false, 0, 2, false);
        else SPLIT_LAUNCH(false, 0, 1, false);
    } else if (place_of(8 * RW + TN, {a.rows_need, a.bvalid, a.npairs, a.code_blocks ? a.code_blocks : a.npairs, cus}, &place, &grid)) {
        extra[0] = (unsigned)place.row_tiles | (unsigned)place.token_tiles << 16;
        extra[1] = (unsigned)place.row_log2 | (unsigned)place.group_tiles << 2 | (unsigned)place.group_rows << 17;
        SPLIT_STAGE(true);
    } else {
        SPLIT_STAGE(false);
    }
#undef SPLIT_STAGE
#undef SPLIT_LAUNCH
    return hipGetLastError();
}

}  // namespace

hipError_t tsvd_fp6_split_init() {
    hipError_t e;
    if ((e = init_shape<2, 4>()) != hipSuccess) return e;
    if ((e = init_shape<2, 2>()) != hipSuccess) return e;
    if ((e = init_shape<1, 2>()) != hipSuccess) return e;
    return init_shape<1, 1>();
}

// shape: rows / 128 of a tile * 8 + token tiles of 16
static hipError_t launch_any(int shape, bool stage2, const gemm_args& a, int ex, const split_x* x, bool f32, long long cus, hipStream_t stream) {
    switch (shape) {
        case 20: return launch_shape<2, 4>(stage2, a, ex, x, f32, cus, stream);
        case 18: return launch_shape<2, 2>(stage2, a, ex, x, f32, cus, stream);
        case 10: return launch_shape<1, 2>(stage2, a, ex, x, f32, cus, stream);
        case 9: return launch_shape<1, 1>(stage2, a, ex, x, f32, cus, stream);
        default: return hipErrorInvalidValue;
    }
}
hipError_t tsvd_fp6_split_launch(int shape, bool stage2, const gemm_args& a, int ex, long long cus, hipStream_t stream) {
    return launch_any(shape, stage2, a, ex, nullptr, false, cus, stream);
}
bool tsvd_fp6_split_placed(int shape, const split_sizes& s) {
    split_place place;
    dim3 grid;
    return place_of(shape, s, &place, &grid);
}
// Two steps of 16 records hold all of x of a token tile.
bool tsvd_fp6_split_makes_x(int shape, int blocks) { return shape != 0 && blocks * (shape & 7) <= 32; }
hipError_t tsvd_fp6_split_launch_x(int shape, const gemm_args& a, const void* x, bool f32, bool token_major, long long ld, int N, hipStream_t stream) {
    if (!f32 && !token_major && (N - 1) * ld + a.bvalid < 8) return hipErrorInvalidValue;
    const split_x xs = {x, ld, token_major, N};
    return launch_any(shape, false, a, 0, &xs, f32, 0, stream);
}

hipError_t tsvd_fp6_split_planes(const void* x, bool f32, bool token_major, long long ld, int N, int B, int blocks, unsigned char* planes,
                                 hipStream_t stream) {
    if (!f32 && !token_major && (N - 1) * ld + B < 8) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((B + 63) / 64), (unsigned)blocks), block(256);
    if (f32) hipLaunchKernelGGL(tsvd_planes_kernel<true>, grid, block, 0, stream, x, ld, (int)token_major, N, B, blocks, planes);
    else hipLaunchKernelGGL(tsvd_planes_kernel<false>, grid, block, 0, stream, x, ld, (int)token_major, N, B, blocks, planes);
    return hipGetLastError();
}
