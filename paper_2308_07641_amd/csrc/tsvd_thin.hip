// Both stages of a batch in one launch: Y = U (S (V X)) for 16 or 32 tokens per workgroup, on fp4 codes x fp6 planes.
//
// The token-panel kernel of tsvd_fp6.hip gives a workgroup 64 tokens and holds x and then z in LDS, which bounds N and K by 1024
// and needs some 10000 tokens to reach most compute units.  A panel of 16 (32) tokens needs a quarter (half) of both: K + N of
// thousands fit, and 200 panels are 3200 tokens.  Against separate stages it saves the operand pass, the round trip of z, two launches
// with their ramps, and the stores of y run while other units multiply (a stage whose tiles all end together pays for
// them on top: 10 of 54 us on a 16384 x 8192 stage of 256 tokens).  Every workgroup streams all code words, so
// they have to stay in the L2s.
//
// Eight wavefronts.  Planes of x are made block by block (a wavefront per record: gather, convert); wavefront w multiplies the
// rank blocks w, w + 8, ... of stage V (128 rows x the panel; its result lanes are stage U's operand lanes, see tsvd_panel_fp6_kernel)
// and writes their planes of z beside those of x; then stage U runs in units of 16 UTM rows, no barrier between them.
// Where stage V's rank blocks do not go round, wavefronts share some: each a part of the contraction, sums added in LDS (3 x 3 from 310 channels, rank 119, two images of 28 x 28: 18.8 -> 14.2 us;
// 5 x 5 from 198, rank 213, twelve of 28 x 28: 100 -> 88; 3456 x 7104 x 193, rows of tokens, at 2801 40.3 -> 35.6; 512 x 1536 x 1280, rows of tokens, at 13568 82.9 -> 79.1: each with arguments preloaded, 0.4 to 0.5 us).
// Where x does not fit beside z its blocks pass through in chunks, two in LDS: four of the wavefronts multiply the one before
// they make their records of the next, the other four after, so that on every SIMD matrix and vector instructions overlap.
// Code words go from the L2s to registers, one fetch ahead across rank blocks and units (those of the next unit are in
// before a unit's stores are issued: loads and stores share one counter); a fetch is 16 bytes per lane and strip, the words of
// 256 contraction indices.
// A convolution's columns are gathered straight from the images: a table of offsets per index in LDS, and per token a bit
// mask of the taps that fall outside its image.  Rows of three taps come as one load of four elements each, six for sixteen indices, with a table and a mask of rows: the
// address unit's requests bound the gather (3 x 3: 256 x 2304 x 116 at 14896 positions 52.4 -> 42.6 us, 89 x 1683 x 78 at 3920 19.1 -> 14.8, 128 x 621 x 412 at 27440
// 56.8 -> 46.7; 60 drawn convolutions, 25 of them with such rows, 0.946 of the time).
// Measured on MI355X: 3072 x 768 x 1545 bf16 at 3152 tokens, token-major: 71.5 -> 39.2 us (ring kernels with a copy of x before; 16 tokens per panel); the
// map of a 3 x 3 convolution, 256 x 2304 x 768 at 6272 positions: 75.5 -> 34.3 us (columns written and read before; 32).
// What bounds them: the matrix instructions of the panels' last round, and the code words that every workgroup pulls from its L2.  By
// counters the matrix pipes are busy 0.43 of the compute units' cycles in the first and 0.28 in the second (which has 196 panels, and six rank blocks
// in stage V for eight wavefronts).
#include "../../include/tsvd_tuning.h"
#include "tsvd_thin.h"

#include <algorithm>
#include <type_traits>

#include "tsvd_fp6_common.h"

namespace {

struct thin_args {
    const uint32_t *tiles_v, *tiles_u;
    unsigned tile_v_bytes, tile_u_bytes;
    int nkt_v, nkt_u, nvb, nub;              // tiles of 256 per strip; 128-index blocks of N and K that hold anything
    const uint16_t* x;
    unsigned x_bytes;                        // below 2^31
    int N, B, chunk, buffers;        // blocks of x per chunk, chunks in LDS (1: all of x, or 2)
    unsigned char whole, shared, parts;      // SHARED: of stage V's last rank blocks the first `whole` a wavefront each, `shared` more 1 << parts wavefronts each (thin_shares)
    long long ldx;
    int images, H, W, kv1, kv2, Hv, Wv, s1, s2, p1, p2, d1, d2;
    const float* S;
    void* y;
    long long ldy;
    const float* bias;
    int M, out_bf16, token_major, utm;       // utm: 16-row blocks per unit of stage U
    int runs;                                // neighbouring panels on one XCD
    int slices;                              // workgroups of a panel, each with the whole z and its part of y's rows
};
// They are passed so that the fourteen words which come preloaded in registers are what stage V needs: a load from the others takes 0.3 us, and everything waits
// for it (742 x 106 x 103 at 29 tokens 5.3 -> 4.8 us, 388 x 120 x 256 at 33 5.45 -> 4.95, 359 x 100 x 81 at 1569 5.7 -> 5.2; 3072 x 768 x 1545 at 3152, 39 us, as before).
struct thin_rest {
    void* y;
    long long ldy;
    const float* bias;
    int M;
};
struct thin_images {
    int images, H, W, kv1, kv2, Hv, Wv, s1, s2, p1, p2, d1, d2;
};
unsigned thin_form(const thin_args& a) {
    return (unsigned)a.chunk | (unsigned)(a.buffers - 1) << 6 | (unsigned)a.nub << 7 | (unsigned)a.whole << 12 | (unsigned)a.shared << 15 | (unsigned)a.parts << 19 | (unsigned)a.runs << 21 |
           (unsigned)a.utm << 22 | (a.out_bf16 ? 1u << 26 : 0u) | (a.token_major ? 1u << 27 : 0u);
}
__device__ __forceinline__ thin_args thin_arguments(const uint16_t* x, const uint32_t* tiles_v, const uint32_t* tiles_u, const float* S, unsigned x_bytes, int N, int B, int ldx, unsigned form,
                                                    int slices, const thin_rest& r, const thin_images& c) {
    thin_args p;
    p.x = x, p.tiles_v = tiles_v, p.tiles_u = tiles_u, p.S = S, p.x_bytes = x_bytes, p.N = N, p.B = B, p.ldx = ldx, p.slices = slices;
    p.chunk = form & 63, p.buffers = 1 + (form >> 6 & 1), p.nub = form >> 7 & 31, p.whole = form >> 12 & 7, p.shared = form >> 15 & 15, p.parts = form >> 19 & 3, p.runs = form >> 21 & 1;
    p.utm = form >> 22 & 15, p.out_bf16 = form >> 26 & 1, p.token_major = form >> 27 & 1;
    p.nvb = (N + 127) >> 7, p.nkt_v = (N + 255) >> 8, p.nkt_u = (p.nub + 1) >> 1;
    p.tile_v_bytes = (unsigned)p.nkt_u * (unsigned)p.nkt_v << 14, p.tile_u_bytes = (unsigned)((r.M + 255) >> 8) * (unsigned)p.nkt_u << 14;
    p.y = r.y, p.ldy = r.ldy, p.bias = r.bias, p.M = r.M;
    p.images = c.images, p.H = c.H, p.W = c.W, p.kv1 = c.kv1, p.kv2 = c.kv2, p.Hv = c.Hv, p.Wv = c.Wv, p.s1 = c.s1, p.s2 = c.s2, p.p1 = c.p1, p.p2 = c.p2, p.d1 = c.d1, p.d2 = c.d2;
    return p;
}

// bytes of LDS for records of x, and then for the sums of the wavefronts that share a block
__host__ __device__ inline int thin_x_bytes(const thin_args& p, int tiles, bool shared) {
    const int records = p.buffers * p.chunk * tiles * FP6_REC_BYTES, sums = shared ? p.shared * ((1 << p.parts) - 1) * tiles * 8192 : 0;
    return records > sums ? records : sums;
}

// THIN_CONV whose V takes rows of three taps side by side, of images of four columns and more: a row is one load of four elements.
constexpr int THIN_CONV_ROWS = 3;

template <int TN, int RB, int SOURCE, bool CHUNKED, bool SHARED>
__global__ void __launch_bounds__(512, 2)
tsvd_thin_panel_kernel(const uint16_t* p_x, const uint32_t* p_tiles_v, const uint32_t* p_tiles_u, const float* p_S, unsigned p_x_bytes, int p_N, int p_B, int p_ldx, unsigned p_form, int p_slices,
                       thin_rest p_rest, thin_images p_images) {
    const thin_args p = thin_arguments(p_x, p_tiles_v, p_tiles_u, p_S, p_x_bytes, p_N, p_B, p_ldx, p_form, p_slices, p_rest, p_images);
    constexpr int NW = 8;
    using words = u32x4;
    extern __shared__ __align__(16) unsigned char smem[];    // records [block][tile]: chunk blocks of x, then nub blocks of z
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = lane & 15, g = lane >> 4;
    // workgroups go to the eight XCDs in turn; with p.runs each XCD takes a run of neighbouring panels, so that the lines that
    // panels share (32 or 64 bytes of a feature-major row each) are fetched into one L2
    // (the workgroups of a panel lie a round of panels apart.  As a second dimension of the grid they cost launches without any 0.1 us: 512 x 128 x 97, rows of
    // tokens, at 4166 8.82 -> 8.91, now 8.71)
    const int panels = (p.B + 16 * TN - 1) / (16 * TN), slice = p.slices > 1 ? (int)blockIdx.x / panels : 0, panel = blockIdx.x - slice * panels;
    const int xcd = panel & 7, per = panels >> 3, more = panels & 7;
    const int b0 = (p.runs ? xcd * per + min(xcd, more) + (panel >> 3) : panel) * 16 * TN;
    unsigned char* xrec = smem;
    unsigned char* zrec = smem + thin_x_bytes(p, TN, SHARED);
    const int* ktab = reinterpret_cast<const int*>(zrec + p.nub * TN * FP6_REC_BYTES);   // THIN_CONV: byte offset of index k in the images
    const __amdgpu_buffer_rsrc_t v_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(p.tiles_v), 0, p.tile_v_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t u_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(p.tiles_u), 0, p.tile_u_bytes, 0x00020000);

    // ---- the record of (block, tile) of x, by one wavefront.  What does not exist (indices beyond N, taps outside the image) is
    // read at an offset beyond the buffer, where loads give zero; tokens beyond the batch repeat the last one (never stored)
    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.x), 0, p.x_bytes, 0x00020000);
    int conv_base = 0;                       // THIN_CONV: byte offset of this lane's token (its tile is the wavefront's), and the taps (rows of taps) outside
    uint64_t conv_outside = 0;               // its image as a bit mask, repeated with the period of the taps (of the rows)
    int conv_right = 0, conv_left = 0;       // THIN_CONV_ROWS: bits by which what a load of a row begins with lies before the first tap, and behind it
    if constexpr (SOURCE == THIN_CONV) {
        const int taps = p.kv1 * p.kv2, channel = p.images * p.H * p.W;
        for (int k = threadIdx.x; k < 128 * p.nvb; k += 512) {
            const int t = k / p.kv2, dx = k - t * p.kv2, ci = t / p.kv1, dy = t - ci * p.kv1;
            const_cast<int*>(ktab)[k] = k < p.N ? 2 * (ci * channel + dy * p.d1 * p.W + dx * p.d2) : (int)0x80000000;
        }
        const int tok = min(b0 + 16 * (wave % TN) + i, p.B - 1), plane = p.Hv * p.Wv, img = tok / plane, at = tok - img * plane, py = at / p.Wv,
                  px = at - py * p.Wv, y0 = py * p.s1 - p.p1, x0 = px * p.s2 - p.p2;
        conv_base = 2 * (img * p.H * p.W + y0 * p.W + x0);
        for (int dy = 0; dy < p.kv1; ++dy)
            for (int dx = 0; dx < p.kv2; ++dx)
                if ((unsigned)(y0 + dy * p.d1) >= (unsigned)p.H || (unsigned)(x0 + dx * p.d2) >= (unsigned)p.W)
                    for (int b = dy * p.kv2 + dx; b < 64; b += taps) conv_outside |= 1ull << b;
        __syncthreads();
    }
    if constexpr (SOURCE == THIN_CONV_ROWS) {
        const int channel = p.images * p.H * p.W;
        for (int r = threadIdx.x; r < 128 * p.nvb / 3 + 2; r += 512) {
            const int ci = r / p.kv1, dy = r - ci * p.kv1;
            const_cast<int*>(ktab)[r] = 3 * r < p.N ? 2 * (ci * channel + dy * p.d1 * p.W) : (int)0x80000000;
        }
        const int tok = min(b0 + 16 * (wave % TN) + i, p.B - 1), plane = p.Hv * p.Wv, img = tok / plane, at = tok - img * plane, py = at / p.Wv,
                  px = at - py * p.Wv, y0 = py * p.s1 - p.p1, x0 = px * p.s2 - p.p2, from = max(0, min(x0, p.W - 4)), by = x0 - from;
        conv_base = 2 * (img * p.H * p.W + y0 * p.W + from);
        conv_right = 16 * max(0, min(by, 3));
        conv_left = 16 * max(0, min(-by, 3));
        for (int dy = 0; dy < p.kv1; ++dy)
            if ((unsigned)(y0 + dy * p.d1) >= (unsigned)p.H || by > 3 || by < -3)
                for (int b = dy; b < 64; b += p.kv1) conv_outside |= 1ull << b;
        __syncthreads();
    }
    auto make_record = [&](int block, int tile, unsigned char* rec) __attribute__((always_inline)) {
        int tok = min(b0 + 16 * tile + i, p.B - 1);
        const int k0 = block * 128 + 64 * (g & 1) + 16 * (g >> 1);
        asm volatile("" : "+v"(tok));                                // (what follows from it is formed here, not kept in registers over the MFMAs)
        float v[32];
        uint16_t raw[32];
        auto gather = [&](int e, int off) {
            raw[e] = __builtin_amdgcn_raw_buffer_load_b16(x_rsrc, off, 0, 0);
            if (e % 8 == 7) __builtin_amdgcn_sched_barrier(0);      // (the offsets of all 32 at once would not fit the registers)
        };
        if constexpr (SOURCE == THIN_CONV_ROWS) {
            // the rows of three that sixteen indices from k on lie in, six of them
            u32x2 rows[2][6];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int r = (k0 + 32 * h) / 3;
                const uint32_t out = (uint32_t)(conv_outside >> (r % p.kv1));
#pragma unroll
                for (int j = 0; j < 6; ++j)
                    rows[h][j] = __builtin_amdgcn_raw_buffer_load_b64(x_rsrc, (ktab[r + j] + conv_base) | (int)((out << (31 - j)) & 0x80000000u), 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t s[9];                                       // eighteen values, two in a word
#pragma unroll
                for (int j = 0; j < 6; ++j) {                        // (shifts bring zeros in where taps lie beside the image)
                    rows[h][j] = __builtin_bit_cast(u32x2, __builtin_bit_cast(uint64_t, rows[h][j]) >> conv_right << conv_left);
                    if (j % 2) {
                        const u32x2 a = rows[h][j - 1], b = rows[h][j];
                        s[3 * (j / 2)] = a.x;
                        s[3 * (j / 2) + 1] = __builtin_amdgcn_perm(b.x, a.y, 0x05040100u);
                        s[3 * (j / 2) + 2] = __builtin_amdgcn_alignbit(b.y, b.x, 16);
                    }
                }
                const int first = (k0 + 32 * h) % 3;
                const uint32_t half = first == 1 ? 16 : 0;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t two = __builtin_amdgcn_alignbit(s[e + 1], first == 2 ? s[e + 1] : s[e], half);
                    v[16 * h + 2 * e] = __uint_as_float(two << 16);
                    v[16 * h + 2 * e + 1] = __uint_as_float(two & 0xFFFF0000u);
                }
            }
        } else if constexpr (SOURCE == THIN_CONV) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int k = k0 + 32 * h, first = k % (p.kv1 * p.kv2);
                const uint32_t out = (uint32_t)(conv_outside >> first);         // bit e: index k + e lies outside the image
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const i32x4 off = *reinterpret_cast<const i32x4*>(ktab + k + 4 * c);
#pragma unroll
                    for (int e = 0; e < 4; ++e) gather(16 * h + 4 * c + e, (off[e] + conv_base) | (int)((out << (31 - 4 * c - e)) & 0x80000000u));
                }
            }
        } else if constexpr (SOURCE == THIN_TOKEN_MAJOR) {
            tsvd_gather_row(p.x + (size_t)tok * p.ldx, k0, p.N, block * 128 + 128 <= p.N, v);
        } else {
            // Rows at scalar offsets, those beyond N at the buffer's end: 587 x 99 x 82 at 29 tokens 5.4 -> 5.2 us against an address and a test for each value.
            // They are formed here: the compiler kept the products of all 32 rows in scalar registers over the whole kernel, of which it has 102, and spilled up to 94
            // of others in panels of several chunks (576 x 640 x 356 at 7947 tokens 15.8 -> 14.9 us, 2164 x 1579 x 428 at 9285 61.7 -> 60.5, 896 x 1203 x 913 at 6592 30.5 -> 29.9).
            // Chunks of eight tokens, transposed in LDS, as the split tiles read them, are of no use here since: 192 x 4961 x 82 at 7561 40.8 against 34.5 us, 384 x 1535 x 218 at 845 11.6
            // against 10.8; on 51 feature-major calls 0.98 of the time without, two of them longer (916 x 4224 x 448 at 589 19.1 -> 19.5, 233 x 5661 x 881 at 261 19.1 -> 19.3).
            int ld2 = 2 * (int)p.ldx;
            asm volatile("" : "+s"(ld2));
            const int lane_off = (64 * (g & 1) + 16 * (g >> 1)) * ld2 + 2 * tok;
#pragma unroll
            for (int e = 0; e < 32; ++e)
                raw[e] = __builtin_amdgcn_raw_buffer_load_b16(x_rsrc, lane_off, tsvd_buffer_offset((block * 128 + 32 * (e >> 4) + (e & 15)) * ld2, p.x_bytes), 0);
        }
        if constexpr (SOURCE == THIN_CONV || SOURCE == THIN_FEATURE_MAJOR) {
#pragma unroll
            for (int e = 0; e < 32; ++e) v[e] = __uint_as_float((uint32_t)raw[e] << 16);
        }
        tsvd_planes_of_32(v, rec, lane);
    };

    // ---- TM row blocks times blocks [0, count) of the records at recs.  w0: the next fetch of the stream of code words that
    // next(words) continues, on return the one after the last pair's.  The operand of MFMA step t + 2 (a plane of a
    // record, TM row blocks) is read before the MFMAs of step t.
    auto run = [&](auto tm_c, const unsigned char* recs, int count, auto& w0, auto next, auto& acc) {
        constexpr int TM = decltype(tm_c)::value, STEPS = 6 * TN;
        words w1[TM];
        u32x4 lo[3];
        u32x2 hi[3];
        uint32_t sc[2];
        const int last = count * TN - 1;
        auto read_step = [&](int pair, int st) {              // step st of the pair of blocks (3 per record)
            const unsigned char* rec = recs + min(pair * 2 * TN + st / 3, last) * FP6_REC_BYTES;
            const int pl = st % 3;
            lo[pl] = *reinterpret_cast<const u32x4*>(rec + pl * 1024 + lane * 16);
            hi[pl] = *reinterpret_cast<const u32x2*>(rec + 3072 + pl * 512 + lane * 8);
            if (pl == 0) sc[(st / 3) & 1] = *reinterpret_cast<const uint32_t*>(rec + 4608 + lane * 4);
        };
        auto half = [&](int pair, auto h_c, const words (&w)[TM]) {        // one block of a pair
            constexpr int h = decltype(h_c)::value, at = 2 * h;
            u32x4 av[TM];
#pragma unroll
            for (int a = 0; a < TM; ++a)
                av[a] = u32x4{(w[a][at] << 2) & 0xCCCCCCCCu, w[a][at] & 0xCCCCCCCCu, (w[a][at + 1] << 2) & 0xCCCCCCCCu, w[a][at + 1] & 0xCCCCCCCCu};
#pragma unroll
            for (int t = 0; t < 3 * TN; ++t) {
                const int st = 3 * TN * h + t, b = t / 3, nx = st + 2;
                read_step(pair + nx / STEPS, nx % STEPS);
                __builtin_amdgcn_sched_barrier(0);
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
        };
        const std::integral_constant<int, 0> first{};
        const std::integral_constant<int, 1> second{};
        const int fetches = (count + 1) / 2;
        read_step(0, 0);
        read_step(0, 1);
        for (int q = 0; q < fetches; q += 2) {
            next(w1);
            half(q, first, w0);
            if (2 * q + 1 < count) half(q, second, w0);
            if (q + 1 < fetches) {
                next(w0);
                half(q + 1, first, w1);
                if (2 * q + 3 < count) half(q + 1, second, w1);
            } else {
#pragma unroll
                for (int a = 0; a < TM; ++a) w0[a] = w1[a];
            }
        }
    };
    // 1-KiB tiles: a lane's 16 bytes are the words of two blocks
    auto fetch = [&](__amdgpu_buffer_rsrc_t r, int voff, int tile_bytes, int block) -> words {
        return buf_load128(r, voff, tile_bytes + (block >> 1) * 1024);
    };
    constexpr int PER = 2;                                    // blocks per fetch

    // ================= stage V =================
    {
        f32x4 acc[RB][8][TN];
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int a = 0; a < 8; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b) acc[r][a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int gg = i >> 2, vv = i & 3;
        const int voff = ((4 * (gg & 1) + (gg >> 1)) * p.nkt_v) * 1024 + (g * 16 + vv) * 16;
        // this wavefront's last rank block, and its part of the block's contraction
        const int mine = wave - p.whole;
        const bool helps = SHARED && mine >= 0;
        const int part = helps ? mine >> (p.shared - 1) : 0, last_rank = NW * (RB - 1) + (helps ? p.whole + (mine & (p.shared - 1)) : wave);
        const bool has_last = SHARED ? !helps || part >> p.parts == 0 : last_rank < p.nub;
        const int ranks_most = wave < p.nub ? (p.nub - 1 - wave) / NW + 1 : 0;
        int nc = 0, nr = 0, nb = 0, ranks = ranks_most, from = 0, to = 0;     // the next fetch: first block of the chunk, rank block, block of the chunk; rank blocks, and blocks of the last one's
        auto next = [&](words (&w)[8]) {
            const bool last = SHARED && (RB == 1 || nr == RB - 1);
            const int rank = last ? last_rank : wave + NW * nr;
#pragma unroll
            for (int a = 0; a < 8; ++a)
                w[a] = fetch(v_rsrc, voff, (8 * rank + 2 * (a >> 2)) * p.nkt_v * 1024 + 4 * (a & 3) * 16, nc + nb);
            if (nb + PER < (last ? to : min(p.chunk, p.nvb - nc))) nb += PER;
            else if (nr + 1 < ranks) {                        // (at the end: the last fetch again)
                ++nr;
                nb = SHARED && nr == RB - 1 ? from : 0;
            }
        };
        auto make = [&](int c0) __attribute__((always_inline)) {
            const int blocks = min(p.chunk, p.nvb - c0);
            unsigned char* rec = xrec + (c0 / p.chunk & (p.buffers - 1)) * p.chunk * TN * FP6_REC_BYTES;
            // Beside the multiplication of a chunk: wavefronts of fewer rank blocks first make as many records as take its time, a fifth of them, then all
            // in turn.  (Records of a convolution's single elements are bound by the address unit, whoever makes them: 315 -> 320 us with this on 228 x 12800 x 388.)
            constexpr int SIDES = NW / TN;
            const int side = wave / TN, tile = wave % TN, heavy = !SHARED ? p.nub % NW : p.whole ? p.whole : p.shared << p.parts;
            const int busy = (heavy + TN - 1 - tile) / TN, idle = SIDES - busy, part_of = SHARED ? blocks * TN >> p.parts : 0;
            const int spare = SHARED && !p.whole ? part_of : blocks * TN - part_of;      // by how much the others multiply less
            const int own = CHUNKED && SOURCE != THIN_CONV && c0 > 0 && busy > 0 && idle > 0 ? idle * min(spare / 5, blocks / idle) : 0;
            const int rest = own + (own ? SIDES - 1 - side : side);
            bool first = own > 0 && side >= busy;
            for (int q = first ? side - busy : rest; q < blocks;) {
                make_record(c0 + q, tile, rec + (q * TN + tile) * FP6_REC_BYTES);
                q += first ? idle : SIDES;
                if (first && q >= own) {
                    first = false;
                    q = rest;
                }
            }
        };
        make(0);
        __syncthreads();
        auto chunks = [&](auto make_first) __attribute__((always_inline)) {
            for (int c0 = 0; c0 < p.nvb; c0 += p.chunk) {
                const int blocks = min(p.chunk, p.nvb - c0);
                const bool more = CHUNKED && c0 + p.chunk < p.nvb;       // (x as a whole: no code for more)
                if (decltype(make_first)::value && more) make(c0 + p.chunk);
                const unsigned char* rec = xrec + (c0 / p.chunk & (p.buffers - 1)) * p.chunk * TN * FP6_REC_BYTES;
                words w0[8];                                  // (not kept over the making of records: the registers are needed there)
                nc = c0;
                nr = nb = 0;
                if (SHARED) to = blocks;
                if (SHARED) from = 0;
                if (helps) {                                  // (whole fetches, of two blocks each)
                    const int fetches = (blocks + PER - 1) / PER;
                    from = PER * (fetches * part >> p.parts);
                    to = min(blocks, PER * (fetches * (part + 1) >> p.parts));
                }
                if constexpr (SHARED) {
                    ranks = RB - 1 + (has_last && from < to ? 1 : 0);
                    if (RB == 1) nb = from;
                }
                if (ranks > 0) next(w0);
#pragma unroll
                for (int r = 0; r < RB; ++r)
                    if (r < ranks) {
                        if (SHARED && r == RB - 1) run(std::integral_constant<int, 8>{}, rec + from * TN * FP6_REC_BYTES, to - from, w0, next, acc[r]);
                        else run(std::integral_constant<int, 8>{}, rec, blocks, w0, next, acc[r]);
                    }
                if (!decltype(make_first)::value && more) make(c0 + p.chunk);
                if (more) __syncthreads();
            }
        };
        if (CHUNKED && wave >= NW / 2) chunks(std::true_type{});
        else chunks(std::false_type{});
        if constexpr (SHARED) {                               // the parts' sums meet where the records of x were
            __syncthreads();
            f32x4* sums = reinterpret_cast<f32x4*>(smem) + lane;
            if (has_last && part > 0) {
#pragma unroll
                for (int a = 0; a < 8; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b) sums[((mine - p.shared) * 8 * TN + a * TN + b) * 64] = acc[RB - 1][a][b];
            }
            __syncthreads();
            if (helps && part == 0) {
                for (int q = 0; q + 1 < 1 << p.parts; ++q)
#pragma unroll
                    for (int a = 0; a < 8; ++a)
#pragma unroll
                        for (int b = 0; b < TN; ++b) acc[RB - 1][a][b] += sums[((mine + q * p.shared) * 8 * TN + a * TN + b) * 64];
            }
        }
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int rank = r == RB - 1 ? last_rank : wave + NW * r;
            if (r == RB - 1 && (!has_last || part > 0)) break;
            f32x4 sv[8];
#pragma unroll
            for (int a = 0; a < 8; ++a)       // z = S (V x) / 4: the codes of either stage multiply as +-2
                sv[a] = 0.25f * *reinterpret_cast<const f32x4*>(p.S + 128 * rank + 64 * (g & 1) + 16 * (g >> 1) + 32 * (a >> 2) + 4 * (a & 3));
#pragma unroll
            for (int b = 0; b < TN; ++b) {
                float v[32];
#pragma unroll
                for (int e = 0; e < 32; ++e) v[e] = acc[r][e >> 2][b][e & 3] * sv[e >> 2][e & 3];
                tsvd_planes_of_32(v, zrec + (rank * TN + b) * FP6_REC_BYTES, lane);
            }
        }
    }

    // ================= stage U =================
    auto stage_u = [&](auto tm_c) {
        constexpr int TM = decltype(tm_c)::value;
        const int units = (p.M + 16 * TM - 1) / (16 * TM);
        // units are dealt to the wavefronts of all slices of the panel
        const int first = wave + NW * slice, stride = NW * p.slices;
        int nu = first, nb = 0;                               // the next fetch: unit, block
        const int last_unit = first + (units - 1 - first) / stride * stride;
        auto next = [&](words (&w)[TM]) {
#pragma unroll
            for (int a = 0; a < TM; ++a) w[a] = fetch(u_rsrc, lane * 16, (nu * TM + a) * p.nkt_u * 1024, nb);
            if (nb + PER < p.nub) nb += PER;
            else if (nu < last_unit) {                        // (at the end: the last fetch again)
                nu += stride;
                nb = 0;
            }
        };
        words w0[TM];
        if (first < units) next(w0);
        __syncthreads();                                      // the planes of z are complete
        for (int unit = first; unit < units; unit += stride) {
            const int strip0 = unit * TM;
            f32x4 acc[TM][TN];
#pragma unroll
            for (int a = 0; a < TM; ++a) {
                f32x4 br = {0.f, 0.f, 0.f, 0.f};
                if (p.bias) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) br[e] = p.bias[min((strip0 + a) * 16 + 4 * g + e, p.M - 1)];
                }
#pragma unroll
                for (int b = 0; b < TN; ++b) acc[a][b] = br;
            }
            run(tm_c, zrec, p.nub, w0, next, acc);
            // (wait for the next unit's code words here, before the stores)
#pragma unroll
            for (int a = 0; a < TM; ++a) asm volatile("" :: "v"(w0[a].x), "v"(w0[a].y));
            if (p.token_major && p.out_bf16 && TM >= 4 && (strip0 + TM) * 16 <= p.M) {
                if constexpr (TM >= 4) {
#pragma unroll
                    for (int b = 0; b < TN; ++b) {
                        const int col = b0 + 16 * b + i;
#pragma unroll
                        for (int a = 0; a < TM; a += 4) {
                            uint32_t d[4][2];
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                d[k][0] = tsvd_pack_bf16(acc[a + k][b][0], acc[a + k][b][1]);
                                d[k][1] = tsvd_pack_bf16(acc[a + k][b][2], acc[a + k][b][3]);
                            }
                            tsvd_store_token_major_bf16_4x16(p.y, p.ldy, col, col < p.B, (strip0 + a) * 16, g, d);
                        }
                    }
                }
                continue;
            }
            if constexpr (SOURCE != THIN_TOKEN_MAJOR) {
                if (!p.token_major && !p.out_bf16 && p.ldy < (1ll << 21)) {
                    // Without a test or an address computation per store: a constant offset per lane plus a scalar; rows beyond M fall
                    // outside the buffer's range, which is exact in the last unit.  (Convolutions 0.97, feature-major calls 0.98 of the time.)
                    const size_t left = ((size_t)(p.M - strip0 * 16) * p.ldy - b0) * 4;
                    const __amdgpu_buffer_rsrc_t y_rsrc = __builtin_amdgcn_make_buffer_rsrc(
                        static_cast<float*>(p.y) + (size_t)strip0 * 16 * p.ldy + b0, 0, (int)(left < 0xFFFFFFFFull ? left : 0xFFFFFFFFull), 0x00020000);
                    const int ld4 = (int)p.ldy * 4, y_voff = 4 * g * ld4 + i * 4;
#pragma unroll
                    for (int b = 0; b < TN; ++b) {
                        if (b0 + 16 * b + i < p.B) {
#pragma unroll
                            for (int a = 0; a < TM; ++a)
#pragma unroll
                                for (int e = 0; e < 4; ++e)
                                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[a][b][e]), y_rsrc, y_voff + 64 * b, (16 * a + e) * ld4, 0);
                        }
                    }
                    continue;
                }
            }
#pragma unroll
            for (int a = 0; a < TM; ++a) {
                const int row0 = (strip0 + a) * 16 + 4 * g;
#pragma unroll
                for (int b = 0; b < TN; ++b) {
                    const int col16 = b0 + 16 * b, col = col16 + i;
                    const f32x4 v = acc[a][b];
                    if (p.token_major) {
                        if (col < p.B) tsvd_store_token_major4(p.y, p.ldy, col, row0, p.M, v[0], v[1], v[2], v[3], p.out_bf16);
                    } else if (p.out_bf16) {
                        tsvd_store_row_pair_bf16(p.y, p.ldy, row0, p.M, col16, i, p.B, v[0], v[1]);
                        tsvd_store_row_pair_bf16(p.y, p.ldy, row0 + 2, p.M, col16, i, p.B, v[2], v[3]);
                    } else if (col < p.B) {
                        float* dst = static_cast<float*>(p.y) + (size_t)row0 * p.ldy + col;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (row0 + e < p.M) dst[(size_t)e * p.ldy] = v[e];
                    }
                }
            }
        }
    };
    if (p.utm == 8) stage_u(std::integral_constant<int, 8>{});
    else if (p.utm == 4) stage_u(std::integral_constant<int, 4>{});
    else stage_u(std::integral_constant<int, 2>{});
}

inline bool thin_rows_of_taps(int source, const thin_args& a) { return source == THIN_CONV && a.kv2 == 3 && a.d2 == 1 && a.W >= 4; }

constexpr int LDS_BYTES = 160 * 1024, MAX_TAPS = 48;

template <int TN, int RB, int SOURCE, bool CHUNKED, bool SHARED>
auto kernel() { return tsvd_thin_panel_kernel<TN, RB, SOURCE, CHUNKED, SHARED>; }
template <int TN, int RB, int SOURCE>
hipError_t launch(const thin_args& a, bool shared, int lds, hipStream_t stream) {
    const dim3 grid((unsigned)((a.B + 16 * TN - 1) / (16 * TN)) * (unsigned)a.slices), block(512);
    auto* k = a.buffers == 2 ? shared ? kernel<TN, RB, SOURCE, true, true>() : kernel<TN, RB, SOURCE, true, false>()
                             : shared ? kernel<TN, RB, SOURCE, false, true>() : kernel<TN, RB, SOURCE, false, false>();
    const thin_rest rest = {a.y, a.ldy, a.bias, a.M};
    const thin_images images = {a.images, a.H, a.W, a.kv1, a.kv2, a.Hv, a.Wv, a.s1, a.s2, a.p1, a.p2, a.d1, a.d2};
    hipLaunchKernelGGL(k, grid, block, lds, stream, a.x, a.tiles_v, a.tiles_u, a.S, a.x_bytes, a.N, a.B, (int)a.ldx, thin_form(a), a.slices, rest, images);
    return hipGetLastError();
}
template <int TN, int RB>
hipError_t launch(int source, const thin_args& a, bool shared, int lds, hipStream_t stream) {
    if (thin_rows_of_taps(source, a)) return launch<TN, RB, THIN_CONV_ROWS>(a, shared, lds, stream);
    if (source == THIN_CONV) return launch<TN, RB, THIN_CONV>(a, shared, lds, stream);
    if (source == THIN_TOKEN_MAJOR) return launch<TN, RB, THIN_TOKEN_MAJOR>(a, shared, lds, stream);
    return launch<TN, RB, THIN_FEATURE_MAJOR>(a, shared, lds, stream);
}
template <int TN, int RB, int SOURCE>
hipError_t init() {
    for (const auto k : {kernel<TN, RB, SOURCE, false, false>(), kernel<TN, RB, SOURCE, true, false>(), kernel<TN, RB, SOURCE, false, true>(), kernel<TN, RB, SOURCE, true, true>()}) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
template <int TN, int RB>
hipError_t init() {
    hipError_t e;
    if ((e = init<TN, RB, THIN_FEATURE_MAJOR>()) != hipSuccess || (e = init<TN, RB, THIN_TOKEN_MAJOR>()) != hipSuccess) return e;
    if ((e = init<TN, RB, THIN_CONV>()) != hipSuccess) return e;
    return init<TN, RB, THIN_CONV_ROWS>();
}

}  // namespace

hipError_t tsvd_thin_init() {
    hipError_t e;
    if ((e = init<1, 1>()) != hipSuccess) return e;
    if ((e = init<1, 2>()) != hipSuccess) return e;
    return init<2, 1>();
}

static size_t tsvd_thin_x_bytes(const tsvd_thin_problem& g) {
    const tsvd_blob_header& hd = *g.hd;
    if (g.source == THIN_CONV) return (size_t)(hd.N / (g.kv1 * g.kv2)) * g.images * g.H * g.W * 2;
    const long long rows = g.source == THIN_TOKEN_MAJOR ? g.B : hd.N, cols = g.source == THIN_TOKEN_MAJOR ? hd.N : g.B;
    return (size_t)((rows - 1) * g.ldx + cols) * 2;
}

// Blocks of x in LDS at a time: all of them if they fit beside those of z, else two chunks of an even number of blocks (a pair
// shares its code words), of about equal length; 0: not possible.
int tsvd_thin_chunk(long long K, long long N, int tiles, bool conv) {
    const long long nvb = (N + 127) / 128, nub = (K + 127) / 128, table = conv ? nvb * 512 : 0;
    if (nub > 16 / tiles) return 0;
    const long long room = ((LDS_BYTES - table) / FP6_REC_BYTES - nub * tiles) / tiles;
    if (nvb <= room) return (int)nvb;
    const long long most = room / 2 & ~1ll;
    if (most < 2) return 0;
    const long long chunks = (nvb + most - 1) / most;
    return (int)std::min(most, ((nvb + chunks - 1) / chunks + 1) & ~1ll);
}

// Stage V's last `left` rank blocks (1 to 8): where one or two are left several wavefronts share each, a part of its contraction everyone; of five or six the first four stay
// whole, one on each SIMD, and the other four wavefronts share the rest.  Of three, four or seven no SIMD has less than without, and shared they cost 3 to 6 % (3 x 3 from 69 channels, rank 412).
// The sums meet behind two more barriers, 0.3 us: worth it from three blocks that the longest part is shorter by, six where a SIMD has a whole one beside (85 channels, rank 704: 12.4 -> 12.7 us).
// Rows of taps in chunks are dear to make: with two rank blocks the six others make them all in the time that these two take (491 channels, rank 147: 36.2 -> 37.7 shared).  The last two of ten in chunks
// of eight blocks leave each of the eight wavefronts a single fetch, and nobody who makes records first (310 channels, rank 1250, 3136 positions: 29.3 -> 30.3 us shared, 4096 features as rows of tokens 41.1 -> 41.7;
// in chunks of ten, 350 channels, 34.4 -> 33.4).
static bool thin_shares(thin_args& a, int tiles, bool conv, bool rows_of_taps) {
    const int left = (a.nub + 7) % 8 + 1, room = LDS_BYTES - a.nub * tiles * FP6_REC_BYTES - (conv ? a.nvb * 512 : 0);
    a.whole = left > 4 ? 4 : 0;
    a.shared = left - a.whole;
    a.parts = 0;
    if (a.shared > 2 || (a.buffers == 2 && a.shared == 2 && (a.nub == 2 ? rows_of_taps : a.nub == 10 && a.chunk <= 8))) return false;
    while (a.shared << (a.parts + 1) <= 8 - a.whole && 2 << a.parts <= (a.chunk + 1) / 2) ++a.parts;
    const int sums = a.shared * ((1 << a.parts) - 1) * tiles * 8192, longest = (a.nvb + (1 << a.parts) - 1) >> a.parts;
    return sums <= room && (a.nvb - longest) * tiles >= (a.whole ? 6 : 3);
}
static void thin_blocks(thin_args& a, long long K, long long N, int tiles, bool conv) {
    a.nvb = (int)((N + 127) / 128);
    a.nub = (int)((K + 127) / 128);
    a.chunk = tsvd_thin_chunk(K, N, tiles, conv);
    a.buffers = a.chunk < a.nvb ? 2 : 1;
}

static int thin_shares_code(const thin_args& a) { return 100 * (a.buffers - 1) + 10 * a.shared + (1 << a.parts); }
static thread_local int thin_last = 0;       // for tsvd_tuning_thin_last

extern "C" int tsvd_tuning_thin_last(void) {
    const int last = thin_last;
    thin_last = 0;
    return last;
}
extern "C" int tsvd_tuning_thin_shares(int64_t K, int64_t N, int tiles, int gathers, int rows_of_taps) {
    thin_args a;
    thin_blocks(a, K, N, tiles, gathers != 0);
    if (a.chunk == 0) return -1;
    return thin_shares(a, tiles, gathers != 0, rows_of_taps != 0) ? thin_shares_code(a) : 0;
}

hipError_t tsvd_thin_launch(const tsvd_thin_problem& g, int tiles, hipStream_t stream) {
    const tsvd_blob_header& hd = *g.hd;
    if (tsvd_thin_x_bytes(g) >= (1ull << 30) || (size_t)hd.Mp * hd.Kp / 4 >= (1ull << 31) || (size_t)hd.Kp * hd.Np / 4 >= (1ull << 31))
        return hipErrorNotSupported;
    thin_args a;
    a.tiles_v = reinterpret_cast<const uint32_t*>(g.blob + hd.off_V);
    a.tiles_u = reinterpret_cast<const uint32_t*>(g.blob + hd.off_U);
    a.tile_v_bytes = (unsigned)((size_t)hd.Kp * hd.Np / 4);
    a.tile_u_bytes = (unsigned)((size_t)hd.Mp * hd.Kp / 4);
    a.nkt_v = (int)(hd.Np / 256);
    a.nkt_u = (int)(hd.Kp / 256);
    a.x = g.x;
    a.x_bytes = (unsigned)tsvd_thin_x_bytes(g);
    a.N = (int)hd.N;
    a.B = (int)g.B;
    a.ldx = g.source == THIN_FEATURE_MAJOR && hd.N == 1 ? g.B : g.ldx;       // (a single row: its distance to the next is any number)
    a.images = g.images; a.H = g.H; a.W = g.W; a.kv1 = g.kv1; a.kv2 = g.kv2; a.Hv = g.Hv; a.Wv = g.Wv;
    a.s1 = g.s1; a.s2 = g.s2; a.p1 = g.p1; a.p2 = g.p2; a.d1 = g.d1; a.d2 = g.d2;
    a.S = reinterpret_cast<const float*>(g.blob + hd.off_S);
    a.y = g.y;
    a.ldy = g.ldy;
    a.bias = g.bias;
    a.M = (int)hd.M;
    a.out_bf16 = g.out_bf16;
    a.token_major = g.y_token_major;
    // Feature-major rows of enough panels, where x is not outweighed by y or the panels share lines of y too: 5019 x 4308 x 768 at 11841
    // tokens 253 -> 199 us, 244 x 2015 x 1536 at 3621 33.9 -> 26.7, 975 x 320 x 125 at 3773 13.3 -> 10.9, 9141 x 731 x 259 at 3805 62.7 -> 44.7.
    // With 50 panels 9.3 -> 10.0 (575 x 177 x 122); with whole lines of y 27.3 -> 29.4 for 2304 rows on 98 (a convolution's columns, which
    // another launch folds), 26.5 -> 27.4 for 7635 on 128, 16.5 -> 17.2 for 933 on 384.  Rows of tokens share nothing; gathered convolutions: 0.95 to 1.1.
    // On 197 random calls (64 .. 2048 ranks, 200 .. 16384 tokens) the rule takes 0.957 of the time without (panels of 16 tokens) and 0.979 (of 32), the better of the two for
    // every call 0.947 and 0.976; where it says yes 0.70 .. 1.02.
    const int piece = a.out_bf16 ? 2 : 4;
    a.runs = g.source == THIN_FEATURE_MAJOR && g.B > 60 * 16 * tiles && (a.ldy * piece % 64 != 0 || a.M * piece <= 6 * a.N);
    // Rows per unit of stage U: the larger units unless they leave wavefronts without one.  Fewer panels than half of the compute units: several workgroups
    // for each, which all make the whole z of their tokens and deal the units among them, as many as shorten stage U (888 x 384 x 69 at 881
    // tokens, 56 panels: 7.8 us with one, 7.0 with two, 6.6 with four; 918 x 348 x 192 at 320 8.0 -> 6.65; convolutions of few positions 0.79 to 0.98 of the time, no call slower).
    auto passes = [&](int utm, int slices) { return ((a.M + 16 * utm - 1) / (16 * utm) + 8 * slices - 1) / (8 * slices) * utm; };
    const long long panels = (g.B + 16 * tiles - 1) / (16 * tiles);
    int best = 1 << 30;
    a.slices = 1;
    for (int slices = 1; slices == 1 || slices * panels <= g.cus; ++slices) {
        for (int utm : {8, 4, 2})
            if (passes(utm, slices) < best) best = passes(utm, slices), a.slices = slices, a.utm = utm;
        if (best == 2) break;
    }
    const bool conv = g.source == THIN_CONV;
    thin_blocks(a, hd.K, hd.N, tiles, conv);
    if (g.source == THIN_FEATURE_MAJOR && 128ll * a.nvb * a.ldx >= 1ll << 30) return hipErrorNotSupported;     // (element loads reach rows, those beyond N too, at 32-bit offsets)
    if (conv && g.kv1 * g.kv2 > MAX_TAPS) return hipErrorNotSupported;
    if (a.chunk == 0) return hipErrorNotSupported;
    const int rb = (a.nub + 7) / 8;
    const bool shared = thin_shares(a, tiles, conv, thin_rows_of_taps(g.source, a));
    thin_last = 1000 * tiles + (shared ? thin_shares_code(a) : 0);
    const int lds = thin_x_bytes(a, tiles, shared) + a.nub * tiles * FP6_REC_BYTES + (conv ? a.nvb * 512 : 0);
    if (tiles == 1 && rb == 1) return launch<1, 1>(g.source, a, shared, lds, stream);
    if (tiles == 1 && rb == 2) return launch<1, 2>(g.source, a, shared, lds, stream);
    if (tiles == 2 && rb == 1) return launch<2, 1>(g.source, a, shared, lds, stream);
    return hipErrorNotSupported;
}
