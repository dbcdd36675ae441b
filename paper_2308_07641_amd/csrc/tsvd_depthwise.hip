// Depth-wise convolutions (one input channel per group) as banded matrix products.
//
// A group's factors collapse to one kernel per output channel, w[dy][dx] = sum over its ranks of U S V, so the ranks cost nothing per
// position; and for a fixed dy a row of 16 outputs is a product of the input row with a banded 16 x 32 matrix of w[dy]: seven matrix
// instructions per 16 x 16 outputs and part of w for a 7 x 7 kernel where vector instructions need 49 per output (or, on the factors, 49 per
// output and rank less the zeros).  w is fp32: it enters as the sum of three bf16 parts, which hold its 24 bits exactly, so products are
// exact and sums are fp32 as before.
//
// The 16 columns of the B operand are strips: R output rows of a column of tiles of one image, as many strips as it takes to fill the chip (images times
// segments of the plane times columns of tiles).  Strips side by side stand in lanes side by side, so that a wavefront's request for a row is
// whole rows of a few images rather than 64 bytes of sixteen, and its stores too: the requests' lines bound the kernel more than its matrix instructions (with sixteen images
// or segments in a wavefront 123 channels of 56 x 56, 5 x 5, 59 images 28.1 us, now 26.0; 558 of 3 x 3, 10 images 22.1 -> 19.5; 201 of 28 x 28, 7 x 7, stride 2, 49 images 15.9 -> 13.1;
// 50 drawn geometries 0.95 of the time, none longer).  A lane's B operand is eight columns of its strip's next row, straight from global memory (16 bytes where
// rows are aligned); the last k1 rows stay in registers, each output row needs stride1 new ones, fetched one output row ahead.
// The banded matrices are the same for every strip and column tile of a channel: the four wavefronts of a workgroup make them
// together, then each keeps all of them in registers.
//
// The zeros of a band meet every column of the window, so an infinite or NaN pixel makes all outputs of its strip's rows NaN, and a
// scale that is not finite all outputs of the channel.  Every such output is itself not finite: a lane that has stored one computes its
// outputs again on the factors, tap by tap, zeros skipped, where only the outputs are touched whose taps hold the value.
//
// Measured on MI355X: 96 channels of 56 x 56, 7 x 7 at rank 5, 32 images, bf16: 14.0 us (14.5 with sixteen images or segments in a wavefront, 68 on the factors): 6.7 of them matrix instructions, about 3.5 the latency of the
// first loads and the bands, 2 the launch; 640 of 28 x 28, 5 x 5, stride 2, 8 images 6.9, 217 of 28 x 28, 7 x 7, 32 images 11.6 (before strips lay along the row 8.3 and 11.8, with rows in loads of two elements and more of them ahead
// 16.6 and 14.5).  60 random geometries of 64 to 768 channels: 1.04 to 41 times the speed of the kernel on the factors.
#include "tsvd_depthwise.h"

#include <algorithm>
#include <utility>

#include "tsvd_epilogue.h"
#include "tsvd_gemm_common.h"
#include "tsvd_kernels.h"
#include "tsvd_layout.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct depthwise_args {
    tsvd_depthwise_problem g;
    int R, segments, col_tiles, strips;              // output rows of a strip, strips to a column of tiles, columns of tiles; strips of all images
    unsigned plane_bytes;                            // of one channel of x
};

// f(0), f(1), ... with compile-time arguments until one returns false.
template <int... u, class F>
__device__ __forceinline__ bool each(std::integer_sequence<int, u...>, F f) {
    return (f(std::integral_constant<int, u>{}) && ...);
}

// The outputs of this lane on the factors, one at a time.  (Everything is derived again from the lane's number: kept in registers over
// the kernel's loop it would cost occupancy.)
template <int STEP>
__device__ __forceinline__ void outputs_on_factors(const depthwise_args& p, int wave) {
    const tsvd_depthwise_problem& g = p.g;
    int all = -1;
    asm volatile("" : "+s"(all));
    const int lane = __builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0));
    const int i = lane & 15, q = lane >> 4, m = blockIdx.y, group = m / g.mg, strip = (blockIdx.x * 4 + wave) * 16 + i;
    const int rest = strip / p.col_tiles, ct = strip - rest * p.col_tiles, img = rest / p.segments, row0 = (rest - img * p.segments) * p.R;
    if (strip >= p.strips) return;
    const int ox = ct * (16 / STEP) + 4 * (STEP == 1 ? q : q & 1), oend = min(ox + 4, g.Wo), yend = min(row0 + p.R, g.Ho);
    const uint16_t* plane = g.x + ((size_t)group * g.images + img) * g.H * g.W;
    const float b = g.bias ? g.bias[m] : 0.f;
    for (int oy = row0 + (STEP == 1 ? 0 : q >> 1); oy < yend; oy += STEP) {
#pragma unroll 1
        for (int c = ox; c < oend; ++c) {
            float y = 0.f;
#pragma unroll 1
            for (int k = 0; k < g.kg; ++k) {
                const int pos = (int)tsvd_rank_position(group * g.kg + k, g.K), u = tsvd_code_at(g.U, g.u_tps, m, pos);
                if (!(u & 1)) continue;
                float z = 0.f;
#pragma unroll 1
                for (int tap = 0; tap < g.k1 * g.k2; ++tap) {
                    const int v = tsvd_code_at(g.V, g.v_tps, pos, tap), dy = tap / g.k2, iy = oy * STEP - g.p1 + dy, ix = c * STEP - g.p2 + tap - dy * g.k2;
                    if (!(v & 1) || (unsigned)iy >= (unsigned)g.H || (unsigned)ix >= (unsigned)g.W) continue;
                    const float xv = __uint_as_float((uint32_t)plane[(size_t)iy * g.W + ix] << 16);
                    z += v & 2 ? -xv : xv;
                }
                z *= g.S[pos];
                y += u & 2 ? -z : z;
            }
            tsvd_store_y(g.y, (((size_t)m * g.images + img) * g.Ho + oy) * g.Wo + c, y + b, g.out_bf16);
        }
    }
}

// ROW: elements per load of a row of x: 8 where rows are aligned to 16 bytes, else 4 at any alignment, or 1 in rows of fewer than four.  (Rows of an even number
// of elements were loaded by 2, odd ones by 1: four and eight requests a row, which keep the address unit busy longer than the row's matrix instructions the
// matrix pipe.)  STEP: both strides.  With stride 2 the window of 16 outputs would not fit 32 columns: a tile is 8 columns of two output rows there, and an input
// row is multiplied by the taps of both.
// VEC: rows of y are a multiple of four elements and y is aligned to four (then a lane's four columns are inside or outside together
// and are stored at once).
template <int K1, int STEP, int ROW, bool VEC>
__global__ void __launch_bounds__(256, K1 == 7 && STEP == 1 ? 3 : 2)
tsvd_depthwise_kernel(depthwise_args p) {
    constexpr int COLS = 16 / STEP, NR = K1 + (STEP - 1) * STEP, ADV = STEP * STEP;      // of a tile: columns, input rows, input rows to the next
    // Rows in registers, and tiles until the slots repeat: as few as pay, since every further row is requested by all wavefronts before the first product, and the
    // loop is unrolled over the slots.  With stride 1 a row is requested two tiles before the one that needs it first (in rows of fewer than four elements: by that tile itself).
    // With stride 2 a tile requests four rows and needs one of them at once (3 x 3 and 7 x 7; 5 x 5 three), so it waits for what it has just asked for, and the SIMD's
    // other wavefronts cover that.  (Three rows ahead with stride 1, 16 or 20 slots with stride 2: 2 % slower with rows by 8, 663 channels of 7 x 7, 3 x 3, stride 2, 2 images
    // 6.3 -> 9.9 us.  12 slots for 5 x 5 with stride 2, whose rows then come a tile ahead: 0.96 to 1.03 of the time of 8 on 14 geometries, 0.995 on the average.)
    constexpr int RING = STEP == 1 ? NR + (ROW == 1 ? 0 : 2) : NR > 8 ? 12 : 8, PERIOD = STEP == 1 ? RING : RING / ADV;
    const tsvd_depthwise_problem& g = p.g;
    __shared__ u32x2 weight[64];                      // of a tap its three parts (bf16: the first two, the last); the last entry is zero
    __shared__ __align__(16) unsigned char bands[NR * 3 * 1024];
    float* const terms = reinterpret_cast<float*>(bands);      // before the bands: U S V per rank and tap
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, q = lane >> 4;
    const int m = blockIdx.y, group = m / g.mg;
    const int scalar_wave = __builtin_amdgcn_readfirstlane(wave);    // (for the outputs that are computed again)

    // ---- this lane's strip and columns; the rows of the first output
    const int strip = (blockIdx.x * 4 + wave) * 16 + i, rest = strip / p.col_tiles, ct = strip - rest * p.col_tiles, img = rest / p.segments, row0 = (rest - img * p.segments) * p.R;
    const int first = ct * 16 - g.p2, c0 = first & ~7;       // window of the tile: columns c0 .. c0 + 31, (COLS - 1) STEP + k2 + 7 <= 29 of them used
    const bool strip_ok = strip < p.strips;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(g.x) + (size_t)group * (p.plane_bytes / 2), 0, (int)p.plane_bytes, 0x00020000);
    const int iy_first = row0 * STEP - g.p1, base = 2 * img * g.H * g.W, pitch = 2 * g.W;
    constexpr unsigned NONE = 0x40000000u;                  // beyond the buffer (below 2^30 bytes): loads give zero
    constexpr int LOADS = 8 / ROW;
    unsigned col_off[LOADS], beyond[LOADS];
#pragma unroll
    for (int e = 0; e < LOADS; ++e) {
        // (columns are multiples of ROW: the four elements of a load lie inside the row, or outside, or their last one to three beyond it)
        const int col = c0 + 8 * q + ROW * e, more = ROW == 4 ? max(0, col + 4 - g.W) : 0;
        col_off[e] = col >= 0 && col < g.W && strip_ok ? (unsigned)(base + 2 * (col - more)) : NONE;
        beyond[e] = 16 * (more & 3);
    }
    auto load_row = [&](int j) __attribute__((always_inline)) {                // row j of the strip's window
        const int iy = iy_first + j;
        const unsigned off = (unsigned)iy < (unsigned)g.H ? (unsigned)(iy * pitch) : NONE;
        if constexpr (ROW == 8) {
            return buf_load128(xr, (int)(off + col_off[0]), 0);
        } else if constexpr (ROW == 4) {
            const u32x2 lo = __builtin_amdgcn_raw_buffer_load_b64(xr, (int)(off + col_off[0]), 0, 0);
            const u32x2 hi = __builtin_amdgcn_raw_buffer_load_b64(xr, (int)(off + col_off[1]), 0, 0);
            return u32x4{lo.x, lo.y, hi.x, hi.y};
        } else {
            u32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t lo = __builtin_amdgcn_raw_buffer_load_b16(xr, (int)(off + col_off[2 * e]), 0, 0);
                const uint32_t hi = __builtin_amdgcn_raw_buffer_load_b16(xr, (int)(off + col_off[2 * e + 1]), 0, 0);
                v[e] = lo | hi << 16;
            }
            return v;
        }
    };
    // Four elements that end with the row where the lane's four do not: those before are shifted out, where the row is first needed (here its loads would
    // be awaited).
    auto in_place = [&](u32x4& v) __attribute__((always_inline)) {
        if constexpr (ROW == 4) {
            const uint64_t lo = ((uint64_t)v.y << 32 | v.x) >> beyond[0], hi = ((uint64_t)v.w << 32 | v.z) >> beyond[1];
            v = u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
        }
    };
    u32x4 ring[RING];                                 // row j in slot j % RING
    // ---- what the first term of this thread is made of, requested ahead of the rows (results come in the order of the requests)
    const int taps = g.k1 * g.k2, ranks = min(g.kg, NR * 3 * 256 / 49);         // (ranks whose terms fit at a time)
    const int idx0 = min((int)threadIdx.x, ranks * taps - 1), pos0 = (int)tsvd_rank_position(group * g.kg + idx0 / taps, g.K), tap0 = idx0 % taps;
    int u_word, u_bit, v_word, v_bit;
    tsvd_code_position(m & 15, pos0 & 255, &u_word, &u_bit);
    tsvd_code_position(pos0 & 15, tap0, &v_word, &v_bit);
    const uint32_t u_codes = g.U[((size_t)(m >> 4) * g.u_tps + (pos0 >> 8)) * 256 + u_word], v_codes = g.V[(size_t)(pos0 >> 4) * g.v_tps * 256 + v_word];
    const float s_first = g.S[pos0];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < RING - ADV; ++j) ring[j] = load_row(j);
    __builtin_amdgcn_sched_barrier(0);

    // ---- the kernel of the channel, then its banded matrices
    float w = 0.f;                                    // of tap threadIdx.x
    for (int k0 = 0; k0 < g.kg; k0 += ranks) {
        const int n = min(ranks, g.kg - k0);
        if (k0) __syncthreads();
        for (int idx = threadIdx.x; idx < n * taps; idx += 256) {
            int u = (int)(u_codes >> u_bit), v = (int)(v_codes >> v_bit);
            float s = s_first;
            if (k0 > 0 || idx >= 256) {
                const int k = idx / taps, pos = (int)tsvd_rank_position(group * g.kg + k0 + k, g.K);
                u = tsvd_code_at(g.U, g.u_tps, m, pos), v = tsvd_code_at(g.V, g.v_tps, pos, idx - k * taps);
                s = g.S[pos];
            }
            terms[idx] = (u & v & 1) ? ((u ^ v) & 2 ? -s : s) : 0.f;
        }
        __syncthreads();
        if ((int)threadIdx.x < taps)
            for (int k = 0; k < n; ++k) w += terms[k * taps + threadIdx.x];
    }
    if (threadIdx.x < 64) {
        uint32_t part[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const uint32_t top = __float_as_uint(w) & 0xFFFF0000u;              // the leading eight bits of what is left: exact
            part[s] = top >> 16;
            w -= __uint_as_float(top);
        }
        weight[threadIdx.x] = u32x2{part[0] | part[1] << 16, part[2]};
    }
    __syncthreads();
    const int from_c0 = -g.p2 & 7;                    // first - c0 (a tile starts at a multiple of 16 columns)
    for (int f = wave; f < NR; f += 4) {
        const int dy = f - i / COLS * STEP;
        const int at = (unsigned)dy < (unsigned)K1 ? dy * g.k2 : 63, first_dx = 8 * q - from_c0 - i % COLS * STEP;   // window column of element 0, from the output's first
        u32x4 part[3];
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const u32x2 w0 = weight[(unsigned)(first_dx + e) < (unsigned)g.k2 ? min(at + first_dx + e, 63) : 63],
                        w1 = weight[(unsigned)(first_dx + e + 1) < (unsigned)g.k2 ? min(at + first_dx + e + 1, 63) : 63];
            part[0][e >> 1] = (w0.x & 0xFFFFu) | w1.x << 16;
            part[1][e >> 1] = w0.x >> 16 | (w1.x & 0xFFFF0000u);
            part[2][e >> 1] = w0.y | w1.y << 16;
        }
#pragma unroll
        for (int s = 0; s < 3; ++s) *reinterpret_cast<u32x4*>(bands + (f * 3 + s) * 1024 + lane * 16) = part[s];
    }
    __syncthreads();
    if ((int)(blockIdx.x * 4 + scalar_wave) * 16 >= p.strips) return;
    bf16x8 band[NR][3];
#pragma unroll
    for (int f = 0; f < NR; ++f)
#pragma unroll
        for (int s = 0; s < 3; ++s) band[f][s] = *reinterpret_cast<const bf16x8*>(bands + (f * 3 + s) * 1024 + lane * 16);

    // ---- R output rows: lane (i, q) ends with four columns of strip i: 4 q .. 4 q + 3 of the row, or 4 (q & 1) .. of the pair's row q >> 1
    const float b = g.bias ? g.bias[m] : 0.f;
    const int ox = ct * COLS + 4 * (STEP == 1 ? q : q & 1), orow = STEP == 1 ? 0 : q >> 1, rows = strip_ok ? min(p.R, g.Ho - row0) : 0;
    // (stores beyond the plane or the strip go to an offset beyond the buffer and are dropped: were they branched around, the wait for a
    // row of x would have to count on stores that may not be there, and wait for those that are)
    const unsigned esize = g.out_bf16 ? 2 : 4, out_plane = (unsigned)(g.images * g.Ho * g.Wo) * esize, yp = (unsigned)(STEP * g.Wo) * esize;
    const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc(static_cast<unsigned char*>(g.y) + (size_t)m * out_plane, 0, (int)out_plane, 0x00020000);
    unsigned at = (unsigned)((img * g.Ho + row0 + orow) * g.Wo + ox) * esize;
    if (VEC && ox >= g.Wo) at = NONE;
    const int tiles = (p.R + STEP - 1) / STEP;
    bool odd = false;                                 // an output was not finite
    auto tile = [&](auto u_c, int t) __attribute__((always_inline)) {          // t % PERIOD = u
        constexpr int u = decltype(u_c)::value;
#pragma unroll
        for (int j = RING - ADV; j < RING; ++j) ring[(u * ADV + j) % RING] = load_row(t * ADV + j);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = NR - ADV; f < NR; ++f) in_place(ring[(u * ADV + f) % RING]);
        f32x4 acc[3];
        acc[0] = f32x4{b, b, b, b};
        acc[1] = acc[2] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int f = 0; f < NR; ++f)
#pragma unroll
            for (int s = 0; s < 3; ++s)
                acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(band[f][s], __builtin_bit_cast(bf16x8, ring[(u * ADV + f) % RING]), acc[s], 0, 0, 0);
        const f32x4 y = acc[0] + (acc[1] + acc[2]);
        const unsigned to = t * STEP + orow < rows ? at : NONE;
        if constexpr (VEC) {
            if (g.out_bf16) __builtin_amdgcn_raw_buffer_store_b64(u32x2{tsvd_pack_bf16(y[0], y[1]), tsvd_pack_bf16(y[2], y[3])}, yr, (int)to, 0, 0);
            else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, y), yr, (int)to, 0, 0);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned te = ox + e < g.Wo ? to + e * esize : NONE;
                if (g.out_bf16) __builtin_amdgcn_raw_buffer_store_b16((short)tsvd_bf16_rne(y[e]), yr, (int)te, 0, 0);
                else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(y[e]), yr, (int)te, 0, 0);
            }
        }
        odd |= !(fabsf(y[0]) < INFINITY);         // (a value that spreads reaches all four)
        at += yp;
    };
#pragma unroll
    for (int f = 0; f < NR - ADV; ++f) in_place(ring[f]);
    int t = 0;
    while (each(std::make_integer_sequence<int, PERIOD>{}, [&](auto u) __attribute__((always_inline)) {
        tile(u, t);
        return ++t < tiles;
    })) {
    }
    if (!odd) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the stores of the same elements are done)
    outputs_on_factors<STEP>(p, scalar_wave);
}

template <int K1, int STEP>
void launch(const depthwise_args& a, int row, dim3 grid, hipStream_t stream) {
    auto go = [&](auto row_c) {
        constexpr int ROW = decltype(row_c)::value;
        const bool vec = a.g.Wo % 4 == 0 && reinterpret_cast<uintptr_t>(a.g.y) % (a.g.out_bf16 ? 8 : 16) == 0;
        if (vec) hipLaunchKernelGGL((tsvd_depthwise_kernel<K1, STEP, ROW, true>), grid, dim3(256), 0, stream, a);
        else hipLaunchKernelGGL((tsvd_depthwise_kernel<K1, STEP, ROW, false>), grid, dim3(256), 0, stream, a);
    };
    if (row == 8) go(std::integral_constant<int, 8>{});
    else if (row == 4) go(std::integral_constant<int, 4>{});
    else go(std::integral_constant<int, 1>{});
}

}  // namespace

hipError_t tsvd_depthwise_launch(const tsvd_depthwise_problem& g, hipStream_t stream) {
    const long long plane_bytes = 2ll * g.images * g.H * g.W, channels = (long long)g.groups * g.mg;
    if ((g.k1 != 3 && g.k1 != 5 && g.k1 != 7) || g.k2 > 7 || g.s1 != g.s2 || g.s1 > 2 || g.d1 != 1 || g.d2 != 1 || plane_bytes >= (1ll << 30) ||
        4ll * g.images * g.Ho * g.Wo >= (1ll << 30) || channels > 65535)
        return hipErrorNotSupported;
    depthwise_args a;
    a.g = g;
    a.plane_bytes = (unsigned)plane_bytes;
    const int cols = 16 / g.s1;
    a.col_tiles = (g.Wo + cols - 1) / cols;
    // Output rows per strip: short strips reload k1 - 1 rows each, long ones leave compute units idle.  In units of a matrix instruction, per
    // round of workgroups: the rows of a strip, and for the bands and the first rows what was best on 27 geometries (100 in place of 60: 1.5 % slower, 30: one of them 18 %).
    long long best = -1;
    for (int n = 1; n <= std::min(g.Ho, 64); ++n) {
        const int R = (g.Ho + n - 1) / n, segments = (g.Ho + R - 1) / R;
        const long long strips = (long long)g.images * segments * a.col_tiles, blocks = (strips + 63) / 64 * channels;
        const long long work = (long long)((R + g.s1 - 1) / g.s1) * 3 * (g.k1 + (g.s1 - 1) * g.s1);
        const long long cost = (blocks + g.cu_count - 1) / g.cu_count * (work + 4 * g.k1 + 60) + work;
        if (best < 0 || cost < best) {
            best = cost;
            a.R = R; a.segments = segments; a.strips = (int)strips;
        }
    }
    const dim3 grid((unsigned)((a.strips + 63) / 64), (unsigned)channels);
    const uintptr_t at = reinterpret_cast<uintptr_t>(g.x);
    const int row = g.W % 8 == 0 && at % 16 == 0 ? 8 : g.W >= 4 ? 4 : 1;
    if (g.s1 == 1) {
        if (g.k1 == 3) launch<3, 1>(a, row, grid, stream);
        else if (g.k1 == 5) launch<5, 1>(a, row, grid, stream);
        else launch<7, 1>(a, row, grid, stream);
    } else {
        if (g.k1 == 3) launch<3, 2>(a, row, grid, stream);
        else if (g.k1 == 5) launch<5, 2>(a, row, grid, stream);
        else launch<7, 2>(a, row, grid, stream);
    }
    return hipGetLastError();
}
