// C ABI entry points that touch the device: upload, forward dispatch, release.
// (The host-only packer lives in tsvd_pack.cpp.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <new>

#include "../../include/tsvd.h"
#include "../../include/tsvd_tuning.h"
#include "tsvd_batch.h"
#include "tsvd_few.h"
#include "tsvd_kernels.h"
#include "tsvd_layout.h"
#include "tsvd_scratch.h"
#include "tsvd_thin.h"

struct tsvd_handle {
    int device;
    tsvd_blob_header hd;
    uint8_t* blob;          // device
    bool owns_blob;
    void* scratch;          // device, handle-owned workspace (grown on demand)
    size_t scratch_bytes;
    void* retired[16];      // earlier, smaller scratch buffers: enqueued work may still use them, so they live until tsvd_free
    int retired_count;
    float bound_V;          // max_k |S_k| * nnz(V[k,:]) : |z_k| <= bound_V * max|x| for every token
    int cu_count;           // compute units of the device
    long long* clocks;      // tuning aid (TSVD_CLOCKS=1 at pack time): phase timestamps of the B <= 2 kernel
    // One-launch single-token path: [counter: 256 B][z as tagged 64-bit words: Kp], device, zeroed at pack
    // (counter = 1); null when the shape does not fit that kernel.  The path belongs to the first stream
    // that uses it: calls on one stream never overlap, calls on other streams take the two-launch kernels.
    uint8_t* dense_u;       // device: U in the denser code (five elements per byte), only with TSVD_DENSE_U = 1 at pack time
    uint8_t* sync;
    std::atomic<int> sync_claimed;
    void* sync_stream;
};

// Workspace of tsvd_forward_noalloc: one array per GPU inside the loaded code object, so the entry point
// never allocates.  The name below is a host-side stand-in; the array's device address differs per GPU
// and is looked up once per device in device_init (noalloc_ptr), which is what host code passes on.
static __device__ __align__(256) unsigned char scratch[TSVD_NOALLOC_MAX_WORKSPACE];
static void* noalloc_ptr[64] = {};

namespace {

int env_int(const char* name, int fallback) { return tsvd_tune(name, fallback); }

size_t round256(size_t v) { return (v + 255) & ~(size_t)255; }

// Options of the last stage (tsvd_forward_ex).
struct out_opts {
    const float* bias;   // device [M] or null
    int out_bf16;
    int token_major;     // y is [B][ldy] instead of [M][ldy]
};

// Token-major activations [B][ldx] -> feature-major [N][ldt] (ldt a multiple of 8 elements, the
// padding columns zero), through 32 x 32 LDS tiles; T is the 16- or 32-bit storage type.
template <typename T>
__global__ void __launch_bounds__(256)
tsvd_transpose_kernel(const T* __restrict__ x, long long ldx, int B, int N, T* __restrict__ xt, long long ldt) {
    __shared__ T tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;          // 32 x 8 threads
    const int n0 = blockIdx.x * 32, b0 = blockIdx.y * 32;
#pragma unroll
    for (int r = ty; r < 32; r += 8) {
        const int b = b0 + r, n = n0 + tx;
        tile[r][tx] = (b < B && n < N) ? x[(size_t)b * ldx + n] : T(0);
    }
    __syncthreads();
#pragma unroll
    for (int r = ty; r < 32; r += 8) {
        const int n = n0 + r, b = b0 + tx;
        if (n < N && b < ldt) xt[(size_t)n * ldt + b] = tile[tx][r];
    }
}

// Feature-major activations with unaligned rows [N][ldx] -> [N][ldt] (ldt a multiple of 8 elements, the padding
// columns zero): eight elements per thread, consecutive threads along a row; the last ones of a row are read to end at its end and shifted.
// (An element per thread: 2 TB/s, 69 us for 4759 rows of 7406 tokens.)
__global__ void __launch_bounds__(256)
tsvd_realign_kernel(const uint16_t* __restrict__ x, long long ldx, int B, uint16_t* __restrict__ xt, long long ldt) {
    typedef unsigned __int128 u128;
    typedef u128 u128_at __attribute__((aligned(2)));
    const int b = (blockIdx.x * 256 + threadIdx.x) * 8;
    const uint16_t* row = x + (size_t)blockIdx.y * ldx;
    if (b >= ldt) return;
    u128 v = 0;
    if (B >= 8) {
        const int first = min(b, B - 8);
        v = *reinterpret_cast<const u128_at*>(row + first) >> (16 * (b - first));
    } else {
        for (int e = 0; e < B; ++e) v |= (u128)row[e] << (16 * e);
    }
    *reinterpret_cast<u128*>(xt + (size_t)blockIdx.y * ldt + b) = v;
}

// One-time, per-device setup (the device is current): kernel attributes, address of the static workspace.
hipError_t device_init(int device) {
    static bool done[64] = {};
    if (device < 0 || device >= 64) return hipErrorInvalidDevice;
    if (done[device]) return hipSuccess;
    void* sp = nullptr;
    hipError_t e = hipGetSymbolAddress(&sp, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!sp || (reinterpret_cast<uintptr_t>(sp) & 255u)) return hipErrorInvalidSymbol;
    noalloc_ptr[device] = sp;
    e = tsvd_skinny_init();
    if (e != hipSuccess) return e;
    e = tsvd_gemm_init();
    if (e != hipSuccess) return e;
    e = tsvd_thin_init();
    if (e != hipSuccess) return e;
    e = tsvd_gemv_init();
    if (e != hipSuccess) return e;
    e = tsvd_mid_init();
    if (e != hipSuccess) return e;
    e = tsvd_few_init();
    if (e != hipSuccess) return e;
    e = tsvd_gemv_dense_init();
    if (e != hipSuccess) return e;
    e = tsvd_transition_init();
    if (e != hipSuccess) return e;
    done[device] = true;
    return hipSuccess;
}

// ---- skinny path (few tokens): two launches per pair of tokens --------------------------------
void shape_skinny(tsvd_skinny_args& a) {
    // LDS: digit planes [8 * tokens][slab_k + 16] bytes + reduction tiles (<= 16 KiB) + 256 B
    const size_t budget = TSVD_SKINNY_MAX_LDS - 16 * 1024 - 1024;
    const int cols = 8 * a.tokens;
    const int slab = (int)std::min<size_t>((size_t)a.nkt, (budget / (size_t)cols - 16) / 256);
    a.slab_tiles = std::max(slab, 1);
    // One workgroup of up to 16 wavefronts per compute unit when the matrix is large enough:
    // sw strips x kw contraction splits, every wavefront streaming nkt / kw tiles.
    int sw = 1;
    while (sw < 16 && a.strips / (sw * 2) >= 256) sw *= 2;
    int kw = 1;
    while (sw * kw * 2 <= 16 && kw * 2 <= a.nkt) kw *= 2;
    a.sw = std::max(1, std::min(16, env_int("TSVD_SKINNY_SW", sw)));
    a.kw = std::max(1, std::min(std::min(16 / a.sw, a.nkt), env_int("TSVD_SKINNY_KW", kw)));
}

// Tokens that the single-token kernels take in one launch (planes of z: 2 MiB at most, K being at most 16384 there).
int gemv_tokens(const tsvd_handle* h, int64_t B) {
    return tsvd_gemv_fits(h->hd.Np, h->hd.Kp) ? (int)std::min<int64_t>(B, TSVD_GEMV_MAX_TOKENS) : 1;
}
size_t skinny_workspace(const tsvd_handle* h, int64_t B) {
    return 256 + (size_t)std::max(16, 8 * gemv_tokens(h, B)) * (size_t)h->hd.Kp;      // exponents, then digit planes of Kp bytes: 8 per token
}

int pow2_ceil(int64_t v) {
    int r = 1;
    while (r < v) r *= 2;
    return r;
}
int pow2_floor(int64_t v) {
    int r = 1;
    while ((int64_t)r * 2 <= v) r *= 2;
    return r;
}

// What decides whether tokens side by side run in one launch (tsvd_gemv_fused_fits), the rest zero.
tsvd_gemv_fused_args gemv_fused_sizes(const tsvd_blob_header& hd, int tokens) {
    tsvd_gemv_fused_args f;
    std::memset(&f, 0, sizeof f);
    f.strips_v = (int)((hd.K + 127) / 128 * 8); f.nkt_v = (int)(hd.Np / 256);
    f.strips_u = (int)((hd.M + 15) / 16); f.nkt_u = (int)(hd.Kp / 256);
    f.N = (int)hd.N; f.Np = (int)hd.Np; f.Kp = (int)hd.Kp; f.M = (int)hd.M;
    f.tokens = tokens;
    return f;
}
// One token through the tsvd_gemv kernels; returns false if the shape does not fit them.
// tokens: each on workgroups of its own, x_token and y_token elements from one to the next
bool try_gemv(const tsvd_handle* h, const void* x, tsvd_dtype x_dtype, int64_t ldx, int tokens, int64_t x_token, void* y, int64_t ldy,
              int64_t y_token, const out_opts& oo, int* meta, unsigned char* planes, hipStream_t stream, tsvd_status* st) {
    const tsvd_blob_header& hd = h->hd;
    if (env_int("TSVD_GEMV", 1) == 0 || !tsvd_gemv_fits(hd.Np, hd.Kp)) return false;
    const int mask = tsvd_stage_mask();
    // (16 bytes of fp32, 8 of bf16 at a time)
    const bool vec = ldx == 1 && hd.N % 4 == 0 && (reinterpret_cast<uintptr_t>(x) & 15u) == 0 && (tokens == 1 || x_token % 4 == 0);
    if (mask == 7 && !h->dense_u && env_int("TSVD_GEMV_FUSED", 1) != 0) {
        // a small V: both stages in one launch
        tsvd_gemv_fused_args f = gemv_fused_sizes(hd, tokens);
        f.tiles_v = h->blob + hd.off_V;
        f.tiles_u = h->blob + hd.off_U;
        f.x = x; f.x_is_bf16 = x_dtype == TSVD_BF16; f.ldx = ldx;
        f.x_vec = vec;
        f.x_token = x_token; f.y_token = y_token;
        f.S = reinterpret_cast<const float*>(h->blob + hd.off_S);
        f.bound_V = h->bound_V;
        f.y = y; f.ldy = ldy; f.bias = oo.bias; f.out_bf16 = oo.out_bf16;
        if (tsvd_gemv_fused_fits(f, h->cu_count)) {
            *st = tsvd_launch_gemv_fused(f, h->cu_count, stream) == hipSuccess ? TSVD_OK : TSVD_EDEVICE;
            return true;
        }
    }
    if (mask == 7 && tokens == 1 && h->sync && !h->dense_u && env_int("TSVD_GEMV_ONEPASS", 0) != 0) {
        // both stages in one launch (z handed over between workgroups through the handle's tagged buffer)
        tsvd_handle* hm = const_cast<tsvd_handle*>(h);
        int expected = 0;
        if (hm->sync_claimed.compare_exchange_strong(expected, 1)) hm->sync_stream = stream;
        tsvd_gemv_onepass_args f;
        std::memset(&f, 0, sizeof f);
        if (hm->sync_stream == (void*)stream && tsvd_gemv_onepass_shape(hd.M, hd.Mp, hd.Kp, hd.Np, h->cu_count, &f)) {
            f.tiles_v = h->blob + hd.off_V;
            f.tiles_u = h->blob + hd.off_U;
            f.N = (int)hd.N; f.Np = (int)hd.Np; f.Kp = (int)hd.Kp; f.M = (int)hd.M;
            f.x = x; f.x_is_bf16 = x_dtype == TSVD_BF16; f.ldx = ldx;
            f.x_vec = vec;
            f.S = reinterpret_cast<const float*>(h->blob + hd.off_S);
            f.bound_V = h->bound_V;
            f.counter = reinterpret_cast<unsigned*>(h->sync);
            f.zbuf = reinterpret_cast<unsigned long long*>(h->sync + 256);
            f.spin_limit = env_int("TSVD_SPIN_LIMIT", 256);
            f.y = y; f.ldy = ldy; f.bias = oo.bias; f.out_bf16 = oo.out_bf16;
            f.clocks = h->clocks;
            *st = tsvd_launch_gemv_onepass(f, stream) == hipSuccess ? TSVD_OK : TSVD_EDEVICE;
            return true;
        }
    }
    // sw strips x kw splits = 16 wavefronts, strips so that no compute unit gets a second workgroup: every workgroup stages its token's
    // planes first, and the second would start with that when the first is done (measured: 12175 x 149 x 7168 15.8 us with two strips,
    // 12.2 with four; 15 tokens of 5290 x 285 x 3200 54 us with one, 17 with sixteen).  Where few splits are possible four strips at least:
    // with 256 columns a workgroup of one strip has one wavefront with work (7978 x 128 x 109: 9.0 -> 7.8 us).
    auto shape = [&](tsvd_gemv_args& a) {
        auto splits = [&](int sw) {
            int kl = 0;
            while ((sw << (kl + 1)) <= 16 && (2 << kl) <= a.nkt) ++kl;
            return kl;
        };
        int sw = 1;
        while (sw < 16 && (long long)((a.strips + sw - 1) / sw) * tokens > h->cu_count) sw *= 2;
        while ((sw << splits(sw)) < 4) sw *= 2;
        a.sw = std::max(1, std::min(16, env_int("TSVD_GEMV_SW", sw)));
        a.kw_log2 = std::max(0, env_int("TSVD_GEMV_KWLOG2", splits(a.sw)));
        while ((a.sw << a.kw_log2) > 16) --a.kw_log2;
    };
    tsvd_gemv_args a;
    std::memset(&a, 0, sizeof a);
    a.N = (int)hd.N; a.Np = (int)hd.Np; a.Kp = (int)hd.Kp;
    a.meta = meta;
    a.tokens = tokens; a.x_token = x_token; a.y_token = y_token;
    a.clocks = h->clocks;
    a.early_tiles = env_int("TSVD_EARLY_TILES", 1);
    if (mask & 2) {
        a.tiles = h->blob + hd.off_V;
        a.strips = (int)(hd.Kp / 16);
        a.nkt = (int)(hd.Np / 256);
        a.rows_out = (int)hd.Kp;
        a.x = x;
        a.x_is_bf16 = x_dtype == TSVD_BF16;
        a.ldx = ldx;
        a.x_vec = vec;
        a.S = reinterpret_cast<const float*>(h->blob + hd.off_S);
        a.bound_V = h->bound_V;
        a.planes_out = planes;
        shape(a);
        if (tsvd_launch_gemv(a, false, stream) != hipSuccess) {
            *st = TSVD_EDEVICE;
            return true;
        }
    }
    if ((mask & 4) && h->dense_u && tsvd_gemv_dense_lds(hd.Kp) <= TSVD_SKINNY_MAX_LDS) {
        tsvd_gemv_dense_args d;
        std::memset(&d, 0, sizeof d);
        d.dense = h->dense_u;
        d.groups = (int)((hd.Mp / 16 + 4) / 5);
        d.nkt = (int)(hd.Kp / 256);
        d.Kp = (int)hd.Kp; d.M = (int)hd.M;
        d.planes_in = planes; d.meta = meta;
        d.y = y; d.ldy = ldy; d.bias = oo.bias; d.out_bf16 = oo.out_bf16;
        *st = tsvd_launch_gemv_dense(d, stream) == hipSuccess ? TSVD_OK : TSVD_EDEVICE;
        return true;
    }
    if (mask & 4) {
        a.tiles = h->blob + hd.off_U;
        a.strips = (int)((hd.M + 15) / 16);
        a.nkt = (int)(hd.Kp / 256);
        a.rows_out = (int)hd.M;
        a.planes_in = planes;
        a.y = y;
        a.ldy = ldy;
        a.bias = oo.bias;
        a.out_bf16 = oo.out_bf16;
        shape(a);
        if (tsvd_launch_gemv(a, true, stream) != hipSuccess) {
            *st = TSVD_EDEVICE;
            return true;
        }
    }
    *st = TSVD_OK;
    return true;
}

// x_token_major: only for calls that gemv_serves
bool gemv_serves(const tsvd_handle* h) { return tsvd_gemv_fits(h->hd.Np, h->hd.Kp) && env_int("TSVD_GEMV", 1) != 0; }
double code_bytes(const tsvd_handle* h) { return (double)h->hd.Kp * (double)(h->hd.Mp + h->hd.Np) / 4.0; }
// 2 - 16 bf16 tokens whose z is kept as in fp32 (side by side on the single-token kernels, or on five planes of the few-token kernels): up to
// 60 MB of code words times tokens.  Beyond, side by side takes longer than z in four planes (0.15 us for every MB and token).
bool z_as_fp32(const tsvd_handle* h, int64_t B, tsvd_dtype x_dtype) {
    return x_dtype == TSVD_BF16 && B >= 2 && B <= 16 && !tsvd_tuning_any() && !h->dense_u && gemv_serves(h) && (double)B * code_bytes(h) <= 60.0e6;
}
// Small factors on five planes, 1 to 16 tokens alike (a token's result does not depend on how many stand beside it): up to 512 ranks and 1 MB of code
// words, and not the smallest (the last lines).  Measured against side by side on 30 such factors: 2 to 8 tokens 0.87 of the time,
// 16 tokens 0.80; at 640 to 2500 ranks one token would take 1.04 .. 1.2 times as long.  One token beyond 768 padded rows is no faster here: two launches, where the
// single-token kernels have one since V is small (36 factors of 769 to 8000 rows: 4.1 to 8.1 us there, 7.4 to 8.1 here, 0.64 of the time on the average).  It stays for its bits,
// the same beside any number of tokens, and its error: against 64 bits 5e-8 to 1.3e-7 of the norm of y, side by side 1e-7 to 4e-6;
// and on rows that avoid features 20 to 30000 times the rest, or where such features cancel, a tenth to a thousandth of that of the integers side by
// side, whose grid is 2^-31 of the largest sum that could be.  (The factors of up to 768 padded rows and 64 tiles a stage, where one workgroup took a token
// fastest when the line was drawn, keep the single-token kernels and with them their bits.)
bool five_planes(const tsvd_handle* h) {
    const tsvd_blob_header& hd = h->hd;
    return !h->dense_u && hd.Kp <= 512 && code_bytes(h) <= 1.0e6 && (!tsvd_gemv_one_workgroup(hd.Mp, hd.Kp, hd.Np) || hd.Mp > 768);
}
// The planes of z of a call of up to 16 tokens on the few-token kernels (0: on others).
int few_planes(const tsvd_handle* h, int64_t B, tsvd_dtype x_dtype, int64_t ldx, bool x_token_major) {
    const tsvd_blob_header& hd = h->hd;
    // (Kp: the records, 50 or 64 bytes a rank, have to fit the fixed workspace of tsvd_forward_noalloc by themselves)
    if (x_dtype != TSVD_BF16 || B > 16 || hd.Kp > (1 << 18) || !tsvd_few_fits(hd, B, ldx, x_token_major)) return 0;
    if (tsvd_tuning_any()) return B <= env_int("TSVD_FEW", 0) ? (env_int("TSVD_FEW_PLANES", 4) == 5 ? 5 : 4) : 0;
    if (five_planes(h)) return 5;
    return B == 1 || z_as_fp32(h, B, x_dtype) ? 0 : 4;
}
tsvd_status forward_skinny(const tsvd_handle* h, const void* x, tsvd_dtype x_dtype, int64_t B, int64_t ldx, bool x_token_major,
                           void* y, int64_t ldy, const out_opts& oo, void* ws, hipStream_t stream) {
    const size_t yelt = oo.out_bf16 ? 2 : 4;
    const tsvd_blob_header& hd = h->hd;
    int* meta = static_cast<int*>(ws);
    unsigned char* planes = static_cast<unsigned char*>(ws) + 256;
    const size_t xelt = x_dtype == TSVD_BF16 ? 2 : 4;
    const int mask = tsvd_stage_mask();
    if (gemv_serves(h)) {
        // tokens side by side through the single-token kernels (each reads the weights; stage U on the denser code: one at a time)
        const int step = h->dense_u ? 1 : gemv_tokens(h, B);
        const int64_t x_token = x_token_major ? ldx : 1, y_token = oo.token_major ? ldy : 1;
        for (int64_t b0 = 0; b0 < B; b0 += step) {
            tsvd_status gst = TSVD_OK;
            // one token's output: column b of y [M][ldy], or row b of y [B][ldy] (then consecutive in memory)
            if (!try_gemv(h, static_cast<const uint8_t*>(x) + (size_t)(b0 * x_token) * xelt, x_dtype, x_token_major ? 1 : ldx,
                          (int)std::min<int64_t>(step, B - b0), x_token, static_cast<uint8_t*>(y) + (size_t)(b0 * y_token) * yelt,
                          oo.token_major ? 1 : ldy, y_token, oo, meta, planes, stream, &gst))
                return TSVD_EUNSUPPORTED;
            if (gst != TSVD_OK) return gst;
        }
        return TSVD_OK;
    }
    for (int64_t b0 = 0; b0 < B; b0 += 2) {
        const int tokens = (int)std::min<int64_t>(2, B - b0);
        tsvd_skinny_args v;
        std::memset(&v, 0, sizeof v);
        v.tiles = h->blob + hd.off_V;
        v.strips = (int)(hd.Kp / 16);           // padded rows give z = 0: every plane byte is written
        v.nkt = (int)(hd.Np / 256);
        v.mode = TSVD_SKINNY_STAGE_V;
        v.in = static_cast<const uint8_t*>(x) + (size_t)b0 * xelt;
        v.in_is_bf16 = x_dtype == TSVD_BF16;
        v.kvalid = (int)hd.N;
        v.ld_in = ldx;
        v.tokens = tokens;
        v.rowscale = reinterpret_cast<const float*>(h->blob + hd.off_S);
        v.bound_V = h->bound_V;
        v.meta_out = meta;
        v.out = planes;
        v.ld_out = hd.Kp;
        v.rows_out = (int)hd.Kp;
        shape_skinny(v);
        if ((mask & 2) && tsvd_launch_skinny(v, stream) != hipSuccess) return TSVD_EDEVICE;

        tsvd_skinny_args u;
        std::memset(&u, 0, sizeof u);
        u.tiles = h->blob + hd.off_U;
        u.strips = (int)((hd.M + 15) / 16);
        u.nkt = (int)(hd.Kp / 256);
        u.mode = TSVD_SKINNY_STAGE_U;
        u.in = planes;
        u.ld_in = hd.Kp;
        u.tokens = tokens;
        u.meta_in = meta;
        u.out = static_cast<uint8_t*>(y) + (oo.token_major ? (size_t)b0 * (size_t)ldy : (size_t)b0) * yelt;
        u.ld_out = ldy;
        u.out_token_major = oo.token_major;
        u.rows_out = (int)hd.M;
        u.bias = oo.bias;
        u.out_bf16 = oo.out_bf16;
        shape_skinny(u);
        if ((mask & 4) && tsvd_launch_skinny(u, stream) != hipSuccess) return TSVD_EDEVICE;
    }
    return TSVD_OK;
}

// ---- slab path for few tokens: groups of up to 16 tokens of bf16 activations, two launches per group ------
// What the few-token kernels (few_planes) do not take: fewer than eight values, odd rows too far apart for them (tsvd_few_fits), and more than 2^18 ranks.
bool use_mid(const tsvd_handle* h, int64_t B, tsvd_dtype x_dtype, int64_t ldx) {
    if (x_dtype != TSVD_BF16 || B < 2 || B > 64 || env_int("TSVD_MID", 1) == 0) return false;
    // (32-bit byte offsets into x in the kernel, which also addresses up to four slabs of 2048 rows
    // beyond the last one: the range check returns zeros there)
    if (((uint64_t)h->hd.Np + 8192) * (uint64_t)ldx * 2 >= (1ull << 31)) return false;
    return B <= std::max(16, env_int("TSVD_MID_MAX_B", 16));       // (tuning switch: largest B served here, in groups of 16)
}

size_t mid_workspace(const tsvd_handle* h) {
    return 256 + (size_t)32 * (size_t)h->hd.Kp;      // per-token maxima, then z fp16 [Kp][16]
}

tsvd_status forward_mid(const tsvd_handle* h, const void* x, int64_t B, int64_t ldx, void* y, int64_t ldy,
                        const out_opts& oo, void* ws, hipStream_t stream) {
    const tsvd_blob_header& hd = h->hd;
    const int mask = tsvd_stage_mask();
    // about one workgroup of 16 wavefronts per compute unit: sw strips x kw contraction splits
    auto shape = [&](tsvd_mid_args& a) {
        int sw = 2;
        while (sw < 16 && a.strips / (sw * 2) >= h->cu_count) sw *= 2;
        int kl = 0;
        while (kl < 3 && (sw << (kl + 1)) <= 16 && (2 << kl) <= a.nkt) ++kl;
        a.sw = std::max(1, std::min(16, env_int("TSVD_MID_SW", sw)));
        a.kw_log2 = std::max(0, std::min(3, env_int("TSVD_MID_KWLOG2", kl)));
        while ((a.sw << a.kw_log2) > 16) --a.kw_log2;
    };
    for (int64_t b0 = 0; b0 < B; b0 += 16) {
    const int64_t nb = std::min<int64_t>(16, B - b0);
    tsvd_mid_args a;
    std::memset(&a, 0, sizeof a);
    a.bvalid = (int)nb;
    a.bound_V = h->bound_V;
    a.colmax = static_cast<float*>(ws);
    a.clocks = h->clocks;
    a.resident_ok = env_int("TSVD_MID_RESIDENT", 1) != 0;
    uint16_t* z = reinterpret_cast<uint16_t*>(static_cast<uint8_t*>(ws) + 256);
    if (mask & 2) {
        a.tiles = h->blob + hd.off_V;
        a.strips = (int)(hd.Kp / 16);
        a.nkt = (int)(hd.Np / 256);
        a.act = static_cast<const uint16_t*>(x) + b0;
        a.ld = ldx;
        a.kvalid = (int)hd.N;
        // extent of x, rounded up to the 4-byte granularity of the buffer range check (for odd B the
        // dword holding the last element would otherwise read as zero; it lies inside an aligned dword
        // whose first half is the caller's, so it cannot cross into an unmapped page)
        a.act_bytes = (unsigned)((((((size_t)hd.N - 1) * (size_t)ldx + (size_t)nb) * 2) + 3) & ~(size_t)3);
        a.S = reinterpret_cast<const float*>(h->blob + hd.off_S);
        a.out = z;
        a.ld_out = 16;
        a.rows_valid = (int)hd.Kp;
        shape(a);
        const bool vec = ldx % 8 == 0 && (reinterpret_cast<uintptr_t>(a.act) & 15u) == 0;
        a.pairs = ldx % 2 == 0 && (reinterpret_cast<uintptr_t>(a.act) & 3u) == 0;
        if (tsvd_launch_mid(a, false, vec, stream) != hipSuccess) return TSVD_EDEVICE;
    }
    if (mask & 4) {
        a.tiles = h->blob + hd.off_U;
        a.strips = (int)((hd.M + 15) / 16);
        a.nkt = (int)(hd.Kp / 256);
        a.act = z;
        a.ld = 16;
        a.kvalid = (int)hd.Kp;
        a.act_bytes = (unsigned)((size_t)hd.Kp * 32);
        a.S = nullptr;
        a.out = static_cast<uint8_t*>(y) + (oo.token_major ? (size_t)b0 * (size_t)ldy : (size_t)b0) * (oo.out_bf16 ? 2 : 4);
        a.ld_out = ldy;
        a.out_token_major = oo.token_major;
        a.rows_valid = (int)hd.M;
        a.bias = oo.bias;
        a.out_bf16 = oo.out_bf16;
        shape(a);
        if (tsvd_launch_mid(a, true, true, stream) != hipSuccess) return TSVD_EDEVICE;
    }
    }
    return TSVD_OK;
}

// (set for the duration of a tsvd_forward_noalloc call whose fp32 batch would not fit the fixed workspace as planes:
// such a call goes one token at a time, as every fp32 batch did before the six-plane path existed)
thread_local bool f32_one_token_at_a_time = false;

bool use_gemm(const tsvd_handle*, int64_t B, tsvd_dtype x_dtype) {
    if (x_dtype == TSVD_F32 && f32_one_token_at_a_time) return false;
    // (fp32 activations: fewer tokens are handled one at a time by the single-token kernels, each pass streaming the weights)
    const int min_b = x_dtype == TSVD_BF16 ? env_int("TSVD_GEMM_MIN_B", 17) : env_int("TSVD_GEMM_MIN_B_F32", 17);
    return B >= min_b;
}

// (set for the duration of a tsvd_forward_noalloc call whose planes would not fit the fixed workspace where z in 16 bits does)
thread_local bool planes_only_by_older_rules = false;

// How a batched call runs that the few-token kernels leave.  copies: x would have to be copied for the kernels that read aligned
// feature-major rows.
tsvd_batch_call batch_call(const tsvd_handle* h, int64_t B, tsvd_dtype x_dtype, bool x_token_major, bool copies, bool y_token_major, bool out_bf16,
                           bool x_aligned, bool few) {
    tsvd_batch_call c = {};
    c.M = h->hd.M; c.K = h->hd.K; c.N = h->hd.N; c.B = B; c.cus = h->cu_count;
    c.f32 = x_dtype == TSVD_F32;
    c.x_token_major = x_token_major; c.y_token_major = y_token_major; c.out_bf16 = out_bf16; c.copies = copies;
    c.whole = tsvd_stage_mask() == 7;
    c.x_aligned = x_aligned;
    c.few = few && !c.f32 && !planes_only_by_older_rules;
    return c;
}
tsvd_batch_plan batch_plan(const tsvd_batch_call& c) {
    tsvd_batch_plan plan = tsvd_plan_batch(c);
    if (planes_only_by_older_rules && !c.f32) plan.split = false;
    return plan;
}

size_t gemm_workspace(const tsvd_handle* h, int64_t B, tsvd_dtype x_dtype) {
    const int64_t Bp = tsvd_round_up(B, 256);
    if (x_dtype == TSVD_F32) return tsvd_gemm_split_bytes(h->hd.K, h->hd.N, B, true);
    // partial column maxima [PARTS][Bp] fp32, then Z as fp16 [Kp][Bp]
    size_t bytes = round256((size_t)(TSVD_COLMAX_PARTS + 1) * Bp * 4) + round256((size_t)h->hd.Kp * (size_t)Bp * 2);
    // (the rule is asked as for aligned rows: a caller with unaligned rows then reserves a little too much)
    if (tsvd_gemm_use_fp6(h->hd.Mp, h->hd.Kp, h->hd.Np, B, h->cu_count, true))      // planes of Z, and of X for stage V
        bytes += round256(tsvd_gemm_fp6_bytes(h->hd.Kp, Bp)) +
                 round256(tsvd_gemm_fp6_bytes((tsvd_gemm_x_twice(h->hd.Mp, h->hd.Kp, h->hd.Np, B, h->cu_count) ? 2 : 1) * h->hd.Np, Bp));
    // (asked as for the call that favours planes most)
    if (use_gemm(h, B, x_dtype) && !planes_only_by_older_rules) {
        const size_t split = tsvd_gemm_split_bytes(h->hd.K, h->hd.N, B, false);
        if (split > bytes && tsvd_batch_may_split(batch_call(h, B, x_dtype, false, true, false, false, true, false))) bytes = split;
    }
    return bytes;
}

}  // namespace

extern "C" tsvd_status tsvd_pack(const int8_t* U, const float* S, const int8_t* V, int64_t M, int64_t K,
                                 int64_t N, void* dev_buf, size_t dev_buf_bytes, tsvd_handle** out) {
    if (!U || !S || !V || !out) return TSVD_EINVAL;
    const size_t bytes = tsvd_packed_bytes(M, K, N);
    if (bytes == 0) return TSVD_EINVAL;
    if (dev_buf && (dev_buf_bytes < bytes || (reinterpret_cast<uintptr_t>(dev_buf) & 255u))) return TSVD_EINVAL;

    void* host = std::malloc(bytes);
    if (!host) return TSVD_ENOMEM;
    tsvd_status st = tsvd_pack_host(U, S, V, M, K, N, host, bytes);
    if (st != TSVD_OK) {
        std::free(host);
        return st;
    }
    tsvd_handle* h = new (std::nothrow) tsvd_handle();
    if (!h) {
        std::free(host);
        return TSVD_ENOMEM;
    }
    std::memcpy(&h->hd, host, sizeof h->hd);
    // bound on |z_k| / max|x|, used to scale the fp16 intermediate of the batched path
    double bound = 0.0;
    for (int64_t k = 0; k < K; ++k) {
        int64_t nz = 0;
        const int8_t* row = V + k * N;
        for (int64_t n = 0; n < N; ++n) nz += row[n] != 0;
        bound = std::max(bound, std::fabs((double)S[k]) * (double)nz);
    }
    h->bound_V = (float)bound;
    h->scratch = nullptr;
    h->scratch_bytes = 0;
    h->retired_count = 0;
    h->clocks = nullptr;
    h->cu_count = 256;
    h->sync = nullptr;
    h->dense_u = nullptr;
    h->sync_claimed.store(0);
    h->sync_stream = nullptr;

    bool ok = hipGetDevice(&h->device) == hipSuccess && device_init(h->device) == hipSuccess;
    if (ok) {
        if (dev_buf) {
            h->blob = static_cast<uint8_t*>(dev_buf);
            h->owns_blob = false;
        } else {
            void* d = nullptr;
            ok = tsvd_device_malloc(&d, bytes) == hipSuccess;
            h->blob = static_cast<uint8_t*>(d);
            h->owns_blob = ok;
        }
    }
    if (ok) ok = hipMemcpy(h->blob, host, bytes, hipMemcpyHostToDevice) == hipSuccess;
    if (ok) {
        {
            int cus = 0;
            if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, h->device) == hipSuccess && cus > 0)
                h->cu_count = cus;
            if (env_int("TSVD_GEMV_ONEPASS", 0) != 0 && tsvd_gemv_onepass_shape(h->hd.M, h->hd.Mp, h->hd.Kp, h->hd.Np, h->cu_count, nullptr)) {
                // hand-over buffer of the one-launch single-token path (small: 8 bytes per rank index)
                const size_t sb = 256 + (size_t)h->hd.Kp * 8;
                void* d = nullptr;
                const unsigned one = 1u;
                ok = tsvd_device_malloc(&d, sb) == hipSuccess;
                if (ok) {
                    h->sync = static_cast<uint8_t*>(d);
                    ok = hipMemset(d, 0, sb) == hipSuccess && hipMemcpy(d, &one, sizeof one, hipMemcpyHostToDevice) == hipSuccess;
                }
            }
            if (ok && env_int("TSVD_DENSE_U", 0) != 0) {
                // measurement switch: a second copy of U in the denser code, used by stage U of single-token calls
                const size_t db = tsvd_dense_bytes(M, K);
                void* hostd = std::malloc(db);
                void* d = nullptr;
                ok = hostd && tsvd_device_malloc(&d, db) == hipSuccess;
                if (ok) {
                    tsvd_internal_dense_from_blob(host, hostd);
                    h->dense_u = static_cast<uint8_t*>(d);
                    ok = hipMemcpy(d, hostd, db, hipMemcpyHostToDevice) == hipSuccess;
                }
                std::free(hostd);
            }
            if (ok && env_int("TSVD_CLOCKS", 0)) {
                void* c = nullptr;
                if (tsvd_device_malloc(&c, TSVD_GEMV_MAX_GRID * 16 * sizeof(long long)) == hipSuccess) {
                    (void)hipMemset(c, 0, TSVD_GEMV_MAX_GRID * 16 * sizeof(long long));
                    h->clocks = static_cast<long long*>(c);
                }
            }
        }
    }
    std::free(host);
    if (!ok) {
        if (h->owns_blob && h->blob) (void)hipFree(h->blob);
        if (h->sync) (void)hipFree(h->sync);
        if (h->dense_u) (void)hipFree(h->dense_u);
        delete h;
        (void)hipGetLastError();
        return TSVD_EDEVICE;
    }
    *out = h;
    return TSVD_OK;
}

extern "C" tsvd_status tsvd_unpack(const tsvd_handle* h, int8_t* U, float* S, int8_t* V) {
    if (!h) return TSVD_EINVAL;
    const size_t bytes = (size_t)h->hd.total_bytes;
    void* host = std::malloc(bytes);
    if (!host) return TSVD_ENOMEM;
    if (hipMemcpy(host, h->blob, bytes, hipMemcpyDeviceToHost) != hipSuccess) {
        std::free(host);
        return TSVD_EDEVICE;
    }
    tsvd_status st = tsvd_unpack_host(host, bytes, U, S, V, nullptr, nullptr, nullptr);
    std::free(host);
    return st;
}

extern "C" tsvd_status tsvd_info(const tsvd_handle* h, int64_t* M, int64_t* K, int64_t* N, int64_t* nnzU,
                                 int64_t* nnzV) {
    if (!h) return TSVD_EINVAL;
    if (M) *M = h->hd.M;
    if (K) *K = h->hd.K;
    if (N) *N = h->hd.N;
    if (nnzU) *nnzU = h->hd.nnzU;
    if (nnzV) *nnzV = h->hd.nnzV;
    return TSVD_OK;
}

namespace {
// What the few-token kernels on planes take, where a call may go to them and it is more than `others`: they read x in place, so this is not beside a copy of x.
size_t few_workspace(const tsvd_handle* h, int64_t B, tsvd_dtype x_dtype, size_t others) {
    if (x_dtype != TSVD_BF16) return 0;
    if (B <= 16) return h->hd.Kp <= (1 << 18) ? round256(tsvd_few_bytes(h->hd.Kp, B, five_planes(h) || tsvd_tuning_any() ? 5 : 4)) : 0;
    const size_t bytes = round256(tsvd_few_bytes(h->hd.Kp, B, 4));
    // (asked as for the call that favours them most: token-major y costs the panels more)
    return use_gemm(h, B, x_dtype) && bytes > others && batch_plan(batch_call(h, B, x_dtype, true, true, true, true, true, true)).few ? bytes : 0;
}
// ... and all other kernels (which of them a call takes depends on the row stride too: cover every candidate).
size_t base_workspace(const tsvd_handle* h, int64_t B, tsvd_dtype x_dtype) {
    const size_t few = round256(std::max(skinny_workspace(h, B), mid_workspace(h)));
    if (use_gemm(h, B, x_dtype)) return std::max(gemm_workspace(h, B, x_dtype), B <= 64 ? few : (size_t)0);
    return few;
}
// (whether a call of few tokens may copy rows that start at odd elements: for the sizes whose workspace stays small.  The slab kernel gains by it, which
// without switches serves what tsvd_few_fits leaves: rows too far apart for 32-bit places, and fewer than eight values)
bool realigns_few(const tsvd_handle* h, int64_t B, tsvd_dtype x_dtype) { return x_dtype == TSVD_BF16 && B > 1 && B <= 16 && h->hd.N <= 65535 && h->hd.Kp <= 65536; }
// feature-major copy of token-major activations: [N][B rounded up to 8] elements
size_t transposed_bytes(const tsvd_handle* h, int64_t B, tsvd_dtype x_dtype) {
    return round256((size_t)h->hd.N * (size_t)tsvd_round_up(B, 8) * (x_dtype == TSVD_BF16 ? 2 : 4));
}
}  // namespace

extern "C" size_t tsvd_workspace_bytes_ex(const tsvd_handle* h, int64_t B, tsvd_dtype x_dtype, tsvd_layout x_layout) {
    if (!h || B <= 0 || (x_dtype != TSVD_F32 && x_dtype != TSVD_BF16)) return 0;
    if (x_layout != TSVD_FEATURE_MAJOR && x_layout != TSVD_TOKEN_MAJOR) return 0;
    // (feature-major rows that are not 16-byte aligned are copied too, when the call goes to the batched kernels:
    // the alignment is not known here, so the room is always there)
    const bool copy = x_layout == TSVD_TOKEN_MAJOR || use_gemm(h, B, x_dtype) || realigns_few(h, B, x_dtype);
    const size_t others = base_workspace(h, B, x_dtype) + (copy ? transposed_bytes(h, B, x_dtype) : 0);
    return std::max(others, few_workspace(h, B, x_dtype, others));
}

extern "C" size_t tsvd_workspace_bytes(const tsvd_handle* h, int64_t B, tsvd_dtype x_dtype) {
    return tsvd_workspace_bytes_ex(h, B, x_dtype, TSVD_FEATURE_MAJOR);
}

extern "C" tsvd_status tsvd_forward_ex(const tsvd_handle* h, const void* x_dev, tsvd_dtype x_dtype, tsvd_layout x_layout,
                                       int64_t B, int64_t ldx, const float* bias_dev, void* y_dev, tsvd_dtype y_dtype,
                                       int64_t ldy, void* workspace, size_t workspace_bytes, void* stream) {
    return tsvd_forward_io(h, x_dev, x_dtype, x_layout, B, ldx, bias_dev, y_dev, y_dtype, TSVD_FEATURE_MAJOR, ldy, workspace,
                           workspace_bytes, stream);
}

extern "C" tsvd_status tsvd_forward_io(const tsvd_handle* h, const void* x_dev, tsvd_dtype x_dtype, tsvd_layout x_layout,
                                       int64_t B, int64_t ldx, const float* bias_dev, void* y_dev, tsvd_dtype y_dtype,
                                       tsvd_layout y_layout, int64_t ldy, void* workspace, size_t workspace_bytes, void* stream) {
    if (!h || !x_dev || !y_dev || B <= 0) return TSVD_EINVAL;
    if (y_layout != TSVD_FEATURE_MAJOR && y_layout != TSVD_TOKEN_MAJOR) return TSVD_EINVAL;
    if (ldy < (y_layout == TSVD_TOKEN_MAJOR ? h->hd.M : B)) return TSVD_EINVAL;
    if (x_dtype != TSVD_F32 && x_dtype != TSVD_BF16) return TSVD_EINVAL;
    if (y_dtype != TSVD_F32 && y_dtype != TSVD_BF16) return TSVD_EINVAL;
    if (x_layout != TSVD_FEATURE_MAJOR && x_layout != TSVD_TOKEN_MAJOR) return TSVD_EINVAL;
    if (ldx < (x_layout == TSVD_TOKEN_MAJOR ? h->hd.N : B)) return TSVD_EINVAL;
    if (B > (int64_t(1) << 24)) return TSVD_EUNSUPPORTED;
    const size_t need = tsvd_workspace_bytes_ex(h, B, x_dtype, x_layout);
    void* ws = workspace;
    if (ws) {
        if (workspace_bytes < need || (reinterpret_cast<uintptr_t>(ws) & 255u)) return TSVD_EINVAL;
    } else {
        if (workspace_bytes != 0) return TSVD_EINVAL;
        tsvd_handle* hm = const_cast<tsvd_handle*>(h);
        if (hm->scratch_bytes < need) {
            // Enqueued work may still use the old buffer.  It is not freed here (hipFree would wait for the whole
            // device): it is kept until tsvd_free, and the new one is at least twice as large, so at most 16
            // buffers ever retire and their sizes sum to less than the live one.  Only when that list is full
            // does the call fall back to draining the device.
            void* d = nullptr;
            const size_t grow = std::max(need, 2 * hm->scratch_bytes);
            if (tsvd_device_malloc(&d, grow) != hipSuccess) {
                (void)hipGetLastError();
                return TSVD_EDEVICE;
            }
            if (hm->scratch) {
                if (hm->retired_count < 16) {
                    hm->retired[hm->retired_count++] = hm->scratch;
                } else {
                    if (hipDeviceSynchronize() != hipSuccess) return TSVD_EDEVICE;
                    (void)hipFree(hm->scratch);
                }
            }
            hm->scratch = d;
            hm->scratch_bytes = grow;
        }
        ws = hm->scratch;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const out_opts oo = {bias_dev, y_dtype == TSVD_BF16, y_layout == TSVD_TOKEN_MAJOR};
    if (x_layout == TSVD_TOKEN_MAJOR && B == 1) {
        // a single token is one contiguous vector in either layout: feature-major with unit row pitch, no copy
        x_layout = TSVD_FEATURE_MAJOR;
        ldx = 1;
    }
    int x_in_place = 0;
    const bool batched = use_gemm(h, B, x_dtype), misaligned = ldx % 8 != 0 || (reinterpret_cast<uintptr_t>(x_dev) & 15u);
    // rows that are not 16-byte aligned get a copy that is, where the kernels of the call do not read them in place anyway (few tokens, panels, planes
    // of x): for more than 16 tokens one pass costs less than the element-wise gathers of the ring and large-tile
    // kernels (stage V of a 4096 x 8192 factor at 300 tokens: 251 us gathered, 3 + 35 us copied), for
    // fewer, on the slab kernel (use_mid), where rows start at odd elements; TSVD_REALIGN=0 keeps the gathers
    const bool realign = x_layout == TSVD_FEATURE_MAJOR && x_dtype == TSVD_BF16 && B > 1 && env_int("TSVD_REALIGN", 1) != 0 && h->hd.N <= 65535 &&
                         (batched ? misaligned : realigns_few(h, B, x_dtype) && (ldx % 2 != 0 || (reinterpret_cast<uintptr_t>(x_dev) & 3u)));
    const int z_planes = few_planes(h, B, x_dtype, ldx, x_layout == TSVD_TOKEN_MAJOR);
    const bool few = !z_planes && !z_as_fp32(h, B, x_dtype) && use_mid(h, B, x_dtype, x_layout == TSVD_TOKEN_MAJOR || realign ? tsvd_round_up(B, 8) : ldx);
    tsvd_batch_plan plan = {};
    if (batched && !few)
        plan = batch_plan(batch_call(h, B, x_dtype, x_layout == TSVD_TOKEN_MAJOR, x_layout == TSVD_TOKEN_MAJOR || misaligned, oo.token_major, oo.out_bf16, !misaligned,
                                     tsvd_few_fits(h->hd, B, ldx, x_layout == TSVD_TOKEN_MAJOR) && tsvd_few_bytes(h->hd.Kp, B, 4) <= need));
    if (plan.split && x_dtype == TSVD_BF16 && tsvd_gemm_split_bytes(h->hd.K, h->hd.N, B, false) > need) plan.split = false;   // (never more than was asked for)
    if (z_planes || plan.few) {
        // few tokens: x in any layout and alignment, planes of z in the workspace
        const tsvd_few_problem f = {h->blob, &h->hd, static_cast<const uint16_t*>(x_dev), B, B == 1 && ldx == 1 ? h->hd.N : ldx, x_layout == TSVD_TOKEN_MAJOR || (B == 1 && ldx == 1), y_dev, ldy,
                                    oo.token_major, oo.out_bf16, bias_dev, static_cast<unsigned char*>(ws), z_planes ? z_planes : 4, h->cu_count,
                                    tsvd_stage_mask()};
        return tsvd_few_launch(f, s) == hipSuccess ? TSVD_OK : TSVD_EDEVICE;
    }
    if (plan.thin) {
        // thin token panels: one launch, x in any layout and alignment, no workspace
        tsvd_thin_problem t = {};
        t.blob = h->blob;
        t.hd = &h->hd;
        t.x = static_cast<const uint16_t*>(x_dev);
        t.source = x_layout == TSVD_TOKEN_MAJOR ? THIN_TOKEN_MAJOR : THIN_FEATURE_MAJOR;
        t.B = B;
        t.ldx = ldx;
        t.y = y_dev;
        t.ldy = ldy;
        t.bias = bias_dev;
        t.out_bf16 = oo.out_bf16;
        t.y_token_major = oo.token_major;
        t.cus = h->cu_count;
        const hipError_t te = tsvd_thin_launch(t, plan.thin, s);
        if (te != hipErrorNotSupported) return te == hipSuccess ? TSVD_OK : TSVD_EDEVICE;
    }
    if (x_layout == TSVD_TOKEN_MAJOR && (plan.split || (!batched && !few && gemv_serves(h)) || (x_dtype == TSVD_BF16 && batched && !few &&
                                                        tsvd_gemm_reads_in_place(h->hd.Mp, h->hd.Kp, h->hd.Np, B, h->cu_count)))) {
        x_in_place = 1;       // the kernels this call takes gather their operand lanes from [B][ldx] themselves
    } else if (x_layout == TSVD_TOKEN_MAJOR) {
        // one pass that rewrites x as [N][B rounded up to 8] at the front of the workspace; the rows
        // of the copy are 16-byte aligned, so every kernel family takes its fast loads
        const int64_t ldt = tsvd_round_up(B, 8);
        const dim3 grid((unsigned)((h->hd.N + 31) / 32), (unsigned)((ldt + 31) / 32));
        if (x_dtype == TSVD_BF16)
            hipLaunchKernelGGL(tsvd_transpose_kernel<uint16_t>, grid, dim3(256), 0, s, static_cast<const uint16_t*>(x_dev), ldx,
                               (int)B, (int)h->hd.N, static_cast<uint16_t*>(ws), ldt);
        else
            hipLaunchKernelGGL(tsvd_transpose_kernel<uint32_t>, grid, dim3(256), 0, s, static_cast<const uint32_t*>(x_dev), ldx,
                               (int)B, (int)h->hd.N, static_cast<uint32_t*>(ws), ldt);
        if (hipGetLastError() != hipSuccess) return TSVD_EDEVICE;
        x_dev = ws;
        ldx = ldt;
        ws = static_cast<uint8_t*>(ws) + transposed_bytes(h, B, x_dtype);
    } else if (realign && (few || (batched && !plan.split && !tsvd_gemm_reads_in_place(h->hd.Mp, h->hd.Kp, h->hd.Np, B, h->cu_count)))) {
        const int64_t ldt = tsvd_round_up(B, 8);
        hipLaunchKernelGGL(tsvd_realign_kernel, dim3((unsigned)((ldt + 2047) / 2048), (unsigned)h->hd.N), dim3(256), 0, s,
                           static_cast<const uint16_t*>(x_dev), (long long)ldx, (int)B, static_cast<uint16_t*>(ws), (long long)ldt);
        if (hipGetLastError() != hipSuccess) return TSVD_EDEVICE;
        x_dev = ws;
        ldx = ldt;
        ws = static_cast<uint8_t*>(ws) + transposed_bytes(h, B, x_dtype);
    }
    if (few) return forward_mid(h, x_dev, B, ldx, y_dev, ldy, oo, ws, s);
    if (use_gemm(h, B, x_dtype)) {
        tsvd_gemm_problem g;
        g.blob = h->blob;
        g.hd = &h->hd;
        g.bound_V = h->bound_V;
        g.x = x_dev;
        g.B = B;
        g.ldx = ldx;
        g.x_token_major = x_in_place;
        g.x_f32 = x_dtype == TSVD_F32;
        g.split = plan.split;
        g.split_v = plan.split_v;
        g.split_u = plan.split_u;
        g.y = y_dev;
        g.ldy = ldy;
        g.bias = oo.bias;
        g.out_bf16 = oo.out_bf16;
        g.y_token_major = oo.token_major;
        g.ws = ws;
        g.cu_count = h->cu_count;
        g.clocks = h->clocks;
        const hipError_t ge = tsvd_forward_gemm(g, s);
        return ge == hipSuccess ? TSVD_OK : ge == hipErrorNotSupported ? TSVD_EUNSUPPORTED : TSVD_EDEVICE;
    }
    return forward_skinny(h, x_dev, x_dtype, B, ldx, x_in_place, y_dev, ldy, oo, ws, s);
}

extern "C" tsvd_status tsvd_forward(const tsvd_handle* h, const void* x_dev, tsvd_dtype x_dtype, int64_t B,
                                    int64_t ldx, void* y_dev, tsvd_dtype y_dtype, int64_t ldy, void* workspace,
                                    size_t workspace_bytes, void* stream) {
    return tsvd_forward_ex(h, x_dev, x_dtype, TSVD_FEATURE_MAJOR, B, ldx, nullptr, y_dev, y_dtype, ldy, workspace,
                           workspace_bytes, stream);
}

extern "C" tsvd_status tsvd_forward_noalloc(const tsvd_handle* h, const void* x_dev, tsvd_dtype x_dtype, tsvd_layout x_layout,
                                            int64_t B, int64_t ldx, const float* bias_dev, void* y_dev, tsvd_dtype y_dtype,
                                            int64_t ldy, void* stream) {
    if (!h || B <= 0) return TSVD_EINVAL;
    if (x_dtype != TSVD_F32 && x_dtype != TSVD_BF16) return TSVD_EINVAL;
    if (x_layout != TSVD_FEATURE_MAJOR && x_layout != TSVD_TOKEN_MAJOR) return TSVD_EINVAL;
    if (h->device < 0 || h->device >= 64 || !noalloc_ptr[h->device]) return TSVD_EDEVICE;
    bool* const smaller = x_dtype == TSVD_F32 ? &f32_one_token_at_a_time : &planes_only_by_older_rules;
    if (tsvd_workspace_bytes_ex(h, B, x_dtype, x_layout) > (size_t)TSVD_NOALLOC_MAX_WORKSPACE) {
        // an fp32 batch whose planes do not fit can still go one token at a time (a small workspace), a bf16 batch
        // on the kernels that keep z in 16 bits
        *smaller = true;
        if (tsvd_workspace_bytes_ex(h, B, x_dtype, x_layout) > (size_t)TSVD_NOALLOC_MAX_WORKSPACE) {
            *smaller = false;
            return TSVD_ETOOLARGE;
        }
    }
    // the workspace contents are undefined on entry for every kernel family (each writes z before it
    // reads it), so nothing has to be cleared between calls
    const tsvd_status st = tsvd_forward_ex(h, x_dev, x_dtype, x_layout, B, ldx, bias_dev, y_dev, y_dtype, ldy, noalloc_ptr[h->device],
                                           (size_t)TSVD_NOALLOC_MAX_WORKSPACE, stream);
    *smaller = false;
    return st;
}

// ---- diagnostic interface (include/tsvd_tuning.h) ------------------------------------------------
namespace {
const char* const tuning_names[] = {
    "TSVD_GEMV", "TSVD_GEMV_FUSED", "TSVD_GEMV_ONEPASS", "TSVD_GEMV_SW", "TSVD_GEMV_KWLOG2", "TSVD_SKINNY_SW", "TSVD_SKINNY_KW",
    "TSVD_FEW", "TSVD_FEW_PLANES", "TSVD_FEW_KWLOG2", "TSVD_FEW_SW_V", "TSVD_FEW_SW_U", "TSVD_FEW_RW_U", "TSVD_MID", "TSVD_MID_MAX_B", "TSVD_MID_SW", "TSVD_MID_KWLOG2", "TSVD_MID_RESIDENT", "TSVD_GEMM_MIN_B", "TSVD_GEMM_MIN_B_F32",
    "TSVD_GEMM_CFG_V", "TSVD_GEMM_CFG_U", "TSVD_FUSEMAX", "TSVD_COLMAX_SCALAR", "TSVD_REALIGN", "TSVD_PANEL",
    "TSVD_PANEL_WAVES", "TSVD_PANEL_FP6", "TSVD_FP6", "TSVD_FP6_V", "TSVD_FP6_TALL", "TSVD_FP6_PLANES", "TSVD_FP6_DIRECT", "TSVD_FP6_TAIL", "TSVD_SPLIT_V", "TSVD_SPLIT_U", "TSVD_SPLIT_X", "TSVD_THIN", "TSVD_TOKEN_MAJOR_COPY", "TSVD_GROUPED_PAIR", "TSVD_DEPTHWISE", "TSVD_CLOCKS",
    "TSVD_SPIN_LIMIT", "TSVD_DENSE_U", "TSVD_EARLY_TILES", "TSVD_TRANSITION_SHIFTED"};
constexpr int tuning_count = (int)(sizeof tuning_names / sizeof tuning_names[0]);
int tuning_value[tuning_count];
bool tuning_is_set[tuning_count];
int tuning_active = 0;                 // number of switches set: 0 in every process that never calls tsvd_tuning_set
thread_local int stage_mask_now = 7;
}  // namespace

bool tsvd_tuning_any() { return tuning_active != 0; }
int tsvd_tune(const char* name, int fallback) {
    if (tuning_active == 0) return fallback;
    for (int i = 0; i < tuning_count; ++i)
        if (tuning_is_set[i] && std::strcmp(name, tuning_names[i]) == 0) return tuning_value[i];
    return fallback;
}
int tsvd_stage_mask() { return stage_mask_now; }

extern "C" int tsvd_tuning_set(const char* name, int value) {
    if (!name) return 1;
    for (int i = 0; i < tuning_count; ++i)
        if (std::strcmp(name, tuning_names[i]) == 0) {
            if (!tuning_is_set[i]) ++tuning_active;
            tuning_is_set[i] = true;
            tuning_value[i] = value;
            return 0;
        }
    return 1;
}

extern "C" void tsvd_tuning_reset(void) {
    for (int i = 0; i < tuning_count; ++i) tuning_is_set[i] = false;
    tuning_active = 0;
}

extern "C" tsvd_status tsvd_tuning_forward_stages(const tsvd_handle* h, const void* x_dev, tsvd_dtype x_dtype, tsvd_layout x_layout,
                                                  int64_t B, int64_t ldx, const float* bias_dev, void* y_dev, tsvd_dtype y_dtype,
                                                  int64_t ldy, void* workspace, size_t workspace_bytes, void* stream, int stage_mask) {
    if (stage_mask < 1 || stage_mask > 7) return TSVD_EINVAL;
    stage_mask_now = stage_mask;
    const tsvd_status st = tsvd_forward_ex(h, x_dev, x_dtype, x_layout, B, ldx, bias_dev, y_dev, y_dtype, ldy, workspace,
                                           workspace_bytes, stream);
    stage_mask_now = 7;
    return st;
}

extern "C" int tsvd_tuning_tile_shapes(const tsvd_handle* h, long long B, int* shape_v, int* shape_u) {
    if (!h || !shape_v || !shape_u || B < 1) return 1;
    *shape_v = *shape_u = -1;
    if (B <= 16 || use_mid(h, B, TSVD_BF16, tsvd_round_up(B, 8))) return 0;
    if (use_gemm(h, B, TSVD_BF16)) {
        const tsvd_batch_plan plan = batch_plan(batch_call(h, B, TSVD_BF16, false, false, false, false, true, true));
        if (plan.few) return 0;
        if (plan.thin) {
            *shape_v = *shape_u = 34;
        } else if (plan.split) {
            *shape_v = plan.split_v ? 100 + plan.split_v : 40;
            *shape_u = plan.split_u ? 100 + plan.split_u : 40;
        } else if (tsvd_gemm_use_panel(h->hd.Mp, h->hd.Kp, h->hd.Np, B, h->cu_count, true)) {
            *shape_v = *shape_u = tsvd_gemm_panel_fp6() ? 33 : 32;   // one token-panel launch (33: on fp4 codes x fp6 planes)
        } else {
            *shape_v = tsvd_gemm_tile_shape(h->hd.Kp, B, h->cu_count, true);
            *shape_u = tsvd_gemm_tile_shape(h->hd.Mp, B, h->cu_count, true);
            if (tsvd_gemm_use_fp6(h->hd.Mp, h->hd.Kp, h->hd.Np, B, h->cu_count, true)) *shape_u = 40;   // fp4 x fp6 planes
            if (tsvd_gemm_use_fp6_v(h->hd.Mp, h->hd.Kp, h->hd.Np, B, h->cu_count, true)) *shape_v = 40;
        }
    }
    return 0;
}

extern "C" int tsvd_tuning_one_launch(const tsvd_handle* h, long long B) {
    if (!h || B < 1 || !gemv_serves(h) || h->dense_u || env_int("TSVD_GEMV_FUSED", 1) == 0) return 0;
    return tsvd_gemv_fused_fits(gemv_fused_sizes(h->hd, (int)std::min<long long>(gemv_tokens(h, B), B)), h->cu_count);
}

extern "C" int tsvd_tuning_split_tiles(const tsvd_handle* h, long long B, tsvd_dtype x_dtype, int* v, int* u) {
    if (!h || !v || !u || B < 1 || !use_gemm(h, B, x_dtype)) return 1;
    const tsvd_batch_plan plan = batch_plan(batch_call(h, B, x_dtype, false, false, false, false, true, true));
    if (!plan.split) return 1;
    *v = plan.split_v, *u = plan.split_u;
    return 0;
}

extern "C" int tsvd_tuning_tiles_by_xcd(const tsvd_handle* h, long long B, tsvd_dtype x_dtype, int* v, int* u) {
    if (!h || !v || !u || B < 1 || !use_gemm(h, B, x_dtype)) return 1;
    const tsvd_batch_plan plan = batch_plan(batch_call(h, B, x_dtype, false, false, false, false, true, true));
    if (!plan.split) return 1;
    const long long nvb = (h->hd.N + 127) / 128, nub = (h->hd.K + 127) / 128, sets = x_dtype == TSVD_F32 ? 2 : 1;
    const bool own_x = tsvd_fp6_split_makes_x(plan.split_v, (int)std::min(sets * nvb, 1ll << 20)) && env_int("TSVD_SPLIT_X", 1) != 0;
    *v = plan.split_v && !own_x && tsvd_fp6_split_placed(plan.split_v, {128 * nub, B, sets * nvb, nvb, h->cu_count});
    *u = plan.split_u && tsvd_fp6_split_placed(plan.split_u, {h->hd.M, B, sets * nub, nub, h->cu_count});
    return 0;
}

const uint8_t* tsvd_internal_blob(const tsvd_handle* h, const tsvd_blob_header** hd) {
    *hd = &h->hd;
    return h->blob;
}

int tsvd_internal_cu_count(const tsvd_handle* h) { return h->cu_count; }

extern "C" int tsvd_tuning_read_clocks(const tsvd_handle* h, long long* out, int workgroups) {
    if (!h || !h->clocks || !out || workgroups < 1 || workgroups > TSVD_GEMV_MAX_GRID) return 1;
    return hipMemcpy(out, h->clocks, (size_t)workgroups * 16 * sizeof(long long), hipMemcpyDeviceToHost) == hipSuccess ? 0 : 4;
}

extern "C" void tsvd_free(tsvd_handle* h) {
    if (!h) return;
    if (h->scratch) (void)hipFree(h->scratch);
    for (int r = 0; r < h->retired_count; ++r) (void)hipFree(h->retired[r]);
    if (h->clocks) (void)hipFree(h->clocks);
    if (h->sync) (void)hipFree(h->sync);
    if (h->dense_u) (void)hipFree(h->dense_u);
    if (h->owns_blob && h->blob) (void)hipFree(h->blob);
    delete h;
}
