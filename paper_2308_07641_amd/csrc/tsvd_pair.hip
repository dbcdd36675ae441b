// Leading singular pair of an fp64 matrix R [M][N] by repeated squaring of its Gram matrix.
//
// With A the Gram matrix on the shorter side (R^T R or R R^T, n = min(M, N)), A^(2^p) tends to the projector onto the
// leading singular direction: p squarings are 2^p power steps.  On the close singular values of a random matrix (gaps of
// 1e-2 .. 1e-4) that takes 10 .. 18 launches that fill the chip, where Lanczos bidiagonalisation takes 60 .. 100 steps
// of four launches each, two of them a single workgroup: 2.5 ms against 0.16 ms for the pair of a [512, 256] Laplace
// matrix (64 steps at 39 us; 11 squarings at 5.2 us in a kernel trace, and 0.1 ms of launches and waits).  Rounding: every squaring perturbs its matrix by a few units in the last place of its norm, so the
// vector is off by rounding over the gap, as with any backward-stable method.
//
// The result is X x_j, with x_j the column of X that has the largest diagonal entry (to nine bits): that entry is at least trace / n, so
// its unit vector e_j has a cosine of at least 1 / sqrt(n) with the leading space whatever the matrix (a fixed vector, as the start
// vector of the Lanczos process, may be orthogonal to it), and the product with X takes the rounding of x_j back to that
// of X itself.  In a degenerate leading space that is one of its vectors.
// The sign is the one with a positive product with the start vector of the Lanczos process, which is also the sign that
// process gives (its tridiagonal matrix has positive off-diagonal entries, its leading eigenvector entries of one sign).
#include "tsvd_pair.h"

#include <algorithm>
#include <cmath>

#include "tsvd_wave.h"

namespace {

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

size_t round256(size_t v) { return (v + 255) & ~(size_t)255; }

// Shorter side up to which the squarings are taken.  A squaring is n^3 multiplications, a Lanczos step two passes over R; how many
// of either are needed depends on the gap.  Measured, squarings against Lanczos: a pair well apart from the rest (6 squarings, 32 steps)
// 0.68 / 1.49 ms at 1024, 2.9 / 2.6 at 2048, 5.1 / 3.0 at 2560, 8.6 / 3.5 at 3072; a Laplace matrix (13 - 15, 96 - 128) 1.0 / 7.1, 4.6 / 17.0,
// 8.9 / 20.4, 17.0 / 30.0 ms.  So the line is where the better case of the Lanczos process begins to win; a Laplace
// matrix would gain from squarings up to 3500 and more, at 2 n^2 doubles of scratch.
constexpr int PAIR_MAX_N = 2048;

// v of lane `from` (uniform).
__device__ __forceinline__ double lane_value(double v, int from) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(double, (uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)b, from) |
                                          ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(b >> 32), from) << 32));
}

// Workgroup (bi, bj), bi <= bj, of Y = c P P^T for P [rows][L]: T x T blocks of 16 x 16, the contraction split over four
// wavefronts (v_mfma_f64_16x16x4), each 64 indices at a time (the Gram matrix of a small n, whose contraction is longer: eight, 32 at a time);
// the block and its mirror image are stored, and the diagonal once more by itself, so that its readers find 256 entries in 16 lines.
//
// The order of the contraction index is free as long as both operands share it: lane group g of a wavefront takes the
// indices 8 t + 2 g, 8 t + 2 g + 1 of its share with load t, so a load is 16 bytes per lane and touches 16 row segments of
// 64 bytes.  Bound by the latency of the loads and of the chain of MFMAs (64 cycles each): small tiles on many
// workgroups while n is small (n = 256: 136 workgroups with a tile, of 160, and 16 MFMAs per wavefront, 5.2 us; on eight wavefronts of 8 MFMAs 5.9 against 5.6 us; the Gram matrix of
// 512 rows 6.2 us on four, 5.7 us on eight), 32 x 32 tiles, which read half as much per product, beyond.
//
// GRAM (first launch): P is R by its rows (TR = false) or columns (TR), any pitch; rows beyond n and indices beyond L read
// as zero, c = 1.  Extra workgroups compute s = R v0 where the shorter side is the rows.
// Otherwise P = X[step & 1], symmetric, zero beyond n, c = 1 / trace^2.  The Gram matrix has the squares of R's magnitudes, and
// their squares would leave the range of fp64 for entries of R beyond 1e77 or below 1e-81: step 0 scales its operands by the power of
// two next to its trace (exact; a reduction and a barrier before the products, in this step only).  So R counts as long as its sum of
// squares does, 1e-150 to 1e150.  The trace of every X from the second on is
// sum lambda^2 / (sum lambda)^2 of the one before, 1 - 2 (lambda_2 / lambda_1)^(2^p) near the end.  Once that is within 1e-6 of
// 1, X itself has the ratio squared, below 2.5e-13, and is the result (X x_j has it squared again, times at most sqrt(n)):
// every workgroup of this and the later launches returns.
//
// Shifts (a sequence of pairs, n <= 768).  A squaring of X - s instead of X maps what lies in [0, 2 s] into [0, s^2] and stretches what lies above: with s halfway to
// the edge e of the part of the spectrum that is not wanted, and the next shift halfway to the image of that edge, s_{k+1} = (s_k / t_k)^2 / 2, p squarings are, on [0, e],
// the Chebyshev polynomial of degree 2^p (plus one, halved), which grows beyond e as cosh(2^p acosh(2 lambda / e - 1)): a distance d = lambda / e - 1 counts like 2 sqrt(d)
// instead of d.  Six squarings leave a residual of [512, 256] Laplace entries at the rank that eight to nine leave it at without (a component 81 -> 72 us, of [300, 700]
// 113 -> 99; the Gram matrix, which traces the value back while it waits for R, 1.1 us longer).  e is a fixed part of the
// second eigenvalue of the pair before, traced back to its own Gram matrix by the shifts and traces of its squarings.  It has to lie below the leading one, which nothing
// guarantees (tsvd_pair_sequence): the tail takes a pair only if the image of e is small against the result.  The matrices are stored with
// the next shift taken off their diagonal, the diagonals by themselves without.
// (GRAM only but for n; the scalars in front of it come preloaded in registers)
struct pair_square_rest {
    int n, M, N;
    const double* v0;
    double* s;
    double edge;             // e as a part of the second eigenvalue of the pair before, 0: no shifts
};
// The tiles of the upper triangle by XCD (workgroups go to the eight of them in turn), where no XCD gets more than one for each of its 32 compute units: the blocks
// of 16 T rows in four groups of k; six XCDs take a pair of groups each, two take two groups' own triangles, so that every L2 fetches half
// of the matrix instead of all of it (with arguments preloaded and results written through: a squaring of n = 256 5.7 -> 5.2 us, a component of [512, 256] 104 -> 96).  With more tiles in turn (768 x 700, where XCDs would get 36 to 42: 2.2 -> 2.9 ms).
// Returns false for workgroups without a tile.
__host__ __device__ constexpr int pair_group(int nb) { return (nb + 3) / 4; }
__host__ __device__ constexpr int pair_grid(int nb) { return pair_group(nb) <= 5 ? 8 * pair_group(nb) * (pair_group(nb) + 1) : nb * (nb + 1) / 2; }
__device__ __forceinline__ bool pair_tile(int nb, int block, int& bi, int& bj) {
    const int k = pair_group(nb), xcd = block & 7, t = block >> 3, half = k * (k + 1) / 2;
    int u = block, from = 0;                 // place in a triangle, its first block
    if (k <= 5) {
        if (xcd < 6) {
            const int gi = xcd < 3 ? 0 : xcd < 5 ? 1 : 2, gj = xcd < 3 ? xcd + 1 : xcd < 5 ? xcd - 1 : 3;
            bi = gi * k + t / k, bj = gj * k + t % k;
            return t < k * k && bj < nb;
        }
        u = t < half ? t : t - half;
        from = (2 * (xcd - 6) + (t >= half)) * k;
    }
    int j = (int)((sqrtf(8.0f * (float)u + 1.0f) - 1.0f) * 0.5f);
    while (j * (j + 1) / 2 > u) --j;
    while ((j + 1) * (j + 2) / 2 <= u) ++j;
    bi = from + u - j * (j + 1) / 2, bj = from + j;
    return bj < nb;
}
template <int T, bool GRAM, bool TR>
__global__ void __launch_bounds__(T == 1 && GRAM ? 512 : 256)
tsvd_pair_square_kernel(const double* __restrict__ P, double* __restrict__ Y, const double* __restrict__ D, double* __restrict__ YD, tsvd_pair_state* state,
                        int np, int step, int sequence, pair_square_rest p) {
    constexpr int W = T == 1 && GRAM ? 8 : 4, SHARE = 256 / W, LOADS = SHARE / 8;      // wavefronts; indices of one at a time
    __shared__ __align__(16) double part[W][T * T * 256];
    __shared__ double red[W];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
    const int nb = np / (16 * T);
    if constexpr (GRAM) {
        if (blockIdx.x == 0 && threadIdx.x == 0) state->last = -1;
        if ((int)blockIdx.x >= pair_grid(nb)) {             // s = R v0, a wavefront per row
            const int m = ((int)blockIdx.x - pair_grid(nb)) * W + wave;
            if (m < p.M) {
                double a = 0.0;
                for (int k = lane; k < p.N; k += 64) a += P[(size_t)m * p.N + k] * p.v0[k];
                a = wave_sum(a);
                if (lane == 0) p.s[m] = a;
            }
            return;
        }
    }
    int bi, bj;
    if (!pair_tile(nb, blockIdx.x, bi, bj)) return;
    const int L = GRAM ? (TR ? p.M : p.N) : np;
    tsvd_pair_shifts* const shifts = reinterpret_cast<tsvd_pair_shifts*>(state);        // (of a sequence)
    f64x4 acc[T][T];
#pragma unroll
    for (int a = 0; a < T; ++a)
#pragma unroll
        for (int b = 0; b < T; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
    const double* arow[T];
    const double* brow[T];
#pragma unroll
    for (int q = 0; q < T; ++q) {
        const int ra = (bi * T + q) * 16 + i, rb = (bj * T + q) * 16 + i;
        arow[q] = GRAM ? P + (TR ? (size_t)min(ra, p.n - 1) : (size_t)min(ra, p.n - 1) * p.N) : P + (size_t)ra * np;
        brow[q] = GRAM ? P + (TR ? (size_t)min(rb, p.n - 1) : (size_t)min(rb, p.n - 1) * p.N) : P + (size_t)rb * np;
    }
    auto load = [&](const double* row, int k) -> f64x2 {     // P[row][k], P[row][k + 1]; GRAM: indices clamped
        if constexpr (!GRAM) return *reinterpret_cast<const f64x2*>(row + k);
        const int k0 = min(k, L - 1), k1 = min(k + 1, L - 1);
        return TR ? f64x2{row[(size_t)k0 * p.N], row[(size_t)k1 * p.N]} : f64x2{row[k0], row[k1]};
    };
    // everything a wavefront needs is requested before anything is waited for
    double tr = 0.0, trace = 0.0, scale = 1.0, shift = 0.0, next_shift = 0.0;
    int done = -1;
    if constexpr (!GRAM) {
        done = state->last;
        if (sequence) shift = step == 0 ? shifts->first : shifts->s[step];
        tr = D[min((int)threadIdx.x, np - 1)];
    }
    auto sum_trace = [&] {                                   // the wavefronts' shares of the trace into red
        if ((int)threadIdx.x >= np) tr = 0.0;
        for (int d = threadIdx.x + 64 * W; d < np; d += 64 * W) tr += D[d];
        tr = wave_sum(tr);
        if (lane == 0) red[wave] = tr;
    };
    auto all = [&] {
        double a = 0.0;
#pragma unroll
        for (int w = 0; w < W; ++w) a += red[w];
        return a;
    };
    if (!GRAM && step == 0) {
        sum_trace();
        __syncthreads();
        trace = all();
        int e = 0;
        (void)frexp(trace, &e);
        scale = ldexp(1.0, -max(e, -1000));
        trace *= scale;
    }
    // (a sequence: what the pair before left, requested ahead of R; lane k holds what belongs to squaring k)
    double lambda = 0.0, before_s = 0.0, before_t = 0.0;
    int before = 0;
    if constexpr (GRAM) {
        if (sequence) {
            lambda = shifts->second, before = shifts->count;
            before_s = shifts->s[min(lane, TSVD_PAIR_MAX_SQUARINGS)], before_t = shifts->t[min(lane, TSVD_PAIR_MAX_SQUARINGS)];
        }
    }
    auto find_shift = [&] {                                  // back to the Gram matrix of that pair (in fp32 where traces are near 1: the edge has 2 % to spare)
        if (lambda > 0.0 && p.edge > 0.0) {
            float l = (float)lambda;
            for (int k = before - 1; k > 0; --k) l = (float)lane_value(before_s, k) + (float)lane_value(before_t, k) * __builtin_amdgcn_sqrtf(l);
            next_shift = 0.5 * p.edge * (lane_value(before_s, 0) + lane_value(before_t, 0) * (double)__builtin_amdgcn_sqrtf(l));
        }
        lambda = 0.0;
    };
    for (int k0 = wave * SHARE; k0 < L; k0 += 256) {
        f64x2 a[T][LOADS], b[T][LOADS];
#pragma unroll
        for (int t = 0; t < LOADS; ++t)
#pragma unroll
            for (int q = 0; q < T; ++q) {
                a[q][t] = load(arow[q], k0 + 8 * t + 2 * g);
                b[q][t] = load(brow[q], k0 + 8 * t + 2 * g);
            }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (GRAM) {
            find_shift();                                    // (while R is awaited)
            // rows beyond n and indices beyond L count as zero
#pragma unroll
            for (int t = 0; t < LOADS; ++t)
#pragma unroll
                for (int q = 0; q < T; ++q)
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const bool in = k0 + 8 * t + 2 * g + e < L;
                        if (!in || (bi * T + q) * 16 + i >= p.n) a[q][t][e] = 0.0;
                        if (!in || (bj * T + q) * 16 + i >= p.n) b[q][t][e] = 0.0;
                    }
        } else if (done >= 0) {
            break;
        } else if (step == 0) {
#pragma unroll
            for (int t = 0; t < LOADS; ++t)
#pragma unroll
                for (int q = 0; q < T; ++q) {
                    a[q][t] *= scale;
                    b[q][t] *= scale;
                }
        }
#pragma unroll
        for (int t = 0; t < LOADS; ++t)
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int qa = 0; qa < T; ++qa)
#pragma unroll
                    for (int qb = 0; qb < T; ++qb)
                        acc[qa][qb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[qa][t][e], b[qb][t][e], acc[qa][qb], 0, 0, 0);
    }
    double c = 1.0;
    if constexpr (!GRAM) {
        if (done >= 0) return;
        if (step > 0) sum_trace();
    } else if (sequence) {
        find_shift();                                        // (wavefronts without a share of the contraction)
        if (blockIdx.x == 0 && threadIdx.x == 0) shifts->first = next_shift;
    }
    // result lane (i, g): column i, rows g + 4 v
#pragma unroll
    for (int qa = 0; qa < T; ++qa)
#pragma unroll
        for (int qb = 0; qb < T; ++qb)
#pragma unroll
            for (int v = 0; v < 4; ++v) part[wave][(qa * T + qb) * 256 + (g + 4 * v) * 16 + i] = acc[qa][qb][v];
    __syncthreads();
    if constexpr (!GRAM) {
        if (step > 0) {
            trace = all();
            if (fabs(1.0 - trace) < 1e-6 && shift == 0.0) {
                if (blockIdx.x == 0 && threadIdx.x == 0) state->last = step;
                return;
            }
        }
        c = trace > 0.0 ? 1.0 / (trace * trace) : 0.0;
        if (sequence) {
            const double part = shift * scale;
            next_shift = 0.5 * part * part * c;
            if (!(next_shift > 1e-30)) next_shift = 0.0;     // (far below the last bit of the leading eigenvalue, which is a share of the trace)
            if (blockIdx.x == 0 && threadIdx.x == 0) {
                if (step == 0) shifts->s[0] = shift;
                shifts->s[step + 1] = next_shift;
                shifts->t[step] = trace / scale;
            }
        }
    }
    // Written through to memory at once: what a launch leaves in the L2s of the XCDs that computed it is written back before the next one starts (0.3 us of
    // 5.7).  (Not for R, the vectors or the system, whose launches write less or in lines of their own: 0.0 to 0.7 us longer.)
    auto store_through = [](double* at, double v) { __hip_atomic_store(at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    // (eight wavefronts: the second half of them writes the mirror image)
    const int r = (threadIdx.x & 255) >> 4, cc = threadIdx.x & 15;
    const bool first = threadIdx.x < 256, second = W == 4 || !first;
#pragma unroll
    for (int qa = 0; qa < T; ++qa)
#pragma unroll
        for (int qb = 0; qb < T; ++qb) {
            const int at = (qa * T + qb) * 256;
            const int row = (bi * T + qa) * 16, col = (bj * T + qb) * 16;
            auto sum = [&](int e) {
                double a = 0.0;
#pragma unroll
                for (int w = 0; w < W; ++w) a += part[w][at + e];
                return a * c;
            };
            if (first) {
                const double y = sum(r * 16 + cc);
                const bool diagonal = row + r == col + cc;
                store_through(&Y[(size_t)(row + r) * np + col + cc], diagonal && row + r < p.n ? y - next_shift : y);
                if (diagonal) store_through(&YD[row + r], y);
            }
            if (second && bi != bj) store_through(&Y[(size_t)(col + r) * np + row + cc], sum(cc * 16 + r));
        }
}

// The fixed start vector of the process, with no special symmetry.
__global__ void __launch_bounds__(256)
tsvd_pair_start_kernel(double* __restrict__ v0, int N, tsvd_pair_state* state) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < N) v0[k] = 1.0 + 0.5 * sin(1.0 + 0.7 * (double)k);
    if (k == 0) {
        state->last = -1;
        state->missed = state->shifted_missed = 0;
        state->needed = state->shifted_needed = state->far = 0;
    }
}

// The vector of the shorter side, a wavefront per row: X x_j, x_j the row (or column) of X with the largest diagonal entry (to
// nine bits: the upper words of the entries, their last bits replaced by the index); its sign that of s x_j.  Every
// workgroup finds j and the sign for itself.  A chain of loads (state, diagonal, x_j): what does not depend on j is requested first.
static_assert(PAIR_MAX_N <= 2048, "eleven bits of an index");
__global__ void __launch_bounds__(256)
tsvd_pair_short_kernel(tsvd_pair_plan p, int count) {
    __shared__ uint32_t most[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = blockIdx.x * 4 + wave;
    const int last = p.state->last;
    const double* X = p.X[(last >= 0 ? last : count) & 1];
    const double* mine = X + (size_t)min(row, p.n - 1) * p.np;
    uint32_t best = 0;
    for (int d = threadIdx.x; d < p.n; d += 256)
        best = max(best, ((uint32_t)(__builtin_bit_cast(uint64_t, X[(size_t)d * (p.np + 1)]) >> 32) & ~2047u) | (uint32_t)(2047 - d));
    double xr[4], sr[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        xr[t] = mine[min(lane + 64 * t, p.n - 1)];
        sr[t] = p.s[min(lane + 64 * t, p.n - 1)];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (last < 0) ++p.state->missed;
        p.state->needed = max(p.state->needed, last < 0 ? count : last + 1);
    }
    best = max(best, lane_xor32<32>(best));
    best = max(best, lane_xor32<16>(best));
    best = max(best, lane_xor32<8>(best));
    best = max(best, lane_xor32<4>(best));
    best = max(best, lane_xor32<2>(best));
    best = max(best, lane_xor32<1>(best));
    if (lane == 0) most[wave] = best;
    __syncthreads();
    const int j = 2047 - (int)(max(max(most[0], most[1]), max(most[2], most[3])) & 2047u);
    const double* x = X + (size_t)j * p.np;
    double a = 0.0, sx = 0.0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const double v = lane + 64 * t < p.n ? x[min(lane + 64 * t, p.n - 1)] : 0.0;
        a += xr[t] * v;
        sx += sr[t] * v;
    }
    for (int k = lane + 256; k < p.n; k += 64) {
        a += mine[k] * x[k];
        sx += p.s[k] * x[k];
    }
    a = wave_sum(a);
    sx = wave_sum(sx);                                       // (of every wavefront: cheaper than a second barrier)
    if (lane == 0 && row < p.n) (p.N <= p.M ? p.v : p.u)[row] = sx < 0.0 ? -a : a;
}

// The same from a squared matrix that is not of rank one yet, n <= 768 (what fits LDS).  After p squarings all but a few eigenvalues are below rounding, and what
// is left of the squarings is work on a matrix of that rank: X = L L^T by a Cholesky factorisation with the largest remaining diagonal entry as the
// pivot (until it is below 2^-50 of the first: X is positive semidefinite, so nothing larger is left anywhere, and the factorisation is as
// accurate as a squaring), S = L^T L [16][16] with the eigenvalues of X, squared until it is of rank one, and the vector L y with y the column
// of S^2 that has the largest diagonal entry.  One workgroup, a row a thread.
//
// Bound by its chain of latencies: a pivot is two barriers and a column of X from L2 (0.5 us), a squaring of S four MFMAs and a trace in one
// wavefront (0.25 us: S is symmetric, so the result registers of the MFMA are its operands of the next).  Loops are kept short rather than
// unrolled: every instruction runs a few times at most, and straight-line code waits for its own fetches (unrolled over the pivots with L in
// registers the kernel took 22 us).  On a [512, 256] Laplace matrix 8 squarings, 6 with shifts, leave 8 .. 14 pivots, in the place of 3 to 6 squarings of
// 6.3 us and of two or three launches that had nothing to do.  More than 16 pivots: the pair counts as missed and is taken again with more squarings.
constexpr int TAIL_RANK = 16, TAIL_PITCH = TAIL_RANK + 1, TAIL_MAX_N = 768;
static_assert(TAIL_MAX_N * TAIL_PITCH * 8 + TAIL_MAX_N / 64 * 2048 + 1024 <= 160 * 1024, "LDS");
__global__ void __launch_bounds__(TAIL_MAX_N)
tsvd_pair_tail_kernel(tsvd_pair_plan p, int count, int shifted) {
    extern __shared__ __align__(16) unsigned char tail_lds[];
    double* L = reinterpret_cast<double*>(tail_lds);         // [threads][TAIL_PITCH]
    __shared__ double row_j[TAIL_RANK + 1], y[TAIL_RANK], tot[TAIL_MAX_N / 64], part[TAIL_MAX_N / 64][256];
    __shared__ uint32_t keys[TAIL_MAX_N / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = p.np >> 6, i = lane & 15, g = lane >> 4;
    const int last = p.state->last;
    const double* X = p.X[(last >= 0 ? last : count) & 1];
    double d = tid < p.n ? p.diag[(last >= 0 ? last : count) & 1][tid] : -1.0;
    const double s = p.s[min(tid, p.n - 1)];
    tsvd_pair_shifts* const shifts = reinterpret_cast<tsvd_pair_shifts*>(p.state);      // (of a sequence)
    const double last_shift = p.sequence ? shifts->s[count] : 0.0, edge = last < 0 ? 2.0 * last_shift : 0.0;
    double* mine = L + tid * TAIL_PITCH;
#pragma unroll
    for (int k = 0; k < TAIL_RANK; ++k) mine[k] = 0.0;
    if (tid <= TAIL_RANK) row_j[tid] = 0.0;
    double tol = 0.0;
    int r = 0;
    bool over = false;
#pragma unroll 1
    for (int k = 0;; ++k) {
        uint32_t best = d > 0.0 ? ((uint32_t)(__builtin_bit_cast(uint64_t, d) >> 32) & ~1023u) | (uint32_t)(1023 - tid) : 0u;
        best = max(best, lane_xor32<32>(best));
        best = max(best, lane_xor32<16>(best));
        best = max(best, lane_xor32<8>(best));
        best = max(best, lane_xor32<4>(best));
        best = max(best, lane_xor32<2>(best));
        best = max(best, lane_xor32<1>(best));
        if (lane == 0) keys[wave] = best;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < TAIL_MAX_N / 64; ++w) best = max(best, keys[min(w, waves - 1)]);
        const int j = min(1023 - (int)(best & 1023u), p.n - 1);
        const double x = X[(size_t)j * p.np + tid];
        if (tid == j) {
            row_j[TAIL_RANK] = best ? d : 0.0;
#pragma unroll 4
            for (int q = 0; q < k; ++q) row_j[q] = mine[q];
        }
        __syncthreads();
        const double dj = row_j[TAIL_RANK];
        if (k == 0) {
            tol = dj * 0x1p-50;
            if (!(edge <= dj * 0x1p-46)) {                   // (shifts: the leading eigenvalue is not known to lie above the edge)
                over = true;
                break;
            }
        }
        // (a matrix that the squarings call of rank one: what a seventeenth pivot would add is below 1e-12 of it)
        over = dj > tol && k == TAIL_RANK && last < 0;
        if (!(dj > tol) || k == TAIL_RANK) break;
        double a = 0.0, b = 0.0;
        for (int q = 0; q < k; q += 4) {                     // (what lies behind k meets zeros)
            a += mine[q] * row_j[q];
            b += mine[q + 1] * row_j[q + 1];
            a += mine[q + 2] * row_j[q + 2];
            b += mine[q + 3] * row_j[q + 3];
        }
        const double root = sqrt(dj), v = tid == j ? root : (x - (a + b)) / root;
        mine[k] = v;
        d = tid == j ? -1.0 : d - v * v;
        r = k + 1;
    }
    if (tid == 0) {
        // squarings that the next such pair (after `over`: this one) should get: halving the exponent nearly doubles the pivots.  After
        // `over`: each squaring doubles the bits between the first pivot and the seventeenth, which are to become fifty; what is missed at the last
        // count that is tried is taken as it is (equal singular values: any vector of theirs will do).
        // (squarings with shifts: one fewer leaves two and a half to four times the pivots)
        int want = r > 12 ? count + 1 : last >= 0 ? last + 1 : r <= (shifted ? 3 : 5) ? max(count - 1, 1) : count;
        if (over && r == TAIL_RANK) {
            constexpr int LAST = TSVD_PAIR_MAX_SQUARINGS - 1;
            const double bits = log2(tol * 0x1p50 / row_j[TAIL_RANK]);      // (not above 0: pivots that are equal, as far as they are compared)
            want = count >= LAST ? TSVD_PAIR_MAX_SQUARINGS : bits > 0x1p-40 ? min(LAST, count + max(1, (int)ceil(log2(50.0 / bits)))) : LAST;
        }
        int* const report = shifted ? &p.state->shifted_missed : &p.state->missed;
        if (over) ++report[0];
        report[1] = max(report[1], want);
    }
    // ---- S = L^T L: a wavefront's share from its own 64 rows, then one wavefront
    f64x4 S = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int t = 0; t < 16; ++t) {
        const double a = L[(wave * 64 + 4 * t + g) * TAIL_PITCH + i];
        S = __builtin_amdgcn_mfma_f64_16x16x4f64(a, a, S, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) part[wave][lane * 4 + v] = S[v];
    __syncthreads();
    if (wave == 0) {
#pragma unroll 1
        for (int w = 1; w < waves; ++w)
#pragma unroll
            for (int v = 0; v < 4; ++v) S[v] += part[w][lane * 4 + v];
        // lane (i, g) holds column i, rows g + 4 v; its diagonal entry, if it has one, v = i / 4
        auto diagonal = [&] {
            const double e = i < 8 ? i < 4 ? S[0] : S[1] : i < 12 ? S[2] : S[3];
            return (i & 3) == g ? e : 0.0;
        };
        const f64x4 S0 = S;
        const double trace0 = wave_sum(diagonal());
        auto square = [&](double c) {
            f64x4 sq = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int t = 0; t < 4; ++t) sq = __builtin_amdgcn_mfma_f64_16x16x4f64(S[t], S[t], sq, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) S[v] = sq[v] * c;
        };
#pragma unroll 1
        for (int step = count; step < TSVD_PAIR_MAX_SQUARINGS; ++step) {
            const double trace = wave_sum(diagonal());
            if (step > count && fabs(1.0 - trace) < 1e-6) break;
            square(trace > 0.0 ? 1.0 / (trace * trace) : 0.0);
        }
        uint32_t best = ((uint32_t)(__builtin_bit_cast(uint64_t, fmax(diagonal(), 0.0)) >> 32) & ~15u) | (uint32_t)(15 - i);
        best = max(best, lane_xor32<32>(best));
        best = max(best, lane_xor32<16>(best));
        best = max(best, lane_xor32<8>(best));
        best = max(best, lane_xor32<4>(best));
        best = max(best, lane_xor32<2>(best));
        best = max(best, lane_xor32<1>(best));
        if (p.sequence) {
            // the second eigenvalue: what the trace holds beside the first one, (S, S0) / tr S (with those behind it, at most fifteen times as much: a value between
            // the first's rounding and itself in the sum, of which the Gram matrix's is the 2^count-th root and less)
            const double first = wave_sum((S[0] * S0[0] + S[1] * S0[1]) + (S[2] * S0[2] + S[3] * S0[3])) / wave_sum(diagonal()), rest = trace0 - first;
            if (lane == 0) {
                shifts->second = !over && rest > 0x1p-46 * first ? fmin(rest, first) : 0.0;
                shifts->count = last >= 0 ? last : count;
                if (!(rest > 0x1p-30 * first)) ++p.state->far;
            }
        }
        square(1.0);
        if (i == 15 - (int)(best & 15u))
#pragma unroll
            for (int v = 0; v < 4; ++v) y[g + 4 * v] = S[v];
    }
    __syncthreads();
    double v = 0.0;
#pragma unroll 4
    for (int k = 0; k < TAIL_RANK; ++k) v += mine[k] * y[k];
    double sx = wave_sum(tid < p.n ? s * v : 0.0);
    if (lane == 0) tot[wave] = sx;
    __syncthreads();
    sx = 0.0;
    for (int w = 0; w < waves; ++w) sx += tot[w];
    if (tid < p.n) (p.N <= p.M ? p.v : p.u)[tid] = sx < 0.0 ? -v : v;
}

// The vector of the longer side.  N <= M: u = R v, a wavefront per row.  M < N: v = R^T u, 64 columns per workgroup, the
// rows in four phases.
__global__ void __launch_bounds__(256)
tsvd_pair_long_kernel(tsvd_pair_plan p, const double* __restrict__ R) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (p.N <= p.M) {
        const int m = blockIdx.x * 4 + wave;
        if (m >= p.M) return;
        const double* row = R + (size_t)m * p.N;
        double a = 0.0;
        for (int k = lane; k < p.N; k += 64) a += row[k] * p.v[k];
        a = wave_sum(a);
        if (lane == 0) p.u[m] = a;
        return;
    }
    __shared__ double red[4][64];
    const int col = blockIdx.x * 64 + lane;
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    if (col < p.N) {
        int m = wave;
        for (; m + 12 < p.M; m += 16)
#pragma unroll
            for (int t = 0; t < 4; ++t) a[t] += R[(size_t)(m + 4 * t) * p.N + col] * p.u[m + 4 * t];
        for (; m < p.M; m += 4) a[0] += R[(size_t)m * p.N + col] * p.u[m];
    }
    red[wave][lane] = (a[0] + a[1]) + (a[2] + a[3]);
    __syncthreads();
    if (wave == 0 && col < p.N) p.v[col] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// Sum of squares over the workgroup (256 threads), in every thread.
__device__ __forceinline__ double norm2(const double* x, int len, double* red) {
    double a = 0.0;
    for (int k = threadIdx.x; k < len; k += 256) a += x[k] * x[k];
    a = wave_sum(a);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// Unit vectors and the singular value: |u| / |v| of the raw pair is sigma (u = R v) or 1 / sigma (v = R^T u).
__global__ void __launch_bounds__(256)
tsvd_pair_normalise_kernel(tsvd_pair_plan p, int count, double* __restrict__ u, double* __restrict__ v, double* __restrict__ sigma,
                           int* __restrict__ steps) {
    __shared__ double red[4];
    const double un = sqrt(norm2(p.u, p.M, red)), vn = sqrt(norm2(p.v, p.N, red));
    const double ui = un > 0.0 ? 1.0 / un : 0.0, vi = vn > 0.0 ? 1.0 / vn : 0.0;
    for (int k = threadIdx.x; k < p.M; k += 256) u[k] = p.u[k] * ui;
    for (int k = threadIdx.x; k < p.N; k += 256) v[k] = p.v[k] * vi;
    if (threadIdx.x == 0) {
        sigma[0] = p.N <= p.M ? un * vi : vn * ui;
        if (steps) steps[0] = p.state->last >= 0 ? p.state->last : count;
    }
}

// R[m][k] -= sigma u[m] v[k] with unit u and v: u_raw v_raw / |the shorter side's raw vector|^2.  A workgroup per row.
__global__ void __launch_bounds__(256)
tsvd_pair_deflate_kernel(tsvd_pair_plan p, double* __restrict__ R) {
    __shared__ double red[4];
    const double n2 = p.N <= p.M ? norm2(p.v, p.N, red) : norm2(p.u, p.M, red);
    const double f = n2 > 0.0 ? p.u[blockIdx.x] / n2 : 0.0;
    double* row = R + (size_t)blockIdx.x * p.N;
    for (int k = threadIdx.x; k < p.N; k += 256) row[k] -= f * p.v[k];
}

}  // namespace

hipError_t tsvd_pair_init() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(tsvd_pair_tail_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, TAIL_MAX_N * TAIL_PITCH * 8);
}

bool tsvd_pair_any_rank(const tsvd_pair_plan& p) { return p.np <= TAIL_MAX_N; }
void tsvd_pair_sequence(tsvd_pair_plan* p, tsvd_pair_shifts* shifts) {
    p->state = &shifts->state;
    p->sequence = tsvd_pair_any_rank(*p);
}
int tsvd_pair_first_squarings(const tsvd_pair_plan& p) { return !tsvd_pair_any_rank(p) ? 16 : p.np <= 128 ? 8 : p.np <= 512 ? 9 : 10; }

bool tsvd_pair_squares(int64_t M, int64_t N) { return std::min(M, N) <= PAIR_MAX_N; }

size_t tsvd_pair_bytes(int64_t M, int64_t N) {
    const size_t np = (size_t)(std::min(M, N) + 63) / 64 * 64;
    return 2 * round256(np * np * 8) + 2 * round256(np * 8) + 3 * round256((size_t)N * 8) + 2 * round256((size_t)M * 8) + 256;
}

void tsvd_pair_prepare(int64_t M, int64_t N, void* mem, tsvd_pair_plan* p, hipStream_t stream) {
    uint8_t* at = static_cast<uint8_t*>(mem);
    auto take = [&](size_t doubles) {
        double* r = reinterpret_cast<double*>(at);
        at += round256(doubles * 8);
        return r;
    };
    p->M = (int)M; p->N = (int)N; p->n = (int)std::min(M, N); p->np = (p->n + 63) / 64 * 64;
    p->X[0] = take((size_t)p->np * p->np);
    p->X[1] = take((size_t)p->np * p->np);
    p->diag[0] = take((size_t)p->np);
    p->diag[1] = take((size_t)p->np);
    p->v0 = take((size_t)N);
    p->s = N <= M ? p->v0 : take((size_t)M);
    p->u = take((size_t)M);
    p->v = take((size_t)N);
    p->state = reinterpret_cast<tsvd_pair_state*>(at);
    p->sequence = false;
    hipLaunchKernelGGL(tsvd_pair_start_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, stream, p->v0, p->N, p->state);
}

void tsvd_pair_square(const tsvd_pair_plan& p, const double* R, int from, int to, bool shifted, hipStream_t stream) {
    const bool big = p.np > 384;
    const int nb = p.np / (big ? 32 : 16);
    const unsigned tiles = (unsigned)pair_grid(nb);
    // The edge for p squarings: at a degree of 2^p the second eigenvalue of the pair before less 2 %, which the leading one is seldom below, comes out 2^52 times the edge's
    // image (cosh 36.7): p = 6 0.90 of it, 7 0.96, 8 0.975.
    const double edge = p.sequence && shifted && from == 0 ? 0.98 / (1.0 + 0.5 * (std::cosh(36.7 / std::ldexp(1.0, to)) - 1.0)) : 0.0;
    const pair_square_rest rest = {p.n, p.M, p.N, p.v0, p.s, edge};
#define PAIR_SQUARE(T, GRAM, TR, grid, threads, in, at, step) \
    hipLaunchKernelGGL((tsvd_pair_square_kernel<T, GRAM, TR>), dim3(grid), dim3(threads), 0, stream, in, p.X[at], p.diag[1 - (at)], p.diag[at], p.state, p.np, step, (int)p.sequence, rest)
    if (from == 0) {
        const bool cols = p.N <= p.M;
        const unsigned grid = tiles + (cols ? 0u : (unsigned)(big ? (p.M + 3) / 4 : (p.M + 7) / 8));
        if (big && cols) PAIR_SQUARE(2, true, true, grid, 256, R, 0, 0);
        else if (big) PAIR_SQUARE(2, true, false, grid, 256, R, 0, 0);
        else if (cols) PAIR_SQUARE(1, true, true, grid, 512, R, 0, 0);
        else PAIR_SQUARE(1, true, false, grid, 512, R, 0, 0);
    }
    for (int step = from; step < to; ++step) {
        const int at = (step + 1) & 1;
        if (big) PAIR_SQUARE(2, false, false, tiles, 256, p.X[1 - at], at, step);
        else PAIR_SQUARE(1, false, false, tiles, 256, p.X[1 - at], at, step);
    }
#undef PAIR_SQUARE
}

void tsvd_pair_vectors(const tsvd_pair_plan& p, const double* R, int count, bool any_rank, bool shifted, hipStream_t stream) {
    if (any_rank) hipLaunchKernelGGL(tsvd_pair_tail_kernel, dim3(1), dim3((unsigned)p.np), (unsigned)(p.np * TAIL_PITCH * 8), stream, p, count, (int)shifted);
    else hipLaunchKernelGGL(tsvd_pair_short_kernel, dim3((unsigned)((p.n + 3) / 4)), dim3(256), 0, stream, p, count);
    const unsigned grid = p.N <= p.M ? (unsigned)((p.M + 3) / 4) : (unsigned)((p.N + 63) / 64);
    hipLaunchKernelGGL(tsvd_pair_long_kernel, dim3(grid), dim3(256), 0, stream, p, R);
}

void tsvd_pair_normalise(const tsvd_pair_plan& p, int count, double* u, double* v, double* sigma, int32_t* steps, hipStream_t stream) {
    hipLaunchKernelGGL(tsvd_pair_normalise_kernel, dim3(1), dim3(256), 0, stream, p, count, u, v, sigma, steps);
}

void tsvd_pair_deflate(const tsvd_pair_plan& p, double* R, hipStream_t stream) {
    hipLaunchKernelGGL(tsvd_pair_deflate_kernel, dim3((unsigned)p.M), dim3(256), 0, stream, p, R);
}
