// Direct transition W -> (U, S, V) on the GPU (paper, section "Direct Transition Algorithm to
// TSVD form": Algorithm 1, Eq. (3), Algorithm 2).  The algorithm runs once per layer and every
// step is small at the paper's matrix sizes ([512, 256] in its random-matrix study), so the steps
// are bound by launch and memory latency, not by arithmetic: each is one launch.  The leading
// singular pair comes from squarings of the Gram matrix (tsvd_pair.hip), beyond its sizes from
// Lanczos steps.  Everything is fp64: the decisions of Algorithm 1 compare sums against cos(theta)
// and must not depend on fp32 noise.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "../../include/tsvd_transition.h"
#include "../../include/tsvd_tuning.h"
#include "tsvd_kernels.h"
#include "tsvd_pair.h"
#include "tsvd_scratch.h"
#include "tsvd_wave.h"

#define TERN_MAX_N 8192
#define FIT_MAX_K 2048

namespace {

size_t round256(size_t v) { return (v + 255) & ~(size_t)255; }

// Sum over the 256 threads of a workgroup, in a fixed order (tree in LDS); result in every thread.
__device__ __forceinline__ double block_sum256(double v, double* red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    return r;
}

// ---- Algorithm 1: one workgroup per vector ---------------------------------------------------
// The magnitudes stay in registers, E per thread (position e * threads + thread), and are sorted largest first by a
// bitonic network: partners less than a wavefront apart meet through cross-lane moves, those in other wavefronts through
// LDS (6 of the 45 stages at 512 entries), those of one thread in its registers.  Then prefix sums in sorted order (wave
// scans and the totals of the wavefronts before), and the smallest q whose cosine reaches cos(theta).  Padding
// (-1) sorts last.  (With the whole list in LDS and 256 threads, every stage behind a barrier, 512 entries took 23 us.)  512 entries take 5.7 us: 1.9
// thousand cycles for the first loads, 7.3 for the network (two wavefronts share a SIMD, and issue some ten operations a stage), 2.3 for
// the sums and the search: 7 before the scan went by moves between lanes and one lane of a wavefront reported (7.8 us).
struct ternarize_job {
    const double* x; long long ldx; int n;
    int8_t* t; long long ldt;
    int* status;             // [rows], or null
    int* failed;             // counts the vectors without a neighbour, or null
};
struct ternarize_args {
    ternarize_job job[2];    // blockIdx.y
    int npow2;
    double cos_theta;
};
#define TERN_THREADS 1024
template <int E>
__global__ void __launch_bounds__(TERN_THREADS)
tsvd_ternarize_kernel(ternarize_args p) {
    __shared__ double keys[2 * TERN_THREADS];
    __shared__ double tot[2][TERN_THREADS / 64];
    __shared__ int qmin;
    __shared__ double threshold;
    const ternarize_job& job = p.job[blockIdx.y];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), T = min(p.npow2, TERN_THREADS), nw = T >> 6, n = job.n;
    const double* xr = job.x + (size_t)blockIdx.x * job.ldx;
    int8_t* tr = job.t + (size_t)blockIdx.x * job.ldt;
    if (tid == 0) qmin = 0x7FFFFFFF;
    double a[E], ss = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int s = e * T + tid;
        const double v = s < n ? xr[s] : 0.0;
        a[e] = s < n ? fabs(v) : -1.0;
        ss += v * v;
    }
    ss = wave_sum(ss);
    if (lane == 0) tot[0][wave] = ss;
    __syncthreads();
    double length = 0.0;
    for (int w = 0; w < nw; ++w) length += tot[0][w];
    length = sqrt(length);
    int flip = 0;
    // Position e T + tid meets the one j away: the larger of the two stays where (position & k) and (position & j) agree.  In a wavefront either
    // condition is a mask of lanes, so a stage is the move, a maximum, a minimum and the choice between them, with nothing that waits for a
    // scalar register (and no quieting of NaNs before the maximum: 165 cycles a stage).
    constexpr uint64_t BIT[6] = {0x5555555555555555ull, 0x3333333333333333ull, 0x0F0F0F0F0F0F0F0Full, 0x00FF00FF00FF00FFull, 0x0000FFFF0000FFFFull, 0x00000000FFFFFFFFull};
    auto meet = [&](int e, uint64_t larger, double b) {
        double hi, lo;
        asm("v_max_f64 %0, %1, %2" : "=v"(hi) : "v"(a[e]), "v"(b));
        asm("v_min_f64 %0, %1, %2" : "=v"(lo) : "v"(a[e]), "v"(b));
        a[e] = __builtin_amdgcn_inverse_ballot_w64(larger) ? hi : lo;
    };
    for (int k = 2; k <= p.npow2; k <<= 1) {
        for (int j = k >> 1; j >= 64; j >>= 1) {
            if (j >= T) {
#pragma unroll
                for (int h = E / 2; h > 0; h >>= 1)
                    if (j == h * T) {
#pragma unroll
                        for (int e = 0; e < E; ++e)
                            if (!(e & h)) {
                                const bool first = ((e * T + tid) & k) == 0;        // largest first
                                const double hi = fmax(a[e], a[e | h]), lo = fmin(a[e], a[e | h]);
                                a[e] = first ? hi : lo;
                                a[e | h] = first ? lo : hi;
                            }
                    }
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    double* buf = keys + flip * TERN_THREADS;                       // (the other one's readers may be behind)
                    buf[tid] = a[e];
                    __syncthreads();
                    const int s = e * T + wave * 64;
                    meet(e, ((s & k) == 0) == ((s & j) == 0) ? ~0ull : 0ull, buf[tid ^ j]);
                    flip ^= 1;
                }
            }
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint64_t mk = __ballot(((e * T + tid) & k) == 0);
            if (k >= 64) meet(e, ~(mk ^ BIT[5]), lane_xor<32>(a[e]));
            if (k >= 32) meet(e, ~(mk ^ BIT[4]), lane_xor<16>(a[e]));
            if (k >= 16) meet(e, ~(mk ^ BIT[3]), lane_xor<8>(a[e]));
            if (k >= 8) meet(e, ~(mk ^ BIT[2]), lane_xor<4>(a[e]));
            if (k >= 4) meet(e, ~(mk ^ BIT[1]), lane_xor<2>(a[e]));
            meet(e, ~(mk ^ BIT[0]), lane_xor<1>(a[e]));
        }
    }
    double carry = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        double run = wave_scan(fmax(a[e], 0.0));
        if (lane == 63) tot[(e + 1) & 1][wave] = run;
        __syncthreads();
        double before = carry;
#pragma unroll 8
        for (int w = 0; w < nw; ++w) {
            const double t = tot[(e + 1) & 1][w];
            if (w < wave) before += t;
            carry += t;
        }
        run += before;
        const int q = e * T + tid + 1;
        // (one lane of a wavefront reports)
        const uint64_t reached = __ballot(a[e] >= 0.0 && length > 0.0 && run / (sqrt((double)q) * length) >= p.cos_theta);
        if (lane == 0 && reached != 0) atomicMin(&qmin, e * T + wave * 64 + __builtin_ctzll(reached) + 1);
    }
    __syncthreads();
    const int q = qmin;
    const bool found = q != 0x7FFFFFFF;
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (e * T + tid + 1 == q) threshold = a[e];
    __syncthreads();
    const double th = threshold;
    for (int s = tid; s < n; s += T) {
        const double v = xr[s];
        tr[s] = (found && fabs(v) >= th) ? (v >= 0.0 ? 1 : -1) : 0;
    }
    if (tid == 0) {
        if (job.status) job.status[blockIdx.x] = found ? 0 : 1;
        if (job.failed && !found) atomicAdd(job.failed, 1);
    }
}

// ---- Eq. (3), left side: G[k][l] = (sum_m U[m][k] U[m][l]) (sum_n V[k][n] V[l][n]) ------------------
// One thread per (k, l), l fastest (U[m][l] is then read along rows; V[l][n] is strided but V is
// small and cached).  Integer sums, exact.
__global__ void __launch_bounds__(256)
tsvd_gram_kernel(const int8_t* __restrict__ U, long long ldu, const int8_t* __restrict__ V, int M, int K, int N,
                 double* __restrict__ G, long long ldg) {
    const int l = blockIdx.x * 256 + threadIdx.x, k = blockIdx.y;
    if (l >= K) return;
    int uu = 0, vv = 0;
    for (int m = 0; m < M; ++m) uu += (int)U[(size_t)m * ldu + k] * (int)U[(size_t)m * ldu + l];
    const int8_t* vk = V + (size_t)k * N;
    const int8_t* vl = V + (size_t)l * N;
    for (int n = 0; n < N; ++n) vv += (int)vk[n] * (int)vl[n];
    G[(size_t)k * ldg + l] = (double)uu * (double)vv;
}

// ---- Eq. (3), right side: d[k] = sum_m sum_n U[m][k] W[m][n] V[k][n]; one workgroup per k ----------
__global__ void __launch_bounds__(256)
tsvd_rhs_kernel(const int8_t* __restrict__ U, long long ldu, const int8_t* __restrict__ V, const double* __restrict__ W, int M,
                int N, double* __restrict__ d) {
    __shared__ double red[256];
    const int k = blockIdx.x;
    const int8_t* vk = V + (size_t)k * N;
    double acc = 0.0;
    for (int m = 0; m < M; ++m) {
        const int um = U[(size_t)m * ldu + k];
        if (um == 0) continue;                                  // (uniform over the workgroup)
        const double* wr = W + (size_t)m * N;
        double row = 0.0;
        for (int n = threadIdx.x; n < N; n += 256) row += (double)vk[n] * wr[n];
        acc += um > 0 ? row : -row;
    }
    const double total = block_sum256(acc, red);
    if (threadIdx.x == 0) d[k] = total;
}

// ---- Eq. (3) inside Algorithm 2: what the components K0 + blockIdx.y (of K by now) add to the system ---------------
// A wavefront each: idx < K: the entry (idx, new) of the Gram matrix and its mirror, four codes per v_dot4; then, for
// every row m of W, U[m][new] sum_n W[m][n] V[new][n] into part[new - K0][m] (summed by the solver).  Ut [rank][mp] and
// V [rank][np] hold one component per row, zero beyond M and N (pitches are multiples of 16).
__global__ void __launch_bounds__(256)
tsvd_system_kernel(const int8_t* __restrict__ Ut, int mp, const int8_t* __restrict__ V, int np, const double* __restrict__ W, int M, int N,
                   int K0, int K, double* __restrict__ G, long long ldg, double* __restrict__ part) {
    const int idx = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, r = K0 + blockIdx.y;
    if (idx < K) {
        auto dot = [&](const int8_t* a, const int8_t* b, int len) {
            int v = 0;
            for (int k = lane * 4; k < len; k += 256)
                v = __builtin_amdgcn_sdot4(*reinterpret_cast<const int*>(a + k), *reinterpret_cast<const int*>(b + k), v, false);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            return v;
        };
        const int uu = dot(Ut + (size_t)idx * mp, Ut + (size_t)r * mp, mp), vv = dot(V + (size_t)idx * np, V + (size_t)r * np, np);
        if (lane == 0) G[(size_t)r * ldg + idx] = G[(size_t)idx * ldg + r] = (double)uu * (double)vv;
    } else if (idx - K < M) {
        const int m = idx - K, um = Ut[(size_t)r * mp + m];
        double a = 0.0;
        if (um != 0) {
            const double* wr = W + (size_t)m * N;
            const int8_t* vr = V + (size_t)r * np;
            for (int n = lane; n < N; n += 64) a += (double)vr[n] * wr[n];
            a = wave_sum(a);
        }
        if (lane == 0) part[(size_t)blockIdx.y * M + m] = um > 0 ? a : -a;
    }
}

// ---- Eq. (3), the solve: conjugate gradients with diagonal scaling, one workgroup -------------
// G s = d for the symmetric positive semi-definite G of the normal equations, started from s = 0,
// so for a singular G the iterates stay in its range and converge to the minimum-norm solution
// (the pseudo-inverse solution).  Stops at |r| <= 1e-13 |d| or after 20 K iterations.
// s0: start from these `fresh` values (and zeros) instead of zero (any least-squares solution gives the
// same residual; the loop of Algorithm 2 starts from the previous scales), or null.  The entries of d from
// `fresh` on are first summed from `part` [K - fresh][M].
//
// An iteration waits for barriers and LDS latency, not for arithmetic: a thread owns a row (its entries of every vector;
// only the direction is shared), rows are read as columns (G is symmetric, so consecutive threads read consecutive
// words), the two sums of an update go through one reduction (wave sums, then every thread adds the wavefronts' totals),
// and a system of up to PCG_LDS_K unknowns runs with G in LDS on as few wavefronts as it has rows.  Larger systems
// re-read G from L2 on 1024 threads, the columns of a row split over 1024 / K groups of threads.
#define PCG_LDS_K 96
__device__ __forceinline__ void solve_pcg(unsigned char* smem, int T, const double* __restrict__ G, long long ldg, double* __restrict__ d, int K,
                                          double* __restrict__ s, const double* __restrict__ s0, int* __restrict__ iters,
                                          const double* __restrict__ part, int fresh, int M) {
    double* xs = reinterpret_cast<double*>(smem);   // [K] solution
    double* r = xs + K;                             // residual
    double* p = r + K;                              // direction
    double* q = p + K;                              // G p
    double* dg = q + K;                             // 1 / diagonal (1 where the diagonal is 0)
    double* sub = dg + K;                           // [1024] partial products of a row
    double* Gl = sub + 1024;                        // [K][K], K <= PCG_LDS_K
    __shared__ double red[2][2][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = T >> 6;
    int flip = 0;
    auto sum2 = [&](double a, double b, double& sa, double& sb) {      // sums over the workgroup, fixed order, in every thread
        a = wave_sum(a);
        b = wave_sum(b);
        if (lane == 0) {
            red[flip][0][wave] = a;
            red[flip][1][wave] = b;
        }
        __syncthreads();
        sa = sb = 0.0;
        for (int w = 0; w < nw; ++w) {
            sa += red[flip][0][w];
            sb += red[flip][1][w];
        }
        flip ^= 1;
    };
    double unused;
    for (int k = fresh; k < K; ++k) {
        double a = 0.0, total;
        for (int m = tid; m < M; m += T) a += part[(size_t)(k - fresh) * M + m];
        sum2(a, 0.0, total, unused);
        if (tid == 0) d[k] = total;
    }
    const bool in_lds = K <= PCG_LDS_K;
    if (in_lds)
        for (int e = tid; e < K * K; e += T) Gl[e] = G[(size_t)(e / K) * ldg + e % K];
    const double* Gm = in_lds ? Gl : G;
    const size_t ld = in_lds ? (size_t)K : (size_t)ldg;
    const int rows = (K + 63) & ~63, groups = rows >= T ? 1 : T / rows, grp = tid / rows;
    auto matvec = [&](const double* in, double* out) {                 // out = G in (owner threads only read their entries of out)
        if (groups == 1) {
            for (int k = tid; k < K; k += T) {
                double v0 = 0.0, v1 = 0.0, v2 = 0.0, v3 = 0.0;
                int l = 0;
                for (; l + 3 < K; l += 4) {
                    v0 += Gm[(size_t)l * ld + k] * in[l];
                    v1 += Gm[(size_t)(l + 1) * ld + k] * in[l + 1];
                    v2 += Gm[(size_t)(l + 2) * ld + k] * in[l + 2];
                    v3 += Gm[(size_t)(l + 3) * ld + k] * in[l + 3];
                }
                for (; l < K; ++l) v0 += Gm[(size_t)l * ld + k] * in[l];
                out[k] = (v0 + v1) + (v2 + v3);
            }
            return;
        }
        const int k = tid - grp * rows;
        if (grp < groups && k < K) {
            const int l0 = K * grp / groups, l1 = K * (grp + 1) / groups;
            double v0 = 0.0, v1 = 0.0, v2 = 0.0, v3 = 0.0;
            int l = l0;
            for (; l + 3 < l1; l += 4) {
                v0 += Gm[(size_t)l * ld + k] * in[l];
                v1 += Gm[(size_t)(l + 1) * ld + k] * in[l + 1];
                v2 += Gm[(size_t)(l + 2) * ld + k] * in[l + 2];
                v3 += Gm[(size_t)(l + 3) * ld + k] * in[l + 3];
            }
            for (; l < l1; ++l) v0 += Gm[(size_t)l * ld + k] * in[l];
            sub[grp * rows + k] = (v0 + v1) + (v2 + v3);
        }
        __syncthreads();
        for (int i = tid; i < K; i += T) {                              // (K < T here)
            double v = 0.0;
            for (int gq = 0; gq < groups; ++gq) v += sub[gq * rows + i];
            out[i] = v;
        }
    };
    for (int k = tid; k < K; k += T) xs[k] = s0 && k < fresh ? s0[k] : 0.0;
    __syncthreads();                                                   // (d, G and xs complete)
    if (s0) matvec(xs, q);
    double a = 0.0, b = 0.0, dd, rz, rr;
    for (int k = tid; k < K; k += T) {
        const double g = Gm[(size_t)k * ld + k], dk = d[k];
        dg[k] = g > 0.0 ? 1.0 / g : 1.0;
        r[k] = dk - (s0 ? q[k] : 0.0);
        p[k] = r[k] * dg[k];
        a += dk * dk;
        b += r[k] * r[k] * dg[k];
    }
    sum2(a, b, dd, rz);
    a = 0.0;
    for (int k = tid; k < K; k += T) a += r[k] * r[k];
    sum2(a, 0.0, rr, unused);
    int it = 0;
    bool converged = !(dd > 0.0) || rr <= 1e-26 * dd;                  // (a warm start may already fit)
    const int max_it = 20 * K + 20;
    while (!converged && it < max_it) {
        matvec(p, q);
        a = 0.0;
        for (int k = tid; k < K; k += T) a += p[k] * q[k];
        double pq;
        sum2(a, 0.0, pq, unused);
        if (!(pq > 0.0)) break;                                        // direction in the null space: done
        const double alpha = rz / pq;
        a = b = 0.0;
        for (int k = tid; k < K; k += T) {
            xs[k] += alpha * p[k];
            const double rk = r[k] - alpha * q[k];
            r[k] = rk;
            a += rk * rk;
            b += rk * rk * dg[k];
        }
        double rz_new;
        sum2(a, b, rr, rz_new);
        ++it;
        if (rr <= 1e-26 * dd) {
            converged = true;
            break;
        }
        const double beta = rz_new / rz;
        rz = rz_new;
        for (int k = tid; k < K; k += T) p[k] = r[k] * dg[k] + beta * p[k];
        __syncthreads();
    }
    for (int k = tid; k < K; k += T) s[k] = xs[k];
    if (tid == 0 && iters) iters[0] = converged ? it : -it;
}
__global__ void __launch_bounds__(1024)
tsvd_pcg_kernel(const double* __restrict__ G, long long ldg, double* __restrict__ d, int K, double* __restrict__ s,
                const double* __restrict__ s0, int* __restrict__ iters, const double* __restrict__ part, int fresh, int M) {
    extern __shared__ __align__(16) unsigned char smem[];
    solve_pcg(smem, (int)blockDim.x, G, ldg, d, K, s, s0, iters, part, fresh, M);
}

// ---- Eq. (3), the solve while Algorithm 2 has at most 64 components: one row of the triangular factor more per component ----
// G = L D L^T (L unit lower triangular) grows by a row and a column per component, and so do L (a forward substitution), D and w = L^-1 d (one
// entry each); only the back substitution L^T s = D^-1 w runs over everything.  One wavefront, a row per lane: a step of either
// substitution is a lane broadcast and a multiply-add on an entry of L that was read ahead; L is held with zeros on and above its diagonal, so
// that lanes already done are left alone without a choice.  32 components take 64 steps, where conjugate gradients took some twenty
// iterations of 2000 cycles (19 us) and a Cholesky factor with a multiplication by 1 / l_jj in every step 170 cycles each: 5.3 us a launch, now 4.3.
// L [CHOL_K][CHOL_K], 1 / D and w live in `factor` between the calls.  A pivot below 1e-10 of its diagonal entry (two components
// that nearly coincide) sets factor's last word, and this and all later calls go through conjugate gradients.
#define CHOL_K 64
#define CHOL_DOUBLES (CHOL_K * CHOL_K + 2 * CHOL_K + 1)
#define CHOL_PITCH (CHOL_K + 1)
__global__ void __launch_bounds__(256)
tsvd_scales_kernel(const double* __restrict__ G, long long ldg, double* __restrict__ d, int K, double* __restrict__ s,
                   const double* __restrict__ s0, const double* __restrict__ part, int fresh, int M, double* __restrict__ factor) {
    extern __shared__ __align__(16) unsigned char smem[];
    double* Ll = reinterpret_cast<double*>(smem);           // [K rounded up to 8][CHOL_PITCH], zero on and above the diagonal
    __shared__ double tot[CHOL_K][4];
    __shared__ int singular;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double* w = factor + CHOL_K * CHOL_K;
    double* dinv = w + CHOL_K;
    double* marked = dinv + CHOL_K;
    if (tid == 0) singular = marked[0] != 0.0;
#pragma unroll 4
    for (int e = tid; e < fresh * CHOL_K; e += 256) Ll[(e >> 6) * CHOL_PITCH + (e & 63)] = factor[e];
    for (int e = fresh * CHOL_K + tid; e < ((K + 7) & ~7) * CHOL_K; e += 256) Ll[(e >> 6) * CHOL_PITCH + (e & 63)] = 0.0;
    for (int k = fresh; k < K; ++k) {
        double a = 0.0;
        for (int m = tid; m < M; m += 256) a += part[(size_t)(k - fresh) * M + m];
        a = wave_sum(a);
        if (lane == 0) tot[k][wave] = a;
    }
    __syncthreads();
    if (wave == 0 && !singular) {
        auto broadcast = [](double v, int from) {
            const uint64_t b = __builtin_bit_cast(uint64_t, v);
            return __builtin_bit_cast(double, (uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)b, from) |
                                                  ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(b >> 32), from) << 32));
        };
        double inv = lane < fresh ? dinv[lane] : 0.0, wl = lane < fresh ? w[lane] : 0.0;
        bool bad = false;
        for (int r = fresh; r < K && !bad; ++r) {
            const double* row = Ll + min(lane, r) * CHOL_PITCH;                // (row r itself is zero still)
            double x = lane <= r ? G[(size_t)r * ldg + lane] : 0.0;
            const double dr = (tot[r][0] + tot[r][1]) + (tot[r][2] + tot[r][3]), grr = broadcast(x, r);
            if (lane >= r) x = 0.0;
            for (int j0 = 0; j0 < r; j0 += 8) {             // (steps at and beyond r meet zeros)
                double e[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) e[t] = row[j0 + t];
#pragma unroll
                for (int t = 0; t < 8; ++t) x -= broadcast(x, j0 + t) * e[t];
            }
            const double l = x * inv, pivot = grr - wave_sum(x * l), dot = wave_sum(l * wl);
            bad = !(pivot > 1e-10 * grr);
            if (lane == r) {
                inv = 1.0 / pivot;
                wl = dr - dot;
                d[r] = dr;
            }
            Ll[r * CHOL_PITCH + lane] = l;
            factor[r * CHOL_K + lane] = l;
        }
        if (bad) {
            if (lane == 0) {
                singular = 1;
                marked[0] = 1.0;
            }
        } else {
            if (lane >= fresh && lane < K) {
                w[lane] = wl;
                dinv[lane] = inv;
            }
            double x = wl * inv;
            for (int j0 = (K - 1) & ~7; j0 >= 0; j0 -= 8) {                     // (rows from K on are zero)
                double e[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) e[t] = Ll[(j0 + t) * CHOL_PITCH + lane];
#pragma unroll
                for (int t = 7; t >= 0; --t) x -= broadcast(x, j0 + t) * e[t];
            }
            if (lane < K) s[lane] = x;
        }
    }
    __syncthreads();
    if (singular) solve_pcg(smem, 256, G, ldg, d, K, s, s0, nullptr, part, fresh, M);
}

// ---- residual: R = W - U diag(S) V and partial sums of |R|_F^2 ----------------------------------
// One workgroup per row m; the scaled row of U (S_k U[m][k], non-zero entries only) is gathered in
// LDS once, then every thread owns columns n, n + 256, ...
__global__ void __launch_bounds__(256)
tsvd_residual_kernel(const double* __restrict__ W, const int8_t* __restrict__ U, long long ldu, const double* __restrict__ S,
                     const int8_t* __restrict__ V, int K, int N, double* __restrict__ R, double* __restrict__ partial) {
    extern __shared__ __align__(16) unsigned char smem[];
    double* us = reinterpret_cast<double*>(smem);               // [K]
    __shared__ double red[256];
    const int m = blockIdx.x;
    for (int k = threadIdx.x; k < K; k += 256) us[k] = (double)U[(size_t)m * ldu + k] * S[k];
    __syncthreads();
    double ss = 0.0;
    for (int n = threadIdx.x; n < N; n += 256) {
        double acc = 0.0;
        for (int k = 0; k < K; ++k) acc += us[k] * (double)V[(size_t)k * N + n];
        const double rv = W[(size_t)m * N + n] - acc;
        R[(size_t)m * N + n] = rv;
        ss += rv * rv;
    }
    const double total = block_sum256(ss, red);
    if (threadIdx.x == 0 && partial) partial[m] = total;
}

// The same inside Algorithm 2, on the component-major factors Ut [rank][mp], V [rank][np]: grid (ceil(N / 256), ceil(M / 4)),
// a wavefront per row, four columns per lane (one 4-byte load of V serves them and hits L1 for three of the four
// wavefronts).  part[m * gridDim.x + blockIdx.x] = sum of squares of that piece, in host memory: the host adds them (a
// copy back to the host after the launch would cost more than the launch); with them goes what the device has to report.
struct transition_state {
    tsvd_pair_shifts pair;
    int failed;              // ternarizations without a result
};
struct transition_report {
    int missed, needed, shifted_missed, shifted_needed;      // of the pairs' squarings (tsvd_pair_state)
    int failed;
    int resolved;            // all pairs have left their second eigenvalue, and none was far below the first
};
static_assert(sizeof(transition_report) % 8 == 0, "doubles follow it");
__global__ void __launch_bounds__(256)
tsvd_residual_rows_kernel(const double* __restrict__ W, const int8_t* __restrict__ Ut, int mp, const double* __restrict__ S,
                          const int8_t* __restrict__ V, int np, int M, int N, int K, double* __restrict__ R, double* __restrict__ part,
                          transition_state* __restrict__ seen, transition_report* __restrict__ told) {
    extern __shared__ __align__(16) unsigned char smem[];
    double* us = reinterpret_cast<double*>(smem);               // [4][K]
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        tsvd_pair_state& of = seen->pair.state;
        told[0] = {of.missed, of.needed, of.shifted_missed, of.shifted_needed, seen->failed, of.far == 0 && seen->pair.second > 0.0};
        of.missed = of.needed = of.shifted_missed = of.shifted_needed = of.far = 0;      // (of one iteration each)
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m0 = blockIdx.y * 4, m = m0 + wave, n = blockIdx.x * 256 + 4 * lane;
    for (int k = threadIdx.x; k < K; k += 256) {
        const int w = *reinterpret_cast<const int*>(Ut + (size_t)k * mp + m0);
        const double sk = S[k];
#pragma unroll
        for (int e = 0; e < 4; ++e) us[e * K + k] = (double)(int8_t)(w >> (8 * e)) * sk;
    }
    __syncthreads();
    if (m >= M) return;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const int nc = min(n, np - 4);
#pragma unroll 8
    for (int k = 0; k < K; ++k) {
        const int w = *reinterpret_cast<const int*>(V + (size_t)k * np + nc);
        const double u = us[wave * K + k];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += u * (double)(int8_t)(w >> (8 * e));
    }
    double ss = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (n + e < N) {
            const double rv = W[(size_t)m * N + n + e] - acc[e];
            R[(size_t)m * N + n + e] = rv;
            ss += rv * rv;
        }
    ss = wave_sum(ss);
    if (lane == 0) part[(size_t)m * ((N + 255) >> 8) + blockIdx.x] = ss;
}

// The result of Algorithm 2 from its component-major scratch: U [M][max_rank] (zero from K on), V [K][N], S [max_rank] (zero from K on).
__global__ void __launch_bounds__(256)
tsvd_emit_kernel(const int8_t* __restrict__ Ut, int mp, const int8_t* __restrict__ Vs, int np, const double* __restrict__ Ss, int M, int N, int K,
                 int max_rank, int8_t* __restrict__ U, int8_t* __restrict__ V, double* __restrict__ S) {
    const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x, all = (size_t)gridDim.x * 256;
    for (size_t e = t; e < (size_t)M * max_rank; e += all) {
        const int m = (int)(e / max_rank), k = (int)(e - (size_t)m * max_rank);
        U[e] = k < K ? Ut[(size_t)k * mp + m] : (int8_t)0;
    }
    for (size_t e = t; e < (size_t)K * N; e += all) {
        const int k = (int)(e / N);
        V[e] = Vs[(size_t)k * np + (e - (size_t)k * N)];
    }
    for (size_t e = t; e < (size_t)max_rank; e += all) S[e] = (int)e < K ? Ss[e] : 0.0;
}

// Sum of `count` partial values in a fixed order (one workgroup).
__global__ void __launch_bounds__(256)
tsvd_sum_kernel(const double* __restrict__ partial, int count, double* __restrict__ out) {
    __shared__ double red[256];
    double v = 0.0;
    for (int i = threadIdx.x; i < count; i += 256) v += partial[i];
    const double total = block_sum256(v, red);
    if (threadIdx.x == 0) out[0] = total;
}

// ---- leading singular pair by Golub-Kahan-Lanczos bidiagonalisation ------------------------------------
// R V_k = U_k B_k with B_k upper bidiagonal (alpha on the diagonal, beta above it):
//   u_i = R v_i - beta_{i-1} u_{i-1},  alpha_i = |u_i|;   w = R^T u_i - alpha_i v_i,  beta_i = |w|,  v_{i+1} = w / beta_i,
// every new vector orthogonalised against all earlier ones (classical Gram-Schmidt, twice).  The
// leading singular triple of the small B_k (found on the host) gives that of R; for the close
// singular values of a random matrix this needs tens of steps where the power iteration needs
// thousands.  A step is four launches: the two matrix-vector products run on all compute units
// (tsvd_gkl_rv_kernel: a wavefront per row; tsvd_gkl_rtu_kernel: 64 columns x a slice of the rows per
// workgroup, partial sums), each followed by one workgroup that orthogonalises and normalises the new
// vector with it in LDS (tsvd_gkl_finish_kernel).  (One workgroup doing everything took 100 us per step on
// a [512, 256] matrix, 95 % of the transition's time.)  The bases ub [kmax][M], vb [kmax + 1][N] live in
// global memory (L2).
#define GKL_MAX_STEPS 128
#define GKL_ROW_SLICES 16

// uw[m] = sum_n R[m][n] v[n] - beta_prev * u_prev[m]: one wavefront per row (grid ceil(M / 4), block 256).
__global__ void __launch_bounds__(256)
tsvd_gkl_rv_kernel(const double* __restrict__ R, int M, int N, const double* __restrict__ v, const double* __restrict__ u_prev,
                   const double* __restrict__ beta_prev, double* __restrict__ uw) {
    const int m = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (m >= M) return;
    const double* row = R + (size_t)m * N;
    double a0 = 0.0, a1 = 0.0;
    int n = lane;
    for (; n + 64 < N; n += 128) {
        a0 += row[n] * v[n];
        a1 += row[n + 64] * v[n + 64];
    }
    if (n < N) a0 += row[n] * v[n];
    double a = a0 + a1;
    for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
    if (lane == 0) uw[m] = a - (u_prev ? beta_prev[0] * u_prev[m] : 0.0);
}

// part[slice][n] = sum over the rows of the slice of R[m][n] u[m]: grid (ceil(N / 64), GKL_ROW_SLICES), block 256 =
// 64 columns x 4 row phases.
__global__ void __launch_bounds__(256)
tsvd_gkl_rtu_kernel(const double* __restrict__ R, int M, int N, const double* __restrict__ u, double* __restrict__ part) {
    __shared__ double red[4][64];
    const int col = blockIdx.x * 64 + (threadIdx.x & 63), phase = threadIdx.x >> 6;
    const int m0 = (int)(((long long)M * blockIdx.y) / GKL_ROW_SLICES), m1 = (int)(((long long)M * (blockIdx.y + 1)) / GKL_ROW_SLICES);
    double a0 = 0.0, a1 = 0.0;
    if (col < N) {
        int m = m0 + phase;
        for (; m + 4 < m1; m += 8) {
            a0 += R[(size_t)m * N + col] * u[m];
            a1 += R[(size_t)(m + 4) * N + col] * u[m + 4];
        }
        if (m < m1) a0 += R[(size_t)m * N + col] * u[m];
    }
    red[phase][threadIdx.x & 63] = a0 + a1;
    __syncthreads();
    if (phase == 0 && col < N) part[(size_t)blockIdx.y * N + col] = (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
}

// One workgroup: x = (raw vector, or the sum of `slices` partial vectors minus scale[0] * sub) orthogonalised twice
// against basis[0 .. count), normalised, written to basis[count]; its norm to norm_out[0].  init: x is the fixed start
// vector instead (count = 0).
__global__ void __launch_bounds__(1024)
tsvd_gkl_finish_kernel(const double* __restrict__ raw, int slices, const double* __restrict__ sub, const double* __restrict__ scale,
                       int len, double* __restrict__ basis, int count, double* __restrict__ norm_out, int init) {
    extern __shared__ __align__(16) unsigned char smem[];
    double* x = reinterpret_cast<double*>(smem);    // [len]
    double* part = x + len;                         // [4][len] partial sums of the projections
    double* coef = part + 4 * (size_t)len;          // [GKL_MAX_STEPS + 1]
    double* red = coef + GKL_MAX_STEPS + 1;         // [1024]
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    if (init) {                  // a fixed start vector with no special symmetry
        for (int n = tid; n < len; n += 1024) x[n] = 1.0 + 0.5 * sin(1.0 + 0.7 * (double)n);
    } else {
        const double sc = sub ? scale[0] : 0.0;
        for (int e = tid; e < len; e += 1024) {
            double a = raw[e];
            for (int q = 1; q < slices; ++q) a += raw[(size_t)q * len + e];
            x[e] = a - (sub ? sc * sub[e] : 0.0);
        }
    }
    __syncthreads();
    for (int pass = 0; pass < 2 && count > 0; ++pass) {
        // four basis vectors per wavefront at a time: their loads overlap
        for (int j0 = wave * 4; j0 < count; j0 += 64) {
            double a[4] = {0.0, 0.0, 0.0, 0.0};
            // (sixteen loads in flight per lane: the loop waits for L2, not for arithmetic; 4.07 -> 3.59 ms per iteration
            // of Algorithm 2 on a [512, 256] matrix; 32 in flight: 3.77)
            for (int e0 = lane; e0 < len; e0 += 256) {
                double b[4][4];
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int t = 0; t < 4; ++t) b[c][t] = basis[(size_t)min(j0 + t, count - 1) * len + min(e0 + 64 * c, len - 1)];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const double xe = e0 + 64 * c < len ? x[e0 + 64 * c] : 0.0;
#pragma unroll
                    for (int t = 0; t < 4; ++t) a[t] += b[c][t] * xe;
                }
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                for (int o = 32; o > 0; o >>= 1) a[t] += __shfl_xor(a[t], o, 64);
                if (lane == 0 && j0 + t < count) coef[j0 + t] = a[t];
            }
        }
        __syncthreads();
        // x[e] -= sum_j coef[j] basis_j[e]: for short vectors the basis range is split over groups of threads
        const int groups = len <= 256 ? 4 : len <= 512 ? 2 : 1, per = 1024 / groups;
        const int grp = tid / per, t = tid - grp * per;
        const int j0 = (count * grp) / groups, j1 = (count * (grp + 1)) / groups;
        for (int e = t; e < len; e += per) {
            double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
            int j = j0;
            for (; j + 3 < j1; j += 4) {
                a0 += coef[j] * basis[(size_t)j * len + e];
                a1 += coef[j + 1] * basis[(size_t)(j + 1) * len + e];
                a2 += coef[j + 2] * basis[(size_t)(j + 2) * len + e];
                a3 += coef[j + 3] * basis[(size_t)(j + 3) * len + e];
            }
            for (; j < j1; ++j) a0 += coef[j] * basis[(size_t)j * len + e];
            part[(size_t)grp * len + e] = (a0 + a1) + (a2 + a3);
        }
        __syncthreads();
        for (int e = tid; e < len; e += 1024) {
            double a = x[e];
            for (int gq = 0; gq < groups; ++gq) a -= part[(size_t)gq * len + e];
            x[e] = a;
        }
        __syncthreads();
    }
    double ss = 0.0;
    for (int e = tid; e < len; e += 1024) ss += x[e] * x[e];
    red[tid] = ss;
    __syncthreads();
    for (int st = 512; st > 0; st >>= 1) {
        if (tid < st) red[tid] += red[tid + st];
        __syncthreads();
    }
    const double nrm = sqrt(red[0]);
    for (int e = tid; e < len; e += 1024) basis[(size_t)count * len + e] = nrm > 0.0 ? x[e] / nrm : 0.0;
    if (tid == 0 && norm_out) norm_out[0] = nrm;
}

// x = sum_j c_j basis_j (j < count), normalised; one workgroup per output vector (blockIdx.x: 0 = u, 1 = v).
__global__ void __launch_bounds__(256)
tsvd_combine_kernel(const double* __restrict__ ub, const double* __restrict__ vb, const double* __restrict__ zc,
                    const double* __restrict__ yc, int count, int M, int N, double* __restrict__ u_out, double* __restrict__ v_out) {
    __shared__ double red[256];
    const bool left = blockIdx.x == 0;
    const double* basis = left ? ub : vb;
    const double* c = left ? zc : yc;
    double* out = left ? u_out : v_out;
    const int len = left ? M : N;
    double ss = 0.0;
    for (int e = threadIdx.x; e < len; e += 256) {
        double a = 0.0;
        for (int j = 0; j < count; ++j) a += c[j] * basis[(size_t)j * len + e];
        out[e] = a;
        ss += a * a;
    }
    const double nrm = sqrt(block_sum256(ss, red));
    for (int e = threadIdx.x; e < len; e += 256) out[e] = nrm > 0.0 ? out[e] / nrm : 0.0;
}

// Largest eigenpair of the symmetric tridiagonal matrix (diagonal d, off-diagonal e) of order k, on
// the host: bisection on the Sturm count, then inverse iteration with a pivoted tridiagonal solve.
double tridiagonal_top_eigenpair(const std::vector<double>& d, const std::vector<double>& e, int k, std::vector<double>& x) {
    double lo = 0.0, hi = 0.0;
    for (int i = 0; i < k; ++i) {
        const double r = (i > 0 ? std::fabs(e[i - 1]) : 0.0) + (i + 1 < k ? std::fabs(e[i]) : 0.0);
        hi = std::max(hi, d[i] + r);
        lo = std::min(lo, d[i] - r);
    }
    auto count_below = [&](double xq) {          // number of eigenvalues < xq
        int c = 0;
        double q = 1.0;
        for (int i = 0; i < k; ++i) {
            q = d[i] - xq - (i > 0 ? e[i - 1] * e[i - 1] / q : 0.0);
            if (q == 0.0) q = 1e-300;
            if (q < 0.0) ++c;
        }
        return c;
    };
    double a = lo, b = hi;
    for (int it = 0; it < 200 && b - a > 4e-16 * std::max(std::fabs(a), std::fabs(b)); ++it) {
        const double mid = 0.5 * (a + b);
        if (count_below(mid) >= k) b = mid; else a = mid;      // the largest eigenvalue lies in (a, b]
    }
    const double lam = 0.5 * (a + b);
    // inverse iteration: (T - lam I) x = rhs by Gaussian elimination with partial pivoting (band of width 2)
    x.assign(k, 0.0);
    std::vector<double> rhs(k);
    for (int i = 0; i < k; ++i) rhs[i] = 1.0 + 0.3 * std::sin(1.0 + (double)i);
    const double shift = lam + 1e-13 * std::max(std::fabs(lam), 1e-300);
    for (int round = 0; round < 4; ++round) {
        std::vector<double> dl(k, 0.0), dm(k), du(k, 0.0), du2(k, 0.0), bb = rhs;
        for (int i = 0; i < k; ++i) {
            dm[i] = d[i] - shift;
            if (i + 1 < k) { du[i] = e[i]; dl[i] = e[i]; }
        }
        for (int i = 0; i + 1 < k; ++i) {
            if (std::fabs(dm[i]) >= std::fabs(dl[i])) {
                if (dm[i] == 0.0) dm[i] = 1e-300;
                const double f = dl[i] / dm[i];
                dm[i + 1] -= f * du[i];
                bb[i + 1] -= f * bb[i];
                dl[i] = 0.0;
            } else {                                            // swap rows i and i + 1
                const double f = dm[i] / dl[i];
                dm[i] = dl[i];
                const double t1 = dm[i + 1];
                dm[i + 1] = du[i] - f * t1;
                du[i] = t1;
                if (i + 2 < k) {
                    du2[i] = du[i + 1];
                    du[i + 1] = -f * du2[i];
                }
                std::swap(bb[i], bb[i + 1]);
                bb[i + 1] -= f * bb[i];
            }
        }
        if (dm[k - 1] == 0.0) dm[k - 1] = 1e-300;
        x[k - 1] = bb[k - 1] / dm[k - 1];
        if (k > 1) x[k - 2] = (bb[k - 2] - du[k - 2] * x[k - 1]) / dm[k - 2];
        for (int i = k - 3; i >= 0; --i) x[i] = (bb[i] - du[i] * x[i + 1] - du2[i] * x[i + 2]) / dm[i];
        double nrm = 0.0;
        for (int i = 0; i < k; ++i) nrm += x[i] * x[i];
        nrm = std::sqrt(nrm);
        for (int i = 0; i < k; ++i) x[i] /= nrm;
        rhs = x;
    }
    return lam;
}

int pow2_at_least(int64_t v) {
    int r = 1;
    while (r < v) r *= 2;
    return r;
}

}  // namespace

// R[m][n] -= sigma u[m] v[n]: removes a converged singular triple, so that the next call for the leading pair
// returns the following one (Algorithm 2 with q > 1 takes the top q vectors of the same residual).
__global__ void __launch_bounds__(256)
tsvd_deflate_kernel(double* __restrict__ R, int M, int N, const double* __restrict__ u, const double* __restrict__ v,
                    const double* __restrict__ sigma) {
    const int m = blockIdx.y;
    const double f = sigma[0] * u[m];
    for (int n = blockIdx.x * 256 + threadIdx.x; n < N; n += gridDim.x * 256) R[(size_t)m * N + n] -= f * v[n];
}

namespace {

// `rows` vectors per job; the jobs of a launch share the length of the sorting network.
hipError_t launch_ternarize(const ternarize_job* jobs, int njobs, unsigned rows, double theta, hipStream_t stream) {
    ternarize_args a;
    int n = 1;
    for (int j = 0; j < njobs; ++j) {
        a.job[j] = jobs[j];
        n = std::max(n, jobs[j].n);
    }
    a.npow2 = std::max(64, pow2_at_least(n));
    a.cos_theta = std::cos(theta);
    const dim3 grid(rows, (unsigned)njobs), block((unsigned)std::min(a.npow2, TERN_THREADS));
    switch (std::max(1, a.npow2 / TERN_THREADS)) {
        case 1: hipLaunchKernelGGL(tsvd_ternarize_kernel<1>, grid, block, 0, stream, a); break;
        case 2: hipLaunchKernelGGL(tsvd_ternarize_kernel<2>, grid, block, 0, stream, a); break;
        case 4: hipLaunchKernelGGL(tsvd_ternarize_kernel<4>, grid, block, 0, stream, a); break;
        default: hipLaunchKernelGGL(tsvd_ternarize_kernel<8>, grid, block, 0, stream, a); break;
    }
    return hipGetLastError();
}

// The K x K system of Eq. (3), by the Cholesky factor kept in `factor` (if any) while it is small, else by conjugate gradients; the last `fresh_count` entries of d come from part [fresh_count][M].
void launch_solve(const double* G, long long ldg, double* d, int K, double* s, const double* s0, int* iters, const double* part, int fresh_count,
                int M, double* factor, hipStream_t stream) {
    const bool lds = K <= PCG_LDS_K;
    const size_t bytes = (size_t)5 * K * 8 + 1024 * 8 + (lds ? (size_t)K * K * 8 : 0);
    if (factor && K <= CHOL_K) {
        const size_t rows = (size_t)((K + 7) & ~7) * CHOL_PITCH * 8;           // the factor, or what conjugate gradients need
        hipLaunchKernelGGL(tsvd_scales_kernel, dim3(1), dim3(256), std::max(bytes, rows), stream, G, ldg, d, K, s, s0, part, K - fresh_count, M, factor);
        return;
    }
    hipLaunchKernelGGL(tsvd_pcg_kernel, dim3(1), dim3(lds ? (unsigned)((K + 63) & ~63) : 1024u), bytes, stream, G, ldg, d, K, s, s0, iters, part,
                       K - fresh_count, M);
}

}  // namespace

extern "C" tsvd_status tsvd_ternarize(const double* x_dev, int64_t n, int64_t count, int64_t ldx, double theta, int8_t* t_dev,
                                      int64_t ldt, int32_t* status_dev, void* stream) {
    if (!x_dev || !t_dev || !status_dev || n < 1 || n > TERN_MAX_N || count < 1 || count > (1 << 30) || ldx < n || ldt < n)
        return TSVD_EINVAL;
    const ternarize_job job = {x_dev, (long long)ldx, (int)n, t_dev, (long long)ldt, status_dev, nullptr};
    return launch_ternarize(&job, 1, (unsigned)count, theta, static_cast<hipStream_t>(stream)) == hipSuccess ? TSVD_OK : TSVD_EDEVICE;
}

extern "C" size_t tsvd_fit_scales_workspace(int64_t K) {
    if (K < 1 || K > FIT_MAX_K) return 0;
    return round256((size_t)K * (size_t)K * 8) + round256((size_t)K * 8);      // G, d
}

extern "C" tsvd_status tsvd_fit_scales(const int8_t* U_dev, int64_t ldu, const int8_t* V_dev, const double* W_dev, int64_t M,
                                       int64_t K, int64_t N, double* S_dev, void* workspace, size_t workspace_bytes,
                                       int32_t* iters_dev, void* stream) {
    if (!U_dev || !V_dev || !W_dev || !S_dev || !workspace || M < 1 || N < 1 || K < 1 || K > FIT_MAX_K || ldu < K ||
        M > (1 << 30) || N > (1 << 30))
        return TSVD_EINVAL;
    if (workspace_bytes < tsvd_fit_scales_workspace(K) || (reinterpret_cast<uintptr_t>(workspace) & 255u)) return TSVD_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    double* G = static_cast<double*>(workspace);
    double* d = reinterpret_cast<double*>(static_cast<uint8_t*>(workspace) + round256((size_t)K * (size_t)K * 8));
    hipLaunchKernelGGL(tsvd_gram_kernel, dim3((unsigned)((K + 255) / 256), (unsigned)K), dim3(256), 0, s, U_dev, (long long)ldu,
                       V_dev, (int)M, (int)K, (int)N, G, (long long)K);
    hipLaunchKernelGGL(tsvd_rhs_kernel, dim3((unsigned)K), dim3(256), 0, s, U_dev, (long long)ldu, V_dev, W_dev, (int)M, (int)N, d);
    launch_solve(G, (long long)K, d, (int)K, S_dev, nullptr, iters_dev, nullptr, 0, 0, nullptr, s);
    return hipGetLastError() == hipSuccess ? TSVD_OK : TSVD_EDEVICE;
}

extern "C" tsvd_status tsvd_residual(const double* W_dev, const int8_t* U_dev, int64_t ldu, const double* S_dev,
                                     const int8_t* V_dev, int64_t M, int64_t K, int64_t N, double* R_dev, double* norm2_dev,
                                     void* stream) {
    if (!W_dev || !U_dev || !S_dev || !V_dev || !R_dev || M < 1 || N < 1 || K < 1 || K > FIT_MAX_K || ldu < K || M > (1 << 30) ||
        N > (1 << 30))
        return TSVD_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    double* partial = nullptr;
    if (norm2_dev) {
        // (the partial sums use the output matrix's own stream order: a scratch array per call)
        hipError_t e = hipMallocAsync(reinterpret_cast<void**>(&partial), (size_t)M * 8, s);
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            tsvd_idle_scratch().release();
            e = hipMallocAsync(reinterpret_cast<void**>(&partial), (size_t)M * 8, s);
        }
        if (e != hipSuccess) return TSVD_EDEVICE;
    }
    hipLaunchKernelGGL(tsvd_residual_kernel, dim3((unsigned)M), dim3(256), (size_t)K * 8, s, W_dev, U_dev, (long long)ldu, S_dev,
                       V_dev, (int)K, (int)N, R_dev, partial);
    if (norm2_dev) {
        hipLaunchKernelGGL(tsvd_sum_kernel, dim3(1), dim3(256), 0, s, partial, (int)M, norm2_dev);
        (void)hipFreeAsync(partial, s);
    }
    return hipGetLastError() == hipSuccess ? TSVD_OK : TSVD_EDEVICE;
}

extern "C" size_t tsvd_leading_singular_pair_workspace(int64_t M, int64_t N) {
    if (M < 1 || N < 1 || M > TERN_MAX_N || N > TERN_MAX_N) return 0;
    if (tsvd_pair_squares(M, N)) return tsvd_pair_bytes(M, N);
    return round256((size_t)GKL_MAX_STEPS * M * 8) + round256((size_t)(GKL_MAX_STEPS + 1) * N * 8) + 4 * round256(GKL_MAX_STEPS * 8) +
           round256((size_t)M * 8) + round256((size_t)GKL_ROW_SLICES * N * 8);      // raw R v, partial R^T u
}

extern "C" tsvd_status tsvd_leading_singular_pair(const double* R_dev, int64_t M, int64_t N, int32_t max_steps, double* u_dev,
                                                  double* v_dev, double* sigma_dev, int32_t* steps_dev, void* workspace,
                                                  size_t workspace_bytes, void* stream) {
    if (!R_dev || !u_dev || !v_dev || !sigma_dev || !workspace || M < 1 || N < 1 || M > TERN_MAX_N || N > TERN_MAX_N ||
        max_steps < 1)
        return TSVD_EINVAL;
    if (workspace_bytes < tsvd_leading_singular_pair_workspace(M, N) || (reinterpret_cast<uintptr_t>(workspace) & 255u))
        return TSVD_EINVAL;
    if (tsvd_pair_squares(M, N)) {
        // squarings until the matrix is numerically of rank one; the host looks at the state now and then
        hipStream_t s = static_cast<hipStream_t>(stream);
        tsvd_pair_plan plan;
        tsvd_pair_prepare(M, N, workspace, &plan, s);
        const int limit = std::min(TSVD_PAIR_MAX_SQUARINGS, std::max(1, (int)max_steps));
        int count = 0;
        for (tsvd_pair_state state = {-1, 0, 0, 0, 0, 0}; count < limit && state.last < 0;) {
            const int to = std::min(limit, count == 0 ? 16 : count + 8);
            tsvd_pair_square(plan, R_dev, count, to, false, s);
            count = to;
            if (hipMemcpyAsync(&state, plan.state, sizeof state, hipMemcpyDeviceToHost, s) != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
                return TSVD_EDEVICE;
        }
        tsvd_pair_vectors(plan, R_dev, count, false, false, s);
        tsvd_pair_normalise(plan, count, u_dev, v_dev, sigma_dev, steps_dev, s);
        return hipGetLastError() == hipSuccess ? TSVD_OK : TSVD_EDEVICE;
    }
    auto finish_lds = [](int64_t len) { return ((size_t)5 * (size_t)len + GKL_MAX_STEPS + 1 + 1024) * 8; };
    if (finish_lds(std::max(M, N)) > 150 * 1024) return TSVD_EUNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint8_t* w8 = static_cast<uint8_t*>(workspace);
    double* ub = reinterpret_cast<double*>(w8);
    double* vb = reinterpret_cast<double*>(w8 + round256((size_t)GKL_MAX_STEPS * M * 8));
    double* alpha = reinterpret_cast<double*>(reinterpret_cast<uint8_t*>(vb) + round256((size_t)(GKL_MAX_STEPS + 1) * N * 8));
    double* beta = alpha + round256(GKL_MAX_STEPS * 8) / 8;
    double* zc = beta + round256(GKL_MAX_STEPS * 8) / 8;
    double* yc = zc + round256(GKL_MAX_STEPS * 8) / 8;
    double* uw = yc + round256(GKL_MAX_STEPS * 8) / 8;                          // R v_i before orthogonalisation
    double* wpart = uw + round256((size_t)M * 8) / 8;                           // [GKL_ROW_SLICES][N] partial R^T u_i
    const int kmax = (int)std::min<int64_t>(GKL_MAX_STEPS, std::min(M, N));   // the Krylov space cannot outgrow the matrix
    std::vector<double> ha(GKL_MAX_STEPS), hb(GKL_MAX_STEPS), d, e, y, z;
    int total = 0, fresh = 1;
    double theta = 0.0;
    for (;;) {
        int k = 0;
        bool done = false;
        while (!done) {
            const int k1 = std::min(kmax, k == 0 ? std::min(32, kmax) : k + 16);
            if (k == 0 && fresh)       // a restart finds its start vector in vb[0]
                hipLaunchKernelGGL(tsvd_gkl_finish_kernel, dim3(1), dim3(1024), finish_lds(N), s, static_cast<const double*>(nullptr), 0,
                                   static_cast<const double*>(nullptr), static_cast<const double*>(nullptr), (int)N, vb, 0,
                                   static_cast<double*>(nullptr), 1);
            for (int i = k; i < k1; ++i) {
                const double* vi = vb + (size_t)i * N;
                hipLaunchKernelGGL(tsvd_gkl_rv_kernel, dim3((unsigned)((M + 3) / 4)), dim3(256), 0, s, R_dev, (int)M, (int)N, vi,
                                   i > 0 ? ub + (size_t)(i - 1) * M : static_cast<const double*>(nullptr), i > 0 ? beta + (i - 1) : beta, uw);
                hipLaunchKernelGGL(tsvd_gkl_finish_kernel, dim3(1), dim3(1024), finish_lds(M), s, uw, 1, static_cast<const double*>(nullptr),
                                   static_cast<const double*>(nullptr), (int)M, ub, i, alpha + i, 0);
                hipLaunchKernelGGL(tsvd_gkl_rtu_kernel, dim3((unsigned)((N + 63) / 64), GKL_ROW_SLICES), dim3(256), 0, s, R_dev, (int)M, (int)N,
                                   ub + (size_t)i * M, wpart);
                hipLaunchKernelGGL(tsvd_gkl_finish_kernel, dim3(1), dim3(1024), finish_lds(N), s, wpart, GKL_ROW_SLICES, vi, alpha + i, (int)N,
                                   vb, i + 1, beta + i, 0);
            }
            if (hipMemcpyAsync(ha.data(), alpha, (size_t)k1 * 8, hipMemcpyDeviceToHost, s) != hipSuccess ||
                hipMemcpyAsync(hb.data(), beta, (size_t)k1 * 8, hipMemcpyDeviceToHost, s) != hipSuccess ||
                hipStreamSynchronize(s) != hipSuccess)
                return TSVD_EDEVICE;
            total += k1 - k;
            k = k1;
            // leading singular triple of the k x k upper bidiagonal B through T = B^T B
            d.assign(k, 0.0);
            e.assign(k > 1 ? k - 1 : 0, 0.0);
            for (int i = 0; i < k; ++i) {
                d[i] = ha[i] * ha[i] + (i > 0 ? hb[i - 1] * hb[i - 1] : 0.0);
                if (i + 1 < k) e[i] = ha[i] * hb[i];
            }
            const double lam = tridiagonal_top_eigenpair(d, e, k, y);
            theta = std::sqrt(std::max(lam, 0.0));
            z.assign(k, 0.0);
            for (int i = 0; i < k; ++i) z[i] = theta > 0.0 ? (ha[i] * y[i] + (i + 1 < k ? hb[i] * y[i + 1] : 0.0)) / theta : 0.0;
            const double resid = hb[k - 1] * std::fabs(z[k - 1]);        // |R^T u - theta v| of the Ritz pair
            done = resid <= 1e-12 * theta || k >= kmax || total >= max_steps || !(theta > 0.0);
            if (done) {
                if (hipMemcpyAsync(zc, z.data(), (size_t)k * 8, hipMemcpyHostToDevice, s) != hipSuccess ||
                    hipMemcpyAsync(yc, y.data(), (size_t)k * 8, hipMemcpyHostToDevice, s) != hipSuccess)
                    return TSVD_EDEVICE;
                hipLaunchKernelGGL(tsvd_combine_kernel, dim3(2), dim3(256), 0, s, ub, vb, zc, yc, k, (int)M, (int)N, u_dev, v_dev);
                if (hipStreamSynchronize(s) != hipSuccess) return TSVD_EDEVICE;    // (z, y are host vectors reused below)
                if (resid <= 1e-12 * theta || total >= max_steps || !(theta > 0.0) || kmax < GKL_MAX_STEPS) {
                    if (hipMemcpy(sigma_dev, &theta, 8, hipMemcpyHostToDevice) != hipSuccess) return TSVD_EDEVICE;
                    if (steps_dev && hipMemcpy(steps_dev, &total, 4, hipMemcpyHostToDevice) != hipSuccess) return TSVD_EDEVICE;
                    return hipGetLastError() == hipSuccess ? TSVD_OK : TSVD_EDEVICE;
                }
            }
        }
        // not converged within the basis: restart from the current estimate of v
        if (hipMemcpyAsync(vb, v_dev, (size_t)N * 8, hipMemcpyDeviceToDevice, s) != hipSuccess) return TSVD_EDEVICE;
        fresh = 0;
    }
}

hipError_t tsvd_transition_init() {
    hipError_t e;
    if ((e = tsvd_pair_init()) != hipSuccess) return e;
    if ((e = hipFuncSetAttribute(reinterpret_cast<const void*>(tsvd_pcg_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 std::max(5 * FIT_MAX_K * 8, 5 * PCG_LDS_K * 8 + PCG_LDS_K * PCG_LDS_K * 8) + 1024 * 8)) != hipSuccess) return e;
    if ((e = hipFuncSetAttribute(reinterpret_cast<const void*>(tsvd_residual_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 FIT_MAX_K * 8)) != hipSuccess) return e;
    if ((e = hipFuncSetAttribute(reinterpret_cast<const void*>(tsvd_residual_rows_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 4 * FIT_MAX_K * 8)) != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(tsvd_gkl_finish_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
}

namespace {
// of this thread's last transition, for tsvd_tuning_transition_shifts
thread_local int shifts_kept = 0, shifts_again = 0;
}  // namespace

extern "C" tsvd_status tsvd_transition(const double* W_dev, int64_t M, int64_t N, double theta, double tol, int64_t max_rank,
                                       int8_t* U_dev, double* S_dev, int8_t* V_dev, int64_t* rank_out, double* errors_host,
                                       void* stream) {
    return tsvd_transition_q(W_dev, M, N, theta, tol, max_rank, 1, U_dev, S_dev, V_dev, rank_out, errors_host, stream);
}

extern "C" tsvd_status tsvd_transition_q(const double* W_dev, int64_t M, int64_t N, double theta, double tol, int64_t max_rank,
                                         int64_t q, int8_t* U_dev, double* S_dev, int8_t* V_dev, int64_t* rank_out,
                                         double* errors_host, void* stream) {
    if (!W_dev || !U_dev || !S_dev || !V_dev || !rank_out || M < 1 || N < 1 || M > TERN_MAX_N || N > TERN_MAX_N || max_rank < 1 ||
        max_rank > FIT_MAX_K || !(tol >= 0.0) || q < 1 || q > max_rank || q > std::min(M, N))
        return TSVD_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    *rank_out = 0;
    shifts_kept = shifts_again = 0;
    // The host waits for what is enqueued, so there is nothing to capture; refused before anything is, or a graph could be left with work on scratch that belongs to the next call.
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();
        return TSVD_EDEVICE;
    }
    const bool squares = tsvd_pair_squares(M, N);
    const int mp = (int)((M + 15) & ~15), np = (int)((N + 15) & ~15);       // pitches of the component-major factors
    const int pieces = (int)((N + 255) / 256);                              // pieces of a row of the residual
    // scratch
    size_t total = 0;
    auto reserve = [&](size_t bytes) {
        const size_t at = total;
        total += round256(bytes);
        return at;
    };
    const size_t at_R = reserve((size_t)M * N * 8);
    const size_t at_Rwork = reserve(q > 1 ? (size_t)M * N * 8 : 0);          // working copy for the second .. q-th triple
    const size_t at_Ut = reserve((size_t)max_rank * mp), at_V = reserve((size_t)max_rank * np);
    const size_t scale_bytes = round256((size_t)max_rank * 8);
    const size_t at_S = reserve(3 * scale_bytes), at_d = reserve((size_t)max_rank * 8);
    const size_t at_G = reserve((size_t)max_rank * max_rank * 8);
    const size_t at_factor = reserve((size_t)CHOL_DOUBLES * 8);
    const size_t at_part = reserve((size_t)q * M * 8);
    const size_t at_report = reserve(sizeof(transition_state));
    const size_t at_u = reserve((size_t)M * 8), at_v = reserve((size_t)N * 8), at_sigma = reserve(8);
    const size_t bytes_svd = tsvd_leading_singular_pair_workspace(M, N), at_svd = reserve(bytes_svd);
    // what the host reads after an iteration (two in turn, written by the device): the report, and the residual's sums of squares
    const size_t told_bytes = round256(sizeof(transition_report) + (size_t)M * pieces * 8);
    tsvd_scratch scratch;
    if (!tsvd_idle_scratch().take(total, 2 * told_bytes + sizeof(tsvd_pair_shifts), &scratch)) return TSVD_EDEVICE;
    uint8_t *const base = scratch.base, *const pinned = scratch.pinned;
    hipEvent_t* const event = scratch.event;
    double* R = reinterpret_cast<double*>(base + at_R);
    double* Rwork = reinterpret_cast<double*>(base + at_Rwork);
    int8_t* Ut = reinterpret_cast<int8_t*>(base + at_Ut);                    // [max_rank][mp]
    int8_t* Vs = reinterpret_cast<int8_t*>(base + at_V);                     // [max_rank][np]
    double* scales[3];                                                       // of iteration i in [i % 3]; 0: none yet
    for (int e = 0; e < 3; ++e) scales[e] = reinterpret_cast<double*>(base + at_S + e * scale_bytes);
    double* dvec = reinterpret_cast<double*>(base + at_d);
    double* G = reinterpret_cast<double*>(base + at_G);                      // [max_rank][max_rank], grown row by row
    double* factor = reinterpret_cast<double*>(base + at_factor);
    double* part = reinterpret_cast<double*>(base + at_part);
    transition_state* rep = reinterpret_cast<transition_state*>(base + at_report);
    double* u = reinterpret_cast<double*>(base + at_u);
    double* v = reinterpret_cast<double*>(base + at_v);
    double* sigma = reinterpret_cast<double*>(base + at_sigma);

    tsvd_status st = TSVD_OK;
    auto ok = [&](hipError_t e) {
        if (e != hipSuccess && st == TSVD_OK) st = TSVD_EDEVICE;
        return e == hipSuccess;
    };
    // the residual after iteration i, with K components, and the report of it
    auto residual = [&](int64_t i, int64_t K) {
        uint8_t* told = pinned + (i & 1) * told_bytes;
        hipLaunchKernelGGL(tsvd_residual_rows_kernel, dim3((unsigned)pieces, (unsigned)((M + 3) / 4)), dim3(256), (size_t)4 * K * 8, s, W_dev, Ut, mp,
                           scales[i % 3], Vs, np, (int)M, (int)N, (int)K, R, reinterpret_cast<double*>(told + sizeof(transition_report)), rep,
                           reinterpret_cast<transition_report*>(told));
        ok(hipGetLastError());
        ok(hipEventRecord(event[i & 1], s));
    };
    transition_report seen = {};
    double rnorm2 = 0.0;
    auto wait_for = [&](int64_t i) {
        if (st == TSVD_EDEVICE || !ok(hipEventSynchronize(event[i & 1]))) return false;
        const uint8_t* told = pinned + (i & 1) * told_bytes;
        std::memcpy(&seen, told, sizeof seen);
        const double* sq = reinterpret_cast<const double*>(told + sizeof(transition_report));
        rnorm2 = 0.0;
        for (size_t e = 0; e < (size_t)M * pieces; ++e) rnorm2 += sq[e];
        return true;
    };
    ok(hipMemsetAsync(Ut, 0, at_S - at_Ut, s));                              // the padding of the factors
    ok(hipMemsetAsync(rep, 0, sizeof(transition_state), s));
    ok(hipMemsetAsync(factor, 0, (size_t)CHOL_DOUBLES * 8, s));
    tsvd_pair_plan plan;
    if (squares) {
        tsvd_pair_prepare(M, N, base + at_svd, &plan, s);
        plan.state = &rep->pair.state;
        if (q == 1) tsvd_pair_sequence(&plan, &rep->pair);
        u = plan.u;
        v = plan.v;
    }
    residual(0, 0);                                                          // R = W, |W|^2
    // Squarings enqueued per pair: what the iteration before found right (tsvd_pair_tail_kernel).  Where they have to lead to rank one: sixteen
    // (those beyond the ones a pair needs return at once), and two more than the last iteration needed where that is more.  Too few
    // cost the iteration again.
    const bool any_rank = squares && tsvd_pair_any_rank(plan);
    int squarings = squares ? tsvd_pair_first_squarings(plan) : 0;
    // What the first matrix needs is not known: its leading pair is taken before the host waits, and squared on from where it is until that will do,
    // which costs only what is missing.  (Singular values in clusters need up to 35 squarings and equal ones all.  When the whole iteration was
    // taken again, with three squarings more each time, the first 24 components of [512, 256] with all values within 1e-6, four an
    // iteration, took 11.3 ms, now 3.7; a Laplace matrix 2.4 either way.)
    bool first_pair = false;                                                 // in the plan already
    int least = 1;                                                           // squarings that iterations before `least_until` get
    int64_t least_until = 0;
    // With q = 1 pairs are shifted from the second iteration on (tsvd_pair_square), two squarings fewer than without.  One that has to be taken again costs itself, the one behind it and a
    // wait, what 20 to 40 shifted ones save, so shifts are left to where they hold:
    //   - eight to ten squarings.  With fewer the spectrum falls: there is little to save, and shifted pairs could need more than others.  With eleven the edge, 2 % below the second eigenvalue,
    //     leaves more directions above it than plain squarings do (700 x 600, values from 1 down to a half: 6.8 -> 7.2 ms), and where more are needed there are clusters, whose squarings
    //     end by themselves without shifts;
    //   - a second eigenvalue that the last iteration known has not lost beside the first, and more than three directions left in it: behind fewer a step down may lie, from where
    //     the shifts reach too little;
    //   - 128 values and more: the gaps of fewer vary more from one pair to the next (188 x 112, 8 components: 0.65 -> 0.75 ms with shifts, 192 x 125, 40: 3.10 -> 3.26; 512 x 128, 15: 1.23 -> 1.09);
    //   - after one that was taken again only where PAYS_FROM components are left, never after the second.
    // Of 1380 random spectra (128 to 768 values, 6 to 40 components) three take more than 1.05 of the time that they take without shifts, up to 1.10: Laplace, normal, ternary and linear
    // ones 0.89 on the average, groups of equal values 0.97, values above a bulk 0.955, exponentials and low rank with noise 0.98, power laws and close values 1.00.  (With shifts from six squarings on, and as few as
    // three of them, 0.05 of such spectra took 1.15 to 1.6 of it: power laws 1.11 on the average, values above a bulk 1.08, groups 1.05.)  (With more pairs an iteration one that misses
    // takes all of them again: Laplace matrices gained 0.94, four an iteration, a linear spectrum took 1.5 times as long.)
    constexpr int SHIFTS_FROM = 8, SHIFTS_TO = 10, PAYS_FROM = 24;
    const int forced = tsvd_tune("TSVD_TRANSITION_SHIFTED", 0);
    bool resolved = false;
    int shifted[2] = {0, 0};                                                 // squarings of iteration i, where they are shifted, in [i & 1]
    if (any_rank && st == TSVD_OK) {
        tsvd_pair_shifts* left = reinterpret_cast<tsvd_pair_shifts*>(pinned + 2 * told_bytes);
        tsvd_pair_state* state = &left->state;
        for (int from = 0, step = 0;;) {
            tsvd_pair_square(plan, R, from, squarings, false, s);
            tsvd_pair_vectors(plan, R, squarings, true, false, s);
            if (!ok(hipMemcpyAsync(left, &rep->pair, sizeof *left, hipMemcpyDeviceToHost, s)) || !ok(hipStreamSynchronize(s))) break;
            from = squarings;
            first_pair = state->missed == 0 || squarings == TSVD_PAIR_MAX_SQUARINGS;
            squarings = std::min(TSVD_PAIR_MAX_SQUARINGS, first_pair ? std::max(1, state->needed) : std::max(squarings + step + 1, state->needed));
            resolved = left->second > 0.0 && state->far == 0;
            if (first_pair) break;
            step += 4;                                                       // (equal values beside others: the estimate stays short)
            if (!ok(hipMemsetAsync(&rep->pair.state.missed, 0, 5 * sizeof(int), s))) break;       // (and what it needed)
        }
    }
    double wnorm2 = 0.0;
    if (wait_for(0)) wnorm2 = rnorm2;
    // Iteration i: components first .. first + take - 1 from the residual of the one before.
    auto enqueue = [&](int64_t i, int64_t first, int64_t take, bool again) {
        const bool by_shifts = any_rank && q == 1 && std::min(M, N) >= 128 && i > 1 && resolved && !again &&
                               (forced > 0 || (squarings >= SHIFTS_FROM && squarings <= SHIFTS_TO)) && (shifts_again == 0 || (shifts_again == 1 && max_rank - first >= PAYS_FROM));
        const int count = !by_shifts ? squarings : forced > 0 ? std::min(forced, TSVD_PAIR_MAX_SQUARINGS) : squarings - 2;
        shifted[i & 1] = by_shifts ? count : 0;
        // the top q singular triples of the residual, one after the other: the leading triple of R, then of R with
        // that triple removed, ... (the last iteration takes what still fits below max_rank)
        const double* src = R;
        if (take > 1) {
            if (!ok(hipMemcpyAsync(Rwork, R, (size_t)M * N * 8, hipMemcpyDeviceToDevice, s))) return;
            src = Rwork;
        }
        for (int64_t j = 0; j < take; ++j) {
            if (squares) {
                if (!first_pair) {
                    tsvd_pair_square(plan, src, 0, count, by_shifts, s);
                    tsvd_pair_vectors(plan, src, count, any_rank, by_shifts, s);
                }
                first_pair = false;
                if (j + 1 < take) tsvd_pair_deflate(plan, Rwork, s);
            } else {
                const tsvd_status ps = tsvd_leading_singular_pair(src, M, N, 4 * GKL_MAX_STEPS, u, v, sigma, nullptr, base + at_svd, bytes_svd, s);
                if (ps != TSVD_OK) {
                    st = ps;
                    return;
                }
                if (j + 1 < take)
                    hipLaunchKernelGGL(tsvd_deflate_kernel, dim3((unsigned)std::min<int64_t>(16, (N + 255) / 256), (unsigned)M), dim3(256), 0, s,
                                       Rwork, (int)M, (int)N, u, v, sigma);
            }
            const ternarize_job jobs[2] = {{u, M, (int)M, Ut + (size_t)(first + j) * mp, mp, nullptr, &rep->failed},
                                           {v, N, (int)N, Vs + (size_t)(first + j) * np, np, nullptr, &rep->failed}};
            if (!ok(launch_ternarize(jobs, 2, 1, theta, s))) return;
        }
        // Eq. (3) with what changed only: the new rows / columns of the Gram matrix and entries of the right
        // side; the solve starts from the previous scales (the new ones at 0)
        const int64_t K = first + take;
        hipLaunchKernelGGL(tsvd_system_kernel, dim3((unsigned)((K + M + 3) / 4), (unsigned)take), dim3(256), 0, s, Ut, mp, Vs, np, W_dev, (int)M, (int)N,
                           (int)first, (int)K, G, (long long)max_rank, part);
        launch_solve(G, (long long)max_rank, dvec, (int)K, scales[i % 3], scales[(i + 2) % 3], nullptr, part, (int)take, (int)M, factor, s);
        residual(i, K);
    };
    // With squarings one iteration is always enqueued beyond the one the host waits for: it costs nothing where the loop goes on, and
    // where the loop ends nothing of it is used (its components lie beyond the rank, its scales in a buffer of their own).  The
    // Lanczos process waits for the device itself: there the next iteration is enqueued once the loop is known to go on.
    int64_t K = 0, i = 1, ahead = 0;                                         // ahead: components enqueued
    int64_t take = std::min<int64_t>(q, max_rank);
    if (st == TSVD_OK && wnorm2 > 0.0) {
        enqueue(1, 0, take, false);
        ahead = take;
        while (st == TSVD_OK) {
            const int64_t next = std::min<int64_t>(q, max_rank - ahead);
            if (squares && next > 0) enqueue(i + 1, ahead, next, false);
            if (st != TSVD_OK || !wait_for(i)) break;
            resolved = seen.resolved != 0;
            const bool missed = seen.missed != 0 && seen.needed < TSVD_PAIR_MAX_SQUARINGS;
            if (missed || seen.shifted_missed != 0) {
                // some pair needed more squarings: back to the residual before this iteration, with more of them, and for a while
                // with one more than were too few (spectra on the edge of two counts missed every eighth iteration)
                if (seen.shifted_missed != 0) {
                    ++shifts_again;
                    squarings = std::max(squarings, std::min(seen.shifted_needed + 1, tsvd_pair_first_squarings(plan)));      // (without shifts; not known where many are alike)
                }
                if (missed) {
                    if (any_rank && i > 1) {
                        least = std::min(seen.needed, squarings + 1);
                        least_until = i + 16;
                    }
                    squarings = std::min(TSVD_PAIR_MAX_SQUARINGS, seen.needed + (any_rank ? 0 : 8));
                }
                if (!ok(hipStreamSynchronize(s)) || !ok(hipMemsetAsync(rep, 0, sizeof(transition_state), s))) break;
                residual(i - 1, K);
                enqueue(i, K, take, true);
                ahead = K + take;
                continue;
            }
            if (seen.failed != 0) {
                st = TSVD_EVALUE;           // no ternary vector within theta: the components of an unfinished iteration are dropped
                break;
            }
            if (const int had = shifted[i & 1]; had > 0) {
                ++shifts_kept;
                if (seen.shifted_needed < had) resolved = false;             // (few directions left: a step down may lie ahead)
                squarings = std::max(squarings, std::min(TSVD_PAIR_MAX_SQUARINGS, seen.shifted_needed + 2));
            }
            if (seen.needed > 0 || !any_rank) squarings = std::min(TSVD_PAIR_MAX_SQUARINGS, any_rank ? std::max(i < least_until ? least : 1, seen.needed) : std::max(16, seen.needed + 2));
            const double err = std::sqrt(rnorm2 / wnorm2);
            if (errors_host)
                for (int64_t r = K; r < K + take; ++r) errors_host[r] = err;      // (one error per iteration, repeated for its components)
            K += take;
            *rank_out = K;
            if (err <= tol || next <= 0) break;
            if (!squares) enqueue(i + 1, ahead, next, false);
            take = next;
            ahead += next;
            ++i;
        }
    }
    const int64_t kept = K == 0 ? 0 : st == TSVD_OK ? i : i - 1;              // the last complete iteration
    if (st == TSVD_OK || st == TSVD_EVALUE)
        hipLaunchKernelGGL(tsvd_emit_kernel, dim3(256), dim3(256), 0, s, Ut, mp, Vs, np, scales[kept % 3], (int)M, (int)N, (int)*rank_out, (int)max_rank, U_dev, V_dev,
                           S_dev);
    const bool done = hipStreamSynchronize(s) == hipSuccess;
    tsvd_idle_scratch().give(scratch, done);
    return st;
}

extern "C" void tsvd_tuning_transition_shifts(int* kept, int* again) {
    *kept = shifts_kept;
    *again = shifts_again;
}

extern "C" void tsvd_transition_release(void) { tsvd_idle_scratch().release(); }
