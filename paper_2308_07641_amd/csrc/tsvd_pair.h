// Leading singular pair of an fp64 matrix by repeated squaring of its Gram matrix (tsvd_pair.hip), as the transition
// (tsvd_transition.hip) uses it.  Everything is enqueued; nothing here waits for the device.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#define TSVD_PAIR_MAX_SQUARINGS 48

// What the device reports about the squarings of one pair.
struct tsvd_pair_state {
    int last;            // index of the squared matrix that is numerically of rank one, -1 while there is none
    int missed;          // pairs since it was last cleared whose squarings were not enough
    int needed;          // most squarings that a pair since it was last cleared should have had
    int shifted_missed, shifted_needed;      // the same of pairs whose squarings were shifted
    int far;             // pairs whose second eigenvalue came out below 2^-30 of the first: with little more between them it is lost in rounding
};
// ... and what pairs leave to the next one of the same sequence (tsvd_pair_sequence): the shifts s and traces t of X_{k+1} = ((X_k - s_k) / t_k)^2, and the second
// eigenvalue of the X_{count} that the pair ended with.
struct tsvd_pair_shifts {
    tsvd_pair_state state;
    int count;
    double second;       // 0: not known
    double first;        // s_0 of the pair that is being squared
    double s[TSVD_PAIR_MAX_SQUARINGS + 1], t[TSVD_PAIR_MAX_SQUARINGS + 1];
};

struct tsvd_pair_plan {
    int M, N;            // of R
    int n, np;           // the shorter side, and rounded up to 64
    double* X[2];        // [np][np] the squared matrices in turn
    double* diag[2];     // [np] their diagonals
    double* v0;          // [N] start vector
    double* s;           // [n] start vector on the shorter side (v0 itself where that is the columns)
    tsvd_pair_state* state;
    bool sequence;       // state is that of a tsvd_pair_shifts
    double *u, *v;       // [M], [N]: the pair, not normalised
};

// Whether the squarings are the faster method for an M x N matrix (the others take Lanczos steps).
bool tsvd_pair_squares(int64_t M, int64_t N);
size_t tsvd_pair_bytes(int64_t M, int64_t N);
// Lays the plan out in `mem` (tsvd_pair_bytes, 256-byte aligned) and enqueues the start vector.
void tsvd_pair_prepare(int64_t M, int64_t N, void* mem, tsvd_pair_plan* plan, hipStream_t stream);
// Makes the pairs taken with the plan a sequence: each one's leading value is expected at the second of the one before or a little above (of 3700 iterations on 240 random matrices 98 in 100 had
// it at 0.99 to 1.3 of it, the lowest at 0.83).  That is no bound: a matrix of rank one taken away would give one, but all scales are fitted again, and residuals differ by as many terms as there
// are.  What results rest on is the tail's look at the image of the edge, and the pair that is taken again without shifts.
void tsvd_pair_sequence(tsvd_pair_plan* plan, tsvd_pair_shifts* shifts);
// Gram matrix of R [M][N] and its squarings `from` .. `to` - 1 (from = 0 computes the Gram matrix first).  shifted (in a sequence, from = 0, of `to` squarings in all): the
// squarings are shifted by what the pair before left.
void tsvd_pair_square(const tsvd_pair_plan& plan, const double* R, int from, int to, bool shifted, hipStream_t stream);
// plan.u and plan.v from the last squared matrix; `count` squarings were enqueued in total.  any_rank: it need not be of rank one (where
// tsvd_pair_any_rank).  shifted: as they were enqueued.
void tsvd_pair_vectors(const tsvd_pair_plan& plan, const double* R, int count, bool any_rank, bool shifted, hipStream_t stream);
bool tsvd_pair_any_rank(const tsvd_pair_plan& plan);
// Squarings after which that is likely to do for a matrix of which nothing is known (sixteen where they have to lead to rank one); the
// device then says what it wants (tsvd_pair_state).
int tsvd_pair_first_squarings(const tsvd_pair_plan& plan);
hipError_t tsvd_pair_init();
// Unit vectors, singular value and number of squarings (steps may be null) of the pair in the plan.
void tsvd_pair_normalise(const tsvd_pair_plan& plan, int count, double* u, double* v, double* sigma, int32_t* steps, hipStream_t stream);
// R -= sigma u v^T for the pair in the plan.
void tsvd_pair_deflate(const tsvd_pair_plan& plan, double* R, hipStream_t stream);
