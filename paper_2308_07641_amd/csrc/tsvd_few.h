// Few tokens of bf16 activations, groups of 16 side by side (tsvd_few.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

struct tsvd_blob_header;

struct tsvd_few_args {
    const unsigned char* tiles;           // stage V: V, Kp / 16 strips of Np / 256 tiles; stage U: U, ceil(M / 16) of Kp / 256
    int strips, nkt;
    int strips_wg, rows_log2;             // strips of a workgroup (1 .. 16, a power of two; stage V: 2 at least), log2 of their rows
    int B;
    long long ld;                         // stage V: of x; stage U: of y
    int token_major;                      // likewise
    const uint16_t* x;                    // stage V: bf16 [N][ld] or [B][ld]
    int N;
    const float* S;
    unsigned char* planes;                // records of z [groups of 16 tokens][blocks], Kp / 128 blocks
    int blocks, z_planes;                 // 4 or 5 planes
    void* y;                              // stage U: fp32 or bf16 [M][ld] or [B][ld]
    const float* bias;
    int out_bf16, M;
};

struct tsvd_few_problem {
    const uint8_t* blob;
    const tsvd_blob_header* hd;
    const uint16_t* x;
    long long B, ldx;
    int x_token_major;
    void* y;
    long long ldy;
    int y_token_major, out_bf16;
    const float* bias;
    unsigned char* planes;                // tsvd_few_bytes
    int z_planes;                         // 4 (z off by 2^-19 of the largest of 32 neighbours), or 5 (2^-24)
    int cu_count, stages;                 // (2: stage V, 4: stage U)
};
hipError_t tsvd_few_init();
size_t tsvd_few_bytes(long long Kp, long long B, int z_planes);
// Whether the kernels take such a call: 32-bit offsets reach everything, and there are eight values to read.
bool tsvd_few_fits(const tsvd_blob_header& hd, long long B, long long ldx, bool x_token_major);
hipError_t tsvd_few_launch(const tsvd_few_problem& f, hipStream_t stream);

// Estimate of a call on four planes in microseconds.
struct tsvd_few_call {
    long long M, N, K, B, cus;
    bool x_token_major, x_aligned, out_bf16;      // x_aligned: rows of x start on 16 bytes
};
double tsvd_few_cost(const tsvd_few_call& c);
