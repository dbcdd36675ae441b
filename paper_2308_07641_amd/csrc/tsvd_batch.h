// Which kernels a batched linear map runs on (tsvd_batch.hip).
#pragma once
struct tsvd_batch_call {
    long long M, K, N, B, cus;
    bool f32;                       // fp32 activations
    bool x_token_major, y_token_major, out_bf16;
    bool copies;                    // kernels that read aligned feature-major rows would need a copy of x first
    bool x_aligned;                 // rows of x start on 16 bytes
    bool few;                       // the few-token kernels (tsvd_few.hip) may take it
    bool conv;                      // x is the columns of a convolution: other kernels need them written first
    bool whole;                     // both stages run (no diagnostic stage mask)
};
struct tsvd_batch_plan {
    bool few;                       // on the few-token kernels, z in four planes; what follows then says what the call would take else
    int thin;                       // token tiles of a thin panel (tsvd_thin.hip), 0: not on those
    bool split;                     // planes of x, stage V to planes of z, stage U from those (the plane path of tsvd_forward_gemm) ...
    int split_v, split_u;           // ... with these shapes of tsvd_fp6_split_launch, 0: the launches of tsvd_fp6.hip
};
tsvd_batch_plan tsvd_plan_batch(const tsvd_batch_call& c);
// Whether such a call is on the plane path in either layout of x (their margins differ).
bool tsvd_batch_may_split(tsvd_batch_call c);
