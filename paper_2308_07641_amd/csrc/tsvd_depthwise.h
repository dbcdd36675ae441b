// Depth-wise convolutions on the matrix cores (tsvd_depthwise.hip): the interface to tsvd_conv.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

struct tsvd_depthwise_problem {
    const uint32_t *U, *V;          // code words, and their tiles per 16-row strip
    int u_tps, v_tps;
    const float* S;
    int K, groups, mg, kg;          // rank of the packed triple; per group (one input channel): output channels, ranks
    const uint16_t* x;              // bf16 [groups][images][H][W]
    void* y;                        // fp32 or bf16 [groups mg][images][Ho][Wo]
    const float* bias;
    int out_bf16;
    int images, H, W, Ho, Wo, k1, k2, s1, s2, p1, p2, d1, d2;
    int cu_count;
};
// Enqueues the launch; hipErrorNotSupported where the geometry is not served (nothing is enqueued then).
hipError_t tsvd_depthwise_launch(const tsvd_depthwise_problem& g, hipStream_t stream);
