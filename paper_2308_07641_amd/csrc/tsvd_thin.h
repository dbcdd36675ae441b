// Both stages of a batch in one launch by thin token panels (tsvd_thin.hip): the interface to the dispatch of the linear map
// (tsvd_api.hip) and to the convolution forms (tsvd_conv.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tsvd_layout.h"

// Where the activations come from.  The gather of a convolution: column (image, py, px) of index (ci, dy, dx) is
// x[ci][image][py s1 + dy d1 - p1][px s2 + dx d2 - p2], zero outside the image.
enum { THIN_FEATURE_MAJOR, THIN_TOKEN_MAJOR, THIN_CONV };
struct tsvd_thin_problem {
    const uint8_t* blob;
    const tsvd_blob_header* hd;
    const uint16_t* x;              // bf16
    int source;
    long long B, ldx;
    int images, H, W, kv1, kv2, Hv, Wv, s1, s2, p1, p2, d1, d2;   // THIN_CONV
    void* y;                        // fp32 (or bf16 with out_bf16) [M][ldy], or [B][ldy] with y_token_major
    long long ldy;
    const float* bias;
    int out_bf16, y_token_major;
    int cus;                        // compute units of the device
};
// Blocks of 128 indices of x that a panel of `tiles` token tiles holds in LDS at a time, 0 where such panels are not possible.
int tsvd_thin_chunk(long long K, long long N, int tiles, bool conv);
hipError_t tsvd_thin_init();
hipError_t tsvd_thin_launch(const tsvd_thin_problem& g, int tiles, hipStream_t stream);
