"""Both stages of a few tokens in one launch (tsvd_gemv_fused_kernel): the bits of the two launches, which share its arithmetic, over the ends
of its tiles, splits and rounds; and exact on integer instances."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import to_device
from test_gpu_planes import tsvd  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu

CALLS = [
    # M, N, K, B: one tile per stage; one rank, one row, one column; ends beside a strip, a tile and a block of 128 ranks
    (16, 256, 16, 1), (1, 1, 1, 1), (17, 255, 127, 3), (33, 257, 129, 2), (65, 130, 256, 16),
    # columns of V of a wavefront and of two; rounds of strips; the most columns
    (300, 200, 640, 1), (300, 500, 320, 2), (300, 1000, 250, 1), (300, 2000, 128, 4), (500, 3072, 96, 1), (500, 3071, 90, 2),
    # the most tiles of V, ranks beyond 1024 (two for a thread), rows that need several strips a workgroup, and all of a device's workgroups
    (700, 256, 1500, 1), (700, 250, 1536, 2), (5000, 300, 600, 1), (16384, 250, 500, 1), (12000, 100, 1025, 1), (3000, 500, 600, 16)]


@pytest.mark.parametrize("M,N,K,B", CALLS)
@pytest.mark.parametrize("x_dtype", ["f32", "bf16"])
def test_bits_of_the_two_launches(tsvd, M, N, K, B, x_dtype):  # noqa: F811
    import torch
    print(f"case one launch {M} {N} {K} {B} {x_dtype}", flush=True)
    for make in (workloads.make_inputs, workloads.make_integer_inputs):
        i = make(M, N, K, B, 0.5, 0.02, x_dtype, seed=M + K) if make is workloads.make_inputs else make(M, N, K, B, 0.5, x_dtype, seed=M + K)
        h = tsvd.tsvd_pack(i.U, i.S, i.V)
        x = to_device(i)
        assert tsvd.tsvd_tuning_one_launch(h, B)              # (else both calls would take the two launches)
        bias = torch.arange(M, dtype=torch.float32, device="cuda:0") % 7
        rows = torch.full((B, N + 3), float("nan"), dtype=x.dtype, device="cuda:0")      # rows at odd elements, what lies between them is no number
        rows[:, 1:1 + N] = x.t()
        out = []
        for fused in (1, 0):
            # (the switch that is set keeps bf16 calls on the single-token kernels too: no other switch is)
            tsvd.tsvd_tuning_set("TSVD_GEMV_FUSED", fused)
            tsvd.tsvd_tuning_set("TSVD_MID", 0)
            marked = torch.full((B, M + 5), -3.0, dtype=torch.bfloat16, device="cuda:0")
            tsvd.tsvd_forward_io(h, rows[:, 1:1 + N], tsvd.TSVD_TOKEN_MAJOR, bias, marked[:, 2:2 + M], tsvd.TSVD_BF16, tsvd.TSVD_TOKEN_MAJOR)
            out.append((tsvd.tsvd_forward(h, x), marked))
            tsvd.tsvd_tuning_reset()
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
        if make is workloads.make_integer_inputs:
            assert np.array_equal(out[0][0].cpu().numpy(), oracle.forward(i.U, i.S, i.V, i.X))
        tsvd.tsvd_free(h)
