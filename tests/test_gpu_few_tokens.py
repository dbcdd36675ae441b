"""A few tokens on the single-token kernels side by side, and on the few-token kernels, in every layout: exact on integer
instances, and the bits of single calls for fp32."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import to_device
from test_gpu_planes import _check, tsvd  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("x_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("M,N,K,B", [
    (70, 60, 40, 2), (250, 200, 250, 16),        # one workgroup per token
    (300, 513, 270, 3), (5000, 130, 100, 16),    # two launches; several strips per workgroup, wavefronts without a split
    (40, 4500, 2100, 7), (2100, 300, 4200, 5)])  # several load rounds
def test_tokens_side_by_side(tsvd, M, N, K, B, x_dtype):  # noqa: F811
    import torch
    print(f"case side by side {M} {N} {K} {B} {x_dtype}", flush=True)
    _check(tsvd, M, N, K, B, x_dtype, {})
    i = workloads.make_inputs(M, N, K, B, 0.6, 0.02, x_dtype, seed=M + B)
    h = tsvd.tsvd_pack(i.U, i.S, i.V)
    x = to_device(i)
    y = tsvd.tsvd_forward(h, x)
    for b in range(B):
        assert torch.equal(y[:, b], tsvd.tsvd_forward(h, x[:, b:b + 1].contiguous())[:, 0])
    tsvd.tsvd_free(h)


@pytest.mark.parametrize("M,N,K,B", [(70, 60, 40, 2), (300, 513, 270, 3), (515, 300, 777, 15), (40, 4500, 2100, 7), (640, 2100, 300, 16)])
def test_few_token_kernels(tsvd, M, N, K, B):  # noqa: F811
    """(TSVD_MID = 1 keeps a call of few tokens on them); rows at odd element offsets are copied, with TSVD_REALIGN = 0 gathered."""
    print(f"case few tokens {M} {N} {K} {B}", flush=True)
    _check(tsvd, M, N, K, B, "bf16", {"TSVD_MID": 1}, 1e-3)
    _check(tsvd, M, N, K, B, "bf16", {"TSVD_MID": 1, "TSVD_REALIGN": 0}, 1e-3)


def test_rows_at_odd_offsets_beyond_the_side_by_side_range(tsvd):  # noqa: F811
    """7 tokens of 12 MB of code words: the few-token kernels, on a copy of rows of 7 elements."""
    i = workloads.make_integer_inputs(4096, 4096, 5900, 7, 0.5, "bf16", seed=77)
    h = tsvd.tsvd_pack(i.U, i.S, i.V)
    assert np.array_equal(tsvd.tsvd_forward(h, to_device(i)).cpu().numpy(), oracle.forward(i.U, i.S, i.V, i.X))
    tsvd.tsvd_free(h)
