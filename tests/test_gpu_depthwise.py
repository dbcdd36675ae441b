"""Depth-wise convolutions on the matrix cores, at the edges of their tiles and strips, against the oracle: exact on integer
instances, fp32 sums on random ones."""
import numpy as np
import pytest

import workloads
from oracle import conv as oc
from test_gpu_conv import _run, tsvd  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu

CASES = [
    # channels, multiplier, ranks, k1, k2, stride, pad, images, H, W
    (3, 1, 5, 7, 7, 1, 3, 2, 56, 56),       # 16-byte rows, strips of several row counts
    (2, 1, 64, 3, 3, 1, 1, 5, 9, 16),       # the most ranks per group (64)
    (4, 2, 3, 5, 5, 1, 2, 3, 14, 14),       # rows of an even number of elements, two outputs per channel
    (5, 1, 2, 3, 5, 1, 0, 17, 7, 7),        # odd rows, no padding, several images per tile, kernel not square
    (3, 1, 4, 7, 7, 2, 3, 2, 31, 40),       # stride 2: two output rows per tile, an odd number of them
    (2, 3, 3, 5, 3, 2, 4, 4, 12, 10),       # padding wider than half the kernel
    (2, 1, 6, 3, 7, 2, 1, 3, 15, 13),
    (1025, 1, 1, 7, 1, 1, 3, 1, 1, 27),     # one row, a last column tile of one column
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}x{c[1]}_r{c[2]}_{c[3]}x{c[4]}_s{c[5]}_{c[8]}x{c[9]}" for c in CASES])
def test_depthwise_exact_and_random(tsvd, case):  # noqa: F811
    C, mg, kg, k1, k2, st, pad, images, H, W = case
    rng = np.random.default_rng(C + 7 * kg + H)
    G, K, co = max(C, 2), max(C, 2) * kg, max(C, 2) * mg
    geom = ((st, st), (pad, pad), (1, 1))
    print(f"case depthwise {case}", flush=True)
    U = rng.choice([-1, 0, 1], size=(co, K), p=[0.3, 0.4, 0.3]).astype(np.int8)
    V = rng.choice([-1, 0, 1], size=(K, k1 * k2), p=[0.15, 0.7, 0.15]).astype(np.int8)
    S = rng.integers(-2, 3, size=K).astype(np.float32)
    x = rng.integers(-2, 3, size=(images, G, H, W)).astype(np.float32)
    bias = rng.integers(-4, 5, size=co).astype(np.float32)
    ref = oc.tsvd_conv2d(x, U, S, V, 0, co, G, k1, k2, *geom, bias=bias, groups=G)
    for y_dtype in (tsvd.TSVD_F32, tsvd.TSVD_BF16):
        got = _run(tsvd, U, S, V, 0, co, G, k1, k2, workloads.f32_to_bf16_bits(x), geom, bias, y_dtype, G)
        assert got.shape == ref.shape
        want = ref if y_dtype == tsvd.TSVD_F32 else workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(ref.astype(np.float32)))
        assert np.array_equal(got, want)
    S = (rng.standard_normal(K) * 0.3).astype(np.float32)
    xb = workloads.f32_to_bf16_bits(rng.standard_normal(x.shape).astype(np.float32))
    ref = oc.tsvd_conv2d(workloads.bf16_bits_to_f32(xb), U, S, V, 0, co, G, k1, k2, *geom, bias=bias, groups=G)
    got = _run(tsvd, U, S, V, 0, co, G, k1, k2, xb, geom, bias, tsvd.TSVD_F32, G)
    assert np.abs(got - ref).max() <= 1e-6 * np.abs(ref).max()
