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


@pytest.mark.parametrize("W", [1, 2, 3, 4, 5, 6, 7, 8, 11, 16, 18, 29])
@pytest.mark.parametrize("k,st", [(3, 1), (5, 1), (7, 1), (3, 2), (5, 2), (7, 2)])
@pytest.mark.parametrize("offset", [0, 1])
def test_depthwise_rows_of_any_width_at_any_element(tsvd, offset, k, st, W):  # noqa: F811
    """Rows of every remainder, x at 16 bytes and one element beyond: the loads that end with a row, at the ends of x too, with infinities on both sides
    of x (nothing from there may reach a result).  Exact."""
    import ctypes

    import torch
    G, kg, images, H = 3, 6, 18, 9
    rng = np.random.default_rng(100 * W + k)
    U = np.kron(np.eye(G, dtype=np.int8), rng.choice([-1, 1], size=(1, kg)).astype(np.int8))
    V = rng.integers(-1, 2, size=(G * kg, k * k)).astype(np.int8)
    S = rng.integers(-2, 3, size=G * kg).astype(np.float32)
    x = rng.integers(-2, 3, size=(images, G, H, W)).astype(np.float32)
    ref = oc.tsvd_conv2d(x, U, S, V, 0, G, G, k, k, (st, st), (k // 2, k // 2), (1, 1), groups=G).transpose(1, 0, 2, 3).reshape(-1)
    xd = torch.full((x.size + 48,), float("inf"), dtype=torch.bfloat16, device="cuda:0")
    xd[16 + offset:16 + offset + x.size] = torch.from_numpy(np.ascontiguousarray(x.transpose(1, 0, 2, 3))).to("cuda:0").to(torch.bfloat16).flatten()
    y = torch.empty(ref.size, dtype=torch.float32, device="cuda:0")
    ws = torch.empty(256, dtype=torch.uint8, device="cuda:0")
    h = tsvd.tsvd_pack(U, S, V)
    geometry = (ctypes.c_int32 * 12)(0, G, G, k, k, st, st, k // 2, k // 2, 1, 1, G)
    p, i64 = ctypes.c_void_p, ctypes.c_int64
    print(f"case depthwise rows of {W} at element {offset}, {k} x {k}, stride {st}", flush=True)
    forward = ctypes.CDLL(tsvd.lib_path()).tsvd_conv2d_forward
    status = forward(p(h.ptr), geometry, p(xd[16 + offset:].data_ptr()), i64(images), i64(H), i64(W), p(None), p(y.data_ptr()), ctypes.c_int(tsvd.TSVD_F32),
                     p(ws.data_ptr()), ctypes.c_size_t(256), p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    tsvd.tsvd_free(h)
    assert status == 0
    assert np.array_equal(y.cpu().numpy(), ref)


@pytest.mark.parametrize("y_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("offset", [0, 1, 2, 3, 4])
def test_depthwise_result_at_any_element(tsvd, offset, y_dtype):  # noqa: F811
    """The C ABI takes any y aligned to its elements: rows of a multiple of four elements that start `offset` elements
    beyond a 16-byte boundary, exact, and nothing written beside them."""
    import ctypes

    import torch
    G, kg, k, images, H, W = 3, 2, 5, 2, 12, 16
    rng = np.random.default_rng(offset)
    U = np.kron(np.eye(G, dtype=np.int8), rng.choice([-1, 1], size=(1, kg)).astype(np.int8))
    V = rng.integers(-1, 2, size=(G * kg, k * k)).astype(np.int8)
    S = rng.integers(-2, 3, size=G * kg).astype(np.float32)
    x = rng.integers(-2, 3, size=(images, G, H, W)).astype(np.float32)
    ref = oc.tsvd_conv2d(x, U, S, V, 0, G, G, k, k, (1, 1), (2, 2), (1, 1), groups=G).transpose(1, 0, 2, 3).reshape(-1)
    dtype = torch.float32 if y_dtype == "f32" else torch.bfloat16
    xd = torch.from_numpy(np.ascontiguousarray(x.transpose(1, 0, 2, 3))).to("cuda:0").to(torch.bfloat16)
    buf = torch.full((ref.size + 16,), -77.0, dtype=dtype, device="cuda:0")
    ws = torch.empty(256, dtype=torch.uint8, device="cuda:0")
    h = tsvd.tsvd_pack(U, S, V)
    geometry = (ctypes.c_int32 * 12)(0, G, G, k, k, 1, 1, 2, 2, 1, 1, G)
    p, i64 = ctypes.c_void_p, ctypes.c_int64
    print(f"case depthwise y at element {offset} {y_dtype}", flush=True)
    forward = ctypes.CDLL(tsvd.lib_path()).tsvd_conv2d_forward
    st = forward(p(h.ptr), geometry, p(xd.data_ptr()), i64(images), i64(H), i64(W), p(None), p(buf[offset:].data_ptr()),
                 ctypes.c_int(tsvd.TSVD_F32 if y_dtype == "f32" else tsvd.TSVD_BF16), p(ws.data_ptr()), ctypes.c_size_t(256),
                 p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    got = buf.float().cpu().numpy()
    tsvd.tsvd_free(h)
    assert st == 0
    assert np.array_equal(got[offset:offset + ref.size], ref)
    assert (got[:offset] == -77.0).all() and (got[offset + ref.size:] == -77.0).all()


@pytest.mark.parametrize("k1,k2,st,pad,H,W", [(7, 7, 1, 3, 20, 40), (3, 5, 1, 1, 17, 19), (5, 5, 2, 2, 22, 36)])
def test_depthwise_values_that_are_not_finite_stay_with_their_taps(tsvd, k1, k2, st, pad, H, W):  # noqa: F811
    """Infinite and NaN pixels, and an infinite scale, reach the outputs whose own taps hold them and no others."""
    G, kg, images = 3, 3, 2
    rng = np.random.default_rng(k1 + 10 * k2 + st)
    U = np.zeros((G, G * kg), dtype=np.int8)
    for g in range(G):
        U[g, g * kg:(g + 1) * kg] = [1, -1, 0]
    V = rng.choice([-1, 0, 1], size=(G * kg, k1 * k2), p=[0.2, 0.6, 0.2]).astype(np.int8)
    S = (rng.standard_normal(G * kg) * 0.3).astype(np.float32)
    S[2 * kg] = np.inf                                            # the last channel
    S[2] = np.nan                                                 # of a rank that no output uses
    x = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(rng.standard_normal((images, G, H, W)).astype(np.float32)))
    x[0, 0, 3, 5], x[0, 0, 9, W - 1], x[1, 0, 0, 0], x[1, 1, H - 1, 17] = np.inf, np.nan, -np.inf, np.inf
    Ho, Wo = (H + 2 * pad - k1) // st + 1, (W + 2 * pad - k2) // st + 1
    ref = np.zeros((images, G, Ho, Wo))
    with np.errstate(invalid="ignore"):
        for i, g, oy, ox in np.ndindex(*ref.shape):
            for k in range(g * kg, g * kg + 2):
                z = 0.0
                for t in np.nonzero(V[k])[0]:
                    iy, ix = oy * st - pad + t // k2, ox * st - pad + t % k2
                    if 0 <= iy < H and 0 <= ix < W:
                        z += float(V[k, t]) * float(x[i, g, iy, ix])
                ref[i, g, oy, ox] += float(U[g, k]) * (float(S[k]) * z)
    print(f"case depthwise not finite {k1} {k2} {st}", flush=True)
    got = _run(tsvd, U, S, V, 0, G, G, k1, k2, workloads.f32_to_bf16_bits(x), ((st, st), (pad, pad), (1, 1)), None, tsvd.TSVD_F32, G)
    finite = np.isfinite(ref)
    assert finite[:, :2].mean() > 0.5 and not finite.all()
    assert np.array_equal(np.isfinite(got), finite)
    assert np.array_equal(got[~finite], ref[~finite], equal_nan=True)
    assert np.abs(got[finite] - ref[finite]).max() <= 1e-6 * np.abs(ref[finite]).max()
