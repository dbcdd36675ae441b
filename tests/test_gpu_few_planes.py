"""The few-token kernels on planes of z (tsvd_few.hip): exact on integer instances and within the bounds of include/tsvd.h on random ones, over
launch shapes, layouts, alignments and the ends of rows and of the array."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import rel_err, to_device
from test_gpu_planes import _check, tsvd  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu

SHAPES = [{}, {"TSVD_FEW_SW_V": 4, "TSVD_FEW_SW_U": 1, "TSVD_FEW_RW_U": 1}, {"TSVD_FEW_SW_U": 4, "TSVD_FEW_RW_U": 4}, {"TSVD_FEW_KWLOG2": 1}]


CALLS = [
    (70, 60, 40, 2),                # one column of tiles for either stage
    (300, 9, 40, 2),                # hardly more than one chunk of a row
    (300, 513, 270, 8), (515, 300, 777, 9),                 # eight tokens and one more
    (256, 255, 300, 9), (256, 257, 300, 5), (256, 263, 300, 18), (100, 511, 700, 31),      # ends of rows beside a chunk and a tile
    (40, 4500, 2100, 7), (2100, 9000, 520, 20),             # several columns for a wavefront
    (130, 64, 60, 33), (300, 1030, 1024, 47), (640, 200, 300, 96)]      # groups of tokens, the last one of one token and full


@pytest.mark.parametrize("planes,M,N,K,B", [(4, *c) for c in CALLS] + [(5, *c) for c in CALLS if c[3] <= 16])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_few_tokens_on_planes(tsvd, planes, M, N, K, B, shape):  # noqa: F811
    """(1e-6 for five planes: fp32 sums of a few hundred to a few thousand terms over 2^-24 of z; four planes: 2^-19, a 32nd of the 1e-4
    that three planes are allowed, and some.)"""
    print(f"case few on planes {M} {N} {K} {B} {shape} {planes}", flush=True)
    _check(tsvd, M, N, K, B, "bf16", {"TSVD_FEW": 128, "TSVD_FEW_PLANES": planes, **shape}, 1e-5 if planes == 4 else 1e-6)


@pytest.mark.parametrize("B,ld,col0", [(3, 10, 0), (5, 10, 2), (4, 9, 1), (9, 24, 8), (16, 40, 5), (19, 33, 7)])
def test_neighbours_that_are_not_finite(tsvd, B, ld, col0):  # noqa: F811
    """Columns of a wider matrix, NaN beside them; and rows of tokens that begin at odd elements, NaN between."""
    import torch
    i = workloads.make_integer_inputs(90, 700, 300, B, 0.5, "bf16", seed=77 + B + ld)
    ref = oracle.forward(i.U, i.S, i.V, i.X)
    h = tsvd.tsvd_pack(i.U, i.S, i.V)
    tsvd.tsvd_tuning_set("TSVD_FEW", 64)
    print(f"case few neighbours {B} {ld} {col0}", flush=True)
    wide = torch.full((700, ld), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    wide[:, col0:col0 + B] = to_device(i)
    assert np.array_equal(tsvd.tsvd_forward(h, wide[:, col0:col0 + B]).cpu().numpy(), ref)
    rows = torch.full((B, 700 + ld), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    rows[:, col0:col0 + 700] = to_device(i).t()
    y = tsvd.tsvd_forward_io(h, rows[:, col0:col0 + 700], x_layout=tsvd.TSVD_TOKEN_MAJOR, y_layout=tsvd.TSVD_TOKEN_MAJOR)
    assert np.array_equal(y.cpu().numpy().T, ref)
    tsvd.tsvd_free(h)


@pytest.mark.parametrize("M,N,K,B", [(1100, 700, 500, 1), (1100, 700, 500, 6), (4096, 4096, 5900, 7), (2500, 640, 1300, 40), (500, 2400, 130, 300)])
def test_calls_that_take_them_by_default(tsvd, M, N, K, B):  # noqa: F811
    """Five planes on small factors (error of fp32 sums), four beyond; the bits of the same kernels asked for by name (no other kernel has them), for
    either layout of x and y, and replayed from a captured graph; nothing behind the workspace that was asked for."""
    import torch
    i = workloads.make_inputs(M, N, K, B, 0.6, 0.02, "bf16", seed=M + B)
    ref = oracle.forward(i.U, i.S, i.V, i.X)
    h = tsvd.tsvd_pack(i.U, i.S, i.V)
    x = to_device(i)
    print(f"case few by default {M} {N} {K} {B}", flush=True)
    y = tsvd.tsvd_forward(h, x)
    assert rel_err(y.cpu().numpy().astype(np.float64), ref) <= (1e-6 if B <= 6 else 1e-5)
    yt = tsvd.tsvd_forward_io(h, x.t().contiguous(), x_layout=tsvd.TSVD_TOKEN_MAJOR, y_layout=tsvd.TSVD_TOKEN_MAJOR)
    assert torch.equal(yt.t(), y)
    for k, v in {"TSVD_FEW": 1024, "TSVD_FEW_PLANES": 5 if K <= 512 and B <= 16 else 4}.items():
        tsvd.tsvd_tuning_set(k, v)
    assert torch.equal(tsvd.tsvd_forward(h, x), y)
    tsvd.tsvd_tuning_set("TSVD_FEW", 0)
    assert not torch.equal(tsvd.tsvd_forward(h, x), y)
    tsvd.tsvd_tuning_reset()
    need = tsvd.tsvd_workspace_bytes(h, B, tsvd.TSVD_BF16)
    marked = torch.full((need + (1 << 16),), 93, dtype=torch.uint8, device="cuda:0")
    ws, out = marked[:need], torch.zeros_like(y)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tsvd.tsvd_forward(h, x, out, workspace=ws)
    for _ in range(3):
        out.zero_()
        ws.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, y) and (marked[need:] == 93).all()
    tsvd.tsvd_free(h)


@pytest.mark.parametrize("M,N,K,B,switch", [(256, 640, 500, 16, 64), (200, 700, 1300, 40, 64), (512, 4096, 7000, 16, None)])
def test_ranks_beside_those_of_massive_outliers(tsvd, M, N, K, B, switch):  # noqa: F811
    """Three features 2000 times the rest, seen by half of the ranks, these among the others; rows of y that use only the others.  z of four planes is off by
    2^-20 of the largest of 32 neighbours at most (here: of 128), and has to keep what 11 bits of each value would."""
    import torch
    rng = np.random.default_rng(M + K)
    U, V = (rng.choice([-1, 0, 1], size=s, p=[0.25, 0.5, 0.25]).astype(np.int8) for s in ((M, K), (K, N)))
    S = np.abs(rng.standard_normal(K)).astype(np.float32)
    massive, free, rows = [3, N // 3, N // 2 + 1], rng.permutation(K)[:K // 2], M // 2
    V[np.ix_(free, massive)] = 0
    U[:rows, np.setdiff1d(np.arange(K), free)] = 0
    x = rng.standard_normal((B, N))
    x[:, massive] *= 2000.0
    xd = torch.from_numpy(x).to("cuda:0").to(torch.bfloat16)
    x = xd.double().cpu().numpy()
    h = tsvd.tsvd_pack(U, S, V)
    if switch:
        tsvd.tsvd_tuning_set("TSVD_FEW", switch)
    print(f"case few beside outliers {M} {N} {K} {B}", flush=True)
    y = tsvd.tsvd_forward_io(h, xd, x_layout=tsvd.TSVD_TOKEN_MAJOR, y_layout=tsvd.TSVD_TOKEN_MAJOR).cpu().numpy().astype(np.float64)
    z = (x @ V.T.astype(np.float64)) * S
    want = z @ U.T.astype(np.float64)
    pad = np.pad(np.abs(z), ((0, 0), (0, -K % 128)))
    e2 = (2.0 ** -20 * np.repeat(pad.reshape(B, -1, 128).max(axis=2), 128, axis=1)[:, :K]) ** 2
    bound, size = np.sqrt(e2 @ (U != 0).T)[:, :rows], np.linalg.norm(want[:, :rows])
    err = np.linalg.norm((y - want)[:, :rows])
    assert err <= np.linalg.norm(bound) + 1e-6 * size
    assert err <= 2.0 ** -12 * size
    tsvd.tsvd_free(h)


@pytest.mark.parametrize("M,N,K,B,switch", [(1100, 700, 500, 1, None), (1100, 700, 500, 6, None), (900, 1030, 270, 16, None), (4096, 4096, 5900, 7, None), (2500, 640, 1300, 40, None),
                                            (70, 600, 300, 9, {"TSVD_FEW_SW_V": 4}), (300, 2100, 300, 16, {"TSVD_FEW_KWLOG2": 1})])
@pytest.mark.parametrize("size,scale", [(1e37, 1e-10), (2.0 ** 127, 2.0 ** -126), (1e-30, 1.0), (1e-36, 1.0)])
def test_activations_near_the_ends_of_fp32(tsvd, M, N, K, B, switch, size, scale):  # noqa: F811
    """Sums of doubled activations beyond fp32 where z and y are numbers again, and z whose last planes are below 2^-126: the bounds of ordinary sizes."""
    import torch
    rng = np.random.default_rng(M + N + K + B)
    U, V = (rng.choice([-1, 0, 1], size=s, p=[0.25, 0.5, 0.25]).astype(np.int8) for s in ((M, K), (K, N)))
    S = (rng.uniform(0.5, 1.0, K) * scale).astype(np.float32)
    x = torch.from_numpy(rng.uniform(-1, 1, (B, N)) * size).to(torch.bfloat16)
    want = ((x.double().numpy() @ V.T.astype(np.float64)) * S.astype(np.float64)) @ U.T.astype(np.float64)
    h = tsvd.tsvd_pack(U, S, V)
    for k, v in ({"TSVD_FEW": 64, **switch} if switch else {}).items():
        tsvd.tsvd_tuning_set(k, v)
    print(f"case few near the ends {M} {N} {K} {B} {size} {scale}", flush=True)
    y = tsvd.tsvd_forward_io(h, x.to("cuda:0"), x_layout=tsvd.TSVD_TOKEN_MAJOR, y_layout=tsvd.TSVD_TOKEN_MAJOR).double().cpu().numpy()
    y2 = tsvd.tsvd_forward(h, x.t().clone(memory_format=torch.contiguous_format).to("cuda:0")).t().double().cpu().numpy()
    for got in (y, y2):
        assert np.linalg.norm(got - want) <= (1e-6 if K <= 512 and not switch else 1e-5) * np.linalg.norm(want)
    tsvd.tsvd_free(h)


def test_z_beyond_fp32_is_no_number_in_y(tsvd):  # noqa: F811
    """z of one token beyond fp32: not a number (rather than an ordinary one) in the rows of that token, all others as they are."""
    import torch
    M, N, K, B = 300, 640, 300, 9
    rng = np.random.default_rng(5)
    U, V = (rng.choice([-1, 1], size=s).astype(np.int8) for s in ((M, K), (K, N)))
    h = tsvd.tsvd_pack(U, np.full(K, 3.0, np.float32), V)
    x = torch.from_numpy(rng.integers(-2, 3, (B, N)).astype(np.float32)).to(torch.bfloat16)
    big = x.clone()
    big[4] = torch.from_numpy(np.where(V[7] > 0, 1e38, -1e38)).to(torch.bfloat16)
    for switches in ({"TSVD_FEW": 16, "TSVD_FEW_PLANES": 4}, {"TSVD_FEW": 16, "TSVD_FEW_PLANES": 5}):
        for k, v in switches.items():
            tsvd.tsvd_tuning_set(k, v)
        print(f"case few z beyond fp32 {switches}", flush=True)
        y, plain = (tsvd.tsvd_forward_io(h, v.to("cuda:0"), x_layout=tsvd.TSVD_TOKEN_MAJOR, y_layout=tsvd.TSVD_TOKEN_MAJOR).cpu() for v in (big, x))
        others = [t for t in range(B) if t != 4]
        assert not torch.isfinite(y[4]).any() and torch.equal(y[others], plain[others])
        assert torch.equal(plain[others].double(), (x[others].double() @ torch.from_numpy(V).double().t() * 3.0) @ torch.from_numpy(U).double().t())
    tsvd.tsvd_free(h)


@pytest.mark.parametrize("M,N,K", [(1100, 700, 500), (900, 4099, 250), (3000, 2000, 300)])
def test_a_token_has_the_same_bits_among_others(tsvd, M, N, K):  # noqa: F811
    """1 to 16 tokens on small factors."""
    import torch
    i = workloads.make_inputs(M, N, K, 16, 0.6, 0.02, "bf16", seed=M + N)
    h = tsvd.tsvd_pack(i.U, i.S, i.V)
    x = to_device(i)
    print(f"case few tokens' bits {M} {N} {K}", flush=True)
    alone = torch.cat([tsvd.tsvd_forward(h, x[:, t:t + 1].clone()) for t in range(16)], dim=1)
    for B in (2, 8, 9, 16):
        for first in {0, 16 - B}:
            xb = x[:, first:first + B]
            assert torch.equal(tsvd.tsvd_forward(h, xb), alone[:, first:first + B])
            assert torch.equal(tsvd.tsvd_forward_io(h, xb.t().contiguous(), x_layout=tsvd.TSVD_TOKEN_MAJOR), alone[:, first:first + B])
    tsvd.tsvd_free(h)


@pytest.mark.parametrize("M,N,K", [(900, 4000, 256), (800, 14000, 200), (3000, 2000, 300)])
@pytest.mark.parametrize("kind", ["offset", "outliers", "opposite"])
def test_sums_that_cancel_on_five_planes(tsvd, M, N, K, kind):  # noqa: F811
    """Activations with a common offset, or a few far above the rest, and rows of V in which these cancel.  An fp32 sum is off by 2^-24 of its partial sums, at
    most of the sum of magnitudes, at each of its additions: one for each 8 values of a wavefront's columns and each wavefront.  The
    integers of the single-token kernels, on a grid of 2^-31 of the largest sum that could be, do not come closer."""
    import torch
    rng = np.random.default_rng(N + K)
    half = N // 4
    V = np.zeros((K, N), np.int8)
    for k in range(K):
        at = rng.permutation(N)
        V[k, at[:half]], V[k, at[half:2 * half]] = 1, -1
    x = rng.standard_normal(N)
    if kind == "offset":
        x += 100.0
    elif kind == "outliers":
        x[rng.permutation(N)[:N // 100]] *= 200.0
    else:
        x[[3, N - 2]] = 3000.0, -3000.0
        V[:, 3] = V[:, N - 2] = 1
    U = rng.choice([-1, 0, 1], size=(M, K), p=[0.25, 0.5, 0.25]).astype(np.int8)
    S = np.abs(rng.standard_normal(K)).astype(np.float32)
    xb = torch.from_numpy(x).to(torch.bfloat16)
    x = xb.double().numpy()
    z = (V.astype(np.float64) @ x) * S
    want = U.astype(np.float64) @ z
    nkt = -(-N // 256)
    kw = min(16, 1 << (nkt.bit_length() - 1))
    adds = 32 * -(-nkt // kw) + kw
    dz = adds * 2.0 ** -24 * S * (np.abs(V).astype(np.float64) @ np.abs(x)) + 2.0 ** -23 * np.abs(z).max()
    h = tsvd.tsvd_pack(U, S, V)
    print(f"case few sums that cancel {M} {N} {K} {kind}", flush=True)
    xd = xb.to("cuda:0")[:, None].contiguous()
    y = tsvd.tsvd_forward(h, xd).double().cpu().numpy()[:, 0]
    tsvd.tsvd_tuning_set("TSVD_FEW", 0)
    integers = tsvd.tsvd_forward(h, xd).double().cpu().numpy()[:, 0]
    assert not np.array_equal(y, integers)
    assert (np.abs(y - want) <= np.abs(U) @ dz + 2.0 ** -20 * (np.abs(U) @ np.abs(z))).all()
    print(f"{np.linalg.norm(y - want) / np.linalg.norm(want):.1e}, integers {np.linalg.norm(integers - want) / np.linalg.norm(want):.1e}", flush=True)
    assert np.linalg.norm(y - want) <= np.linalg.norm(integers - want)
    tsvd.tsvd_free(h)
