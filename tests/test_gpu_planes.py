"""The plane path's split tiles and the thin token panels at the edges of their tiles, against the oracle: exact on
integer instances (every layout, bias and output type), within a fraction of the tolerance on random ones."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import rel_err, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tsvd():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: the HIP path has no fallback")
    import paper_2308_07641_amd as t
    t.load_library()
    return t


def _check(tsvd, M, N, K, B, x_dtype, switches, bf16_tol=1e-4):
    import torch
    i = workloads.make_integer_inputs(M, N, K, B, 0.5, x_dtype, seed=M + N + K + B)
    ref = oracle.forward(i.U, i.S, i.V, i.X)
    h = tsvd.tsvd_pack(i.U, i.S, i.V)
    for k, v in switches.items():
        tsvd.tsvd_tuning_set(k, v)
    x = to_device(i)
    assert np.array_equal(tsvd.tsvd_forward(h, x).cpu().numpy(), ref)
    bias = np.arange(M, dtype=np.float32) % 7 - 3
    wide = torch.full((B, N + 3), float("nan"), dtype=x.dtype, device="cuda:0")       # rows of tokens, not 16-byte aligned, NaN beyond
    wide[:, :N] = x.t()
    y = tsvd.tsvd_forward_io(h, wide[:, :N], x_layout=tsvd.TSVD_TOKEN_MAJOR, y_layout=tsvd.TSVD_TOKEN_MAJOR, bias=torch.from_numpy(bias).to("cuda:0"))
    assert np.array_equal(y.cpu().numpy().T, ref + bias[:, None])
    y = tsvd.tsvd_forward_io(h, x.t().contiguous(), x_layout=tsvd.TSVD_TOKEN_MAJOR, y_layout=tsvd.TSVD_TOKEN_MAJOR, y_dtype=tsvd.TSVD_BF16)
    assert torch.equal(y.cpu(), torch.from_numpy(np.ascontiguousarray(ref.T)).to(torch.bfloat16))
    y = tsvd.tsvd_forward_ex(h, x[:, :B - 1], y_dtype=tsvd.TSVD_BF16)                 # a row pitch longer than the row
    assert torch.equal(y.cpu(), torch.from_numpy(ref[:, :B - 1].copy()).to(torch.bfloat16))
    tsvd.tsvd_free(h)
    j = workloads.make_inputs(M, N, K, B, 0.6, 0.02, x_dtype, seed=M + 2 * N + K + B)
    h = tsvd.tsvd_pack(j.U, j.S, j.V)
    e = rel_err(tsvd.tsvd_forward(h, to_device(j)).cpu().numpy().astype(np.float64), oracle.forward(j.U, j.S, j.V, j.X))
    assert e <= (1e-6 if x_dtype == "f32" else bf16_tol)
    tsvd.tsvd_free(h)


@pytest.mark.parametrize("x_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("own_x", [0, 1])
@pytest.mark.parametrize("v,u", [(9, 10), (10, 18), (18, 20), (20, 9), (0, 9), (20, 0)])
@pytest.mark.parametrize("M,N,K,B", [(130, 64, 60, 65), (515, 300, 777, 130), (256, 1300, 2500, 17)])
def test_split_tiles(tsvd, M, N, K, B, v, u, own_x, x_dtype):
    """One block and many, rows and tokens beside a tile's multiple, more steps than groups of wavefronts; planes of x made by
    stage V or by their own pass."""
    print(f"case split {M} {N} {K} {B} {v} {u} {own_x} {x_dtype}", flush=True)
    _check(tsvd, M, N, K, B, x_dtype, {"TSVD_MID": 0, "TSVD_PANEL": 0, "TSVD_SPLIT_V": v, "TSVD_SPLIT_U": u, "TSVD_SPLIT_X": own_x})


@pytest.mark.parametrize("tiles", [1, 2])
@pytest.mark.parametrize("M,N,K,B", [(130, 64, 60, 65), (515, 300, 777, 130), (300, 1030, 1024, 47), (200, 2600, 900, 40), (200, 3200, 2048, 19), (64, 100, 2049, 33)])
def test_thin_panels(tsvd, M, N, K, B, tiles):
    """x in LDS as a whole and in chunks, one and two rank blocks per wavefront, and sizes that no such panel holds (these take the other
    kernels)."""
    print(f"case thin {M} {N} {K} {B} {tiles}", flush=True)
    _check(tsvd, M, N, K, B, "bf16", {"TSVD_MID": 0, "TSVD_PANEL": 0, "TSVD_THIN": tiles, "TSVD_SPLIT_V": 9, "TSVD_SPLIT_U": 9})


@pytest.mark.parametrize("tiles", [1, 2])
@pytest.mark.parametrize("form,ci,co,k1,k2,geom", [
    (0, 5, 7, 3, 3, ((1, 1), (1, 1), (1, 1))), (0, 150, 40, 5, 5, ((2, 1), (2, 2), (1, 1))), (2, 20, 33, 3, 2, ((1, 2), (1, 0), (2, 1))),
    (3, 64, 9, 7, 1, ((2, 2), (3, 0), (1, 1))), (0, 3, 5, 7, 7, ((1, 1), (3, 3), (1, 1)))])
def test_thin_panels_gather_convolutions(tsvd, form, ci, co, k1, k2, geom, tiles):
    """Taps outside the image, strides and dilations, x in chunks, and more taps than the bit mask holds (the columns are written
    then)."""
    import torch
    from oracle import conv as oc
    K, images, H, W = 150, 3, 12, 9
    rows, cols = {0: (co, ci * k1 * k2), 2: (co * k1, ci * k2), 3: (co * k2, ci * k1)}[form]
    rng = np.random.default_rng(form + ci + k1)
    print(f"case thin conv {form} {ci} {co} {k1}x{k2} {tiles}", flush=True)
    U = rng.choice([-1, 0, 1], size=(rows, K), p=[0.15, 0.7, 0.15]).astype(np.int8)
    V = rng.choice([-1, 0, 1], size=(K, cols), p=[0.15, 0.7, 0.15]).astype(np.int8)
    S = rng.integers(-2, 3, size=K).astype(np.float32)
    x = rng.integers(-2, 3, size=(images, ci, H, W)).astype(np.float32)
    bias = rng.integers(-4, 5, size=co).astype(np.float32)
    ref = oc.tsvd_conv2d(x, U, S, V, form, co, ci, k1, k2, *geom, bias=bias)
    h = tsvd.tsvd_pack(U, S, V)
    tsvd.tsvd_tuning_set("TSVD_THIN", tiles)
    xd = torch.from_numpy(np.ascontiguousarray(x.transpose(1, 0, 2, 3))).to("cuda:0").to(torch.bfloat16)
    for y_dtype in (tsvd.TSVD_F32, tsvd.TSVD_BF16):
        y = tsvd.tsvd_conv2d_forward(h, form, ci, co, k1, k2, xd, *geom, bias=torch.from_numpy(bias).to("cuda:0"), y_dtype=y_dtype)
        want = torch.from_numpy(np.ascontiguousarray(ref.transpose(1, 0, 2, 3))).to(y.dtype)
        assert torch.equal(y.cpu(), want)
    tsvd.tsvd_free(h)


PLANE_PATHS = [{"TSVD_THIN": 1}, {"TSVD_THIN": 2}, {"TSVD_SPLIT_V": 9, "TSVD_SPLIT_U": 10}, {"TSVD_SPLIT_V": 18, "TSVD_SPLIT_U": 20, "TSVD_SPLIT_X": 1}]


def _on_planes(tsvd, h, x, switches):
    for k, v in {"TSVD_MID": 0, "TSVD_PANEL": 0, **switches}.items():
        tsvd.tsvd_tuning_set(k, v)
    return tsvd.tsvd_forward_io(h, x, x_layout=tsvd.TSVD_TOKEN_MAJOR, y_layout=tsvd.TSVD_TOKEN_MAJOR).cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("switches", PLANE_PATHS, ids=str)
def test_values_within_two_to_the_seven_of_their_neighbours_are_exact(tsvd, switches):
    """What tsvd.h states for bf16 activations on planes: each value that is at least 2^-7 of the largest of its 32 neighbours enters
    exactly.  V and U pick one entry per row, so y is x itself, permuted."""
    import torch
    rng = np.random.default_rng(7)
    N, B = 333, 70
    pick, place, sign = rng.permutation(N), rng.permutation(N), rng.choice([-1, 1], N)
    V, U = np.zeros((N, N), np.int8), np.zeros((N, N), np.int8)
    V[np.arange(N), pick] = sign
    U[place, np.arange(N)] = 1
    x = rng.choice([-1, 1], (B, N)) * np.ldexp(rng.integers(128, 256, (B, N)) / 128.0, rng.integers(-6, 1, (B, N)))      # 2^-6 .. 2 - 2^-7
    h = tsvd.tsvd_pack(U, np.ones(N, np.float32), V)
    print(f"case exact values {switches}", flush=True)
    y = _on_planes(tsvd, h, torch.from_numpy(x).to("cuda:0").to(torch.bfloat16), switches)
    want = np.empty_like(x)
    want[:, place] = x[:, pick] * sign
    assert np.array_equal(y, want)
    tsvd.tsvd_free(h)


@pytest.mark.parametrize("outlier", [200.0, 2000.0])
@pytest.mark.parametrize("switches", PLANE_PATHS, ids=str)
def test_rows_free_of_massive_outliers(tsvd, switches, outlier):
    """Three features far above the rest, seen by a third of the ranks; rows of y that use none of those keep the precision that
    tsvd.h states.  An x smaller than 2^-7 of the largest m of its neighbours is off by 2^-15 m at most, so y = U (S (V x)) by a sum of such
    errors with the signs of V and U (bounded here by its root mean square over those, neighbours taken as 64); z of such ranks shares its
    neighbours with others of them only: 2^-14 of a block's largest value, which is four times its rms at most, 2.5e-4 of y."""
    import torch
    rng = np.random.default_rng(int(outlier))
    M, N, K, B, free_ranks, free_rows = 256, 640, 384, 70, 256, 128
    U, V = (rng.choice([-1, 0, 1], size=s, p=[0.25, 0.5, 0.25]).astype(np.int8) for s in ((M, K), (K, N)))
    S = np.abs(rng.standard_normal(K)).astype(np.float32)
    massive = [3, 200, 333]
    V[:free_ranks, massive] = 0
    U[:free_rows, free_ranks:] = 0
    x = rng.standard_normal((B, N))
    x[:, massive] *= outlier
    xd = torch.from_numpy(x).to("cuda:0").to(torch.bfloat16)
    x = xd.double().cpu().numpy()
    h = tsvd.tsvd_pack(U, S, V)
    print(f"case massive outliers {outlier} {switches}", flush=True)
    y = _on_planes(tsvd, h, xd, switches)
    z = (x @ V.T.astype(np.float64)) * S
    want = z @ U.T.astype(np.float64)
    e2 = (2.0 ** -15 * np.repeat(np.abs(x).reshape(B, N // 64, 64).max(axis=2), 64, axis=1)) ** 2
    bound = np.sqrt(((e2 @ (V != 0).T) * S ** 2) @ (U != 0).T)[:, :free_rows]
    err = (y - want)[:, :free_rows]
    assert np.linalg.norm(err) <= np.linalg.norm(bound) + 2.5e-4 * np.linalg.norm(want[:, :free_rows])
    assert rel_err(y, want) <= 1e-4                                                # the whole of y
    tsvd.tsvd_free(h)


TWO_SETS = [{"TSVD_PANEL": 0, "TSVD_FP6": 1, "TSVD_FP6_V": 2, "TSVD_GEMM_CFG_V": 3, "TSVD_FP6_TALL": tall} for tall in (0, 1)]


@pytest.mark.parametrize("switches", TWO_SETS, ids=str)
@pytest.mark.parametrize("M,N,K,B", [(130, 64, 60, 65), (515, 300, 777, 130), (300, 129, 512, 47), (200, 1280, 1025, 129)])
def test_stage_v_on_two_sets_of_planes(tsvd, M, N, K, B, switches):
    """An odd and an even number of blocks, one and several, tokens beside a tile's multiple."""
    print(f"case two sets {M} {N} {K} {B} {switches}", flush=True)
    _check(tsvd, M, N, K, B, "bf16", switches)


@pytest.mark.parametrize("outlier", [200.0, 2000.0, 30000.0])
@pytest.mark.parametrize("M,N,K,B,switches", [(256, 640, 768, 130, TWO_SETS[0]), (256, 640, 768, 130, TWO_SETS[1]), (2048, 512, 2304, 8192, {})], ids=str)
def test_large_batches_with_massive_outliers(tsvd, M, N, K, B, switches, outlier):
    """Rows of y that use only ranks which avoid three features far above the rest, in blocks of their own: what is off there is z on
    three planes, 2^-14 of a block's largest value, four times its rms at most; x counts as it is.  (The last call takes these kernels by itself.)"""
    import torch
    g = torch.Generator(device="cuda:0")
    g.manual_seed(int(outlier) + K)
    U, V = (torch.randint(0, 4, s, generator=g, device="cuda:0").sub_(1).clamp_(max=1).double() for s in ((M, K), (K, N)))
    U, V = U * torch.randint(0, 2, U.shape, generator=g, device="cuda:0"), V * torch.randint(0, 2, V.shape, generator=g, device="cuda:0")
    S = torch.randn(K, generator=g, device="cuda:0", dtype=torch.float64).abs().float()
    massive, free_ranks, free_rows = [3, 200, 333], K // 2, M // 2
    V[:free_ranks, massive] = 0
    U[:free_rows, free_ranks:] = 0
    x = torch.randn((B, N), generator=g, device="cuda:0")
    x[:, massive] *= outlier
    x = x.to(torch.bfloat16)
    h = tsvd.tsvd_pack(U.to(torch.int8).cpu().numpy(), S.cpu().numpy(), V.to(torch.int8).cpu().numpy())
    for k, v in switches.items():
        tsvd.tsvd_tuning_set(k, v)
    print(f"case large batch, massive outliers {outlier} {switches}", flush=True)
    want = ((x.double() @ V.t().contiguous()) * S.double()) @ U.t().contiguous()
    y = tsvd.tsvd_forward_io(h, x, x_layout=tsvd.TSVD_TOKEN_MAJOR, y_layout=tsvd.TSVD_TOKEN_MAJOR).double()
    assert (y - want)[:, :free_rows].norm() <= 2.5e-4 * want[:, :free_rows].norm()
    y2 = tsvd.tsvd_forward(h, x.t().contiguous()).double().t()
    assert (y2 - want)[:, :free_rows].norm() <= 2.5e-4 * want[:, :free_rows].norm()
    assert (y - want).norm() <= 2.5e-4 * want.norm()
    tsvd.tsvd_free(h)


@pytest.mark.parametrize("M,N,K,B", [(1, 40, 70, 20), (31, 300, 130, 33), (33, 129, 260, 17), (129, 300, 900, 40), (2050, 200, 130, 50), (4100, 130, 1020, 18), (9000, 257, 100, 65),
                                     (520, 140, 257, 2040), (300, 260, 90, 2049)])
@pytest.mark.parametrize("tiles", [1, 2])
def test_thin_panels_of_several_workgroups(tsvd, M, N, K, B, tiles):
    """Few panels: the rows of y dealt among several workgroups of a panel, down to units of 32 rows, the last ones without any; and the numbers of
    panels where two workgroups a panel begin.  (The bits of one workgroup a panel: the bound is that of test_thin_panels.)"""
    print(f"case thin of several workgroups {M} {N} {K} {B} {tiles}", flush=True)
    _check(tsvd, M, N, K, B, "bf16", {"TSVD_THIN": tiles})


@pytest.mark.parametrize("M,N,K,B,tiles,shares", [
    (70, 700, 128, 33, 1, 12), (40, 900, 100, 17, 1, 14), (50, 2000, 60, 35, 1, 18), (30, 4300, 100, 50, 1, 114), (30, 5600, 128, 40, 1, 118), (70, 700, 129, 40, 1, 22),
    (40, 900, 256, 17, 1, 24), (30, 4200, 250, 40, 1, 124), (40, 1030, 640, 31, 1, 14), (30, 3800, 600, 33, 1, 114), (70, 1600, 700, 33, 1, 22), (30, 3700, 760, 20, 1, 122),
    (60, 1030, 1100, 20, 1, 14), (60, 2000, 1025, 20, 1, 18), (30, 3300, 1100, 18, 1, 114), (60, 900, 1250, 35, 1, 24), (60, 3200, 1280, 18, 1, 124), (30, 2100, 1664, 35, 1, 14),
    (30, 2800, 1600, 33, 1, 114), (30, 1600, 1700, 33, 1, 22), (30, 3000, 1790, 33, 1, 122), (60, 3000, 1280, 18, 1, 0),
    (40, 600, 128, 33, 2, 12), (40, 1000, 100, 50, 2, 14), (50, 1900, 60, 35, 2, 18), (30, 2100, 100, 40, 2, 112), (70, 520, 256, 40, 2, 22), (40, 900, 250, 65, 2, 24),
    (30, 2000, 200, 33, 2, 122), (40, 760, 600, 31, 2, 12), (40, 900, 640, 33, 2, 14), (30, 1600, 620, 33, 2, 112), (70, 800, 700, 33, 2, 22), (30, 1500, 760, 40, 2, 122)])
def test_thin_panels_share_rank_blocks(tsvd, M, N, K, B, tiles, shares):
    """One, two, five and six rank blocks that do not go round, alone or behind eight that do: two to eight wavefronts share a block's contraction, some with nothing of
    it where there is little or in the last chunk; x as a whole and in chunks (`shares`: 10 x blocks + wavefronts of each, + 100 in chunks; these are the kernels that
    run).  (The bound is that of test_thin_panels: sums of fp32 in another order.)"""
    print(f"case thin shares {M} {N} {K} {B} {tiles}", flush=True)
    tsvd.tsvd_tuning_thin_last()
    _check(tsvd, M, N, K, B, "bf16", {"TSVD_MID": 0, "TSVD_PANEL": 0, "TSVD_THIN": tiles, "TSVD_SPLIT_V": 9, "TSVD_SPLIT_U": 9})
    assert tsvd.tsvd_tuning_thin_last() == 1000 * tiles + shares


@pytest.mark.parametrize("M,N,K,B,v,u", [
    (300, 260, 200, 17, 9, 9), (700, 600, 500, 700, 9, 10), (1500, 300, 200, 700, 9, 0), (200, 2000, 1500, 511, 10, 9), (2000, 1200, 700, 700, 10, 18), (2000, 1200, 700, 1000, 10, 0),
    (130, 500, 1800, 700, 18, 9), (3000, 1500, 1500, 700, 18, 0), (3000, 1500, 1500, 1000, 18, 20), (600, 300, 3000, 700, 20, 9), (600, 300, 3000, 1000, 20, 10),
    (700, 600, 500, 1024, 9, 10), (700, 600, 500, 1025, 10, 10), (130, 500, 1800, 1024, 18, 9), (130, 500, 1800, 1025, 20, 9)])
def test_fp32_calls_choose_their_tiles(tsvd, M, N, K, B, v, u):
    """Calls of fp32 activations without switches: each tile of either stage as the estimates choose it (on 256 compute units), and both sides of the 1024 tokens where
    the other factors begin."""
    print(f"case fp32 choice {M} {N} {K} {B}", flush=True)
    h = tsvd.tsvd_pack(np.zeros((M, K), np.int8), np.ones(K, np.float32), np.zeros((K, N), np.int8))
    assert tsvd.tsvd_tuning_split_tiles(h, B, tsvd.TSVD_F32) == (v, u)
    tsvd.tsvd_free(h)
    _check(tsvd, M, N, K, B, "f32", {})


@pytest.mark.parametrize("x_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("own_x", [0, 1])
@pytest.mark.parametrize("v,u", [(9, 9), (10, 10)])
@pytest.mark.parametrize("M,N,K,B", [(20, 30, 20, 17), (128, 1024, 1024, 32), (129, 1025, 1025, 33), (300, 2050, 3100, 47), (100, 4100, 140, 16 + 17)])
def test_blocks_of_a_wavefront(tsvd, M, N, K, B, v, u, own_x, x_dtype):
    """Tiles of 128 rows, each wavefront with blocks of its own: fewer blocks than wavefronts, one for each, one more; more than are in flight; planes of x
    made in registers or by their own pass."""
    print(f"case blocks of a wavefront {M} {N} {K} {B} {v} {u} {own_x} {x_dtype}", flush=True)
    _check(tsvd, M, N, K, B, x_dtype, {"TSVD_MID": 0, "TSVD_PANEL": 0, "TSVD_SPLIT_V": v, "TSVD_SPLIT_U": u, "TSVD_SPLIT_X": own_x})


@pytest.mark.parametrize("x_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("own_x", [0, 1])
@pytest.mark.parametrize("v,u", [(18, 18), (20, 20)])
@pytest.mark.parametrize("M,N,K,B", [(20, 30, 20, 17), (257, 500, 510, 64), (300, 1025, 1150, 65), (512, 1030, 2050, 31), (130, 3330, 3900, 97), (90, 640, 900, 1025)])
def test_blocks_of_a_pair(tsvd, M, N, K, B, v, u, own_x, x_dtype):
    """Tiles of 256 rows, each pair of wavefronts with blocks of its own: pairs without any, with one, an odd and an even number of steps, a last step
    that is not full; planes of x made by all wavefronts first or by their own pass."""
    print(f"case blocks of a pair {M} {N} {K} {B} {v} {u} {own_x} {x_dtype}", flush=True)
    _check(tsvd, M, N, K, B, x_dtype, {"TSVD_MID": 0, "TSVD_PANEL": 0, "TSVD_SPLIT_V": v, "TSVD_SPLIT_U": u, "TSVD_SPLIT_X": own_x})


@pytest.mark.parametrize("x_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("M,N,K,B,v,u,placed", [
    (700, 5000, 2600, 300, 9, 9, (False, True)), (700, 5000, 1300, 150, 9, 9, (True, False)), (1900, 4500, 2100, 130, 10, 10, (True, True)), (2600, 4300, 2300, 200, 18, 18, (True, True)),
    (2050, 8300, 1100, 513, 20, 20, (True, True)), (4100, 8300, 2100, 72, 18, 9, (True, True))])
def test_tiles_by_xcd(tsvd, M, N, K, B, v, u, placed, x_dtype):
    """Launches of one round whose tiles are dealt to the XCDs in groups that do not divide evenly: every tile is computed, those beyond the matrix write
    nothing (the call's own workspace ends where the planes of z do)."""
    import torch
    print(f"case tiles by XCD {M} {N} {K} {B} {v} {u} {x_dtype}", flush=True)
    _check(tsvd, M, N, K, B, x_dtype, {"TSVD_MID": 0, "TSVD_PANEL": 0, "TSVD_SPLIT_V": v, "TSVD_SPLIT_U": u, "TSVD_SPLIT_X": 0})
    i = workloads.make_integer_inputs(M, N, K, B, 0.5, x_dtype, seed=M + B)
    h = tsvd.tsvd_pack(i.U, i.S, i.V)
    for name, value in {"TSVD_MID": 0, "TSVD_PANEL": 0, "TSVD_SPLIT_V": v, "TSVD_SPLIT_U": u, "TSVD_SPLIT_X": 0}.items():
        tsvd.tsvd_tuning_set(name, value)
    dtype = tsvd.TSVD_BF16 if x_dtype == "bf16" else tsvd.TSVD_F32
    assert tsvd.tsvd_tuning_tiles_by_xcd(h, B, dtype) == placed
    need = tsvd.tsvd_workspace_bytes(h, B, dtype)
    guarded = torch.full((need + (1 << 20),), 0x5A, dtype=torch.uint8, device="cuda:0")
    y = tsvd.tsvd_forward(h, to_device(i), workspace=guarded[:need])
    assert np.array_equal(y.cpu().numpy(), oracle.forward(i.U, i.S, i.V, i.X))
    assert bool((guarded[need:] == 0x5A).all())
    tsvd.tsvd_free(h)


def _gather_rows_of_three(tsvd, form, ci, co, k1, K, H, W, geom, tiles, shares=None):
    import torch
    from oracle import conv as oc
    k2, images = 3, 5
    rows, cols = {0: (co, ci * k1 * k2), 2: (co * k1, ci * k2)}[form]
    rng = np.random.default_rng(form + ci + k1 + K + W)
    print(f"case thin rows of three {form} {ci} {co} {k1} {K} {H} {W} {geom} {tiles}", flush=True)
    U = rng.choice([-1, 0, 1], size=(rows, K), p=[0.05, 0.9, 0.05]).astype(np.int8)
    V = rng.choice([-1, 0, 1], size=(K, cols), p=[0.05, 0.9, 0.05]).astype(np.int8)
    S = rng.integers(-1, 2, size=K).astype(np.float32)
    x = rng.integers(-1, 2, size=(images, ci, H, W)).astype(np.float32)
    ref = oc.tsvd_conv2d(x, U, S, V, form, co, ci, k1, k2, *geom)
    h = tsvd.tsvd_pack(U, S, V)
    tsvd.tsvd_tuning_set("TSVD_THIN", tiles)
    xd = torch.full((x.size + 9,), float("nan"), dtype=torch.bfloat16, device="cuda:0")        # (nothing from beside x may reach y)
    xd = xd[1:1 + x.size].view(ci, images, H, W).copy_(torch.from_numpy(x.transpose(1, 0, 2, 3)))
    tsvd.tsvd_tuning_thin_last()
    y = tsvd.tsvd_conv2d_forward(h, form, ci, co, k1, k2, xd, *geom)
    assert shares is None or tsvd.tsvd_tuning_thin_last() == 1000 * tiles + shares
    assert torch.equal(y.cpu(), torch.from_numpy(np.ascontiguousarray(ref.transpose(1, 0, 2, 3))).to(y.dtype))
    tsvd.tsvd_free(h)


@pytest.mark.parametrize("tiles", [1, 2])
@pytest.mark.parametrize("form,ci,co,k1,K,H,W,geom", [
    (0, 5, 7, 3, 60, 6, 4, ((1, 1), (1, 1), (1, 1))), (0, 5, 7, 3, 60, 6, 3, ((1, 1), (1, 1), (1, 1))), (0, 43, 9, 3, 150, 5, 9, ((2, 3), (4, 5), (2, 1))),
    (0, 20, 9, 5, 150, 7, 11, ((1, 2), (0, 3), (1, 1))), (2, 90, 3, 2, 300, 6, 5, ((1, 1), (1, 2), (1, 1))), (0, 20, 9, 3, 150, 7, 11, ((1, 1), (2, 2), (1, 2))),
    (0, 300, 5, 3, 150, 5, 7, ((1, 1), (1, 1), (1, 1))), (0, 460, 5, 3, 777, 5, 5, ((1, 1), (1, 1), (1, 1))), (0, 460, 5, 3, 1100, 5, 5, ((1, 1), (0, 1), (1, 1)))])
def test_thin_panels_gather_rows_of_three(tsvd, form, ci, co, k1, K, H, W, geom, tiles):
    """Rows of three taps in loads of four elements: images as wide as a load and narrower (which take element loads, as dilated rows do), taps that
    begin more than a load before or behind a row, kernels of more and fewer rows, x at an odd element; and x in chunks that wavefronts of
    fewer rank blocks make more records of.  Exact."""
    _gather_rows_of_three(tsvd, form, ci, co, k1, K, H, W, geom, tiles)


@pytest.mark.parametrize("ci,co,K,H,W,tiles,shares", [
    (430, 5, 100, 5, 7, 1, 114), (120, 9, 640, 6, 5, 1, 14), (380, 5, 600, 5, 7, 1, 114), (180, 9, 700, 7, 5, 1, 22), (380, 5, 768, 5, 7, 1, 122), (150, 9, 1100, 5, 9, 1, 14),
    (340, 5, 1030, 5, 7, 1, 114), (150, 9, 1250, 6, 6, 1, 24), (360, 5, 1280, 5, 7, 1, 124), (290, 5, 1600, 5, 5, 1, 114), (270, 5, 1700, 5, 7, 1, 122),
    (240, 9, 128, 5, 7, 2, 112), (110, 9, 200, 6, 9, 2, 24), (200, 9, 600, 5, 7, 2, 112), (256, 5, 768, 7, 7, 2, 122), (256, 33, 700, 5, 8, 2, 122), (320, 5, 256, 5, 7, 2, 0)])
def test_thin_panels_gather_rows_of_three_and_share_rank_blocks(tsvd, ci, co, K, H, W, tiles, shares):
    """The same where rank blocks are shared (as test_thin_panels_share_rank_blocks has it), and where two are not because of the rows."""
    _gather_rows_of_three(tsvd, 0, ci, co, 3, K, H, W, ((1, 1), (1, 1), (1, 1)), tiles, shares)


@pytest.mark.parametrize("switches", [{"TSVD_THIN": 1}, {"TSVD_THIN": 2}, {"TSVD_SPLIT_V": 9, "TSVD_SPLIT_U": 10}, {"TSVD_SPLIT_V": 10, "TSVD_SPLIT_U": 10, "TSVD_SPLIT_X": 1},
                                      {"TSVD_SPLIT_V": 9, "TSVD_SPLIT_U": 9, "TSVD_SPLIT_X": 1}, {"TSVD_SPLIT_V": 20, "TSVD_SPLIT_U": 18, "TSVD_SPLIT_X": 1}], ids=str)
@pytest.mark.parametrize("N,B,pad", [(1153, 17, 0), (1157, 23, 3), (1279, 33, 0), (1280, 40, 1), (129, 50, 0), (8, 17, 0), (1, 19, 5), (4097, 30, 2)])
def test_columns_of_feature_major_x(tsvd, N, B, pad, switches):
    """Feature-major bf16 x read in chunks of eight tokens: rows at odd elements, a last chunk that ends with x, features one beyond a block, the last rows of
    a block, one row.  What stands beside the tokens, and behind x where the rows of a whole block would be, is no number and reaches no result.  Exact."""
    import torch
    M, K = 70, 150
    print(f"case columns {N} {B} {pad} {switches}", flush=True)
    rng = np.random.default_rng(N + B)
    U = rng.choice([-1, 0, 1], size=(M, K), p=[0.1, 0.8, 0.1]).astype(np.int8)
    V = rng.choice([-1, 0, 1], size=(K, N), p=[0.05, 0.9, 0.05]).astype(np.int8)
    S = rng.integers(-1, 2, size=K).astype(np.float32)
    X = rng.integers(-1, 2, size=(N, B)).astype(np.float32)
    h = tsvd.tsvd_pack(U, S, V)
    for k, v in {"TSVD_MID": 0, "TSVD_PANEL": 0, **switches}.items():
        tsvd.tsvd_tuning_set(k, v)
    x = torch.full(((N + 256) * (B + pad) + B + 1,), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    view = torch.as_strided(x, (N, B), (B + pad, 1), 1).copy_(torch.from_numpy(X))
    y = tsvd.tsvd_forward(h, view)
    assert np.array_equal(y.cpu().numpy(), oracle.forward(U, S, V, X).astype(np.float32))
    tsvd.tsvd_free(h)


@pytest.mark.parametrize("v,u,own_x", [(9, 9, 1), (10, 10, 1), (10, 18, 0), (20, 20, 1)])
@pytest.mark.parametrize("N,B,ld", [(1, 2, 2), (1, 7, 7), (2, 3, 4), (3, 2, 2), (1, 3, 4000), (1, 8, 8), (2, 4, 4), (4, 2, 2)])
def test_split_tiles_of_fewer_values_than_a_chunk(tsvd, N, B, ld, v, u, own_x):
    """Feature-major bf16 x of fewer than the eight values that the split tiles read at a time, and of eight.  Exact."""
    import torch
    M, K = 40, 70
    print(f"case fewer than a chunk {N} {B} {ld} {v} {u} {own_x}", flush=True)
    i = workloads.make_integer_inputs(M, N, K, B, 0.3, "bf16", seed=N + B)
    h = tsvd.tsvd_pack(i.U, i.S, i.V)
    for name, value in {"TSVD_GEMM_MIN_B": 2, "TSVD_MID": 0, "TSVD_PANEL": 0, "TSVD_SPLIT_V": v, "TSVD_SPLIT_U": u, "TSVD_SPLIT_X": own_x, "TSVD_REALIGN": 0}.items():
        tsvd.tsvd_tuning_set(name, value)
    held = torch.full(((N - 1) * ld + B + 64,), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    x = torch.as_strided(held, (N, B), (ld, 1)).copy_(to_device(i))
    assert np.array_equal(tsvd.tsvd_forward(h, x).cpu().numpy(), oracle.forward(i.U, i.S, i.V, i.X))
    tsvd.tsvd_free(h)
