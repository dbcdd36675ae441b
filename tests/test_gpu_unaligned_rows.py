"""Rows of tokens, and of features, at any element: activations are read and results written 16 bytes at a time at addresses that are no multiple of it.  Integer instances
are exact; beside x lies NaN and beside y a mark that has to stay."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import to_device
from test_gpu_planes import tsvd  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu

# fp16 z, token panels of 64, thin panels of 16 and of 32, split tiles on their own x and on planes of it, plane path on large tiles
ROUTES = [{"TSVD_FP6": 0, "TSVD_PANEL": 0}, {"TSVD_PANEL": 1}, {"TSVD_THIN": 1}, {"TSVD_THIN": 2}, {"TSVD_PANEL": 0, "TSVD_SPLIT_V": 10, "TSVD_SPLIT_U": 10, "TSVD_SPLIT_X": 1},
          {"TSVD_PANEL": 0, "TSVD_SPLIT_V": 10, "TSVD_SPLIT_U": 10, "TSVD_SPLIT_X": 0}, {"TSVD_PANEL": 0, "TSVD_FP6": 1},
          {"TSVD_PANEL": 0, "TSVD_FP6": 1, "TSVD_FP6_V": 1, "TSVD_GEMM_CFG_V": 3, "TSVD_FP6_TALL": 0}]      # (the last: planes of z from stage V)


@pytest.mark.parametrize("M,N,K,B", [(64, 5, 40, 17), (66, 8, 70, 40), (131, 127, 60, 33), (129, 129, 130, 65), (257, 251, 200, 130), (67, 263, 300, 49)])
@pytest.mark.parametrize("route", ROUTES, ids=str)
@pytest.mark.parametrize("x_dtype,y_dtype", [("bf16", "bf16"), ("bf16", "f32"), ("f32", "bf16"), ("f32", "f32")])
def test_rows_at_any_element(tsvd, M, N, K, B, route, x_dtype, y_dtype):  # noqa: F811
    import torch
    i = workloads.make_integer_inputs(M, N, K, B, 0.5, x_dtype, seed=M + N + K + B)
    ref = torch.from_numpy(np.ascontiguousarray(oracle.forward(i.U, i.S, i.V, i.X).T))
    h = tsvd.tsvd_pack(i.U, i.S, i.V)
    for k, v in route.items():
        tsvd.tsvd_tuning_set(k, v)
    x, out = to_device(i), torch.bfloat16 if y_dtype == "bf16" else torch.float32
    for before, after in ((0, 0), (1, 0), (3, 2), (8, 8)):
        print(f"case rows at any element {M} {N} {K} {B} {route} {x_dtype} {y_dtype} {before} {after}", flush=True)
        wide = torch.full((B, before + N + after), float("nan"), dtype=x.dtype, device="cuda:0")
        wide[:, before:before + N] = x.t()
        y = torch.full((B, before + M + after), -77.0, dtype=out, device="cuda:0")
        tsvd.tsvd_forward_io(h, wide[:, before:before + N], x_layout=tsvd.TSVD_TOKEN_MAJOR, y=y[:, before:before + M], y_dtype=tsvd.TSVD_BF16 if y_dtype == "bf16" else tsvd.TSVD_F32,
                             y_layout=tsvd.TSVD_TOKEN_MAJOR)
        got = y.cpu()
        assert torch.equal(got[:, before:before + M], ref.to(out))
        assert (got[:, :before] == -77).all() and (got[:, before + M:] == -77).all()
        xf = torch.full((N, before + B + after), float("nan"), dtype=x.dtype, device="cuda:0")
        xf[:, before:before + B] = x
        f = torch.full((M, before + B + after), -77.0, dtype=out, device="cuda:0")      # feature-major y: pairs of tokens per store
        tsvd.tsvd_forward_ex(h, xf[:, before:before + B], y=f[:, before:before + B], y_dtype=tsvd.TSVD_BF16 if y_dtype == "bf16" else tsvd.TSVD_F32)
        got = f.cpu()
        assert torch.equal(got[:, before:before + B], ref.to(out).t())
        assert (got[:, :before] == -77).all() and (got[:, before + B:] == -77).all()
    tsvd.tsvd_free(h)


@pytest.mark.parametrize("M,N,K,B", [(805, 144, 1604, 866), (1572, 113, 2093, 900), (2216, 122, 832, 697), (1466, 250, 2301, 216), (1241, 315, 733, 419)])
def test_workspace_of_rows_of_tokens_is_enough(tsvd, M, N, K, B):  # noqa: F811
    """Calls that take the split tiles for rows of tokens only: nothing is written beyond the workspace that was asked for."""
    import torch
    i = workloads.make_integer_inputs(M, N, K, B, 0.5, "bf16", seed=M + B)
    ref = torch.from_numpy(np.ascontiguousarray(oracle.forward(i.U, i.S, i.V, i.X).T))
    h = tsvd.tsvd_pack(i.U, i.S, i.V)
    x = to_device(i).t().contiguous()
    need = tsvd.tsvd_workspace_bytes_ex(h, B, tsvd.TSVD_BF16, tsvd.TSVD_TOKEN_MAJOR)
    ws = torch.full((need + (32 << 20),), 93, dtype=torch.uint8, device="cuda:0")
    print(f"case workspace {M} {N} {K} {B} {need}", flush=True)
    y = tsvd.tsvd_forward_io(h, x, x_layout=tsvd.TSVD_TOKEN_MAJOR, y_layout=tsvd.TSVD_TOKEN_MAJOR, workspace=ws[:need])
    assert (ws[need:] == 93).all()
    assert torch.equal(y.cpu(), ref)
    tsvd.tsvd_free(h)


# (beside those: the single-token kernels, slabs, few tokens, ring and large tiles, narrow tiles on planes, six planes of x, the 16-bit token panel)
MORE_ROUTES = [{}, {"TSVD_GEMV": 0, "TSVD_MID": 1}, {"TSVD_FEW": 64}, {"TSVD_PANEL": 0, "TSVD_GEMM_CFG_U": 14, "TSVD_GEMM_CFG_V": 15}, {"TSVD_PANEL": 0, "TSVD_GEMM_CFG_U": 16, "TSVD_GEMM_CFG_V": 16},
               {"TSVD_PANEL": 0, "TSVD_GEMM_CFG_U": 0, "TSVD_GEMM_CFG_V": 1}, {"TSVD_PANEL": 0, "TSVD_GEMM_CFG_U": 2, "TSVD_GEMM_CFG_V": 3},
               {"TSVD_PANEL": 0, "TSVD_FP6": 1, "TSVD_FP6_V": 1, "TSVD_GEMM_CFG_V": 3, "TSVD_FP6_TALL": 3}, {"TSVD_PANEL": 0, "TSVD_FP6": 1, "TSVD_FP6_V": 2, "TSVD_GEMM_CFG_V": 3, "TSVD_FP6_TALL": 1},
               {"TSVD_PANEL": 1, "TSVD_PANEL_FP6": 0}]


@pytest.mark.parametrize("M,N,K,B", [(66, 8, 70, 40), (131, 127, 60, 33), (257, 251, 200, 136), (520, 64, 300, 16), (300, 100, 80, 1)])
@pytest.mark.parametrize("route", ROUTES + MORE_ROUTES, ids=str)
def test_what_lies_behind_y_stays(tsvd, M, N, K, B, route):  # noqa: F811
    """Rows of tiles beyond y's last row, and tokens beyond the last token, are not stored: what lies there in memory keeps its mark.  (Tests beside the columns of y
    do not show this: stores without a test of the row rest on the range of a buffer that ends with y.)"""
    import torch
    i = workloads.make_integer_inputs(M, N, K, B, 0.5, "bf16", seed=M + N + K + B)
    ref = torch.from_numpy(np.ascontiguousarray(oracle.forward(i.U, i.S, i.V, i.X)))
    h = tsvd.tsvd_pack(i.U, i.S, i.V)
    for k, v in route.items():
        tsvd.tsvd_tuning_set(k, v)
    x = to_device(i)
    for out, code in ((torch.float32, tsvd.TSVD_F32), (torch.bfloat16, tsvd.TSVD_BF16)):
        for tokens in (False, True):
            for beside in (0, 3):
                print(f"case behind y {M} {N} {K} {B} {route} {out} {tokens} {beside}", flush=True)
                rows, cols = (B, M) if tokens else (M, B)
                y = torch.full((rows + 520, cols + beside), -77.0, dtype=out, device="cuda:0")
                if tokens:
                    tsvd.tsvd_forward_io(h, x.t().contiguous(), x_layout=tsvd.TSVD_TOKEN_MAJOR, y=y[:rows, :cols], y_dtype=code, y_layout=tsvd.TSVD_TOKEN_MAJOR)
                else:
                    tsvd.tsvd_forward_ex(h, x, y=y[:rows, :cols], y_dtype=code)
                got = y.cpu()
                assert torch.equal(got[:rows, :cols], (ref.t() if tokens else ref).to(out))
                assert (got[rows:] == -77).all() and (got[:rows, cols:] == -77).all()
    tsvd.tsvd_free(h)


@pytest.mark.parametrize("M,N,K,B", [(66, 8, 70, 40), (40, 1, 60, 33), (257, 251, 200, 136), (70, 129, 60, 24), (520, 64, 300, 16), (300, 100, 80, 1)])
@pytest.mark.parametrize("route", ROUTES + MORE_ROUTES, ids=str)
def test_what_lies_behind_x_reaches_nothing(tsvd, M, N, K, B, route):  # noqa: F811
    """Features of a block beyond x's last row are not read: no number stands there in memory, for more rows than any kernel takes at a time.  Exact."""
    import torch
    i = workloads.make_integer_inputs(M, N, K, B, 0.5, "bf16", seed=M + N + K + B)
    ref = oracle.forward(i.U, i.S, i.V, i.X)
    h = tsvd.tsvd_pack(i.U, i.S, i.V)
    for k, v in route.items():
        tsvd.tsvd_tuning_set(k, v)
    x = to_device(i)
    print(f"case behind x {M} {N} {K} {B} {route}", flush=True)
    for ld in (B, B + 8 - B % 8):                 # the last one aligned
        held = torch.full(((N + 2304) * ld,), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        view = torch.as_strided(held, (N, B), (ld, 1)).copy_(x)
        assert np.array_equal(tsvd.tsvd_forward(h, view).cpu().numpy(), ref)
    held = torch.full(((B + 256) * N,), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    held[:B * N] = x.t().flatten()
    y = tsvd.tsvd_forward_io(h, held[:B * N].view(B, N), x_layout=tsvd.TSVD_TOKEN_MAJOR, y_layout=tsvd.TSVD_TOKEN_MAJOR)
    assert np.array_equal(y.cpu().numpy().T, ref)
    tsvd.tsvd_free(h)


@pytest.mark.parametrize("form,co,k,groups", [(0, 33, 3, 1), (1, 21, 3, 1), (2, 40, 3, 1), (3, 9, 5, 1), (0, 12, 5, 12)])
@pytest.mark.parametrize("tiles", [0, 1, 2])
def test_what_lies_behind_a_convolution_stays(tsvd, form, co, k, groups, tiles):  # noqa: F811
    import ctypes
    import torch
    from oracle import conv as oc
    ci, rank, images, H, W = (co if groups > 1 else 24), 20, 3, 11, 9
    mu, nv = {0: (1, k * k), 1: (k * k, 1), 2: (k, k), 3: (k, k)}[form]
    rng = np.random.default_rng(form + co)
    K = rank * groups
    U = rng.choice([-1, 0, 1], size=(co * mu, K), p=[0.2, 0.6, 0.2]).astype(np.int8)
    if groups > 1:
        U *= (np.arange(co)[:, None] // (co // groups) == np.arange(K)[None, :] // rank).astype(np.int8)
    V = rng.choice([-1, 0, 1], size=(K, ci // groups * nv), p=[0.2, 0.6, 0.2]).astype(np.int8)
    S = rng.integers(-2, 3, size=K).astype(np.float32)
    h = tsvd.tsvd_pack(U, S, V)
    if tiles:
        tsvd.tsvd_tuning_set("TSVD_THIN", tiles)
    x = torch.from_numpy(rng.integers(-2, 3, size=(ci, images, H, W)).astype(np.float32)).to("cuda:0").to(torch.bfloat16)
    print(f"case behind a convolution {form} {co} {k} {groups} {tiles}", flush=True)
    want = tsvd.tsvd_conv2d_forward(h, form, ci, co, k, k, x, (1, 1), (k // 2, k // 2), groups=groups)
    lib, geometry = tsvd.load_library(), (ctypes.c_int32 * 12)(form, ci, co, k, k, 1, 1, k // 2, k // 2, 1, 1, groups)
    need = lib.tsvd_conv2d_workspace_bytes(h.ptr, ctypes.addressof(geometry), images, H, W)
    ws = torch.empty(need + (1 << 16), dtype=torch.uint8, device="cuda:0").fill_(93)
    y = torch.full((co + 64, images, H, W), -77.0, device="cuda:0")
    assert lib.tsvd_conv2d_forward(h.ptr, ctypes.addressof(geometry), x.data_ptr(), images, H, W, None, y.data_ptr(), 0, ws.data_ptr(), need, None) == 0
    torch.cuda.synchronize()
    assert torch.equal(y[:co], want) and (y[co:] == -77).all() and (ws[need:] == 93).all()
    if groups == 1:
        ref = oc.tsvd_conv2d(x.float().cpu().numpy().transpose(1, 0, 2, 3), U, S, V, form, co, ci, k, k, (1, 1), (k // 2, k // 2), (1, 1))
        assert np.array_equal(want.cpu().numpy(), ref.transpose(1, 0, 2, 3))
    tsvd.tsvd_free(h)
