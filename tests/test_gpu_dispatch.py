"""GPU parity where a dispatch rule changes kernels: the smallest and largest sizes of each path, the edges of its
tiles and the operand alignments that it has to tell apart.  Same oracle and bars as test_gpu_ops.py."""
import ctypes
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2201_11990_amd as M
from paper_2201_11990_amd import binding as B
from parity import TOL, assert_close, dev, to_np
import test_gpu_ops
from test_gpu_ops import DT, gemm_oracle, randn

pytestmark = pytest.mark.gpu


def operands(layout, Mm, N, K, dtype, seed=3):
    return (randn((Mm, K) if layout != B.GEMM_TN else (K, Mm), dtype, seed),
            randn((N, K) if layout == B.GEMM_NT else (K, N), dtype, seed + 1, 0.3))


def shifted(t, by):
    """The same values on the device, ``by`` elements past an allocation's start: contiguous, but aligned to one element only."""
    buf = torch.empty(t.numel() + by, dtype=t.dtype, device="cuda")
    out = buf[by:].view(t.shape)
    out.copy_(t)
    return out


TILES = ("stream 256x256", "stream 256x320", "ragged 256", "ragged 128", "ragged 128 deep")   # enum gemm_tile


def picked_tile(layout, Mm, N, K, ws_bytes=0):
    """The tile that the dispatch takes for a bf16 product, None if the bf16 kernels do not take it."""
    fn = B.lib()._ZN5mtnlg19gemm_mfma_pick_tileEilllm
    fn.argtypes, fn.restype = [ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_size_t], ctypes.c_int
    t = fn(layout, Mm, N, K, ws_bytes)
    return None if t < 0 else TILES[t]


def gemm_on_tile(tile, layout, a, b, C, epilogue=0, bias=None, aux=None, workspace=None):
    """A bf16 product on the named tile, whatever the dispatch would take."""
    fn = B.lib()._ZN5mtnlg14gemm_mfma_bf16EilllPKvS1_PvS1_S2_jS2_mP12ihipStream_tii
    vp, i64 = ctypes.c_void_p, ctypes.c_int64
    fn.argtypes = [ctypes.c_int, i64, i64, i64, vp, vp, vp, vp, vp, ctypes.c_uint32, vp, ctypes.c_size_t, vp, ctypes.c_int, ctypes.c_int]
    fn.restype = ctypes.c_int
    ptr = lambda t: 0 if t is None else t.data_ptr()
    K = a.shape[0] if layout == B.GEMM_TN else a.shape[1]
    status = fn(layout, C.shape[0], C.shape[1], K, ptr(a), ptr(b), ptr(C), ptr(bias), ptr(aux), epilogue, ptr(workspace),
                0 if workspace is None else workspace.numel(), torch.cuda.current_stream().cuda_stream, -1, TILES.index(tile))
    assert status == 0


def small_fp32_tile(layout, Mm, N):
    fn = B.lib()._ZN5mtnlg23gemm_generic_small_tileEill
    fn.argtypes, fn.restype = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64], ctypes.c_bool
    return fn(layout, Mm, N)


# Rows so long that a tile's DMA offsets pass 2^31 bytes (K-contiguous from 4.2 M elements on, row-contiguous from 16.8 M): still
# the bf16 kernels, and the right rows.
@pytest.mark.parametrize("layout,shape", [(B.GEMM_NT, (136, 128, 9000008)), (B.GEMM_NN, (8, 16777224, 72)),
                                          (B.GEMM_TN, (8, 16777224, 69)), (B.GEMM_TN, (16777224, 8, 72))])
def test_bf16_gemm_on_very_long_rows(layout, shape):
    Mm, N, K = shape
    assert picked_tile(layout, Mm, N, K) is not None
    gen = torch.Generator(device="cuda").manual_seed(3)
    a = torch.randn((K, Mm) if layout == B.GEMM_TN else (Mm, K), device="cuda", generator=gen, dtype=torch.bfloat16)
    b = torch.randn((N, K) if layout == B.GEMM_NT else (K, N), device="cuda", generator=gen, dtype=torch.bfloat16)
    C = torch.full((Mm, N), float("nan"), device="cuda")
    M.mtnlg_gemm(layout, a, b, C, epilogue=B.EPI_OUT_F32)
    want = torch.zeros((Mm, N), dtype=torch.float64, device="cuda")
    for k0 in range(0, K, 1 << 18):
        k = slice(k0, k0 + (1 << 18))
        x = a[k].double().T.contiguous() if layout == B.GEMM_TN else a[:, k].double().contiguous()
        want += x @ (b[:, k].double().T.contiguous() if layout == B.GEMM_NT else b[k].double())
    # fp32 sums of K terms in one chain: relative error of about 2^-24 sqrt(K) of the result
    tol = max(TOL["fp32"], 2.0 ** -24 * math.sqrt(K) * 4)
    assert float((C - want).norm() / want.norm()) <= tol
    assert float((C - want).abs().max() / want.square().mean().sqrt()) <= 8 * tol


# fp32 matrix-instruction GEMM: one element; K shorter than a chunk of 16 and than a wave's share; the 32 and 64 tiles
# with remainders on every side; widths that are no multiple of 4 take the scalar accesses.
F32_SHAPES = [(1, 4, 4), (1, 1, 1), (33, 36, 20), (31, 64, 132), (900, 1156, 44), (1000, 3076, 20), (2044, 2052, 36), (66, 130, 17)]


@pytest.mark.parametrize("layout", [B.GEMM_NT, B.GEMM_NN, B.GEMM_TN])
@pytest.mark.parametrize("shape", F32_SHAPES)
def test_fp32_gemm_tiles_and_remainders(layout, shape):
    Mm, N, K = shape
    A, Bm = operands(layout, Mm, N, K, "fp32")
    C = torch.full((Mm, N), float("nan"), device="cuda")
    M.mtnlg_gemm(layout, dev(A), dev(Bm), C)
    want = gemm_oracle(layout, A, Bm)
    assert_close(C, want, TOL["fp32"], f"f32 gemm {layout} {shape}")
    M.mtnlg_gemm(layout, dev(A), dev(Bm), C, epilogue=B.EPI_ACCUMULATE)
    assert_close(C, 2 * want, TOL["fp32"], f"f32 gemm {layout} {shape} accumulate")


# The 64 x 64 tiles with several 32-k chunks for each of the four waves of a K split and a K tail; bf16: row lengths that are
# multiples of 4 but not of 8.
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("layout", [B.GEMM_NT, B.GEMM_NN, B.GEMM_TN])
@pytest.mark.parametrize("shape", [(1020, 1020, 1044), (1024, 1012, 268), (960, 1020, 132)])
def test_fp32_gemm_large_tile_with_long_k(dtype, layout, shape):
    Mm, N, K = shape
    assert not small_fp32_tile(layout, Mm, N)
    assert dtype == "fp32" or N % 8 or K % 8   # not a product of the bf16 kernels
    A, Bm = operands(layout, Mm, N, K, dtype)
    bias, res = randn((N,), dtype, 7), randn((Mm, N), dtype, 8)
    a, b = dev(A), dev(Bm)
    want = gemm_oracle(layout, A, Bm)
    C = torch.full((Mm, N), float("nan"), device="cuda")
    M.mtnlg_gemm(layout, a, b, C, epilogue=B.EPI_OUT_F32 if dtype == "bf16" else 0)
    assert_close(C, want, TOL["fp32"], f"{dtype} gemm {layout} {shape}")
    out, Z = (torch.full((Mm, N), float("nan"), dtype=DT[dtype], device="cuda") for _ in range(2))
    M.mtnlg_gemm(layout, a, b, out, bias=dev(bias), aux=dev(res), epilogue=B.EPI_BIAS | B.EPI_RESIDUAL)
    assert_close(out, want + to_np(bias) + to_np(res), TOL[dtype], f"{dtype} gemm {layout} {shape} bias + residual")
    M.mtnlg_gemm(layout, a, b, out, bias=dev(bias), aux=Z, epilogue=B.EPI_BIAS | B.EPI_GELU)
    assert_close(Z, want + to_np(bias), TOL[dtype], f"{dtype} gemm {layout} {shape} pre-activation")
    assert_close(out, oracle.gelu(want + to_np(bias)), TOL[dtype], f"{dtype} gemm {layout} {shape} GeLU")


# The limits of GeLU and GeLU' on these kernels, whose epilogues are the same for aligned rows and for others: z or 0, and 1 or 0.
@pytest.mark.parametrize("layout", [B.GEMM_NT, B.GEMM_NN, B.GEMM_TN])
@pytest.mark.parametrize("N", [68, 70])
def test_bf16_gemm_without_dma_at_the_limits_of_gelu(layout, N):
    Mm, K = 36, 44
    A, Bm = operands(layout, Mm, N, K, "bf16")
    acc = gemm_oracle(layout, A, Bm)
    z = torch.tensor([1e14, -1e14, 1e18, -1e18])[torch.arange(N) % 4].to(torch.bfloat16)
    aux, C = (torch.full((Mm, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    M.mtnlg_gemm(layout, dev(A), dev(Bm), C, bias=dev(z), aux=aux, epilogue=B.EPI_BIAS | B.EPI_GELU)
    rows = z.expand(Mm, N)
    assert torch.equal(aux.cpu(), rows) and torch.equal(C.cpu(), rows.clamp(min=0.0))
    out = torch.full((Mm, N), float("nan"), device="cuda")
    M.mtnlg_gemm(layout, dev(A), dev(Bm), out, aux=dev(rows.contiguous()), epilogue=B.EPI_GELU_GRAD | B.EPI_OUT_F32)
    assert_close(out, acc * (to_np(rows) > 0), TOL["fp32"], f"bf16 gemm {layout} {N} GeLU' at its limits")


# bf16 products of these kernels either side of the rule for their tiles, which is one for their times on the bf16 instructions: 72 tiles
# of 64 x 64 or 272 of 32 x 32; 272 or 1056, which went out in five rounds of small tiles where two of large ones take less; by the layout
# at 72 or 272.
@pytest.mark.parametrize("layout,shape,small", [(B.GEMM_NT, (508, 516, 260), True), (B.GEMM_NN, (508, 516, 260), True), (B.GEMM_TN, (508, 516, 259), False),
                                                (B.GEMM_NT, (1020, 1028, 132), False), (B.GEMM_NN, (1020, 1028, 132), False),
                                                (B.GEMM_NT, (252, 1020, 68), True), (B.GEMM_TN, (252, 1020, 69), True)])
def test_bf16_gemm_without_dma_on_either_tile(layout, shape, small):
    Mm, N, K = shape
    fn = B.lib()._ZN5mtnlg28gemm_generic_small_tile_bf16Eill
    fn.argtypes, fn.restype = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64], ctypes.c_bool
    assert N % 8 and fn(layout, Mm, N) == small   # N % 8: not a product of the kernels with DMA
    A, Bm = operands(layout, Mm, N, K, "bf16")
    C = torch.full((Mm, N), float("nan"), device="cuda")
    M.mtnlg_gemm(layout, dev(A), dev(Bm), C, epilogue=B.EPI_OUT_F32)
    assert_close(C, gemm_oracle(layout, A, Bm), TOL["fp32"], f"bf16 gemm {layout} {shape}")


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("layout", [B.GEMM_NT, B.GEMM_NN, B.GEMM_TN])
@pytest.mark.parametrize("Mm", [70, 72])   # 72: the weight-gradient form has 4-element accesses to lose
def test_vector_gemm_takes_operands_aligned_to_one_element(dtype, layout, Mm):
    N, K = 68, 52   # bf16: a K (NT, NN) or an N (TN) that the bf16 kernels do not take
    A, Bm = operands(layout, Mm, N, K, dtype)
    bias, res = randn((N,), dtype, 7), randn((Mm, N), dtype, 8)
    want = gemm_oracle(layout, A, Bm) + to_np(bias) + to_np(res)
    for which in range(5):
        t = [shifted(x, 1 if i == which else 0) for i, x in enumerate((A, Bm, bias, res, torch.zeros(Mm, N, dtype=DT[dtype])))]
        M.mtnlg_gemm(layout, t[0], t[1], t[4], bias=t[2], aux=t[3], epilogue=B.EPI_BIAS | B.EPI_RESIDUAL)
        assert_close(t[4], want, TOL[dtype], f"gemm {layout} {dtype} operand {which} shifted")


# Token search of the embedding gradient: less than one 64-token mask, more than one round of 4096 tokens; vocabulary rows
# that are no multiple of the 8 of a workgroup; columns beyond one 2048-column chunk; one id that takes most tokens.
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("b,s,h,V,vs", [(1, 3, 8, 8, 0), (1, 63, 2056, 24, 8), (2, 4133, 40, 16, 1000), (3, 1400, 4104, 40, 5)])
def test_embedding_token_search_and_positions(dtype, b, s, h, V, vs):
    T = b * s
    g = torch.Generator().manual_seed(5)
    tokens = torch.randint(max(0, vs - 3), vs + V + 3, (T,), generator=g, dtype=torch.int32)
    tokens[torch.rand(T, generator=g) < 0.4] = vs + V - 1
    E, P, dx = randn((V, h), dtype, 1), randn((s, h), dtype, 2), randn((T, h), dtype, 3)
    desc = B.head_desc(h, V, vs, s, b, dtype)
    x = torch.full((T, h), float("nan"), dtype=DT[dtype], device="cuda")
    M.mtnlg_embedding_fwd(desc, tokens.cuda(), dev(E), dev(P), x)
    assert_close(x, oracle.embedding_fwd(to_np(tokens), to_np(E), to_np(P), s, vs), TOL[dtype], "embedding")
    x2 = torch.empty_like(x)   # with a hook between the lookup and the positions: the same values bit for bit
    M.mtnlg_embedding_fwd(desc, tokens.cuda(), dev(E), dev(P), x2, reduce=lambda *a: None)
    assert torch.equal(x, x2)
    dE, dP = torch.full((V, h), float("nan"), dtype=DT[dtype], device="cuda"), torch.empty((s, h), dtype=DT[dtype], device="cuda")
    M.mtnlg_embedding_bwd(desc, tokens.cuda(), dev(dx), dE, dP)
    dE_o, dP_o = oracle.embedding_bwd(to_np(tokens), to_np(dx), V, s, vs)
    assert_close(dE, dE_o, TOL[dtype], "embedding gradient")
    assert_close(dP, dP_o, TOL[dtype], "position gradient")


# bf16 MFMA GEMM, one shape or more per tile kind: 128 x 128 (one element wide, less than a tile, K tails), the same with deep
# rings (more and fewer slabs than stages), 256 x 256 with ragged edges, and the aligned 256 x 256 and 256 x 320 tiles.  In
# the weight-gradient form K is not even a multiple of 8.
BF16_TILES = [((1, 8, 8), "ragged 128"), ((129, 136, 72), "ragged 128"), ((256, 128, 192), "ragged 128"),
              ((136, 264, 1032), "ragged 128 deep"), ((72, 136, 1096), "ragged 128 deep"), ((2047, 8184, 72), "ragged 256"),
              ((2048, 8192, 128), "stream 256x256"), ((2048, 10240, 64), "stream 256x320")]


@pytest.mark.parametrize("layout", [B.GEMM_NT, B.GEMM_NN, B.GEMM_TN])
@pytest.mark.parametrize("shape,tile", BF16_TILES)
def test_bf16_gemm_tile_kinds_and_ragged_edges(layout, shape, tile):
    Mm, N, K = shape
    if layout == B.GEMM_TN and K % 64:
        Mm, K = (Mm + 7) // 8 * 8 if Mm < 2000 else Mm // 8 * 8, K - 5
    assert picked_tile(layout, Mm, N, K) == tile
    check_bf16_gemm(layout, Mm, N, K, M.mtnlg_gemm)


# Every tile by name, small enough for all elements: 1 slab to more than twice the stages of any of its rings, several tiles each
# way, and (256 x 256) the last round split along K with a part of 8 slabs and one of fewer.
NAMED = [("stream 256x256", 256, 256), ("stream 256x320", 256, 320), ("ragged 256", 264, 328), ("ragged 128", 136, 264),
         ("ragged 128 deep", 264, 136)]


@pytest.mark.parametrize("layout", [B.GEMM_NT, B.GEMM_NN, B.GEMM_TN])
@pytest.mark.parametrize("slabs", [1, 2, 3, 4, 5, 9])
@pytest.mark.parametrize("tile,rows,cols", NAMED)
def test_bf16_gemm_on_each_tile_by_slabs(layout, slabs, tile, rows, cols):
    for Mm, N in ((rows, cols), (2 * rows, 3 * cols)) if slabs in (4, 9) else ((rows, cols),):
        K = 64 * slabs - (16 if tile.startswith("ragged") else 0)
        check_bf16_gemm(layout, Mm, N, K, lambda *a, **k: gemm_on_tile(tile, *a, **k))


@pytest.mark.parametrize("layout", [B.GEMM_NT, B.GEMM_NN, B.GEMM_TN])
@pytest.mark.parametrize("tile,Mm,N,K", [("stream 256x256", 256, 512, 2048), ("stream 256x256", 512, 256, 64 * 25),
                                         ("ragged 256", 264, 520, 64 * 31 + 8)])
def test_bf16_gemm_split_along_k(layout, tile, Mm, N, K):
    ws = torch.full((M.mtnlg_gemm_workspace(B.BF16, layout, Mm, N, K),), 0xFF, dtype=torch.uint8, device="cuda")
    assert ws.numel() > 0
    check_bf16_gemm(layout, Mm, N, K, lambda *a, **k: gemm_on_tile(tile, *a, workspace=ws, **k))
    assert not bool((ws == 0xFF).all()), "the partial tiles went somewhere else"


# Small problems and the fp32 ones: K split over the eight waves of a workgroup, 32 x 32 or 64 x 64 tiles.  Less than a tile and a
# slab; fewer slabs than waves, as many, and a ninth; ragged on every side.
WAVE_SHAPES = [(8, 8, 8), (40, 72, 104), (64, 64, 256), (72, 136, 520), (136, 40, 584), (96, 32, 1096)]


def gemm_by_waves(tile, layout, a, b, C, epilogue=0, bias=None, aux=None):
    fn = B.lib()._ZN5mtnlg9gemm_waveEiilllPKvS1_PvS1_S2_jiP12ihipStream_t
    vp, i64 = ctypes.c_void_p, ctypes.c_int64
    fn.argtypes = [ctypes.c_int, ctypes.c_int, i64, i64, i64, vp, vp, vp, vp, vp, ctypes.c_uint32, ctypes.c_int, vp]
    ptr = lambda t: 0 if t is None else t.data_ptr()
    K = a.shape[0] if layout == B.GEMM_TN else a.shape[1]
    assert fn(B.F32 if a.dtype == torch.float32 else B.BF16, layout, C.shape[0], C.shape[1], K, ptr(a), ptr(b), ptr(C), ptr(bias), ptr(aux),
              epilogue, tile, torch.cuda.current_stream().cuda_stream) == 0


def gemm_without_lds(layout, a, b, C, epilogue=0, bias=None, aux=None):   # fp32, 64 x 64 tiles, operands straight to registers
    fn = B.lib()._ZN5mtnlg12gemm_genericEiilllPKvS1_PvS1_S2_jP12ihipStream_t
    vp, i64 = ctypes.c_void_p, ctypes.c_int64
    fn.argtypes = [ctypes.c_int, ctypes.c_int, i64, i64, i64, vp, vp, vp, vp, vp, ctypes.c_uint32, vp]
    ptr = lambda t: 0 if t is None else t.data_ptr()
    K = a.shape[0] if layout == B.GEMM_TN else a.shape[1]
    assert fn(B.F32, layout, C.shape[0], C.shape[1], K, ptr(a), ptr(b), ptr(C), ptr(bias), ptr(aux), epilogue,
              torch.cuda.current_stream().cuda_stream) == 0


def gemm_in_parts(layout, a, b, C, epilogue=0, bias=None, aux=None):   # fp32, 128 x 128 tiles
    fn = B.lib()._ZN5mtnlg10gemm_partsEilllPKvS1_PvS1_S2_jP12ihipStream_t
    vp, i64 = ctypes.c_void_p, ctypes.c_int64
    fn.argtypes = [ctypes.c_int, i64, i64, i64, vp, vp, vp, vp, vp, ctypes.c_uint32, vp]
    ptr = lambda t: 0 if t is None else t.data_ptr()
    K = a.shape[0] if layout == B.GEMM_TN else a.shape[1]
    assert fn(layout, C.shape[0], C.shape[1], K, ptr(a), ptr(b), ptr(C), ptr(bias), ptr(aux), epilogue, torch.cuda.current_stream().cuda_stream) == 0


@pytest.mark.parametrize("layout", [B.GEMM_NT, B.GEMM_NN, B.GEMM_TN])
@pytest.mark.parametrize("shape", WAVE_SHAPES)
@pytest.mark.parametrize("tile", [32, 64])
def test_gemm_with_k_split_over_waves(tile, shape, layout):
    Mm, N, K = shape
    check_bf16_gemm(layout, Mm, N, K - 5 if layout == B.GEMM_TN else K, lambda *a, **k: gemm_by_waves(tile, *a, **k))
    K = K // 2 + 4   # slabs of 32
    check_fp32_gemm(layout, Mm, N, K - 3 if layout == B.GEMM_TN else K, lambda *a, **k: gemm_by_waves(tile, *a, **k), f"waves {tile}")


class GemmCall(ctypes.Structure):
    _fields_ = [("M", ctypes.c_int64), ("N", ctypes.c_int64), ("K", ctypes.c_int64), ("A", ctypes.c_void_p), ("B", ctypes.c_void_p),
                ("C", ctypes.c_void_p), ("aux", ctypes.c_void_p), ("epi", ctypes.c_uint32)]


class ColumnSums(ctypes.Structure):
    _fields_ = [("count", ctypes.c_int), ("rows", ctypes.c_int64), ("C", ctypes.c_int64), ("in_f32", ctypes.c_bool), ("out_f32", ctypes.c_bool),
                ("accumulate", ctypes.c_bool), ("of", ctypes.c_void_p * 6)]


# A linear layer's backward in one launch: both products, and no column sums, the bias gradient, or three of fp32 partial sums.  Less than
# a tile, ragged on every side, several tiles and slabs for every wave; 1 to 300 rows to sum.
@pytest.mark.parametrize("dtype,tile", [("bf16", 32), ("bf16", 64), ("fp32", 32)])
@pytest.mark.parametrize("T,I,O", [(8, 8, 8), (40, 72, 136), (136, 264, 72), (300, 128, 200)])
@pytest.mark.parametrize("sums", [0, 1, 3])
def test_linear_backward_in_one_launch(dtype, tile, T, I, O, sums):
    dY, X, W, z = randn((T, O), dtype, 1), randn((T, I), dtype, 2), randn((O, I), dtype, 3), randn((T, I), dtype, 4)
    code, td = (B.F32, torch.float32) if dtype == "fp32" else (B.BF16, torch.bfloat16)
    accumulate = sums != 1
    dX = torch.full((T, I), float("nan"), dtype=td, device="cuda")
    dW = torch.full((O, I), 2.0, device="cuda")
    a, x, w, zz = dev(dY), dev(X), dev(W), dev(z)
    nn = GemmCall(T, I, O, a.data_ptr(), w.data_ptr(), dX.data_ptr(), zz.data_ptr(), B.EPI_GELU_GRAD)
    tn = GemmCall(O, I, T, a.data_ptr(), x.data_ptr(), dW.data_ptr(), None, B.EPI_ACCUMULATE | (0 if dtype == "fp32" else B.EPI_OUT_F32))
    rows = 1 if T == 8 else T
    parts = [dY] if sums == 1 else [randn((rows, O), "fp32", 10 + i) for i in range(sums)]
    ins, out_f32 = [dev(p) for p in parts], dtype == "fp32" or sums == 1
    outs = [torch.full((O,), 3.0, dtype=torch.float32 if out_f32 else td, device="cuda") for _ in parts]
    cs = ColumnSums(sums, T if sums == 1 else rows, O, sums != 1 or dtype == "fp32", out_f32, accumulate)
    for i in range(sums):
        cs.of[2 * i], cs.of[2 * i + 1] = ins[i].data_ptr(), outs[i].data_ptr()
    fn = B.lib()._ZN5mtnlg15gemm_wave_groupEiRKNS_8GemmCallES2_RKNS_10ColumnSumsEiP12ihipStream_t
    fn.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    assert fn(code, ctypes.byref(nn), ctypes.byref(tn), ctypes.byref(cs), tile, torch.cuda.current_stream().cuda_stream) == 0
    assert_close(dX, gemm_oracle(B.GEMM_NN, dY, W) * oracle.gelu_grad(to_np(z)), TOL[dtype], f"dX {dtype} {tile} {T} {I} {O}")
    assert_close(dW - 2.0, gemm_oracle(B.GEMM_TN, dY, X), TOL["fp32"], f"dW {dtype} {tile} {T} {I} {O}")
    for part, out in zip(parts, outs):
        assert_close(out, to_np(part).sum(0) + (3.0 if accumulate else 0.0), TOL["fp32"] if out_f32 else TOL[dtype], f"sums {dtype} {T} {O}")


# fp32 on 128 x 128 tiles: less than a tile and a slab; 1 to 9 slabs through the ring of 3, with K tails; more row tiles than a group of 8,
# ragged on every side, where a wave's whole half of the tile lies outside.
@pytest.mark.parametrize("layout", [B.GEMM_NT, B.GEMM_NN, B.GEMM_TN])
@pytest.mark.parametrize("Mm,N,K", [(4, 4, 4), (128, 128, 32), (60, 260, 64), (132, 72, 100), (256, 128, 128), (200, 196, 156), (128, 256, 168),
                                    (1100, 136, 200), (136, 1036, 256), (192, 64, 288)])
def test_fp32_gemm_on_128_tiles(layout, Mm, N, K):
    check_fp32_gemm(layout, Mm, N, K - 3 if layout == B.GEMM_TN else K, gemm_in_parts, "128 x 128")


# fp32 on the 64 x 64 tiles without LDS in bf16 parts (sums of more than 256): less than a tile; one chunk of 32 for some of the four waves, and
# several with a tail; widths that are no multiple of 4 (scalar accesses).
@pytest.mark.parametrize("layout", [B.GEMM_NT, B.GEMM_NN, B.GEMM_TN])
@pytest.mark.parametrize("Mm,N,K", [(4, 4, 260), (60, 72, 264), (132, 196, 612), (66, 130, 301)])
def test_fp32_gemm_without_lds(layout, Mm, N, K):
    check_fp32_gemm(layout, Mm, N, K - 3 if layout == B.GEMM_TN else K, gemm_without_lds, "without LDS")


# Pointers aligned to 4 bytes only, which the kernels with DMA take: every operand and result 4 bytes past an allocation.
@pytest.mark.parametrize("layout", [B.GEMM_NT, B.GEMM_NN, B.GEMM_TN])
@pytest.mark.parametrize("route", [32, 64, 128])
def test_gemm_with_pointers_aligned_to_four_bytes(route, layout):
    Mm, N, K = 72, 136, 104
    for dtype in ("fp32", "bf16") if route < 128 else ("fp32",):
        by = 1 if dtype == "fp32" else 2
        gemm = gemm_in_parts if route == 128 else lambda *a, **k: gemm_by_waves(route, *a, **k)
        A, Bm = operands(layout, Mm, N, K, dtype)
        bias, aux, C = randn((N,), dtype, 7), randn((Mm, N), dtype, 8), shifted(torch.zeros((Mm, N), dtype=DT[dtype]), by)
        gemm(layout, shifted(A, by), shifted(Bm, by), C, bias=shifted(bias, by), aux=shifted(aux, by), epilogue=B.EPI_BIAS | B.EPI_RESIDUAL)
        assert_close(C, gemm_oracle(layout, A, Bm) + to_np(bias) + to_np(aux), TOL[dtype], f"{dtype} {route} {layout} aligned to 4 bytes")


def check_fp32_gemm(layout, Mm, N, K, gemm, what):
    shape = (Mm, N, K)
    A, Bm = operands(layout, Mm, N, K, "fp32")
    bias, aux = randn((N,), "fp32", 7), randn((Mm, N), "fp32", 8)
    want = gemm_oracle(layout, A, Bm)
    C = torch.full((Mm, N), float("nan"), device="cuda")
    gemm(layout, dev(A), dev(Bm), C)
    assert_close(C, want, TOL["fp32"], f"fp32 {what} {layout} {shape}")
    gemm(layout, dev(A), dev(Bm), C, epilogue=B.EPI_ACCUMULATE)
    assert_close(C, 2 * want, TOL["fp32"], f"fp32 {what} {layout} {shape} accumulate")
    gemm(layout, dev(A), dev(Bm), C, bias=dev(bias), aux=dev(aux), epilogue=B.EPI_BIAS | B.EPI_RESIDUAL)
    assert_close(C, want + to_np(bias) + to_np(aux), TOL["fp32"], f"fp32 {what} {layout} {shape} bias + residual")
    gemm(layout, dev(A), dev(Bm), C, aux=dev(aux), epilogue=B.EPI_GELU_GRAD)
    assert_close(C, want * oracle.gelu_grad(to_np(aux)), TOL["fp32"], f"fp32 {what} {layout} {shape} GeLU'")


# fp32 values in three bf16 parts: what the parts cannot say goes the way of the fp32 instructions.  Values whose third part or
# whose rounded first part leaves bf16's range, an infinity, a NaN; 32 x 32, 64 x 64, 128 x 128 and the 64 x 64 tiles without LDS.
@pytest.mark.parametrize("layout", [B.GEMM_NT, B.GEMM_NN, B.GEMM_TN])
@pytest.mark.parametrize("route", [32, 64, 128, 0])
def test_fp32_gemm_at_the_ends_of_the_range(route, layout):
    Mm, N, K = 96, 72, 136 if route else 280   # (up to 256 the tiles without LDS multiply on the fp32 instructions)
    gemm = {0: gemm_without_lds, 128: gemm_in_parts}.get(route, lambda *a: gemm_by_waves(route, *a))
    A, Bm = operands(layout, Mm, N, K, "fp32")
    for scale_a, scale_b in ((2.0 ** -118, 1.0), (2.0 ** -100, 2.0 ** -24), (2.0 ** 90, 2.0 ** 30)):
        C = torch.full((Mm, N), float("nan"), device="cuda")
        gemm(layout, dev(A * scale_a), dev(Bm * scale_b), C)
        assert_close(C / scale_a / scale_b if scale_a < 1 else C * (1 / scale_a) * (1 / scale_b), gemm_oracle(layout, A, Bm), TOL["fp32"],
                     f"fp32 gemm {route} {layout} scaled")
    row = (lambda t, m: t[:, m]) if layout == B.GEMM_TN else (lambda t, m: t[m])
    for bad in (float("inf"), float("nan"), 3.4e38):   # 3.4e38 rounds to an infinity in bf16
        X, Y = A.clone(), Bm.clone()
        row(X, 5)[7] = bad
        if bad == 3.4e38:
            row(X, 5)[:7] = row(X, 5)[8:] = 0.0
            Y *= 0.25
        C = torch.full((Mm, N), 7.0, device="cuda")
        gemm(layout, dev(X), dev(Y), C)
        x, y = (X.T if layout == B.GEMM_TN else X).double(), (Y.T if layout == B.GEMM_NT else Y).double()
        want = x @ y
        rest = [m for m in range(Mm) if m != 5]
        assert_close(C[rest], want[rest].numpy(), TOL["fp32"], "the other rows")
        if bad == 3.4e38:
            assert_close(C[5] * 2.0 ** -100, want[5].numpy() * 2.0 ** -100, TOL["fp32"], "the row of the large value")
        else:
            assert torch.equal(torch.isnan(C[5].cpu()), torch.isnan(want[5])) and torch.equal(torch.isinf(C[5].cpu()), torch.isinf(want[5]))


# ... and small values whose products with large ones are ordinary numbers: every digit of an fp32 value down to the smallest one has to be
# in its parts, whatever the size of the sum.  Both operands either way, and one such term among ordinary ones (in the second case
# of it the large values are beyond what the parts can say).
@pytest.mark.parametrize("layout", [B.GEMM_NT, B.GEMM_NN, B.GEMM_TN])
@pytest.mark.parametrize("route", [32, 64, 128, 0])
def test_fp32_gemm_of_small_values_times_large_ones(route, layout):
    Mm, N, K = 96, 72, 136 if route else 280
    gemm = {0: gemm_without_lds, 128: gemm_in_parts}.get(route, lambda *a: gemm_by_waves(route, *a))
    A, Bm = operands(layout, Mm, N, K, "fp32")

    def check(X, Y, what):
        C = torch.full((Mm, N), float("nan"), device="cuda")
        gemm(layout, dev(X), dev(Y), C)
        assert_close(C, gemm_oracle(layout, X, Y), TOL["fp32"], f"fp32 gemm {route} {layout} {what}")

    for small, large in ((-112, 60), (-118, 60), (-130, 90), (-136, 30), (-140, 125)):
        check(A * 2.0 ** small, Bm * 2.0 ** large, f"2^{small} x 2^{large}")
        check(A * 2.0 ** large, Bm * 2.0 ** small, f"2^{large} x 2^{small}")
    for small, large in ((-126, 100), (-124, 124)):
        X, Y = A * 2.0 ** (small + large), Bm.clone()
        col, row = (X[7], Y[7]) if layout == B.GEMM_TN else (X[:, 7], Y[:, 7] if layout == B.GEMM_NT else Y[7])
        col.zero_()
        col[5] = 1.37 * 2.0 ** small
        row *= 2.0 ** large
        check(X, Y, f"one term 2^{small} x 2^{large}")


def check_bf16_gemm(layout, Mm, N, K, gemm):
    A, Bm = operands(layout, Mm, N, K, "bf16")
    what = f"bf16 gemm {layout} {Mm} {N} {K}"
    want = gemm_oracle(layout, A, Bm)
    a, b = dev(A), dev(Bm)
    C = torch.full((Mm, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    gemm(layout, a, b, C)
    assert_close(C, want, TOL["bf16"], what)
    bias, res = randn((N,), "bf16", 7), randn((Mm, N), "bf16", 8)
    C.fill_(float("nan"))
    gemm(layout, a, b, C, bias=dev(bias), aux=dev(res), epilogue=B.EPI_BIAS | B.EPI_RESIDUAL)
    assert_close(C, want + to_np(bias) + to_np(res), TOL["bf16"], f"{what} bias + residual")
    C32 = torch.full((Mm, N), float("nan"), device="cuda")
    gemm(layout, a, b, C32, epilogue=B.EPI_OUT_F32)
    assert_close(C32, want, TOL["fp32"], f"{what} fp32 out")
    gemm(layout, a, b, C32, epilogue=B.EPI_OUT_F32 | B.EPI_ACCUMULATE)
    assert_close(C32, 2 * want, TOL["fp32"], f"{what} fp32 accumulate")


@pytest.mark.parametrize("layout", [B.GEMM_NT, B.GEMM_NN, B.GEMM_TN])
def test_bf16_gemm_writes_nothing_outside_a_ragged_result(layout):
    """Guard rows before and after C and poisoned memory after A and B: edges of every tile kind stay inside."""
    for Mm, N, K in [(136, 264, 1032), (72, 136, 72)]:
        A, Bm = operands(layout, Mm, N, K, "bf16")

        def fenced(t):
            buf = torch.full((t.numel() + 8192,), float("nan"), dtype=torch.bfloat16, device="cuda")
            v = buf[4096:4096 + t.numel()].view(t.shape)
            v.copy_(t)
            return v

        buf = torch.full((Mm * N + 8192,), 7.0, dtype=torch.bfloat16, device="cuda")
        C = buf[4096:4096 + Mm * N].view(Mm, N)
        M.mtnlg_gemm(layout, fenced(A), fenced(Bm), C)
        assert_close(C, gemm_oracle(layout, A, Bm), TOL["bf16"], f"fenced {layout}")
        assert bool((buf[:4096] == 7.0).all()) and bool((buf[4096 + Mm * N:] == 7.0).all())


# fp32 matrix-instruction attention: head sizes at and between the multiples of 32 that it is compiled for, sequences around
# the 16 rows of a wave, the 32 keys of a forward step and the 64 rows of a workgroup.
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("b,s,n,d", [(2, 17, 3, 24), (1, 65, 2, 72), (1, 129, 8, 96), (2, 100, 9, 104), (1, 15, 2, 136), (1, 79, 1, 168),
                                     (1, 33, 2, 192), (1, 90, 2, 200), (2, 70, 2, 232), (1, 64, 1, 256), (3, 1, 2, 40)])
def test_attention_at_every_compiled_head_size(dtype, b, s, n, d):
    test_gpu_ops.test_attention_fwd_bwd(dtype, b, s, n, d)


# ... with 64 rows to a workgroup (above 512 groups of 16 rows, and up to 32 rows), and at the edges of the rule: the last
# shapes with 16 rows to a workgroup and the streamed side split over its waves.
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("b,s,n,d", [(3, 100, 25, d) for d in (24, 56, 72, 104, 136, 168, 200, 232)]
                         + [(1, 32, 2, 200), (1, 33, 3, 72), (4, 250, 8, 40), (3, 250, 11, 40), (1, 530, 2, 56)])
def test_attention_by_rows_of_a_workgroup(dtype, b, s, n, d):
    test_gpu_ops.test_attention_fwd_bwd(dtype, b, s, n, d)


# fp32 at the edges of the rule for 16 or 64 rows to a workgroup, which depends on the sequence, the head size, the direction and whether there are several sequences: above
# 512 groups of 16 rows, on both sides of a limit (groups, then 1 where forward and backward take 16 rows).
@pytest.mark.parametrize("b,s,n,d", [(1, 192, 64, 32), (1, 192, 86, 32), (2, 192, 32, 64), (1, 256, 64, 88), (1, 257, 61, 64),      # 768 11, 1032 00, 768 11, 1024 01, 1037 00
                                     (1, 256, 48, 128), (1, 256, 64, 160), (1, 272, 31, 232), (1, 520, 47, 64), (1, 512, 49, 96),   # 768 11, 1024 01, 527 11, 1551 01, 1568 00
                                     (2, 256, 32, 88), (1, 513, 31, 128), (1, 513, 30, 248), (3, 513, 10, 248)])                    # 1024 11, 1023 01, 990 00, 990 11
def test_fp32_attention_by_groups_of_rows(b, s, n, d):
    test_gpu_ops.test_attention_fwd_bwd("fp32", b, s, n, d)


def attention_fwd_without_lds(b, s, n, d, scale, qkv, a, lse):
    fn = B.lib()._ZN5mtnlg17attention_fwd_f32EiiiiifPKvPvPfP12ihipStream_t
    fn.argtypes = [ctypes.c_int] * 5 + [ctypes.c_float] + [ctypes.c_void_p] * 4
    assert fn(B.F32 if qkv.dtype == torch.float32 else B.BF16, b, s, n, d, scale, qkv.data_ptr(), a.data_ptr(), lse.data_ptr(),
              torch.cuda.current_stream().cuda_stream) == 0


def attention_bwd_without_lds(b, s, n, d, scale, qkv, a, lse, da, dqkv, ws):
    fn = B.lib()._ZN5mtnlg17attention_bwd_f32EiiiiifPKvS1_PKfS1_PvS4_P12ihipStream_t
    fn.argtypes = [ctypes.c_int] * 5 + [ctypes.c_float] + [ctypes.c_void_p] * 7
    assert fn(B.F32 if qkv.dtype == torch.float32 else B.BF16, b, s, n, d, scale, qkv.data_ptr(), a.data_ptr(), lse.data_ptr(),
              da.data_ptr(), dqkv.data_ptr(), ws.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0


# bf16 with 64 rows to a workgroup and no LDS, at every compiled head size: what calls take whose sequences the DMA's 32-bit offsets do not reach.
@pytest.mark.parametrize("d", [24, 64, 72, 96, 104, 136, 160, 184])
def test_bf16_attention_without_lds(d):
    b, s, n = 3, 100, 25
    qkv, da = randn((b * s, 3 * n * d), "bf16", 21), randn((b * s, n * d), "bf16", 22)
    dims = oracle.Dims(hidden=8, heads=n, head_dim=d, ffn=8, seq=s, batch=b)
    a, dqkv = torch.full_like(da, float("nan"), device="cuda"), torch.full_like(qkv, float("nan"), device="cuda")
    lse = torch.full((b, n, s), float("nan"), device="cuda")
    ws = torch.empty(M.mtnlg_attention_bwd_workspace(b, s, n, d), dtype=torch.uint8, device="cuda")
    x, g = dev(qkv), dev(da)
    attention_fwd_without_lds(b, s, n, d, 1.0 / math.sqrt(d), x, a, lse)
    attention_bwd_without_lds(b, s, n, d, 1.0 / math.sqrt(d), x, a, lse, g, dqkv, ws)
    assert_close(a, oracle.attention_fwd(dims, to_np(qkv)), TOL["bf16"], "attention out")
    assert_close(dqkv, oracle.attention_bwd(dims, to_np(qkv), to_np(da)), TOL["bf16"], "attention dqkv")


# bf16, P and dS in fp32, streamed side through LDS: the edges of its rule (513 groups of 16 rows, s 33; s 193 / 257 with fewer), of
# the 64 rows of a block and of the head sizes that a tile of 32 k columns holds.
@pytest.mark.parametrize("b,s,n,d", [(3, 33, 58, 8), (2, 64, 65, 32), (1, 65, 104, 40), (1, 129, 58, 88), (2, 127, 33, 96), (1, 191, 43, 104),
                                     (1, 193, 3, 184), (1, 257, 2, 72), (1, 257, 17, 56), (1, 513, 1, 192), (1, 300, 2, 136)])
def test_attention_with_exact_weights(b, s, n, d):
    test_gpu_ops.test_attention_fwd_bwd("bf16", b, s, n, d)


# ... and dS of any size: one key takes all but 2^-20 of the weight and the gradient is small, so dS is about 2^-135 and every digit of it that
# fp32 holds has to be in its parts.  dq where the keys are large, dk where the queries are; without the dominating key and the column
# of its score, in which dP - D has no digits left.
@pytest.mark.parametrize("part", [0, 1])
@pytest.mark.parametrize("b,s,n,d", [(1, 257, 2, 96), (1, 100, 80, 40), (1, 257, 3, 184)])
def test_attention_with_small_score_gradients(b, s, n, d, part):
    dims = oracle.Dims(hidden=8, heads=n, head_dim=d, ffn=8, seq=s, batch=b)
    x, da = randn((b, s, n, 3, d), "fp32", 31), randn((b, s, n, d), "fp32", 32) * 2.0 ** -114
    x[..., 0, 0], x[..., 1, 0] = 32.0, 0.0
    x[:, 0, :, 1] = 0.0
    x[:, 0, :, 1, 0] = 16.0 * math.sqrt(d) / 32.0
    x[..., part, :] *= 2.0 ** -50
    x[..., 1 - part, :] *= 2.0 ** 50
    qkv, da = x.reshape(b * s, -1).to(torch.bfloat16), da.reshape(b * s, -1).to(torch.bfloat16)
    a, dqkv = torch.empty_like(da, device="cuda"), torch.empty_like(qkv, device="cuda")
    lse = torch.empty((b, n, s), device="cuda")
    ws = torch.empty(M.mtnlg_attention_bwd_workspace(b, s, n, d), dtype=torch.uint8, device="cuda")
    M.mtnlg_attention_fwd(b, s, n, d, 1.0 / math.sqrt(d), dev(qkv), a, lse)
    M.mtnlg_attention_bwd(b, s, n, d, 1.0 / math.sqrt(d), dev(qkv), a, lse, dev(da), dqkv, ws)
    want = oracle.attention_bwd(dims, to_np(qkv), to_np(da)).reshape(b, s, n, 3, d)
    got = dqkv.reshape(b, s, n, 3, d)
    assert_close(got[:, 1:, :, part, 1:], want[:, 1:, :, part, 1:], TOL["bf16"], "dq" if part == 0 else "dk")


# ... and weights of any size that fp32 has: one key scores 90 (natural units) above the others, whose weights are about 2^-130.  What they
# weigh is large and what the dominating key weighs is 0, so they are all of the result: V in a, dO in dv.  The key at the start, and in the
# third tile, where the sums of the tiles before it are scaled down by as much.
@pytest.mark.parametrize("at", [0, 150])
@pytest.mark.parametrize("b,s,n,d", [(1, 257, 17, 56), (1, 200, 40, 96), (1, 257, 3, 184)])
def test_attention_with_small_weights(b, s, n, d, at):
    dims = oracle.Dims(hidden=8, heads=n, head_dim=d, ffn=8, seq=s, batch=b)
    x, da = randn((b, s, n, 3, d), "fp32", 33), randn((b, s, n, d), "fp32", 34) * 2.0 ** 40
    x[..., 0, 0], x[..., 1, 0] = 32.0, 0.0
    x[:, at, :, 1] = 0.0
    x[:, at, :, 1, 0] = 90.0 * math.sqrt(d) / 32.0
    x[..., 2, :] *= 2.0 ** 60
    x[:, at, :, 2] = 0.0
    qkv, da = x.reshape(b * s, -1).to(torch.bfloat16), da.reshape(b * s, -1).to(torch.bfloat16)
    a, dqkv = torch.empty_like(da, device="cuda"), torch.empty_like(qkv, device="cuda")
    lse = torch.empty((b, n, s), device="cuda")
    ws = torch.empty(M.mtnlg_attention_bwd_workspace(b, s, n, d), dtype=torch.uint8, device="cuda")
    M.mtnlg_attention_fwd(b, s, n, d, 1.0 / math.sqrt(d), dev(qkv), a, lse)
    M.mtnlg_attention_bwd(b, s, n, d, 1.0 / math.sqrt(d), dev(qkv), a, lse, dev(da), dqkv, ws)
    want = oracle.attention_fwd(dims, to_np(qkv)).reshape(b, s, n, d)
    # rows that see the dominating key: of such a row the others' weights are left
    first = max(at, 1)
    assert_close(a.reshape(b, s, n, d)[:, first:], want[:, first:], TOL["bf16"], "a")
    want = oracle.attention_bwd(dims, to_np(qkv), to_np(da)).reshape(b, s, n, 3, d)
    assert_close(dqkv.reshape(b, s, n, 3, d)[:, at + 1:, :, 2], want[:, at + 1:, :, 2], TOL["bf16"], "dv")


# ... and values whose sums leave the range of the scaled parts, but not that of fp32: V (dP stays ordinary, the gradient is small), then K with
# the gradient (P stays ordinary, Q is small).
@pytest.mark.parametrize("b,s,n,d", [(1, 100, 80, 40), (1, 257, 3, 96)])
@pytest.mark.parametrize("part", [1, 2])
def test_attention_with_large_values(b, s, n, d, part):
    dims = oracle.Dims(hidden=8, heads=n, head_dim=d, ffn=8, seq=s, batch=b)
    x, da = randn((b, s, n, 3, d), "fp32", 35), randn((b, s, n, d), "fp32", 36)
    if part == 2:
        x[..., 2, :] *= 2.0 ** 112
        da *= 2.0 ** -100
    else:
        x[..., 0, :] *= 2.0 ** -60
        x[..., 1, :] *= 2.0 ** 60
        da *= 2.0 ** 50
    qkv, da = x.reshape(b * s, -1).to(torch.bfloat16), da.reshape(b * s, -1).to(torch.bfloat16)
    a, dqkv = torch.empty_like(da, device="cuda"), torch.empty_like(qkv, device="cuda")
    lse = torch.empty((b, n, s), device="cuda")
    ws = torch.empty(M.mtnlg_attention_bwd_workspace(b, s, n, d), dtype=torch.uint8, device="cuda")
    M.mtnlg_attention_fwd(b, s, n, d, 1.0 / math.sqrt(d), dev(qkv), a, lse)
    M.mtnlg_attention_bwd(b, s, n, d, 1.0 / math.sqrt(d), dev(qkv), a, lse, dev(da), dqkv, ws)
    assert_close(a, oracle.attention_fwd(dims, to_np(qkv)), TOL["bf16"], "a")
    want, got = oracle.attention_bwd(dims, to_np(qkv), to_np(da)).reshape(b, s, n, 3, d), dqkv.reshape(b, s, n, 3, d)
    for i in range(3):
        assert_close(got[:, :, :, i], want[:, :, :, i], TOL["bf16"], f"d{'qkv'[i]}")


# Backward in one launch, dk / dv with a D of its own: two rows (with one dq is the rounding of dP - D), the edges of a 64-row block and of the 128 rows that a pass of D takes, and
# either side of the rule (up to 320 blocks, 296 for s 65 to 96; head size 64 up to 768, 256 beyond s 1024).
@pytest.mark.parametrize("b,s,n,d", [(1, 2, 1, 128), (2, 63, 3, 64), (1, 64, 2, 160), (1, 65, 1, 128), (1, 129, 2, 64), (3, 191, 1, 160), (1, 1030, 1, 64),
                                     (4, 64, 64, 128), (1, 64, 257, 160), (3, 100, 128, 64), (1, 97, 385, 64), (1, 64, 320, 128), (1, 64, 321, 160), (1, 70, 148, 160), (1, 70, 149, 128),
                                     (1, 1030, 16, 64)])
def test_attention_backward_in_one_launch(b, s, n, d):
    test_gpu_ops.test_attention_fwd_bwd("bf16", b, s, n, d)


# Backward in two launches at head sizes 128 and 160 (from 321 blocks of 64 rows on), workgroups of 64 own rows and of 128 rows with tiles of 32 (s 65 to 128; s 129 to 1024 from 513 blocks on; others
# from 768 on, but s 33 to 64 never): either side of the rules, ends of sequences at the edges of a 32-row part, of a tile and of the own rows.
@pytest.mark.parametrize("b,s,n,d", [(1, 64, 321, 128), (1, 33, 321, 128), (1, 96, 161, 160), (3, 127, 64, 128), (1, 97, 192, 160), (1, 191, 170, 128), (1, 191, 255, 128),
                                     (1, 95, 384, 128), (3, 129, 85, 160), (2, 129, 128, 160), (1, 32, 768, 128), (1, 64, 768, 160), (2, 161, 128, 128), (1, 257, 154, 160),
                                     (1, 200, 81, 160)])
def test_attention_backward_by_rows_of_a_workgroup(b, s, n, d):
    test_gpu_ops.test_attention_fwd_bwd("bf16", b, s, n, d)


# Forward by workgroups of 64 and of 128 own rows: either side of the rules (by workgroups of 128 rows: 448, 512 and 1024; head size 64: 896 and 1024, s from 512 on, and 896 blocks of 64 rows below),
# sequences that end at the edges of a 32-row part, of a tile and of the own rows, two rows (with one dq is the rounding of dP - D) and one head; and the short
# sequences that have 16 rows to a wave (head size 64 up to 512 blocks, others up to 32 tokens); a number of heads that is no multiple of 4 (257 to 512 blocks).
@pytest.mark.parametrize("b,s,n,d", [(1, 2, 1, 128), (2, 31, 3, 160), (1, 33, 2, 64), (1, 64, 448, 128), (3, 65, 150, 160), (1, 97, 512, 128), (1, 96, 513, 160),
                                     (1, 129, 511, 128), (4, 127, 256, 160), (1, 161, 256, 128), (1, 257, 342, 128), (1, 513, 180, 64), (2, 545, 102, 64), (1, 640, 205, 64),
                                     (1, 64, 512, 64), (1, 49, 513, 64), (2, 65, 65, 64), (1, 128, 256, 64), (1, 95, 257, 64), (1, 127, 449, 64), (1, 205, 225, 64),
                                     (1, 32, 9, 128), (1, 17, 255, 160), (1, 200, 81, 128), (1, 385, 47, 160), (1, 100, 129, 160), (1, 769, 21, 128), (1, 384, 86, 160), (1, 768, 23, 128), (1, 120, 140, 160), (1, 600, 91, 128), (1, 1030, 57, 160)])
def test_attention_forward_by_rows_of_a_workgroup(b, s, n, d):
    test_gpu_ops.test_attention_fwd_bwd("bf16", b, s, n, d)


# With fp32 weights, forward and backward on 16 or 32 rows to a wave and 64 or 128 to a workgroup: either side of the rules (704, 768 and 2048 blocks of 64 rows; short sequences up to 512,
# 384 and 256 blocks by head size; backward by head size, sequence and blocks).
@pytest.mark.parametrize("b,s,n,d", [(3, 100, 30, 24), (1, 65, 383, 40), (2, 96, 192, 56), (1, 127, 351, 72), (1, 97, 352, 88), (1, 33, 2047, 96), (1, 95, 1024, 104),
                                     (1, 129, 683, 152), (2, 161, 342, 80), (1, 513, 17, 112), (1, 35, 2048, 184),
                                     (1, 64, 384, 72), (1, 63, 256, 104), (1, 49, 257, 120), (1, 128, 256, 112), (1, 65, 129, 152), (1, 48, 200, 144), (1, 66, 129, 40), (1, 200, 81, 144), (1, 270, 90, 72),
                                     (1, 33, 513, 88), (1, 96, 129, 96), (1, 95, 128, 96), (1, 191, 257, 80), (1, 193, 193, 72), (1, 385, 30, 72), (1, 100, 129, 128), (1, 520, 80, 56),
                                     (1, 780, 40, 48), (1, 50, 257, 136), (1, 129, 257, 136), (1, 65, 200, 168), (1, 97, 200, 192)])
def test_attention_with_exact_weights_by_rows(b, s, n, d):
    test_gpu_ops.test_attention_fwd_bwd("bf16", b, s, n, d)


@pytest.mark.parametrize("n,d", [(44, 24), (70, 56), (352, 88), (384, 40), (70, 104), (1024, 120), (70, 152), (250, 192)])
def test_attention_with_exact_weights_by_rows_non_finite_token(n, d):
    check_non_finite_token("bf16", n, d, 37, float("inf"), M.mtnlg_attention_fwd, M.mtnlg_attention_bwd)


# The same for the kernels without LDS: fp32 and small bf16 calls on either side of the rules (512, 256 and 128 groups of 16 rows), head sizes that have
# no such launch, one row (dq is exactly zero).
@pytest.mark.parametrize("dtype,b,s,n,d", [("fp32", 1, 1, 1, 64), ("fp32", 1, 64, 128, 96), ("fp32", 1, 64, 129, 96), ("fp32", 2, 127, 16, 128),
                                           ("fp32", 1, 33, 42, 160), ("fp32", 1, 33, 43, 160), ("fp32", 1, 100, 2, 192), ("bf16", 1, 1, 2, 96),
                                           ("bf16", 1, 128, 32, 72), ("bf16", 1, 49, 65, 24), ("bf16", 1, 99, 18, 184), ("bf16", 1, 113, 16, 256)])
def test_attention_backward_in_one_launch_without_lds(dtype, b, s, n, d):
    test_gpu_ops.test_attention_fwd_bwd(dtype, b, s, n, d)


# An infinity or NaN in one token reaches only what depends on that token.  K and V of token t0: outputs and dq of the rows before it
# stay as they were; Q and dO of token t0: dk and dv of the keys after it.  t0 at the start, inside and at the end of a 16-row
# block, and the last token, whose block hangs over the end of the sequence.
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("t0", [0, 32, 37, 63, 89])
# 2 heads: 16 rows to a workgroup (head size 224: the backward kernels in two launches); 44 heads: 64 rows, and bf16 up to head size 192
# through LDS, in tiles of as many columns, of an even number of 32, and with columns past the head size.
@pytest.mark.parametrize("dtype,n,d", [("fp32", 2, 24), ("fp32", 2, 64), ("fp32", 2, 96), ("fp32", 2, 224), ("bf16", 2, 40), ("bf16", 2, 96),
                                       ("fp32", 44, 24), ("fp32", 44, 96), ("bf16", 44, 96), ("bf16", 44, 40), ("bf16", 44, 184), ("bf16", 44, 200)])
def test_attention_non_finite_token_stays_where_it_belongs(dtype, n, d, t0, bad):
    check_non_finite_token(dtype, n, d, t0, bad, M.mtnlg_attention_fwd, M.mtnlg_attention_bwd)


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("t0", [0, 37, 63, 89])
@pytest.mark.parametrize("d", [40, 96])   # bf16, 64 rows to a workgroup without LDS
def test_attention_without_lds_non_finite_token_stays_where_it_belongs(d, t0, bad):
    check_non_finite_token("bf16", 44, d, t0, bad, attention_fwd_without_lds, attention_bwd_without_lds)


def check_non_finite_token(dtype, n, d, t0, bad, attention_fwd, attention_bwd):
    b, s, col = 2, 90, 5
    dims = oracle.Dims(hidden=8, heads=n, head_dim=d, ffn=8, seq=s, batch=b)
    qkv, da = randn((b, s, n, 3, d), dtype, 51), randn((b, s, n, d), dtype, 52)
    flat = lambda t: dev(t.reshape(b * s, -1))

    def run(x, g):
        a, dx = torch.full_like(g, 7.0, device="cuda").reshape(b * s, -1), torch.full_like(x, 7.0, device="cuda").reshape(b * s, -1)
        lse = torch.full((b, n, s), 7.0, device="cuda")
        ws = torch.empty(M.mtnlg_attention_bwd_workspace(b, s, n, d), dtype=torch.uint8, device="cuda")
        fx, fg = flat(x), flat(g)
        attention_fwd(b, s, n, d, 1.0 / math.sqrt(d), fx, a, lse)
        attention_bwd(b, s, n, d, 1.0 / math.sqrt(d), fx, a, lse, fg, dx, ws)
        return a.reshape(b, s, n, d), lse, dx.reshape(b, s, n, 3, d)

    want_a = oracle.attention_fwd(dims, to_np(qkv).reshape(b * s, -1)).reshape(b, s, n, d)
    want_dx = oracle.attention_bwd(dims, to_np(qkv).reshape(b * s, -1), to_np(da).reshape(b * s, -1)).reshape(b, s, n, 3, d)
    _, lse0, _ = run(qkv, da)
    for part in (1, 2):   # K, V of token t0 in head 1 of sequence 0
        x = qkv.clone()
        x[0, t0, 1, part, col] = bad
        a, lse, dx = run(x, da)
        for name, got, want in (("a", a, want_a), ("dq", dx[:, :, :, 0], want_dx[:, :, :, 0])):
            assert_close(got[:, :, 0], want[:, :, 0], TOL[dtype], f"{name} of the other head")
            assert_close(got[1], want[1], TOL[dtype], f"{name} of the other sequence")
            if t0 > 0:
                assert_close(got[0, :t0, 1], want[0, :t0, 1], TOL[dtype], f"{name} before token {t0}")
        assert torch.equal(lse[1], lse0[1]) and torch.equal(lse[0, 0], lse0[0, 0])
        if t0 > 0:
            assert_close(lse[0, 1, :t0], to_np(lse0[0, 1, :t0]), TOL["fp32"], f"lse before token {t0}")
        if part == 2:   # V enters one column of the output, in every later row
            assert not bool(torch.isfinite(a[0, t0:, 1, col].float()).any())
            rest = [c for c in range(d) if c != col]
            assert_close(a[0, :, 1][:, rest], want_a[0, :, 1][:, rest], TOL[dtype], "the other columns")
    for poison_q in (True, False):   # Q, dO of token t0
        x, g = qkv.clone(), da.clone()
        if poison_q:
            x[0, t0, 1, 0, col] = bad
        else:
            g[0, t0, 1, col] = bad
        _, _, dx = run(x, g)
        for i in (1, 2):
            assert_close(dx[1, :, :, i], want_dx[1, :, :, i], TOL[dtype], "the other sequence")
            if t0 + 1 < s:
                assert_close(dx[0, t0 + 1:, 1, i], want_dx[0, t0 + 1:, 1, i], TOL[dtype], f"d{'qkv'[i]} after token {t0}")
            if not poison_q and i == 2:
                assert not bool(torch.isfinite(dx[0, :t0 + 1, 1, 2, col].float()).any())


# Backward at head sizes 128 and 160, one launch and two, 64 and 128 own rows: an infinity in V of one key, with a and lse from before it, enters dP of that key only;
# so dk of the other keys, and all of dv, keep every bit (dk / dv hands P on through LDS that V of its own rows came through).
@pytest.mark.parametrize("b,s,n,d", [(1, 64, 6, 128), (1, 64, 330, 128), (1, 128, 400, 128), (1, 64, 330, 160), (1, 128, 400, 160)])
def test_attention_backward_infinity_in_one_key(b, s, n, d):
    qkv, da = randn((b * s, n, 3, d), "bf16", 53), dev(randn((b * s, n * d), "bf16", 54))
    x, a, lse = dev(qkv.reshape(b * s, -1)), torch.empty_like(da), torch.empty((b, n, s), device="cuda")
    ws = torch.empty(M.mtnlg_attention_bwd_workspace(b, s, n, d), dtype=torch.uint8, device="cuda")
    M.mtnlg_attention_fwd(b, s, n, d, 1.0 / math.sqrt(d), x, a, lse)

    def backward(x):
        dx = torch.full_like(x, 7.0)
        M.mtnlg_attention_bwd(b, s, n, d, 1.0 / math.sqrt(d), x, a, lse, da, dx, ws)
        return dx.reshape(s, n, 3, d)

    want = backward(x)
    for key in (3, s - 28):
        bad = x.clone()
        bad.reshape(s, n, 3, d)[key, 1, 2, 5] = float("inf")
        got = backward(bad)
        others = [t for t in range(s) if t != key]
        assert torch.equal(got[others][:, :, 1], want[others][:, :, 1]), f"dk of the keys besides {key}"
        assert torch.equal(got[:, :, 2], want[:, :, 2]), "dv"


# Head sizes 64, 128 and 160 without the slow path: an infinity or NaN in K or V of one token reaches outputs of the token's 64-row tile and of later rows,
# whatever the number of rows of a workgroup (forward: 64, and 128 from 449 to 512 and from 1024 workgroups of 128 rows on; head size 64 from 897 to 1024).  The rows
# before, the other heads and the other sequence keep every bit.
REACH_CASES = [(2, 200, 3, 64), (2, 520, 100, 64), (2, 200, 3, 128), (2, 200, 120, 128), (2, 200, 260, 128), (2, 200, 3, 160), (2, 200, 120, 160)]


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("t0", [70, 127, 199])
@pytest.mark.parametrize("b,s,n,d", REACH_CASES)
def test_attention_forward_non_finite_token_reach(b, s, n, d, t0, bad):
    qkv = dev(randn((b * s, 3 * n * d), "bf16", 55))

    def forward(x):
        a, lse = torch.full((b, s, n, d), 7.0, device="cuda", dtype=torch.bfloat16), torch.full((b, n, s), 7.0, device="cuda")
        M.mtnlg_attention_fwd(b, s, n, d, 1.0 / math.sqrt(d), x, a.view(b * s, -1), lse)
        return a, lse

    a0, lse0 = forward(qkv)
    first = t0 // 64 * 64
    for part in (1, 2):   # K, V of token t0 in head 1 of sequence 0
        x = qkv.clone()
        x.view(b, s, n, 3, d)[0, t0, 1, part, 5] = bad
        a, lse = forward(x)
        assert torch.equal(a[1], a0[1]) and torch.equal(lse[1], lse0[1]), "the other sequence"
        others = [j for j in range(n) if j != 1]
        assert torch.equal(a[0][:, others], a0[0][:, others]) and torch.equal(lse[0][others], lse0[0][others]), "the other heads"
        assert torch.equal(a[0, :first, 1], a0[0, :first, 1]) and torch.equal(lse[0, 1, :first], lse0[0, 1, :first]), f"rows before {first}"


# Backward: K or V of the token reach dq of its tile and of later rows; Q or dO of it dk and dv of the keys up to the end of its tile.  (One launch; two, with 64 rows to a workgroup; with 128.)
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("t0", [70, 127, 199])
@pytest.mark.parametrize("b,s,n,d", [(2, 200, 3, 64), (2, 200, 3, 128), (2, 200, 60, 128), (2, 200, 120, 128), (2, 200, 3, 160), (2, 200, 60, 160), (2, 230, 120, 160)])
def test_attention_backward_non_finite_token_reach(b, s, n, d, t0, bad):
    qkv, da = dev(randn((b * s, 3 * n * d), "bf16", 55)), dev(randn((b * s, n * d), "bf16", 56))

    def step(x, g):
        a, dx, lse = torch.empty_like(g), torch.full_like(x, 7.0), torch.empty((b, n, s), device="cuda")
        ws = torch.empty(M.mtnlg_attention_bwd_workspace(b, s, n, d), dtype=torch.uint8, device="cuda")
        M.mtnlg_attention_fwd(b, s, n, d, 1.0 / math.sqrt(d), x, a, lse)
        M.mtnlg_attention_bwd(b, s, n, d, 1.0 / math.sqrt(d), x, a, lse, g, dx, ws)
        return dx.view(b, s, n, 3, d)

    want = step(qkv, da)
    first, end = t0 // 64 * 64, t0 // 64 * 64 + 64
    for part in range(4):   # Q, K, V, dO of token t0 in head 1 of sequence 0
        x, g = qkv.clone(), da.clone()
        (g.view(b, s, n, 1, d) if part == 3 else x.view(b, s, n, 3, d))[0, t0, 1, part % 3, 5] = bad
        got = step(x, g)
        others = [j for j in range(n) if j != 1]
        assert torch.equal(got[1], want[1]) and torch.equal(got[0][:, others], want[0][:, others]), "the other sequence and heads"
        if part in (1, 2):
            assert torch.equal(got[0, :first, 1, 0], want[0, :first, 1, 0]), f"dq of the rows before {first}"
        else:
            assert torch.equal(got[0, end:, 1, 1:], want[0, end:, 1, 1:]), f"dk, dv of the keys from {end} on"


# Weights in fp32 with each half of the keys under a maximum of its own: lse of scores around 160, which are whole numbers times the scale, so that only the softmax rounds.  What is left is the rounding of
# the result, half a unit in its last place, and the error of a logarithm and a sum of fp32 weights, below 1e-6 where that unit is 1.5e-5: 0.57 of it in all.
@pytest.mark.parametrize("s,n,d", [(512, 16, 96), (330, 8, 120), (300, 4, 152)])
def test_attention_with_exact_weights_lse_of_large_scores(s, n, d):
    g = torch.Generator().manual_seed(57)
    qkv = torch.randint(-3, 4, (s, n, 3, d), generator=g).float()
    qkv[:, :, 0, 0] = 16.0
    qkv[:, :, 1, 0] = 100.0
    scale = float(np.float32(0.0971))
    x = dev(qkv.reshape(s, -1).bfloat16())
    a, lse = torch.empty((s, n * d), device="cuda", dtype=torch.bfloat16), torch.empty((1, n, s), device="cuda")
    M.mtnlg_attention_fwd(1, s, n, d, scale, x, a, lse)
    S = np.einsum("snd,tnd->nst", qkv[:, :, 0].double().numpy(), qkv[:, :, 1].double().numpy()) * scale
    S = np.where(np.tril(np.ones((s, s), bool)), S, -np.inf)
    want = np.log(np.exp(S - S.max(-1, keepdims=True)).sum(-1)) + S.max(-1)
    ulps = np.abs(lse[0].double().cpu().numpy() - want) / np.spacing(want.astype(np.float32)).astype(np.float64)
    assert ulps.max() <= 0.57, ulps.max()


# The weights of head sizes 64, 128 and 160 are rounded to bf16 relative to a running maximum, whose own weight rounds to itself.  The error of a is no larger than with the maximum of the first 64 keys, moved
# when a later one is 2^8 beyond it (the bound: 0.5 %, twice what draws of the inputs differ by); workgroups of 128 queries, and of 64.
@pytest.mark.parametrize("b,s,n,d", [(2, 512, 60, 128), (1, 900, 64, 160), (1, 640, 200, 64), (1, 600, 8, 128)])
def test_attention_forward_error_of_rounded_weights(b, s, n, d):
    g = torch.Generator(device="cuda").manual_seed(58)
    qkv = torch.randn((b, s, n, 3, d), generator=g, device="cuda").bfloat16()
    a, lse = torch.empty((b * s, n * d), device="cuda", dtype=torch.bfloat16), torch.empty((b, n, s), device="cuda")
    M.mtnlg_attention_fwd(b, s, n, d, 1.0 / math.sqrt(d), qkv.view(b * s, -1), a, lse)
    got, mask = a.view(b, s, n, d).double(), torch.ones(s, s, dtype=torch.bool, device="cuda").triu(1)
    ours = theirs = 0.0
    for i in range(b):
        for j in range(n):
            q, k, v = (qkv[i, :, j, c].double().contiguous() for c in range(3))
            x = (q @ k.t().contiguous() / math.sqrt(d) * math.log2(math.e)).masked_fill(mask, -math.inf)
            p = torch.softmax(x * math.log(2), -1)
            want, m, num, den = p @ v, torch.full((s,), -math.inf, device="cuda", dtype=torch.float64), 0.0, 0.0
            for u in range(0, s, 64):
                top = x[:, u:u + 64].amax(-1)
                m_new = torch.where(top > m + 8, top, m)
                w, alpha = torch.exp2(x[:, u:u + 64] - m_new[:, None]), torch.exp2(m - m_new)[:, None]
                num, den, m = num * alpha + w.bfloat16().double() @ v[u:u + 64], den * alpha + w.sum(-1, keepdim=True), m_new
            ours += ((got[i, :, j] - want) ** 2).sum().item()
            theirs += (((num / den).bfloat16().double() - want) ** 2).sum().item()
    assert math.sqrt(ours / theirs) <= 1.005, math.sqrt(ours / theirs)


# Matrix-core attention over very many heads, whose workgroups are dealt out in rows of a few heads each, in the backward kernels
# of others than in the forward kernel: sequences do not depend on each other, so two calls on parts give the same bytes.
def test_attention_batches_of_several_grid_rows():
    b, s, n, d = 4001, 2, 17, 64
    gen = torch.Generator(device="cuda").manual_seed(3)
    qkv = torch.randn(b * s, 3 * n * d, device="cuda", generator=gen).bfloat16()
    da = torch.randn(b * s, n * d, device="cuda", generator=gen).bfloat16()

    def run(lo, hi):
        x, g = qkv[lo * s:hi * s], da[lo * s:hi * s]
        a, dx = torch.full_like(g, float("nan")), torch.full_like(x, float("nan"))
        lse = torch.full((hi - lo, n, s), float("nan"), device="cuda")
        ws = torch.empty(M.mtnlg_attention_bwd_workspace(hi - lo, s, n, d), dtype=torch.uint8, device="cuda")
        M.mtnlg_attention_fwd(hi - lo, s, n, d, 0.125, x, a, lse)
        M.mtnlg_attention_bwd(hi - lo, s, n, d, 0.125, x, a, lse, g, dx, ws)
        return a, lse, dx

    for whole, first, second in zip(run(0, b), run(0, 2000), run(2000, b)):
        assert torch.equal(whole, torch.cat([first, second]))


# Many heads.  Backward: one launch (the first two cases), two blocks of a head to a workgroup (head size 64, s 65 to 128), 128 rows and 64 (the last case but one) to a workgroup.  Forward: 64 queries to a workgroup,
# and 128 (24 x 128 and the last case).  The heads in several grid rows, the last one shorter and no multiple of 8: forward all but the first three cases and 24 x 128, backward all but the first three.
@pytest.mark.parametrize("b,s,n,d", [(5, 192, 20, 128), (12, 100, 25, 64), (16, 100, 25, 64), (12, 130, 25, 128), (12, 130, 25, 160), (24, 128, 25, 64),
                                     (12, 260, 25, 128), (12, 260, 25, 160), (20, 449, 13, 64), (12, 130, 43, 160)])
def test_attention_of_many_heads(b, s, n, d):
    qkv, da = randn((b * s, 3 * n * d), "bf16", 21), randn((b * s, n * d), "bf16", 22)
    dims = oracle.Dims(hidden=8, heads=n, head_dim=d, ffn=8, seq=s, batch=b)
    scale = 1.0 / math.sqrt(d)
    a = torch.full((b * s, n * d), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((b, n, s), float("nan"), device="cuda")
    M.mtnlg_attention_fwd(b, s, n, d, scale, dev(qkv), a, lse)
    ws = torch.empty(M.mtnlg_attention_bwd_workspace(b, s, n, d), dtype=torch.uint8, device="cuda")
    dqkv = torch.full(qkv.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    M.mtnlg_attention_bwd(b, s, n, d, scale, dev(qkv), a, lse, dev(da), dqkv, ws)
    assert_close(a, oracle.attention_fwd(dims, to_np(qkv)), TOL["bf16"], "attention out")
    assert_close(dqkv, oracle.attention_bwd(dims, to_np(qkv), to_np(da)), TOL["bf16"], "attention dqkv")


# One key that scores 100 (natural units) above all others, head by head at every position modulo 16 and, by sequence, in the
# first tile, a middle one and the last: exponents taken from any but the maximum over all keys overflow.  208 rows: 16 heads x 3
# and x 18 sequences go to workgroups of 64 queries, whose halves of the keys have a maximum each, x 32 to workgroups of 128 at head sizes 128 and 160.
@pytest.mark.parametrize("d", [64, 128, 160])
@pytest.mark.parametrize("b", [3, 18, 32])
def test_attention_with_one_dominating_key(b, d):
    s, n = 208, 16
    g = torch.Generator().manual_seed(17)
    qkv = torch.randn((b, s, n, 3, d), generator=g)
    qkv[..., 0, 0] = 32.0
    qkv[..., 1, 0] = 0.0
    for bi in range(b):
        for j in range(n):
            first = (0, 64 + 16 * (bi // 3 % 8), 192)[bi % 3]
            qkv[bi, first + j, j, 1, 0] = 104.0 * math.sqrt(d) / 32.0   # + the other products, a few units
    qkv = qkv.reshape(b * s, 3 * n * d).to(torch.bfloat16)
    da = randn((b * s, n * d), "bf16", 18)
    dims = oracle.Dims(hidden=8, heads=n, head_dim=d, ffn=8, seq=s, batch=b)
    scale = 1.0 / math.sqrt(d)
    a = torch.full((b * s, n * d), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((b, n, s), float("nan"), device="cuda")
    M.mtnlg_attention_fwd(b, s, n, d, scale, dev(qkv), a, lse)
    ws = torch.empty(M.mtnlg_attention_bwd_workspace(b, s, n, d), dtype=torch.uint8, device="cuda")
    dqkv = torch.full(qkv.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    M.mtnlg_attention_bwd(b, s, n, d, scale, dev(qkv), a, lse, dev(da), dqkv, ws)
    for name, t in (("a", a), ("lse", lse), ("dqkv", dqkv)):
        bad = ~torch.isfinite(t.float())
        assert not bool(bad.any()), f"{name}: {int(bad.sum())} of {bad.numel()} not finite"
    assert_close(a, oracle.attention_fwd(dims, to_np(qkv)), TOL["bf16"], "attention out")
    assert_close(dqkv, oracle.attention_bwd(dims, to_np(qkv), to_np(da)), TOL["bf16"], "attention dqkv")


# LayerNorm backward: the widths between which the number of waves to a row changes (512, 1024, 2048, 4096 columns; below 2^18
# elements all 16 whatever the width) and the row count per thread (8192, 16384, 24576); fewer rows than a workgroup takes at a time,
# and several turns of the row loop with and without a remainder.
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("T,h", [(1, 8), (3, 512), (700, 512), (259, 520), (40, 1024), (9, 1032), (1030, 2048), (511, 512), (513, 512), (505, 520), (515, 1024), (300, 1032), (130, 2056), (1100, 8), (5, 2056), (600, 4096),
                                 (3, 4104), (300, 8192), (2, 8200), (2, 16392), (2, 24584)])
def test_layernorm_backward_widths_and_rows(dtype, T, h):
    x, dout, dres = randn((T, h), dtype, 1), randn((T, h), dtype, 2), randn((T, h), dtype, 3)
    gamma = randn((h,), dtype, 4)
    _, mean, rstd = oracle.layernorm_fwd(to_np(x), to_np(gamma), np.zeros(h), 1e-5)
    mean_d, rstd_d = (torch.tensor(v, dtype=torch.float32, device="cuda") for v in (mean, rstd))
    ws = torch.empty(M.mtnlg_layernorm_bwd_workspace(T, h), dtype=torch.uint8, device="cuda")
    o_dx, o_dg, o_db = oracle.layernorm_bwd(to_np(x), to_np(gamma), mean, rstd, to_np(dout))
    for res in (None, dres):
        dx = torch.full((T, h), float("nan"), dtype=DT[dtype], device="cuda")
        dg, db, cs = (torch.full((h,), float("nan"), device="cuda") for _ in range(3))
        M.mtnlg_layernorm_bwd(dev(x), dev(gamma), mean_d, rstd_d, dev(dout), dx, dg, db, ws, grad_f32=True,
                              dres=None if res is None else dev(res), colsum_dx=None if res is None else cs)
        want = o_dx if res is None else o_dx + to_np(res)
        assert_close(dx, want, TOL[dtype], f"dx {T} {h}")
        assert_close(dg, o_dg, TOL[dtype], f"dgamma {T} {h}")
        assert_close(db, o_db, TOL[dtype], f"dbeta {T} {h}")
        if res is not None:
            assert_close(cs, to_np(dx).sum(0), TOL["fp32"], f"column sum of the stored dx {T} {h}")


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("T,C", [(1, 8), (15, 520), (64, 512), (65, 1032), (700, 64), (2049, 520), (5000, 8)])
def test_column_sums_row_remainders(dtype, T, C):
    x = randn((T, C), dtype, 5)
    ws = torch.empty(M.mtnlg_colsum_workspace(T, C), dtype=torch.uint8, device="cuda")
    out = torch.full((C,), float("nan"), device="cuda")
    M.mtnlg_colsum(dev(x), out, ws)
    assert_close(out, to_np(x).sum(0), TOL["fp32"], f"colsum {T} {C}")
