"""The fast mode's short-K kernel (K = 64 .. 256, the Backward GEMM of a layer)
against the streamed kernel, whose instruction and lane layout it shares: the
same bits, at the edges of its 32-row blocks and 128-column tiles, at every
slab count, with chunks of one and of several slabs, on both epilogues."""
import numpy as np
import pytest
import torch

import oracle
import paper_1812_08011_amd as fp8t
from tests.gpu_util import DEV, dev, gemm, host, say
from tests.test_gpu_kernels import check_fast

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fp8t.lib()
    yield


@pytest.mark.parametrize("K,CL", [(64, 64), (128, 64), (192, 64), (256, 64), (128, 128),
                                  (192, 128), (256, 128), (256, 256), (192, 192)])
@pytest.mark.parametrize("M,N,tb,pad,special", [
    (1, 1, 1, 0, ""), (33, 129, 1, 0, ""), (31, 127, 0, 16, ""), (161, 300, 1, 16, "overflow"),
    (128, 256, 0, 0, "nan"), (95, 160, 1, 0, "nan")])
def test_short_k(monkeypatch, M, N, K, CL, tb, pad, special):
    rng = np.random.default_rng(1000 * K + CL + M)
    A = oracle.fp8_quantize(rng.standard_normal((M, K)).astype(np.float32))
    B = oracle.fp8_quantize(rng.standard_normal((N, K) if tb else (K, N)).astype(np.float32))
    Bn = B if tb else B.T                      # rows are the outputs' columns
    if special == "overflow":
        # one block's sums leave FP16's range
        A[70, :] = 0x7A
        Bn[40, :] = 0x7A
    elif special == "nan":
        A[3, K - 1] = 0x7C                     # +Inf
        Bn[N - 1, K // 2] = 0x7D               # NaN
    lda = K + pad
    ldb = (K if tb else N) + pad
    Ap = np.full((M, lda), 0x7D, np.uint8)     # padding that must not be used
    Bp = np.full((B.shape[0], ldb), 0x7D, np.uint8)
    Ap[:, :K] = A
    Bp[:, :B.shape[1]] = B
    Ad, Bd = dev(Ap), dev(Bp)
    got = {}
    for tile, wgs in (("2", "0"), ("5", "0"), ("5", "2")):     # wgs 2: the kernel for any K
        monkeypatch.setenv("FP8T_MFMA_TILE", tile)
        monkeypatch.setenv("FP8T_GEMM_WGS", wgs)
        for guard in ("1", "0"):
            monkeypatch.setenv("FP8T_GEMM_GUARD", guard)
            say(f"short K tile={tile} wgs={wgs} guard={guard} tb={tb} {M}x{N}x{K} CL={CL} pad={pad}")
            got[tile, wgs, guard] = host(gemm(Ad, Bd, M, N, K, CL, 0, tb, mode=fp8t.FAST, lda=lda,
                                              ldb=ldb))
    ref = got["2", "0", "1"]
    for key, C in got.items():
        assert np.array_equal(C, ref), (key, np.argwhere(C != ref)[:5])
    # the FP8 result of the same pass, rows padded, with and without C
    monkeypatch.setenv("FP8T_MFMA_TILE", "5")
    monkeypatch.setenv("FP8T_GEMM_WGS", "0")
    monkeypatch.setenv("FP8T_GEMM_GUARD", "1")
    for with_c in (True, False):
        C8 = torch.full((M, N + 3), 0xEE, dtype=torch.uint8, device=DEV)
        C = torch.empty((M, N), dtype=torch.uint16, device=DEV) if with_c else None
        nb = fp8t.chunk_gemm_fp8_workspace_size(0, tb, M, N, K, CL, fp8t.FAST)
        ws = torch.empty(max(nb, 1), dtype=torch.uint8, device=DEV)
        fp8t.chunk_gemm_fp8(0, tb, M, N, K, CL, Ad, lda, Bd, ldb, C, N, C8, N + 3, 0.5, fp8t.FAST,
                            ws, nb)
        q8 = host(C8)
        assert np.all(q8[:, N:] == 0xEE)
        assert np.array_equal(q8[:, :N], oracle.fp8_quantize(ref, 0.5))
        if with_c:
            assert np.array_equal(host(C), ref)


@pytest.mark.parametrize("K", [64, 128, 192, 256])
def test_short_k_64_row_tiles(monkeypatch, K):
    # 3250 tiles of 64 x 128: enough for the 64-row tiles (12 per CU of 256);
    # ragged in both directions, one block that overflows and a NaN
    M, N, CL = 16 * 64 * 4 + 40, 6400 - 10, 64
    gen = torch.Generator(device=DEV).manual_seed(K)
    A, B = (torch.randn(s, generator=gen, device=DEV) for s in ((M, K), (N, K)))
    A[70, :], B[40, :] = 49152.0, 49152.0
    Ad, Bd = (torch.empty(x.shape, dtype=torch.uint8, device=DEV) for x in (A, B))
    fp8t.fp8_quantize(A, Ad)
    fp8t.fp8_quantize(B, Bd)
    Bd[N - 1, K // 2] = 0x7D
    got = []
    for tile in ("2", "5"):
        monkeypatch.setenv("FP8T_MFMA_TILE", tile)
        say(f"short K, 64-row tiles: tile={tile} {M}x{N}x{K}")
        got.append(host(gemm(Ad, Bd, M, N, K, CL, 0, 1, mode=fp8t.FAST)))
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("K,CL,tb", [(64, 64, 1), (128, 64, 0), (128, 128, 1), (192, 64, 1),
                                     (192, 192, 0), (256, 64, 1), (256, 128, 0), (256, 256, 1)])
def test_short_k_64_row_tiles_aligned_results(monkeypatch, K, CL, tb):
    """Rows of results that allow the 16-byte stores of C and the 8-byte ones
    of C8, on the 64-row tiles: chunks of one and of several slabs, both
    layouts of B, both epilogues, blocks that overflow and hold Inf and NaN;
    against the streamed kernel everywhere and the fast mode's bounds on
    sampled rows and columns."""
    M, N = 16 * 64 * 4 + 40, 6400
    gen = torch.Generator(device=DEV).manual_seed(7 * K + CL)
    A = torch.randn((M, K), generator=gen, device=DEV)
    B = torch.randn((N, K) if tb else (K, N), generator=gen, device=DEV)
    Bn = B if tb else B.T                      # rows are the outputs' columns
    A[70, :], Bn[40, :] = 49152.0, 49152.0
    Ad, Bd = (torch.empty(x.shape, dtype=torch.uint8, device=DEV) for x in (A, B))
    fp8t.fp8_quantize(A, Ad)
    fp8t.fp8_quantize(B.contiguous(), Bd)
    Ad[M - 1, 3] = 0x7C                        # +Inf
    (Bd if tb else Bd.T)[N - 1, K // 2] = 0x7D    # NaN
    got = {}
    for tile, guard in (("2", "1"), ("5", "1"), ("5", "0")):
        monkeypatch.setenv("FP8T_MFMA_TILE", tile)
        monkeypatch.setenv("FP8T_GEMM_GUARD", guard)
        say(f"short K, 64-row tiles, aligned: tile={tile} guard={guard} tb={tb} {M}x{N}x{K} CL={CL}")
        got[tile, guard] = host(gemm(Ad, Bd, M, N, K, CL, 0, tb, mode=fp8t.FAST))
    ref = got["2", "1"]
    for key, C in got.items():
        assert np.array_equal(C, ref), (key, np.argwhere(C != ref)[:5])
    monkeypatch.setenv("FP8T_GEMM_GUARD", "1")
    for with_c in (True, False):
        C8 = torch.full((M, N), 0xEE, dtype=torch.uint8, device=DEV)
        C = torch.empty((M, N), dtype=torch.uint16, device=DEV) if with_c else None
        nb = fp8t.chunk_gemm_fp8_workspace_size(0, tb, M, N, K, CL, fp8t.FAST)
        ws = torch.empty(max(nb, 1), dtype=torch.uint8, device=DEV)
        fp8t.chunk_gemm_fp8(0, tb, M, N, K, CL, Ad, K, Bd, Bd.shape[1], C, N, C8, N, 0.5,
                            fp8t.FAST, ws, nb)
        assert np.array_equal(host(C8), oracle.fp8_quantize(ref, 0.5))
        if with_c:
            assert np.array_equal(host(C), ref)
    # rows of both 32-row halves of tiles, the last tile, the planted ones
    rows = np.array([0, 31, 32, 63, 64, 70, 2047, M - 41, M - 40, M - 2, M - 1])
    cols = np.array([0, 31, 32, 40, 127, 128, 3333, N - 33, N - 2, N - 1])
    Ah = host(Ad)[rows]
    Bh = host(Bd)[cols] if tb else np.ascontiguousarray(host(Bd)[:, cols])
    check_fast(ref[np.ix_(rows, cols)], Ah, Bh, CL, 0, tb, f"short K {K} CL={CL}")


@pytest.mark.parametrize("M,N,tb", [(33, 128, 1), (95, 264, 0)])
@pytest.mark.parametrize("K,CL", [(64, 64), (192, 64), (256, 128)])
def test_short_k_32_row_tiles_aligned_fp8_result(monkeypatch, M, N, tb, K, CL):
    """The 8-byte stores of C8 (rows a multiple of 8 bytes apart) on the 32-row
    tiles, and the result against the fast mode's bounds."""
    monkeypatch.setenv("FP8T_MFMA_TILE", "5")
    rng = np.random.default_rng(2000 * K + CL + M)
    A = oracle.fp8_quantize(rng.standard_normal((M, K)).astype(np.float32))
    B = oracle.fp8_quantize(rng.standard_normal((N, K) if tb else (K, N)).astype(np.float32))
    Ad, Bd = dev(A), dev(B)
    ldc8 = N + 8
    C8 = torch.full((M, ldc8), 0xEE, dtype=torch.uint8, device=DEV)
    C = torch.empty((M, N), dtype=torch.uint16, device=DEV)
    nb = fp8t.chunk_gemm_fp8_workspace_size(0, tb, M, N, K, CL, fp8t.FAST)
    ws = torch.empty(max(nb, 1), dtype=torch.uint8, device=DEV)
    say(f"short K, aligned C8: tb={tb} {M}x{N}x{K} CL={CL}")
    fp8t.chunk_gemm_fp8(0, tb, M, N, K, CL, Ad, K, Bd, B.shape[1], C, N, C8, ldc8, 0.5, fp8t.FAST,
                        ws, nb)
    ref, q8 = host(C), host(C8)
    check_fast(ref, A, B, CL, 0, tb, f"short K {M}x{N}x{K} CL={CL}")
    assert np.all(q8[:, N:] == 0xEE)
    assert np.array_equal(q8[:, :N], oracle.fp8_quantize(ref, 0.5))
