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
