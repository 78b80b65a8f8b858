"""GPU parity of the chunk-per-wave exact kernel (configurations 12-17: 4 x 4
and 2 x 2 outputs per lane, 4, 8 or 16 waves): chunk counts that do and do not
fill a round of waves, chunk lengths that are not whole operand slabs, ragged
edges, shared tiles, unaligned operands and pieces that fail the guard."""
import numpy as np
import pytest
import torch

import oracle
import paper_1812_08011_amd as fp8t
from .gpu_util import DEV, dev, gemm, host, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fp8t.lib()
    yield


TILES = ["12", "13", "14", "15", "16", "17"]
SHAPES = [
    # M, N, K, CL
    (130, 67, 333, 64),       # ragged everywhere, last chunk 13
    (16, 17, 70, 32),         # the smallest sizes it takes, last chunk 6
    (33, 40, 1030, 100),      # chunks of 6.25 slabs
    (64, 96, 2240, 64),       # 35 chunks: rounds of 16 and 3
    (45, 31, 700, 33),        # odd chunk length: unaligned chunk starts
    (32, 32, 65, 64),         # a last chunk of one product
]


def operands(rng, M, N, K, ta, tb):
    a = rng.standard_normal((M, K)).astype(np.float32)
    b = rng.standard_normal((K, N)).astype(np.float32)
    a[rng.random(a.shape) < 0.05] = 0.0
    b[rng.random(b.shape) < 0.02] *= 64.0
    return (oracle.fp8_quantize(np.ascontiguousarray(a.T if ta else a)),
            oracle.fp8_quantize(np.ascontiguousarray(b.T if tb else b)))


@pytest.mark.parametrize("plan", ["whole", "3", "7"])
@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_chunk_per_wave_matches_oracle(tile, ta, tb, plan, monkeypatch):
    monkeypatch.setenv("FP8T_VALU_TILE", tile)
    monkeypatch.setenv("FP8T_GEMM_SPLIT", "0" if plan == "whole" else "1")
    if plan != "whole":
        monkeypatch.setenv("FP8T_GEMM_WGS", plan)
    rng = np.random.default_rng(900 + 2 * ta + tb)
    for (M, N, K, CL) in SHAPES:
        A, B = operands(rng, M, N, K, ta, tb)
        say(f"chunk per wave tile={tile} plan={plan} ta={ta} tb={tb} {M}x{N}x{K} CL={CL}")
        got = host(gemm(dev(A), dev(B), M, N, K, CL, ta, tb))
        ref = oracle.chunk_gemm(A, B, CL, ta, tb)
        assert np.array_equal(got, ref), (M, N, K, CL, np.argwhere(got != ref)[:5])


@pytest.mark.parametrize("guard", ["1", "0"])
@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("wgs", ["0", "5"])
def test_chunk_per_wave_specials(tile, guard, wgs, monkeypatch):
    """Inf and NaN operands, sums that overflow FP16 on the way, subnormal and
    zero rows, some in tiles next to ordinary ones: both paths, whole and
    shared tiles, with the FP8 result."""
    monkeypatch.setenv("FP8T_VALU_TILE", tile)
    monkeypatch.setenv("FP8T_GEMM_GUARD", guard)
    if wgs != "0":
        monkeypatch.setenv("FP8T_GEMM_SPLIT", "1")
        monkeypatch.setenv("FP8T_GEMM_WGS", wgs)
    rng = np.random.default_rng(951)
    M, N, K, CL = 70, 50, 640, 64
    A, B = operands(rng, M, N, K, 0, 0)
    A[3, :] = 0x7B                       # 57344: overflows part-way
    A[7, 5] = 0x7C
    A[9, 600] = 0x7F
    A[40, :] = 0x01                      # 2^-16
    A[41, :] = 0x80                      # -0
    B[:, 11] = 0x01
    Ad, Bd = dev(A), dev(B)
    ref = oracle.chunk_gemm(A, B, CL)
    say(f"chunk per wave specials tile={tile} guard={guard} wgs={wgs}")
    assert np.array_equal(host(gemm(Ad, Bd, M, N, K, CL)), ref)
    for with_c in (True, False):
        wb = fp8t.chunk_gemm_fp8_workspace_size(0, 0, M, N, K, CL, fp8t.EXACT)
        ws = torch.empty(wb, dtype=torch.uint8, device=DEV) if wb else None
        C = torch.zeros((M, N), dtype=torch.uint16, device=DEV) if with_c else None
        C8 = torch.zeros((M, N), dtype=torch.uint8, device=DEV)
        fp8t.chunk_gemm_fp8(0, 0, M, N, K, CL, Ad, K, Bd, N, C, N, C8, N, 0.25, fp8t.EXACT, ws, wb)
        assert np.array_equal(host(C8), oracle.fp8_quantize(ref, 0.25))
        if with_c:
            assert np.array_equal(host(C), ref)


@pytest.mark.parametrize("tile", ["12", "14", "16"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_chunk_per_wave_unaligned_operands(tile, ta, tb, monkeypatch):
    """Operands at odd addresses with odd leading dimensions, results too."""
    monkeypatch.setenv("FP8T_VALU_TILE", tile)
    rng = np.random.default_rng(970)
    M, N, K, CL = 67, 35, 391, 64
    A, B = operands(rng, M, N, K, ta, tb)
    lda, ldb, ldc = A.shape[1] + 3, B.shape[1] + 5, N + 1
    Ap = np.full(1 + A.shape[0] * lda, 0x7F, np.uint8)       # padding is NaN
    Bp = np.full(3 + B.shape[0] * ldb, 0x7F, np.uint8)
    Ap[1:].reshape(A.shape[0], lda)[:, :A.shape[1]] = A
    Bp[3:].reshape(B.shape[0], ldb)[:, :B.shape[1]] = B
    Ad, Bd = dev(Ap), dev(Bp)
    C = torch.zeros((M, ldc), dtype=torch.uint16, device=DEV)
    say(f"chunk per wave unaligned tile={tile} ta={ta} tb={tb}")
    fp8t.chunk_gemm(ta, tb, M, N, K, CL, Ad[1:], lda, Bd[3:], ldb, C, ldc, fp8t.EXACT)
    got = host(C)
    assert np.array_equal(got[:, :N], oracle.chunk_gemm(A, B, CL, ta, tb))
    assert not got[:, N:].any()
