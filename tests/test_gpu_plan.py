"""The planner: queries from several threads, and the kernel families that
calls of few or short chunks are given."""
import threading

import pytest
import torch

import paper_1812_08011_amd as fp8t
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fp8t.lib()
    yield


def test_queries_from_several_threads():
    """Every thread's first queries fill the table of resident workgroups
    together; all get the answers of one thread."""
    def query():
        return [fp8t.chunk_gemm_workspace_size(ta, tb, m, 384, k, cl, mode)
                for ta in (0, 1) for tb in (0, 1) for m in (100, 2304) for k in (700, 9000)
                for cl in (8, 64) for mode in (fp8t.EXACT, fp8t.FAST)] + \
               [fp8t.chunk_gemm_p16_workspace_size(ta, tb, 300, 384, 900, 64)
                for ta in (0, 1) for tb in (0, 1)] + \
               [fp8t.chunk_gemm_sr_workspace_size(ta, 0, 300, 384, 900, 64) for ta in (0, 1)]
    got = [None] * 8

    def work(i):
        got[i] = query()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(8)]
    say("plan queries from 8 threads")
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    ref = query()
    assert all(g == ref for g in got)


def chosen(capfd, kind, what):
    lines = [l for l in capfd.readouterr().err.splitlines() if f"] chose kind {kind} " in l]
    assert lines, what
    f = lines[-1].split()
    return int(f[f.index("cfg") + 1]), int(f[f.index("L") + 1])


# Plans that had become slower than others (times with both, microseconds).
@pytest.mark.parametrize("ta,tb,M,N,K,CL,slow", [
    (0, 1, 21, 3241, 947, 4, (5, True)),       # 53 against 30 on the chain kernel
    (1, 0, 960, 104, 7226, 4, (8, True)),      # 249 / 145
    (1, 1, 28688, 32, 720, 4, (5, False)),     # 131 / 68
    (0, 1, 3392, 416, 1216, 16, (5, False)),   # 230 / 126
    (0, 1, 29601, 35, 14, 128, (11, False)),   # 19.0 / 8.9
])
def test_short_chunks_and_short_sums(ta, tb, M, N, K, CL, slow, monkeypatch, capfd):
    monkeypatch.setenv("FP8T_GEMM_VERBOSE", "1")
    fp8t.chunk_gemm_workspace_size(ta, tb, M, N, K, CL, fp8t.EXACT)
    cfg, L = chosen(capfd, 0, (M, N, K, CL))
    say(f"plan {M}x{N}x{K} CL={CL}: cfg {cfg} L {L}")
    assert (cfg, L > 0) != slow


@pytest.mark.parametrize("ta,tb,M,N,K,CL,slow", [
    (0, 0, 150, 1938, 1079, 256, 13),          # 118 against 58 (5 chunks for 8 waves)
    (0, 1, 3385, 1203, 10, 8, 5),              # 35 / 26 on the 64 x 64 tile
    (0, 0, 704, 5952, 16, 48, 5),              # 36 / 23
])
def test_fp16_operands_few_and_short_chunks(ta, tb, M, N, K, CL, slow, monkeypatch, capfd):
    monkeypatch.setenv("FP8T_GEMM_VERBOSE", "1")
    fp8t.chunk_gemm_p16_workspace_size(ta, tb, M, N, K, CL)
    cfg, L = chosen(capfd, 3, (M, N, K, CL))
    say(f"plan p16 {M}x{N}x{K} CL={CL}: cfg {cfg} L {L}")
    assert cfg != slow
