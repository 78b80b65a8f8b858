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
