"""Host threads that share one stream, and so its workspace, while one of them
makes it grow.  Integer inputs make every sum exact, so each result must equal
the oracle bit for bit."""
import threading

import numpy as np
import pytest
import torch

import oracle
from paper_1905_03136_amd import api, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_threads_on_one_stream():
    cases = []
    for K, M, N in [(10007, 4, 4), (9001, 8, 8), (200000, 8, 8), (70001, 24, 20)]:
        A = inputs.host_integers(K, M, 98, inputs.STREAM_A)
        B = inputs.host_integers(K, N, 98, inputs.STREAM_B)
        cases.append((torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV), oracle.tsmttsm(A, B)))
    ones = torch.ones(300000, 64, dtype=torch.float64, device=DEV)
    torch.cuda.synchronize()
    for turn in range(6):
        print("shared stream, turn %d" % turn, flush=True)
        s = torch.cuda.Stream()  # a new stream's workspace starts small
        got, fail = [], []

        def work(i):
            try:
                with torch.cuda.stream(s):
                    for n in range(12):
                        if i == 0:  # rows for a larger workspace each time
                            K = 25000 * (n + 1)
                            got.append((api.tsmttsm(ones[:K], ones[:K]), np.full((64, 64), float(K))))
                        else:
                            A, B, ref = cases[(i + n) % 4]
                            got.append((api.tsmttsm(A, B), ref))
            except Exception as e:  # noqa: BLE001
                fail.append(e)

        threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        s.synchronize()
        assert not fail, fail
        assert len(got) == 48
        for C, ref in got:
            assert np.array_equal(C.cpu().numpy(), ref)
