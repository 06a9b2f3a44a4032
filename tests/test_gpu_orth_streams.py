"""Batches on several streams at once, whose blocks share the compute units:
no launch holds all of its blocks from the start.  Integer inputs make
C = V^T W and W - V C exact."""
import numpy as np
import pytest
import torch

from paper_1905_03136_amd import api, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("graph", [True, False])
def test_batches_side_by_side(graph):
    host = []
    for i in range(24):
        K, M, N = 6000 + 977 * i, (5, 17, 33, 64)[i % 4], (1, 4, 16)[i % 3]
        host.append((inputs.host_integers(K, M, 53, 10 + 2 * i, False, -3, 3),
                     inputs.host_integers(K, N, 53, 11 + 2 * i, False, -3, 3)))
    ref = [V.T @ W for V, W in host]
    streams = [torch.cuda.Stream() for _ in range(3)]
    plans = []
    try:
        for _ in streams:
            plans.append(api.OrthPlan([(torch.from_numpy(V).to(DEV), torch.from_numpy(W).to(DEV)) for V, W in host]))
        fresh = [torch.from_numpy(W).to(DEV) for _, W in host]
        for turn in range(8):
            print("orth side by side, graph %s, turn %d" % (graph, turn), flush=True)
            torch.cuda.synchronize()
            for s, plan in zip(streams, plans):
                with torch.cuda.stream(s):
                    for (_, dW), W in zip(plan.pairs, fresh):
                        dW.copy_(W)
            for s, plan in zip(streams, plans):
                with torch.cuda.stream(s):
                    plan.launch() if graph else plan.run()
            for plan in plans:
                plan.check()
                for (V, W), C, (_, dW), dC in zip(host, ref, plan.pairs, plan.C):
                    assert np.array_equal(dC.cpu().numpy(), C)
                    assert np.array_equal(dW.cpu().numpy(), W - V @ C)
    finally:
        for plan in plans:
            plan.close()
