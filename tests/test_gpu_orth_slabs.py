"""Slab counts of the batched orthogonalisation around its groups of sixteen
and beyond sixteen groups, batches of the automatic slab size, and workspaces
that hold fewer slabs than a batch would have.  Integer inputs make C = V^T W
and W - V C exact."""
import numpy as np
import pytest
import torch

from paper_1905_03136_amd import _lib, api, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def instances(shapes, seed):
    out = []
    for i, (K, M, N) in enumerate(shapes):
        V = inputs.host_integers(K, M, seed, 10 + 2 * i, False, -3, 3)
        W = inputs.host_integers(K, N, seed, 11 + 2 * i, False, -3, 3)
        out.append((V, W))
    return out


def check(host, pairs, C):
    for (V, W), (_, dW), dC in zip(host, pairs, C):
        ref = V.T @ W if len(V) else np.zeros((V.shape[1], W.shape[1]))
        assert np.array_equal(dC.cpu().numpy(), ref)
        assert np.array_equal(dW.cpu().numpy(), W - V @ ref)


def on_device(host):
    return [(torch.from_numpy(V).to(DEV), torch.from_numpy(W).to(DEV)) for V, W in host]


@pytest.mark.parametrize("slabs", [1, 15, 16, 17, 255, 256, 257, 600])
def test_slab_counts(slabs):
    print("orth slabs %d" % slabs, flush=True)
    host = instances([(16 * slabs - 3, 33, 16), (16 * slabs, 5, 3), (0, 2, 2), (1, 64, 1)], 51)
    plan = api.OrthPlan(on_device(host), rows_per_item=16)
    try:
        for how in (plan.launch, plan.run):
            for (_, W), (_, dW) in zip(host, plan.pairs):
                dW.copy_(torch.from_numpy(W))
            how()
            plan.check()
            check(host, plan.pairs, plan.C)
    finally:
        plan.close()


@pytest.mark.parametrize("count,K,M,N", [(1, 300001, 17, 5), (40, 1203, 9, 16), (3, 40000, 64, 16)])
def test_automatic_slabs_and_small_workspaces(count, K, M, N):
    print("orth auto %d x %d" % (count, K), flush=True)
    host = instances([(K + 7 * i, M, N) for i in range(count)], 52)
    pairs = on_device(host)
    batch = api.OrthBatch(pairs)
    full = batch.workspace
    # queue room, and partial sums for the automatic slabs or for fewer larger ones
    queue = _lib.tsg_workspace_size(_lib.TSG_KIND_ORTH, _lib.TSG_R64, 1, 1, 1, count) - 8 * (544 + 2 * count)
    for doubles in (None, 600 * M * N, (count + 16) * M * N):
        ws = full if doubles is None else full[:min(full.numel(), queue + 8 * doubles)]
        batch.workspace = ws
        for (_, W), (_, dW) in zip(host, pairs):
            dW.copy_(torch.from_numpy(W))
        batch.run()
        batch.check()
        check(host, pairs, batch.C)
