"""GPU parity of cr_sample_blocks, bit for bit, at the sizes where its kernels take other shapes."""
import numpy as np
import pytest

import oracle
from test_gpu_sampling import DeviceGraph, compare, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_mod():
    import torch
    assert torch.cuda.is_available()
    return torch


def mixed_graph(n):
    """Node i has i % 37 neighbours, every 50th node 300: empty rows, rows that share a pass, rows longer than a pass."""
    rng = np.random.default_rng(n)
    rows = [np.sort(rng.permutation(n)[:300 if i % 50 == 0 else i % 37]).astype(np.int32) for i in range(n)]
    indptr = np.zeros(n + 1, dtype=np.int64)
    indptr[1:] = np.cumsum([len(r) for r in rows])
    return indptr, np.concatenate(rows), (np.arange(n) // (n // 8 + 1)).astype(np.int32)


# a wave takes 2, 8, 16 or 32 destination rows, by the number of rows in the group
@pytest.mark.parametrize("batch_size,n_batches", [(33, 1), (400, 9), (500, 40)])
@pytest.mark.parametrize("p", [0.5, 0.9, 1.0])
def test_rows_per_wave(torch_mod, batch_size, n_batches, p):
    graph = mixed_graph(24_000)
    dg = DeviceGraph(torch_mod, graph, 8, edge_classes=True)
    roots = np.random.default_rng(1).permutation(24_000).astype(np.int32)[:batch_size * n_batches - 5]
    print(f"case rows per wave: {n_batches} batches of {batch_size}, p={p}", flush=True)
    layers, nb = run_gpu(torch_mod, dg, roots, [4, 7], p, False, 3, 1, 2, batch_size)
    compare(layers, nb, graph, roots, [4, 7], p, False, 3, 1, 2, batch_size, f"rows per wave p={p}")
