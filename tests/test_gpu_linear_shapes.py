"""GPU parity of the dense calls at the sizes where they take other kernels, against float64 on the same bf16 operands."""
import ctypes as C

import numpy as np
import pytest

import oracle
from gpu_util import assert_close, bf16_tensor_to_float
from paper_2504_18082_amd import synth
from test_gpu_linear import hdr_for, to_bf16_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_mod():
    import torch
    assert torch.cuda.is_available()
    return torch


# capacities from 16384 rows on: the weight gradient in two halves per workgroup (one step, an odd number of steps, a last split
# with a single row, every split full), the input gradient by the kernels for many rows (N = 256: streaming and wide)
@pytest.mark.parametrize("M,F_in,F_out,n_op", [(1, 128, 256, 2), (33, 100, 64, 2), (97, 64, 128, 1), (16384, 128, 256, 2), (16417, 256, 192, 1),
                                               (24_577, 602, 256, 1), (20_001, 128, 320, 2), (66_000, 128, 256, 2)])
def test_many_rows(torch_mod, M, F_in, F_out, n_op):
    torch = torch_mod
    from paper_2504_18082_amd import binding as B
    print(f"case many rows M={M} F_in={F_in} F_out={F_out} operands={n_op}", flush=True)
    rng = np.random.default_rng(M + F_in)
    cap = max(16384, M + 9)
    W = (rng.standard_normal((n_op * F_in, F_out)) / np.sqrt(n_op * F_in)).astype(np.float32)
    layer = B.SageLayer(W, np.zeros(F_out, np.float32), n_operands=n_op)
    layer.refresh()
    x = [rng.standard_normal((M, F_in)).astype(np.float32) for _ in range(n_op)]
    dz = (rng.standard_normal((M, F_out)) / 64).astype(np.float32)
    pad = lambda a: np.pad(a, ((0, cap - M), (0, 0)), constant_values=3.0)      # junk rows past the live count
    dev = [to_bf16_dev(torch, pad(a), layer.F_pad) for a in x]
    d_dz = to_bf16_dev(torch, pad(dz), layer.N_pad)
    hdr = hdr_for(torch, M)
    h_self, agg = (dev[0], dev[1]) if n_op == 2 else (None, dev[0])
    out_b = torch.full((cap, layer.N_pad), 0x7FC0, dtype=torch.int16, device="cuda")
    B.cr_sage_linear_fwd(layer, C.c_void_p(hdr.data_ptr()), cap, h_self, agg, layer.F_pad, True, None, out_b)
    ws = torch.empty(B.cr_sage_linear_bwd_workspace_bytes(F_in, F_out, cap), dtype=torch.uint8, device="cuda")
    dW = torch.zeros((n_op * F_in, F_out), dtype=torch.float32, device="cuda")
    db = torch.zeros(F_out, dtype=torch.float32, device="cuda")
    want_input = (n_op * layer.F_pad) % 64 == 0
    d_in = torch.full((cap, n_op * layer.F_pad), 0x7FC0, dtype=torch.int16, device="cuda") if want_input else None
    B.cr_sage_linear_bwd(layer, C.c_void_p(hdr.data_ptr()), cap, h_self, agg, layer.F_pad, d_dz, 0.0, 0.0, None, None, ws, dW, db, d_in_bf16=d_in)
    torch.cuda.synchronize()
    bf = lambda a: torch.from_numpy(oracle.round_bf16(a)).cuda().double()
    X, Z, Wb = torch.cat([bf(a) for a in x], 1), bf(dz), bf(W)
    # float sums of M terms of size ~1/64: 2^-24 sqrt(M) of the terms' magnitude, an order of magnitude in hand
    assert_close(dW.cpu().numpy(), (X.t() @ Z).cpu().numpy(), 1e-5, "dW", scale=np.sqrt(M) / 64)
    assert_close(db.cpu().numpy(), Z.sum(0).cpu().numpy(), 1e-5, "db", scale=np.sqrt(M) / 64)
    # one rounding to bf16 (2^-8 relative) of a float sum
    assert_close(bf16_tensor_to_float(out_b)[:M, :F_out], (X @ Wb).clamp_min(0).cpu().numpy(), 2.0 ** -8, "out", scale=1e-4)
    assert np.all(out_b.cpu().numpy()[M:].view(np.uint16) == 0x7FC0)
    if want_input:
        got, want = bf16_tensor_to_float(d_in)[:M], (Z @ Wb.t()).cpu().numpy()
        for part in range(n_op):
            cols = slice(part * layer.F_pad, part * layer.F_pad + F_in)
            assert_close(got[:, cols], want[:, part * F_in:(part + 1) * F_in], 2.0 ** -8, "d_in", scale=1e-4)
        assert np.all(d_in.cpu().numpy()[M:].view(np.uint16) == 0x7FC0)



# rows that are not finite through the kernels for many rows, N = 256: forward and input gradient, streaming (K = 256) and wide
# (K = 320).  What the sums make of them comes out -- NaN stays NaN, with ReLU too, as it does below 16384 rows and in the oracle
@pytest.mark.parametrize("F_in,F_out,cap", [(128, 256, 16384), (128, 320, 16384), (160, 256, 16384), (128, 256, 4096)])
def test_rows_that_are_not_finite(torch_mod, F_in, F_out, cap):
    torch = torch_mod
    from paper_2504_18082_amd import binding as B
    M = cap - 7
    print(f"case not finite F_in={F_in} F_out={F_out} capacity={cap}", flush=True)
    rng = np.random.default_rng(F_out)

    def spoiled(cols):
        x = rng.standard_normal((M, cols)).astype(np.float32)
        for r in (0, 5, M - 1):
            x[r, r % cols] = np.nan
        x[17, 3], x[18, 3], x[19, 3], x[19, 4] = np.inf, -np.inf, np.inf, -np.inf
        return x

    W = np.abs(rng.standard_normal((2 * F_in, F_out)) / 16).astype(np.float32)       # (of one sign: row 19 meets inf and -inf)

    def new_layer():                    # (a step on these gradients leaves NaN in the weights)
        layer = B.SageLayer(W, np.zeros(F_out, np.float32))
        layer.refresh()
        return layer

    layer = new_layer()
    hdr = hdr_for(torch, M)
    pad = lambda a: np.pad(a, ((0, cap - M), (0, 0)))
    dz = spoiled(F_out)
    d_dz = to_bf16_dev(torch, pad(dz), layer.N_pad)
    clean = to_bf16_dev(torch, np.zeros((cap, F_in), np.float32), layer.F_pad)
    ws = torch.empty(B.cr_sage_linear_bwd_workspace_bytes(F_in, F_out, cap), dtype=torch.uint8, device="cuda")
    dW, db = torch.zeros((2 * F_in, F_out), device="cuda"), torch.zeros(F_out, device="cuda")
    d_in = [torch.zeros((cap, 2 * layer.F_pad), dtype=torch.int16, device="cuda") for _ in range(2)]
    B.cr_sage_linear_bwd(layer, C.c_void_p(hdr.data_ptr()), cap, clean, clean, layer.F_pad, d_dz, 0.0, 0.0, None, None, ws, dW, db, d_in_bf16=d_in[0])
    layer = new_layer()
    B.cr_sage_linear_bwd_input(layer, C.c_void_p(hdr.data_ptr()), cap, d_dz, None, None, d_in_bf16=d_in[1])
    bf = lambda a: torch.from_numpy(oracle.round_bf16(a)).double()
    Wb = bf(W)

    def same(got, want, what):
        assert np.array_equal(np.isnan(got), np.isnan(want)), f"{what}: NaN in other places"
        assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)]), f"{what}: infinities"
        fin = np.isfinite(want)
        assert_close(got[fin], want[fin], 2.0 ** -8, what, scale=1e-2)       # one rounding to bf16 of a float sum of ~13 in magnitude

    want = (bf(dz) @ Wb.t()).numpy()
    for t in d_in:
        same(bf16_tensor_to_float(t)[:M], want, "d_in")
    x = spoiled(2 * F_in)
    hs, ag = to_bf16_dev(torch, pad(x[:, :F_in]), layer.F_pad), to_bf16_dev(torch, pad(x[:, F_in:]), layer.F_pad)
    want = (bf(x) @ Wb).numpy()
    for relu in (False, True):
        out = torch.zeros((cap, layer.N_pad), dtype=torch.int16, device="cuda")
        B.cr_sage_linear_fwd(layer, C.c_void_p(hdr.data_ptr()), cap, hs, ag, layer.F_pad, relu, None, out)
        same(bf16_tensor_to_float(out)[:M, :F_out], np.where(want < 0, 0.0, want) if relu else want, f"out relu={relu}")


def launches(torch, call):
    """Number of kernels a call launches (nodes of its captured graph)."""
    from paper_2504_18082_amd import binding as B
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    n = C.c_size_t(0)
    assert B.lib().hipGraphGetNodes(C.c_void_p(graph.raw_cuda_graph()), None, C.byref(n)) == 0
    return n.value


# the weight gradient and the input gradient go side by side in one launch at every number of rows (two launches are slower up to
# 131072 rows, by half at 16384), the reduction of the weight gradient's partial sums is the other
@pytest.mark.parametrize("cap,F_out,n_op", [(4096, 256, 2), (16384, 256, 2), (16384, 256, 1), (66_000, 320, 2)])
def test_backward_products_share_a_launch(torch_mod, cap, F_out, n_op):
    torch = torch_mod
    from paper_2504_18082_amd import binding as B
    print(f"case shared launch, capacity {cap}", flush=True)
    layer = B.SageLayer(np.zeros((n_op * 128, F_out), np.float32), np.zeros(F_out, np.float32), n_operands=n_op)
    layer.refresh()
    rows = lambda cols: torch.zeros((cap, cols), dtype=torch.int16, device="cuda")
    hdr, x, dz, d_in = hdr_for(torch, cap - 5), rows(128), rows(layer.N_pad), rows(n_op * 128)
    ws = torch.empty(B.cr_sage_linear_bwd_workspace_bytes(128, F_out, cap), dtype=torch.uint8, device="cuda")
    dW, db = torch.zeros((n_op * 128, F_out), device="cuda"), torch.zeros(F_out, device="cuda")
    for out in (d_in, None):
        call = lambda: B.cr_sage_linear_bwd(layer, C.c_void_p(hdr.data_ptr()), cap, x if n_op == 2 else None, x, 128, dz, 0.0, 0.0, None, None, ws,
                                            dW, db, d_in_bf16=out)
        call()                                   # (the kernels are loaded by now)
        torch.cuda.synchronize()
        assert launches(torch, call) == 2
