"""GPU parity: cr_sample_blocks against the oracle, bit-exact on every array of every block."""
import numpy as np
import pytest

import oracle
from paper_2504_18082_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_mod():
    import torch
    assert torch.cuda.is_available()
    return torch


class DeviceGraph:
    def __init__(self, torch, graph, n_comm, edge_classes=False):
        from paper_2504_18082_amd import binding as B
        indptr, indices, comm = graph
        self.indptr = torch.from_numpy(np.ascontiguousarray(indptr, dtype=np.int64)).cuda()
        self.indices = torch.from_numpy(np.ascontiguousarray(indices, dtype=np.int32)).cuda()
        self.comm = torch.from_numpy(np.ascontiguousarray(comm, dtype=np.int32)).cuda()
        self.c = B.make_graph(self.indptr, self.indices, self.comm, n_comm)
        self.n_nodes = len(indptr) - 1
        if edge_classes:
            self.bits = B.cr_graph_edge_classes(self.c)
            self.c.edge_intra = self.bits.data_ptr()


def run_gpu(torch, dg, roots, fanouts, p, strict, seed, epoch, first_batch, batch_size, hash_dedup=False, input_global=False,
            exact_ranking=False):
    from paper_2504_18082_amd import binding as B
    n_batches = -(-len(roots) // batch_size)
    flags = (B.CR_SAMPLE_STRICT_INTRA if strict else 0) | (B.CR_SAMPLE_HASH_DEDUP if hash_dedup else 0)
    flags |= B.CR_SAMPLE_INPUT_GLOBAL_IDS if input_global else 0
    flags |= B.CR_SAMPLE_EXACT_RANKING if exact_ranking else 0
    cfg = B.make_sample_cfg(fanouts, p, seed, epoch, first_batch, flags)
    layers = B.alloc_block_sets(cfg, dg.n_nodes, batch_size, n_batches)
    ws = torch.empty(B.cr_sample_blocks_workspace_bytes(cfg, dg.n_nodes, batch_size, n_batches), dtype=torch.uint8, device="cuda")
    d_roots = torch.from_numpy(np.ascontiguousarray(roots, dtype=np.int32)).cuda()
    B.cr_sample_blocks(dg.c, cfg, d_roots, len(roots), batch_size, n_batches, ws, layers)
    torch.cuda.synchronize()
    return layers, n_batches


def compare(layers, n_batches, graph, roots, fanouts, p, strict, seed, epoch, first_batch, batch_size, what, input_global=False):
    pos = np.full(len(graph[0]) - 1, -1, dtype=np.int32)
    host = [dict(hdr=b.hdr.cpu().numpy(), src=b.src_ids.cpu().numpy(), indptr=b.indptr.cpu().numpy(),
                 indices=b.indices.cpu().numpy(),
                 gather_ids=None if b.gather_ids is None else b.gather_ids.cpu().numpy(),
                 t_indptr=None if b.t_indptr is None else b.t_indptr.cpu().numpy(),
                 t_indices=None if b.t_indices is None else b.t_indices.cpu().numpy()) for b in layers]
    for g in range(n_batches):
        want = oracle.sample_blocks(graph, roots[g * batch_size:(g + 1) * batch_size], fanouts, p, strict, seed, epoch,
                                    first_batch + g, pos)
        for l, blk in enumerate(want):
            h = host[l]
            tag = f"{what} batch {g} layer {l}"
            if l == 0 and input_global:
                # input-side block left in global ids: sizes, row pointers, per-edge global ids, destination nodes
                assert h["hdr"][g, :4].tolist() == [blk.n_dst, -1, blk.nnz, 0], tag
                assert np.array_equal(h["src"][g, :blk.n_dst], blk.src_ids[:blk.n_dst]), tag + " src_ids head"
                assert np.array_equal(h["indptr"][g, :blk.n_dst + 1], blk.indptr), tag + " indptr"
                assert np.array_equal(h["gather_ids"][g, :blk.nnz], blk.src_ids[blk.indices]), tag + " gather_ids"
                continue
            assert h["hdr"][g, :4].tolist() == [blk.n_dst, blk.n_src, blk.nnz, 0], tag
            assert np.array_equal(h["src"][g, :blk.n_src], blk.src_ids), tag + " src_ids"
            assert np.array_equal(h["indptr"][g, :blk.n_dst + 1], blk.indptr), tag + " indptr"
            assert np.array_equal(h["indices"][g, :blk.nnz], blk.indices), tag + " indices"
            if h["gather_ids"] is not None:
                assert np.array_equal(h["gather_ids"][g, :blk.nnz], blk.src_ids[blk.indices]), tag + " gather_ids"
            if l >= 1:
                assert np.array_equal(h["t_indptr"][g, :blk.n_src + 1], blk.t_indptr), tag + " t_indptr"
                assert np.array_equal(h["t_indices"][g, :blk.nnz], blk.t_indices), tag + " t_indices"


@pytest.mark.parametrize("p,strict", [(0.5, False), (0.9, False), (1.0, False), (1.0, True), (0.75, False)])
def test_tiny_group_of_batches(torch_mod, tiny_workload, p, strict):
    w = tiny_workload
    dg = DeviceGraph(torch_mod, w.graph, w.cfg.n_comm)
    perm = oracle.build_batches(oracle.COMM_RAND, 6, 0, 2, w.train_ids, w.comm, w.cfg.n_comm)
    roots = perm[:256 * 3 + 100]                      # four batches, the last one short
    print(f"case tiny p={p} strict={strict}", flush=True)
    layers, nb = run_gpu(torch_mod, dg, roots, w.cfg.fanouts, p, strict, 0, 2, 5, 256)
    assert nb == 4
    compare(layers, nb, w.graph, roots, w.cfg.fanouts, p, strict, 0, 2, 5, 256, f"tiny p={p}")


@pytest.mark.parametrize("p,hash_dedup", [(0.5, False), (0.9, False), (1.0, False), (0.5, True), (1.0, True)])
def test_arxiv_three_layers(torch_mod, arxiv_workload, p, hash_dedup):
    # both frontier de-duplication tables: direct-address (the input-side hop at this size; the hops above it go without a table) and
    # open addressing (every hop)
    w = arxiv_workload
    dg = DeviceGraph(torch_mod, w.graph, w.cfg.n_comm)
    perm = oracle.build_batches(oracle.RAND, 1, 3, 1, w.train_ids, w.comm, w.cfg.n_comm)
    roots = perm[:1024 + 1000]
    print(f"case arxiv p={p} hash_dedup={hash_dedup}", flush=True)
    layers, nb = run_gpu(torch_mod, dg, roots, w.cfg.fanouts, p, False, 3, 1, 0, 1024, hash_dedup)
    compare(layers, nb, w.graph, roots, w.cfg.fanouts, p, False, 3, 1, 0, 1024, f"arxiv p={p}")


def test_hub_rows_and_isolated_nodes(torch_mod):
    # a hub with 5000 neighbours in two communities, leaves of degree 1, and isolated nodes
    g = synth.star_graph(3000, 2000)
    indptr = np.concatenate([g[0], [g[0][-1]] * 3])             # three isolated nodes at the end
    comm = np.concatenate([g[2], [0, 1, 1]]).astype(np.int32)
    graph = (indptr, g[1], comm)
    dg = DeviceGraph(torch_mod, graph, 2)
    roots = np.array([0, 5001, 17, 5003, 4000], dtype=np.int32)
    for p, strict in ((0.5, False), (0.9, False), (1.0, False), (1.0, True)):
        for fan in ([3, 64], [64, 7]):
            print(f"case hub p={p} strict={strict} fanouts={fan}", flush=True)
            layers, nb = run_gpu(torch_mod, dg, roots, fan, p, strict, 9, 0, 3, 8, hash_dedup=(fan[0] == 3))
            compare(layers, nb, graph, roots, fan, p, strict, 9, 0, 3, 8, f"hub p={p} {fan}")


def test_single_layer_and_determinism(torch_mod, tiny_workload):
    w = tiny_workload
    dg = DeviceGraph(torch_mod, w.graph, w.cfg.n_comm)
    roots = w.train_ids[:77]
    layers, nb = run_gpu(torch_mod, dg, roots, [7], 0.9, False, 1, 1, 0, 128)
    compare(layers, nb, w.graph, roots, [7], 0.9, False, 1, 1, 0, 128, "single layer")
    a, _ = run_gpu(torch_mod, dg, w.train_ids[:600], [10, 5], 0.9, False, 4, 4, 2, 256)
    b, _ = run_gpu(torch_mod, dg, w.train_ids[:600], [10, 5], 0.9, False, 4, 4, 2, 256)
    # compare the valid parts batch by batch
    for x, y in zip(a, b):
        hdr = x.hdr.cpu().numpy()
        for g in range(3):
            n_dst, n_src, nnz = hdr[g, :3]
            assert np.array_equal(x.src_ids[g, :n_src].cpu().numpy(), y.src_ids[g, :n_src].cpu().numpy())
            assert np.array_equal(x.indices[g, :nnz].cpu().numpy(), y.indices[g, :nnz].cpu().numpy())
            if x.t_indices is not None:
                assert np.array_equal(x.t_indices[g, :nnz].cpu().numpy(), y.t_indices[g, :nnz].cpu().numpy())


@pytest.mark.parametrize("p,hash_dedup", [(0.5, False), (0.9, True)])
def test_input_block_in_global_ids(torch_mod, tiny_workload, p, hash_dedup):
    """CR_SAMPLE_INPUT_GLOBAL_IDS: the layers above are unchanged, the input-side block carries row pointers and
    per-edge global ids only; also with a single layer (the roots' own block is the input-side one)."""
    w = tiny_workload
    dg = DeviceGraph(torch_mod, w.graph, w.cfg.n_comm)
    perm = oracle.build_batches(oracle.RAND, 1, 0, 4, w.train_ids, w.comm, w.cfg.n_comm)
    roots = perm[:256 * 2 + 31]
    for fanouts in (w.cfg.fanouts, [7, 4, 3], [12]):
        print(f"case input-global p={p} fanouts={fanouts}", flush=True)
        layers, nb = run_gpu(torch_mod, dg, roots, fanouts, p, False, 0, 4, 2, 256, hash_dedup, input_global=True)
        compare(layers, nb, w.graph, roots, fanouts, p, False, 0, 4, 2, 256, f"input-global {fanouts}", input_global=True)


def test_edge_class_bits(torch_mod, tiny_workload, arxiv_workload):
    """cr_graph_edge_classes against its definition (bit e = both ends of entry e in one community), and sampling
    with the bits against the oracle: same blocks as without them, for every p and also for long rows."""
    for w in (tiny_workload, arxiv_workload):
        dg = DeviceGraph(torch_mod, w.graph, w.cfg.n_comm, edge_classes=True)
        torch_mod.cuda.synchronize()
        rows = np.repeat(np.arange(w.cfg.n_nodes), np.diff(w.indptr))
        want = (w.comm[rows] == w.comm[w.indices]).astype(np.uint8)
        got = np.unpackbits(dg.bits.cpu().numpy().view(np.uint8), bitorder="little")[:len(want)]
        assert np.array_equal(got, want)
        tail = np.unpackbits(dg.bits.cpu().numpy().view(np.uint8), bitorder="little")[len(want):]
        assert not tail.any()                              # padding bits of the last word are zero
    w = arxiv_workload
    dg = DeviceGraph(torch_mod, w.graph, w.cfg.n_comm, edge_classes=True)
    perm = oracle.build_batches(oracle.COMM_RAND, 60, 0, 1, w.train_ids, w.comm, w.cfg.n_comm)
    roots = perm[:1024 + 77]
    for p, strict in ((0.9, False), (1.0, False), (1.0, True), (0.5, False)):
        print(f"case edge bits p={p} strict={strict}", flush=True)
        layers, nb = run_gpu(torch_mod, dg, roots, w.cfg.fanouts, p, strict, 0, 1, 3, 1024)
        compare(layers, nb, w.graph, roots, w.cfg.fanouts, p, strict, 0, 1, 3, 1024, f"edge bits p={p}")


def many_hubs_graph(seed=0, n_hubs=48, n_leaves=6000, n_comm=4, degrees=(65, 66, 100, 128, 129, 255, 257, 700, 3000)):
    """Hubs of degree 65..3000 whose neighbours are 0 %, a few, half, most or all in the hub's own community
    (symmetrised); exercises every long-row path of the selection kernels."""
    rng = np.random.default_rng(seed)
    n = n_hubs + n_leaves
    comm = np.concatenate([rng.integers(0, n_comm, n_hubs), rng.integers(0, n_comm, n_leaves)]).astype(np.int32)
    leaves_of = [n_hubs + np.nonzero(comm[n_hubs:] == c)[0] for c in range(n_comm)]
    others_of = [n_hubs + np.nonzero(comm[n_hubs:] != c)[0] for c in range(n_comm)]
    rows, cols = [], []
    for h in range(n_hubs):
        deg = int(rng.choice(list(degrees)))
        frac = float(rng.choice([0.0, 0.02, 0.1, 0.5, 0.9, 1.0]))
        n_in = min(int(round(deg * frac)), len(leaves_of[comm[h]]))
        n_out = min(deg - n_in, len(others_of[comm[h]]))
        nb = np.concatenate([rng.choice(leaves_of[comm[h]], n_in, replace=False), rng.choice(others_of[comm[h]], n_out, replace=False)])
        rows += [np.full(len(nb), h), nb]
        cols += [nb, np.full(len(nb), h)]
    r, c = np.concatenate(rows), np.concatenate(cols)
    key = np.unique(r.astype(np.int64) * n + c)
    r, c = key // n, (key % n).astype(np.int32)
    indptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(r, minlength=n), out=indptr[1:])
    return (indptr, c, comm), n_hubs


@pytest.mark.parametrize("edge_classes", [True, False])
def test_long_rows_all_paths(torch_mod, edge_classes):
    graph, n_hubs = many_hubs_graph()
    dg = DeviceGraph(torch_mod, graph, 4, edge_classes=edge_classes)
    roots = np.arange(n_hubs, dtype=np.int32)
    for p in (0.5, 0.75, 0.9, 0.99, 1.0):
        for fan in ([5], [15], [25], [64]):
            print(f"case long rows p={p} fanout={fan} bits={edge_classes}", flush=True)
            layers, nb = run_gpu(torch_mod, dg, roots, fan, p, False, 5, 1, 0, 16)
            compare(layers, nb, graph, roots, fan, p, False, 5, 1, 0, 16, f"long rows p={p} {fan}")
    layers, nb = run_gpu(torch_mod, dg, roots, [15], 1.0, True, 5, 1, 0, 16)
    compare(layers, nb, graph, roots, [15], 1.0, True, 5, 1, 0, 16, "long rows strict")


@pytest.mark.parametrize("degrees", [(17, 24, 40, 64), (65, 100, 128, 200, 255, 256), (5, 17, 40, 100, 200, 256)])
def test_medium_rows_both_rankings(torch_mod, degrees):
    """Rows of 5..256 neighbours, 160 of them side by side (ten waves of sixteen rows): passes of many short rows, where
    every lane ranks its own four slots, passes of one or two long rows with few candidates, where a lane ranks one
    candidate, and mixtures of both."""
    graph, n_hubs = many_hubs_graph(seed=3, n_hubs=160, n_leaves=4000, n_comm=4, degrees=degrees)
    dg = DeviceGraph(torch_mod, graph, 4, edge_classes=True)
    roots = np.arange(n_hubs, dtype=np.int32)
    for p in (0.5, 0.9, 1.0):
        for fan in ([5], [15], [30]):
            print(f"case medium rows degrees={degrees} p={p} fanout={fan}", flush=True)
            layers, nb = run_gpu(torch_mod, dg, roots, fan, p, False, 11, 2, 0, 160, input_global=(fan[0] == 15))
            compare(layers, nb, graph, roots, fan, p, False, 11, 2, 0, 160, f"medium rows p={p} {fan}", input_global=(fan[0] == 15))


def test_clock_approximation_bound(torch_mod):
    """The weighted selection ranks single-precision keys and accepts a row only if the integer keys provably give the same
    result; that rests on a bound on the error of the single-precision clock, measured here over all 2^32 words."""
    from paper_2504_18082_amd import binding as B
    res = torch_mod.full((4,), -1.0, dtype=torch_mod.float32, device="cuda")
    B.cr_selftest_clock_approximation(res)
    torch_mod.cuda.synchronize()
    worst_abs, worst_rel, worst_ratio, zero = res.cpu().numpy().tolist()
    print(f"clock approximation: |error| <= {worst_abs:.3f} units of 2^-24 (small clocks), relative <= {worst_rel:.3e} (large clocks), "
          f"fraction of the assumed bound {worst_ratio:.3f}", flush=True)
    assert zero == 0.0
    assert 0.0 < worst_ratio <= 0.5           # a factor of two in hand


@pytest.mark.parametrize("edge_classes", [True, False])
def test_exact_ranking_path(torch_mod, arxiv_workload, edge_classes):
    """CR_SAMPLE_EXACT_RANKING sends every row through the path that otherwise only redoes the rare rows whose pre-filter
    threshold let too few slots through or whose boundary words are equal: same blocks, for short and long rows."""
    w = arxiv_workload
    dg = DeviceGraph(torch_mod, w.graph, w.cfg.n_comm, edge_classes=edge_classes)
    perm = oracle.build_batches(oracle.RAND, 1, 0, 2, w.train_ids, w.comm, w.cfg.n_comm)
    roots = perm[:1024 + 300]
    for p, strict in ((0.5, False), (1.0, False), (1.0, True), (0.9, False)):
        print(f"case exact ranking arxiv p={p} strict={strict} bits={edge_classes}", flush=True)
        layers, nb = run_gpu(torch_mod, dg, roots, w.cfg.fanouts, p, strict, 2, 2, 1, 1024, input_global=not strict, exact_ranking=True)
        compare(layers, nb, w.graph, roots, w.cfg.fanouts, p, strict, 2, 2, 1, 1024, f"exact ranking p={p}", input_global=not strict)
    graph, n_hubs = many_hubs_graph(seed=3)
    dg = DeviceGraph(torch_mod, graph, 4, edge_classes=edge_classes)
    roots = np.arange(n_hubs, dtype=np.int32)
    for p in (0.5, 1.0):
        for fan in ([15], [64]):
            print(f"case exact ranking long rows p={p} fanout={fan} bits={edge_classes}", flush=True)
            layers, nb = run_gpu(torch_mod, dg, roots, fan, p, False, 5, 1, 0, 16, exact_ranking=True)
            compare(layers, nb, graph, roots, fan, p, False, 5, 1, 0, 16, f"exact ranking long rows p={p} {fan}")


@pytest.mark.parametrize("n_comm,input_global", [(50, True), (50, False), (9000, True)])
def test_row_order_groups_destinations_by_community(torch_mod, tiny_workload, n_comm, input_global):
    """cr_block_set.row_order: per batch a permutation of the destination rows, communities ascending (folded onto
    4096 buckets in order when there are more communities); everything else of the blocks is unchanged."""
    from paper_2504_18082_amd import binding as B
    torch = torch_mod
    w = tiny_workload
    rng = np.random.default_rng(n_comm)
    comm = w.comm if n_comm == 50 else rng.integers(0, n_comm, size=w.cfg.n_nodes).astype(np.int32)
    graph = (w.indptr, w.indices, comm)
    dg = DeviceGraph(torch, graph, n_comm)
    fanouts, batch_size, seed, epoch = [10, 5], 256, 3, 1
    roots = w.train_ids[:3 * batch_size + 77]
    n_batches = 4
    flags = (B.CR_SAMPLE_INPUT_GLOBAL_IDS if input_global else 0) | B.CR_SAMPLE_ROW_ORDER
    cfg = B.make_sample_cfg(fanouts, 0.5, seed, epoch, 0, flags)
    print(f"case row order n_comm={n_comm} input_global={input_global}", flush=True)
    layers = B.alloc_block_sets(cfg, dg.n_nodes, batch_size, n_batches, order_input=True)
    layers[1] = B.BlockSet(n_batches, fanouts[1], layers[1].cap_dst, layers[1].cap_src, layers[1].cap_nnz, True, row_order=True)
    for b in layers:
        b.row_order.fill_(-7)
    ws = torch.empty(B.cr_sample_blocks_workspace_bytes(cfg, dg.n_nodes, batch_size, n_batches), dtype=torch.uint8, device="cuda")
    ws.fill_(0xAB)                                       # nothing may rely on a clean workspace
    d_roots = torch.from_numpy(np.ascontiguousarray(roots, dtype=np.int32)).cuda()
    for rep in range(2):
        B.cr_sample_blocks(dg.c, cfg, d_roots, len(roots), batch_size, n_batches, ws, layers)
        torch.cuda.synchronize()
        for l, b in enumerate(layers):
            hdr = b.hdr.cpu().numpy()
            order = b.row_order.cpu().numpy()
            src = b.src_ids.cpu().numpy()
            for g in range(n_batches):
                n_dst = hdr[g, 0]
                o = order[g, :n_dst]
                assert np.array_equal(np.sort(o), np.arange(n_dst)), f"layer {l} batch {g}: not a permutation"
                assert np.all(order[g, n_dst:] == -7)
                c = comm[src[g, :n_dst]][o].astype(np.int64)
                bucket = c if n_comm <= 4096 else c * 4096 // n_comm
                assert np.all(np.diff(bucket) >= 0), f"layer {l} batch {g}: buckets not ascending"
    compare(layers, n_batches, graph, roots, fanouts, 0.5, False, seed, epoch, 0, batch_size, "row order", input_global=input_global)
