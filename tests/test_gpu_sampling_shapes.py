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


# blocks whose row pointers the selection works out itself (at most 512 rows by capacity) and just not: rows at the root and one hop on,
# empty and long rows among them, a short last batch, with the input block in global ids and relabelled
@pytest.mark.parametrize("batch_size,n_batches,p", [(1, 3, 0.5), (63, 2, 0.9), (64, 1, 1.0), (102, 5, 0.5), (103, 5, 0.9), (512, 3, 1.0), (513, 2, 0.5)])
@pytest.mark.parametrize("input_global", [False, True])
def test_row_pointers_in_the_selection(torch_mod, batch_size, n_batches, p, input_global):
    from paper_2504_18082_amd import binding as B
    torch = torch_mod
    n = 3000
    graph = mixed_graph(n)
    dg = DeviceGraph(torch, graph, 8, edge_classes=True)
    n_roots = batch_size * n_batches - batch_size // 2
    roots = np.random.default_rng(4).permutation(n).astype(np.int32)[:n_roots]
    print(f"case row pointers in the selection: {n_batches} batches of {batch_size}, p={p}, global {input_global}", flush=True)
    cfg = B.make_sample_cfg([7, 4], p, 3, 1, 2, B.CR_SAMPLE_INPUT_GLOBAL_IDS if input_global else 0)
    layers = B.alloc_block_sets(cfg, n, batch_size, n_batches)
    ws = torch.full((B.cr_sample_blocks_workspace_bytes(cfg, n, batch_size, n_batches),), 0xAB, dtype=torch.uint8, device="cuda")
    B.cr_sample_blocks(dg.c, cfg, torch.from_numpy(roots).cuda(), n_roots, batch_size, n_batches, ws, layers)
    torch.cuda.synchronize()
    compare(layers, n_batches, graph, roots, [7, 4], p, False, 3, 1, 2, batch_size, f"row pointers p={p}", input_global=input_global)


def fixed_rows(n_nodes, rows):
    """Graph whose node i has the neighbours rows(i) (ascending, distinct)."""
    r = [np.sort(np.asarray(rows(i), dtype=np.int32)) for i in range(n_nodes)]
    indptr = np.zeros(n_nodes + 1, dtype=np.int64)
    indptr[1:] = np.cumsum([len(x) for x in r])
    return indptr, np.concatenate(r), (np.arange(n_nodes) // (n_nodes // 4 + 1)).astype(np.int32)


def check(torch_mod, graph, n_roots, batch_size, fanouts, p, what):
    dg = DeviceGraph(torch_mod, graph, 4, edge_classes=True)
    roots = np.random.default_rng(2).permutation(len(graph[0]) - 1).astype(np.int32)[:n_roots]
    print(f"case {what}: {n_roots} roots in batches of {batch_size}, fanouts {fanouts}, p={p}", flush=True)
    layers, nb = run_gpu(torch_mod, dg, roots, fanouts, p, False, 5, 1, 0, batch_size)
    compare(layers, nb, graph, roots, fanouts, p, False, 5, 1, 0, batch_size, what)


# ids of a hop (rows and chosen neighbours): just one part (11264) and just not, and two sizes of sixteen parts
@pytest.mark.parametrize("batch_size,fanout", [(1, 1), (64, 1), (1024, 10), (1025, 10), (1024, 64), (11915, 10), (11916, 10)])
def test_frontier_parts(torch_mod, batch_size, fanout):
    rng = np.random.default_rng(batch_size)
    n = 20_000
    graph = fixed_rows(n, lambda i: np.unique(rng.integers(0, n, size=i % (2 * fanout + 1))))
    check(torch_mod, graph, min(n, 2 * batch_size - batch_size // 3), batch_size, [2, fanout], 0.5, "frontier parts")


def wide_graph(n, n_rows, degree):
    """n nodes, the first n_rows of them with `degree` neighbours anywhere: a hop at those reaches almost as many ids as it has edges."""
    rng = np.random.default_rng(degree)
    r = np.sort(rng.integers(0, n - degree, size=(n_rows, degree)), axis=1) + np.arange(degree)          # ascending, distinct
    indptr = np.minimum(np.arange(n + 1, dtype=np.int64), n_rows) * degree
    return indptr, r.reshape(-1).astype(np.int32), (np.arange(n) // (n // 4 + 1)).astype(np.int32)


def sample_wide(torch, batch_size, fanout, flags=0, p=0.5, cut=0, n_batches=1):
    """Batches at the head of wide_graph, two hops; the first hop's frontier array `cut` entries short of what the first batch needs."""
    from paper_2504_18082_amd import binding as B
    n, n_roots = 1_200_000, batch_size * n_batches
    graph = wide_graph(n, n_roots + 1000, fanout + 1)
    roots = np.random.default_rng(2).permutation(n_roots + 1000).astype(np.int32)[:n_roots]
    want = oracle.sample_blocks(graph, roots[:batch_size], [1, fanout], p, bool(flags & B.CR_SAMPLE_STRICT_INTRA), 5, 1, 0, np.full(n, -1, dtype=np.int32))
    cfg = B.make_sample_cfg([1, fanout], p, 5, 1, 0, flags | (B.CR_SAMPLE_SMALL_FRONTIER if cut else 0))
    layers = B.alloc_block_sets(cfg, n, batch_size, n_batches)
    if cut:
        cap_src = want[1].n_src - cut
        layers = [B.BlockSet(1, 1, cap_src, 2 * cap_src, cap_src, False), B.BlockSet(1, fanout, batch_size, cap_src, batch_size * fanout, True)]
    ws = torch.full((B.cr_sample_blocks_workspace_bytes(cfg, n, batch_size, n_batches),), 0xAB, dtype=torch.uint8, device="cuda")
    dg = DeviceGraph(torch, graph, 4, edge_classes=True)
    B.cr_sample_blocks(dg.c, cfg, torch.from_numpy(roots).cuda(), n_roots, batch_size, n_batches, ws, layers)
    torch.cuda.synchronize()
    return graph, roots, want, layers, ws


# ids of a hop where the parts double (73728, 147456) and where the tables in memory take over (73728 for one batch, 147456 for a group
# of two, 294912 for any): just at and just above, each with its transposed block; nearly every edge is a first appearance.  The
# direct-address table leaves its cleared words behind
@pytest.mark.parametrize("batch_size,n_batches,table", [(8192, 1, False), (8193, 1, True), (8193, 2, False), (16384, 2, False), (16385, 2, True),
                                                        (16385, 4, False), (32768, 4, False), (32769, 4, True)])
def test_frontier_parts_double(torch_mod, batch_size, n_batches, table):
    from paper_2504_18082_amd import binding as B
    print(f"case frontier of {n_batches} x {9 * batch_size} ids", flush=True)
    graph, roots, want, layers, ws = sample_wide(torch_mod, batch_size, 8, B.CR_SAMPLE_INPUT_GLOBAL_IDS, n_batches=n_batches)
    compare(layers, n_batches, graph, roots, [1, 8], 0.5, False, 5, 1, 0, batch_size, "parts double", input_global=True)
    assert want[1].n_src > 0.8 * 9 * batch_size
    words = (ws[:ws.numel() // 4 * 4].view(torch_mod.int32) == 0x7FFFFFFF).sum()
    assert int(words) >= n_batches * 1_200_000 if table else int(words) == 0


# transposed blocks of more than forty ranges (368640 edges) or of 131072 rows and more: counters, scan and ranks in memory, behind
# either table
@pytest.mark.parametrize("hash_dedup", [False, True])
@pytest.mark.parametrize("batch_size,fanout", [(40_961, 9), (131_072, 1), (131_073, 2)])
def test_transpose_in_memory(torch_mod, batch_size, fanout, hash_dedup):
    from paper_2504_18082_amd import binding as B
    print(f"case transpose in memory: {batch_size} rows of {fanout}, hash {hash_dedup}", flush=True)
    graph, roots, _, layers, _ = sample_wide(torch_mod, batch_size, fanout, B.CR_SAMPLE_HASH_DEDUP if hash_dedup else 0)
    compare(layers, 1, graph, roots, [1, fanout], 0.5, False, 5, 1, 0, batch_size, "transpose in memory")


# a frontier cut short where several workgroups number the hop (27 K ids), and where the tables do (the same with the open-addressing
# table, strict sampling): marked, the length that was needed reported, every local id inside the arrays
@pytest.mark.parametrize("strict,hash_dedup", [(False, False), (False, True), (True, False)])
def test_cut_frontier(torch_mod, strict, hash_dedup):
    from paper_2504_18082_amd import binding as B
    torch = torch_mod
    flags = (B.CR_SAMPLE_STRICT_INTRA if strict else 0) | (B.CR_SAMPLE_HASH_DEDUP if hash_dedup else 0)
    status = torch.zeros(B.CR_CTX_STATUS_WORDS, dtype=torch.int64, device="cuda")
    ctx = B.Context(status=status)
    ctx.make_current()
    try:
        print(f"case cut frontier strict={strict} hash={hash_dedup}", flush=True)
        _, _, want, layers, _ = sample_wide(torch, 3000, 8, flags, 1.0 if strict else 0.5, cut=101)
        blk, b, low = want[1], layers[1], layers[0]
        assert ctx.poll_error() == (B.CR_ERR_ASYNC_OVERFLOW, blk.n_src)
        n_src = blk.n_src - 101
        hdr = b.hdr[0, :4].cpu().tolist()
        assert hdr[:3] == [blk.n_dst, n_src, blk.nnz] and hdr[3] != 0 and int(low.hdr[0, 3]) != 0
        assert np.array_equal(b.src_ids[0, :n_src].cpu().numpy(), blk.src_ids[:n_src])
        idx = b.indices[0, :blk.nnz].cpu().numpy()
        assert np.array_equal(idx, np.where(blk.indices < n_src, blk.indices, 0))
        t_indptr, t_idx = b.t_indptr[0, :n_src + 1].cpu().numpy(), b.t_indices[0, :blk.nnz].cpu().numpy()
        assert t_indptr[0] == 0 and t_indptr[-1] == blk.nnz and np.all(np.diff(t_indptr) == np.bincount(idx, minlength=n_src))
        assert t_idx.min() >= 0 and t_idx.max() < blk.n_dst
        assert int(low.hdr[0, 0]) == n_src and int(low.hdr[0, 2]) <= n_src
    finally:
        B.Context.make_none_current()
        ctx.destroy()


@pytest.mark.parametrize("batch_size", [700, 3000])
def test_hash_dedup_flag_takes_the_table(torch_mod, batch_size):
    """CR_SAMPLE_HASH_DEDUP names the open-addressing table, which has at least twice as many words as the frontier has ids: half
    of them stay as they were cleared (all ones, which nothing else leaves in the workspace).  One hop only: the input-side block
    is left in global ids."""
    from paper_2504_18082_amd import binding as B
    print(f"case hash flag: {batch_size} rows", flush=True)
    for flags, table in ((B.CR_SAMPLE_INPUT_GLOBAL_IDS, False), (B.CR_SAMPLE_INPUT_GLOBAL_IDS | B.CR_SAMPLE_HASH_DEDUP, True)):
        graph, roots, want, layers, ws = sample_wide(torch_mod, batch_size, 8, flags)
        compare(layers, 1, graph, roots, [1, 8], 0.5, False, 5, 1, 0, batch_size, "hash flag", input_global=True)
        cleared = int((ws[:ws.numel() // 8 * 8].view(torch_mod.int64) == -1).sum())
        assert cleared >= want[1].n_src if table else cleared == 0


# a handful of nodes that every row chooses: lists of a part and of a range of sources that overflow, ranges whose rows are sorted
# rather than ranked, in one window (15000 edges) and in many (108000)
@pytest.mark.parametrize("batch_size,hubs", [(3000, 5), (12_000, 9)])
def test_every_row_shares_its_neighbours(torch_mod, batch_size, hubs):
    graph = fixed_rows(30_000, lambda i: 7 * np.arange(hubs) + 400)
    check(torch_mod, graph, 2 * batch_size, batch_size, [3, hubs], 0.5, "shared neighbours")


# rows whose neighbours follow a power law, and hops of one part, several and many: ranges ranked next to ranges taken by windows (with
# a list that overflows, and with one that does not), windows with many sources, a last window of a few edges
@pytest.mark.parametrize("batch_size,fanout", [(700, 15), (1500, 15), (4097, 12), (9000, 15), (18_000, 15)])
def test_skewed_neighbours(torch_mod, batch_size, fanout):
    rng = np.random.default_rng(batch_size)
    n = 40_000
    graph = fixed_rows(n, lambda i: np.unique((rng.random(fanout + 5) ** 4 * n).astype(np.int32)))
    check(torch_mod, graph, 2 * batch_size - 3, batch_size, [2, fanout], 0.5, "skewed")


def test_one_part_gets_every_id(torch_mod):
    """More distinct ids in one part than the table holds: the part is taken in slices."""
    n = 420_000
    ids = np.arange(n, dtype=np.uint32)
    fold = ids ^ (ids >> 15)
    part0 = ids[((fold ^ (fold >> 5) ^ (fold >> 10)) & 15) == 0].astype(np.int32)       # the kernel's choice of the part, sixteen parts
    assert len(part0) > 20_000
    rng = np.random.default_rng(1)
    picks = np.sort(part0[(rng.integers(0, len(part0) - 20, size=(n, 1)) + np.arange(15))], axis=1)
    graph = (np.arange(n + 1, dtype=np.int64) * 15, picks.reshape(-1), (np.arange(n) // (n // 4 + 1)).astype(np.int32))
    check(torch_mod, graph, 16_000, 8000, [2, 15], 0.5, "one part")


@pytest.mark.parametrize("n_batches,parts", [(1, 32), (2, 32), (32, 8)])
def test_one_part_gets_every_id_of_a_group(torch_mod, n_batches, parts):
    """The same with as many parts as small groups (32) and large ones (8) are cut into, and batches without an edge behind them."""
    n, batch_size = 27_000 * parts, 4000 if n_batches < 32 else 900
    ids = np.arange(n, dtype=np.uint32)
    fold = ids ^ (ids >> 15)
    part0 = ids[((fold ^ (fold >> 5) ^ (fold >> 10)) & (parts - 1)) == 0].astype(np.int32)
    assert len(part0) > 20_000
    rng = np.random.default_rng(parts)
    picks = np.sort(part0[(rng.integers(0, len(part0) - 20, size=(n, 1)) + np.arange(15))], axis=1)
    degree = np.where(np.arange(n) % 7 == 3, 0, 15)
    graph = (np.concatenate([[0], np.cumsum(degree)]).astype(np.int64), picks[degree > 0].reshape(-1), (np.arange(n) // (n // 4 + 1)).astype(np.int32))
    check(torch_mod, graph, n_batches * batch_size - 5, batch_size, [2, 15], 0.5, "one part of a group")


# destination rows of a whole group in community order: one workgroup (at most 8192 rows by capacity), just not, many buckets
@pytest.mark.parametrize("batch_size,n_batches,n_comm", [(64, 1, 5), (409, 4, 4096), (410, 4, 9000), (1024, 8, 70)])
def test_group_order(torch_mod, batch_size, n_batches, n_comm):
    from paper_2504_18082_amd import binding as B
    torch = torch_mod
    graph = mixed_graph(24_000)
    comm = np.sort(np.random.default_rng(n_comm).integers(0, n_comm, size=24_000)).astype(np.int32)
    dg = DeviceGraph(torch, (graph[0], graph[1], comm), n_comm, edge_classes=True)
    print(f"case group order: {n_batches} batches of {batch_size}, {n_comm} communities", flush=True)
    cfg = B.make_sample_cfg([3, 4], 0.5, 3, 1, 0, B.CR_SAMPLE_INPUT_GLOBAL_IDS | B.CR_SAMPLE_ROW_ORDER)
    layers = B.alloc_block_sets(cfg, 24_000, batch_size, n_batches, group_order_input=True)
    layers[0].group_order.fill_(-1)
    ws = torch.empty(B.cr_sample_blocks_workspace_bytes(cfg, 24_000, batch_size, n_batches), dtype=torch.uint8, device="cuda")
    roots = torch.from_numpy(np.random.default_rng(1).permutation(24_000).astype(np.int32)[:batch_size * n_batches - 3]).cuda()
    B.cr_sample_blocks(dg.c, cfg, roots, roots.numel(), batch_size, n_batches, ws, layers)
    torch.cuda.synchronize()
    b = layers[0]
    n_dst, src, order = b.hdr[:, 0].cpu().numpy(), b.src_ids.cpu().numpy(), b.group_order.cpu().numpy()
    n = int(n_dst.sum())
    assert order[n_batches * b.cap_dst] == n and np.all(b.hdr[:, 1].cpu().numpy() == -1)
    want = np.concatenate([g * b.cap_dst + np.arange(n_dst[g]) for g in range(n_batches)])
    assert np.array_equal(np.sort(order[:n]), want)
    c = comm[src.reshape(n_batches, -1)[order[:n] // b.cap_dst, order[:n] % b.cap_dst]].astype(np.int64)
    assert np.all(np.diff(c if n_comm <= 4096 else c * 4096 // n_comm) >= 0)


# the bound that parts kept from left-out neighbours: one left out, one kept, rows that fill a pass, one class short of the fanout
@pytest.mark.parametrize("p", [0.5, 0.51, 0.9, 0.97, 1.0])
@pytest.mark.parametrize("fanout", [1, 15, 64])
def test_rows_just_above_the_fanout(torch_mod, fanout, p):
    rng = np.random.default_rng(fanout)
    n = 4096
    degrees = [fanout + 1, fanout + 2, 256, 255, 254, max(1, fanout), 5, 4, 3, 257, fanout + 1, 64]

    def rows(i):
        deg = degrees[i % len(degrees)]
        near = rng.integers(0, deg + 1) if i % 3 else deg - (i % 2)      # how many lie in the node's own community
        home = i // (n // 4 + 1) * (n // 4 + 1)
        own = np.arange(home, min(n, home + n // 4 + 1))
        other = np.setdiff1d(np.arange(n), own)
        return np.concatenate([rng.choice(own, near, replace=False), rng.choice(other, deg - near, replace=False)])

    check(torch_mod, fixed_rows(n, rows), n - 3, 1000, [fanout], p, f"rows of about {fanout} neighbours, p={p}")


# rows longer than a pass: one slot more than a pass, whole stretches and one slot more, candidates of one and of two per lane
@pytest.mark.parametrize("p", [0.5, 0.51, 0.9, 0.97, 1.0])
@pytest.mark.parametrize("fanout", [1, 25, 64])
def test_long_rows(torch_mod, fanout, p):
    rng = np.random.default_rng(fanout)
    n, degrees = 4096, [257, 300, 511, 512, 513, 1000, 3000]
    home = np.arange(n) // (n // 4 + 1)

    def rows(i):
        if i >= 280:
            return rng.choice(n, i % 3, replace=False)
        deg = degrees[i % len(degrees)]
        own, other = np.flatnonzero(home == home[i]), np.flatnonzero(home != home[i])
        near = min(len(own), [deg // 2, fanout, fanout - 1, deg - 1, 0][i // len(degrees) % 5])      # how many lie in the node's own community
        near = max(near, deg - len(other))
        return np.concatenate([rng.choice(own, near, replace=False), rng.choice(other, deg - near, replace=False)])

    check(torch_mod, fixed_rows(n, rows), n - 3, 1000, [fanout], p, f"long rows, fanout {fanout}, p={p}")
