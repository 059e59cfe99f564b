"""The work that a user of this framework has it do, as timed and compared cases.

A case is a dict of plain values; `path` says which part of a training program it is:

  roots     the epoch's permutation of the training set (once per epoch)
  sample    the blocks of a group of mini-batches (once per group)
  gather    input-feature gather + aggregation of a sampled group (once per group)
  input     the dense part of the first layer, forward and backward with its SGD step (every mini-batch)
  sage      one GraphSAGE layer above the first, forward and backward; the last one with the loss (every mini-batch)
  gcn       the same for a GCN layer
  gat       one graph-attention layer, forward and backward, the first one with its row gather (every mini-batch)
  train     a sampled group and its training steps, through the Trainer (what a training program spends its time on)

Graphs are the planted-community stand-ins of the paper's data sets that `synth` describes, at full or reduced scale,
drawn on the GPU; `graph` and `scale` name them.
"""
from __future__ import annotations

import copy
import math

import numpy as np
import torch

from paper_2504_18082_amd import binding as B
from paper_2504_18082_amd import synth, synth_gpu
from paper_2504_18082_amd.trainer import Trainer

DEV = "cuda"
POLICIES = {"norand": B.CR_ROOTS_NORAND, "mix": B.CR_ROOTS_COMM_RAND, "rand": B.CR_ROOTS_RAND}
LR, DECAY = 0.01, 5e-4


def listed():
    return [
        # epoch start of the largest workload under the paper's favoured setting (MIX-12.5 %): both sorts of the step
        dict(name="roots_papers_mix", path="roots", n_nodes=111_000_000, n_train=1_221_000, n_comm=100_000, policy="mix", percent=12.5),
        # the sampler as the trainer calls it: a group of 32 mini-batches, input block in global ids, community order
        dict(name="sample_products_uniform", path="sample", graph="products", scale=1.0, batches=32, batch_size=1024, p=0.5,
             layout="global"),
        # hub rows, weighted selection and the de-duplicated, transposed input block that graph attention needs
        dict(name="sample_reddit_weighted", path="sample", graph="reddit", scale=1.0, batches=8, batch_size=1024, p=0.9,
             layout="transposed"),
        # layer-0 gather: narrow bf16 rows from a table far beyond the caches (a tenth of papers: 2.8 GB) ...
        dict(name="gather_papers_bf16", path="gather", graph="papers", scale=0.1, batches=32, batch_size=1024, p=0.5, model="sage"),
        # ... and rows of 2.4 KB, float, taken in column panels
        dict(name="gather_reddit_f32", path="gather", graph="reddit", scale=1.0, batches=16, batch_size=1024, p=0.5, model="sage"),
        # papers' input layer: 2 x 128 -> 256 over the destination rows of one mini-batch
        dict(name="input_layer_papers", path="input", rows=60_800, cap=67_584, f_in=128, f_out=256, operands=2),
        # the layer above it, 6 K rows on a products block
        dict(name="hidden_layer_products", path="sage", graph="products", scale=1.0, batch_size=1024, p=0.5, layer=1, n_classes=47),
        # the layer next to the loss with more classes than one column tile holds
        dict(name="top_layer_172", path="sage", graph="products", scale=1.0, batch_size=1024, p=0.5, layer=2, n_classes=172),
        # GCN's middle layer
        dict(name="gcn_layer_arxiv", path="gcn", graph="arxiv", scale=1.0, batch_size=1024, p=1.0, layer=1, n_classes=40),
        # the attention layer that dominates a GAT step: 130 K source rows of 602 features, 4 heads of 64
        dict(name="gat_layer_reddit", path="gat", graph="reddit", scale=1.0, batch_size=1024, p=0.5, layer=0, heads=4),
        # the default benchmark workload: one group of 32 mini-batches of the full 111 M node graph
        dict(name="train_papers", path="train", graph="papers", scale=1.0, model="sage", batches=32, batch_size=1024, policy="rand",
             percent=0.0, p=0.5),
        # a single small step, where launches and latency are all there is
        dict(name="train_tiny", path="train", graph="tiny", scale=1.0, model="sage", batches=1, batch_size=64, policy="mix",
             percent=12.5, p=1.0),
    ]


# ------------------------------------------------------------------------------------------------ drawn cases
SCALES = {"tiny": (1.0, 4.0), "arxiv": (0.1, 4.0), "reddit": (0.05, 1.0), "products": (0.02, 1.0), "papers": (0.005, 0.2)}


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _whole(rng, lo, hi):
    return min(hi, max(lo, int(round(_log(rng, lo, hi)))))


def _graph(rng, names):
    g = rng.choice(names)
    return g, round(_log(rng, *SCALES[g]), 4)


def draw(rng):
    path = rng.choice(["roots", "sample", "sample", "gather", "gather", "input", "sage", "sage", "gcn", "gat", "train", "train"])
    p = rng.choice([0.5, 0.5, 0.9, 1.0])
    if path == "roots":
        n_train = _whole(rng, 300, 1_221_000)
        return dict(path=path, n_nodes=max(n_train * rng.randint(2, 20), 1000), n_train=n_train, n_comm=_whole(rng, 3, max(4, min(100_000, n_train // 10))),
                    policy=rng.choice(["mix", "mix", "rand", "rand", "norand"]), percent=rng.choice([0.0, 12.5, 25.0, 50.0]))
    if path == "input":
        rows, operands = _whole(rng, 900, 66_000), rng.choice([1, 2, 2])
        return dict(path=path, rows=rows, cap=rows + rng.randint(0, max(1, rows // 6)), f_in=rng.choice([64, 100, 128, 128, 602, rng.randint(17, 300)]),
                    f_out=rng.choice([256, 256, 128, rng.randint(33, 256)]), operands=operands)
    batch = rng.choice([64, 1024, 1024, rng.randint(33, 1024)])
    if path == "sample":
        graph, scale = _graph(rng, ["tiny", "arxiv", "reddit", "products", "papers"])
        return dict(path=path, graph=graph, scale=scale, batches=_whole(rng, 1, 32 if graph != "reddit" else 8), batch_size=batch, p=p,
                    layout=rng.choice(["global", "global", "relabelled", "transposed"]))
    if path == "gather":
        graph, scale = _graph(rng, ["tiny", "arxiv", "reddit", "products", "papers"])
        return dict(path=path, graph=graph, scale=scale, batches=_whole(rng, 1, 32 if graph != "reddit" else 16), batch_size=batch, p=p,
                    model=rng.choice(["sage", "sage", "gcn"]))
    if path in ("sage", "gcn"):
        graph, scale = _graph(rng, ["arxiv", "reddit", "products", "papers"])
        layers = len(synth.CONFIGS[graph].fanouts)
        return dict(path=path, graph=graph, scale=min(scale, 0.1) if graph == "papers" else scale, batch_size=batch, p=p, layer=rng.randint(1, layers - 1),
                    n_classes=rng.choice([10, 40, 41, 47, 172, rng.randint(5, 200)]))
    if path == "gat":
        graph, scale = _graph(rng, ["tiny", "arxiv", "reddit", "products"])
        return dict(path=path, graph=graph, scale=scale, batch_size=batch, p=p, layer=rng.randint(0, len(synth.CONFIGS[graph].fanouts) - 2),
                    heads=rng.choice([1, 2, 4, 4, 8]))
    graph, scale = _graph(rng, ["tiny", "arxiv", "reddit", "products", "papers"])
    model = rng.choice(["sage", "sage", "gcn", "gat"])
    if graph == "papers" and model == "gat":
        model = "sage"
    return dict(path=path, graph=graph, scale=scale, model=model, batches=_whole(rng, 1, 32 if model != "gat" else 8), batch_size=batch,
                policy=rng.choice(["rand", "mix", "norand"]), percent=12.5, p=p)


# ------------------------------------------------------------------------------------------------ inputs
def _config(case):
    cfg = synth.scaled(synth.CONFIGS[case["graph"]], case["scale"]) if case["scale"] != 1.0 else copy.deepcopy(synth.CONFIGS[case["graph"]])
    cfg.batch_size = case.get("batch_size", cfg.batch_size)
    cfg.n_classes = case.get("n_classes", cfg.n_classes)
    return cfg


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 13)
    return g


def _bf16(x):
    """Raw bf16 words, as the library takes them."""
    return x.to(torch.bfloat16).view(torch.int16)


def _as_bf16(t):
    return t.view(torch.bfloat16)


def _rows(n, width, real, gen, relu=False, scale=1.0, cap=None):
    """bf16 [cap or n][width] of normal values in the first `real` columns (and n rows), zeros elsewhere."""
    t = torch.zeros((cap or n, width), dtype=torch.int16, device=DEV)
    x = torch.randn((n, real), device=DEV, generator=gen) * scale
    t[:n, :real] = _bf16(x.clamp_min_(0.0) if relu else x)
    return t


def _weights(fan_in, rows, cols, gen):
    a = math.sqrt(6.0 / (fan_in + cols))
    return ((torch.rand((rows, cols), device=DEV, generator=gen) * 2 - 1) * a).cpu().numpy()


def _sampled(case, seed, batches, with_features=False, layout="global"):
    """A graph and the blocks of one group of mini-batches on it."""
    cfg = _config(case)
    w = synth_gpu.make_workload_gpu(cfg, seed, with_features=with_features)
    gen = _gen(seed)
    want = batches * cfg.batch_size
    roots = w.train_ids[torch.randperm(w.train_ids.numel(), generator=gen, device=DEV)][:want].contiguous()
    batches = max(1, -(-roots.numel() // cfg.batch_size))        # a small training set fills fewer mini-batches
    flags = {"global": B.CR_SAMPLE_INPUT_GLOBAL_IDS | B.CR_SAMPLE_ROW_ORDER, "relabelled": 0, "transposed": B.CR_SAMPLE_TRANSPOSE_INPUT}[layout]
    scfg = B.make_sample_cfg(cfg.fanouts, case["p"], seed, 1, 0, flags)
    graph = B.make_graph(w.indptr, w.indices, w.comm, cfg.n_comm)
    bits = B.cr_graph_edge_classes(graph)
    graph.edge_intra = bits.data_ptr()
    blocks = B.alloc_block_sets(scfg, cfg.n_nodes, cfg.batch_size, batches, DEV, transpose_input=layout == "transposed",
                                group_order_input=layout == "global")
    ws = torch.empty(B.cr_sample_blocks_workspace_bytes(scfg, cfg.n_nodes, cfg.batch_size, batches), dtype=torch.uint8, device=DEV)
    return dict(cfg=cfg, w=w, roots=roots, batches=batches, scfg=scfg, graph=graph, bits=bits, blocks=blocks, ws=ws, gen=gen)


def _sample(s):
    B.cr_sample_blocks(s["graph"], s["scfg"], s["roots"], s["roots"].numel(), s["cfg"].batch_size, s["batches"], s["ws"], s["blocks"])


def _header(blk, g=0):
    return [int(x) for x in blk.hdr[g, :3].cpu().tolist()]       # n_dst, n_src, nnz


def _zeros(*shape, dtype=torch.float32):
    return torch.zeros(shape, dtype=dtype, device=DEV)


def _prepare_layer(case, seed, operands):
    """What the layers above the first have in common: a block, the activations below, weights, buffers."""
    s = _sampled(case, seed, 1, layout="global")
    _sample(s)
    cfg, gen, l = s["cfg"], s["gen"], case["layer"]
    blk, top = s["blocks"][l], l == len(cfg.fanouts) - 1
    n_dst, n_src, _ = _header(blk)
    f_out = cfg.n_classes if top else cfg.hidden
    lay = B.SageLayer(_weights(cfg.hidden, operands * cfg.hidden, f_out, gen), np.zeros(f_out, dtype=np.float32), DEV, operands)
    lay.refresh()
    wide = lay.F_pad
    s.update(blk=blk, top=top, n_dst=n_dst, n_src=n_src, lay=lay, h=_rows(n_src, wide, cfg.hidden, gen, relu=True, cap=blk.cap_src),
             agg=_zeros(blk.cap_dst, wide, dtype=torch.int16), d_in=_zeros(blk.cap_dst, operands * wide, dtype=torch.int16),
             d_src=_zeros(blk.cap_src, wide, dtype=torch.int16),
             ws_bwd=torch.empty(B.cr_sage_linear_bwd_workspace_bytes(lay.F_in, lay.F_out, blk.cap_dst), dtype=torch.uint8, device=DEV))
    if top:
        s.update(out=_zeros(blk.cap_dst, lay.N_pad), dz=_zeros(blk.cap_dst, lay.N_pad, dtype=torch.int16), loss=_zeros(1), row_loss=_zeros(blk.cap_dst),
                 scratch=torch.zeros(B.CR_XENT_SCRATCH_BYTES, dtype=torch.uint8, device=DEV))
    else:
        s.update(out=_zeros(blk.cap_dst, lay.N_pad, dtype=torch.int16),
                 dz=_rows(n_dst, lay.N_pad, f_out, gen, scale=1.0 / cfg.batch_size, cap=blk.cap_dst))
    return s


def prepare(case, seed):
    path = case["path"]
    if path == "roots":
        gen = _gen(seed)
        comm = torch.sort(torch.randint(0, case["n_comm"], (case["n_nodes"],), dtype=torch.int32, device=DEV, generator=gen)).values
        picks = torch.randint(0, case["n_nodes"], (int(case["n_train"] * 1.1) + 64,), device=DEV, generator=gen)
        train = torch.unique(picks).to(torch.int32)
        n = min(case["n_train"], int(train.numel()))
        train = torch.sort(train[torch.randperm(train.numel(), device=DEV, generator=gen)[:n]]).values.contiguous()
        in_train = int(torch.unique(comm[train.to(torch.int64)]).numel())
        return dict(case=case, seed=seed, comm=comm, train=train, perm=torch.zeros_like(train), mix=B.cr_mix_count_from_percent(case["percent"], in_train),
                    ws=torch.empty(B.cr_build_batches_workspace_bytes(n, case["n_comm"]), dtype=torch.uint8, device=DEV))
    if path == "sample":
        return dict(_sampled(case, seed, case["batches"], layout=case["layout"]), case=case)
    if path == "gather":
        s = _sampled(case, seed, case["batches"], with_features=True)
        _sample(s)
        blk, cfg = s["blocks"][0], s["cfg"]
        f_pad, _ = B.cr_sage_padded_dims(cfg.n_feat, cfg.hidden)
        s.update(case=case, f_pad=f_pad, agg=_zeros(s["batches"], blk.cap_dst, f_pad, dtype=torch.int16))
        if case["model"] == "sage":
            s["self"] = _zeros(s["batches"], blk.cap_dst, f_pad, dtype=torch.int16)
        else:
            s["norm"] = B.cr_graph_gcn_norm(s["graph"])
        return s
    if path == "input":
        gen, rows, n_op = _gen(seed), case["rows"], case["operands"]
        lay = B.SageLayer(_weights(case["f_in"], n_op * case["f_in"], case["f_out"], gen), np.zeros(case["f_out"], dtype=np.float32), DEV, n_op)
        lay.refresh()
        x = [_rows(rows, lay.F_pad, case["f_in"], gen, cap=case["cap"]) for _ in range(n_op)]
        return dict(case=case, lay=lay, x_self=x[0] if n_op == 2 else None, x_agg=x[-1], hdr=torch.tensor([rows, rows, 0, 0, 0, 0, 0, 0], dtype=torch.int32, device=DEV),
                    out=_zeros(case["cap"], lay.N_pad, dtype=torch.int16),
                    dz=_rows(rows, lay.N_pad, case["f_out"], gen, scale=1.0 / 1024, cap=case["cap"]),
                    ws=torch.empty(B.cr_sage_linear_bwd_workspace_bytes(lay.F_in, lay.F_out, case["cap"]), dtype=torch.uint8, device=DEV))
    if path == "sage":
        return dict(_prepare_layer(case, seed, 2), case=case)
    if path == "gcn":
        s = _prepare_layer(case, seed, 1)
        s.update(case=case, norm=B.cr_graph_gcn_norm(s["graph"]), blk_norm=_zeros(s["blk"].cap_src + 2 * s["blk"].cap_dst))
        return s
    if path == "gat":
        l, heads = case["layer"], case["heads"]
        s = _sampled(case, seed, 1, with_features=l == 0, layout="transposed")
        _sample(s)
        cfg, gen, blk = s["cfg"], s["gen"], s["blocks"][l]
        n_dst, n_src, _ = _header(blk)
        f_in = cfg.n_feat if l == 0 else cfg.hidden
        lay = B.SageLayer(_weights(f_in, f_in, cfg.hidden, gen), np.zeros(cfg.hidden, dtype=np.float32), DEV, 1)
        lay.drop_bias()
        lay.refresh()
        att = [_weights(1, cfg.hidden, 1, gen)[:, 0] * 0.2 for _ in range(2)]
        par = B.GatParams(att[0], att[1], np.zeros(cfg.hidden, dtype=np.float32), heads, lay.N_pad, 0.2, DEV)
        i16 = torch.int16
        s.update(case=case, blk=blk, n_dst=n_dst, n_src=n_src, lay=lay, par=par, f_in=f_in,
                 x=_zeros(blk.cap_src, lay.F_pad, dtype=i16) if l == 0 else _rows(n_src, lay.F_pad, f_in, gen, relu=True, cap=blk.cap_src),
                 z=_zeros(blk.cap_src, lay.N_pad, dtype=i16), el=_zeros(blk.cap_src, heads), er=_zeros(blk.cap_src, heads), stat=_zeros(blk.cap_dst, 4 * heads),
                 out=_zeros(blk.cap_dst, lay.N_pad, dtype=i16), dz=_zeros(blk.cap_src, lay.N_pad, dtype=i16),
                 d_out=_rows(n_dst, lay.N_pad, cfg.hidden, gen, scale=1.0 / cfg.batch_size, cap=blk.cap_dst),
                 # the forward output whose sign masks the gradient: given, so that a last-bit change of z that turns an
                 # output's sign does not show as a different gradient
                 relu_out=_rows(n_dst, lay.N_pad, cfg.hidden, gen, relu=True, cap=blk.cap_dst),
                 d_in=_zeros(blk.cap_src, lay.F_pad, dtype=i16) if l > 0 else None,
                 ws_att=torch.empty(B.cr_gat_attention_bwd_workspace_bytes(blk.cap_dst, lay.N_pad, heads), dtype=torch.uint8, device=DEV),
                 ws_bwd=torch.empty(B.cr_sage_linear_bwd_workspace_bytes(lay.F_in, lay.F_out, blk.cap_src), dtype=torch.uint8, device=DEV))
        s["rows_hdr"] = B.C.c_void_p(blk.hdr_ptr(0).value + 4 * B.CR_HDR_N_SRC)
        return s
    if path == "train":
        cfg = _config(case)
        w = synth_gpu.make_workload_gpu(cfg, seed)
        tr = Trainer(w, group_size=case["batches"], lr=LR, weight_decay=DECAY, seed=seed, model=case["model"])
        n_batches = tr.build_batches(POLICIES[case["policy"]], B.cr_mix_count_from_percent(case["percent"], w.n_comm_in_train), 1)
        return dict(case=case, tr=tr, batches=min(case["batches"], n_batches))
    raise ValueError(path)


# ------------------------------------------------------------------------------------------------ one pass
def run(s):
    case = s["case"]
    path = case["path"]
    if path == "roots":
        n = B.cr_build_batches(POLICIES[case["policy"]], s["mix"], 1024, s["seed"], 3, s["train"], s["comm"], case["n_comm"], s["ws"], s["perm"])
        return s["perm"], n
    if path == "sample":
        _sample(s)
        return [[t for t in (b.hdr, b.src_ids, b.indptr, b.indices, b.t_indptr, b.t_indices, b.gather_ids) if t is not None] for b in s["blocks"]]
    if path == "gather":
        blk, cfg, w = s["blocks"][0], s["cfg"], s["w"]
        dtype, ld = B.CR_BF16 if cfg.feat_dtype == "bf16" else B.CR_F32, int(w.features.shape[1])
        if case["model"] == "gcn":
            B.cr_gcn_aggregate_fwd_group(blk, s["norm"], w.features, dtype, ld, cfg.n_feat, s["agg"], blk.cap_dst, s["f_pad"])
            return _as_bf16(s["agg"])
        B.cr_gather_aggregate_fwd_group(blk, w.features, dtype, ld, cfg.n_feat, s["agg"], s["self"], blk.cap_dst, s["f_pad"])
        return _as_bf16(s["agg"]), _as_bf16(s["self"])
    if path == "input":
        lay, hdr, cap = s["lay"], B._ptr(s["hdr"]), case["cap"]
        B.cr_sage_linear_fwd(lay, hdr, cap, s["x_self"], s["x_agg"], lay.F_pad, True, None, s["out"])
        B.cr_sage_linear_bwd(lay, hdr, cap, s["x_self"], s["x_agg"], lay.F_pad, s["dz"], LR, DECAY, None, None, s["ws"])
        return _as_bf16(s["out"]), lay.W, lay.bias
    if path in ("sage", "gcn"):
        return _run_layer(s, path == "gcn")
    if path == "gat":
        return _run_gat(s)
    tr = s["tr"]
    tr.sample_group(0, s["batches"], case["p"], 1)
    for g in range(s["batches"]):
        tr.train_batch(g)
    return [tr.out[-1], tr.loss] + [lay.W for lay in tr.layers]


def _run_layer(s, gcn):
    cfg, blk, lay, top, wide = s["cfg"], s["blk"], s["lay"], s["top"], s["lay"].F_pad
    if gcn:
        B.cr_gcn_block_norm(blk, 0, s["norm"], s["blk_norm"])
        B.cr_gcn_aggregate_fwd(blk, 0, s["norm"], s["blk_norm"], s["h"], B.CR_BF16, wide, cfg.hidden, False, None, s["agg"], wide)
    else:
        B.cr_gather_aggregate_fwd(blk, 0, s["h"], B.CR_BF16, wide, cfg.hidden, False, None, s["agg"], None, wide)
    h_self = None if gcn else s["h"]
    if top:
        B.cr_sage_linear_fwd_xent(lay, blk.hdr_ptr(0), blk.cap_dst, h_self, s["agg"], wide, s["out"], cfg.n_classes, s["w"].labels,
                                  blk.src_ids_ptr(0), s["loss"], s["row_loss"], s["dz"], s["scratch"])
    else:
        B.cr_sage_linear_fwd(lay, blk.hdr_ptr(0), blk.cap_dst, h_self, s["agg"], wide, True, None, s["out"])
    if gcn:
        B.cr_sage_linear_bwd(lay, blk.hdr_ptr(0), blk.cap_dst, None, s["agg"], wide, s["dz"], LR, DECAY, None, None, s["ws_bwd"], d_in_bf16=s["d_in"])
        B.cr_gcn_aggregate_bwd(blk, 0, s["blk_norm"], s["d_in"], wide, cfg.hidden, s["h"], wide, None, s["d_src"], wide, relu_dtype=B.CR_BF16,
                               in_dtype=B.CR_BF16)
    else:
        B.cr_sage_layer_bwd(lay, blk, 0, h_self, s["agg"], wide, s["dz"], LR, DECAY, s["d_in"], s["h"], wide, s["d_src"], wide, s["ws_bwd"])
    got = [_as_bf16(s["agg"]), s["out"] if top else _as_bf16(s["out"]), _as_bf16(s["d_src"]), lay.W, lay.bias]
    return got + ([s["loss"], _as_bf16(s["dz"])] if top else [])


def _first_layer(s):
    return s["case"]["layer"] == 0


def _run_gat(s):
    cfg, blk, lay, par = s["cfg"], s["blk"], s["lay"], s["par"]
    if _first_layer(s):
        w = s["w"]
        B.cr_gather_rows_bf16(w.features, B.CR_BF16 if cfg.feat_dtype == "bf16" else B.CR_F32, int(w.features.shape[1]), cfg.n_feat,
                              blk.src_ids_ptr(0), blk.hdr_ptr(0), B.CR_HDR_N_SRC, blk.cap_src, s["x"], lay.F_pad)
    B.cr_sage_linear_fwd(lay, s["rows_hdr"], blk.cap_src, None, s["x"], lay.F_pad, False, None, s["z"])
    B.cr_gat_attention_fwd(blk, 0, par, s["z"], lay.N_pad, True, s["el"], s["er"], s["stat"], None, s["out"])
    B.cr_gat_attention_bwd(blk, 0, par, s["z"], lay.N_pad, s["el"], s["stat"], s["d_out"], lay.N_pad, s["relu_out"], LR, DECAY, s["dz"], s["ws_att"])
    B.cr_sage_linear_bwd(lay, s["rows_hdr"], blk.cap_src, None, s["x"], lay.F_pad, s["dz"], LR, DECAY, None, None, s["ws_bwd"], d_in_bf16=s["d_in"])
    got = [_as_bf16(s["out"]), _as_bf16(s["dz"]), lay.W, par.attn]
    return got + ([_as_bf16(s["d_in"])] if s["d_in"] is not None else [])


# ------------------------------------------------------------------------------------------------ work and tolerance
def _expected(case, batches=None):
    """Expected rows per layer of one mini-batch: [(n_dst, n_src, nnz)], input side first.  Closed form on the
    configuration alone: rows are expanded by min(fanout, mean degree), frontiers draw distinct nodes at random."""
    cfg = _config(case)
    deg = 2.0 * cfg.n_edges_undirected / cfg.n_nodes
    n, out = float(min(cfg.batch_size, cfg.train_fraction * cfg.n_nodes)), []
    for f in reversed(cfg.fanouts):
        nnz = n * min(f, deg)
        new = cfg.n_nodes * (1.0 - math.exp(-nnz / cfg.n_nodes))
        out.append((n, min(cfg.n_nodes, n + new), nnz))
        n = out[-1][1]
    return cfg, out[::-1]


def _dense(rows, k, n):
    return 2.0 * rows * k * n


def work(case):
    path = case["path"]
    if path == "roots":
        words = case["n_train"] * (2 if case["policy"] != "mix" else 3)          # ids in and out, a community per node
        return dict(bytes=4.0 * words, flops=0.0)
    if path == "input":
        k, n, rows = case["operands"] * case["f_in"], case["f_out"], case["rows"]
        # operands once per direction, dZ, the output; weights in and out
        return dict(bytes=2.0 * rows * (2 * k + 2 * n) + 12.0 * k * n, flops=2 * _dense(rows, k, n))
    cfg, layers = _expected(case)
    elem = 2 if cfg.feat_dtype == "bf16" else 4
    batches = case.get("batches", 1)
    if path == "sample":
        total = 0.0
        for l, (n_dst, n_src, nnz) in enumerate(layers):
            # ids and row pointers in; the chosen neighbours in and out, row pointers and frontier out
            total += 4 * n_dst + 16 * n_dst + 4 * nnz + 4 * nnz + 4 * n_dst
            if l > 0 or case["layout"] != "global":
                total += 4 * n_src
            if l > 0 or case["layout"] == "transposed":
                total += 4 * nnz + 4 * n_src
        return dict(bytes=total * batches, flops=0.0)
    if path == "gather":
        n_dst, n_src, nnz = layers[0]
        outs = 2 if case["model"] == "sage" else 1
        distinct = cfg.n_nodes * (1.0 - math.exp(-batches * n_src / cfg.n_nodes))
        return dict(bytes=distinct * cfg.n_feat * elem + batches * (4 * nnz + 8 * n_dst + outs * 2 * n_dst * cfg.n_feat), flops=batches * nnz * cfg.n_feat * 1.0)
    if path in ("sage", "gcn"):
        n_dst, n_src, nnz = layers[case["layer"]]
        n_op, h = (2 if path == "sage" else 1), cfg.hidden
        f_out = cfg.n_classes if case["layer"] == len(cfg.fanouts) - 1 else h
        moved = 2 * n_src * h * 2 + 4 * nnz * 2 + 2 * n_dst * (h + 2 * f_out) + 12 * n_op * h * f_out
        return dict(bytes=float(moved), flops=3 * _dense(n_dst, n_op * h, f_out) + 4.0 * nnz * h)
    if path == "gat":
        n_dst, n_src, nnz = layers[case["layer"]]
        f_in, h = (cfg.n_feat if case["layer"] == 0 else cfg.hidden), cfg.hidden
        moved = n_src * f_in * (elem if case["layer"] == 0 else 2) + 2 * n_src * h + 4 * n_dst * h + 8 * nnz + 12 * f_in * h
        return dict(bytes=float(moved), flops=(2 if case["layer"] == 0 else 3) * _dense(n_src, f_in, h) + 8.0 * nnz * h)
    # train: the input rows once per group, activations in and out once each way, weights
    flops = moved = 0.0
    n_op = 2 if case["model"] == "sage" else 1
    dims = synth.layer_dims(cfg)
    for l, ((f_in, f_out), (n_dst, n_src, nnz)) in enumerate(zip(dims, layers)):
        rows = n_src if case["model"] == "gat" else n_dst
        flops += (2 if l == 0 else 3) * _dense(rows, n_op * f_in, f_out) + (2 if l == 0 else 4) * nnz * f_in
        moved += 8 * nnz + (4 * n_src * f_in if l else 0) + 4 * n_dst * f_out + 12 * n_op * f_in * f_out
    n_src0 = layers[0][1]
    moved = moved * batches + cfg.n_nodes * (1.0 - math.exp(-batches * n_src0 / cfg.n_nodes)) * cfg.n_feat * elem
    return dict(bytes=float(moved), flops=float(flops * batches))


def tolerance(case):
    if case["path"] in ("roots", "sample"):
        return "exact"
    if case["path"] == "train":      # roundings of one layer travel through the next ones and through the steps
        return {"rel": 1e-2, "max": 0.2}
    # bf16 operands, float sums, bf16 results: a result rounded once is 1.7e-3 off in the 2-norm, one that is computed
    # from rounded ones 2e-3 to 3e-3
    return {"rel": 8e-3, "max": 0.1}


# ------------------------------------------------------------------------------------------------ the same in 64 bits
def _edges(blk, g=0):
    """(destination row, local source, global source or None) of every edge of a block, on the GPU."""
    n_dst, _, nnz = _header(blk, g)
    ptr = blk.indptr[g, :n_dst + 1].to(torch.int64)
    rows = torch.repeat_interleave(torch.arange(n_dst, device=DEV), ptr[1:] - ptr[:-1])
    return rows, blk.indices[g, :nnz].to(torch.int64), blk.gather_ids[g, :nnz].to(torch.int64) if blk.gather_ids is not None else None


def _f64(t):
    return _as_bf16(t).double() if t.dtype == torch.int16 else t.double()


def _sum_rows(n, rows, values):
    return torch.zeros((n, values.shape[1]), dtype=torch.float64, device=DEV).index_add_(0, rows, values)


def _pad(x, rows, cols):
    out = torch.zeros((rows, cols), dtype=torch.float64, device=DEV)
    out[:x.shape[0], :x.shape[1]] = x
    return out


def _bf16_weights(lay):
    return lay.W.to(torch.bfloat16).double()                     # the products take their weights in bf16


def _step(lay, dW, db):
    W = lay.W.double() * (1 - LR * DECAY) - LR * dW
    bias = None if lay.bias is None else lay.bias.double()
    if bias is not None and db is not None:
        bias[:db.numel()] -= LR * db
    return W, bias


def exact(case, seed):
    path = case["path"]
    if path == "train":
        return _exact_train(case, seed) if case["model"] == "sage" and case["batches"] <= 2 and case["graph"] != "papers" else None
    if path not in ("gather", "input", "sage", "gcn", "gat"):
        return None
    s = prepare(case, seed)
    torch.cuda.synchronize()
    if path == "gather":
        return _exact_gather(s)
    if path == "input":
        lay, n = s["lay"], case["rows"]
        x = torch.cat([_f64(t[:n, :case["f_in"]]) for t in (s["x_self"], s["x_agg"]) if t is not None], 1)
        out = (x @ _bf16_weights(lay) + lay.bias[:lay.F_out].double()).clamp_min(0)
        dz = _f64(s["dz"][:n, :lay.F_out])
        W, bias = _step(lay, x.t() @ dz, dz.sum(0))
        return _pad(out, case["cap"], lay.N_pad), W, bias
    if path == "gat":
        return _exact_gat(s)
    return _exact_layer(s, path == "gcn")


def _exact_gather(s):
    case, cfg, blk, feats = s["case"], s["cfg"], s["blocks"][0], s["w"].features
    agg = torch.zeros(s["agg"].shape, dtype=torch.float64, device=DEV)
    own = torch.zeros_like(agg) if case["model"] == "sage" else None
    deg = (s["w"].indptr[1:] - s["w"].indptr[:-1]).double()
    for g in range(s["batches"]):
        n_dst, _, _ = _header(blk, g)
        rows, _, ids = _edges(blk, g)
        dst = blk.src_ids[g, :n_dst].to(torch.int64)
        count = torch.bincount(rows, minlength=n_dst).double().clamp_min(1).unsqueeze(1)
        for c in range(0, cfg.n_feat, 128):                      # by columns: a whole block in 64 bits is large
            cols = slice(c, min(c + 128, cfg.n_feat))
            x, me = _f64(feats[:, cols][ids].contiguous()), _f64(feats[:, cols][dst].contiguous())
            if case["model"] == "sage":
                agg[g, :n_dst, cols] = _sum_rows(n_dst, rows, x) / count
                own[g, :n_dst, cols] = me
            else:
                v = (deg[dst] + 1).unsqueeze(1)
                near = _sum_rows(n_dst, rows, x / (deg[ids] + 1).sqrt().unsqueeze(1))
                agg[g, :n_dst, cols] = me / v + deg[dst].unsqueeze(1) / count / v.sqrt() * near
    return (agg, own) if own is not None else agg


def _exact_layer(s, gcn):
    cfg, blk, lay, top, n_dst, n_src = s["cfg"], s["blk"], s["lay"], s["top"], s["n_dst"], s["n_src"]
    H, F, wide = cfg.hidden, lay.F_out, lay.F_pad
    rows, src, _ = _edges(blk)
    h = _f64(s["h"][:n_src, :H])
    count = torch.bincount(rows, minlength=n_dst).double().clamp_min(1)
    if gcn:
        ids = blk.src_ids[0, :n_src].to(torch.int64)
        deg = (s["w"].indptr[1:] - s["w"].indptr[:-1]).double()[ids]
        w_src, w_dst = 1 / (deg + 1).sqrt(), deg[:n_dst] / count / (deg[:n_dst] + 1).sqrt()
        edge, own = w_dst[rows] * w_src[src], 1 / (deg[:n_dst] + 1)
    else:
        edge, own = (1 / count)[rows], torch.zeros(n_dst, dtype=torch.float64, device=DEV)
    agg = _sum_rows(n_dst, rows, h[src] * edge.unsqueeze(1)) + h[:n_dst] * own.unsqueeze(1)
    x = agg if gcn else torch.cat([h[:n_dst], agg], 1)
    Wb = _bf16_weights(lay)
    out = x @ Wb + lay.bias[:F].double()
    if top:
        labels = s["w"].labels[blk.src_ids[0, :n_dst].to(torch.int64)].to(torch.int64)
        logp = torch.log_softmax(out, 1)
        loss = -logp.gather(1, labels.unsqueeze(1)).mean().reshape(1)
        dz = logp.exp()
        dz[torch.arange(n_dst, device=DEV), labels] -= 1
        dz /= n_dst
    else:
        out, dz = out.clamp_min(0), _f64(s["dz"][:n_dst, :F])
    W, bias = _step(lay, x.t() @ dz, dz.sum(0))
    d_in = dz @ Wb.t()
    d_agg = d_in if gcn else d_in[:, H:]
    d_src = _sum_rows(n_src, src, d_agg[rows] * edge.unsqueeze(1))
    d_src[:n_dst] += d_agg * own.unsqueeze(1) if gcn else d_in[:, :H]
    d_src = d_src * (h > 0)
    got = [_pad(agg, blk.cap_dst, wide), _pad(out, blk.cap_dst, lay.N_pad), _pad(d_src, blk.cap_src, wide), W, bias]
    return got + ([loss, _pad(dz, blk.cap_dst, lay.N_pad)] if top else [])


def _exact_gat(s):
    cfg, blk, lay, par, n_dst, n_src = s["cfg"], s["blk"], s["lay"], s["par"], s["n_dst"], s["n_src"]
    H, heads, f_in = cfg.hidden, s["case"]["heads"], s["f_in"]
    D = H // heads
    if _first_layer(s):                                         # the projection takes its rows in bf16
        feats, ids = s["w"].features, blk.src_ids[0, :n_src].to(torch.int64)
        x = feats[ids, :f_in]
        x = _as_bf16(x).double() if x.dtype == torch.int16 else x.to(torch.bfloat16).double()
    else:
        x = _f64(s["x"][:n_src, :f_in])
    Wb = _bf16_weights(lay)
    z = x @ Wb
    a_l, a_r, b = (par.attn[i, :H].double() for i in range(3))
    rows, src, _ = _edges(blk)
    zh = z.view(n_src, heads, D)
    score = (zh * a_l.view(heads, D)).sum(2)[src] + (zh * a_r.view(heads, D)).sum(2)[:n_dst][rows]
    e = torch.where(score > 0, score, score * par.slope)
    top = torch.full((n_dst, heads), -1e300, dtype=torch.float64, device=DEV).scatter_reduce_(0, rows.unsqueeze(1).expand(-1, heads), e, "amax")
    ex = (e - top[rows]).exp()
    alpha = ex / _sum_rows(n_dst, rows, ex)[rows]
    wide = lambda t: t.repeat_interleave(D, 1)                   # a value per head, repeated over its columns
    out = (_sum_rows(n_dst, rows, wide(alpha) * z[src]) + b).clamp_min(0)
    d_out = _f64(s["d_out"][:n_dst, :H]) * (_f64(s["relu_out"][:n_dst, :H]) > 0)
    d_alpha = (d_out[rows] * z[src]).view(-1, heads, D).sum(2)
    t = _sum_rows(n_dst, rows, alpha * d_alpha)
    d_score = alpha * (d_alpha - t[rows]) * torch.where(score > 0, 1.0, par.slope)
    d_el, d_er = _sum_rows(n_src, src, d_score), _sum_rows(n_dst, rows, d_score)
    dz = _sum_rows(n_src, src, wide(alpha) * d_out[rows]) + wide(d_el) * a_l
    dz[:n_dst] += wide(d_er) * a_r
    att = torch.zeros_like(par.attn, dtype=torch.float64)
    att[0, :H] = a_l * (1 - LR * DECAY) - LR * (wide(d_el) * z).sum(0)
    att[1, :H] = a_r * (1 - LR * DECAY) - LR * (wide(d_er) * z[:n_dst]).sum(0)
    att[2, :H] = b - LR * d_out.sum(0)
    W, _ = _step(lay, x.t() @ dz, None)
    got = [_pad(out, blk.cap_dst, lay.N_pad), _pad(dz, blk.cap_src, lay.N_pad), W, att]
    return got + ([_pad(dz @ Wb.t(), blk.cap_src, lay.F_pad)] if s["d_in"] is not None else [])


def _exact_train(case, seed):
    """GraphSAGE steps in 64 bits on the blocks the sampler gives (whole numbers, compared by themselves elsewhere)."""
    s = prepare(case, seed)
    tr, cfg = s["tr"], s["tr"].cfg
    flags = tr.sample_flags & ~B.CR_SAMPLE_INPUT_GLOBAL_IDS
    tr.sample_group(0, s["batches"], case["p"], 1, flags=flags)
    torch.cuda.synchronize()
    W = [lay.W.double() for lay in tr.layers]
    bias = [lay.bias[:lay.F_out].double() for lay in tr.layers]
    loss = out = None
    for g in range(s["batches"]):
        dst = [_header(b, g)[0] for b in tr.blocks]
        xs, hs = [], []
        blk0 = tr.blocks[0]
        h = _f64(tr.table[blk0.src_ids[g, :_header(blk0, g)[1]].to(torch.int64), :cfg.n_feat].contiguous())
        edges = []
        for l, blk in enumerate(tr.blocks):
            rows, src, _ = _edges(blk, g)
            inv = 1 / torch.bincount(rows, minlength=dst[l]).double().clamp_min(1)
            edges.append((rows, src, inv))
            x = torch.cat([h[:dst[l]], _sum_rows(dst[l], rows, h[src]) * inv.unsqueeze(1)], 1)
            hs.append(h)
            xs.append(x)
            h = x @ W[l].float().to(torch.bfloat16).double() + bias[l]
            if l < tr.L - 1:
                h = h.clamp_min(0)
        out = h
        labels = tr.labels[tr.blocks[-1].src_ids[g, :dst[-1]].to(torch.int64)].to(torch.int64)
        logp = torch.log_softmax(out, 1)
        loss = -logp.gather(1, labels.unsqueeze(1)).mean().reshape(1)
        dz = logp.exp()
        dz[torch.arange(dst[-1], device=DEV), labels] -= 1
        dz /= dst[-1]
        for l in range(tr.L - 1, -1, -1):
            d_in = dz @ W[l].float().to(torch.bfloat16).double().t()
            W[l] = W[l] * (1 - LR * DECAY) - LR * (xs[l].t() @ dz)
            bias[l] = bias[l] - LR * dz.sum(0)
            if l:
                rows, src, inv = edges[l]
                half = d_in.shape[1] // 2
                dz = _sum_rows(hs[l].shape[0], src, d_in[:, half:][rows] * inv[rows].unsqueeze(1))
                dz[:dst[l]] += d_in[:, :half]
                dz = dz * (hs[l] > 0)
    return [_pad(out, tr.out[-1].shape[0], tr.layers[-1].N_pad), loss] + W
