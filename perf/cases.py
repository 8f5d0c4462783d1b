"""The work that programs have this library do, as cases to time.

A case names a mask family, its sizes and the path that is taken through the library's public entry points:

* ``forward``  attention over a mask whose block index the program already holds (one mask, many layers or calls);
* ``step``     a mask that is new in every call: block index, then the forward (decoding with a token tree, dynamic
               sparsity, the step that the benchmark's headline measures);
* ``layer``    forward and backward of one layer over a block index that the program holds (one mask for all layers);
* ``train``    as ``layer``, with the block index and the column list built in the call (packed batches: every batch has
               its own mask);
* ``reorder``  a very sparse mask with scattered entries: ordering, permuted mask and gathered rows, then the block
               index, the forward, and the output rows put back in the caller's order.

Masks come from the families of the benchmark and of the tests (`workloads/`): random blocks, packed sequences (causal,
or with a part of every sequence seen in both directions), a token tree behind a prefix, windows (plain and dilated),
a window with global tokens and random blocks, a power-law graph with locality, causal and all-ones masks.  They are
drawn on the GPU, so that making a state takes milliseconds.  Q, K, V and dO are N(0,1) in bf16, the only data type
that the library takes; head sizes 64 and 128; tile heights 64, 128 (the default) and 256; the softmax scale is
1/sqrt(d) unless the case has a sharper one.
"""
import math

import numpy as np
import torch

import paper_2409_15097_amd as bbm

BC = 64  # keys per block column

# What the reordered power-law graph needs, per query row: tiles of 128 x 64 that hold at least one edge, in keys.
GRAPH_KEYS = 3900.0


def listed():
    case = lambda name, path, family, B, H, Nq, Nk, d, **more: dict(  # noqa: E731
        name=name, path=path, family=family, B=B, H=H, Nq=Nq, Nk=Nk, d=d,
        **{**dict(masks=1, Br=128, sharper=1.0), **more})
    return [
        # the smallest call: a mask of two block rows and two heads, where launches and latency are all there is
        case("tiny-step", "step", "blocks", 1, 2, 256, 256, 64),
        # decoding with a candidate tree: 256 tree tokens of 8 sequences against a 1024-token prefix and themselves
        case("tree-decode", "step", "tree", 8, 32, 256, 1280, 128),
        # the same for one sequence with a long prefix: few query rows, very long lists
        case("tree-decode-long", "step", "tree", 1, 32, 256, 16640, 128),
        # prefill of prefix and tree together
        case("tree-prefill", "step", "tree", 8, 32, 1280, 1280, 128),
        # fine-tuning on packed sequences, a mask for every batch entry
        case("packed-train", "train", "packed", 4, 16, 4096, 4096, 64, masks=4),
        # the same with a length that no tile divides, the prompt part seen in both directions, and a sharper softmax
        case("packed-ragged-train", "train", "packed_bidir", 2, 12, 3001, 3001, 128, masks=2, sharper=1.5),
        # long-context training: window, global tokens and random blocks
        case("longctx-layer", "layer", "longctx", 1, 16, 16384, 16384, 64),
        # ordinary causal layers at both head sizes; the second is the largest case
        case("causal-layer-64", "layer", "causal", 4, 16, 4096, 4096, 64),
        case("causal-layer-128", "layer", "causal", 2, 32, 8192, 8192, 128),
        # nothing is masked: the plain attention forward
        case("dense-forward-128", "forward", "full", 2, 32, 8192, 8192, 128),
        # the headline workload of the benchmark: a graph whose nodes are already in a good order
        case("graph-step", "step", "graph", 1, 8, 32768, 32768, 64),
        # a graph as it arrives, its node labels scattered
        case("graph-reorder", "reorder", "graph", 1, 8, 32768, 32768, 64),
    ]


def _log_int(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi], odd ones among them."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    largest = work(next(c for c in listed() if c["name"] == "causal-layer-128"))
    while True:
        path = rng.choice(["forward", "step", "step", "layer", "layer", "train", "reorder"])
        d = rng.choice([64, 128])
        c = dict(path=path, d=d, B=_log_int(rng, 1, 8), H=_log_int(rng, 2, 32), masks=1, Br=rng.choice([128, 128, 128, 64, 256]),
                 sharper=rng.choice([1.0, 1.0, 1.0, 1.5, 2.5]))
        if path == "reorder":
            c.update(family="graph", B=1)
            c["Nq"] = c["Nk"] = _log_int(rng, 8192, 32768)
        elif path == "step" and rng.random() < 0.5:  # decoding: a tree behind a prefix
            tree = _log_int(rng, 16, 256)
            c.update(family="tree", Nq=tree, Nk=tree + _log_int(rng, 256, 32768))
        else:
            c["family"] = rng.choice(["blocks", "tree", "packed", "packed_bidir", "longctx", "window", "dilated", "causal", "full", "graph"])
            n = _log_int(rng, 8192, 32768) if c["family"] == "graph" else _log_int(rng, 256, 16384)
            if c["family"] in ("blocks", "longctx"):  # made of whole 64 x 64 blocks
                n = max(256, n // 64 * 64)
            c["Nq"] = c["Nk"] = n
            if c["family"] in ("packed", "packed_bidir"):
                c["masks"] = rng.choice([1, c["B"]])
        w = work(c)
        if (w["flops"] <= largest["flops"] and w["bytes"] <= 4 * largest["bytes"] and c["masks"] * c["Nq"] * c["Nk"] <= 1 << 30
                and c["B"] * c["H"] * c["Nk"] * d <= 1 << 27):
            return c


# ---- masks, on the GPU

def _packed_ids(N, rng):
    """Sequence number of every position (-1: padding) and its place in the sequence and the sequence's length."""
    hi = min(1024, max(16, N // 4))
    mu = 5.3 if N >= 4096 else math.log(max(20.0, N / 20.0))
    ids, place, length = (np.full(N, -1, dtype=np.int64) for _ in range(3))
    pos = n = 0
    while True:
        L = int(np.clip(np.rint(rng.lognormal(mu, 0.7)), 16, hi))
        if pos + L > N:
            return ids, place, length
        ids[pos:pos + L], place[pos:pos + L], length[pos:pos + L] = n, np.arange(L), L
        pos, n = pos + L, n + 1


def _tree_ancestors(T, rng):
    """[T, T]: token t sees its ancestors and itself, in a random tree of T nodes with at most four levels."""
    parent = np.full(T, -1, dtype=np.int64)
    level = np.zeros(T, dtype=np.int64)
    for t in range(1, T):
        p = int(rng.integers(-1, t))
        if p >= 0 and level[p] < 3:
            parent[t], level[t] = p, level[p] + 1
    sees = np.zeros((T, T), dtype=np.uint8)
    for t in range(T):
        if parent[t] >= 0:
            sees[t] = sees[parent[t]]
        sees[t, t] = 1
    return sees


def _graph(N, gen, scattered):
    """Power-law graph with locality and self loops: node i draws h_i neighbours within +-max(h_i, 8)."""
    f = min(1.0, 4.0 * N / 32768.0)
    xm, cap = 84.0 * f, int(2000 * f)
    u = torch.rand(N, generator=gen, device="cuda").clamp_(min=1e-6)
    h = torch.minimum((xm * u ** (-1.0 / 1.5)).floor(), torch.tensor(float(cap), device="cuda")).long()
    src = torch.repeat_interleave(torch.arange(N, device="cuda"), h)
    reach = torch.repeat_interleave(h.clamp(min=8), h)
    off = ((torch.rand(src.numel(), generator=gen, device="cuda") * 2 - 1) * (reach + 1)).floor().long()
    dst = (src + off).clamp_(0, N - 1)
    if scattered:
        label = torch.randperm(N, generator=gen, device="cuda")
        src, dst = label[src], label[dst]
    m = torch.zeros((N, N), dtype=torch.uint8, device="cuda")
    m[src, dst] = 1
    m[dst, src] = 1
    m.fill_diagonal_(1)
    return m


def _mask(case, seed, gen):
    family, Nq, Nk = case["family"], case["Nq"], case["Nk"]
    rng = np.random.Generator(np.random.PCG64(seed))
    i = torch.arange(Nq, device="cuda")[:, None]
    j = torch.arange(Nk, device="cuda")[None, :]
    if family == "packed" or family == "packed_bidir":
        out = torch.empty((case["masks"], Nq, Nk), dtype=torch.uint8, device="cuda")
        for m in range(case["masks"]):
            ids, place, length = (torch.from_numpy(x).cuda() for x in _packed_ids(Nq, rng))
            seen = i >= j
            if family == "packed_bidir":  # the first 40 % of a sequence attends in both directions
                prompt = place < (0.4 * length).round().long()
                seen = seen | (prompt[:, None] & prompt[None, :])
            out[m] = seen & (ids[:, None] == ids[None, :]) & (ids[:, None] >= 0)
        return out
    if family == "tree":
        tree = min(Nq, 256) if Nq != Nk else max(1, min(256, Nq // 5))
        full = (j <= i + (Nk - Nq)).to(torch.uint8)
        full[Nq - tree:, Nk - tree:] = torch.from_numpy(_tree_ancestors(tree, rng)).cuda()
        return full[None].contiguous()
    if family == "blocks":  # empty, full and half-full 64 x 64 blocks
        nb = Nq // 64
        kind = torch.rand((nb, nb), generator=gen, device="cuda").repeat_interleave(64, 0).repeat_interleave(64, 1)
        half = torch.rand((Nq, Nk), generator=gen, device="cuda") < 0.5
        return ((kind < 0.3) | ((kind < 0.6) & half) | (i == j)).to(torch.uint8)[None].contiguous()
    if family == "longctx":
        nb = Nq // 64
        m = ((i - j).abs() <= min(256, Nq // 16)) | (i < min(64, Nq // 16)) | (j < min(64, Nq // 16))
        pick = torch.zeros((nb, nb), dtype=torch.bool, device="cuda")
        pick.scatter_(1, torch.randint(0, nb, (nb, 3), generator=gen, device="cuda"), True)
        return (m | pick.repeat_interleave(64, 0).repeat_interleave(64, 1)).to(torch.uint8)[None].contiguous()
    if family == "window" or family == "dilated":
        w = 256 if Nq >= 16384 else max(32, Nq // 32)
        m = (i - j).abs() <= w if family == "window" else ((i - j).abs() <= 2 * w) & ((i - j) % 2 == 0)
        return m.to(torch.uint8)[None].contiguous()
    if family == "causal":
        return (i >= j).to(torch.uint8)[None].contiguous()
    if family == "full":
        return torch.ones((1, Nq, Nk), dtype=torch.uint8, device="cuda")
    return _graph(Nq, gen, scattered=case["path"] == "reorder")[None]


def _keys_per_row(case):
    """Keys that a query row meets, on average: allowed ones where the mask is made of runs or whole blocks, those of the
    tiles it cannot skip where single entries are scattered over them."""
    family, Nq, Nk = case["family"], case["Nq"], case["Nk"]
    if family in ("packed", "packed_bidir"):
        mean = min(1024, Nk / 4, math.exp((5.3 if Nq >= 4096 else math.log(max(20.0, Nq / 20.0))) + 1.5 * 0.49))
        return mean / 2 if family == "packed" else 0.58 * mean
    if family == "tree":
        return Nk - 128.0 if Nq != Nk else Nk / 2
    if family == "blocks":
        return 0.6 * Nk
    if family == "longctx":
        return min(Nk, 2 * min(256, Nq // 16) + 2 * min(64, Nq // 16) + 3 * 64)
    if family == "window" or family == "dilated":
        w = 256 if Nq >= 16384 else max(32, Nq // 32)
        return min(Nk, 2.0 * w if family == "window" else 4.0 * w)
    if family == "causal":
        return Nk / 2
    if family == "full":
        return float(Nk)
    return min(Nk, GRAPH_KEYS * min(1.0, 4.0 * Nk / 32768.0))


# ---- one pass

def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B, H, Nq, Nk, d, Br = (case[x] for x in ("B", "H", "Nq", "Nk", "d", "Br"))
    normal = lambda n: torch.randn((B, H, n, d), generator=gen, device="cuda").to(torch.bfloat16)  # noqa: E731
    s = dict(case=case, scale=case["sharper"] * d ** -0.5, q=normal(Nq), k=normal(Nk), v=normal(Nk), mask=_mask(case, seed, gen))
    backward = case["path"] in ("layer", "train")
    # the block index (for a path that rebuilds it, the tensors it is rebuilt in), outputs and workspaces
    s["idx"] = bbm.build_index(s["mask"], Br, BC, columns=backward)
    s["o"] = torch.empty_like(s["q"])
    s["lse"] = torch.empty((B, H, Nq), dtype=torch.float32, device="cuda")
    s["ws"] = torch.zeros(max(16, bbm.bbm_attn_fwd_workspace_bytes(B, H, Nq, d, Br, BC, bbm.BBM_MODE_AUTO)), dtype=torch.uint8, device="cuda")
    if backward:
        s["d_o"] = normal(Nq)
        s["dq"], s["dk"], s["dv"] = (torch.empty_like(s["q"]) for _ in range(3))
        s["ws_bwd"] = torch.zeros(bbm.bbm_attn_bwd_workspace_bytes(B, H, Nq, d, Br), dtype=torch.uint8, device="cuda")
    if case["path"] == "reorder":
        s["perm"] = torch.empty(Nq, dtype=torch.int32, device="cuda")
        s["ws_order"] = torch.empty(bbm.bbm_rcm_workspace_bytes(Nq), dtype=torch.uint8, device="cuda")
        s["mask_p"] = torch.empty_like(s["mask"])
        s["qp"], s["kp"], s["vp"], s["op"] = (torch.empty_like(s["q"]) for _ in range(4))
    return s


def run(s):
    path, idx, Br = s["case"]["path"], s["idx"], s["case"]["Br"]
    if path == "reorder":
        bbm.bbm_rcm_order(s["mask"][0], perm=s["perm"], workspace=s["ws_order"])
        bbm.bbm_permute_mask(s["mask"], s["perm"], out=s["mask_p"])
        for x, y in (("q", "qp"), ("k", "kp"), ("v", "vp")):
            bbm.bbm_gather_rows(s[x], s["perm"], out=s[y])
        bbm.build_index(s["mask_p"], Br, BC, idx=idx)
        bbm.bbm_attn_fwd(s["qp"], s["kp"], s["vp"], idx, softmax_scale=s["scale"], out=s["op"], lse=s["lse"], workspace=s["ws"])
        bbm.bbm_gather_rows(s["op"], s["perm"], inverse=True, out=s["o"])
        return dict(perm=s["perm"], mask=s["mask_p"], blocks=idx.blk_class, o=s["o"], lse=s["lse"])
    if path in ("step", "train"):
        bbm.build_index(s["mask"], Br, BC, idx=idx, columns=path == "train")
    bbm.bbm_attn_fwd_rect(s["q"], s["k"], s["v"], idx, softmax_scale=s["scale"], out=s["o"], lse=s["lse"], workspace=s["ws"])
    out = dict(o=s["o"], lse=s["lse"])
    if path in ("step", "train"):
        out.update(blocks=idx.blk_class, bin_blk_mat=idx.bin_blk_mat, offset=idx.offset, total_ones=idx.total_ones, row_ptr=idx.row_ptr)
    if path in ("layer", "train"):
        bbm.bbm_attn_bwd(s["q"], s["k"], s["v"], s["o"], s["d_o"], s["lse"], idx, softmax_scale=s["scale"],
                         dq=s["dq"], dk=s["dk"], dv=s["dv"], workspace=s["ws_bwd"])
        out.update(dq=s["dq"], dk=s["dk"], dv=s["dv"])
    return out


def work(case):
    """Two products in the forward, five in the backward, over the keys a row meets; every tensor once."""
    B, H, Nq, Nk, d, path = (case[x] for x in ("B", "H", "Nq", "Nk", "d", "path"))
    product = 2.0 * B * H * Nq * _keys_per_row(case) * d
    rows_q, rows_k = 2.0 * B * H * Nq * d, 2.0 * B * H * Nk * d  # bytes of Q, O, dQ .. and of K, V ..
    mask = float(case["masks"] * Nq * Nk)
    flops, nbytes = 2 * product, 2 * rows_q + 2 * rows_k + 4.0 * B * H * Nq
    if path in ("step", "train", "reorder"):
        nbytes += mask
    if path in ("layer", "train"):
        flops += 5 * product
        nbytes += 3 * rows_q + 2 * rows_k + 3 * rows_q  # Q, O, dO, K, V read, dQ, dK, dV written
    if path == "reorder":
        nbytes += 4 * 2 * rows_q  # three gathers and one scatter; the permuted mask is an output of the path
        nbytes += mask
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Four times the largest error seen against the same formulas in 64 bits, over all listed cases and 14 drawn ones
    # (first and last head).  Forward: O 2.9e-3 of its norm, single values 6.5e-2 of the larger of their size and the rms.
    # Backward: dQ 3.1e-3, dK 3.6e-3, dV 3.5e-3, single values 0.16 (a gradient is a sum of products of either sign).
    # Block classes, run index, list positions and the ordering are whole numbers and have to be the same.
    if case["path"] in ("layer", "train"):
        return {"rel": 1.4e-2, "max": 0.6}
    return {"rel": 1.2e-2, "max": 0.26}
