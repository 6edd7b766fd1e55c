"""The work that a user of this library has it do, as cases that can be timed.

A case is a dict of plain values.  Its `kind` says which calls one pass makes, in the order in which a speculative
decoder makes them:

  layer    top-p selection of one layer's draft rows, then sparse attention over the lists (single positions or
           chunks; contiguous cache or paged pool; with or without the new tokens behind the cache)
  step     one verify step: one batched selection for the rows of all mapped layers, then the attention of layer
           after layer - over index lists (`route` "list") or through the fused call over the kept mask ("mask")
  dense    attention of a layer that is kept dense (no list)
  union    selection of every draft step and draft head with the union of the kept sets, then attention over it
  mapping  the offline layer mapping of a model pair: similarity matrix and monotonic alignment

Draft rows follow the recipe of `paper_2510_27641_amd.workloads` (sink, recency band, log-normal or heavy-tailed bulk,
sparse strongly attended positions), drawn on the device; Q, K and V are N(0, 1).
"""
import math

import numpy as np
import torch

from paper_2510_27641_amd import binding as sa
from paper_2510_27641_amd import workloads as W

PAGE = W.PAGE_SIZE
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
ELEM_BYTES = {"f32": 4, "bf16": 2, "f16": 2}


def _layer(name, dtype, d, B, H_q, H_kv, T, n, top_p, *, chunk=1, paged=False, ragged=False, new_tokens=False, lowp=False,
           tail="normal"):
    return dict(name=name, kind="layer", dtype=dtype, d=d, B=B, H_q=H_q, H_kv=H_kv, T=T, n=n, top_p=top_p, chunk=chunk,
                paged=paged, ragged=ragged, new_tokens=new_tokens, lowp=lowp, tail=tail)


def _step(name, route, layers, B, n, top_p, dtype="bf16", H_q=32, H_kv=8, T=5, d=128):
    return dict(name=name, kind="step", route=route, layers=layers, dtype=dtype, d=d, B=B, H_q=H_q, H_kv=H_kv, T=T, n=n,
                top_p=top_p, tail="normal")


def _dense(name, dtype, B, n, ragged, H_q=32, H_kv=8, T=5, d=128):
    return dict(name=name, kind="dense", dtype=dtype, d=d, B=B, H_q=H_q, H_kv=H_kv, T=T, n=n, ragged=ragged)


def _union(name, B, H_draft, S, n, top_p, dtype="bf16", H_q=32, H_kv=8, T=5, d=128):
    return dict(name=name, kind="union", dtype=dtype, d=d, B=B, H_q=H_q, H_kv=H_kv, T=T, n=n, H_draft=H_draft, S=S,
                top_p=top_p, tail="normal")


def _mapping(name, m, n_layers, rows, L):
    return dict(name=name, kind="mapping", m=m, n_layers=n_layers, rows=rows, L=L)


def listed():
    return [
        # The smallest call: one sequence, fp32, 64-wide heads, a context of 1024 - what a first integration and every
        # parity check run.  Latency and launches are all there is to it.
        _layer("tiny_fp32", "f32", 64, 1, 8, 8, 5, 1024, 0.9),
        # The paper's own setting: 32 heads without grouping, fp16, a context just short of 2048, chunks of 16
        # positions, the tokens being verified behind the cache and an output copy for the next projection.
        _layer("paper_2k_chunks", "f16", 128, 1, 32, 32, 5, 2044, 0.97, chunk=16, new_tokens=True, lowp=True),
        # One layer of a single interactive session: one sequence of 8192 tokens, grouped heads, bf16.
        _layer("single_8k", "bf16", 128, 1, 32, 8, 5, 8192, 0.95),
        # A small verifier: 64-wide heads in groups of 8, bf16, a small batch at an ordinary length.
        _layer("small_heads_8k", "bf16", 64, 4, 32, 4, 5, 8192, 0.9),
        # A larger verifier with 8 query heads per kv head (40 query rows each with 5 tokens), at a length that is no
        # multiple of anything: contexts grow token by token.
        _layer("wide_group_13k", "bf16", 128, 8, 64, 8, 5, 13001, 0.95),
        # The headline workload: verify step of a batch of 8 at 32768 positions, selection of all layers in one call.
        # (16 layers: twice that is the same again.)
        _step("step_32k", "list", 16, 8, 32768, 0.9),
        # The same through the fused call, which never has an index list.
        _step("step_32k_fused", "mask", 16, 8, 32768, 0.9),
        # Long documents: few rows of 131072 positions with heavy-tailed logits.
        _layer("long_128k", "bf16", 128, 4, 32, 8, 5, 131072, 0.9, tail="heavy"),
        # A serving batch: 64 sequences of very different lengths over a shared pool of 16-token pages.
        _layer("ragged_paged", "bf16", 128, 64, 32, 8, 5, 65536, 0.95, paged=True, ragged=True),
        # The first layers of the verifier, which stay dense: a batch of sequences of different lengths.
        _dense("dense_first_layers", "bf16", 8, 32768, True),
        # Algorithm 2 as a whole: four draft steps, four draft heads per kv head, union of the kept sets.
        _union("union_4x4", 8, 32, 4, 32768, 0.9),
        # Offline, once per model pair: which draft layer serves which verifier layer (22 against 32 layers).
        _mapping("layer_mapping", 22, 32, 64, 2048),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    p = round(rng.uniform(0.8, 0.99), 3)
    pick = rng.random()
    if pick < 0.10:                                            # fp32, both head sizes
        d = rng.choice([64, 128])
        H_kv = rng.choice([4, 8])
        return _layer("", "f32", d, rng.randint(1, 4), H_kv * rng.choice([1, 2, 4]), H_kv, rng.randint(1, 8), _log_int(rng, 256, 8192), p)
    if pick < 0.20:                                            # short contexts in chunks, new tokens behind the cache
        H_kv = rng.choice([8, 32])
        return _layer("", rng.choice(["f16", "bf16"]), 128, rng.randint(1, 8), 32, H_kv, rng.randint(2, 6), _log_int(rng, 512, 16384), p,
                      chunk=rng.choice([8, 16, 32]), new_tokens=True, lowp=rng.random() < 0.5)
    if pick < 0.35:                                            # single sessions and small batches, any length
        return _layer("", rng.choice(["bf16", "f16"]), 128, rng.randint(1, 4), 32, 8, rng.randint(1, 8), _log_int(rng, 1024, 65536), p,
                      new_tokens=rng.random() < 0.3)
    if pick < 0.45:                                            # 64-wide heads
        H_kv = rng.choice([4, 8])
        return _layer("", rng.choice(["bf16", "f16"]), 64, rng.randint(1, 8), 32, H_kv, rng.randint(1, 8), _log_int(rng, 1024, 16384), p)
    if pick < 0.55:                                            # large groups of query heads
        return _layer("", "bf16", 128, rng.randint(1, 8), rng.choice([64, 128]), 8, rng.randint(3, 8), _log_int(rng, 2048, 32768), p)
    if pick < 0.70:                                            # verify steps
        return _step("", rng.choice(["list", "mask"]), rng.randint(4, 12), rng.randint(1, 8), _log_int(rng, 4096, 32768), p)
    if pick < 0.78:                                            # long documents
        return _layer("", "bf16", 128, rng.randint(1, 4), 32, 8, rng.randint(1, 6), _log_int(rng, 65536, 262144), p, tail="heavy")
    if pick < 0.86:                                            # serving batches
        return _layer("", "bf16", 128, _log_int(rng, 8, 64), 32, 8, rng.randint(1, 6), PAGE * _log_int(rng, 512, 4096), p, paged=True, ragged=True)
    if pick < 0.92:                                            # dense layers
        return _dense("", rng.choice(["bf16", "f16"]), rng.randint(1, 8), _log_int(rng, 1024, 32768), rng.random() < 0.5, T=rng.randint(1, 6))
    if pick < 0.97:                                            # unions
        return _union("", rng.randint(1, 8), rng.choice([8, 16, 32]), rng.randint(2, 6), _log_int(rng, 2048, 32768), p)
    return _mapping("", rng.randint(8, 32), rng.randint(12, 48), _log_int(rng, 16, 96), _log_int(rng, 512, 2048))


def draw(rng):
    most = max(work(c)["bytes"] for c in listed())
    while True:
        case = _draw_once(rng)
        if work(case)["bytes"] <= most:
            del case["name"]
            return case


# ------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------
def _bulk(gen, shape, tail):
    z = torch.randn(shape, generator=gen, device="cuda")
    if tail == "heavy":                                        # Student-t with 3 degrees of freedom, clipped
        chi = torch.randn((3, *shape), generator=gen, device="cuda").square_().sum(0)
        return (2.0 * z / (chi / 3.0).sqrt()).clamp_(-8.0, 8.0)
    return 2.0 * z


def _shape_rows(gen, logit, lens, tail):
    """Sink, recency band and strongly attended positions on rows of bulk logits [rows, n]; positions at and beyond a
    row's length become -inf."""
    rows, n = logit.shape
    pos = torch.arange(n, device="cuda")
    end = torch.full((rows, 1), n, device="cuda") if lens is None else lens.view(-1, 1)
    logit[:, 0] += 6.0
    logit += 3.0 * ((pos >= end - 64) & (pos < end))
    k = n // 100 if tail == "normal" else 0
    if k > 0:
        width = n // k                                         # one strongly attended position per stretch of the row
        where = torch.arange(k, device="cuda") * width + (torch.rand((rows, k), generator=gen, device="cuda") * width).long().clamp_(max=width - 1)
        rank = torch.rand((rows, k), generator=gen, device="cuda").argsort(1).float() + 1.0
        logit.scatter_add_(1, where, 4.0 * rank.pow(-1.1))
    if lens is not None:
        logit.masked_fill_(pos >= end, -math.inf)
    return logit


def _draft_rows(gen, rows, n, *, lens=None, tail="normal"):
    out = torch.empty((rows, n), device="cuda")
    per = max(1, (1 << 26) // n)
    for r in range(0, rows, per):
        m = min(per, rows - r)
        out[r:r + m] = _shape_rows(gen, _bulk(gen, (m, n), tail), None if lens is None else lens[r:r + m], tail).softmax(1)
    return out


def _step_rows(gen, B, H_draft, S, n):
    """[B, H_draft, S, n]: the rows of one (sequence, head) share their logits up to a perturbation per step."""
    out = torch.empty((B, H_draft, S, n), device="cuda")
    for b in range(B):
        base = _shape_rows(gen, _bulk(gen, (H_draft, n), "normal"), None, "normal")
        out[b] = (base[:, None, :] + 0.7 * torch.randn((H_draft, S, n), generator=gen, device="cuda")).softmax(2)
    return out


def _normal(gen, shape, dtype):
    return torch.empty(shape, dtype=DTYPES[dtype], device="cuda").normal_(generator=gen)


def _bind_workspace(args, nbytes):
    ws = sa.alloc_workspace(nbytes)
    args.workspace, args.workspace_bytes = ws.data_ptr(), ws.numel()
    return ws


def _lens(rng, case):
    """Lengths of a ragged batch: uniform from a sixteenth of the longest to the longest."""
    if not case["ragged"]:
        return None
    lens = rng.integers(max(1, case["n"] // 16), case["n"] + 1, size=case["B"])
    lens[int(rng.integers(case["B"]))] = case["n"]
    return lens.astype(np.int32)


def _prepare_layer(case, seed, gen):
    B, H_q, H_kv, T, d, n = (case[k] for k in ("B", "H_q", "H_kv", "T", "d", "n"))
    rng = np.random.default_rng(seed)
    lens = _lens(rng, case)
    sl = None if lens is None else torch.from_numpy(lens).cuda()
    row_lens = None if sl is None else sl.long().repeat_interleave(H_kv)
    probs = _draft_rows(gen, B * H_kv, n, lens=row_lens, tail=case["tail"]).view(B, H_kv, n)
    chunk = case["chunk"]
    cap = -(-n // chunk)
    idx = torch.zeros((B * H_kv, cap), dtype=torch.int32, device="cuda")
    counts = torch.zeros(B * H_kv, dtype=torch.int32, device="cuda")
    sel = sa.select_args(probs, case["top_p"], indices=idx, counts=counts, seq_lens=sl, chunk_size=chunk if chunk > 1 else 0)
    need = sa.specattn_workspace_size(sel, None)
    sel_ws = sa.alloc_workspace(need) if need else None

    q = _normal(gen, (B, H_q, T, d), case["dtype"])
    extra = {}
    if case["paged"]:
        pages = -(-lens // PAGE)
        total = int(pages.sum())
        table = np.zeros((B, -(-n // PAGE)), dtype=np.int32)
        perm = rng.permutation(total).astype(np.int32)
        at = 0
        for b in range(B):
            table[b, :pages[b]] = perm[at:at + pages[b]]
            at += int(pages[b])
        shape = (total, H_kv, PAGE, d)
        extra = dict(page_table=torch.from_numpy(table).cuda(), page_size=PAGE, n_max=n)
    else:
        shape = (B, H_kv, n, d)
    k, v = _normal(gen, shape, case["dtype"]), _normal(gen, shape, case["dtype"])
    if case["new_tokens"]:
        extra.update(k_new=_normal(gen, (B, H_kv, T, d), case["dtype"]), v_new=_normal(gen, (B, H_kv, T, d), case["dtype"]))
    out = torch.zeros((B, H_q, T, d), dtype=torch.float32, device="cuda")
    outputs = [idx, counts, out]
    if case["lowp"]:
        extra["out_lowp"] = torch.zeros((B, H_q, T, d), dtype=DTYPES[case["dtype"]], device="cuda")
        outputs.append(extra["out_lowp"])
    attn = sa.attn_args(q, k, v, out=out, indices=idx, counts=counts, seq_lens=sl, chunk_size=chunk if chunk > 1 else 0, **extra)
    ws = _bind_workspace(attn, sa.specattn_workspace_size(None, attn))
    return dict(kind="layer", sel=sel, sel_ws=sel_ws, attn=attn, outputs=outputs, keep=(probs, sl, q, k, v, ws, extra))


def _prepare_step(case, seed, gen):
    L, B, H_q, H_kv, T, d, n = (case[k] for k in ("layers", "B", "H_q", "H_kv", "T", "d", "n"))
    R = B * H_kv
    probs = _draft_rows(gen, L * R, n).view(L * B, H_kv, n)
    q = _normal(gen, (L * B, H_q, T, d), case["dtype"])
    k, v = _normal(gen, (L * B, H_kv, n, d), case["dtype"]), _normal(gen, (L * B, H_kv, n, d), case["dtype"])
    out = torch.zeros((L * B, H_q, T, d), dtype=torch.float32, device="cuda")
    counts = torch.zeros(L * R, dtype=torch.int32, device="cuda")
    part = lambda l: slice(l * B, (l + 1) * B)
    rows = lambda l: slice(l * R, (l + 1) * R)
    calls = []
    if case["route"] == "list":
        idx = torch.zeros((L * R, n), dtype=torch.int32, device="cuda")
        sel = sa.select_args(probs, case["top_p"], indices=idx, counts=counts)
        for l in range(L):
            calls.append((sa.attn_args(q[part(l)], k[part(l)], v[part(l)], out=out[part(l)], indices=idx[rows(l)], counts=counts[rows(l)]),))
        need = sa.specattn_workspace_size(None, calls[0][0])
        outputs = [idx, counts, out]
    else:
        blocks = -(-n // sa.SEL_BLOCK)
        tau = torch.zeros(L * R, dtype=torch.float32, device="cuda")
        bc = torch.zeros((L * R, blocks), dtype=torch.int32, device="cuda")
        mask = torch.zeros((L * R, blocks * (sa.SEL_BLOCK // 32)), dtype=torch.int32, device="cuda")
        state = dict(indices=None, thresholds=tau, block_counts=bc, kept_mask=mask)
        sel = sa.select_args(probs, case["top_p"], counts=counts, **state)
        for l in range(L):
            s = sa.select_args(probs[part(l)], case["top_p"], indices=None, counts=counts[rows(l)], thresholds=tau[rows(l)],
                               block_counts=bc[rows(l)], kept_mask=mask[rows(l)], reuse_selection=True)
            calls.append((s, sa.attn_args(q[part(l)], k[part(l)], v[part(l)], out=out[part(l)])))
        need = sa.specattn_workspace_size(*calls[0])
        outputs = [counts, tau, bc, mask, out]
    ws = sa.alloc_workspace(need)
    for c in calls:
        c[-1].workspace, c[-1].workspace_bytes = ws.data_ptr(), ws.numel()
    need = sa.specattn_workspace_size(sel, None) if case["route"] == "list" else 0
    sel_ws = sa.alloc_workspace(need) if need else None
    return dict(kind="step", sel=sel, sel_ws=sel_ws, calls=calls, outputs=outputs, keep=(probs, q, k, v, ws))


def _prepare_dense(case, seed, gen):
    B, H_q, H_kv, T, d, n = (case[k] for k in ("B", "H_q", "H_kv", "T", "d", "n"))
    lens = _lens(np.random.default_rng(seed), case)
    sl = None if lens is None else torch.from_numpy(lens).cuda()
    q = _normal(gen, (B, H_q, T, d), case["dtype"])
    k, v = _normal(gen, (B, H_kv, n, d), case["dtype"]), _normal(gen, (B, H_kv, n, d), case["dtype"])
    k_new, v_new = _normal(gen, (B, H_kv, T, d), case["dtype"]), _normal(gen, (B, H_kv, T, d), case["dtype"])
    out = torch.zeros((B, H_q, T, d), dtype=torch.float32, device="cuda")
    attn = sa.attn_args(q, k, v, out=out, seq_lens=sl, k_new=k_new, v_new=v_new)
    ws = _bind_workspace(attn, sa.specattn_workspace_size(None, attn))
    return dict(kind="dense", attn=attn, outputs=[out], keep=(q, k, v, k_new, v_new, sl, ws))


def _prepare_union(case, seed, gen):
    B, H_q, H_kv, T, d, n = (case[k] for k in ("B", "H_q", "H_kv", "T", "d", "n"))
    probs = _step_rows(gen, B, case["H_draft"], case["S"], n)
    idx = torch.zeros((B * H_kv, n), dtype=torch.int32, device="cuda")
    counts = torch.zeros(B * H_kv, dtype=torch.int32, device="cuda")
    uni = sa.union_args(probs, case["top_p"], H_kv, indices=idx, counts=counts)
    uni_ws = sa.alloc_workspace(sa.specattn_union_workspace_size(uni))
    q = _normal(gen, (B, H_q, T, d), case["dtype"])
    k, v = _normal(gen, (B, H_kv, n, d), case["dtype"]), _normal(gen, (B, H_kv, n, d), case["dtype"])
    out = torch.zeros((B, H_q, T, d), dtype=torch.float32, device="cuda")
    attn = sa.attn_args(q, k, v, out=out, indices=idx, counts=counts)
    ws = _bind_workspace(attn, sa.specattn_workspace_size(None, attn))
    return dict(kind="union", union=uni, union_ws=uni_ws, attn=attn, outputs=[idx, counts, out], keep=(probs, q, k, v, ws))


def _attention_maps(gen, layers, lens, content, L):
    """Causal attention rows of a model (the device counterpart of workloads.layer_attention_maps): a sink that grows
    and a recency window that narrows with depth, content positions shared by both models, noise per layer."""
    rows = lens.numel()
    pos = torch.arange(L, device="cuda")
    out = torch.empty((layers, rows, L), device="cuda")
    for i in range(layers):
        t = i / max(layers - 1, 1)
        logit = 0.5 * torch.randn((rows, L), generator=gen, device="cuda")
        logit[:, 0] += 2.0 + 4.0 * t
        width = (lens * (0.25 - 0.2 * t)).round().clamp_(min=2.0)
        logit += 2.0 * ((pos >= (lens - width).view(-1, 1)) & (pos < lens.view(-1, 1)))
        logit.scatter_add_(1, content, torch.full(content.shape, 1.0 + 3.0 * math.sin(math.pi * t), device="cuda"))
        logit.masked_fill_(pos >= lens.view(-1, 1), -math.inf)
        out[i] = logit.softmax(1)
    return out


def _prepare_mapping(case, seed, gen):
    m, n, rows, L = case["m"], case["n_layers"], case["rows"], case["L"]
    lens = torch.randint(max(8, L // 8), L + 1, (rows,), generator=gen, device="cuda").float()
    # eight different positions per row: one in each eighth of what the row sees
    content = ((torch.arange(8, device="cuda") + torch.rand((rows, 8), generator=gen, device="cuda") * 0.99) * (lens // 8).view(-1, 1)).long()
    draft, verifier = _attention_maps(gen, m, lens, content, L), _attention_maps(gen, n, lens, content, L)
    S = torch.zeros((m, n), dtype=torch.float64, device="cuda")
    f = torch.zeros(n, dtype=torch.int32, device="cuda")
    total = torch.zeros(1, dtype=torch.float64, device="cuda")
    ws = sa.alloc_workspace(int(sa.load().specattn_layer_similarity_workspace_size(m, n, rows, L)))
    ws_map = sa.alloc_workspace(int(sa.load().specattn_layer_map_workspace_size(m, n)))
    return dict(kind="mapping", args=(draft, verifier, S, ws), map_args=(S, f, total, ws_map), outputs=[S, f, total])


_PREPARE = dict(layer=_prepare_layer, step=_prepare_step, dense=_prepare_dense, union=_prepare_union, mapping=_prepare_mapping)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return _PREPARE[case["kind"]](case, seed, gen)


def run(state):
    kind = state["kind"]
    if kind == "layer":
        sa.specattn_topp_select(state["sel"], state["sel_ws"])
        sa.specattn_sparse_decode_attn(state["attn"])
    elif kind == "step":
        sa.specattn_topp_select(state["sel"], state["sel_ws"])
        for call in state["calls"]:
            if len(call) == 1:
                sa.specattn_sparse_decode_attn(call[0])
            else:
                sa.specattn_fused(*call)
    elif kind == "dense":
        sa.specattn_sparse_decode_attn(state["attn"])
    elif kind == "union":
        sa.specattn_topp_select_union(state["union"], state["union_ws"])
        sa.specattn_sparse_decode_attn(state["attn"])
    else:
        sa.specattn_layer_similarity(*state["args"])
        sa.specattn_layer_map(*state["map_args"])
    return state["outputs"]


# ------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------
def _kept(rows, top_p):
    """Boolean kept sets of rows of scores, by sorting."""
    order = np.argsort(-rows, axis=-1, kind="stable")
    mass = np.cumsum(np.take_along_axis(rows, order, -1), -1, dtype=np.float64)
    need = (mass < top_p * mass[..., -1:]).sum(-1) + 1
    rank = np.empty_like(order)
    np.put_along_axis(rank, order, np.broadcast_to(np.arange(rows.shape[-1]), rows.shape), -1)
    return rank < need[..., None]


def _kept_fraction(case, n):
    """Share of n positions that the recipe's rows keep, from a few rows drawn on the host."""
    rng = np.random.default_rng(0)
    if case["kind"] == "union":
        rows = W.draft_step_probs(rng, 1, case["H_draft"] // case["H_kv"], case["S"], n)
        return float(_kept(rows, case["top_p"]).any(axis=(0, 1, 2)).mean())
    heavy = dict(student_t_nu=3.0, logit_clip=8.0, spike_frac=0.0) if case["tail"] == "heavy" else {}
    rows = W.draft_probs(rng, 2, n, **heavy)
    chunk = case.get("chunk", 1)
    if chunk > 1:
        rows = np.pad(rows, ((0, 0), (0, -n % chunk))).reshape(2, -1, chunk).sum(-1)
    return float(_kept(rows, case["top_p"]).mean())


def work(case):
    """Draft rows read once and lists (or mask) written once; the K and V rows of the kept positions and Q read once,
    the output written once.  Two products of 2 * d operations per query row and kept position."""
    if case["kind"] == "mapping":
        m, n, E = case["m"], case["n_layers"], case["rows"] * case["L"]
        # the maps in, the similarity out; a logarithm per entry and a multiply-add per term
        return {"bytes": 4 * (m + n) * E + 8 * m * n + 4 * n, "flops": 2 * m * n * E + (m + n) * E}
    B, H_q, H_kv, T, d, n = (case[k] for k in ("B", "H_q", "H_kv", "T", "d", "n"))
    es = ELEM_BYTES[case["dtype"]]
    mean_len = n * 17 / 32 if case.get("ragged") else n
    layers = case.get("layers", 1)
    positions = layers * B * H_kv * mean_len
    bytes_ = layers * B * H_q * T * d * (es + 4)
    if case["kind"] == "dense":
        kept = positions
    else:
        kept = positions * _kept_fraction(case, int(mean_len))
        members = case["H_draft"] // H_kv * case["S"] if case["kind"] == "union" else 1
        bytes_ += 4 * members * positions
        bytes_ += positions / 8 if case.get("route") == "mask" else 4 * kept / case.get("chunk", 1)
    if case.get("new_tokens") or case["kind"] == "dense":
        bytes_ += 2 * B * H_kv * T * d * es
    if case.get("lowp"):
        bytes_ += B * H_q * T * d * es
    bytes_ += kept * 2 * d * es
    return {"bytes": int(bytes_), "flops": int(kept * (H_q // H_kv) * T * 4 * d)}


def tolerance(case):
    """Lists, counts, masks and maps are exact.  Attention against the same path in 64 bits: 2.2e-7 to 4.8e-7 where the
    weights keep 22 bits or more (fp32, fp16, and bf16 with 64-wide heads), 1.6e-6 to 2.4e-6 for bf16 with 128-wide
    heads; the output copy in the inputs' type moves by 1.6e-5 (fp16) and 6.4e-5 (bf16) where a value is rounded the
    other way.  Similarities with their sums split and reordered in 64 bits: 7e-14.  Stated: about four times that."""
    if case["kind"] == "mapping":
        return {"rel": 3e-13}
    short = case["dtype"] == "bf16" and case["d"] == 128
    if case.get("lowp"):
        return {"rel": 2.5e-4 if short else 6.5e-5}
    return {"rel": 1e-5 if short else 2e-6}
