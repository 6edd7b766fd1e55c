#!/usr/bin/env python3
"""Benchmark of the SpecAttn hot path on one MI355X: top-p selection + sparse decode attention.

A "step" is one verify step of the 32-layer workload (Llama-3-8B-shaped layers, B=8, n=32768,
gamma=4, bf16 K/V, top_p=0.9): selection for the rows of all 32 mapped layers (one batched launch -
every layer's selection depends only on the draft model's output, Algorithm 1), then sparse attention
layer by layer (one launch sequence per layer, as a real verifier runs them).  Inputs are synthetic,
seeded, and resident in HBM before the timed region.

Prints ONE JSON line: selected-KV GB/s of the whole step (`value`), with the fused and unfused
paths, the roofline of the dominant kernel (HIP-event timed), and the CPU oracle timed on a bounded
sample of the same workload.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0     # MI355X HBM3E, published


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--layers", type=int, default=32)
    ap.add_argument("--batch", type=int, default=8)
    ap.add_argument("--context", type=int, default=32768)
    ap.add_argument("--top-p", type=float, default=0.9)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-other-configs", action="store_true", help="skip the bounded summary of the other configurations")
    ap.add_argument("--path", choices=["both", "unfused", "fused"], default="both")
    ap.add_argument("--workload", choices=["headline", "side"], default="headline",
                    help="headline: the 32-layer verify step (one JSON line).  side: the other workloads and calls "
                         "(8k layer, long-context sweep, ragged paged batch, dense, new tokens, chunks, union, large "
                         "GQA group, offline layer mapping), one JSON line each")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="also run one 1 GiB device copy (reference for rocprofv3 --pmc byte counters)")
    return ap.parse_args()


def side_workloads(torch, sa, W):
    """The workloads besides the headline one, and the calls beyond the selection + attention pair: HIP-event
    times of each call (mean of 20 after 3 warm-up calls, layer instances rotating so that nothing is served from
    the Infinity Cache unless the workload itself is that small)."""
    H_q, H_kv, T, d = 32, 8, 5, 128

    def timed(fn, reps=20, warm=3):
        for _ in range(warm):
            fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps * 1e3          # us

    def emit(name, **kw):
        print(json.dumps(dict(workload=name, **kw)), flush=True)

    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)

    def kv(shape):
        return (torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16),
                torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16))

    def pair(name, probs_np, top_p, B, n, *, H_q=H_q, seq_lens=None, page_table=None, pool_pages=0, copies=1):
        """selection + attention of one layer; `copies` layer instances are rotated through."""
        R = B * H_kv
        p = torch.from_numpy(probs_np).cuda()
        sl = None if seq_lens is None else torch.from_numpy(seq_lens.astype(np.int32)).cuda()
        pt = None if page_table is None else torch.from_numpy(page_table).cuda()
        idx = torch.empty((R, n), dtype=torch.int32, device="cuda")
        cnt = torch.zeros(R, dtype=torch.int32, device="cuda")
        s = sa.select_args(p, top_p, indices=idx, counts=cnt, seq_lens=sl)
        need = sa.specattn_workspace_size(s, None)
        ws_s = sa.alloc_workspace(need) if need else None
        out = torch.empty((B, H_q, T, d), dtype=torch.float32, device="cuda")
        calls = []
        for _ in range(copies):
            q = torch.randn((B, H_q, T, d), generator=gen, device="cuda").to(torch.bfloat16)
            k, v = kv((pool_pages, H_kv, 16, d) if pool_pages else (B, H_kv, n, d))
            extra = dict(page_table=pt, page_size=16, n_max=n) if pt is not None else {}
            a = sa.attn_args(q, k, v, out=out, indices=idx, counts=cnt, **extra)
            ws = sa.alloc_workspace(sa.specattn_workspace_size(None, a))
            a.workspace, a.workspace_bytes = ws.data_ptr(), ws.numel()
            calls.append((a, ws, q, k, v))
        t_sel = timed(lambda: sa.specattn_topp_select(s, ws_s))
        state = {"i": 0}

        def attend():
            sa.specattn_sparse_decode_attn(calls[state["i"] % copies][0])
            state["i"] += 1
        t_att = timed(attend)
        kept = int(cnt.sum().item())
        total = int(seq_lens.sum()) * H_kv if seq_lens is not None else R * n
        emit(name, rows=R, n=n, top_p=top_p, kept_fraction=round(kept / total, 4), select_us=round(t_sel, 1),
             split_selection=bool(need), attention_us=round(t_att, 1), kept_kv_MB=round(kept * 512 / 1e6, 1),
             attention_GBps=round(kept * 512.0 / t_att / 1e3, 1))

    w = W.llama8b_layer(seed=1, with_kv=False)
    pair("llama8b_layer n=8192 p=0.95 (cache-resident)", w.probs, 0.95, 1, 8192)
    for clip in (None, 8.0):
        w = W.long_context(seed=3, B=4, n=131072, logit_clip=clip, with_kv=False)
        for tp in (0.8, 0.9, 0.95, 0.99):
            pair(f"long_context B=4 n=131072 logits {'literal' if clip is None else 'clipped to 8'}", w.probs, tp, 4, 131072)
    w = W.ragged_paged(seed=0, B=64, with_kv=False)
    pair("ragged_paged B=64 lens 4096..65536, 16-token pages", w.probs, 0.95, 64, w.n, seq_lens=w.seq_lens,
         page_table=w.page_table, pool_pages=w.n_pool_pages)

    # ---- the calls beyond the pair, at the headline layer shape ---------------------------------------------
    B, n, L = 8, 32768, 6
    R = B * H_kv
    rng = np.random.default_rng(11)
    probs = torch.from_numpy(W.draft_probs(rng, L * R, n).reshape(L * B, H_kv, n)).cuda()
    k, v = kv((L * B, H_kv, n, d))
    k_new, v_new = kv((L * B, H_kv, T, d))
    idx = torch.zeros((L * R, n), dtype=torch.int32, device="cuda")
    cnt = torch.zeros((L * R,), dtype=torch.int32, device="cuda")
    sel = sa.select_args(probs, 0.9, indices=idx, counts=cnt)
    sa.specattn_topp_select(sel)
    torch.cuda.synchronize()
    kept_bytes = float(cnt.sum().item()) / L * 512

    def layer_calls(H_q_, **kw):
        q = torch.randn((L * B, H_q_, T, d), generator=gen, device="cuda").to(torch.bfloat16)
        out = torch.empty((B, H_q_, T, d), dtype=torch.float32, device="cuda")
        calls = []
        for l in range(L):
            b, r = slice(l * B, (l + 1) * B), slice(l * R, (l + 1) * R)
            extra = {key: (val[b] if key in ("k_new", "v_new") else val[r] if key in ("indices", "counts") else val)
                     for key, val in kw.items()}
            a = sa.attn_args(q[b], k[b], v[b], out=out, **extra)
            ws = sa.alloc_workspace(sa.specattn_workspace_size(None, a))
            a.workspace, a.workspace_bytes = ws.data_ptr(), ws.numel()
            calls.append((a, ws))
        return calls, q, out

    def per_layer(calls):
        return timed(lambda: [sa.specattn_sparse_decode_attn(a) for a, _ in calls]) / L

    c, *_k = layer_calls(H_q, indices=idx, counts=cnt)
    t = per_layer(c)
    emit("headline layer, list", attention_us=round(t, 1), attention_GBps=round(kept_bytes / t / 1e3, 1))
    c, *_k = layer_calls(H_q, indices=idx, counts=cnt, k_new=k_new, v_new=v_new)
    emit("headline layer, list + new tokens behind the cache", attention_us=round(per_layer(c), 1))
    c, *_k = layer_calls(H_q)
    t = timed(lambda: [sa.specattn_sparse_decode_attn(a) for a, _ in c], reps=5) / L
    emit("headline layer, dense (no list)", attention_us=round(t, 1), attention_GBps=round(R * n * 512.0 / t / 1e3, 1))
    for hq in (64, 128):
        c, *_k = layer_calls(hq, indices=idx, counts=cnt)
        t = per_layer(c)
        emit(f"headline layer, {hq // H_kv} query heads per kv head", attention_us=round(t, 1),
             kept_kv_GBps_counted_once=round(kept_bytes / t / 1e3, 1))
    nc = n // 16
    idc = torch.zeros((L * R, nc), dtype=torch.int32, device="cuda")
    cc = torch.zeros((L * R,), dtype=torch.int32, device="cuda")
    selc = sa.select_args(probs, 0.9, indices=idc, counts=cc, chunk_size=16)
    wsc = sa.alloc_workspace(sa.specattn_workspace_size(selc, None))
    t_tok = timed(lambda: sa.specattn_topp_select(sel))
    t_chk = timed(lambda: sa.specattn_topp_select(selc, wsc))
    chunk_bytes = float(cc.sum().item()) / L * 16 * 512
    c, *_k = layer_calls(H_q, indices=idc, counts=cc, chunk_size=16)
    t = per_layer(c)
    emit("selection in chunks of 16 + attention over chunk lists", rows=L * R, n=n, select_tokens_us=round(t_tok, 1),
         select_chunks_us=round(t_chk, 1), kept_chunk_fraction=round(float(cc.float().mean().item()) / nc, 4),
         attention_us=round(t, 1), attention_GBps=round(chunk_bytes / t / 1e3, 1))
    # ---- offline layer mapping (runs once per model pair, not per decoding step) --------------------------------
    for (m_, n_, rows_, L_) in ((22, 32, 64, 2048), (32, 80, 256, 4096)):
        ad, av = W.layer_attention_maps(seed=0, m=m_, n=n_, rows=rows_, L=L_)
        ad_d, av_d = torch.from_numpy(ad).cuda(), torch.from_numpy(av).cuda()
        S = torch.empty((m_, n_), dtype=torch.float64, device="cuda")
        fmap = torch.empty((n_,), dtype=torch.int32, device="cuda")
        tot = torch.empty((1,), dtype=torch.float64, device="cuda")
        ws1 = sa.alloc_workspace(int(sa.load().specattn_layer_similarity_workspace_size(m_, n_, rows_, L_)))
        ws2 = sa.alloc_workspace(int(sa.load().specattn_layer_map_workspace_size(m_, n_)))
        t_sim = timed(lambda: sa.specattn_layer_similarity(ad_d, av_d, S, ws1), reps=5, warm=1)
        t_map = timed(lambda: sa.specattn_layer_map(S, fmap, tot, ws2), reps=5, warm=1)
        terms = m_ * n_ * rows_ * L_
        emit(f"offline layer mapping, {m_} draft x {n_} verifier layers, {rows_} rows x {L_} positions",
             similarity_us=round(t_sim, 1), terms=terms, Gterms_per_s=round(terms / t_sim / 1e3, 2),
             input_MB=round((m_ + n_) * rows_ * L_ * 4 / 1e6, 1), alignment_us=round(t_map, 1),
             total_score=round(float(tot.item()), 4))
    for hd, steps in ((8, 4), (32, 4)):
        pu = torch.from_numpy(W.draft_step_probs(np.random.default_rng(2), B, hd, steps, n)).cuda()
        iu = torch.zeros((R, n), dtype=torch.int32, device="cuda")
        cu = torch.zeros((R,), dtype=torch.int32, device="cuda")
        ua = sa.union_args(pu, 0.9, H_kv, indices=iu, counts=cu)
        wsu = sa.alloc_workspace(sa.specattn_union_workspace_size(ua))
        t = timed(lambda: sa.specattn_topp_select_union(ua, wsu))
        emit(f"union over {steps} draft steps x {hd // H_kv} draft heads per kv head", member_rows=B * hd * steps, n=n,
             probs_MB=round(B * hd * steps * n * 4 / 1e6, 1), union_us=round(t, 1),
             union_fraction=round(float(cu.float().mean().item()) / n, 4))


def compare_lists(ref, idx, cnt, tau):
    """Rows the oracle flags as near the boundary, and rows whose device result (count, tau*, list) differs from the
    oracle's: (flagged, mismatched among the flagged, mismatched among the others)."""
    NEAR = 2
    flagged = mism_flagged = mism_clear = 0
    for r in range(ref.counts.size):
        c = int(ref.counts[r])
        same = int(cnt[r]) == c and tau[r] == ref.tau[r] and np.array_equal(idx[r, :c], ref.indices[r, :c])
        if ref.flags[r] & NEAR:
            flagged += 1
            mism_flagged += 0 if same else 1
        else:
            mism_clear += 0 if same else 1
    return flagged, mism_flagged, mism_clear


def other_configs(torch, sa, W, oracle):
    """The workload's other configurations, bounded so that the default run stays short: selection and attention
    times (HIP events, mean of 10 after 2 warm-up calls), kept fraction, and the device lists against the oracle's."""
    H_q, H_kv, T, d = 32, 8, 5, 128
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)

    def timed(fn, reps=10, warm=2):
        for _ in range(warm):
            fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps * 1e3          # us

    def pair(w, dtype, *, paged=False, copies=1, physical=False):
        B, H, n = w.probs.shape
        R = B * H
        p = torch.from_numpy(w.probs).cuda()
        sl = None if w.seq_lens is None else torch.from_numpy(w.seq_lens.astype(np.int32)).cuda()
        pt = torch.from_numpy(w.page_table).cuda() if paged else None
        idx = torch.zeros((R, n), dtype=torch.int32, device="cuda")
        cnt = torch.zeros(R, dtype=torch.int32, device="cuda")
        tau = torch.zeros(R, dtype=torch.float32, device="cuda")
        s = sa.select_args(p, w.top_p, indices=idx, counts=cnt, thresholds=tau, seq_lens=sl)
        need = sa.specattn_workspace_size(s, None)
        ws_s = sa.alloc_workspace(need) if need else None
        t_sel = timed(lambda: sa.specattn_topp_select(s, ws_s))
        ref = oracle.topp_select(w.probs.reshape(R, n), w.top_p, None if w.seq_lens is None else np.repeat(w.seq_lens, H))
        flagged, mf, mc = compare_lists(ref, idx.cpu().numpy(), cnt.cpu().numpy(), tau.cpu().numpy())
        H_qw = w.H_q
        out = torch.empty((B, H_qw, w.T, w.d), dtype=torch.float32, device="cuda")
        calls = []
        for _ in range(copies):
            q = torch.randn((B, H_qw, w.T, w.d), generator=gen, device="cuda").to(dtype)
            shape = (w.n_pool_pages, H, W.PAGE_SIZE, w.d) if paged else (B, H, n, w.d)
            k = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(dtype) if dtype == torch.float32 else \
                torch.empty(shape, device="cuda", dtype=dtype).normal_(generator=gen)
            v = torch.empty(shape, device="cuda", dtype=dtype).normal_(generator=gen)
            extra = dict(page_table=pt, page_size=W.PAGE_SIZE, n_max=n) if paged else {}
            a = sa.attn_args(q, k, v, out=out, indices=idx, counts=cnt, **extra)
            ws = sa.alloc_workspace(sa.specattn_workspace_size(None, a))
            a.workspace, a.workspace_bytes = ws.data_ptr(), ws.numel()
            calls.append((a, ws, q, k, v))
        state = {"i": 0}

        def attend():
            sa.specattn_sparse_decode_attn(calls[state["i"] % copies][0])
            state["i"] += 1
        t_att = timed(attend)
        kept = int(cnt.sum().item())
        total = int(w.seq_lens.sum()) * H if w.seq_lens is not None else R * n
        row_bytes = 2 * w.d * (4 if dtype == torch.float32 else 2)
        return dict(rows=R, n=n, top_p=w.top_p, kept_fraction=round(kept / total, 5), select_us=round(t_sel, 1),
                    attention_us=round(t_att, 1), kept_kv_MB=round(kept * row_bytes / 1e6, 2),
                    attention_GBps=round(kept * row_bytes / t_att / 1e3, 1),
                    pct_hbm_peak=round(kept * row_bytes / t_att / 1e3 / HBM_PEAK_GBPS * 100, 2),
                    flagged_rows=flagged, mismatched_flagged_rows=mf, mismatched_rows=mc)

    res = {}
    res["config1 tiny fp32 (B=1, H=8, n=1024, d=64, p=0.9)"] = pair(W.tiny_f32(), torch.float32)
    res["config2 llama3-8b layer (B=1, n=8192, p=0.95; 11 MB kept: cache-resident)"] = \
        pair(W.llama8b_layer(seed=1, with_kv=False), torch.bfloat16, copies=4)
    for clip in (None, 8.0):
        for tp in (0.8, 0.9, 0.95, 0.99):
            w = W.long_context(seed=3, B=4, n=131072, top_p=tp, logit_clip=clip, with_kv=False)
            res[f"config4 long context (B=4, n=131072), logits {'literal' if clip is None else 'clipped to +-8'}, p={tp}"] = \
                pair(w, torch.bfloat16)
    w = W.ragged_paged(seed=0, B=64, with_kv=False)
    res["config5 ragged paged (B=64, lens 4096..65536, 16-token pages, p=0.95)"] = pair(w, torch.bfloat16, paged=True)
    return res


def main():
    args = parse()
    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU; --gpus must be 1 (no multi-GPU path exists)",
              file=sys.stderr)
        sys.exit(2)
    import torch
    from paper_2510_27641_amd import binding as sa
    from paper_2510_27641_amd import workloads as W

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    torch.cuda.set_device(0)
    sa.load()
    if args.workload == "side":
        side_workloads(torch, sa, W)
        return
    L, B, n, top_p = args.layers, args.batch, args.context, args.top_p
    H_q, H_kv, T, d = 32, 8, 5, 128
    R = B * H_kv

    # ---- synthetic inputs, resident in HBM ---------------------------------------------------
    t0 = time.time()
    probs_host = np.empty((L * B, H_kv, n), dtype=np.float32)
    for layer in range(L):
        w = W.llama8b_layer(seed=1000 + layer, B=B, n=n, top_p=top_p, with_kv=False)
        probs_host[layer * B:(layer + 1) * B] = w.probs
    probs = torch.from_numpy(probs_host).cuda()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2024)
    # one allocation per tensor kind, [L*B, ...]: layer l is the slice [l*B, (l+1)*B)
    q_all = torch.empty((L * B, H_q, T, d), device="cuda", dtype=torch.bfloat16)
    k_all = torch.empty((L * B, H_kv, n, d), device="cuda", dtype=torch.bfloat16)
    v_all = torch.empty((L * B, H_kv, n, d), device="cuda", dtype=torch.bfloat16)
    qs, ks, vs = [], [], []
    for layer in range(L):
        sl_ = slice(layer * B, (layer + 1) * B)
        q_all[sl_] = torch.randn((B, H_q, T, d), generator=gen, device="cuda", dtype=torch.float32).to(torch.bfloat16)
        k_all[sl_].normal_(generator=gen)
        v_all[sl_].normal_(generator=gen)
        qs.append(q_all[sl_])
        ks.append(k_all[sl_])
        vs.append(v_all[sl_])
    torch.cuda.synchronize()
    t_gen = time.time() - t0

    # ---- outputs and argument structs --------------------------------------------------------
    idx = torch.empty((L * R, n), dtype=torch.int32, device="cuda")
    counts = torch.zeros((L * R,), dtype=torch.int32, device="cuda")
    tau = torch.empty((L * R,), dtype=torch.float32, device="cuda")
    flags = torch.empty((L * R,), dtype=torch.int32, device="cuda")
    outs = [torch.empty((B, H_q, T, d), dtype=torch.float32, device="cuda") for _ in range(L)]
    sel_all = sa.select_args(probs, top_p, indices=idx, counts=counts, thresholds=tau, row_flags=flags)
    attn = []
    ws = None
    for layer in range(L):
        a = sa.attn_args(qs[layer], ks[layer], vs[layer], out=outs[layer],
                         indices=idx[layer * R:(layer + 1) * R], counts=counts[layer * R:(layer + 1) * R])
        if ws is None:
            ws = sa.alloc_workspace(sa.specattn_workspace_size(None, a))
        a.workspace, a.workspace_bytes = ws.data_ptr(), ws.numel()
        attn.append(a)

    def step_unfused():
        sa.specattn_topp_select(sel_all)
        for a in attn:
            sa.specattn_sparse_decode_attn(a)

    # fused: the index list never goes through HBM.  One threshold launch for the rows of all layers
    # writes tau*, counts and per-block counts; each layer's attention rebuilds its lists on chip.
    fused_ok = True
    nblk = (n + sa.SEL_BLOCK - 1) // sa.SEL_BLOCK
    counts_f = torch.zeros((L * R,), dtype=torch.int32, device="cuda")
    tau_f = torch.empty((L * R,), dtype=torch.float32, device="cuda")
    bc_f = torch.empty((L * R, nblk), dtype=torch.int32, device="cuda")
    km_f = torch.empty((L * R, nblk * (sa.SEL_BLOCK // 32)), dtype=torch.int32, device="cuda")
    outs_f = [torch.empty((B, H_q, T, d), dtype=torch.float32, device="cuda") for _ in range(L)]
    sel_all_f = sa.select_args(probs, top_p, indices=None, counts=counts_f, thresholds=tau_f, block_counts=bc_f,
                               kept_mask=km_f)
    sel_layer, attn_f, ws_f = [], [], None
    for layer in range(L):
        rows = slice(layer * R, (layer + 1) * R)
        s = sa.select_args(probs[layer * B:(layer + 1) * B], top_p, indices=None, counts=counts_f[rows],
                           thresholds=tau_f[rows], block_counts=bc_f[rows], kept_mask=km_f[rows], reuse_selection=True)
        a = sa.attn_args(qs[layer], ks[layer], vs[layer], out=outs_f[layer])
        if ws_f is None:
            ws_f = sa.alloc_workspace(sa.specattn_workspace_size(s, a))
        a.workspace, a.workspace_bytes = ws_f.data_ptr(), ws_f.numel()
        sel_layer.append(s)
        attn_f.append(a)

    def step_fused():
        sa.specattn_topp_select(sel_all_f)
        for s, a in zip(sel_layer, attn_f):
            sa.specattn_fused(s, a)

    def timed(fn, steps, warmup):
        for _ in range(warmup):
            fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(steps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / steps          # ms per step

    if args.calibrate_copy:
        src = torch.empty(1 << 30, dtype=torch.uint8, device="cuda").fill_(1)
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    results = {}
    if args.path in ("both", "unfused"):
        results["unfused"] = timed(step_unfused, args.steps, args.warmup)
    if args.path in ("both", "fused"):
        try:
            results["fused"] = timed(step_fused, args.steps, args.warmup)
        except sa.SpecAttnError as e:
            fused_ok = False
            results["fused_error"] = str(e)
            if args.path == "fused":
                raise
    if "unfused" not in results:
        sa.specattn_topp_select(sel_all)            # counts for the byte accounting
        torch.cuda.synchronize()

    cnt = (counts if "unfused" in results else counts_f).cpu().numpy().astype(np.int64)
    sel_bytes_step = float(cnt.sum()) * 2 * d * 2   # K and V rows of d bf16 per kept position
    sel_frac = float(cnt.mean()) / n

    # ---- dominant kernel: sparse attention, HIP-event timed over its own launches ------------
    def attn_only():
        for a in attn:
            sa.specattn_sparse_decode_attn(a)
    if "unfused" not in results:
        sa.specattn_topp_select(sel_all)
    ms_attn = timed(attn_only, max(args.steps // 2, 3), 1) / L      # per layer launch
    ms_sel = timed(lambda: sa.specattn_topp_select(sel_all), max(args.steps // 2, 3), 1)
    # secondary figure: the same layers as independent instances of ONE bigger batch (groups of 16 layers per
    # call) - what the kernel sustains once the fixed start/end phases of a launch are amortised
    grp = 16 if L % 16 == 0 else 1
    out_b = torch.empty((grp * B, H_q, T, d), dtype=torch.float32, device="cuda")
    batched = []
    for g0 in range(0, L, grp):
        rows_b = slice(g0 * R, (g0 + grp) * R)
        ab = sa.attn_args(q_all[g0 * B:(g0 + grp) * B], k_all[g0 * B:(g0 + grp) * B], v_all[g0 * B:(g0 + grp) * B],
                          out=out_b, indices=idx[rows_b], counts=counts[rows_b])
        wsb = sa.alloc_workspace(sa.specattn_workspace_size(None, ab))
        ab.workspace, ab.workspace_bytes = wsb.data_ptr(), wsb.numel()
        batched.append((ab, wsb))

    def attn_batched():
        for ab, _ in batched:
            sa.specattn_sparse_decode_attn(ab)
    ms_batched = timed(attn_batched, max(args.steps // 2, 3), 1)
    # the same grouping on the fused path (lists rebuilt on chip from probs, tau* and the block counts)
    ms_batched_f = None
    if fused_ok and "fused" in results:
        batched_f = []
        for g0 in range(0, L, grp):
            rows_b = slice(g0 * R, (g0 + grp) * R)
            sb = sa.select_args(probs[g0 * B:(g0 + grp) * B], top_p, indices=None, counts=counts_f[rows_b],
                                thresholds=tau_f[rows_b], block_counts=bc_f[rows_b], kept_mask=km_f[rows_b],
                                reuse_selection=True)
            ab = sa.attn_args(q_all[g0 * B:(g0 + grp) * B], k_all[g0 * B:(g0 + grp) * B], v_all[g0 * B:(g0 + grp) * B], out=out_b)
            wsb = sa.alloc_workspace(sa.specattn_workspace_size(sb, ab))
            ab.workspace, ab.workspace_bytes = wsb.data_ptr(), wsb.numel()
            batched_f.append((sb, ab, wsb))

        def fused_batched():
            for sb, ab, _ in batched_f:
                sa.specattn_fused(sb, ab)
        ms_batched_f = timed(fused_batched, max(args.steps // 2, 3), 1)

    # whole steps in that grouping: the batched selection (or threshold pass) followed by the grouped calls
    def step_batched():
        sa.specattn_topp_select(sel_all)
        attn_batched()
    ms_step_b = timed(step_batched, max(args.steps // 2, 3), 1)
    ms_step_bf = None
    if ms_batched_f is not None:
        def step_batched_f():
            sa.specattn_topp_select(sel_all_f)
            fused_batched()
        ms_step_bf = timed(step_batched_f, max(args.steps // 2, 3), 1)
    # the grouped calls compute the same thing: the last group's outputs against the per-layer calls' outputs
    # (only the fp32 summation order differs, with the split of the rows over the workgroups)
    attn_only()
    attn_batched()
    torch.cuda.synchronize()
    grouped_diff = float((out_b.view(grp, B, H_q, T, d) - torch.stack(outs[L - grp:])).abs().max().item())
    if ms_batched_f is not None:
        step_fused()
        fused_batched()
        torch.cuda.synchronize()
        grouped_diff = max(grouped_diff, float((out_b.view(grp, B, H_q, T, d) - torch.stack(outs_f[L - grp:])).abs().max().item()))
    # ceiling of this machine: a plain 16 B per lane read over distinct 4 GiB pieces of the K cache
    piece = max(1, (4 << 30) // (k_all[0].numel() * 2))
    pieces = [k_all[i * piece:(i + 1) * piece] for i in range(min(3, k_all.shape[0] // piece))]
    state = {"i": 0}

    def stream_read():
        sa.specattn_stream_read(pieces[state["i"] % len(pieces)])
        state["i"] += 1
    ms_read = timed(stream_read, 6, 2)
    stream_gbps = pieces[0].numel() * 2 / (ms_read * 1e-3) / 1e9
    bytes_launch = sel_bytes_step / L
    achieved = bytes_launch / (ms_attn * 1e-3) / 1e9

    best = min(v for k, v in results.items() if k in ("unfused", "fused"))
    best_name = [k for k in ("fused", "unfused") if results.get(k) == best][0]
    value = sel_bytes_step / (best * 1e-3) / 1e9

    # HBM bytes per launch from rocprofv3 --pmc: taken from the committed summary only if that summary was made
    # from the kernel sources this run is built from (it records their hash); otherwise null
    traffic, traffic_source = None, None
    pmc = os.path.join(ROOT, "profiles", "sparse_decode_attn_config3_pmc.txt")
    if os.path.exists(pmc):
        import hashlib
        src = [os.path.join(ROOT, "paper_2510_27641_amd", "csrc", f) for f in ("attn_mfma.hip", "attn_mfma_kernel.h")]
        digest = hashlib.sha256(b"".join(open(f, "rb").read() for f in src)).hexdigest()[:16]
        found, val = None, None
        for ln in open(pmc):
            if ln.startswith("traffic_bytes_per_launch:"):
                val = float(ln.split(":")[1])
            if ln.startswith("attn_mfma_hip_sha256_16:"):
                found = ln.split(":")[1].strip()
        if val is not None and found == digest:
            traffic, traffic_source = val, "profiles/sparse_decode_attn_config3_pmc.txt (same kernel source, sha256/16 " + digest + ")"
        else:
            traffic_source = "profiles/sparse_decode_attn_config3_pmc.txt was made from other kernel sources: not quoted"
    line = {
        "metric": "selected_kv_GBps_topp_select_plus_sparse_decode_attn_32k",
        "value": round(value, 1), "unit": "GB/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(best, 4), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16", "data": "synthetic",
        "config": {"workload": f"llama3-8b-shaped verify step: {L} layers x (B={B}, n={n}, H_q=32, H_kv=8, d=128, "
                               f"T=5 queries), top_p={top_p}, bf16 K/V",
                   "path": best_name, "selected_fraction": round(sel_frac, 4),
                   "selected_kv_bytes_per_step": int(sel_bytes_step)},
        "pct_hbm_peak": round(100.0 * value / HBM_PEAK_GBPS, 2),
        "stream_read_GBps": round(stream_gbps, 1), "pct_of_stream_read": round(100.0 * value / stream_gbps, 2),
        "verify_steps_per_s": round(1e3 / best, 2),
        "selection_rows_per_s": round(L * R / (best * 1e-3), 1),
        "paths": {k: {"ms_per_step": round(v, 4), "GBps": round(sel_bytes_step / (v * 1e-3) / 1e9, 1)}
                  for k, v in results.items() if k in ("unfused", "fused")},
        "kernels": {"select_all_layers_ms": round(ms_sel, 4), "attention_per_layer_ms": round(ms_attn, 5)},
        "batched_instances": {"what": f"attention of all {L} layers as {L // grp} calls of {grp} independent layer instances each "
                                      "(the workload's layers are independent instances, so the figures hold for it; a verifier cannot run its "
                                      "layers this way, each layer's Q/K/V depending on the layer before, which is why `value` "
                                      "is the per-layer figure; shows the rate with the launch phases amortised)",
                              "ms": round(ms_batched, 4), "GBps": round(sel_bytes_step / (ms_batched * 1e-3) / 1e9, 1),
                              "fused_ms": None if ms_batched_f is None else round(ms_batched_f, 4),
                              "fused_GBps": None if ms_batched_f is None else round(sel_bytes_step / (ms_batched_f * 1e-3) / 1e9, 1),
                              "max_abs_diff_to_per_layer_calls": grouped_diff,
                              "whole_step": {"what": "selection of all rows + the grouped attention calls",
                                             "unfused_ms": round(ms_step_b, 4),
                                             "unfused_GBps": round(sel_bytes_step / (ms_step_b * 1e-3) / 1e9, 1),
                                             "fused_ms": None if ms_step_bf is None else round(ms_step_bf, 4),
                                             "fused_GBps": None if ms_step_bf is None else round(sel_bytes_step / (ms_step_bf * 1e-3) / 1e9, 1)}},
        "roofline": {"bound": "hbm", "kernel": "specattn_sparse_decode_attn = attn_mfma_kernel + merge_partials_kernel, one layer (HIP events around the layer loop)",
                     "achieved": round(achieved, 1), "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBPS, 4), "traffic": traffic, "traffic_source": traffic_source,
                     "algorithmic_bytes_per_launch": int(bytes_launch), "launch_us": round(ms_attn * 1e3, 2),
                     "frac_of_stream_read": round(achieved / stream_gbps, 4)},
        "roofline_select": {"bound": "hbm", "kernel": "specattn_topp_select = topp_select_kernel, the rows of all layers in one launch",
                            "algorithmic_bytes_per_launch": int(L * R * n * 4 + float(cnt.sum()) * 4),
                            "achieved": round((L * R * n * 4 + float(cnt.sum()) * 4) / (ms_sel * 1e-3) / 1e9, 1),
                            "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                            "frac": round((L * R * n * 4 + float(cnt.sum()) * 4) / (ms_sel * 1e-3) / 1e9 / HBM_PEAK_GBPS, 4),
                            "launch_us": round(ms_sel * 1e3, 1),
                            "what": "4 B per context position read once + 4 B per kept position written"},
        "input_generation_s": round(t_gen, 1),
    }
    if not fused_ok:
        line["fused_error"] = results.get("fused_error")

    # ---- CPU baseline: the oracle as it stands, on a bounded sample of the same workload ------
    if not args.no_cpu_baseline:
        import oracle
        cores = oracle.set_threads(0)
        budget_s = 20.0                                             # whole layers 0, 1, ... until about this much CPU work
        n_samp = 0
        t_sel = t_att = 0.0
        samp_bytes = 0.0
        worst = 0.0
        flagged = mism_flagged = mism_clear = 0
        sa.specattn_topp_select(sel_all)
        torch.cuda.synchronize()
        idx_h, cnt_h, tau_h = idx.cpu().numpy(), counts.cpu().numpy(), tau.cpu().numpy()
        for layer in range(L):
            if t_sel + t_att > budget_s:
                break
            n_samp += 1
            rows_s = probs_host[layer * B:(layer + 1) * B].reshape(R, n)
            t0 = time.time()
            ref = oracle.topp_select(rows_s, top_p)
            t_sel += time.time() - t0
            rs = slice(layer * R, (layer + 1) * R)
            f_, mf_, mc_ = compare_lists(ref, idx_h[rs], cnt_h[rs], tau_h[rs])
            flagged += f_; mism_flagged += mf_; mism_clear += mc_
            mask = ref.mask().reshape(B, H_kv, n)
            q0 = qs[layer].view(torch.int16).cpu().numpy().view(np.uint16)
            k0 = ks[layer].view(torch.int16).cpu().numpy().view(np.uint16)
            v0 = vs[layer].view(torch.int16).cpu().numpy().view(np.uint16)
            t0 = time.time()
            o_ref, _ = oracle.masked_attention(q0, k0, v0, mask, bf16=True)
            t_att += time.time() - t0
            samp_bytes += float(ref.counts.sum()) * 2 * d * 2
            # the same sample doubles as a full-size check of the device result
            got = (outs if "unfused" in results else outs_f)[layer].cpu().numpy()
            err = np.abs(got - o_ref).max(axis=-1) / np.abs(o_ref).max(axis=-1)
            worst = max(worst, float(err.max()))
        line["cpu_baseline"] = {
            "value": round(samp_bytes / (t_sel + t_att) / 1e9, 4), "unit": "GB/s", "cores": cores, "kind": "oracle",
            "sample": f"layers 0..{n_samp - 1} of the step ({n_samp * R} selection rows, {n_samp * B * H_q * T} query rows): "
                      f"oracle selection {t_sel:.2f} s + masked dense attention {t_att:.2f} s wall on {cores} threads; "
                      f"rate = kept K/V bytes of the sample / that time"}
        line["full_size_check_row_rel_err"] = worst
        line["selection_check"] = {"rows_checked": n_samp * R, "flagged_rows": flagged,
                                   "mismatched_flagged_rows": mism_flagged, "mismatched_rows": mism_clear,
                                   "what": "device lists, counts and tau* of the checked layers against the oracle's: rows whose "
                                           "kept or strictly-above mass lies within 1e-6 of the target are flagged and counted; "
                                           "mismatches are counted separately among them and among the others"}
        if not args.no_other_configs:
            line["other_configs"] = other_configs(torch, sa, W, oracle)

    print(json.dumps(line))


if __name__ == "__main__":
    main()
