"""One to four tiles of 16 query rows per kv head in one launch, and 64-wide heads, on the matrix-core kernel, at the
sizes where tiles begin and end.

Bounds: 128-wide heads as everywhere (2e-3; the bf16 weights carry 16 bits).  64-wide heads hand their weights over
in three parts, 24 bits, so what is left is the fp32 accumulation over at most a few thousand terms, the bound of the fp32
route (1e-5)."""
import numpy as np
import pytest
import torch

import oracle
from helpers import TOL, dev, gpu_attention, kv_tensors, oracle_attention, row_rel_err
from paper_2510_27641_amd import binding as sa
from paper_2510_27641_amd import workloads as W

pytestmark = pytest.mark.gpu


def lists(mask):
    B, H, n = mask.shape
    idx = np.zeros((B * H, n), dtype=np.int32)
    cnt = np.zeros(B * H, dtype=np.int32)
    for r, m in enumerate(mask.reshape(B * H, n)):
        at = np.flatnonzero(m)
        idx[r, :at.size], cnt[r] = at, at.size
    return dev(idx), dev(cnt)


def tol(w):
    return TOL["f32"] if w.d == 64 else TOL[w.dtype]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,T", [(1, 1), (2, 8), (17, 1), (4, 8), (11, 3), (8, 6), (7, 7), (8, 8), (13, 5), (16, 8)])
def test_query_rows_around_the_tiles(d, G, T, dtype):
    # 1, 16, 17, 32, 33, 48, 49 and 64 query rows in one launch; 65 and 128 in two shares of heads (d = 128 only)
    if d == 64 and G * T > 64:
        z = torch.zeros((1, 2 * G, T, d), dtype=torch.bfloat16, device="cuda")
        a = sa.attn_args(z, z[:, :2], z[:, :2], out=z.float(), indices=None, counts=None)
        with pytest.raises(RuntimeError, match="query rows"):
            sa.specattn_sparse_decode_attn(a)
        return
    w = W.llama8b_layer(seed=G * T, B=2, n=900, H_q=2 * G, H_kv=2, T=T, d=d, dtype=dtype)
    mask = oracle.topp_select(w.probs.reshape(-1, w.n), w.top_p).mask().reshape(w.B, w.H_kv, w.n)
    q, k, v = kv_tensors(w)
    idx, cnt = lists(mask)
    out, lse = gpu_attention(q, k, v, idx, cnt)
    ref, ref_lse = oracle_attention(w, mask)
    assert row_rel_err(out, ref) <= tol(w)
    assert np.abs(lse - ref_lse).max() <= 1e-3


@pytest.mark.parametrize("G", [4, 8])
@pytest.mark.parametrize("count", [0, 1, 63, 64, 65, 127, 128, 129, 8 * 64 - 1, 8 * 64 + 1, 2000])
def test_counts_around_the_tiles_of_64_wide_heads(count, G):
    w = W.llama8b_layer(seed=3, B=1, n=2048, H_q=3 * G, H_kv=3, T=5, d=64)
    rng = np.random.default_rng(count)
    mask = np.zeros((1, 3, w.n), dtype=np.uint8)
    for h in range(3):
        mask[0, h, rng.choice(w.n, size=max(0, count - h), replace=False)] = 1
    q, k, v = kv_tensors(w)
    idx, cnt = lists(mask)
    out, lse = gpu_attention(q, k, v, idx, cnt)
    ref, ref_lse = oracle_attention(w, mask)
    assert row_rel_err(out, ref) <= tol(w)
    if count == 0:
        assert (out == 0).all() and np.isneginf(lse).all()


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("G,T", [(1, 1), (4, 5), (8, 8)])
@pytest.mark.parametrize("capacity", [1, 17, 128, 129])
def test_short_lists_of_64_wide_heads(capacity, G, T, dtype):
    """On both sides of the line from which on such lists leave the kernel that finishes a row in one launch."""
    w = W.llama8b_layer(seed=capacity, B=2, n=700, H_q=3 * G, H_kv=3, T=T, d=64, dtype=dtype)
    rng = np.random.default_rng(capacity)
    mask = np.zeros((2, 3, w.n), dtype=np.uint8)
    for r, count in enumerate((0, 1, capacity, max(1, capacity // 2), capacity, capacity - 1)):
        mask[r // 3, r % 3, rng.choice(w.n, size=count, replace=False)] = 1
    k_new, v_new = (rng.standard_normal((2, 3, T, 64), dtype=np.float32) for _ in range(2))
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    bits = W.round_to_bf16_bits if dtype == "bf16" else lambda a: a.astype(np.float16).view(np.uint16)
    q, k, v = kv_tensors(w)
    idx, cnt = lists(mask)
    for new in ({}, dict(k_new=dev(k_new, dt), v_new=dev(v_new, dt))):
        out, lse = torch.full(q.shape, float("nan"), device="cuda"), torch.full(q.shape[:3], float("nan"), device="cuda")
        att = sa.attn_args(q, k, v, out=out, lse=lse, indices=idx[:, :capacity].contiguous(), counts=cnt, **new)
        ws = sa.alloc_workspace(sa.specattn_workspace_size(None, att))
        att.workspace, att.workspace_bytes = ws.data_ptr(), ws.numel()
        sa.specattn_sparse_decode_attn(att)
        torch.cuda.synchronize()
        ref, ref_lse = oracle.masked_attention(*(bits(a).reshape(a.shape) for a in (w.q, w.k, w.v)), mask, bf16=dtype == "bf16", f16=dtype == "f16",
                                               **(dict(k_new=bits(k_new).reshape(k_new.shape), v_new=bits(v_new).reshape(v_new.shape)) if new else {}))
        assert row_rel_err(out.cpu().numpy(), ref) <= TOL["f32"]
        fin, got = np.isfinite(ref_lse), lse.cpu().numpy()
        assert np.array_equal(np.isneginf(got), ~fin) and np.abs(got[fin] - ref_lse[fin]).max() <= 1e-3


@pytest.mark.parametrize("mode", ["table", "physical"])
@pytest.mark.parametrize("d,H_q", [(64, 16), (64, 24), (128, 24), (128, 32)])
def test_paged_layouts(mode, d, H_q):
    w = W.ragged_paged(seed=5, B=4, len_lo=50, len_hi=3000, H_q=H_q, H_kv=2, T=4, d=d)
    ref = oracle.topp_select(w.probs.reshape(-1, w.n), w.top_p, np.repeat(w.seq_lens, w.H_kv))
    mask = ref.mask().reshape(w.B, w.H_kv, w.n)
    idx, cnt = lists(mask)
    if mode == "physical":
        i = idx.cpu().numpy()
        for r in range(i.shape[0]):
            c = int(ref.counts[r])
            i[r, :c] = w.page_table[r // w.H_kv, i[r, :c] // W.PAGE_SIZE] * W.PAGE_SIZE + i[r, :c] % W.PAGE_SIZE
        idx = dev(i)
    q, k, v = kv_tensors(w)
    out, _ = gpu_attention(q, k, v, idx, cnt, page_table=dev(w.page_table) if mode == "table" else None,
                           page_size=W.PAGE_SIZE, physical=mode == "physical", n_max=w.n)
    want, _ = oracle_attention(w, mask)
    assert row_rel_err(out, want) <= tol(w)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("layout", ["table", "physical", "odd stride", "contiguous"])
def test_rows_beyond_64_gib(layout, dtype):
    """64-wide heads in pools of more than 64 GiB (row offsets of 16 bytes would need more than 32 bits), with pages whose
    stride is no multiple of a row, and in a contiguous cache whose positions lie that far apart."""
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 80 GiB")
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    n, H, T = 600, 2, 5
    w = W.llama8b_layer(seed=6, B=1, n=n, H_q=4 * H, H_kv=H, T=T, d=64, dtype=dtype)
    mask = oracle.topp_select(w.probs.reshape(-1, n), w.top_p).mask().reshape(1, H, n)
    idx, cnt = lists(mask)
    q, k, v = kv_tensors(w)
    kw = dict(n_max=n)
    if layout == "contiguous":
        stride = 36 * 2 ** 30 // n // 64 * 64                  # elements: n rows over 72 GiB
        buf = torch.empty(n * stride + 4 * n * 64, dtype=dt, device="cuda")
        kp, vp = (buf[at:].as_strided((1, H, n, 64), (2 * stride, 64, stride, 1)) for at in (0, 256))
        kp.copy_(k), vp.copy_(v)
    else:
        page, extra = 16, 8 if layout == "odd stride" else 0   # a page's rows, then 16 bytes of something else
        per = H * page * 64 + extra
        pages = 36 * 2 ** 30 // (2 * per)                       # of K and V, 72 GiB
        buf = torch.empty(pages * 2 * per, dtype=dt, device="cuda")
        kp, vp = (buf[at:].as_strided((pages, H, page, 64), (2 * per, page * 64, 64, 1)) for at in (0, per))
        at = np.linspace(0, pages - 1, -(-n // page)).astype(np.int32)[::-1].copy()
        for i, p in enumerate(at):
            m = min(page, n - i * page)
            kp[p, :, :m], vp[p, :, :m] = k[0, :, i * page:i * page + m], v[0, :, i * page:i * page + m]
        kw.update(page_size=page)
        if layout == "physical":
            idx = (dev(at)[(idx // page).long()] * page + idx % page).to(torch.int32)
            kw.update(physical=True)
        else:
            kw.update(page_table=dev(at.reshape(1, -1)))
    out, _ = gpu_attention(q, kp, vp, idx, cnt, **kw)
    del buf, kp, vp
    torch.cuda.empty_cache()
    assert row_rel_err(out, oracle_attention(w, mask)[0]) <= TOL["f32"]


@pytest.mark.parametrize("shape", [dict(B=40, n=250, H_q=64, H_kv=8, T=8), dict(B=1, n=60, H_q=7 * 512, H_kv=512, T=7)])
def test_small_workspace(shape):
    """The built-in 16 MiB do not hold partials of 64 query rows for all rows of these calls: the first goes out in
    batches of fewer rows, the second (one sequence of 512 rows) in shares of at most 32 query rows."""
    w = W.llama8b_layer(seed=8, **shape)
    mask = oracle.topp_select(w.probs.reshape(-1, w.n), w.top_p).mask().reshape(w.B, w.H_kv, w.n)
    q, k, v = kv_tensors(w)
    idx, cnt = lists(mask)
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
    sa.specattn_sparse_decode_attn_static(sa.attn_args(q, k, v, out=out, indices=idx, counts=cnt))
    torch.cuda.synchronize()
    assert row_rel_err(out.cpu().numpy(), oracle_attention(w, mask)[0]) <= TOL["bf16"]


def generic_bytes(w, capacity):
    rows, splits = w.B * w.H_kv, max(1, min(-(-1024 // (w.B * w.H_kv)), -(-capacity // 256), 64))
    return -(-rows * splits * (w.H_q // w.H_kv) * w.T * (w.d + 2) * 4 // 256) * 256


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("shape", [dict(d=64, B=1, n=1000, H_q=8, H_kv=8, T=1), dict(d=64, B=2, n=3000, H_q=16, H_kv=2, T=6),
                                   dict(d=128, B=2, n=3000, H_q=16, H_kv=2, T=6)])
def test_workspaces_for_two_query_tiles_are_accepted(shape, fused):
    """64-wide heads run with room for the partials of the fp32 kernel, 128-wide ones with room for two query tiles
    (256 workgroups plus one slot per row, and the cost prefix)."""
    w = W.llama8b_layer(seed=4, **shape)
    mask = oracle.topp_select(w.probs.reshape(-1, w.n), w.top_p).mask().reshape(w.B, w.H_kv, w.n)
    q, k, v = kv_tensors(w)
    rows = w.B * w.H_kv
    need = generic_bytes(w, w.n)
    if w.d == 128:
        G, heads = w.H_q // w.H_kv, 32 // w.T
        per = -(-G // -(-G // heads))                          # heads per launch of at most 32 query rows
        need = max(need, 256 + (256 + rows) * -(-per * w.T // 16) * 16 * (w.d + 2) * 4)
    probs = dev(w.probs)
    counts = torch.zeros(rows, dtype=torch.int32, device="cuda")
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
    if fused:
        sel = sa.select_args(probs, w.top_p, indices=None, counts=counts)
        att = sa.attn_args(q, k, v, out=out)
        need += sa.specattn_workspace_size(sel, att) - sa.specattn_workspace_size(None, att)
    else:
        idx, cnt = lists(mask)
        att = sa.attn_args(q, k, v, out=out, indices=idx, counts=cnt)
    ws = sa.alloc_workspace(need)
    att.workspace, att.workspace_bytes = ws.data_ptr(), need
    sa.specattn_fused(sel, att) if fused else sa.specattn_sparse_decode_attn(att)
    torch.cuda.synchronize()
    assert row_rel_err(out.cpu().numpy(), oracle_attention(w, mask)[0]) <= tol(w)
    att.workspace_bytes = need - 256
    with pytest.raises(RuntimeError, match="needed"):
        sa.specattn_fused(sel, att) if fused else sa.specattn_sparse_decode_attn(att)


@pytest.mark.parametrize("route", ["list", "dense"])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("G,T", [(1, 1), (4, 5), (7, 6), (8, 8)])
def test_infinite_values_decide_their_columns(G, T, dtype, route):
    """Infinite and NaN values at kept positions - inside a tile, in a row's last, partial tile, in one of several tiles of a
    wave, of both signs in one column - give what the sum of positive weights times values gives, in their columns alone."""
    n = 3001
    w = W.llama8b_layer(seed=G, B=1, n=n, H_q=3 * G, H_kv=3, T=T, d=64, dtype=dtype)
    mask = np.ones((1, 3, n), dtype=np.uint8)
    if route == "list":
        mask[0, 0, 21:] = 0
        mask[0, 2, n - 1] = 0
    ref, _ = oracle_attention(w, mask)
    for h, j, c, x in [(0, 20, 3, np.inf), (0, 7, 63, -np.inf), (1, n - 2, 8, np.inf), (1, 5, 9, -np.inf), (1, 2000, 9, np.inf),
                       (1, 33, 12, np.nan), (1, 1234, 40, -np.inf), (1, 2900, 40, -np.inf)]:
        w.v[0, h, j, c] = x
        column = ref[:, h * G:(h + 1) * G, :, c]
        column[...] = x if np.isfinite(column).all() or (column == x).all() else np.nan
    if route == "list":
        w.v[0, 2, n - 1, 0] = np.inf                           # not kept
    q, k, v = kv_tensors(w)
    out, _ = gpu_attention(q, k, v, *(lists(mask) if route == "list" else (None, None)))
    fin = np.isfinite(ref)
    assert np.array_equal(out[~fin], ref[~fin], equal_nan=True)
    assert row_rel_err(np.where(fin, out, 0.0), np.where(fin, ref, 0.0)) <= TOL["f32"]


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("mode", ["list", "dense", "chunks", "fused", "fused chunks"])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d,G,T", [(64, 4, 5), (64, 8, 8), (128, 7, 6), (128, 8, 8)])
def test_options_together(d, G, T, dtype, mode, paged):
    """Ragged lengths (an empty sequence, partial chunks), lists of positions or chunks, dense calls and the fused call, in
    both layouts, each without and with new tokens behind the cache and the copy of the output in the inputs' type; 64-wide
    heads, and three and four query tiles.  Every chunk list ends in the partial chunk of its row (the recency band)."""
    w = W.ragged_paged(seed=d + G, B=4, len_lo=33, len_hi=2300, H_q=2 * G, H_kv=2, T=T, d=d)
    w.seq_lens[2] = 0
    w.probs[2] = 0.0
    B, H, n = w.probs.shape
    rng = np.random.default_rng(9)
    k_new, v_new = (rng.standard_normal((B, H, T, d), dtype=np.float32) for _ in range(2))
    if dtype == "f16":
        w.dtype = "f16"
        w.q, w.k, w.v = (a.astype(np.float16).astype(np.float32) for a in (w.q, w.k, w.v))
        bits = lambda a: a.astype(np.float16).view(np.uint16)
    else:
        bits = lambda a: W.round_to_bf16_bits(a).reshape(a.shape)
    lens, chunk = w.row_lens(), 16 if "chunks" in mode else 0
    if mode == "dense":
        mask = np.arange(n) < lens[:, None]
    elif chunk:
        ref = oracle.topp_select_chunks(w.probs.reshape(-1, n), w.top_p, chunk, lens=lens)
        mask = oracle.chunk_token_mask(ref, chunk, n, lens)
    else:
        ref = oracle.topp_select(w.probs.reshape(-1, n), w.top_p, lens)
        mask = ref.mask()
    mask = mask.reshape(B, H, n).astype(np.uint8)
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    kw = dict(seq_lens=dev(w.seq_lens))
    if paged:
        kw.update(page_table=dev(w.page_table), page_size=W.PAGE_SIZE, n_max=n)
        q, k, v = kv_tensors(w)
    else:
        q, k, v = (dev(a, dt) for a in (w.q, w.k, w.v))
    sel, call = None, sa.specattn_sparse_decode_attn
    counts = torch.zeros(B * H, dtype=torch.int32, device="cuda")
    if mode in ("list", "chunks"):
        cap = -(-n // chunk) if chunk else n
        kw.update(indices=dev(np.ascontiguousarray(ref.indices[:, :cap])), counts=dev(ref.counts), chunk_size=chunk)
    elif mode != "dense":
        probs = dev(w.probs)
        sel = sa.select_args(probs, w.top_p, indices=None, counts=counts, seq_lens=kw["seq_lens"], chunk_size=chunk)
        call = lambda a: sa.specattn_fused(sel, a)
    for more in (False, True):
        out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
        lse = torch.full(q.shape[:3], float("nan"), dtype=torch.float32, device="cuda")
        low = torch.full(q.shape, float("nan"), dtype=dt, device="cuda")
        new = dict(k_new=dev(k_new, dt), v_new=dev(v_new, dt), out_lowp=low) if more else {}
        att = sa.attn_args(q, k, v, out=out, lse=lse, **kw, **new)
        ws = sa.alloc_workspace(sa.specattn_workspace_size(sel, att))
        att.workspace, att.workspace_bytes = ws.data_ptr(), ws.numel()
        call(att)
        torch.cuda.synchronize()
        want, want_lse = oracle.masked_attention(bits(w.q), bits(w.k), bits(w.v), mask, bf16=dtype == "bf16", f16=dtype == "f16",
                                                 lens=w.seq_lens, **(dict(k_new=bits(k_new), v_new=bits(v_new)) if more else {}))
        assert row_rel_err(out.cpu().numpy(), want) <= tol(w)
        fin = np.isfinite(want_lse)
        got = lse.cpu().numpy()
        assert np.array_equal(np.isneginf(got), ~fin) and np.abs(got[fin] - want_lse[fin]).max() <= 1e-3
        if more:
            assert torch.equal(low, out.to(dt))


@pytest.mark.parametrize("new_tokens", [False, True])
@pytest.mark.parametrize("B,H_kv,G,T,n", [(1, 1, 1, 1, 700), (4, 16, 3, 3, 700), (13, 5, 5, 7, 700), (9, 7, 9, 6, 700), (2, 33, 2, 5, 700),
                                          (1, 3, 4, 5, 9001), (1, 4, 2, 5, 2500), (2, 4, 4, 4, 4100), (2, 8, 1, 8, 2600), (4, 8, 2, 3, 330)])
def test_rows_and_their_shares(B, H_kv, G, T, n, new_tokens):
    """63, 64 and 65 rows and few ones, head and token counts that are no powers of two, empty rows among full ones, rows inside
    one workgroup and over many, lines of 64, 128 and 256 shares, in a workspace that holds anything."""
    d = 128
    rng = np.random.default_rng(B * 100 + H_kv)
    w = W.llama8b_layer(seed=G, B=B, n=n, H_q=G * H_kv, H_kv=H_kv, T=T, d=d, dtype="f16")
    keep = rng.integers(0, n + 1, size=(B, H_kv)) * (rng.random((B, H_kv)) < 0.8)
    keep[0, 0] = n
    mask = (np.arange(n) < keep[..., None]).astype(np.uint8)
    q, k, v = kv_tensors(w)
    idx, cnt = lists(mask)
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
    extra, ref = {}, None
    if new_tokens:
        nk, nv = (rng.standard_normal((B, H_kv, T, d)).astype(np.float16) for _ in range(2))
        extra = dict(k_new=dev(nk), v_new=dev(nv))
        ref, _ = oracle.masked_attention(*(x.astype(np.float16).view(np.uint16) for x in (w.q, w.k, w.v)), mask, f16=True,
                                         k_new=nk.view(np.uint16), v_new=nv.view(np.uint16))
    else:
        ref, _ = oracle_attention(w, mask)
    att = sa.attn_args(q, k, v, out=out, indices=idx, counts=cnt, **extra)
    ws = sa.alloc_workspace(sa.specattn_workspace_size(None, att))
    ws.copy_(torch.from_numpy(rng.integers(0, 256, size=ws.numel(), dtype=np.uint8)))
    att.workspace, att.workspace_bytes = ws.data_ptr(), ws.numel()
    for _ in range(2):                                         # the second pass finds what the first one left
        sa.specattn_sparse_decode_attn(att)
        torch.cuda.synchronize()
        assert row_rel_err(out.cpu().numpy(), ref) <= TOL["f16"]


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("B,H_kv", [(1, 2), (2, 4), (2, 8), (8, 8), (13, 5)])
@pytest.mark.parametrize("others", [0, 3])
def test_one_long_row_among_short_ones(d, B, H_kv, others):
    """One row holds nearly all of the line, the others a few positions or none: 64, 128 and 256 shares, and 65 rows."""
    n, T = 9001, 5
    rng = np.random.default_rng(B * 10 + H_kv)
    w = W.llama8b_layer(seed=d, B=B, n=n, H_q=2 * H_kv, H_kv=H_kv, T=T, d=d, dtype="f16")
    keep = np.full((B, H_kv), others)
    keep[B // 2, H_kv // 2] = n
    mask = (rng.permuted(np.broadcast_to(np.arange(n), (B, H_kv, n)), axis=2) < keep[..., None]).astype(np.uint8)
    q, k, v = kv_tensors(w)
    idx, cnt = lists(mask)
    out, lse = gpu_attention(q, k, v, idx, cnt)
    ref, want_lse = oracle_attention(w, mask)
    assert row_rel_err(out, ref) <= TOL["f16"]
    fin = np.isfinite(want_lse)
    assert np.array_equal(np.isneginf(lse), ~fin) and np.abs(lse[fin] - want_lse[fin]).max() <= 1e-3


@pytest.mark.parametrize("B,H_kv,tiles", [(1, 2, 8), (1, 2, 9), (1, 2, 128), (1, 2, 129), (1, 1, 192), (1, 1, 193), (1, 1, 1152), (1, 1, 1153),
                                          (1, 8, 872), (1, 8, 873), (2, 4, 1308), (2, 4, 1309), (1, 8, 1745), (1, 8, 5232), (1, 8, 5233),
                                          (8, 8, 768), (8, 8, 769), (4, 16, 1152), (8, 8, 3072), (8, 8, 3073), (3, 11, 3488), (5, 13, 300),
                                          (1, 1, 1536), (1, 1, 1537), (1, 2, 3072), (1, 2, 3073), (3, 11, 3489),
                                          (3, 11, 8203), (3, 11, 8204), (3, 11, 8205), (5, 13, 8203), (5, 13, 8204), (5, 13, 8205), (2, 4, 12000)])
def test_shares_of_whole_tiles(B, H_kv, tiles):
    """Totals of tiles at which the shares of up to 64 rows become longer (3, 4, 6, 8, ... 32 tiles) and go over to the line's, in rows
    of uneven lengths with an empty one among them; 65 rows; lines around 32 tiles to each of 256 shares (12 less for an empty row),
    from which on every second boundary is moved."""
    n_tiles = rng_tiles(tiles, B * H_kv)
    n = 32 * int(n_tiles.max())
    w = W.llama8b_layer(seed=tiles, B=B, n=n, H_q=2 * H_kv, H_kv=H_kv, T=2, d=128, dtype="f16")
    rng = np.random.default_rng(tiles)
    keep = np.maximum(n_tiles * 32 - rng.integers(0, 32, size=B * H_kv) * (n_tiles > 0), 0).reshape(B, H_kv)
    mask = (np.arange(n) < keep[..., None]).astype(np.uint8)
    q, k, v = kv_tensors(w)
    idx, cnt = lists(mask)
    out, lse = gpu_attention(q, k, v, idx, cnt)
    ref, want_lse = oracle_attention(w, mask)
    assert row_rel_err(out, ref) <= TOL["f16"]
    fin = np.isfinite(want_lse)
    assert np.array_equal(np.isneginf(lse), ~fin) and np.abs(lse[fin] - want_lse[fin]).max() <= 1e-3


def rng_tiles(total, rows):
    """`rows` tile counts that add up to `total`: the last one 0 where there are more than two, the others uneven."""
    rng = np.random.default_rng(total * 100 + rows)
    full = rows - 1 if rows > 2 else rows
    part = np.floor(total * rng.dirichlet(np.full(full, 8.0))).astype(int)
    part[0] += total - part.sum()
    return np.concatenate([part, np.zeros(rows - full, dtype=int)])


@pytest.mark.parametrize("rows", [63, 64, 65])
@pytest.mark.parametrize("kind", ["positions", "chunks", "dense"])
@pytest.mark.parametrize("d,G,T", [(128, 4, 5), (128, 8, 8), (64, 8, 5)])
def test_forms_of_the_kernel_at_the_line_between_them(d, G, T, kind, rows):
    """Up to 64 rows and more run in kernels of their own, lists of single positions apart from chunk lists and dense calls, and four query tiles
    of 128 apart from fewer: every sequence on its own against the oracle, some of them without a kept position."""
    n, chunk = 333, 8
    w = W.llama8b_layer(seed=rows + G, B=rows, n=n, H_q=G, H_kv=1, T=T, d=d)
    rng = np.random.default_rng(rows)
    keep = rng.random((rows, -(-n // chunk))) < 0.3
    keep[::7] = False
    keep[1::7, -1] = True                                      # (the partial chunk at the end)
    mask = np.ones((rows, 1, n), dtype=np.uint8)
    kw = {}
    if kind == "chunks":
        mask = np.repeat(keep, chunk, axis=1)[:, :n].astype(np.uint8).reshape(rows, 1, n)
        idx, cnt = lists(keep.reshape(rows, 1, -1))
        kw = dict(indices=idx, counts=cnt, chunk_size=chunk)
    elif kind == "positions":
        mask = (rng.random((rows, 1, n)) < 0.3).astype(np.uint8)
        mask[::7] = 0
        idx, cnt = lists(mask)
        kw = dict(indices=idx, counts=cnt)
    q, k, v = kv_tensors(w)
    out = torch.full(q.shape, float("nan"), device="cuda")
    a = sa.attn_args(q, k, v, out=out, **kw)
    ws = sa.alloc_workspace(sa.specattn_workspace_size(None, a))
    a.workspace, a.workspace_bytes = ws.data_ptr(), ws.numel()
    sa.specattn_sparse_decode_attn(a)
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    ref, _ = oracle_attention(w, mask)
    if kind != "dense":
        assert (out[::7] == 0).all()
    assert row_rel_err(out, ref) <= tol(w)
