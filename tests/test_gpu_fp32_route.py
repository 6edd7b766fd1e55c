"""The fp32 attention kernel at the sizes where its work is cut: tiles of 16 positions over eight waves, one or several
splits per row, tiles of 16 query rows, new tokens behind the cache; and with 16-bit inputs where the 16-bit route does
not take the call.

Bound: fp32 products and sums over at most a few thousand terms (the 1e-5 of every fp32 test)."""
import numpy as np
import pytest
import torch

import oracle
from helpers import TOL, dev, gpu_attention, kv_tensors, oracle_attention, row_rel_err
from paper_2510_27641_amd import binding as sa
from paper_2510_27641_amd import workloads as W

pytestmark = pytest.mark.gpu


def lists(mask, cap):
    B, H, n = mask.shape
    idx = np.zeros((B * H, cap), dtype=np.int32)
    cnt = np.zeros(B * H, dtype=np.int32)
    for r, m in enumerate(mask.reshape(B * H, n)):
        at = np.flatnonzero(m)
        idx[r, :at.size], cnt[r] = at, at.size
    return dev(idx), dev(cnt)


@pytest.mark.parametrize("d,cap", [(64, 1100), (64, 3000), (128, 1000), (128, 3000)])     # one split, several splits
@pytest.mark.parametrize("count", [0, 1, 15, 16, 17, 127, 128, 129, 144, 1000])
def test_counts_around_the_tiles(d, cap, count):
    w = W.tiny_f32(seed=count, n=3000, B=2, H=3, T=5, d=d)
    rng = np.random.default_rng(count)
    mask = np.zeros((2, 3, w.n), dtype=np.uint8)
    for b in range(2):
        for h in range(3):
            mask[b, h, rng.choice(w.n, size=max(0, count - 7 * h - b), replace=False)] = 1
    q, k, v = kv_tensors(w)
    out, lse = gpu_attention(q, k, v, *lists(mask, cap))
    ref, ref_lse = oracle_attention(w, mask)
    assert row_rel_err(out, ref) <= TOL["f32"]
    live = np.isfinite(ref_lse)
    assert np.abs(lse[live] - ref_lse[live]).max(initial=0.0) <= 1e-5 and np.isneginf(lse[~live]).all()
    assert (out[~live] == 0).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [300, 2500])
@pytest.mark.parametrize("G,T", [(1, 1), (2, 8), (17, 1), (4, 8), (11, 3), (8, 6), (7, 7), (8, 8)])
def test_query_rows_around_the_tiles_with_new_tokens(d, n, G, T):
    w = W.llama8b_layer(seed=G * T, B=1, n=n, H_q=3 * G, H_kv=3, T=T, d=d, dtype="f32")
    mask = oracle.topp_select(w.probs.reshape(-1, w.n), w.top_p).mask().reshape(w.B, w.H_kv, w.n)
    mask[0, 1] = 0                                             # this row attends to new tokens only
    rng = np.random.default_rng(n)
    k_new, v_new = (rng.standard_normal((1, 3, T, d), dtype=np.float32) for _ in range(2))
    v_new[0, 2, T - 1] = np.inf                                # seen by the last query alone
    q, k, v = kv_tensors(w)
    idx, cnt = lists(mask, n)
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
    low = torch.zeros_like(out)
    args = sa.attn_args(q, k, v, out=out, out_lowp=low, indices=idx, counts=cnt, k_new=dev(k_new), v_new=dev(v_new))
    ws = sa.alloc_workspace(sa.specattn_workspace_size(None, args))
    args.workspace, args.workspace_bytes = ws.data_ptr(), ws.numel()
    sa.specattn_sparse_decode_attn(args)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    v_new[0, 2, T - 1] = 0.0
    ref = oracle.masked_attention(w.q, w.k, w.v, mask, k_new=k_new, v_new=v_new)[0]
    assert np.isinf(got[0, 2 * G:, T - 1]).all()
    seen = np.ones(got.shape[:3], dtype=bool)
    seen[0, 2 * G:, T - 1] = False
    assert row_rel_err(got[seen], ref[seen]) <= TOL["f32"]
    assert torch.equal(out, low)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [300, 2500])
@pytest.mark.parametrize("G,T", [(1, 1), (2, 8), (17, 1), (4, 8), (11, 3), (8, 6), (7, 7), (8, 8)])
def test_query_rows_around_the_tiles(d, n, G, T):
    """Contiguous lists of single positions alone, which have a form of their own up to three query tiles of 128."""
    w = W.llama8b_layer(seed=G * T, B=2, n=n, H_q=3 * G, H_kv=3, T=T, d=d, dtype="f32")
    mask = oracle.topp_select(w.probs.reshape(-1, w.n), w.top_p).mask().reshape(w.B, w.H_kv, w.n)
    mask[1, 1] = 0
    q, k, v = kv_tensors(w)
    out, lse = gpu_attention(q, k, v, *lists(mask, n))
    ref, want_lse = oracle_attention(w, mask)
    assert row_rel_err(out, ref) <= TOL["f32"] and (out[1, G:2 * G] == 0).all()
    live = np.isfinite(want_lse)
    assert np.abs(lse[live] - want_lse[live]).max() <= 1e-5 and np.isneginf(lse[~live]).all()


def test_infinite_value_in_a_partial_tile():
    """A kept position with an infinite value in the row's last, partial tile: it alone decides, nothing turns into NaN."""
    w = W.tiny_f32(seed=1, n=600, H=2, d=64)
    mask = np.zeros((1, 2, w.n), dtype=np.uint8)
    mask[0, :, :21] = 1
    w.v[0, 0, 20] = np.inf
    q, k, v = kv_tensors(w)
    out, _ = gpu_attention(q, k, v, *lists(mask, w.n))
    assert np.isposinf(out[0, 0]).all() and np.isfinite(out[0, 1]).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_many_kv_heads_in_16_bits(dtype, d):
    """More than 512 kv heads are beyond the 16-bit kernel's tables."""
    w = W.llama8b_layer(seed=2, B=1, n=40, H_q=1026, H_kv=513, T=3, d=d, dtype=dtype)
    mask = oracle.topp_select(w.probs.reshape(-1, w.n), w.top_p).mask().reshape(w.B, w.H_kv, w.n)
    q, k, v = kv_tensors(w)
    out, _ = gpu_attention(q, k, v, *lists(mask, w.n))
    assert row_rel_err(out, oracle_attention(w, mask)[0]) <= TOL["f32"]


@pytest.mark.parametrize("mode", ["table", "physical"])
def test_paged_layouts(mode):
    w = W.ragged_paged(seed=5, B=3, len_lo=50, len_hi=3000, H_q=8, H_kv=2, T=4, d=64)
    w.dtype = "f32"
    mask = oracle.topp_select(w.probs.reshape(-1, w.n), w.top_p, np.repeat(w.seq_lens, w.H_kv)).mask().reshape(w.B, w.H_kv, w.n)
    idx, cnt = lists(mask, w.n)
    if mode == "physical":
        i, c = idx.cpu().numpy(), cnt.cpu().numpy()
        for r in range(i.shape[0]):
            i[r, :c[r]] = w.page_table[r // w.H_kv, i[r, :c[r]] // W.PAGE_SIZE] * W.PAGE_SIZE + i[r, :c[r]] % W.PAGE_SIZE
        idx = dev(i)
    q, k, v = kv_tensors(w)
    out, _ = gpu_attention(q, k, v, idx, cnt, page_table=dev(w.page_table) if mode == "table" else None,
                           page_size=W.PAGE_SIZE, physical=mode == "physical", n_max=w.n)
    assert row_rel_err(out, oracle_attention(w, mask)[0]) <= TOL["f32"]
