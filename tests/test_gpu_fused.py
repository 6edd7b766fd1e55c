"""GPU parity of specattn_fused (selection + attention without an index list in HBM) against
oracle selection followed by oracle masked attention."""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_27641_amd import binding as sa
from paper_2510_27641_amd import workloads as W
from helpers import TOL, dev, kv_tensors, oracle_attention, row_rel_err

pytestmark = pytest.mark.gpu


def _fused(w, *, reuse=False, give_state=False, want_lse=True):
    """Run specattn_fused on workload w; returns (out, lse, counts, tau)."""
    q, k, v = kv_tensors(w)
    probs = dev(w.probs)
    R = w.B * w.H_kv
    counts = torch.full((R,), -7, dtype=torch.int32, device="cuda")
    sl = None if w.seq_lens is None else dev(w.seq_lens.astype(np.int32))
    pt = None if w.page_table is None else dev(w.page_table)
    nblk = (w.n + sa.SEL_BLOCK - 1) // sa.SEL_BLOCK
    tau = torch.zeros((R,), dtype=torch.float32, device="cuda") if (give_state or reuse) else None
    bc = torch.full((R, nblk), -1, dtype=torch.int32, device="cuda") if (give_state or reuse) else None
    km = torch.full((R, nblk * 32), -1, dtype=torch.int32, device="cuda") if (give_state or reuse) else None
    out = torch.full((w.B, w.H_q, w.T, w.d), float("nan"), dtype=torch.float32, device="cuda")
    lse = torch.full((w.B, w.H_q, w.T), float("nan"), dtype=torch.float32, device="cuda") if want_lse else None
    if reuse:      # the threshold phase as a separate (batchable) call that writes no index list
        s0 = sa.select_args(probs, w.top_p, indices=None, counts=counts, thresholds=tau, seq_lens=sl,
                            block_counts=bc, kept_mask=km)
        sa.specattn_topp_select(s0)
    sel = sa.select_args(probs, w.top_p, indices=None, counts=counts, thresholds=tau, seq_lens=sl,
                         block_counts=bc, kept_mask=km, reuse_selection=reuse)
    kw = dict(page_table=pt, page_size=W.PAGE_SIZE, n_max=w.n) if pt is not None else dict(n_max=w.n)
    att = sa.attn_args(q, k, v, out=out, lse=lse, seq_lens=sl, **kw)
    ws = sa.alloc_workspace(sa.specattn_workspace_size(sel, att))
    att.workspace, att.workspace_bytes = ws.data_ptr(), ws.numel()
    sa.specattn_fused(sel, att)
    torch.cuda.synchronize()
    return (out.cpu().numpy(), None if lse is None else lse.cpu().numpy(), counts.cpu().numpy(),
            None if tau is None else tau.cpu().numpy())


def test_kept_mask_and_block_counts_equal_the_oracle_set():
    """The selection state the fused call works from: one bit per position and kept counts per 1024 positions,
    bit for bit the oracle's kept set (off the rows the oracle flags as near the boundary)."""
    for w in (W.llama8b_layer(seed=8, B=2, n=5000, top_p=0.9), W.ragged_paged(seed=4, B=6, len_lo=50, len_hi=7000),
              W.llama8b_layer(seed=9, B=1, n=70001, H_q=8, H_kv=2, top_p=0.95)):
        probs = dev(w.probs)
        R = w.B * w.H_kv
        nblk = (w.n + sa.SEL_BLOCK - 1) // sa.SEL_BLOCK
        counts = torch.full((R,), -7, dtype=torch.int32, device="cuda")
        bc = torch.full((R, nblk), -1, dtype=torch.int32, device="cuda")
        km = torch.full((R, nblk * 32), -1, dtype=torch.int32, device="cuda")
        sl = None if w.seq_lens is None else dev(w.seq_lens.astype(np.int32))
        sa.specattn_topp_select(sa.select_args(probs, w.top_p, indices=None, counts=counts, seq_lens=sl,
                                               block_counts=bc, kept_mask=km))
        torch.cuda.synchronize()
        ref = oracle.topp_select(w.probs.reshape(-1, w.n), w.top_p, w.row_lens())
        want = np.zeros((R, nblk * 1024), dtype=np.uint8)
        want[:, :w.n] = ref.mask().reshape(R, w.n)
        got = np.unpackbits(km.cpu().numpy().view(np.uint8), axis=1, bitorder="little")
        clear = (ref.flags & oracle.ROW_NEAR_BOUNDARY) == 0
        assert clear.any()
        assert np.array_equal(got[clear], want[clear])
        assert np.array_equal(bc.cpu().numpy()[clear], want.reshape(R, nblk, 1024).sum(axis=2)[clear])
        assert np.array_equal(counts.cpu().numpy()[clear], ref.counts[clear])


def _reference(w, which=None):
    ref = oracle.topp_select(w.probs.reshape(-1, w.n), w.top_p, w.row_lens())
    mask = ref.mask().reshape(w.B, w.H_kv, w.n)
    o, lse = oracle_attention(w, mask, which=which)
    return ref, o, lse


def _check_counts(counts, ref):
    clear = (ref.flags & oracle.ROW_NEAR_BOUNDARY) == 0
    assert np.array_equal(counts[clear], ref.counts[clear])


@pytest.mark.parametrize("mode", ["one_call", "state_given", "reuse"])
def test_llama_layer_8k(mode):
    w = W.llama8b_layer(seed=1)
    out, lse, counts, tau = _fused(w, reuse=(mode == "reuse"), give_state=(mode == "state_given"))
    ref, o, l = _reference(w)
    _check_counts(counts, ref)
    assert row_rel_err(out, o) <= TOL["bf16"]
    assert np.abs(lse - l).max() <= 2e-3
    if tau is not None:
        clear = (ref.flags & oracle.ROW_NEAR_BOUNDARY) == 0
        assert np.array_equal(tau[clear], ref.tau[clear])


def test_batch_of_32k_rows_sampled():
    w = W.llama8b_layer(seed=3, B=2, n=32768, top_p=0.9)
    out, _, counts, _ = _fused(w)
    rng = np.random.default_rng(1)
    which = [(int(rng.integers(w.B)), int(rng.integers(w.H_q)), int(rng.integers(w.T))) for _ in range(48)]
    ref, o, _ = _reference(w, which=which)
    _check_counts(counts, ref)
    got = np.stack([out[b, h, t] for b, h, t in which])
    assert row_rel_err(got, o) <= TOL["bf16"]


@pytest.mark.parametrize("n", [33, 1000, 1024, 1025, 5000, 70001])
def test_row_lengths(n):
    w = W.llama8b_layer(seed=20 + n % 7, B=2, n=n, H_q=8, H_kv=2, top_p=0.9)
    out, _, counts, _ = _fused(w)
    ref, o, _ = _reference(w)
    _check_counts(counts, ref)
    assert row_rel_err(out, o) <= TOL["bf16"]


def test_sparse_rows_whose_tiles_span_many_mask_words():
    """Kept positions far apart: the 32 positions of a tile lie in more than the 64 mask words fetched ahead
    (row 0: one kept position in about 130; row 1: two clusters 30000 positions apart; row 2: 3 kept positions;
    row 3 as drawn), so the on-chip decode takes further rounds over the following words."""
    w = W.llama8b_layer(seed=31, B=1, n=40000, H_q=8, H_kv=4, top_p=0.9)
    rng = np.random.default_rng(5)
    base = rng.random((3, w.n)).astype(np.float32) * 1e-9
    spikes = np.sort(rng.choice(w.n, size=300, replace=False))
    base[0, spikes] = 1.0 + rng.random(300).astype(np.float32)
    base[1, 100:140] = 1.0
    base[1, 30100:30140] = 1.0
    base[2, [5, 20000, 39999]] = 1.0
    w.probs[0, :3] = base
    out, lse, counts, _ = _fused(w)
    ref, o, l = _reference(w)
    _check_counts(counts, ref)
    assert 200 < counts[0] < 300 and counts[1] == 80 and counts[2] == 3      # (ties at the threshold are all kept)
    assert row_rel_err(out, o) <= TOL["bf16"]
    assert np.abs(lse - l).max() <= 2e-3


def _rows_of_every_density(rng, R, n, first):
    """Kept rows [R, n], row r of kind (first + r) % 8: all positions, all but a few, words full and words empty in turns, one in 4, one in 50,
    one in 300, the ends of the blocks, six in ten; one of the last two positions is always kept."""
    kept = np.zeros((R, n), dtype=bool)
    pos = np.arange(n)
    for r in range(R):
        kind = (first + r) % 8
        if kind == 2:
            kept[r] = (pos >> 5) % 3 == 0
        elif kind == 6:
            kept[r] = (pos % 1024 >= 900) | (pos > n - 7)
        else:
            kept[r] = rng.random(n) < (2.0, 0.998, 0.0, 0.25, 0.02, 1 / 300, 0.0, 0.6)[kind]
        kept[r, n - 1 - r % 2] = True
    return kept


def _sparse_rows(rng, R, n, densities):
    """Kept rows [R, n], a part densities[r % len] of row r's positions at random; row 1 keeps none in its middle half."""
    kept = np.stack([rng.random(n) < densities[r % len(densities)] for r in range(R)])
    kept[1, n // 4:3 * n // 4] = False
    return kept


def _check_mask_against_lists(kept, B, H_q, H_kv, T, shared_pool=False):
    """The fused call over a given selection state against the attention over the same positions as lists.  shared_pool: all sequences
    read the same pages, each in an order of its own."""
    R, n = kept.shape
    nblk = -(-n // sa.SEL_BLOCK)
    counts = kept.sum(axis=1).astype(np.int32)
    idx = np.zeros((R, n), dtype=np.int32)
    for r in range(R):
        idx[r, :counts[r]] = np.flatnonzero(kept[r])
    padded = np.zeros((R, nblk * sa.SEL_BLOCK), dtype=np.uint8)
    padded[:, :n] = kept
    bc = dev(padded.reshape(R, nblk, -1).sum(axis=2).astype(np.int32))
    km, d_idx = dev(np.packbits(padded, axis=1, bitorder="little").view(np.int32)), dev(idx)
    gen = torch.Generator(device="cuda").manual_seed(n)
    draw = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    q, kw = draw(B, H_q, T, 128), {}
    if shared_pool:
        pages = -(-n // W.PAGE_SIZE)
        order = np.stack([np.random.default_rng(b).permutation(pages) for b in range(B)]).astype(np.int32)
        kw = dict(page_table=dev(order), page_size=W.PAGE_SIZE, n_max=n)
        k, v = draw(pages, H_kv, W.PAGE_SIZE, 128), draw(pages, H_kv, W.PAGE_SIZE, 128)
    else:
        k, v = draw(B, H_kv, n, 128), draw(B, H_kv, n, 128)
    outs = []
    for fused in (False, True):
        out = torch.full((B, H_q, T, 128), float("nan"), device="cuda")
        d_counts = dev(counts)
        if fused:
            probs = torch.full((B, H_kv, n), 1.0 / n, device="cuda")
            tau = torch.zeros(R, device="cuda")
            sel = sa.select_args(probs, 0.9, indices=None, counts=d_counts, thresholds=tau, block_counts=bc, kept_mask=km, reuse_selection=True)
            att = sa.attn_args(q, k, v, out=out, **kw)
        else:
            sel, att = None, sa.attn_args(q, k, v, out=out, indices=d_idx, counts=d_counts, **kw)
        ws = sa.alloc_workspace(sa.specattn_workspace_size(sel, att))
        att.workspace, att.workspace_bytes = ws.data_ptr(), ws.numel()
        if fused:
            sa.specattn_fused(sel, att)
        else:
            sa.specattn_sparse_decode_attn(att)
        torch.cuda.synchronize()
        outs.append(out.cpu().numpy())
    # (the same weights and products, summed in another order: fp32 sums of 16-bit weight parts, 2.4e-6 against 64 bits)
    assert row_rel_err(outs[1], outs[0]) <= 2e-5


@pytest.mark.parametrize("B,H_q,H_kv,T,n,first", [(1, 8, 2, 5, 40000, 0), (1, 8, 2, 5, 40000, 2), (1, 8, 2, 5, 40000, 4), (1, 8, 2, 5, 40000, 6),
                                                  (3, 24, 2, 4, 9001, 0), (18, 8, 4, 3, 2500, 0)])
def test_positions_of_any_density_come_out_of_the_mask(B, H_q, H_kv, T, n, first):
    """Rows of every density against the same attention over lists, a few tiles to a wave: two query tiles, three, and more rows than a wave scans by itself."""
    rng = np.random.default_rng(n)
    _check_mask_against_lists(_rows_of_every_density(rng, B * H_kv, n, first), B, H_q, H_kv, T)


@pytest.mark.parametrize("B,H_q,H_kv,T,n,first,shared_pool", [(2, 8, 8, 5, 131072, 0, False), (2, 32, 8, 5, 131072, 3, False), (2, 64, 8, 6, 100001, 5, True),
                                                              (9, 32, 8, 1, 30000, 1, False), (9, 32, 8, 5, 30000, 6, True), (11, 40, 10, 8, 20011, 4, True), (11, 60, 10, 8, 20011, 7, False)])
def test_waves_that_take_many_tiles_from_the_mask(B, H_q, H_kv, T, n, first, shared_pool):
    """8 and more tiles of a row to a wave, so that its buffer of positions is filled again and again inside the tile loop and what is left in it moves to the front;
    rows of up to 128 blocks (two rounds of the search for a wave's first one); up to 64 rows and more, one to three query tiles."""
    rng = np.random.default_rng(n + first)
    _check_mask_against_lists(_rows_of_every_density(rng, B * H_kv, n, first), B, H_q, H_kv, T, shared_pool)


@pytest.mark.parametrize("B,H_kv,G,T,densities", [(8, 8, 4, 5, (1 / 40, 1 / 50, 1 / 70, 1 / 100)), (8, 8, 1, 3, (1 / 50, 1 / 66, 1 / 80, 1 / 60)), (8, 8, 8, 5, (1 / 70,)),
                                                  (24, 4, 4, 5, (1 / 100,)), (24, 4, 2, 5, (1 / 60, 1 / 300, 1 / 90)), (24, 4, 8, 5, (1 / 80,)), (96, 4, 4, 4, (1 / 300,))])
def test_waves_that_take_sparse_tiles_from_the_mask(B, H_kv, G, T, densities):
    """Three and more tiles to a wave whose positions span more than the 64 words fetched ahead, so that a tile's positions are completed from memory
    inside the tile loop; rows of 256 blocks, a pool shared by all sequences."""
    n = 262144
    rng = np.random.default_rng(B + G)
    _check_mask_against_lists(_sparse_rows(rng, B * H_kv, n, densities), B, G * H_kv, H_kv, T, shared_pool=True)


@pytest.mark.parametrize("B", [80, 200])
def test_many_rows_through_the_mask_source(B):
    # 640 rows (two rounds of the workgroup-wide cost prefix) and 1600 rows (1536 + 64: two launches)
    w = W.llama8b_layer(seed=33, B=B, n=300, H_q=16, H_kv=8, T=2, top_p=0.8)
    out, lse, counts, _ = _fused(w)
    ref, o, l = _reference(w)
    _check_counts(counts, ref)
    assert row_rel_err(out, o) <= TOL["bf16"]


def test_paged_ragged_batch_through_page_table():
    w = W.ragged_paged(seed=4, B=6, len_lo=50, len_hi=7000)
    out, lse, counts, _ = _fused(w)
    ref, o, l = _reference(w)
    _check_counts(counts, ref)
    assert row_rel_err(out, o) <= TOL["bf16"]


def test_invalid_and_empty_rows_give_zero_output():
    w = W.llama8b_layer(seed=5, n=3000, H_q=8, H_kv=4)
    w.probs[0, 1, 17] = np.nan
    w.probs[0, 2, :] = 0.0
    out, lse, counts, _ = _fused(w)
    ref, o, l = _reference(w)
    assert counts[1] == 0 and counts[2] == 0
    G = w.G
    assert (out[0, 1 * G:(2 + 1) * G] == 0).all()
    assert np.isneginf(lse[0, 1 * G:(2 + 1) * G]).all()
    assert row_rel_err(out, o) <= TOL["bf16"]


def test_top_p_one_selects_everything():
    w = W.llama8b_layer(seed=6, n=2100, top_p=1.0, H_q=8, H_kv=2)
    out, _, counts, _ = _fused(w)
    ref, o, _ = _reference(w)
    assert (counts == 2100).all()
    assert row_rel_err(out, o) <= TOL["bf16"]


def test_tiny_fp32_workload_through_the_fused_entry():
    """fp32, d = 64: the fused entry runs the selection into its workspace and attends over that list."""
    w = W.tiny_f32()
    out, lse, counts, _ = _fused(w)
    ref, o, l = _reference(w)
    _check_counts(counts, ref)
    assert row_rel_err(out, o) <= TOL["f32"]
    assert np.abs(lse - l).max() <= 1e-4
    with pytest.raises(sa.SpecAttnError) as e:          # the on-chip selection state does not exist on this route
        _fused(w, give_state=True)
    assert e.value.status == sa.EUNSUPPORTED


@pytest.mark.parametrize("chunk", [16, 64])
def test_chunk_granular_selection_through_the_fused_entry(chunk):
    """sel.chunk_size > 1: top-p over chunk masses, attention over every position of the kept chunks."""
    w = W.llama8b_layer(seed=13, B=2, n=5000, top_p=0.9)
    q, k, v = kv_tensors(w)
    probs = dev(w.probs)
    R = w.B * w.H_kv
    counts = torch.full((R,), -7, dtype=torch.int32, device="cuda")
    out = torch.full((w.B, w.H_q, w.T, w.d), float("nan"), dtype=torch.float32, device="cuda")
    sel = sa.select_args(probs, w.top_p, indices=None, counts=counts, chunk_size=chunk)
    att = sa.attn_args(q, k, v, out=out, n_max=w.n)
    ws = sa.alloc_workspace(sa.specattn_workspace_size(sel, att))
    att.workspace, att.workspace_bytes = ws.data_ptr(), ws.numel()
    sa.specattn_fused(sel, att)
    torch.cuda.synchronize()
    ref = oracle.topp_select_chunks(w.probs.reshape(-1, w.n), w.top_p, chunk)
    clear = (ref.flags & oracle.ROW_NEAR_BOUNDARY) == 0
    assert np.array_equal(counts.cpu().numpy()[clear], ref.counts[clear])
    mask = oracle.chunk_token_mask(ref, chunk, w.n, np.full(R, w.n, dtype=np.int32)).reshape(w.B, w.H_kv, w.n)
    o, _ = oracle_attention(w, mask)
    assert row_rel_err(out.cpu().numpy(), o) <= TOL["bf16"]


@pytest.mark.parametrize("n,chunk", [(1030, 1024), (1025, 512), (1279, 256), (1280, 256)])
def test_rows_just_above_whole_chunks_run_in_the_size_asked_for(n, chunk):
    """A list of whole chunks stands for more positions than the row has, and its splits for more partials."""
    w = W.llama8b_layer(seed=n, B=8, n=n, H_q=64, H_kv=8, T=2, d=64, dtype="f32", top_p=0.9)
    q, k, v = kv_tensors(w)
    R = w.B * w.H_kv
    counts = torch.full((R,), -7, dtype=torch.int32, device="cuda")
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
    probs = dev(w.probs)
    sel = sa.select_args(probs, w.top_p, indices=None, counts=counts, chunk_size=chunk)
    att = sa.attn_args(q, k, v, out=out, n_max=n)
    ws = sa.alloc_workspace(sa.specattn_workspace_size(sel, att))
    att.workspace, att.workspace_bytes = ws.data_ptr(), ws.numel()
    sa.specattn_fused(sel, att)
    torch.cuda.synchronize()
    ref = oracle.topp_select_chunks(w.probs.reshape(-1, n), w.top_p, chunk)
    assert np.array_equal(counts.cpu().numpy(), ref.counts)
    mask = oracle.chunk_token_mask(ref, chunk, n, np.full(R, n, dtype=np.int32)).reshape(w.B, w.H_kv, n)
    assert row_rel_err(out.cpu().numpy(), oracle_attention(w, mask)[0]) <= TOL["f32"]


def test_physical_indices_do_not_apply_to_the_fused_entry():
    w = W.ragged_paged(seed=4, B=2, len_lo=50, len_hi=900)
    q, k, v = kv_tensors(w)
    probs = dev(w.probs)
    counts = torch.zeros((w.B * w.H_kv,), dtype=torch.int32, device="cuda")
    out = torch.zeros((w.B, w.H_q, w.T, w.d), dtype=torch.float32, device="cuda")
    sel = sa.select_args(probs, w.top_p, indices=None, counts=counts, seq_lens=dev(w.seq_lens.astype(np.int32)))
    att = sa.attn_args(q, k, v, out=out, page_size=W.PAGE_SIZE, n_max=w.n, indices_are_physical=True)
    ws = sa.alloc_workspace(1 << 24)
    att.workspace, att.workspace_bytes = ws.data_ptr(), ws.numel()
    with pytest.raises(sa.SpecAttnError) as e:
        sa.specattn_fused(sel, att)
    assert e.value.status == sa.EUNSUPPORTED
