"""Chunk-granular selection (chunk masses, exact top-p over them) and attention over chunk lists, against the
oracle: chunk lists and thresholds bit-exact off the near-boundary rows, outputs within the attention tolerance."""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_27641_amd import binding as sa
from paper_2510_27641_amd import workloads as W

from helpers import TOL, compare_select, dev, kv_tensors, oracle_attention, row_rel_err

pytestmark = pytest.mark.gpu


def gpu_select_chunks(probs, top_p, chunk, *, seq_lens=None, capacity=None):
    p = dev(probs)
    B, H, n = p.shape
    R = B * H
    nc = (n + chunk - 1) // chunk
    cap = nc if capacity is None else capacity
    idx = torch.full((R, cap), -7, dtype=torch.int32, device="cuda")
    counts = torch.full((R,), -7, dtype=torch.int32, device="cuda")
    tau = torch.full((R,), -7.0, dtype=torch.float32, device="cuda")
    flags = torch.full((R,), 0x7FFFFFFF, dtype=torch.int32, device="cuda")
    sl = None if seq_lens is None else dev(np.asarray(seq_lens, dtype=np.int32))
    a = sa.select_args(p, top_p, indices=idx, counts=counts, thresholds=tau, row_flags=flags, seq_lens=sl,
                       chunk_size=chunk)
    ws = sa.alloc_workspace(sa.specattn_workspace_size(a, None))
    sa.specattn_topp_select(a, ws)
    torch.cuda.synchronize()
    return dict(indices=idx.cpu().numpy(), counts=counts.cpu().numpy(), tau=tau.cpu().numpy(),
                flags=flags.cpu().numpy().astype(np.uint32), d_indices=idx, d_counts=counts, d_lens=sl)


@pytest.mark.parametrize("chunk", [2, 16, 64])
@pytest.mark.parametrize("n", [16, 1000, 4096, 40000])
def test_chunk_lists_match_oracle(chunk, n):
    rng = np.random.default_rng(n + chunk)
    probs = W.draft_probs(rng, 6, n).reshape(2, 3, n)
    got = gpu_select_chunks(probs, 0.9, chunk)
    ref = oracle.topp_select_chunks(probs.reshape(6, n), 0.9, chunk)
    flagged, mism = compare_select(got, ref)
    assert mism == 0


def test_ragged_lengths_partial_chunks_and_invalid_rows():
    rng = np.random.default_rng(3)
    lens = np.array([5000, 0, 4999, 17, 16, 1], dtype=np.int32)
    probs = W.draft_probs(rng, 12, 5000, lens=np.repeat(lens, 2)).reshape(6, 2, 5000)
    probs[0, 1, 77] = -1.0                     # hides inside a positive chunk mass unless checked per entry
    got = gpu_select_chunks(probs, 0.95, 16, seq_lens=lens)
    ref = oracle.topp_select_chunks(probs.reshape(12, 5000), 0.95, 16, lens=np.repeat(lens, 2))
    flagged, mism = compare_select(got, ref)
    assert mism == 0
    assert got["flags"][1] & sa.ROW_INVALID and got["flags"][2] & sa.ROW_INVALID


@pytest.mark.parametrize("B,H,n,chunk", [(64, 17, 3000, 16), (64, 17, 20003, 16), (60, 18, 9001, 4), (64, 17, 49153, 16), (64, 17, 60001, 64)])
def test_more_ragged_rows_than_fit_the_chip(B, H, n, chunk):
    """Chunk sums of rows that the workgroups take in turns, in the order of the batch and, long ones, from the longest sequence down
    (lengths that are no whole chunks, one length, an empty row)."""
    rng = np.random.default_rng(B * n)
    lens = rng.integers(0, n + 1, size=B).astype(np.int32)
    lens[: B // 3] = lens[0]
    lens[-1], lens[B // 3] = 0, n
    probs = W.draft_probs(rng, 8, n)[rng.integers(0, 8, size=B * H)].reshape(B, H, n)
    probs *= np.exp2(rng.integers(-3, 4, size=(B, H, 1))).astype(np.float32)     # (no two rows alike)
    got = gpu_select_chunks(probs, 0.9, chunk, seq_lens=lens)
    ref = oracle.topp_select_chunks(probs.reshape(B * H, n), 0.9, chunk, lens=np.repeat(lens, H))
    flagged, _ = compare_select(got, ref)
    assert flagged < B * H // 2


@pytest.mark.parametrize("paged", [False, True])
def test_attention_over_chunk_lists(paged):
    if paged:
        w = W.ragged_paged(seed=11, B=5, len_lo=40, len_hi=6000)
        lens = w.seq_lens
    else:
        w = W.llama8b_layer(seed=12, B=3, n=5000, top_p=0.9)
        lens = np.array([5000, 4097, 33], dtype=np.int32)        # partial last chunks (the recency band keeps them)
        w.seq_lens = lens
        for b in range(3):
            w.probs[b, :, lens[b]:] = 0.0
    B, H, n = w.probs.shape
    got = gpu_select_chunks(w.probs, w.top_p, 16, seq_lens=lens)
    ref = oracle.topp_select_chunks(w.probs.reshape(B * H, n), w.top_p, 16, lens=np.repeat(lens, H))
    flagged, mism = compare_select(got, ref)
    assert mism == 0
    mask = oracle.chunk_token_mask(ref, 16, n, np.repeat(lens, H)).reshape(B, H, n)
    q, k, v = kv_tensors(w)
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
    lse = torch.full(q.shape[:3], float("nan"), dtype=torch.float32, device="cuda")
    pt = dev(w.page_table) if paged else None
    a = sa.attn_args(q, k, v, out=out, lse=lse, indices=got["d_indices"], counts=got["d_counts"], seq_lens=got["d_lens"],
                     page_table=pt, page_size=W.PAGE_SIZE if paged else 0, n_max=n, chunk_size=16)
    ws = sa.alloc_workspace(sa.specattn_workspace_size(None, a))
    a.workspace, a.workspace_bytes = ws.data_ptr(), ws.numel()
    sa.specattn_sparse_decode_attn(a)
    torch.cuda.synchronize()
    o_ref, l_ref = oracle_attention(w, mask)
    assert row_rel_err(out.cpu().numpy(), o_ref) <= TOL["bf16"]
    assert np.abs(lse.cpu().numpy() - l_ref).max() <= 1e-3


def test_tiny_fp32_chunks_through_the_portable_kernel():
    w = W.tiny_f32(seed=13)
    B, H, n = w.probs.shape
    got = gpu_select_chunks(w.probs, 0.9, 16)
    ref = oracle.topp_select_chunks(w.probs.reshape(B * H, n), 0.9, 16)
    assert compare_select(got, ref)[1] == 0
    mask = oracle.chunk_token_mask(ref, 16, n).reshape(B, H, n)
    q, k, v = kv_tensors(w)
    out = torch.empty(q.shape, dtype=torch.float32, device="cuda")
    a = sa.attn_args(q, k, v, out=out, indices=got["d_indices"], counts=got["d_counts"], chunk_size=16)
    ws = sa.alloc_workspace(sa.specattn_workspace_size(None, a))
    a.workspace, a.workspace_bytes = ws.data_ptr(), ws.numel()
    sa.specattn_sparse_decode_attn(a)
    torch.cuda.synchronize()
    o_ref, _ = oracle_attention(w, mask)
    assert row_rel_err(out.cpu().numpy(), o_ref) <= TOL["f32"]


@pytest.mark.parametrize("rows", [3, 600])
@pytest.mark.parametrize("n, chunk", [(1, 2), (7, 2), (2049, 2), (4095, 2), (4097, 2), (8191, 2), (8192, 2), (8193, 2), (16383, 16)])
def test_rows_at_the_edges_of_the_chunk_summing_selection(rows, n, chunk):
    """Up to 4096 chunks the selection adds the chunks up itself, one more and they come through memory; few and many rows
    take different workgroups; last chunks are partial, rows start off 16-byte boundaries, one row is invalid."""
    rng = np.random.default_rng(n + rows)
    lens = rng.integers(0, n + 1, size=rows).astype(np.int32)
    lens[0] = n
    probs = W.draft_probs(rng, rows, n, lens=np.maximum(lens, 1))
    probs[1, 0] = -1.0
    lens[1] = n
    got = gpu_select_chunks(probs.reshape(rows, 1, n), 0.95, chunk, seq_lens=lens)
    ref = oracle.topp_select_chunks(probs, 0.95, chunk, lens=lens)
    flagged, mism = compare_select(got, ref)
    assert mism == 0
    assert got["flags"][1] & sa.ROW_INVALID and got["counts"][1] == 0


@pytest.mark.parametrize("rows", [3, 80])
def test_few_long_rows_of_chunks_come_through_memory(rows):
    """Rows of 60000 positions or more: their masses come through memory unless there are many of them."""
    n, chunk = 60001, 32
    probs = W.draft_probs(np.random.default_rng(rows), rows, n)
    got = gpu_select_chunks(probs.reshape(rows, 1, n), 0.9, chunk)
    ref = oracle.topp_select_chunks(probs, 0.9, chunk)
    flagged, mism = compare_select(got, ref)
    assert mism == 0


def chunk_masses(row, chunk):
    """fp64 sums of the row's chunks, rounded to fp32 (as the definition has them)."""
    row = np.pad(row.astype(np.float64), (0, -row.size % chunk)).reshape(-1, chunk)
    return row.cumsum(1)[:, -1].astype(np.float32).astype(np.float64)


def least_kept_at_top_p_one(mass):
    """The least positive entry but, from the smallest octave up, those octaves that together add less than a unit in the last place of the sum."""
    octave = np.frexp(np.maximum(mass, 2.0 ** -127))[1]
    low = [x for x in range(-126, 129) if mass[octave <= x].sum() < np.spacing(mass.sum())]
    return mass[(mass > 0) & (octave > (max(low) if low else -127))].min()


@pytest.mark.parametrize("rows", [9, 603])
@pytest.mark.parametrize("chunks", [1, 2, 15, 63, 64, 65, 127, 128, 129])
def test_short_rows_of_chunks(rows, chunks):
    """Rows of up to 128 chunks compare their masses with each other: of every kind, shorter ones among them, the last chunk partial."""
    n = chunks * 16 - 3
    rng = np.random.default_rng(chunks)
    z = rng.standard_normal((9, n))
    kinds = np.exp(2.0 * z)
    kinds[1] = 1.0                                             # ties (but for the last chunk)
    kinds[2] = np.where(np.arange(n) // 16 % 3 == 1, kinds[2], 0.0)           # chunks without mass
    kinds[2, 0] += 1.0
    kinds[3] = kinds[3] * 2.0 ** -140                          # subnormal entries and masses
    kinds[4] = 2.0 ** -(np.arange(n) // 16).astype(float)      # one octave down per chunk
    kinds[5, -1] = np.inf
    kinds[6] = 3e38                                            # finite entries, infinite masses
    kinds[7] = 0.0
    kinds[8] = np.exp(10.0 * z[8])
    lens = np.where(np.arange(rows) % 2 == 0, n, np.maximum(1, n - np.arange(rows) % n)).astype(np.int32)
    lens[:9] = n
    probs = np.ascontiguousarray(kinds.astype(np.float32)[np.arange(rows) % 9])
    for p in (0.3, 0.9, 0.99999, 1.0):
        got = gpu_select_chunks(probs.reshape(rows, 1, n), p, 16, seq_lens=lens)
        ref = oracle.topp_select_chunks(probs, p, 16, lens=lens)
        _, mism = compare_select(got, ref)
        if p < 1.0:
            assert mism == 0
        else:                                                  # (every valid row is flagged, and the oracle stops one entry at a time)
            for r in list(range(9)) + [rows - 1]:
                if r % 9 not in (5, 6, 7):
                    mass = chunk_masses(probs[r, :lens[r]], 16)
                    keep = np.flatnonzero(mass >= least_kept_at_top_p_one(mass))
                    assert got["counts"][r] == keep.size and np.array_equal(got["indices"][r, :keep.size], keep), r
        if n > 16:
            assert got["flags"][5] & sa.ROW_INVALID and got["flags"][6] & sa.ROW_INVALID and got["flags"][7] & sa.ROW_INVALID


@pytest.mark.parametrize("rows,chunks", [(8, 40), (8, 1500), (8, 4096), (520, 40), (520, 1500), (520, 2048), (520, 4000)])
def test_short_rows_in_calls_of_long_ones(rows, chunks):
    """Rows of up to 128 chunks beside longer ones, in every shape of workgroup that adds chunks up: what is compared lies in LDS
    behind all the masses that the workgroup has room for.  Nothing is written behind a row's list."""
    n = chunks * 4
    rng = np.random.default_rng(rows + chunks)
    lens = np.minimum(n, np.array([1, 4, 5, 255, 256, 257, 509, 512, 513, n])[np.arange(rows) % 10]).astype(np.int32)
    probs = W.draft_probs(rng, rows, n, lens=lens, recency_len=4)
    got = gpu_select_chunks(probs.reshape(rows, 1, n), 0.97, 4, seq_lens=lens)
    ref = oracle.topp_select_chunks(probs, 0.97, 4, lens=lens)
    assert compare_select(got, ref)[1] == 0
    assert all((got["indices"][r, got["counts"][r]:] == -7).all() for r in range(rows))


@pytest.mark.parametrize("chunk", [2, 4, 8, 16, 32, 1024])
@pytest.mark.parametrize("rows", [6, 70])
def test_odd_entries_in_whole_chunks(rows, chunk):
    """Entries that send a chunk's sum the long way: -0.0 counts as zero, negative, infinite and NaN entries make the row invalid, wherever in
    the chunk they are; with the sums in the selection (few long rows: in a kernel of their own)."""
    for n in ([5 * chunk + 3] if rows > 6 else [5 * chunk + 3, 60000 + chunk]):
        rng = np.random.default_rng(chunk + n)
        probs = (rng.random((rows, n)) + 0.01).astype(np.float32)
        at = chunk + rng.integers(0, chunk, rows)
        bad = np.array([-0.0, -1e-30, np.inf, np.nan, -np.inf, np.float32(2.0 ** -149)], dtype=np.float32)[np.arange(rows) % 6]
        probs[np.arange(rows), at] = bad
        got = gpu_select_chunks(probs.reshape(rows, 1, n), 0.7, chunk)
        ref = oracle.topp_select_chunks(probs, 0.7, chunk)
        assert compare_select(got, ref)[1] == 0
        assert np.array_equal((got["flags"] & sa.ROW_INVALID) != 0, ~np.isin(np.arange(rows) % 6, (0, 5)))
