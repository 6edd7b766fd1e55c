"""GPU parity: specattn_topp_select (HIP, through the C ABI) against the oracle, element by element.

Index lists, counts and thresholds must be bit-exact on every row the oracle does not flag as
near-boundary (kept or strictly-above mass within 1e-6 of p); flagged rows are counted and their
mismatches reported.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_27641_amd import binding as sa
from paper_2510_27641_amd import workloads as W
from helpers import compare_select, dev, gpu_select

pytestmark = pytest.mark.gpu


def _check(probs3, top_p, allow_flagged_mismatch=False, **kw):
    B, H, n = probs3.shape
    lens = kw.get("seq_lens")
    row_lens = None if lens is None else np.repeat(np.asarray(lens, dtype=np.int32), H)
    ref = oracle.topp_select(probs3.reshape(B * H, n), top_p, row_lens)
    got = gpu_select(probs3, top_p, **kw)
    flagged, mism = compare_select(got, ref, capacity=kw.get("capacity"))
    print(f"rows={B * H} n={n} p={top_p} flagged={flagged} flagged_mismatch={mism}")
    if not allow_flagged_mismatch:
        assert mism == 0      # not required by the contract, but expected of fp64 suffix sums
    return got, ref


def test_tiny_f32_workload():
    w = W.tiny_f32()
    _check(w.probs, w.top_p)


def test_llama_layer_8k():
    w = W.llama8b_layer(seed=1, with_kv=False)
    _check(w.probs, w.top_p)


@pytest.mark.parametrize("n", [1, 2, 5, 63, 64, 65, 1000, 1023, 1025, 2047, 3000, 4097, 8191, 12000,
                               16385, 20000, 32768, 40000, 65536])
def test_row_lengths_span_every_kernel_variant(n):
    rng = np.random.default_rng(n)
    probs = W.draft_probs(rng, 6, n, recency_len=min(64, n), spike_frac=0.01).reshape(2, 3, n)
    for p in (0.9, 0.5):
        _check(probs, p)


def test_long_rows_streaming_variant():
    rng = np.random.default_rng(7)
    probs = W.draft_probs(rng, 4, 131072).reshape(2, 2, 131072)
    _check(probs, 0.9)
    probs = W.draft_probs(rng, 2, 70001).reshape(1, 2, 70001)
    _check(probs, 0.95)


def test_32k_batch_like_the_headline_workload():
    w = W.llama8b_layer(seed=3, B=4, n=32768, top_p=0.9, with_kv=False)
    got, ref = _check(w.probs, w.top_p)
    frac = got["counts"].mean() / 32768
    assert 0.15 < frac < 0.35


@pytest.mark.parametrize("top_p", [1.0, 0.999999, 0.99, 0.8, 0.3, 1e-3, 1e-7])
def test_top_p_sweep_including_limits(top_p):
    rng = np.random.default_rng(17)
    probs = W.draft_probs(rng, 8, 5000).reshape(2, 4, 5000)
    got, ref = _check(probs, top_p)
    if top_p == 1.0:
        assert (got["counts"] == 5000).all()
    if top_p == 1e-7:
        assert (got["counts"] == 1).all() and (got["indices"][:, 0] == probs.reshape(8, -1).argmax(1)).all()


def test_heavy_tailed_rows_with_underflowed_zeros():
    w = W.long_context(seed=0, B=1, n=32768, H_kv=4, with_kv=False)
    assert (w.probs == 0).any()
    for p in (0.8, 0.99):
        _check(w.probs, p)
    # p = 1 on a row whose tail lies below 2^-53 of the row sum: the oracle adds its entries one by one and stops where
    # none of them moves the sum, the library where all that are left add less than one unit in its last place
    _check(w.probs, 1.0, allow_flagged_mismatch=True)
    w = W.long_context(seed=1, B=1, n=32768, H_kv=4, logit_clip=8.0, with_kv=False)
    for p in (0.8, 0.9, 0.95, 0.99):
        _check(w.probs, p)


@pytest.mark.parametrize("split", [True, False])
@pytest.mark.parametrize("n", [1000, 4096, 20000, 40000, 100001])
def test_top_p_one_keeps_small_entries_that_add_up(n, split):
    """Entries that are nothing next to the largest one, one by one, but together move the fp64 sum of the row: kept.
    Entries that add less than a unit in its last place (2^-52 of 1.0) all together: not kept."""
    rng = np.random.default_rng(n)
    probs = np.full((1, 6, n), 2.0 ** -54)
    probs[0, 1] = 2.0 ** -70                                   # n of them: below 2^-53
    probs[0, 2, 300:] = 2.0 ** -62                             # 300 of 2^-54 (minus the large one), the others below 2^-46: kept too
    probs[0, 3, 300:] = 2.0 ** -90                             # ... below 2^-73: not kept
    probs[0, 4] = np.where(np.arange(n) < 2, 2.0 ** -54, 0.0)  # 2^-54 or 2^-53: not kept
    probs[0, 5] = np.where(np.arange(n) < 10, 2.0 ** -55, 2.0 ** -140)     # at least 9 * 2^-55, more than 2^-52: kept
    at = rng.integers(0, n, size=6)
    at[2:] = 1
    for r in range(6):
        probs[0, r, at[r]] = 1.0
    got = gpu_select(probs.astype(np.float32), 1.0, split=split)
    want = [n, 1, n if (n - 300) * 2.0 ** -62 >= 2.0 ** -52 else 300, 300, 1, 10]
    assert got["counts"].tolist() == want
    for r in range(6):
        keep = probs[0, r] >= got["tau"][r]
        assert keep.sum() == want[r] and np.array_equal(got["indices"][r, :want[r]], np.flatnonzero(keep))


def test_ties_zeros_denormals_and_scaling():
    rng = np.random.default_rng(23)
    n = 3000
    rows = []
    q = np.round(rng.random(n) * 8) / 8 + 0.125                 # 9 distinct values: massive ties
    rows.append(q)
    rows.append(np.full(n, 0.25))                               # uniform
    z = rng.random(n) ** 4
    z[rng.random(n) < 0.5] = 0.0                                # half zeros
    rows.append(z)
    rows.append(rng.random(n) * 1e-41)                          # all denormal
    mix = rng.random(n) ** 6
    mix[::7] *= 1e-39                                           # denormals among normals
    rows.append(mix)
    rows.append(rng.random(n) * 2.0 ** 100)                     # huge, far from normalised
    one = np.zeros(n)
    one[1234] = 3.0                                             # one non-zero entry
    rows.append(one)
    neg0 = rng.random(n)
    neg0[5] = -0.0
    rows.append(neg0)
    probs = np.stack(rows).astype(np.float32).reshape(1, len(rows), n)
    for p in (0.9, 0.5, 1.0):
        got, ref = _check(probs, p)
    assert got["counts"][1] == n and got["counts"][6] == 1


def test_invalid_rows_are_flagged_and_empty():
    rng = np.random.default_rng(29)
    probs = W.draft_probs(rng, 6, 2000).reshape(1, 6, 2000)
    probs[0, 1, 77] = np.nan
    probs[0, 2, 1999] = -1e-3
    probs[0, 3, :] = 0.0
    probs[0, 4, 3] = np.inf
    got, ref = _check(probs, 0.9)
    assert [bool(f & sa.ROW_INVALID) for f in got["flags"]] == [False, True, True, True, True, False]


def test_sequence_lengths_including_zero():
    rng = np.random.default_rng(31)
    lens = np.array([4096, 1, 0, 777, 4095], dtype=np.int32)
    probs = W.draft_probs(rng, 10, 4096, lens=np.repeat(lens, 2)).reshape(5, 2, 4096)
    probs[3, :, 777:] = 0.5           # garbage past the end must be ignored
    got, ref = _check(probs, 0.9, seq_lens=lens)
    assert (got["counts"][4:6] == 0).all()


def test_capacity_overflow_truncates_and_reports_true_count():
    rng = np.random.default_rng(37)
    probs = W.draft_probs(rng, 4, 8192).reshape(1, 4, 8192)
    got, ref = _check(probs, 0.95, capacity=512)
    assert (got["counts"] > 512).all()
    assert all(f & sa.ROW_OVERFLOW for f in got["flags"])


@pytest.mark.parametrize("capacity", [100, 8192, 9000])
def test_capacity_far_below_a_long_kept_list(capacity):
    # more kept entries than one round of the list staging holds (8192), and a capacity below, at and above that
    rng = np.random.default_rng(38)
    probs = W.draft_probs(rng, 3, 32768).reshape(1, 3, 32768)
    got, ref = _check(probs, 0.995, capacity=capacity)
    assert (got["counts"] > 9000).all()
    assert all(f & sa.ROW_OVERFLOW for f in got["flags"])


def test_strided_and_unaligned_rows():
    rng = np.random.default_rng(41)
    n = 1500
    base = np.zeros((2, 3, 2048 + 3), dtype=np.float32)
    base[:, :, 1:1 + n] = W.draft_probs(rng, 6, n).reshape(2, 3, n)
    t = dev(base)
    view = t[:, :, 1:1 + n]           # rows start 4 bytes off a 16-byte boundary
    ref = oracle.topp_select(base[:, :, 1:1 + n].reshape(6, n), 0.9)
    got = gpu_select(None, 0.9, probs_dev=view)
    assert compare_select(got, ref)[1] == 0


def test_paged_physical_indices():
    w = W.ragged_paged(seed=2, B=5, len_lo=100, len_hi=6000, H_kv=2, H_q=2, with_kv=False)
    ref = oracle.topp_select(w.probs.reshape(-1, w.n), w.top_p, w.row_lens())
    got = gpu_select(w.probs, w.top_p, seq_lens=w.seq_lens, page_table=w.page_table,
                     page_size=W.PAGE_SIZE, emit_physical=True)

    def to_physical(r, pos):
        b = r // w.H_kv
        return w.page_table[b, pos // W.PAGE_SIZE] * W.PAGE_SIZE + pos % W.PAGE_SIZE

    assert compare_select(got, ref, to_physical=to_physical)[1] == 0
    got2 = gpu_select(w.probs, w.top_p, seq_lens=w.seq_lens)       # logical positions
    assert compare_select(got2, ref)[1] == 0


def test_run_to_run_determinism():
    w = W.llama8b_layer(seed=5, B=2, n=16384, with_kv=False)
    a = gpu_select(w.probs, 0.9)
    for _ in range(3):
        b = gpu_select(w.probs, 0.9)
        assert np.array_equal(a["indices"], b["indices"]) and np.array_equal(a["counts"], b["counts"])
        assert np.array_equal(a["tau"], b["tau"]) and np.array_equal(a["flags"], b["flags"])


def test_near_boundary_flag_matches_oracle_on_clear_rows():
    """The device flag is a diagnostic: it must be set on exact hits and clear on wide margins."""
    row = np.array([0.5, 0.25, 0.125, 0.0625, 0.0625], dtype=np.float32).reshape(1, 1, 5)
    assert gpu_select(row, 0.5)["flags"][0] & sa.ROW_NEAR_BOUNDARY
    assert not gpu_select(row, 0.6)["flags"][0] & sa.ROW_NEAR_BOUNDARY


# ---- few long rows: the split path (each row over many workgroups) against the oracle and the one-workgroup path
@pytest.mark.parametrize("rows,n", [(1, 65536), (8, 66000), (3, 70001), (2, 200000), (32, 131072), (64, 131072)])
def test_split_path_matches_oracle_and_single_path(rows, n):
    rng = np.random.default_rng(rows * 7 + n)
    probs = W.draft_probs(rng, rows, n).reshape(1, rows, n)
    got = gpu_select(probs, 0.9)
    assert got["split"], "this shape is expected to take the split path"
    ref = oracle.topp_select(probs.reshape(rows, n), 0.9)
    flagged, mism = compare_select(got, ref)
    assert mism == 0
    one = gpu_select(probs, 0.9, split=False)
    assert np.array_equal(got["counts"], one["counts"]) and np.array_equal(got["tau"], one["tau"])
    assert np.array_equal(got["flags"], one["flags"])
    for r in range(rows):
        assert np.array_equal(got["indices"][r, :got["counts"][r]], one["indices"][r, :one["counts"][r]])


def test_split_path_edge_rows():
    n = 66000
    rng = np.random.default_rng(77)
    probs = W.draft_probs(rng, 8, n).reshape(2, 4, n)
    lens = np.array([n, 20001], dtype=np.int32)
    probs[1] = W.draft_probs(rng, 4, n, lens=np.full(4, 20001))
    probs[0, 0, :] = 0.0; probs[0, 0, 12345] = 1.0            # one entry holds everything (single-entry bins)
    probs[0, 1, :] = np.float32(1.0 / n)                      # all tied: the boundary bin holds the whole row
    probs[0, 2, 777] = np.nan                                 # invalid
    probs[0, 3, :] = 0.0                                      # no mass
    probs[1, 0, 5:15000] = 0.0                                # long run of zeros
    probs[1, 1, 100] = -0.0
    for p in (0.5, 0.9, 1.0):
        got = gpu_select(probs, p, seq_lens=lens, capacity=50000)
        assert got["split"]
        ref = oracle.topp_select(probs.reshape(8, n), p, lens=np.repeat(lens, 4))
        flagged, mism = compare_select(got, ref, capacity=50000)
        assert mism == 0 or p == 1.0
        assert got["counts"][0] == 1 and got["counts"][1] == n
        assert got["flags"][2] & sa.ROW_INVALID and got["flags"][3] & sa.ROW_INVALID
        assert got["flags"][1] & sa.ROW_OVERFLOW


def test_split_path_paged_physical_output():
    w = W.ragged_paged(seed=15, B=2, len_lo=70000, len_hi=90000, with_kv=False)
    got = gpu_select(w.probs, 0.95, seq_lens=w.seq_lens, page_table=w.page_table, page_size=W.PAGE_SIZE, emit_physical=True)
    assert got["split"]
    B, H, n = w.probs.shape
    ref = oracle.topp_select(w.probs.reshape(B * H, n), 0.95, lens=w.row_lens())
    to_phys = lambda r, pos: w.page_table[r // H, pos // W.PAGE_SIZE] * W.PAGE_SIZE + pos % W.PAGE_SIZE
    flagged, mism = compare_select(got, ref, to_physical=to_phys)
    assert mism == 0


@pytest.mark.parametrize("rows,n", [(8, 2047), (520, 2048), (8, 4093), (520, 4095), (9, 8191), (800, 6001), (8, 16383), (300, 16381),
                                    (520, 13001), (520, 15361), (300, 20001), (8, 32767), (5, 40001)])
def test_thread_shapes_and_rows_at_any_address(rows, n):
    """Every shape of workgroup that the row count and the row length lead to, on rows that start at any multiple of four
    bytes (odd lengths): lists, thresholds, bits and block counts."""
    rng = np.random.default_rng(n)
    probs = W.draft_probs(rng, rows, n).reshape(1, rows, n)
    probs[0, 1, n - 1] = 0.5                                   # the entry behind the last whole vector
    probs[0, 2, 3] = -0.0
    got = gpu_select(probs, 0.93, split=False)
    ref = oracle.topp_select(probs.reshape(-1, n), 0.93)
    assert compare_select(got, ref)[1] == 0
    p = dev(probs)
    blocks = -(-n // 1024)
    counts = torch.zeros(rows, dtype=torch.int32, device="cuda")
    bc = torch.full((rows, blocks), -1, dtype=torch.int32, device="cuda")
    bits = torch.full((rows, blocks * 32), -1, dtype=torch.int32, device="cuda")
    sa.specattn_topp_select(sa.select_args(p, 0.93, indices=None, counts=counts, block_counts=bc, kept_mask=bits))
    torch.cuda.synchronize()
    kept = np.unpackbits(bits.cpu().numpy().view(np.uint8), axis=1, bitorder="little")
    assert np.array_equal(kept.sum(1), got["counts"]) and not kept[:, n:].any()
    assert np.array_equal(kept.reshape(rows, blocks, 1024).sum(2), bc.cpu().numpy())
    for r in (0, 1, 2, rows - 1):
        assert np.array_equal(np.flatnonzero(kept[r]), got["indices"][r, :got["counts"][r]])


@pytest.mark.parametrize("rows,n", [(2, 65537), (9, 131075), (40, 200003)])
def test_split_path_flat_rows(rows, n):
    """Rows whose boundary bin holds from a few entries to all of them: kept in LDS, fetched again, or (more than 4096 in
    a slice) read again from the rows; against the path with one workgroup per row."""
    rng = np.random.default_rng(rows)
    spread = np.geomspace(1e-3, 3.0, rows)[:, None]
    logit = spread * rng.standard_normal((rows, n))
    probs = np.exp(logit - logit.max(1, keepdims=True)).astype(np.float32)
    probs /= probs.sum(1, keepdims=True)
    probs[1, ::2] = 0.0
    probs[1, :n // 2] *= np.float32(1e-40) / np.float32(probs[1].max())      # subnormal entries
    probs[0, n - 1] = -0.0
    probs[rows - 1, :] = np.float32(1.0 / n)                   # ties
    for p in (0.6, 0.95):
        got = gpu_select(probs.reshape(1, rows, n), p)
        one = gpu_select(probs.reshape(1, rows, n), p, split=False)
        assert got["split"]
        for k in ("counts", "tau", "flags"):
            assert np.array_equal(got[k], one[k]), k
        assert np.array_equal(got["indices"], one["indices"])


def least_split_bytes(rows, n):
    """32 KiB of counters and a bit per position for every row, with the alignment of each part."""
    a256 = lambda x: -(-x // 256) * 256
    blocks = -(-n // 4096)
    return 3 * a256(rows * 4) + a256(rows * blocks * 4) + a256(rows * blocks * 512) + rows * 32768 + a256(rows * 88)


@pytest.mark.parametrize("rows,n", [(1, 65536), (5, 65539), (32, 131072), (9, 200003), (130, 266241)])
def test_split_path_in_the_least_workspace(rows, n):
    """Less room than is asked for: one histogram per row, and as many collected entries as fit (the flat rows' do not).  The
    results are the same; nothing is written behind the workspace."""
    rng = np.random.default_rng(rows + 1)
    few = min(rows, 12)
    spread = np.geomspace(1e-3, 3.0, few)[:, None]
    logit = spread * rng.standard_normal((few, n), dtype=np.float32)
    probs = np.exp(logit - logit.max(1, keepdims=True)).astype(np.float32)
    probs /= probs.sum(1, keepdims=True)
    probs[0, n - 1] = -0.0
    if few > 4:
        probs[1, ::2] = 0.0
        probs[1, :n // 2] *= np.float32(1e-40) / np.float32(probs[1].max())  # subnormal entries
        probs[2, 77] = np.nan
        probs[3, :] = np.float32(1.0 / n)                                    # ties
    probs = np.resize(probs, (1, rows, n))
    lens = np.array([n - 3], dtype=np.int32)
    least = least_split_bytes(rows, n)
    ws = torch.full((least + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    pr, sl = dev(probs), dev(lens)
    for p in (0.6, 1.0):
        one = gpu_select(None, p, probs_dev=pr, split=False, seq_lens=lens)
        got = gpu_select(None, p, probs_dev=pr, split=least, seq_lens=lens)
        for k in ("counts", "tau", "flags", "indices"):
            assert np.array_equal(got[k], one[k]), k
    idx = torch.full((rows, n), -7, dtype=torch.int32, device="cuda")
    counts = torch.full((rows,), -7, dtype=torch.int32, device="cuda")
    sa.specattn_topp_select(sa.select_args(pr, 1.0, indices=idx, counts=counts, seq_lens=sl), ws[:least])
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), one["indices"]) and (ws[least:] == 0xA5).all().item()
    bits = torch.zeros((rows, -(-n // 1024) * 32), dtype=torch.int32, device="cuda")
    args = sa.select_args(pr, 1.0, indices=idx, counts=counts, seq_lens=sl, kept_mask=bits)
    with pytest.raises(RuntimeError, match="kept_mask"):
        sa.specattn_topp_select(args, ws[:least])
    sa.specattn_topp_select(args, ws[:least // 256 * 256 - 256])             # (not split)
    torch.cuda.synchronize()
    assert np.array_equal(counts.cpu().numpy(), one["counts"])


# every workgroup shape at its edges: (rows, entries) as the launch chooses 256 / 512 / 1024 threads with 1 .. 16 vectors each
SHAPES = [(9, 3), (9, 1024), (9, 1025), (520, 2047), (9, 4096), (515, 4093), (9, 4097), (515, 8192), (9, 8193), (257, 16384),
          (515, 8201), (515, 16383), (9, 16385), (257, 32767), (9, 32769), (9, 36863), (70, 40001), (66, 65536)]


@pytest.mark.parametrize("rows,n", SHAPES)
def test_passes_over_rows_of_every_kind(rows, n):
    """Rows that leave the first pass's window (entries far below the largest one, at and beyond the boundary), whose boundary bin
    holds one, a few, many or all of the entries, or ties alone, subnormal and tiny rows, and zeros."""
    rng = np.random.default_rng(rows + n)
    z = rng.standard_normal((9, n))
    kinds = np.empty((9, n))
    kinds[0] = np.exp(2.0 * z[0])                              # the ordinary kind
    kinds[1] = np.where(rng.random(n) < 0.3, 0.0, np.exp(12.0 * z[1]))        # over 32 octaves and more, zeros
    kinds[2] = 2.0 ** -rng.integers(0, 60, n)                  # one value per octave, half of them below the window
    kinds[3] = 1.0 + rng.random(n) * 2.0 ** -7                 # one bin of the first pass
    kinds[4] = 1.0 + np.floor(rng.random(n) * 3) * 2.0 ** -20  # ... of three values
    kinds[5] = 0.75                                            # ties alone
    kinds[6] = np.exp(2.0 * z[6]) * 2.0 ** -135                # subnormal
    kinds[7] = np.exp(3.0 * z[7]) * 2.0 ** -100                # the window ends at the smallest normal number
    kinds[8] = np.where(np.arange(n) < max(1, n // 2), 1.0, 2.0 ** -40)       # the small half adds nothing to fp32, something to fp64
    probs = np.repeat(kinds.astype(np.float32), -(-rows // 9), axis=0)[:rows].reshape(1, rows, n)
    for p in (0.9, 0.2, 0.9999999):                            # (the last flags every row: _check compares flagged rows, too)
        sub = np.ascontiguousarray(probs if p == 0.9 else probs[:, ::max(1, rows // 9)])
        _check(sub, p)
        if p > 0.99:
            _check(sub, p, split=False)
    got = gpu_select(np.ascontiguousarray(probs[:, ::max(1, rows // 9)]), 1.0)
    for r, row in enumerate(probs[0, ::max(1, rows // 9)].astype(np.float64)):
        # all but the smallest octaves that together add less than a unit in the last place of the sum
        e = np.frexp(np.maximum(row, 2.0 ** -127))[1]
        tail = np.array([row[(e <= x)].sum() for x in range(-126, 129)])
        cut = np.flatnonzero(tail < np.spacing(np.float64(row.sum())))
        least = -126 + cut[-1] if cut.size else -127
        keep = np.flatnonzero((row > 0) & (e > least))
        assert got["counts"][r] == keep.size and np.array_equal(got["indices"][r, :keep.size], keep), r


@pytest.mark.parametrize("values", ["distinct", "tied", "equal"])
@pytest.mark.parametrize("rows,n", [(1, 8193), (1, 16384), (258, 12001), (1, 32767), (258, 20480), (258, 32768), (300, 40001)])
def test_boundary_bins_of_few_entries(rows, n, values):
    """Rows whose threshold lies at the first, a middle and the last entry of a boundary bin (1 to 1 + 1/64) of k entries, below, at and
    beyond the longest list that is compared entry by entry and its halves."""
    rng = np.random.default_rng(n)
    made, taus = [], []
    for k in (1, 2, 3, 4, 5, 31, 32, 33, 63, 64, 65, 66, 127, 128, 129, 200):
        steps = {"distinct": rng.permutation(1 << 17)[:k], "tied": rng.integers(0, 3, k) * 43690, "equal": np.full(k, 77)}[values]
        bin_entries = np.sort(1.0 + steps * 2.0 ** -23)[::-1]
        for j in sorted({0, k // 2, k - 1}):                   # the threshold is the j-th largest
            large = np.full(k // 2 + 1, 4.0)
            reach = large.sum() + bin_entries[:j].sum() + 0.5 * bin_entries[j]
            small = rng.random(n - k - large.size) + 0.5       # they bring the row's sum to twice what is to be reached
            small *= (2.0 * reach - large.sum() - bin_entries.sum()) / small.sum()
            assert small.max() < 0.9
            made.append(rng.permutation(np.concatenate([large, bin_entries, small])).astype(np.float32))
            taus.append(np.float32(bin_entries[j]))
    probs = np.stack(made)[np.arange(max(rows, len(made))) % len(made)].reshape(1, -1, n)
    got, _ = _check(probs, 0.5)
    assert np.array_equal(got["tau"], np.array(taus)[np.arange(probs.shape[1]) % len(taus)])


@pytest.mark.parametrize("rows,n", [(1, 13001), (1, 16384), (300, 16384), (520, 16381), (1, 32767), (300, 32768), (300, 40001), (70, 65536)])
def test_thresholds_below_the_window(rows, n):
    """Rows of one large entry and thousands of ones more than 31 octaves below it: the threshold is the first, the middle or the last of
    their three values, two of which share an octave; with zeros and without."""
    rng = np.random.default_rng(n)
    values = np.array([1.9, 1.2, 0.55]) * 2.0 ** -32
    for zeros in (False, True):
        count = n // 4 if zeros else (n - 1) // 3
        row = np.zeros(n) if zeros else np.full(n, values[2])
        row[:1 + 3 * count] = np.concatenate([[1.0], np.repeat(values, count)])
        mass = count * values
        rows_in = np.tile(rng.permutation(row).astype(np.float32), (1, rows, 1))
        for j in range(3):                                     # (rows the oracle flags are compared, too: the margin is 2e-7 of the sum at least)
            p = float(np.float32((1.0 + mass[:j].sum() + 0.5 * mass[j]) / row.sum()))
            got, _ = _check(rows_in, p)
            assert (got["tau"] == np.float32(values[j])).all()


@pytest.mark.parametrize("rows,n", [(9, 1000), (9, 2048), (520, 2047), (9, 4096), (9, 8191), (520, 8192), (9, 16384), (520, 13001), (520, 16384), (9, 32767), (300, 32768),
                                    (9, 33000), (300, 65536)])
def test_flat_rows(rows, n):
    """Rows whose waves add their entries up by themselves, in the first pass and in later ones: nearly all entries in one bin, a few
    values in it, with zeros and single other entries among them, normal and subnormal."""
    rng = np.random.default_rng(n + rows)
    z, at = rng.random(n), rng.integers(0, n, 5)
    kinds = np.empty((9, n))
    kinds[0] = 1.0 / n
    kinds[1] = np.where(z < 0.4, 0.0, 0.75)                    # zeros between equal entries
    kinds[2] = 1.0 + np.floor(3 * z) * 2.0 ** -20              # three values, apart in the last pass
    kinds[3] = np.where(np.arange(n) < n // 2, 1.0, 1.0 + 2.0 ** -12)           # two values, each in waves of its own or together
    kinds[4] = 0.75
    kinds[4, at] = [4.0, 0.7501, 1e-6, 0.0, 1e-30]             # entries of other bins and below the window in single waves
    kinds[5] = 5 * 2.0 ** -149                                 # subnormal: the lowest bin of the lowest octave
    kinds[6] = np.where(z < 0.4, 0.0, np.floor(1 + 6 * z) * 2.0 ** -149)
    kinds[7] = 2.0 ** -130 * (1.0 + np.floor(2 * z) * 2.0 ** -15)
    kinds[8] = np.where(np.arange(n) % 4096 < 256, 2.0 ** -33, 1.0)             # whole waves below the window
    probs = kinds.astype(np.float32)[np.arange(rows) % 9].reshape(1, rows, n)
    for p in (0.9, 0.35):
        _check(probs, p)


@pytest.mark.parametrize("rows,n", [(3, 5), (3, 1023), (520, 2046), (3, 8191), (520, 13003), (3, 32765), (300, 32768), (3, 33001), (70, 65535)])
def test_rows_that_keep_everything(rows, n):
    """Lists of every position: shorter rows beside them, lists cut at any place, rows of lists at any address, pool slots, and next to them
    rows with a single zero."""
    rng = np.random.default_rng(n)
    probs = np.full((rows, n), 0.25, dtype=np.float32)
    probs[1] = rng.random(n).astype(np.float32) + 0.5          # (top_p = 1 keeps these too)
    probs[2, n // 2] = 0.0
    lens = np.full(rows, n, dtype=np.int32)
    lens[0] = n - 1
    page = 8
    table = rng.permutation(-(-n // page) * rows).astype(np.int32).reshape(rows, -1)
    for cap in (n, n - 3, 3):
        for phys in (False, True):
            paged = dict(page_table=table, page_size=page, emit_physical=True) if phys else {}
            got = gpu_select(probs.reshape(rows, 1, n), 1.0, seq_lens=lens, capacity=cap, split=False, **paged)
            for r in range(rows):
                want = np.flatnonzero(probs[r, :lens[r]])
                assert got["counts"][r] == want.size
                want = (table[r, want // page] * page + want % page if phys else want)[:cap]
                assert np.array_equal(got["indices"][r, :want.size], want) and (got["indices"][r, want.size:] == -7).all()


def _ragged_batch(B, H, n):
    """Rows of B sequences and their lengths: equal ones, some of one level and an empty one among them."""
    rng = np.random.default_rng(B * n)
    lens = rng.integers(0, n + 1, size=B).astype(np.int32)
    lens[: B // 3] = lens[0]                                 # one length
    lens[B // 2 : B // 2 + B // 4] = n - rng.integers(0, 3, size=B // 4)
    lens[-1], lens[B // 3] = 0, n
    probs = W.draft_probs(rng, 8, n, recency_len=min(64, n))[rng.integers(0, 8, size=B * H)].reshape(B, H, n)
    probs *= np.exp2(rng.integers(-3, 4, size=(B, H, 1))).astype(np.float32)     # (no two rows alike)
    return probs, lens


@pytest.mark.parametrize("B,H,n", [(64, 17, 300), (63, 17, 1000), (2, 600, 1500), (37, 8, 33000), (64, 9, 18000), (65, 9, 18000),
                                   (64, 17, 12288), (64, 17, 12289), (64, 12, 33000), (64, 13, 33000)])
def test_more_rows_of_different_lengths_than_fit_the_chip(B, H, n):
    """Workgroups take up to 64 sequences of long rows from the longest down where they come in up to three turns (every thread count; equal
    lengths, lengths of one level and empty rows among them), others in the order of the batch: both sides of each line."""
    probs, lens = _ragged_batch(B, H, n)
    _check(probs, 0.9, allow_flagged_mismatch=True, seq_lens=lens)


@pytest.mark.parametrize("B,H,n", [(64, 17, 1000), (37, 8, 33000), (64, 9, 18000), (64, 17, 13000)])
def test_pool_slots_and_state_of_rows_taken_by_length(B, H, n):
    """The same order where the lists hold pool slots, and where the kept mask and the block counts take their place."""
    probs, lens = _ragged_batch(B, H, n)
    R, page, nblk = B * H, 16, -(-n // sa.SEL_BLOCK)
    ref = oracle.topp_select(probs.reshape(R, n), 0.9, np.repeat(lens, H))
    table = np.random.default_rng(n).permutation(B * -(-n // page)).astype(np.int32).reshape(B, -1)
    got = gpu_select(probs, 0.9, seq_lens=lens, page_table=table, page_size=page, emit_physical=True, split=False)
    compare_select(got, ref, to_physical=lambda r, pos: table[r // H, pos // page] * page + pos % page)

    counts, tau = torch.full((R,), -7, dtype=torch.int32, device="cuda"), torch.full((R,), -7.0, device="cuda")
    bc, km = (torch.full((R, m), -1, dtype=torch.int32, device="cuda") for m in (nblk, nblk * sa.SEL_BLOCK // 32))
    sa.specattn_topp_select(sa.select_args(dev(probs), 0.9, indices=None, counts=counts, thresholds=tau, seq_lens=dev(lens), block_counts=bc, kept_mask=km))
    torch.cuda.synchronize()
    want = np.zeros((R, nblk * sa.SEL_BLOCK), dtype=np.uint8)
    want[:, :n] = ref.mask().reshape(R, n)
    sure = (ref.flags & oracle.ROW_NEAR_BOUNDARY) == 0
    assert sure.sum() > R // 2
    assert np.array_equal(counts.cpu().numpy()[sure], ref.counts[sure])
    valid = sure & ((ref.flags & oracle.ROW_INVALID) == 0)
    assert np.array_equal(tau.cpu().numpy()[valid], ref.tau[valid])
    assert np.array_equal(np.unpackbits(km.cpu().numpy().view(np.uint8), axis=1, bitorder="little")[sure], want[sure])
    assert np.array_equal(bc.cpu().numpy()[sure], want.reshape(R, nblk, -1).sum(axis=2)[sure])
