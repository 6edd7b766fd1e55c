"""GPU parity of the offline layer mapping (Section 3.3, Eq. 4; Appendix B, Algorithm 3) against the oracle.

Similarity: both sides compute in fp64 from the same fp32 inputs; they differ in the order of the sums (chunks
and lanes on the GPU, sequential in the oracle) and in the last bit of the logarithms, so with N terms t_k per
pair |S_gpu - S_ref| <= about N * 2^-53 * sum|t_k| / rows; the sums of |t_k| stay within a few times |S| here,
hence the relative tolerance 1e-9 (N up to 5e5) with an absolute floor of 1e-12.
Alignment: every table entry is one chain of fp64 additions taken in the same order on both sides and the tie
rule is the same (first maximum), so the map and the total are compared exactly."""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_27641_amd import binding as sa
from paper_2510_27641_amd import workloads as W
from helpers import dev

pytestmark = pytest.mark.gpu


def gpu_similarity(ad, av):
    S = torch.full((ad.shape[0], av.shape[0]), float("nan"), dtype=torch.float64, device="cuda")
    sa.specattn_layer_similarity(dev(ad), dev(av), S)
    torch.cuda.synchronize()
    return S.cpu().numpy()


def gpu_map(S):
    m, n = S.shape
    f = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    total = torch.full((1,), float("nan"), dtype=torch.float64, device="cuda")
    sa.specattn_layer_map(dev(S), f, total)
    torch.cuda.synchronize()
    return f.cpu().numpy(), float(total.item())


def close(got, ref):
    fin = np.isfinite(ref)
    assert np.array_equal(np.isneginf(got), np.isneginf(ref))
    assert np.all(np.abs(got[fin] - ref[fin]) <= 1e-9 * np.abs(ref[fin]) + 1e-12)


def test_similarity_tiny_against_the_plain_loops():
    ad, av = W.layer_attention_maps(seed=1, m=3, n=4, rows=5, L=37)
    close(gpu_similarity(ad, av), oracle.layer_similarity(ad, av))


@pytest.mark.parametrize("m,n,rows,L,seed", [(6, 9, 8, 256, 2), (22, 32, 16, 1024, 3), (1, 1, 1, 1, 4), (2, 3, 1, 5000, 5),
                                             (5, 2, 300, 33, 6), (32, 22, 7, 4097, 7)])
def test_similarity_shapes(m, n, rows, L, seed):
    ad, av = W.layer_attention_maps(seed=seed, m=m, n=n, rows=rows, L=L)
    close(gpu_similarity(ad, av), oracle.layer_similarity_fast(ad, av))


def test_similarity_zeros_and_minus_infinity():
    rng = np.random.default_rng(8)
    ad, av = W.layer_attention_maps(seed=8, m=4, n=5, rows=6, L=300)
    av[2, :, 10:20] = 0.0                                     # verifier zeros add nothing
    ad[1, 3, 0] = 0.0                                         # a draft zero under verifier mass: -infinity for draft layer 1
    ref = oracle.layer_similarity_fast(ad, av)
    assert np.isneginf(ref[1]).all() and np.isfinite(ref[[0, 2, 3]]).all()
    close(gpu_similarity(ad, av), ref)
    assert rng is not None


@pytest.mark.parametrize("rows,L", [(1, 40), (3, 700)])
def test_similarity_of_entries_that_are_no_probabilities(rows, L):
    """What the plain sum over p > 0 of p (log p - log q) gives: an infinite draft entry +infinity (NaN beside a zero),
    negative and NaN ones NaN, an infinite verifier entry -infinity; nothing where the verifier has no mass."""
    ad, av = W.layer_attention_maps(seed=20, m=10, n=4, rows=rows, L=L)
    av[:, 0, :12] = np.maximum(av[:, 0, :12], np.float32(1e-30))
    av[1:, 0, 2] = 0.0                                        # only verifier layer 0 has mass at position 2
    ad[0, 0, 2] = np.inf
    ad[1, 0, 3] = np.inf
    ad[2, 0, 3], ad[2, 0, 5] = np.inf, 0.0
    ad[3, 0, 3] = -0.25
    ad[4, 0, 3] = np.nan
    ad[5, 0, 5] = 0.0
    ad[6, 0, 7] = 1.0                                         # under the infinite verifier entry: log q = 0 and above
    ad[7, 0, 7] = 3.0
    ad[8, 0, 2] = np.nan
    av[3, 0, 7] = np.inf
    av[2, 0, 9], av[2, 0, 10] = np.nan, -0.5                  # (not above 0)
    ref, got = oracle.layer_similarity_fast(ad, av), gpu_similarity(ad, av)
    assert np.isposinf(ref[1, :3]).all() and np.isnan(ref[2]).all() and np.isneginf(ref[[0, 5, 6, 7, 9], 3]).all()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
    some = ~np.isnan(ref) & ~np.isposinf(ref)
    close(got[some], ref[some])


@pytest.mark.parametrize("m,n,rows,L", [(16, 16, 1, 63), (17, 15, 1, 64), (33, 31, 1, 65), (32, 33, 1, 511), (31, 65, 3, 171),
                                        (1, 32, 1, 4611), (3, 2, 1, 131072 * 2 + 512 * 3 + 1)])
def test_similarity_tile_edges(m, n, rows, L):
    """Layers around the 16- and 32-wide tiles, entries around a wave's 64 and a workgroup's 512, several runs per
    workgroup (more than 512 entries per CU); values over the whole fp32 range, subnormals and ones among them."""
    rng = np.random.default_rng(m * 100 + n)
    ad = np.exp(rng.uniform(-100, 0, size=(m, rows, L))).astype(np.float32)
    av = np.exp(rng.uniform(-100, 0, size=(n, rows, L))).astype(np.float32)
    ad[:, 0, ::7] = 1.0
    av[:, 0, 1::5] = np.float32(1.0) - np.float32(2.0 ** -24)
    av[:, 0, ::11] = 0.0
    ad[:, :, -1] = np.float32(1e-40)
    close(gpu_similarity(ad, av), oracle.layer_similarity_fast(ad, av))


@pytest.mark.parametrize("m,n", [(63, 20), (65, 33), (128, 200), (129, 7), (1000, 30), (2, 12289), (22, 8), (22, 9)])
def test_alignment_scan_edges(m, n):
    """Draft layers around one wave and several, columns around a block of eight, back pointers in LDS and in memory."""
    rng = np.random.default_rng(m * 7 + n)
    S = np.round(rng.normal(size=(m, n)) * 3) / 2
    f_ref, v_ref = oracle.layer_map(S)
    f, v = gpu_map(S)
    assert v == v_ref and np.array_equal(f, f_ref)


@pytest.mark.parametrize("m,n", [(16, 63), (17, 64), (32, 65), (33, 129), (64, 16), (1, 6145), (3, 6145)])
def test_alignment_in_one_wave(m, n):
    """Draft layers around the lane steps of one wave, columns around its blocks of 16 and 64 and the records LDS holds; ties,
    entries of -infinity, and a NaN, for which the general form (more than 64 layers, the others -infinity) is the measure."""
    rng = np.random.default_rng(m * 11 + n)
    S = np.round(rng.normal(size=(m, n)) * 2)
    S[rng.random(S.shape) < 0.1] = -np.inf
    S[0, ::2] = np.where(np.isneginf(S[0, ::2]), -9.0, S[0, ::2])
    f_ref, v_ref = oracle.layer_map(S)
    f, v = gpu_map(S)
    assert (v == v_ref or (np.isneginf(v) and np.isneginf(v_ref))) and np.array_equal(f, f_ref)
    S[m // 2, n // 3] = np.nan
    f, v = gpu_map(S)
    f_ref, v_ref = gpu_map(np.vstack([S, np.full((65 - m, n), -np.inf)]))
    assert np.array_equal([v], [v_ref], equal_nan=True) and np.array_equal(f, f_ref)


@pytest.mark.parametrize("m,n", [(1, 64), (2, 63), (64, 1), (64, 64), (64, 65), (63, 66), (2, 128), (64, 129), (5, 192), (40, 9900)])
def test_alignment_by_diagonals(m, n):
    """Steps and columns around the blocks of 64, records in LDS and in memory; entries whose sums could end in a NaN, for which the general
    form (more than 64 layers, the others -infinity) is the measure."""
    rng = np.random.default_rng(m * 13 + n)
    S = np.round(rng.normal(size=(m, n)) * 2)
    f_ref, v_ref = oracle.layer_map(S)
    f, v = gpu_map(S)
    assert v == v_ref and np.array_equal(f, f_ref)
    for large in (2e300, np.inf):
        S[rng.integers(m, size=3), rng.integers(n, size=3)] = large
        S[rng.integers(m, size=n), np.arange(n)] = -np.inf
        f, v = gpu_map(S)
        f_ref, v_ref = gpu_map(np.vstack([S, np.full((65 - m, n), -np.inf)]))
        assert np.array_equal([v], [v_ref], equal_nan=True) and np.array_equal(f, f_ref)


@pytest.mark.parametrize("m,n", [(1, 5), (7, 64), (32, 48), (64, 65), (64, 1000), (40, 9900)])
@pytest.mark.parametrize("low", [-9.0, -1e300, -1.5e300, -np.inf])
def test_alignment_of_very_large_entries(m, n, low):
    """Infinities and sums that overflow, alone and beside entries on either side of -1e300, from which the general form takes over
    (more than 64 layers, the others -infinity, is the measure; without a NaN also the oracle)."""
    rng = np.random.default_rng(m * 17 + n)
    S = np.round(rng.normal(size=(m, n)) * 2)
    S[rng.random(S.shape) < 0.1] = low
    for large in (1e300, 1.7e308, np.inf):
        S[rng.integers(m, size=4), rng.integers(n, size=4)] = large
        f, v = gpu_map(S)
        f_ref, v_ref = gpu_map(np.vstack([S, np.full((65 - m, n), -np.inf)]))
        assert np.array_equal([v], [v_ref], equal_nan=True) and np.array_equal(f, f_ref)
        if low > -1e301 and not np.isnan(v):
            with np.errstate(over="ignore"):
                want_f, want_v = oracle.layer_map(S)
            assert v == want_v and np.array_equal(f, want_f)


def test_layers_compared_with_themselves():
    ad, _ = W.layer_attention_maps(seed=9, m=5, n=5, rows=4, L=128)
    S = gpu_similarity(ad, ad)
    assert np.all(np.abs(np.diag(S)) <= 1e-15) and np.all(S[~np.eye(5, dtype=bool)] < 0)


@pytest.mark.parametrize("seed", range(12))
def test_alignment_random_matrices_exact(seed):
    rng = np.random.default_rng(100 + seed)
    m, n = int(rng.integers(1, 40)), int(rng.integers(1, 50))
    if seed % 3 == 0:
        S = np.round(rng.normal(size=(m, n)))                 # many ties
    else:
        S = -rng.gamma(1.0, size=(m, n))
    if seed % 4 == 1:
        S[rng.random(S.shape) < 0.2] = -np.inf
    f_ref, v_ref = oracle.layer_map(S)
    f, v = gpu_map(S)
    assert v == v_ref or (np.isneginf(v) and np.isneginf(v_ref))
    assert np.array_equal(f, f_ref)
    assert np.all(np.diff(f) >= 0) and f.min() >= 0 and f.max() < m


@pytest.mark.parametrize("m,n", [(1, 1), (1, 7), (7, 1), (1024, 3), (3, 1000), (64, 64)])
def test_alignment_edge_sizes(m, n):
    rng = np.random.default_rng(m * 1000 + n)
    S = -rng.gamma(1.0, size=(m, n))
    f_ref, v_ref = oracle.layer_map(S)
    f, v = gpu_map(S)
    assert v == v_ref and np.array_equal(f, f_ref)


def test_alignment_tiny_against_exhaustive_search():
    rng = np.random.default_rng(11)
    for _ in range(10):
        m, n = int(rng.integers(1, 6)), int(rng.integers(1, 6))
        S = np.round(rng.normal(size=(m, n)) * 2) / 2
        best, all_f = oracle.layer_map_exhaustive(S)
        f, v = gpu_map(S)
        assert v == best and tuple(int(x) for x in f) in all_f


def test_whole_mapping_on_synthetic_models():
    """22 draft layers against 32 verifier layers (the depths of the paper's TinyLlama / Llama-2-7b pair)."""
    ad, av = W.layer_attention_maps(seed=0, m=22, n=32, rows=32, L=2048)
    S_ref = oracle.layer_similarity_fast(ad, av)
    f_ref, v_ref = oracle.layer_map(S_ref)
    S = torch.empty((22, 32), dtype=torch.float64, device="cuda")
    f = torch.empty((32,), dtype=torch.int32, device="cuda")
    total = torch.empty((1,), dtype=torch.float64, device="cuda")
    sa.specattn_layer_similarity(dev(ad), dev(av), S)
    sa.specattn_layer_map(S, f, total)
    torch.cuda.synchronize()
    close(S.cpu().numpy(), S_ref)
    got = f.cpu().numpy()
    assert abs(total.item() - v_ref) <= 1e-9 * abs(v_ref)
    assert np.all(np.diff(got) >= 0) and got.min() >= 0 and got.max() < 22
    # the value reached by the GPU's map, evaluated on the oracle's matrix, is the oracle's optimum
    assert abs(sum(S_ref[got[j], j] for j in range(32)) - v_ref) <= 1e-9 * abs(v_ref)
    print("f =", got.tolist())


def test_similarity_in_a_small_workspace():
    """Room for two chunks per layer pair (4 x 256 workgroups over 704 pairs): accepted, in longer chunks; less is not."""
    ad, av = W.layer_attention_maps(seed=12, m=22, n=32, rows=8, L=2048)
    S = torch.full((22, 32), float("nan"), dtype=torch.float64, device="cuda")
    ws = sa.alloc_workspace(22 * 32 * 2 * 8)
    sa.specattn_layer_similarity(dev(ad), dev(av), S, ws)
    torch.cuda.synchronize()
    close(S.cpu().numpy(), oracle.layer_similarity_fast(ad, av))
    with pytest.raises(RuntimeError, match="needed"):
        sa.specattn_layer_similarity(dev(ad), dev(av), S, ws[:22 * 32 * 8])
