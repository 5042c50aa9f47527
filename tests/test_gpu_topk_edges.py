"""ddtree_topk where its bounds are void, tight or wrong: rows of one chunk and of one more element, fewer
group maxima than ranks, a chunk that holds all of the row's top K (its hot list then lacks some of them),
hot lists that overflow, candidates around the switch between the two rankings.  Tokens exactly, the
log-probabilities to the 2 ulp of the other top-K tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402

if torch.cuda.is_available():
    from tests import gpu_util as gu  # noqa: E402
    from tests.test_gpu_parity import ulp_diff  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests selected but no GPU is visible")


def _check(x, K):
    tok_o, lp_o = oracle.topk(x, K)
    tok_g, lp_g = gu.gpu_topk(x, K)
    assert np.array_equal(tok_g[0], tok_o)
    fin = np.isfinite(lp_o)
    assert np.array_equal(np.isfinite(lp_g[0]), fin)
    assert not fin.any() or ulp_diff(lp_g[0][fin], lp_o[fin]).max() <= 2


@pytest.mark.parametrize("V", [3, 33, 255, 1023, 2047, 2049, 4095, 4097, 6143, 6144, 6145, 12289, 50003])
@pytest.mark.parametrize("K", [1, 3, 64, 255, 257, 511, 513, 1024])
def test_sizes(V, K):
    if K > V:
        pytest.skip("more ranks than tokens")
    rng = np.random.default_rng(V * 7 + K)
    _check((rng.standard_normal((5, V)) * 3.0).astype(np.float32), K)


@pytest.mark.parametrize("K", [16, 256, 1024])
def test_top_k_in_one_place(K):
    rng = np.random.default_rng(K)
    x = rng.standard_normal((6, 60001)).astype(np.float32)
    x[0, 7000:7000 + K] += 20.0                       # all of it inside one chunk
    x[1, :K // 2] += 20.0                             # half of it in front, half at the end
    x[1, 60001 - K // 2:] += 20.0
    x[2, 30000:30000 + 2 * K] = 5.0                   # 2 K equal values in one chunk: the first K
    x[3, ::3] = -np.inf
    x[3, 100:100 + K] += 15.0
    x[4, 20000:20000 + K] = np.linspace(50.0, 9.0, K)  # a long ramp far above everything else
    x[5, 59000] = 1000.0                              # the range of the maxima is all one outlier
    _check(x, K)


def _row(kind, rng, V, K):
    x = (rng.standard_normal(V) * 3.0).astype(np.float32)
    lowest = np.finfo(np.float32).min
    kept = np.zeros(V, bool)
    if kind == "outlier":                      # the range of the group maxima is nearly empty
        x[V // 3] = 1000.0
    elif kind == "two clusters":
        x[rng.permutation(V)[:K // 2]] += 5000.0
    elif kind == "masked half, lowest":        # scattered
        x[rng.random(V) < 0.5] = lowest
    elif kind == "masked half, -1e9":          # whole chunks
        x[V // 2:] = -1e9
    elif kind == "masked half, -inf":
        x[V // 2:] = -np.inf
    elif kind == "few kept, -1e4":             # fewer than K at the smaller sizes: masked tokens in the order of ids
        kept[rng.permutation(V)[:min(V, 150)]] = True
        x[~kept] = -1e4
    elif kind == "few kept, -inf":
        kept[rng.permutation(V)[:min(V, 150)]] = True
        x[~kept] = -np.inf
    elif kind == "equal":
        x[:] = 0.25
    elif kind == "steps":
        x = np.round(x * 2) / 2
    elif kind == "zeros of both signs":
        x = np.where(rng.random(V) < 0.5, -0.0, 0.0).astype(np.float32)
        x[rng.permutation(V)[:K // 2]] = 1.0
    elif kind == "powers":                     # a range that no linear scale resolves
        x = np.ldexp(1.0, -rng.integers(0, 120, V)).astype(np.float32) * np.where(rng.random(V) < 0.5, 1, -1)
    elif kind == "whole range":
        x = (x / 16.0 * 3e38).astype(np.float32)
    return x.astype(np.float32)


KINDS = ["outlier", "two clusters", "masked half, lowest", "masked half, -1e9", "masked half, -inf", "few kept, -1e4",
         "few kept, -inf", "equal", "steps", "zeros of both signs", "powers", "whole range"]


@pytest.mark.parametrize("V,K", [(700, 64), (1000, 512), (6144, 200), (6144, 1024), (20011, 100), (50003, 300), (151936, 1024)])
@pytest.mark.parametrize("kind", KINDS)
def test_masks_ties_and_ranges(kind, V, K):
    rng = np.random.default_rng(V + K + len(kind))
    _check(np.stack([_row(kind, rng, V, K) for _ in range(3)]), K)


@pytest.mark.parametrize("V,K", [(400003, 256), (700001, 200), (700001, 1024)])
def test_rows_of_more_than_64_chunks(V, K):
    rng = np.random.default_rng(V)
    x = (rng.standard_normal((7, V)) * 3.0).astype(np.float32)
    x[0, V - 5000:V - 5000 + K] += 30.0               # the top K behind chunk 64, more than its hot list takes
    x[1, [100, V - 7]] = 40.0                         # the maximum on both sides of it
    x[2, V - 6000:] = 20.0                            # equal values: a hot list that overflows there, ties at the K-th
    x[3, :V - 9000] = -np.inf
    x[4] = _row("masked half, -1e9", rng, V, K)
    x[5] = _row("equal", rng, V, K)
    x[6, rng.permutation(V)[:K // 2]] = 7.5
    _check(x, K)


@pytest.mark.parametrize("K", [86, 150, 300])
def test_one_chunk_above_all_others(K):
    # rows of two chunks, every group maximum of one above the other chunk's maximum: the K-th maximum lies above the
    # range that the second largest chunk maximum ends
    rng = np.random.default_rng(K)
    x = rng.standard_normal((16, 16, 12000)).astype(np.float32)
    x[0::2, :, :6000] += 50.0
    x[1::2, :, 6000:] += 50.0 * (1 + np.arange(16))[None, :, None]
    tok_g, lp_g = gu.gpu_topk(x, K)
    for b in (0, 1, 14, 15):
        tok_o, lp_o = oracle.topk(x[b], K)
        assert np.array_equal(tok_g[b], tok_o) and ulp_diff(lp_g[b], lp_o).max() <= 2


def test_many_rows():
    rng = np.random.default_rng(5)
    x = (rng.standard_normal((7, 19, 20011)) * 2.0).astype(np.float32)
    tok_g, lp_g = gu.gpu_topk(x, 100)
    for b in (0, 3, 6):
        tok_o, lp_o = oracle.topk(x[b], 100)
        assert np.array_equal(tok_g[b], tok_o) and ulp_diff(lp_g[b], lp_o).max() <= 2
