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


def test_many_rows():
    rng = np.random.default_rng(5)
    x = (rng.standard_normal((7, 19, 20011)) * 2.0).astype(np.float32)
    tok_g, lp_g = gu.gpu_topk(x, 100)
    for b in (0, 3, 6):
        tok_o, lp_o = oracle.topk(x[b], 100)
        assert np.array_equal(tok_g[b], tok_o) and ulp_diff(lp_g[b], lp_o).max() <= 2
