"""Tree construction where its variants meet: budgets whose frontier just fits one wave (63 nodes), the budgets at
which pops give way to levels (36) and 256 threads to 512 (320), with tied scores, sibling runs, fewer
ranks than budget and the most rows.  Bit for bit against the oracle, under every construction."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402

if torch.cuda.is_available():
    import paper_2604_12989_amd as dd  # noqa: E402
    from tests import gpu_util as gu  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests selected but no GPU is visible")


def _table(kind, rng, B, K):
    if kind == "tied":      # few distinct, exactly representable values: equal sums everywhere
        lp = -0.5 * rng.integers(1, 5, (B, K))
    elif kind == "runs":    # one parent's ranks close together, then a gap: long sibling runs
        lp = -3.0 - 0.01 * rng.random((B, K)) - 2.0 * (np.arange(K) > K // 2)
    else:                   # a confident drafter
        lp = np.where(np.arange(K) == 0, -0.2, -2.5) - 2.0 * rng.random((B, K))
    lp = -np.sort(-lp.astype(np.float32), axis=1)
    return rng.integers(0, 5000, (B, K)).astype(np.int32), lp


@pytest.mark.parametrize("kind", ["tied", "runs", "peaked"])
@pytest.mark.parametrize("N,B,K", [(1, 1, 1), (15, 1, 15), (16, 32, 16), (31, 3, 2), (35, 16, 35), (36, 16, 36), (48, 2, 9),
                                   (62, 32, 62), (63, 16, 63), (64, 16, 64), (319, 16, 319), (320, 16, 320), (321, 5, 64), (1024, 16, 900)])
def test_constructions_meet(kind, N, B, K):
    rng = np.random.default_rng(1000 * N + B)
    tok, lp = _table(kind, rng, B, K)
    o = oracle.build_tree(tok, lp, N, 5)
    mask = oracle.ancestor_mask(o["parent"], o["n_nodes"], T=N + 1)
    try:
        for algo in (dd.BUILD_AUTO, dd.BUILD_POPS, dd.BUILD_LEVELS):
            dd.set_build_algorithm(algo)
            g = gu.gpu_build(tok, lp, N, 5)
            assert int(g["n_nodes"][0]) == o["n_nodes"], algo
            for key in ("tokens", "parent", "depth", "rank"):
                assert np.array_equal(g[key][0], o[key]), (algo, key)
            assert np.array_equal(g["node_score"][0].view(np.uint32), o["score"].view(np.uint32)), algo
            assert np.array_equal(g["ancestor_mask"][0], mask), algo
    finally:
        dd.set_build_algorithm(dd.BUILD_AUTO)
