"""Tree construction where its variants meet: budgets whose frontier just fits one wave (63 nodes), the budgets and the
near-stars at which pops give way to the construction by deviations (28 to 257 nodes), with tied scores, sibling runs, fewer
ranks than budget and the most rows.  Bit for bit against the oracle, by the automatic choice, the pops and the levels."""
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


def _check(tok, lp, N):
    o = oracle.build_tree(tok, lp, N, 5)
    mask = oracle.ancestor_mask(o["parent"], o["n_nodes"], T=N + 1)
    try:
        for algo in (dd.BUILD_AUTO, dd.BUILD_LEVELS):
            dd.set_build_algorithm(algo)
            g = gu.gpu_build(tok, lp, N, 5)
            assert int(g["n_nodes"][0]) == o["n_nodes"], algo
            for key in ("tokens", "parent", "depth", "rank"):
                assert np.array_equal(g[key][0], o[key]), (algo, key)
            assert np.array_equal(g["node_score"][0].view(np.uint32), o["score"].view(np.uint32)), algo
            assert np.array_equal(g["ancestor_mask"][0], mask), algo
    finally:
        dd.set_build_algorithm(dd.BUILD_AUTO)


# wide: nodes off the chain with more than 64 children in the tree; long: continuations of more than 16 nodes; mixed: one
# flat row among peaked ones; twins: equal rows, so that many prefixes have equal scores; masked: ranks of -1e9 and -inf.
# From 28 nodes on the automatic choice builds them by deviations and hands none over, but for 1023 x 24 x 1023, whose table
# leaves no room for anything but pops, and near-stars.
@pytest.mark.parametrize("kind", ["wide", "long", "mixed", "twins", "masked"])
@pytest.mark.parametrize("N,B,K", [(23, 16, 23), (24, 16, 24), (63, 32, 63), (64, 32, 64), (65, 2, 65), (66, 16, 66), (129, 17, 129),
                                   (255, 32, 255), (512, 31, 512), (513, 16, 513), (1000, 24, 1000), (1023, 24, 1023), (1024, 32, 700)])
def test_deviations(kind, N, B, K):
    rng = np.random.default_rng(7 * N + B)
    r = np.arange(K)
    if kind == "wide":
        lp = np.where(r == 0, -0.3, -4.0 - 1e-3 * r - 1e-4 * rng.random((B, K)))
        lp[0] = np.where(r < 3, -1.0 - 0.1 * r, -30.0 - 0.01 * r)
    elif kind == "long":
        lp = np.where(r == 0, -0.01, -3.0 - 0.3 * r) - 0.005 * rng.random((B, K))
    elif kind == "mixed":
        lp = np.where(r == 0, -0.1, -3.5 - 0.02 * r) - 0.01 * rng.random((B, K))
        lp[B // 2] = -5.0 - 1e-3 * rng.random(K)
    elif kind == "twins":
        lp = np.repeat((np.where(r == 0, -0.25, -2.0 - 0.125 * (r // 2)))[None], B, 0)
    else:
        lp = np.where(r == 0, -0.2, -3.0 - 0.1 * r) - 0.01 * rng.random((B, K))
        lp[:, K // 2:] = -1e9
        lp[1::2, 3 * K // 4:] = -np.inf
    lp = -np.sort(-lp.astype(np.float32), axis=1)
    before = dd.build_handovers()
    _check(rng.integers(0, 5000, (B, K)).astype(np.int32), lp, N)
    assert dd.build_handovers() == before


def test_forced_levels_run_alone():
    """Rows of equal values: more prefixes share the last score of the tree than the construction by deviations has room
    for, so that it hands the sequence over.  Forced levels do not try it first."""
    B, K, N = 8, 50, 256
    lp = np.full((B, K), np.float32(-np.log(K)))
    tok = np.tile(np.arange(K, dtype=np.int32), (B, 1))
    o = oracle.build_tree(tok, lp, N, 5)
    try:
        for algo, more in ((dd.BUILD_AUTO, 1), (dd.BUILD_LEVELS, 0), (dd.BUILD_POPS, 0)):
            dd.set_build_algorithm(algo)
            before = dd.build_handovers()
            g = gu.gpu_build(tok, lp, N, 5)
            assert dd.build_handovers() - before == more, algo
            assert np.array_equal(g["parent"][0], o["parent"]) and np.array_equal(g["rank"][0], o["rank"]), algo
    finally:
        dd.set_build_algorithm(dd.BUILD_AUTO)


# Rows without equal scores whose trees are bushy: a few plausible tokens a row (few), none that stands out (gumbel, normal),
# falling by a factor (geometric, zipf), all but some masked.  The construction by deviations finds several
# times as many prefixes as the tree has nodes on the way, and has to have room for them.  The levels are wide here, count
# levels whose candidates do not fit before they write them (few16, masked16), and give up on some (geometric).
@pytest.mark.parametrize("kind", ["few5", "few16", "few40", "gumbel3", "normal6", "geometric", "zipf2", "masked4", "masked16"])
@pytest.mark.parametrize("N,B,K", [(256, 8, 256), (256, 16, 256), (512, 16, 512), (512, 32, 512), (1024, 8, 1024), (1024, 16, 1024),
                                   (700, 24, 700), (1000, 24, 1000), (256, 16, 50), (1024, 16, 200)])
def test_bushy_trees_fit(kind, N, B, K):
    rng = np.random.default_rng(N + B + K)
    V, number = 8192, float("".join(c for c in kind if c.isdigit()) or 0)
    x = rng.standard_normal((B, V))
    if kind.startswith("few"):
        x[:, :int(number)] += 14.0
    elif kind.startswith("gumbel"):
        x = number * rng.gumbel(size=(B, V))
    elif kind.startswith("normal"):
        x *= number
    elif kind == "geometric":
        x = np.log(0.6) * np.arange(V) + 0.05 * x
    elif kind.startswith("zipf"):
        x = 0.3 * x - number * np.log(1.0 + np.arange(V))
    else:
        x[:, int(number):] -= 100.0
    tok, lp = oracle.topk(x.astype(np.float32), K)
    o = oracle.build_tree(tok, lp, N, 5)
    mask = oracle.ancestor_mask(o["parent"], o["n_nodes"], T=N + 1)
    try:
        for algo in (dd.BUILD_AUTO, dd.BUILD_LEVELS):
            dd.set_build_algorithm(algo)
            before, given_up = dd.build_handovers(), dd.build_giveups()
            g = gu.gpu_build(tok, lp, N, 5)
            if algo == dd.BUILD_AUTO:
                assert dd.build_handovers() == before and dd.build_giveups() == given_up
            for key in ("tokens", "parent", "depth", "rank"):
                assert np.array_equal(g[key][0], o[key]), (algo, key)
            assert np.array_equal(g["node_score"][0].view(np.uint32), o["score"].view(np.uint32)), algo
            assert np.array_equal(g["ancestor_mask"][0], mask), algo
    finally:
        dd.set_build_algorithm(dd.BUILD_AUTO)


# equal values: 1 to 4 distinct ones a row, budgets whose members do not fit (they go to the pops, not to the levels and then the
# pops) and others
@pytest.mark.parametrize("values", [1, 2, 4])
@pytest.mark.parametrize("N,B,K", [(28, 4, 20), (64, 8, 50), (64, 8, 7), (100, 16, 60), (128, 5, 40)])
def test_small_budgets_of_equal_scores(values, N, B, K):
    rng = np.random.default_rng(N + K + values)
    lp = -np.sort(rng.integers(0, values, (B, K)), axis=1).astype(np.float32) / 4 - 1
    tok = rng.integers(0, 5000, (B, K)).astype(np.int32)
    before = dd.build_handovers()
    _check(tok, lp, N)
    assert dd.build_handovers() == before


# exactly `below` prefixes of depth 2 reach the worst useful rank of row 0, where the choice between pops and deviations lies;
# the top-1 chain reaches it to its second node, or to its last
@pytest.mark.parametrize("chain", ["short", "long"])
@pytest.mark.parametrize("below", [0, 2, 3, 4, 5])
@pytest.mark.parametrize("N", [27, 28, 35, 36, 47, 48, 99, 100, 128, 129, 256, 257])
def test_choice_between_pops_and_deviations(N, below, chain):
    B, K, rng = 5, N, np.random.default_rng(N + below)
    r = np.arange(K)
    lp = np.empty((B, K))
    lp[0] = -1.0 - 0.01 * r
    lp[1] = -0.01 * (N - below) + 0.004 - 9.0 * (r > 0) - 0.001 * r
    lp[2:] = (-1e-4 if chain == "long" else -9.0) - 9.0 * (r > 0) - 0.001 * r - 1e-5 * rng.random((B - 2, K))
    lp = lp.astype(np.float32)
    assert ((lp[0][:, None] + lp[1][None, :4]) >= lp[0][-1]).sum() == below
    _check(rng.integers(0, 5000, (B, K)).astype(np.int32), lp, N)
