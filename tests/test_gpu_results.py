"""Results that the binding allocates: each in memory of its own, so that keeping one keeps nothing else."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2604_12989_amd as dd  # noqa: E402


def test_every_result_has_memory_of_its_own():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests selected but no GPU is visible")
    batch, B, V, N = 2, 4, 2000, 20
    ws = dd.Workspace(batch, B, V, N, 4, 2, 96, 0)
    x = torch.randn((batch, B, V), device="cuda")
    tok, lp = dd.topk(x, N, ws)
    tree = dd.build(tok, lp, N, torch.zeros(batch, dtype=torch.int32, device="cuda"), ws)
    walk = dd.accept(torch.randn((batch, N + 1, V), device="cuda"), tree["tokens"], tree["parent"], tree["depth"], tree["n_nodes"], B, ws)
    results = [tok, lp, *tree.values(), *walk.values()]
    assert list(tree) == ["tokens", "parent", "depth", "rank", "node_score", "ancestor_mask", "n_nodes"]
    assert list(walk) == ["path", "n_accepted", "bonus_token", "posterior"]
    for t in results:
        assert t._base is None and t.is_contiguous() and t.untyped_storage().nbytes() == t.numel() * t.element_size()
