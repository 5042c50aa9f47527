"""The two matrix-core attention kernels at the sizes where their tiling can go wrong: single rows and
keys, edges of the 32-row and 64-row groups and of the 32-key sub-tiles, more waves than sub-tiles,
key ranges cut differently for every sequence of a batch, scores that keep outgrowing the softmax
reference.  Against the oracle, with the bound of the other bf16 attention tests (1e-2)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import ddtree_inputs as di  # noqa: E402
import oracle  # noqa: E402

if torch.cuda.is_available():
    import paper_2604_12989_amd as dd  # noqa: E402
    from tests import gpu_util as gu  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests selected but no GPU is visible")


def _tree_mask(rng, T, n=None):
    n = T - 1 if n is None else n
    par = np.full(T, -1, np.int32)
    for i in range(1, n + 1):
        par[i] = i - 1 if rng.random() < 0.5 else rng.integers(0, i)
    return oracle.ancestor_mask(par, n, T=T)


def _check(seed, Ts, Ls, Hq, Hkv, D, n_pairs=40, edit=None, n_nodes=None, also=()):
    """A ragged batch of equal T against the oracle on sampled (node, head) pairs, the corners among them."""
    rng = np.random.default_rng(seed)
    T, batch = Ts, len(Ls)
    off = np.concatenate([[0], np.cumsum(Ls)]).astype(np.int32)
    parts = [di.attn_tensors(seed + b, T, Ls[b], Hq, Hkv, D, "bf16") for b in range(batch)]
    masks = [_tree_mask(rng, T, n_nodes) for _ in range(batch)]
    if edit is not None:
        for p in parts:
            edit(*p)
    got = gu.gpu_attn(*(np.concatenate([p[i] for p in parts]) for i in range(5)), np.stack(masks), off, batch, T, "bf16")
    worst = 0.0
    for b in range(batch):
        pairs = np.stack([rng.integers(0, T, n_pairs), rng.integers(0, Hq, n_pairs)], axis=1).astype(np.int32)
        pairs[:4] = [[0, 0], [T - 1, Hq - 1], [0, Hq - 1], [T - 1, 0]]
        pairs[4:4 + len(also)] = np.array(also, np.int32).reshape(-1, 2)
        ref = oracle.verify_attn(*parts[b], masks[b], pairs=pairs)
        worst = max(worst, gu.attn_err(got[b][pairs[:, 0], pairs[:, 1]], ref))
    assert worst < 1e-2, worst


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("T,L,Hq,Hkv", [
    (1, 0, 1, 1), (1, 1, 2, 2), (2, 31, 1, 1), (8, 32, 4, 1), (33, 33, 1, 1), (11, 255, 3, 1), (32, 256, 2, 1),
    (65, 257, 1, 1), (63, 7, 8, 8), (64, 900, 7, 1), (66, 31, 5, 5), (17, 4000, 4, 1), (97, 1025, 4, 2)])
def test_few_rows_edges(T, L, Hq, Hkv, D):
    _check(100 + T, T, [L], Hq, Hkv, D)


@pytest.mark.parametrize("T,Ls,Hq,Hkv,D", [
    (257, [4096], 32, 8, 64), (129, [3000, 0, 65, 1700], 32, 8, 64), (1025, [700], 8, 2, 64),   # 64-row groups
    (273, [5000], 32, 8, 128), (129, [5000, 100, 2600], 32, 8, 128), (257, [9000, 64], 16, 4, 128),  # shared key tiles
    (33, [900, 0, 31, 2500, 64], 12, 4, 128), (20, [40] * 9, 8, 8, 64)])
def test_ragged_batches_with_key_ranges_of_their_own(T, Ls, Hq, Hkv, D):
    _check(300 + T, T, Ls, Hq, Hkv, D, n_pairs=24)


@pytest.mark.parametrize("T,Ls,Hq,Hkv", [
    (130, [4000], 32, 8), (257, [9000, 64], 16, 4),           # fewer key ranges than the whole tiles have
    (1025, [700, 300], 16, 4), (1025, [8192], 32, 8),         # as many, and more
    (96, [6000, 33], 32, 8), (265, [6000, 33], 32, 8), (101, [37, 3001, 900, 1700], 24, 8),  # several blocks
    (257, [4096] * 5, 32, 8), (1025, [0, 0, 1], 32, 8)])      # uncut
def test_blocks_left_beside_whole_row_tiles(T, Ls, Hq, Hkv):
    """The last nodes' rows, which do not fill a tile of 256, take a path of their own."""
    rng = np.random.default_rng(T)
    last = [(T - 1 - i % min(T, 30), int(rng.integers(0, Hq))) for i in range(20)]
    _check(700 + T, T, Ls, Hq, Hkv, 128, n_pairs=40, also=last)


@pytest.mark.parametrize("T,Ls", [(161, [700] * 16), (161, [900, 30] + [700] * 14), (300, [1024] * 8), (545, [4096] * 4)])
def test_whole_row_tiles_in_several_rounds_of_workgroups(T, Ls):
    """More work items than compute units and no block left beside the tiles: every one is run."""
    _check(900 + T, T, Ls, 32, 8, 128, n_pairs=32)


@pytest.mark.parametrize("T,L,Hq,Hkv,D", [(40, 1500, 8, 2, 64), (40, 1500, 8, 2, 128), (257, 4096, 32, 8, 64), (273, 5000, 32, 8, 128)])
def test_scores_that_keep_outgrowing_the_reference(T, L, Hq, Hkv, D):
    # from key 200 on, keys point along a query with a factor that grows to 8: scores up to about 90, so a
    # row's maximum moves again and again by more than the slack of its reference
    def edit(q, kc, vc, kt, vt):
        G = Hq // Hkv
        for j in range(200, L, 3):
            f = 8.0 * (j - 200) / (L - 200)
            for hk in range(Hkv):
                kc[j, hk] = di.round_to_bf16((f * q[j % T, hk * G + j % G]).astype(np.float32))
    _check(500 + T, T, [L], Hq, Hkv, D, edit=edit)


def test_padding_rows_are_zero_in_every_kernel():
    """... and every head of every real row is what the oracle says."""
    for T, L, Hq, Hkv, D in ((80, 50, 4, 2, 64), (80, 50, 4, 2, 128), (300, 6000, 32, 8, 128), (257, 4096, 32, 8, 64)):
        rng = np.random.default_rng(T)
        parts = di.attn_tensors(T, T, L, Hq, Hkv, D, "bf16")
        mask = _tree_mask(rng, T, 40)
        got = gu.gpu_attn(*parts, mask[None], [0, L], 1, T, "bf16")[0]
        assert not got[41:].any() and np.isfinite(got).all()
        assert np.abs(got[:41]).max(axis=2).min() > 0.0
        pairs = np.stack(np.meshgrid(np.arange(41), np.arange(Hq), indexing="ij"), axis=-1).reshape(-1, 2).astype(np.int32)
        assert gu.attn_err(got[pairs[:, 0], pairs[:, 1]], oracle.verify_attn(*parts, mask, pairs=pairs)) < 1e-2


def test_heads_of_64_need_no_scratch():
    """Without a workspace no key range is cut; the result is that of the cut one up to rounding."""
    T, L, Hq, Hkv, D = 65, 3000, 8, 2, 64
    rng = np.random.default_rng(9)
    q, kc, vc, kt, vt = (gu.bf16_dev(a) for a in di.attn_tensors(9, T, L, Hq, Hkv, D, "bf16"))
    mask = gu.to_dev(_tree_mask(rng, T).view(np.int64)[None])
    args = (q, kc, vc, kt, vt, mask, [0, L], 1, T, Hq, Hkv, D, 0.125, dd.DTYPE_BF16)
    a = dd.verify_attn(*args, None)
    b = dd.verify_attn(*args, dd.Workspace(1, 4, 100, T - 1, Hq, Hkv, D, L))
    assert (a.float() - b.float()).abs().max().item() < 1e-2


@pytest.mark.parametrize("T,Ls,Hq,Hkv", [
    (297, [45, 636, 808, 238], 32, 8),                                                # row tiles of the same height
    (94, [366, 13, 40, 442, 104, 275, 5, 142, 304, 99, 220], 15, 5),                  # with blocks left beside them
    (102, [119, 56, 145, 212, 113, 958, 845, 427, 769, 302, 148], 2, 2), (9, [39, 522, 1006, 47, 15, 751, 816], 18, 6)])  # waves
@pytest.mark.parametrize("nodes", [None, 7])
def test_ragged_batches_of_short_caches(T, Ls, Hq, Hkv, nodes):
    """Key ranges are cut for the sake of the longest sequences alone: partial results in fp32."""
    _check(1100 + T, T, Ls, Hq, Hkv, 128, n_pairs=24, n_nodes=nodes)


@pytest.mark.parametrize("scale", [1.0, 2.0 ** 116])
@pytest.mark.parametrize("T,Ls,Hq,Hkv,scratch", [(65, [2047], 16, 4, True), (257, [4096], 32, 8, True), (33, [900, 31, 2500], 12, 4, True),
                                                 (65, [3000], 8, 2, False), (200, [31], 4, 1, True), (257, [4096], 8, 1, True)])
def test_heads_of_64_are_as_exact_as_their_result_type(T, Ls, Hq, Hkv, scratch, scale):
    """fp32 weights, sums and partial results: what is left is the rounding of the result to bf16 (weights of 8 bits
    or partials of 11 add a fifth to a half of it).  With values of 2^116 too: weights above 1 would overflow."""
    batch, rng = len(Ls), np.random.default_rng(T)
    parts = [di.attn_tensors(80 + b, T, Ls[b], Hq, Hkv, 64, "bf16") for b in range(batch)]
    masks = [_tree_mask(rng, T) for _ in Ls]
    off = np.concatenate([[0], np.cumsum(Ls)]).astype(np.int32)
    q, kc, vc, kt, vt = (np.concatenate([p[i] for p in parts]) for i in range(5))
    q = 3.0 * q  # (scores of a few units: references move)
    q, s = di.round_to_bf16(q.astype(np.float32)), np.float32(scale)
    got = dd.verify_attn(*(gu.bf16_dev(a) for a in (q, kc, vc * s, kt, vt * s)), gu.to_dev(np.stack(masks).view(np.int64)), off,
                         batch, T, Hq, Hkv, 64, 0.125, dd.DTYPE_BF16,
                         dd.Workspace(batch, 1, 8, T - 1, Hq, Hkv, 64, int(off[-1])) if scratch else None)
    got = got.double().cpu().numpy().reshape(batch, T, Hq, 64) / scale
    err, rounding = 0.0, 0.0
    for b in range(batch):
        pairs = np.stack([rng.integers(0, T, 200), rng.integers(0, Hq, 200)], axis=1).astype(np.int32)
        ref = np.asarray(oracle.verify_attn(q[b * T:(b + 1) * T], *parts[b][1:], masks[b], pairs=pairs), np.float64)
        err += ((got[b][pairs[:, 0], pairs[:, 1]] - ref) ** 2).sum()
        rounding += ((di.round_to_bf16(ref.astype(np.float32)).astype(np.float64) - ref) ** 2).sum()
    assert np.sqrt(err) < 1.03 * np.sqrt(rounding), (np.sqrt(err), np.sqrt(rounding))


class _Scratch:
    """A workspace of exactly nbytes."""

    def __init__(self, nbytes):
        self.nbytes = nbytes
        self.buf = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
        self.ptr = self.buf.data_ptr() + (-self.buf.data_ptr()) % 256


@pytest.mark.parametrize("T,Ls,Hq,Hkv,D", [
    (17, [600], 32, 8, 128), (17, [1000], 8, 8, 128), (65, [2048], 32, 8, 128), (257, [8192], 32, 8, 128),
    (1025, [900], 8, 2, 128), (33, [900, 0, 31, 2500], 12, 4, 128), (17, [600, 10, 10, 10], 32, 8, 128), (65, [2047], 16, 4, 64)])
def test_a_workspace_of_the_size_that_a_call_uses(T, Ls, Hq, Hkv, D):
    """The scratch of ddtree_verify_attn_workspace_bytes is enough, and gives the result of a larger one bit for bit."""
    batch, rng = len(Ls), np.random.default_rng(T)
    parts = [di.attn_tensors(40 + b, T, Ls[b], Hq, Hkv, D, "bf16") for b in range(batch)]
    q, kc, vc, kt, vt = (gu.bf16_dev(np.concatenate([p[i] for p in parts])) for i in range(5))
    mask = gu.to_dev(np.stack([_tree_mask(rng, T) for _ in Ls]).view(np.int64))
    off = np.concatenate([[0], np.cumsum(Ls)]).astype(np.int32)
    args = (q, kc, vc, kt, vt, mask, off, batch, T, Hq, Hkv, D, 1.0 / np.sqrt(D), dd.DTYPE_BF16)
    need = dd.binding.verify_attn_workspace_bytes(batch, T, Hq, Hkv, D, dd.DTYPE_BF16, int(off[-1]))
    a = dd.verify_attn(*args, _Scratch(need) if need else None)
    b = dd.verify_attn(*args, dd.Workspace(batch, 4, 2000, T - 1, Hq, Hkv, D, int(off[-1])))
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("T,Ls,Hq,Hkv", [(17, [600, 10, 10, 10], 32, 8), (17, [300], 32, 8), (161, [700] * 16, 32, 8)])
def test_short_calls_need_no_workspace(T, Ls, Hq, Hkv):
    """Fewer than eight key tiles a sequence on average, or enough workgroups without a cut."""
    batch, rng = len(Ls), np.random.default_rng(T)
    parts = [di.attn_tensors(60 + b, T, Ls[b], Hq, Hkv, 128, "bf16") for b in range(batch)]
    q, kc, vc, kt, vt = (gu.bf16_dev(np.concatenate([p[i] for p in parts])) for i in range(5))
    masks = [_tree_mask(rng, T) for _ in Ls]
    off = np.concatenate([[0], np.cumsum(Ls)]).astype(np.int32)
    got = dd.verify_attn(q, kc, vc, kt, vt, gu.to_dev(np.stack(masks).view(np.int64)), off, batch, T, Hq, Hkv, 128,
                         1.0 / np.sqrt(128), dd.DTYPE_BF16, None).float().cpu().numpy().reshape(batch, T, Hq, 128)
    for b in range(batch):
        pairs = np.stack([rng.integers(0, T, 24), rng.integers(0, Hq, 24)], axis=1).astype(np.int32)
        assert gu.attn_err(got[b][pairs[:, 0], pairs[:, 1]], oracle.verify_attn(*parts[b], masks[b], pairs=pairs)) < 1e-2
