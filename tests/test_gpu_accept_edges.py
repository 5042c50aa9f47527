"""The sampled walk where keys tie exactly: at a small temperature logit / temperature swamps the noise, so equal
logits give equal keys and the lowest token id wins, as in the greedy walk."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from tests import gpu_util as gu  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests selected but no GPU is visible")


@pytest.mark.parametrize("V", [1027, 2049, 4098, 4099])
def test_equal_keys_take_the_lowest_id(V):
    # Rows of one segment, read as 0-3 single elements, loads of four by 256 threads in turn, 0-3 single elements;
    # the first threads also hold the single ones.  Two equal maxima of one thread, in all pairs of the three.
    T = 9
    rng = np.random.default_rng(V)
    x = rng.standard_normal((T, V)).astype(np.float32)
    want = []
    for i in range(T):
        head = (-i * V) % 4
        nvec = (V - head) // 4
        tail = V - head - 4 * nvec
        t = i % 3                                      # the thread
        places = [head + 4 * t, head + 4 * t + 2]      # its first load
        places += [head + 4 * (t + 256)] if t + 256 < nvec else []
        places += [t] if t < head else []
        places += [head + 4 * nvec + t] if t < tail else []
        a, b = rng.choice(len(places), 2, replace=False) if i >= 3 else (0, len(places) - 1)
        x[i, [places[a], places[b]]] = 500.0
        want.append(min(places[a], places[b]))
    par = np.arange(-1, T - 1).astype(np.int32)
    got = gu.gpu_accept(x, np.zeros(T, np.int32), par, np.arange(T, dtype=np.int32), T - 1, 16, temperature=1e-6, seed=3)
    assert list(got["posterior"][0]) == want
