"""Left-over points of batches of every size, by waves and by tiles; the result is that of all pairs everywhere."""
import numpy as np
import pytest

from tests.test_gpu_knn_search import all_pairs, same

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fp():
    from paper_2507_23480_amd import binding
    binding.load()
    return binding


@pytest.mark.parametrize("B,N", [(1, 4096), (1, 16384), (1, 16385), (5, 13107), (5, 13108), (8, 8192), (8, 8193), (20, 4097)])
def test_left_over_points_of_a_batch(fp, B, N):
    """A radius that settles nothing leaves all points to the brute-force kernels, by waves and by tiles."""
    rng = np.random.default_rng(N)
    x = torch.from_numpy(rng.random((B, N, 3)).astype(np.float32)).cuda()
    s = torch.from_numpy(np.stack([rng.permutation(N)[:70] for _ in range(B)]).astype(np.int32)).cuda()
    s[0, 3], s[0, 4] = -1, N
    for k in (1, 5):
        got = fp.knn_grid(x, s, k, 1e-6, want_deferred=True)
        assert (got[2] >= N - 70).all()
        assert same(got, all_pairs(fp, x, s, k))
