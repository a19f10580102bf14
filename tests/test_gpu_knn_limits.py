"""Where the search through the grid gives up: bunched samples, points beside a clump or far from all samples, left-over
points of batches of every size, and the lines between the routes; the result is that of all pairs everywhere."""
import numpy as np
import pytest

from tests.routes import all_pairs
from tests.test_gpu_knn_search import same, search

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fp():
    from paper_2507_23480_amd import binding
    binding.load()
    return binding


def scene(kind, N, n, rng):
    """Points and sample positions; the share of the points that has to be left over (0: any)."""
    p = rng.random((N, 3))
    s = rng.permutation(N)[:n]
    if kind == "one_cell":                      # nearly all samples in one cell of the grid: nothing is searched
        p[s[: n - n // 50]] = 0.5 + 1e-4 * rng.random((n - n // 50, 3))
        return p, s, 1.0
    if kind == "clump_beside":                  # more samples than a thread looks at two cells away from many points
        m = n // 5
        p[s[:m]] = 0.5 + 1e-3 * rng.random((m, 3))
        return p, s, 0.0
    if kind == "far":                           # half of the points out of reach of the samples' box
        out = np.setdiff1d(np.arange(N), s)[: N // 2]
        p[out] += 50.0
        return p, s, len(out) / N
    if kind == "equal":                         # every sample at one of eight places
        p[s] = rng.integers(0, 2, (n, 3))
        return p, s, 0.0
    return p, s, 0.0


@pytest.mark.parametrize("kind", ["one_cell", "clump_beside", "far", "equal", "even"])
@pytest.mark.parametrize("N,n", [(3000, 300), (9000, 2049), (21000, 6001)])
def test_limits(fp, kind, N, n):
    rng = np.random.default_rng([N, n])
    got = [scene(kind, N, n, rng) for _ in range(2)]
    x = torch.from_numpy(np.stack([g[0] for g in got]).astype(np.float32)).cuda()
    s = torch.from_numpy(np.stack([g[1] for g in got]).astype(np.int32)).cuda()
    for k in (1, 3, 8):
        r = search(fp, x, s, k)
        assert same(r, all_pairs(fp, x, s, k)), k
        assert (r[2] >= got[0][2] * N).all()


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


@pytest.mark.parametrize("n,k", [(1023, 3), (1024, 3), (2047, 4), (2048, 4)])
def test_either_side_of_the_lines(fp, n, k):
    rng = np.random.default_rng(n)
    x = torch.from_numpy(rng.random((2, 4099, 3)).astype(np.float32)).cuda()
    s = torch.from_numpy(np.stack([rng.permutation(4099)[:n] for _ in range(2)]).astype(np.int32)).cuda()
    assert same(fp.knn(x, s, k), all_pairs(fp, x, s, k))
