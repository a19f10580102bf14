"""The k nearest samples through the density-following grid against all pairs, over what the call accepts: samples on
surfaces, in volumes, bunched, all at one place, bad sample indices, points outside the samples' box, coordinates that
are not finite, every k."""
import numpy as np
import pytest

from paper_2507_23480_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fp():
    from paper_2507_23480_amd import binding
    binding.load()
    return binding


def out_for(x, k):
    B, N = x.shape[:2]
    return (torch.empty((B, N, k), dtype=torch.int32, device="cuda"), torch.empty((B, N, k), device="cuda"))


def all_pairs(fp, x, s, k):
    pos, d2 = out_for(x, k)
    st = fp.load().fp_knn(x.data_ptr(), x.shape[0], x.shape[1], s.data_ptr(), s.shape[1], k, pos.data_ptr(), d2.data_ptr(),
                          None, None, None, 0, torch.cuda.current_stream().cuda_stream)
    assert st == 0
    return pos, d2


def search(fp, x, s, k):
    B, N, n = x.shape[0], x.shape[1], s.shape[1]
    pos, d2 = out_for(x, k)
    ws = torch.empty(fp.load().fp_knn_search_workspace_bytes(B, N, n), dtype=torch.uint8, device="cuda")
    left = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    st = fp.load().fp_knn_search(x.data_ptr(), B, N, s.data_ptr(), n, k, pos.data_ptr(), d2.data_ptr(), left.data_ptr(),
                                 ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert st == 0
    return pos, d2, left.cpu().numpy()


def same(a, b):
    return torch.equal(a[0], b[0]) and torch.equal(a[1].view(torch.int32), b[1].view(torch.int32))


def cloud(kind, N, rng):
    if kind == "volume":
        return rng.random((N, 3))
    if kind == "plane":
        p = rng.random((N, 3))
        p[:, 2] = 0.25
        return p
    if kind == "bunched":
        return np.where(rng.random((N, 1)) < 0.95, 1e-3 * rng.normal(size=(N, 3)), 100.0 * rng.normal(size=(N, 3)))
    if kind == "lattice":
        return rng.integers(0, 14, (N, 3)).astype(np.float64)
    if kind == "far":
        return 1e5 + rng.random((N, 3))
    return np.full((N, 3), 2.5)


@pytest.mark.parametrize("kind", ["volume", "plane", "bunched", "lattice", "far", "point"])
@pytest.mark.parametrize("N,n", [(1, 1), (70, 3), (1000, 17), (5003, 1301), (20000, 2000)])
def test_search_is_all_pairs(fp, kind, N, n):
    rng = np.random.default_rng([N, n])
    x = np.stack([cloud(kind, N, rng) for _ in range(2)]).astype(np.float32)
    s = np.stack([rng.permutation(N)[:n] for _ in range(2)]).astype(np.int32)
    if n > 10:
        x[1, 3] = np.nan
        x[1, 4, 2] = np.inf
        s[1, 5], s[1, 6] = -1, N
        s[0, 7] = s[0, 8]                                   # one point twice: equal distances
        half = np.argsort(x[0, :, 0], kind="stable")[:max(n, N // 2)]
        s[0] = rng.permutation(half)[:n]                    # points far outside the samples' box
    xd, sd = torch.from_numpy(x).cuda(), torch.from_numpy(s).cuda()
    for k in {1, min(2, n), min(3, n), min(5, n), min(8, n)}:
        got = search(fp, xd, sd, k)
        assert same(got, all_pairs(fp, xd, sd, k)), k
        assert (got[2] >= 0).all() and (got[2] <= N).all()


@pytest.mark.parametrize("N,n", [(4095, 1024), (4096, 1023), (4096, 1024)])
def test_either_side_of_the_rule(fp, N, n):
    x = torch.from_numpy(np.stack([inputs.make_cloud("C3", 800 + b, N) for b in range(2)])).cuda()
    s = fp.fps_exact(x, n)
    assert same(fp.knn(x, s, 3), all_pairs(fp, x, s, 3))
    assert fp.knn(x, s, 3, want_deferred=True)[2] is None


def test_lists_of_both_lengths(fp):
    # most points left to the brute-force kernels: a few (a wave each), then more than those take
    rng = np.random.default_rng(3)
    for N in (9000, 40000):
        x = rng.random((1, N, 3)).astype(np.float32)
        x[0, : N // 2] *= 1e-4                              # the samples lie in a corner, the points far away
        s = torch.arange(0, 1200, dtype=torch.int32, device="cuda")[None].contiguous()
        xd = torch.from_numpy(x).cuda()
        got = search(fp, xd, s, 4)
        assert N // 4 < got[2][0] <= 16384 if N == 9000 else got[2][0] > 16384
        assert same(got, all_pairs(fp, xd, s, 4))


def test_refused(fp):
    x = torch.zeros((1, 50, 3), device="cuda")
    s = torch.zeros((1, 10), dtype=torch.int32, device="cuda")
    pos, d2 = out_for(x, 3)
    ws = torch.empty(fp.load().fp_knn_search_workspace_bytes(1, 50, 10), dtype=torch.uint8, device="cuda")
    call = lambda n, k, w, wb: fp.load().fp_knn_search(x.data_ptr(), 1, 50, s.data_ptr(), n, k, pos.data_ptr(),  # noqa: E731
                                                       d2.data_ptr(), None, w, wb, None)
    assert call(10, 11, ws.data_ptr(), ws.numel()) == -2 and call(10, 9, ws.data_ptr(), ws.numel()) == -2
    assert call(51, 1, ws.data_ptr(), ws.numel()) == -2 and call(10, 1, None, 0) == -4
    assert call(10, 1, ws.data_ptr(), ws.numel() - 1) == -4
    assert fp.load().fp_knn_search_workspace_bytes(0, 5, 5) == 0
