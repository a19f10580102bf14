"""Exact FPS by local decisions (the cell-ordered fps_exact): the samples and the curve of the index-ordered kernels, bit for
bit, where the sampler and the kernel that puts the samples in sequence change their ways -- one to eight points per
thread, one workgroup and many, lists at their limits, equal distances, n at the edges of a workgroup's keys."""
import numpy as np
import pytest

from tests.routes import exact_by_index

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fp():
    from paper_2507_23480_amd import binding
    binding.load()
    binding.set_wg_per_cloud(0)
    yield binding
    binding.set_wg_per_cloud(0)


def cloud(kind, N):
    rng = np.random.default_rng([N, len(kind)])
    if kind == "sheet":                         # a thin layer: the curve leaves it and comes back elsewhere
        return (rng.random((N, 3)) * [100.0, 100.0, 0.3]).astype(np.float32)
    if kind == "dense corner":                  # the first rounds' candidates sit in a few workgroups
        p = rng.random((N, 3))
        p[: N // 2] = 30.0 + 0.5 * p[: N // 2]
        return p.astype(np.float32)
    if kind == "lattice":
        return rng.permutation(np.stack(np.unravel_index(np.arange(N), (64, 64, (N + 4095) // 4096)), -1)).astype(np.float32)
    return rng.random((N, 3), dtype=np.float32)


def compare(fp, p, n, G, start=None):
    x = torch.from_numpy(p).cuda()
    want = exact_by_index(fp, x, n, want_mdc=True, start_idx=start)
    fp.set_wg_per_cloud(G)
    try:
        got = fp.fps_exact_pruned(x, n, want_mdc=True, want_info=True, start_idx=start)
        torch.cuda.synchronize()
    finally:
        fp.set_wg_per_cloud(0)
    assert all(i.status == 0 for i in fp.parse_info(got[2]))
    assert torch.equal(got[0], want[0]) and torch.equal(got[1].view(torch.int32), want[1].view(torch.int32))


@pytest.mark.parametrize("kind", ["uniform", "sheet", "dense corner"])
@pytest.mark.parametrize("N,G", [(1023, 1), (1025, 1), (4097, 1), (8192, 1), (1025, 2), (8192, 2), (20000, 3), (66000, 33),
                                 (66000, 129), (66000, 256)])
def test_points_per_thread_and_workgroups(fp, kind, N, G):
    compare(fp, cloud(kind, N)[None], min(N, 1200), G)


@pytest.mark.parametrize("n", [1, 2, 3, 4096, 4097, 4098, 8193, 20000])
def test_sequence_at_the_edges(fp, n):
    compare(fp, cloud("uniform", 20000)[None], n, 20)


@pytest.mark.parametrize("N,n,G", [(8192, 5000, 8), (12288, 6000, 3)])
def test_equal_distances(fp, N, n, G):
    compare(fp, cloud("lattice", N)[None], n, G)


def test_duplicates_and_start(fp):
    p = np.repeat(cloud("uniform", 700), 9, axis=0)
    compare(fp, np.stack([p, p[::-1]]), 5000, 6, start=[6299, 17])


def test_more_clouds_than_fit(fp):
    compare(fp, np.stack([cloud("uniform", 3000 + 0 * b) + b for b in range(60)]), 400, 5)
