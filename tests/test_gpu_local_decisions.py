"""Sampling by local decisions (the cell-ordered fps_exact, and mdps_sample_pruned from 5000 samples on): the samples and the curve of the index-ordered kernels, bit for
bit, where the sampler and the kernel that puts the samples in sequence change their ways -- one to eight points per
thread, one workgroup and many, lists at their limits, equal distances, n at the edges of a workgroup's keys."""
import numpy as np
import pytest

from oracle import ref
from tests.routes import exact_by_index, scan

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
    if kind == "path":                          # indices follow a curve, a sensor on its way
        t = np.linspace(0.0, 200.0, N)
        p = np.stack([30.0 * np.cos(t / 7.0) + t / 10.0, 30.0 * np.sin(t / 9.0), 0.02 * t], axis=-1)
        return (p + 0.01 * rng.normal(size=(N, 3))).astype(np.float32)
    if kind == "rows":                          # a lattice by rows and layers
        return np.stack(np.unravel_index(np.arange(N), ((N + 1023) // 1024, 32, 32)), axis=-1).astype(np.float32)
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


# Ranges of more samples than a workgroup has places for in the kernel that puts the samples in sequence: all points sampled,
# the smallest distance far below the others; more than 4096 samples at one distance; both beside ranges of a few
@pytest.mark.parametrize("kind,N,n", [("uniform", 2049, 2049), ("uniform", 3000, 3000), ("uniform", 20000, 20000), ("uniform", 20000, 19000),
                                      ("dense corner", 12289, 12289), ("near", 20000, 19990), ("near", 6145, 6145),
                                      ("lattice", 32768, 16384), ("lattice", 16384, 16384)])
def test_long_ranges(fp, kind, N, n):
    p = cloud("uniform" if kind == "near" else kind, N)
    if kind == "near":                          # a pair of points, the closer the more ranges lie above the others
        p[5] = p[6] + np.float32(1e-7) * np.arange(3, dtype=np.float32)
    compare(fp, p[None], n, 8)


def test_equal_samples_of_a_prefix(fp):
    """index 0 some thousand times, at the end of a prefix longer than the cloud has different points"""
    p = np.resize(cloud("uniform", 700), (60000, 3))
    compare_mdps(fp, p[None], 50000, 60, fp.MdpsParams(exponent=0.7, bias=1.05, p=0.2), 0.05)


def test_all_points_sampled_in_time(fp):
    """Twice the samples, the last of them at distances far below the others, take about twice the time."""
    x = torch.from_numpy(cloud("uniform", 20000)[None]).cuda()

    def best(n):
        times = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            fp.fps_exact_pruned(x, n)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)
    assert best(20000) < 4.0 * best(10000)


def test_duplicates_and_start(fp):
    p = np.repeat(cloud("uniform", 700), 9, axis=0)
    compare(fp, np.stack([p, p[::-1]]), 5000, 6, start=[6299, 17])


def test_more_clouds_than_fit(fp):
    compare(fp, np.stack([cloud("uniform", 3000 + 0 * b) + b for b in range(60)]), 400, 5)


def info_words(fp, info):
    return [(i.m, i.et_index, list(i.level_start), list(i.level_exhausted), list(i.thr2), i.status)
            for i in fp.parse_info(info)]


def compare_mdps(fp, p, n, G, prm, radius, start=None):
    """From 5000 samples on the cell-ordered MDPS runs by local decisions: against the index-ordered kernels, the record
    against the scan of all points."""
    x = torch.from_numpy(p).cuda()
    want, winfo = fp.mdps_sample(x, n, prm, want_info=True, start_idx=start)
    cache = fp.new_bq_cache(x, n)
    fp.set_wg_per_cloud(G)
    try:
        got, info = fp.mdps_sample_pruned(x, n, prm, want_info=True, start_idx=start)
        rec = fp.mdps_sample_pruned(x, n, prm, start_idx=start, bq_cache=cache, bq_radius=radius)
        torch.cuda.synchronize()
    finally:
        fp.set_wg_per_cloud(0)
    assert torch.equal(got, want) and torch.equal(rec, want)
    assert info_words(fp, info) == info_words(fp, winfo)
    for a, b in zip(fp.ball_query(x, rec, radius, 16, bq_cache=cache), scan(fp, x, rec, radius, 16)):
        assert torch.equal(a, b)
    return fp.bq_cache_stats(cache)


# bias: levels cut by their quota (0.8), exhausted (1.05), exhausted early, so that most of the samples are a remainder (2.0)
@pytest.mark.parametrize("bias", [0.8, 1.05, 2.0])
@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("N,G", [(8192, 1), (8192, 2), (12001, 3), (12001, 12), (40000, 40), (66000, 129)])
def test_mdps(fp, order, N, G, bias):
    stats = compare_mdps(fp, cloud("uniform", N)[None], 5000, G, fp.MdpsParams(exponent=0.7, bias=bias, scan_order=order), 0.04)
    assert stats["cell_order"] and not any(stats["incomplete"])


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("kind", ["sheet", "dense corner", "lattice"])
def test_mdps_uneven(fp, kind, order):
    radius = {"sheet": 1.0, "dense corner": 0.03, "lattice": 1.5}[kind]
    prm = fp.MdpsParams(exponent=1.0, bias=1.05, scan_order=order)
    compare_mdps(fp, np.stack([cloud(kind, 20480), cloud(kind, 20480)[::-1]]), 5003, 20, prm, radius, start=[20479, 5])


# Samples that wait for one another: lists settled in order.  Levels cut by their quota inside a list, exhausted, followed by a
# remainder; a list's candidates in one wave and in all; one workgroup and many; both scan orders
@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("kind,N,G,R", [("path", 8192, 1, 0.9), ("path", 8192, 3, 0.9), ("path", 40000, 40, 0.9), ("path", 40000, 7, 2.0),
                                        ("path", 40000, 256, 0.2), ("rows", 8192, 2, 2.5), ("rows", 32768, 32, 3.1)])
def test_mdps_chains(fp, kind, N, G, R, order):
    p = cloud(kind, N)
    thr = [(f * R) ** 2 for f in (1.6, 1.0, 0.6, 0.25)]
    prm = fp.MdpsParams(p=0.002, nseg=4, m_min=4, thr_override=thr, scan_order=order)
    compare_mdps(fp, np.stack([p, p[::-1]]), 5000, G, prm, R, start=[N - 1, 3])


def test_mdps_chains_take_few_rounds(fp):
    """A path of 40000 points, 6000 samples: 256 candidates settled in order a round take 248 to 760 rounds, a sample per chain
    and round 1228 to 3242."""
    x = torch.from_numpy(cloud("path", 40000)[None]).cuda()
    r = 200 * 4.0 / 6000
    for prm in (fp.MdpsParams(p=0.01, exponent=2.0), fp.MdpsParams(p=0.001, exponent=2.0),
                fp.MdpsParams(p=0.001, nseg=3, thr_override=[(1.6 * r) ** 2, r ** 2, (0.5 * r) ** 2])):
        got, info = fp.mdps_sample_pruned(x, 6000, prm, want_info=True)
        assert fp.parse_info(info)[0].rounds < 300
        assert torch.equal(got, fp.mdps_sample(x, 6000, prm))


@pytest.mark.parametrize("order", [0, 1])
def test_mdps_duplicates(fp, order):
    """More samples than different points: exact FPS repeats index 0, in the prefix already or at the end."""
    for different in (300, 4000):
        p = np.resize(cloud("uniform", different), (9000, 3))
        compare_mdps(fp, p[None], 6000, 9, fp.MdpsParams(exponent=0.7, bias=1.05, scan_order=order), 0.05)


def test_mdps_given_thresholds_small_record_and_short_prefix(fp):
    p = cloud("uniform", 20000)[None]
    x = torch.from_numpy(p).cuda()
    thr = [0.004, 0.0025, 0.0012]
    compare_mdps(fp, p, 5000, 20, fp.MdpsParams(p=0.001, nseg=3, m_min=1, thr_override=thr), 0.04)
    compare_mdps(fp, p, 5000, 20, fp.MdpsParams(p=0.9999, exponent=0.7), 0.04)          # the prefix is everything
    prm = fp.MdpsParams(exponent=0.7, bias=1.05, scan_order=1)
    small = fp.new_bq_cache(x, 5000, 256)
    got = fp.mdps_sample_pruned(x, 5000, prm, bq_cache=small, bq_radius=0.04)
    assert all(fp.bq_cache_stats(small)["incomplete"])
    for a, b in zip(fp.ball_query(x, got, 0.04, 16, bq_cache=small), scan(fp, x, got, 0.04, 16)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("G", [1, 3, 8])
def test_stamps_start_again_in_a_cloud(fp, G):
    """Equal distances take a round a sample: the stamps of published candidates start again (after 100 rounds with a
    number of workgroups forced) within one cloud; with one workgroup there is nothing to renew."""
    x = torch.from_numpy(cloud("lattice", 8192)[None]).cuda()
    want = exact_by_index(fp, x, 3000, want_mdc=True)
    fp.set_wg_per_cloud(G)
    try:
        idx, mdc, info = fp.fps_exact_pruned(x, 3000, want_mdc=True, want_info=True)
    finally:
        fp.set_wg_per_cloud(0)
    assert fp.parse_info(info)[0].status == 0 and fp.parse_info(info)[0].rounds > 3 * 100
    assert torch.equal(idx, want[0]) and torch.equal(mdc.view(torch.int32), want[1].view(torch.int32))


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("G", [1, 64, 128])
def test_stamps_start_again_between_clouds(fp, G, order):
    """The rounds of a group go on over its clouds."""
    clouds = 256 // G * 10
    x = torch.stack([torch.from_numpy(cloud("uniform", 8192) + np.float32(b)).cuda() for b in range(5)]).repeat(clouds // 5, 1, 1)
    prm = fp.MdpsParams(exponent=0.7, bias=1.05, scan_order=order)
    want = [fp.mdps_sample(x[:5], 5000, prm), exact_by_index(fp, x[:5], 3000)]
    fp.set_wg_per_cloud(G)
    try:
        got, info = fp.mdps_sample_pruned(x, 5000, prm, want_info=True)
        got, info = [got, None], [info, None]
        got[1], info[1] = fp.fps_exact_pruned(x, 3000, want_info=True)
    finally:
        fp.set_wg_per_cloud(0)
    for g, w, i in zip(got, want, info):
        rounds = [k.rounds for k in fp.parse_info(i)]
        assert sum(rounds[::256 // G]) > 2 * 100 and all(k.status == 0 for k in fp.parse_info(i))
        assert all(torch.equal(g[b], w[b % 5]) for b in range(clouds))


def test_more_above_a_level_than_16_bits_count(fp):
    """a hemisphere of a million points just below the fourth level of the first list, 66200 of them just above: evenly
    mixed, so that no part of the cloud has more of them than it may list, and 664 too many for 16 bits"""
    rng = np.random.default_rng(9)
    N, above = 1000000, 66200
    u = rng.normal(size=(N, 3))
    u[:, 0] = -np.abs(u[:, 0]) - 0.05
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    r2 = np.full(N, 0.510)
    r2[rng.choice(np.arange(2, N), above, replace=False)] = 0.514
    p = (u * np.sqrt(r2)[:, None]).astype(np.float32)
    p[0], p[1] = 0.0, (1.0, 0.0, 0.0)
    n = 300
    idx, mdc = fp.fps_exact_pruned(torch.from_numpy(p[None]).cuda(), n, want_mdc=True)
    want, wmdc = ref.fps_exact(p, n)
    assert np.array_equal(idx.cpu().numpy()[0], want) and np.array_equal(mdc.cpu().numpy()[0], wmdc)
