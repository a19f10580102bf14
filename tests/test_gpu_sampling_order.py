"""Clouds in sampling order -- the gathered samples of an earlier stage, which sample to 0, 1, 2, ... again -- and clouds that
are so only up to some point: the samplers follow such a sequence without searching for it.  Against the oracle: the
sequence complete, broken off at the borders of the stretches it is tried in (64, 512, 4096) and beside them, points moved
by little, equal points, another start; exact FPS and MDPS, with and without a record, one workgroup and many."""
import numpy as np
import pytest

from oracle import ref
from paper_2507_23480_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fp():
    from paper_2507_23480_amd import binding
    binding.load()
    binding.set_wg_per_cloud(0)
    yield binding
    binding.set_wg_per_cloud(0)


ORDERED = {}


def ordered(N, kind="C3"):
    if (N, kind) not in ORDERED:
        p = inputs.make_cloud(kind, 77, 3 * N)
        ORDERED[N, kind] = p[ref.fps_exact(p, N)[0]]
    return ORDERED[N, kind].copy()


def check(fp, p, n, bias=1.05, radius=0.3, starts=None):
    x = torch.from_numpy(p[None]).cuda()
    start = None if starts is None else [starts]
    widx, wmdc = ref.fps_exact(p, n, start=starts or 0)
    for f in (fp.fps_exact, fp.fps_exact_pruned):
        idx, mdc = f(x, n, want_mdc=True, start_idx=start)
        assert np.array_equal(idx.cpu().numpy()[0], widx) and np.array_equal(mdc.cpu().numpy()[0], wmdc)
    rp, prm = ref.MdpsParams(exponent=0.8, bias=bias), fp.MdpsParams(exponent=0.8, bias=bias)
    wm, winfo = ref.mdps_sample(p, n, rp, start=starts or 0)
    wbq, wcnt = ref.ball_query(p, wm, radius, 16)
    for sample in (fp.mdps_sample, fp.mdps_sample_pruned):
        m, info = sample(x, n, prm, want_info=True, start_idx=start)
        cache = fp.new_bq_cache(x, n)
        r, rinfo = sample(x, n, prm, want_info=True, start_idx=start, bq_cache=cache, bq_radius=radius)
        bq, cnt = fp.ball_query(x, r, radius, 16, bq_cache=cache)
        assert np.array_equal(m.cpu().numpy()[0], wm) and np.array_equal(r.cpu().numpy()[0], wm)
        for i in fp.parse_info(info) + fp.parse_info(rinfo):
            assert i.status == 0 and i.m == winfo.m and i.et_index == winfo.et_index
            assert list(i.level_start)[:6] == list(winfo.level_start)[:6]
            assert list(i.level_exhausted)[:6] == list(winfo.level_exhausted)[:6]
            assert np.array_equal(np.array(list(i.thr2)[:6], np.float32), np.asarray(winfo.thr2, np.float32)[:6])
        assert np.array_equal(bq.cpu().numpy()[0], wbq) and np.array_equal(cnt.cpu().numpy()[0], wcnt)
        assert not any(fp.bq_cache_stats(cache)["incomplete"])


@pytest.mark.parametrize("bias", [0.9, 1.05, 1.4])
@pytest.mark.parametrize("N,n", [(100, 15), (100, 16), (375, 94), (1500, 375), (1024, 512), (3000, 3000), (6000, 1500), (9000, 1600)])
def test_in_order(fp, N, n, bias):
    check(fp, ordered(N), n, bias)


# the sequence breaks off at point `at`: two points exchanged, or everything behind it shuffled
@pytest.mark.parametrize("how", ["swap", "shuffle"])
@pytest.mark.parametrize("N,n,at", [(1500, 375, a) for a in (2, 63, 64, 65, 300)] +
                         [(6000, 1500, a) for a in (7, 63, 64, 511, 512, 513, 1400)] + [(9000, 5000, a) for a in (4095, 4096, 4999)])
def test_breaks_off(fp, N, n, at, how):
    p = ordered(N)
    if how == "swap":
        p[[at, at + 7]] = p[[at + 7, at]]
    else:
        p[at:] = np.random.default_rng(at).permutation(p[at:])
    check(fp, p, n)


@pytest.mark.parametrize("how", ["swap", "shuffle"])
@pytest.mark.parametrize("N,n,at", [(6000, 1500, 513), (6000, 1500, 1000), (6000, 1500, 1400), (9000, 5000, 4097)])
def test_goes_on_where_it_breaks_off(fp, N, n, at, how):
    """The samples in front of the break are kept: the rounds are those for the rest, a part of those for the cloud in no
    order (some waves of both sizes hold no points)."""
    p = ordered(N)
    q = np.random.default_rng(1).permutation(p)
    if how == "swap":
        p[[at, at + 7]] = p[[at + 7, at]]
    else:
        p[at:] = np.random.default_rng(at).permutation(p[at:])
    rounds = [fp.parse_info(fp.fps_exact_pruned(torch.from_numpy(c[None]).cuda(), n, want_info=True)[1])[0].rounds for c in (p, q)]
    # (the curve falls with the number of samples, and the lists follow it down by some factor a round)
    assert rounds[0] < (0.5 if at < n / 2 else 0.25) * rounds[1]


def test_moved_equal_and_other_start(fp):
    p = ordered(6000)
    check(fp, p, 1600, starts=5)
    q = p.copy()
    q[1200] = q[40]                         # lies on a sample: never one itself
    check(fp, q, 1600)
    q = p.copy()
    q[5000] += np.float32(2.0)              # no sample of the first 1600, but farther than one of them
    check(fp, q, 1600)
    q = p.copy()
    q[5500] = np.nan
    check(fp, q[:5400], 1600)
    x = torch.from_numpy(q[None]).cuda()
    want = ref.fps_exact(q, 40)[0]
    assert np.array_equal(fp.fps_exact(x, 40).cpu().numpy()[0], want)


def test_batch_of_both_kinds(fp):
    ps = [ordered(2000), inputs.make_cloud("C3", 5, 2000), ordered(2000)[::-1].copy(), ordered(2000, "C1")] * 3
    x = torch.from_numpy(np.stack(ps)).cuda()
    for G in (0, 1, 4):
        fp.set_wg_per_cloud(G)
        try:
            got = fp.fps_exact(x, 700), fp.fps_exact_pruned(x, 700)
        finally:
            fp.set_wg_per_cloud(0)
        for b, p in enumerate(ps):
            want = ref.fps_exact(p, 700)[0]
            assert all(np.array_equal(g[b].cpu().numpy(), want) for g in got)


def test_several_clouds_to_a_group(fp):
    """more clouds than groups of workgroups: one group follows cloud after cloud, some of them in order to the end, others
    up to some point"""
    p = ordered(6000)
    q = p.copy()
    q[900:] = np.random.default_rng(3).permutation(q[900:])
    x = torch.from_numpy(np.stack([p, q, p, p, q, q, p] * 3)).cuda()
    want = [ref.fps_exact(c, 1500) for c in (p, q)]
    for G in (64, 100):                     # 4 groups, 2 groups
        fp.set_wg_per_cloud(G)
        try:
            got = [f(x, 1500, want_mdc=True) for f in (fp.fps_exact, fp.fps_exact_pruned)]
        finally:
            fp.set_wg_per_cloud(0)
        for b, k in enumerate([0, 1, 0, 0, 1, 1, 0] * 3):
            for idx, mdc in got:
                assert np.array_equal(idx[b].cpu().numpy(), want[k][0]) and np.array_equal(mdc[b].cpu().numpy(), want[k][1])


@pytest.mark.parametrize("G", [5, 33, 128])
def test_followed_behind_searched(fp, G):
    """clouds in order next to clouds in none in the turn of a group, with few samples and so short lists, which most
    workgroups have no share of"""
    p = ordered(3000)
    q = np.random.default_rng(4).permutation(p)
    kinds = ([0] * (256 // G) + [1] * (256 // G)) * 6
    x = torch.stack([torch.from_numpy(p).cuda(), torch.from_numpy(q).cuda()])[torch.tensor(kinds)].contiguous()
    for n in (20, 300):
        want = [ref.fps_exact(c, n)[0] for c in (p, q)]
        fp.set_wg_per_cloud(G)
        try:
            got = [f(x, n).cpu().numpy() for f in (fp.fps_exact, fp.fps_exact_pruned)]
        finally:
            fp.set_wg_per_cloud(0)
        for b, k in enumerate(kinds):
            assert all(np.array_equal(g[b], want[k]) for g in got)
