"""The number of samples decides whether a sampler sorts the cloud into cells first: either side of the lines the same
samples, and the layout the rule names.  It is told by the number of rounds: an index-ordered run always takes the same,
a cell-ordered one fewer, which may differ by a few from run to run (points of one cell lie in no fixed order)."""
import numpy as np
import pytest

from paper_2507_23480_amd import inputs
from tests.routes import exact_by_index, in_cells, scan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fp():
    from paper_2507_23480_amd import binding
    binding.load()
    binding.set_wg_per_cloud(0)
    yield binding
    binding.set_wg_per_cloud(0)


def rounds(fp, info):
    return [i.rounds for i in fp.parse_info(info)]


@pytest.mark.parametrize("B,N,n", [(2, 6000, 40), (2, 6000, 1499), (2, 6000, 1500), (1, 5120, 1500), (1, 5121, 1500),
                                   (2, 40001, 1499), (2, 40001, 1500), (140, 5121, 2999), (140, 5121, 3000)])
def test_exact(fp, B, N, n):
    x = torch.from_numpy(np.stack([inputs.make_cloud("C3", 40 + b % 3, N) for b in range(B)])).cuda()
    few = 256 // B <= 2                                     # workgroups per cloud
    want, ordered = exact_by_index(fp, x, n, want_info=True)
    cells, sorted_ = in_cells(fp, x, lambda: fp.fps_exact_pruned(x, n, want_info=True))
    assert torch.equal(cells, want) and rounds(fp, sorted_) != rounds(fp, ordered)
    many = n >= (3000 if few else 1500)
    for f, cell_order in ((fp.fps_exact, many and N >= 5121), (fp.fps_exact_pruned, many)):
        got, info = f(x, n, want_info=True)
        assert torch.equal(got, want)
        assert (rounds(fp, info) == rounds(fp, ordered)) == (not cell_order)


@pytest.mark.parametrize("order,n", [(0, 1999), (0, 2000), (1, 1499), (1, 1500)])
@pytest.mark.parametrize("N", [2049, 2100, 20011])
def test_mdps(fp, order, n, N):
    x = torch.from_numpy(np.stack([inputs.make_cloud("C3", 60 + b, N) for b in range(2)])).cuda()
    prm = fp.MdpsParams(exponent=0.8, bias=1.05, scan_order=order)
    want, ordered = fp.mdps_sample(x, n, prm, want_info=True)
    cells, sorted_ = in_cells(fp, x, lambda: fp.mdps_sample_pruned(x, n, prm, want_info=True))
    got, info = fp.mdps_sample_pruned(x, n, prm, want_info=True)
    assert torch.equal(cells, want) and torch.equal(got, want)
    assert rounds(fp, sorted_) != rounds(fp, ordered)
    assert (rounds(fp, info) == rounds(fp, ordered)) == (n % 100 != 0)


@pytest.mark.parametrize("N,n", [(12000, 5100), (12000, 5110), (12000, 5120), (12000, 5130), (12000, 300)])
@pytest.mark.parametrize("order", [0, 1])
def test_prefix_either_side_of_the_sweeps(fp, N, n, order):
    """A prefix of a tenth of the samples: 511 to 513 picks, and a short one, with and without a record."""
    x = torch.from_numpy(np.stack([inputs.make_cloud("C3", 70 + b, N) for b in range(2)])).cuda()
    prm = fp.MdpsParams(exponent=0.8, bias=1.05, scan_order=order)
    want = fp.mdps_sample(x, n, prm)
    cache = fp.new_bq_cache(x, n)
    assert torch.equal(in_cells(fp, x, lambda: fp.mdps_sample_pruned(x, n, prm)), want)
    assert torch.equal(fp.mdps_sample_pruned(x, n, prm, bq_cache=cache, bq_radius=0.1), want)
    wanted = scan(fp, x, want, 0.1, 16)
    got = fp.ball_query(x, want, 0.1, 16, bq_cache=cache)
    assert torch.equal(got[0], wanted[0]) and torch.equal(got[1], wanted[1])


@pytest.mark.parametrize("places", [1, 6, 7, 12, 13, 27, 60])
def test_a_far_point_leaves_few_cells(fp, places):
    """Waves whose points share that many cells, and a last wave that is not full: the sort into cells loses no point."""
    N, n = 5185, 1600
    rng = np.random.default_rng(places)
    x = rng.random((2, N, 3)).astype(np.float32)
    x[..., 0] += 15.625 * rng.integers(0, places, (2, N))
    x[:, N // 3, 0] = 1000.0
    x = torch.from_numpy(x).cuda()
    want = exact_by_index(fp, x, n)
    assert torch.equal(in_cells(fp, x, lambda: fp.fps_exact_pruned(x, n)), want) and torch.equal(fp.fps_exact(x, n), want)
    c = want[:, ::7].contiguous()
    for r in (0.05, 0.3):
        for a, b in zip(fp.ball_query_grid(x, c, r, 16), scan(fp, x, c, r, 16)):
            assert torch.equal(a, b)
