"""Exact rounds settled in sweeps, and the size rule that picks a sampler's layout: the cell-ordered kernels and
the index-ordered ones have to agree bit for bit, on clouds where most candidates of a round touch each
other (lattices, lines, duplicates, clusters of nearly equal points) and on either side of the rule's lines."""

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


def clouds(kind, N, seed):
    rng = np.random.default_rng([seed, N])
    if kind == "lattice":                      # equal distances everywhere
        s = int(np.ceil(N ** (1 / 3)))
        p = np.stack(np.meshgrid(*[np.arange(s)] * 3, indexing="ij"), -1).reshape(-1, 3)[:N]
        return rng.permutation(p).astype(np.float32)
    if kind == "line":                         # long chains of candidates that lower each other
        p = np.zeros((N, 3))
        p[:, 0] = np.arange(N)
        return p.astype(np.float32)
    if kind == "duplicates":
        return rng.integers(0, 12, (N, 3)).astype(np.float32)
    if kind == "clusters":
        return (rng.normal(size=(7, 3))[rng.integers(0, 7, N)] + 1e-3 * rng.normal(size=(N, 3))).astype(np.float32)
    return rng.random((N, 3), dtype=np.float32)


def index_ordered(fp, x, n, start=None):
    """fps_exact_static: its fixed scratch keeps it on the index-ordered kernels at every size."""
    B = x.shape[0]
    idx = torch.empty((B, n), dtype=torch.int32, device="cuda")
    mdc = torch.empty((B, n), dtype=torch.float32, device="cuda")
    fp.fps_exact_static(x, n, idx, mdc, start)
    return idx, mdc


@pytest.mark.parametrize("kind", ["lattice", "line", "duplicates", "clusters", "uniform"])
@pytest.mark.parametrize("N,G", [(63, 1), (257, 1), (1000, 1), (1500, 2), (3000, 5), (4096, 1), (5200, 6)])
def test_sweeps_match_oracle(fp, kind, N, G):
    p = clouds(kind, N, 5)
    n = min(N, 700)
    fp.set_wg_per_cloud(G)                     # the cell-ordered kernels whatever the size
    try:
        idx, mdc = fp.fps_exact_pruned(torch.from_numpy(p[None]).cuda(), n, want_mdc=True)
        torch.cuda.synchronize()
    finally:
        fp.set_wg_per_cloud(0)
    want = ref.fps_exact(p, n)
    assert np.array_equal(idx.cpu().numpy()[0], want[0])
    assert np.array_equal(mdc.cpu().numpy()[0], want[1])


@pytest.mark.parametrize("N", [2048, 2049, 5120, 5121, 8191, 8192, 20011])
def test_either_side_of_the_rule(fp, N):
    x = torch.from_numpy(np.stack([clouds(k, N, 7) for k in ("uniform", "clusters", "lattice")])).cuda()
    n = N // 5
    start = torch.tensor([0, N - 1, 17], dtype=torch.int32, device="cuda")
    want = index_ordered(fp, x, n, start)
    for f in (fp.fps_exact, fp.fps_exact_pruned):
        got = f(x, n, start_idx=start, want_mdc=True)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    for order in (0, 1):
        prm = fp.MdpsParams(exponent=0.8, bias=1.05, scan_order=order)
        assert torch.equal(fp.mdps_sample(x, n, prm), fp.mdps_sample_pruned(x, n, prm))


@pytest.mark.parametrize("N", [3000, 6000])
def test_small_workspace_and_odd_coordinates(fp, N):
    p = clouds("uniform", N, 9)
    p[5] = np.nan
    p[11, 1] = np.inf
    p[12, 2] = -np.inf
    p[20] = 3e38
    x = torch.from_numpy(p[None]).cuda()
    want = index_ordered(fp, x, 300)
    got = fp.fps_exact(x, 300, want_mdc=True)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1].view(torch.int32), want[1].view(torch.int32))
    # the workspace of the index-ordered kernels stays enough
    small = torch.empty(int(fp.load().fp_workspace_bytes(1, 10)), dtype=torch.uint8, device="cuda")
    assert torch.equal(fp.fps_exact(x, 300, ws=small), want[0])


def test_captured(fp):
    x = torch.from_numpy(np.stack([inputs.make_cloud("C3", 600, 9000) for _ in range(2)])).cuda()
    ws = fp.new_workspace(x.device, 2, 9000)
    idx = torch.empty((2, 900), dtype=torch.int32, device="cuda")
    fp.set_cooperative_launch(False)
    try:
        lib = fp.load()
        side = torch.cuda.Stream()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            status = lib.fp_fps_exact(x.data_ptr(), 2, 9000, 900, None, idx.data_ptr(), None, None, None, 0, 0.0,
                                      ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
        assert status == 0
        for rep in range(3):
            x.copy_(torch.from_numpy(np.stack([inputs.make_cloud("C3", 600 + rep + b, 9000) for b in range(2)])))
            idx.fill_(-7)
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(idx, index_ordered(fp, x, 900)[0])
    finally:
        fp.set_cooperative_launch(True)
