"""The grid query leaves clouds whose balls, or whose one far point, make its cells useless to a look at all points in
index order: the bytes are those of the scan either way, also where a batch holds clouds of both kinds."""
import numpy as np
import pytest

from tests.routes import scan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fp():
    from paper_2507_23480_amd import binding
    binding.load()
    return binding


def scene(kind, N, rng):
    p = rng.random((N, 3))
    if kind == "far_point":                     # the other points share a cell
        p[N // 3] = 1e5
    elif kind == "spread":                      # balls of a point or two: the cells are used
        p *= 100.0
    elif kind == "odd":
        p[5], p[6, 1], p[7] = np.nan, np.inf, 3e38
    elif kind == "one_place":
        p[:] = 0.25
    return p


@pytest.mark.parametrize("kinds", [("wide",), ("far_point",), ("one_place",), ("odd",), ("wide", "spread", "far_point"),
                                   ("spread", "wide")])
@pytest.mark.parametrize("N", [1, 63, 300, 4096, 4097, 5200, 13001])
def test_same_bytes(fp, kinds, N):
    rng = np.random.default_rng([len(kinds), N])
    B = len(kinds)
    x = torch.from_numpy(np.stack([scene(k if N > 8 else "wide", N, rng) for k in kinds]).astype(np.float32)).cuda()
    for M in (1, 7, 33, 259):
        c = rng.integers(0, N, (B, M)).astype(np.int32)
        if M > 8:
            c[0, 2], c[B - 1, 6] = -1, N
        c = torch.from_numpy(c).cuda()
        for r, k in ((0.5, 16), (0.02, 5), (3.0, 254), (0.2, 1), (1e30, 65)):
            want = scan(fp, x, c, r, k)
            for f in (fp.ball_query, fp.ball_query_grid):
                got = f(x, c, r, k)
                assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), (M, r, k)


def test_without_counts(fp):
    x = torch.from_numpy(np.random.default_rng(1).random((1, 6000, 3)).astype(np.float32)).cuda()
    c = torch.arange(0, 6000, 20, dtype=torch.int32, device="cuda")[None].contiguous()
    ws = torch.empty(int(fp.load().fp_ball_query_grid_workspace_bytes(1, 6000)), dtype=torch.uint8, device="cuda")
    idx = torch.empty((1, 300, 12), dtype=torch.int32, device="cuda")
    assert fp.load().fp_ball_query_grid(x.data_ptr(), 1, 6000, c.data_ptr(), 300, 0.6, 12, idx.data_ptr(), None,
                                        ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(idx, scan(fp, x, c, 0.6, 12)[0])


def test_lines_of_the_route(fp):
    for B, N, M, grid in ((1, 5120, 500, False), (1, 5121, 500, True), (8, 5121, 64, True), (9, 5121, 500, False),
                          (9, 10000, 500, True), (1, 11999, 63, False), (1, 12000, 63, True), (9, 12000, 1, True)):
        assert fp.grid_query(B, N, M) == grid
