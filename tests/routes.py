"""One kernel by name where a public call picks between several: the references that tests of the others compare with."""
import ctypes

import torch


def own_workgroups(fp, B, N):
    """The number of workgroups per cloud the library would choose; forced, it keeps an entry point's own layout."""
    g, t, p = ctypes.c_int32(), ctypes.c_int32(), ctypes.c_int32()
    assert fp.load().fp_plan(B, N, ctypes.byref(g), ctypes.byref(t), ctypes.byref(p)) == 0
    return g.value


def in_cells(fp, x, call):
    """call() of a _pruned sampler on the cell-ordered kernels whatever the number of samples."""
    fp.set_wg_per_cloud(own_workgroups(fp, x.shape[0], x.shape[1]))
    try:
        return call()
    finally:
        fp.set_wg_per_cloud(0)


def exact_by_index(fp, x, n, **kw):
    """fps_exact on the index-ordered kernels: their workspace has no room for a cell-ordered copy."""
    ws = torch.empty(int(fp.load().fp_workspace_bytes(1, 1)), dtype=torch.uint8, device="cuda")
    return fp.fps_exact(x, n, ws=ws, **kw)


def scan(fp, x, c, r, k):
    """The ball query by a scan of all points."""
    B, N = x.shape[:2]
    M = c.shape[1]
    idx = torch.empty((B, M, k), dtype=torch.int32, device="cuda")
    cnt = torch.empty((B, M), dtype=torch.int32, device="cuda")
    assert fp.load().fp_ball_query(x.data_ptr(), B, N, c.data_ptr(), M, float(r), k, idx.data_ptr(), cnt.data_ptr(),
                                   None, torch.cuda.current_stream().cuda_stream) == 0
    return idx, cnt


def all_pairs(fp, x, s, k):
    """The k nearest samples by comparing every point with every sample."""
    B, N = x.shape[:2]
    pos = torch.empty((B, N, k), dtype=torch.int32, device="cuda")
    d2 = torch.empty((B, N, k), device="cuda")
    assert fp.load().fp_knn(x.data_ptr(), B, N, s.data_ptr(), s.shape[1], k, pos.data_ptr(), d2.data_ptr(),
                            None, None, None, 0, torch.cuda.current_stream().cuda_stream) == 0
    return pos, d2
