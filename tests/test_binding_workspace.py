"""The samplers' shared workspace keeps its address: a graph captured from one call replays into it after calls on
larger clouds."""
import pytest

torch = pytest.importorskip("torch")


@pytest.fixture()
def fp(monkeypatch):
    from paper_2507_23480_amd import binding
    binding.load()
    monkeypatch.setattr(binding, "_workspaces", {})
    return binding


def test_shared_workspace_is_one_for_all_shapes(fp):
    ws = fp.workspace(torch.device("cpu"), 1, 4096)
    assert ws.numel() >= max(int(fp.load().fp_workspace_bytes(b, n)) for b, n in ((1, 1), (8, 4096)))
    assert fp.workspace(torch.device("cpu"), 4, 120000).data_ptr() == ws.data_ptr()


@pytest.mark.parametrize("call", ["fps_exact", "mdps_sample"])
def test_default_workspace_survives_larger_clouds(fp, monkeypatch, call):
    """The address handed to the library for a small cloud stays that of a live tensor after a larger call."""
    seen = []

    class Lib:
        def __getattr__(self, name):
            if name in ("fp_fps_exact", "fp_mdps_sample"):
                return lambda *args: seen.append((args[1:3], args[-3])) or 0
            return getattr(real, name)

    real = fp.load()
    monkeypatch.setattr(fp, "load", Lib)
    monkeypatch.setattr(fp, "_stream", lambda: 0)
    monkeypatch.setattr(fp, "_xyz", lambda x: (int(x.shape[0]), int(x.shape[1])))
    args = (64,) if call == "fps_exact" else (64, fp.MdpsParams())
    for n in (4096, 120000, 4096):
        getattr(fp, call)(torch.zeros((1, n, 3)), *args)
    small, _, again = [ptr for _, ptr in seen]
    assert small == again
    assert small in [t.data_ptr() for t in fp._workspaces.values()]


@pytest.mark.gpu
def test_graph_replays_after_a_larger_call(fp):
    from paper_2507_23480_amd import inputs
    import numpy as np
    x = torch.from_numpy(inputs.make_batch("C1")).cuda()                       # 4096 points, four workgroups
    want = fp.fps_exact(x, 512)
    torch.cuda.synchronize()
    fp.set_cooperative_launch(False)
    try:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=torch.cuda.Stream()):
            idx = fp.fps_exact(x, 512)
        big = torch.from_numpy(np.stack([inputs.make_cloud("C3", 900, 20000)])).cuda()
        for _ in range(3):
            idx.fill_(-7)
            fp.fps_exact(big, 2000)
            keep = torch.zeros(8 << 20, dtype=torch.uint8, device="cuda")      # takes up whatever was freed
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(idx, want) and int(keep.sum()) == 0
    finally:
        fp.set_cooperative_launch(True)
