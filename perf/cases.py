"""The work a user has this library do, as cases of one pass each.

A pass goes through the public entry points of paper_2507_23480_amd.binding the way a network's
sampling layer calls them: set abstraction (a sampler, the ball query around its samples and, in a
hierarchy, the gather that feeds the next stage), the k-NN of an up-sampling layer, and exclusion
lists built as a data structure.  Sizes and clouds are those of the repository's five workloads
(paper_2507_23480_amd/inputs.py) and of the ranges around them.

Paths:
  exact         fps_exact, ball_query, gather_xyz between stages
  fastpoint     MDPS recording its radius tests, ball_query reading the record, gather_xyz between
                stages; from 16384 points per cloud the cell-ordered sampler with the scattered scan
                order, below that the index-ordered one (what bench.py runs)
  pruned        fps_exact_pruned, ball_query_grid, gather_xyz between stages
  upsample      knn: the k nearest samples of every point
  upsample_grid knn_grid, the search radius three times the samples' coverage radius
  lists         fp_excl_count and fp_excl_fill at the six MDPS thresholds and the query radius into
                buffers of a fixed capacity, ball_query_lists
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2507_23480_amd import binding as fp
from paper_2507_23480_amd import calibration, inputs

# scene: workload whose clouds and MDPS constants it has, its points per cloud and first radius there,
# dimension in which its points spread (radius and spacing go with N ** (-1 / dim))
SCENES = {"cube": ("C1", 4096, 0.1, 3), "object": ("C2", 1024, 0.2, 2), "room": ("C3", 24000, 0.1, 2),
          "lidar": ("C4", 120000, 1.0, 2), "clusters": ("C5", 1000000, 0.5, 3)}
PRUNED_FROM = 16384
# exclusion-list members per point over the seven levels when a quarter of a room's points is sampled
ROOM_LIST_MEMBERS = 156
LIST_CAPACITY = 400         # members per point a caller that does not read the total back makes room for
# blocks of 64 radius tests a LiDAR cloud's record has room for, per point (its balls near the sensor
# hold thousands of points); the other scenes take the library's default capacity
LIDAR_ENTRIES_PER_POINT = 10


def listed():
    case = lambda name, path, scene, B, N, n, k, stages, ratio: {  # noqa: E731
        "name": name, "path": path, "scene": scene, "B": B, "N": N, "n": n, "k": k, "stages": stages, "ratio": ratio}
    return [
        # one small cloud, alone: a robot's or an interactive user's single object; latency counts
        case("cube_exact", "exact", "cube", 1, 4096, 1024, 32, 1, 4),
        # object classification, two stages of a batch: the exact layer and FastPoint's
        case("objects_exact", "exact", "object", 16, 1024, 512, 32, 2, 4),
        case("objects_fastpoint", "fastpoint", "object", 16, 1024, 512, 32, 2, 4),
        # indoor segmentation, the encoder's four stages at a quarter each
        case("rooms_exact", "exact", "room", 8, 24000, 6000, 32, 4, 4),
        case("rooms_fastpoint", "fastpoint", "room", 8, 24000, 6000, 32, 4, 4),
        # the same layer on a few clouds of an odd size through the pruned sampler and the grid query
        case("rooms_ragged_pruned", "pruned", "room", 3, 30011, 7501, 24, 2, 4),
        # LiDAR sweeps: the largest batch
        case("lidar_exact", "exact", "lidar", 4, 120000, 16384, 16, 1, 4),
        case("lidar_fastpoint", "fastpoint", "lidar", 4, 120000, 16384, 16, 1, 4),
        # the decoder's up-sampling step of a LiDAR batch (three neighbours, as interpolation takes them)
        case("lidar_upsample", "upsample", "lidar", 4, 120000, 16384, 3, 1, 4),
        # a scanned site in one piece: the largest cloud
        case("clusters_exact", "exact", "clusters", 1, 1000000, 65536, 32, 1, 4),
        case("clusters_fastpoint", "fastpoint", "clusters", 1, 1000000, 65536, 32, 1, 4),
        # neighbour structure of a batch of rooms kept for several later queries
        case("rooms_lists", "lists", "room", 8, 24000, 6000, 32, 1, 4),
    ]


def draw(rng):
    path = rng.choice(["exact", "exact", "fastpoint", "fastpoint", "pruned", "upsample", "upsample_grid", "lists"])
    scene = "room" if path == "lists" else rng.choice(list(SCENES))
    lo, hi, most_b = {"cube": (1000, 16384, 4), "object": (512, 4096, 32), "room": (4000, 48000, 8),
                      "lidar": (20000, 120000, 4), "clusters": (60000, 1000000, 1)}[scene]
    if path == "lists":
        hi = 24000
    N = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    first = {"cube": 4, "object": 2, "room": 4, "lidar": 7, "clusters": 15}[scene]
    n = N // 4 if path == "lists" else max(64, int(N / (first * rng.uniform(0.7, 1.5))))
    stages = 1 if path in ("upsample", "upsample_grid", "lists") else rng.choice([1, 1, 2, 3])
    k = rng.choice([1, 3, 3, 5]) if path.startswith("upsample") else rng.choice([16, 24, 32, 48, 64])
    return {"path": path, "scene": scene, "B": rng.randint(1, most_b), "N": N, "n": n, "k": k, "stages": stages,
            "ratio": 4}


def _stages(case):
    """(points, samples, radius) of each stage: a later one keeps 1 / ratio of what reaches it, at twice the radius."""
    _, N0, r0, dim = SCENES[case["scene"]]
    N, n, r = case["N"], case["n"], r0 * (N0 / case["N"]) ** (1.0 / dim)
    out = []
    for _ in range(case["stages"]):
        out.append((N, n, r))
        N, n, r = n, max(1, n // case["ratio"]), 2.0 * r
    return out


def _lidar(B, N, seed):
    """Sweeps like those of inputs.py (64 rings x 4000 steps over a ground plane and 20 to 60 boxes, ring-major
    order, decimated to N), with the rays cast on the GPU."""
    rng = np.random.default_rng([20250723, seed])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dev = {"device": "cuda", "dtype": torch.float64}
    elev = torch.deg2rad(torch.linspace(-24.0, 2.0, 64, **dev))[:, None]
    az = (torch.arange(4000, **dev) * (2.0 * math.pi / 4000))[None, :]
    d = torch.stack([elev.cos() * az.cos(), elev.cos() * az.sin(), elev.sin().expand(64, 4000)], dim=2).reshape(-1, 3)
    origin = torch.tensor([0.0, 0.0, 1.7], **dev)
    clouds = []
    for _ in range(B):
        nbox = int(rng.integers(20, 61))
        foot, height = rng.uniform(1.0, 6.0, (nbox, 2)), rng.uniform(1.0, 4.0, nbox)
        ang, rad = rng.uniform(0.0, 2.0 * math.pi, nbox), rng.uniform(4.0, 48.0, nbox)
        cxy = np.stack([rad * np.cos(ang), rad * np.sin(ang)], axis=1)
        lo = torch.as_tensor(np.concatenate([cxy - 0.5 * foot, np.zeros((nbox, 1))], axis=1), **dev)
        hi = torch.as_tensor(np.concatenate([cxy + 0.5 * foot, height[:, None]], axis=1), **dev)
        t = torch.where(d[:, 2] < -1e-9, -origin[2] / d[:, 2], math.inf)
        inv = 1.0 / d
        for b in range(nbox):
            t0, t1 = (lo[b] - origin) * inv, (hi[b] - origin) * inv
            tn, tf = torch.minimum(t0, t1).nan_to_num(-math.inf).amax(1), torch.maximum(t0, t1).nan_to_num(math.inf).amin(1)
            t = torch.where((tn <= tf) & (tn > 0.0) & (tn < t), tn, t)
        t = t + 0.02 * torch.randn(t.shape, generator=gen, **dev)
        ok = torch.isfinite(t) & (t > 0.5) & (t <= 50.0)
        pts = origin + t[ok, None] * d[ok]
        keep = torch.randperm(pts.shape[0], generator=gen, device="cuda")[:N].sort().values
        if keep.numel() < N:
            raise RuntimeError("too few returns")
        clouds.append(pts[keep].float())
    return torch.stack(clouds).contiguous()


def _clouds(case, seed):
    if case["scene"] == "lidar":
        return _lidar(case["B"], case["N"], seed % (1 << 31))
    base = 10_000_000 + (seed % (1 << 31)) * 64         # clouds no workload and no calibration run draws
    name = SCENES[case["scene"]][0]
    return torch.from_numpy(np.stack([inputs.make_cloud(name, base + b, case["N"]) for b in range(case["B"])])).cuda()


def prepare(case, seed):
    name = SCENES[case["scene"]][0]
    xyz = _clouds(case, seed)
    state = {"case": case, "xyz": xyz, "stages": _stages(case)}
    if case["path"] == "fastpoint":
        known = len(inputs.WORKLOADS[name].stages)
        state["prm"], state["cache"] = [], []
        for s, (N, n, _) in enumerate(state["stages"]):
            prm = calibration.params_for(name, min(s, known - 1))
            state["prm"].append(dataclasses.replace(prm, scan_order=1) if N >= PRUNED_FROM else prm)
            entries = LIDAR_ENTRIES_PER_POINT * N if case["scene"] == "lidar" and s == 0 else 0
            shape = xyz if s == 0 else torch.empty((case["B"], N, 3), device="cuda")
            state["cache"].append(fp.new_bq_cache(shape, n, entries))
    elif case["path"].startswith("upsample"):
        state["samples"] = fp.fps_exact_pruned(xyz, case["n"])
        if case["path"] == "upsample_grid":
            state["radius"] = 3.0 * float(fp.coverage2(xyz, state["samples"]).max()) ** 0.5
    elif case["path"] == "lists":
        prm = calibration.params_for(name, 0)
        state["samples"], info = fp.mdps_sample(xyz, case["n"], prm, want_info=True)
        r2 = float(np.float32(state["stages"][0][2]) * np.float32(state["stages"][0][2]))
        state["thr2"] = torch.tensor([[i.thr2[j] for j in range(prm.nseg)] + [r2] for i in fp.parse_info(info)],
                                     dtype=torch.float32, device="cuda")
        B, N, L = case["B"], case["N"], prm.nseg + 1
        state["offsets"] = torch.empty(L * B * N + 1, dtype=torch.int64, device="cuda")
        state["entries"] = torch.zeros(LIST_CAPACITY * B * N, dtype=torch.int32, device="cuda")
        state["ws"] = torch.empty(fp.load().fp_excl_workspace_bytes(B, N, L), dtype=torch.uint8, device="cuda")
    return state


def _lists(state):
    """Both passes of the exclusion lists through the C ABI, nothing read back between them."""
    lib, x, thr2, ws = fp.load(), state["xyz"], state["thr2"], state["ws"]
    offsets, entries = state["offsets"], state["entries"]
    B, N, L = x.shape[0], x.shape[1], thr2.shape[1]
    stream = torch.cuda.current_stream().cuda_stream
    status = lib.fp_excl_count(x.data_ptr(), B, N, thr2.data_ptr(), L, offsets.data_ptr(), ws.data_ptr(), ws.numel(), stream)
    if status == 0:
        status = lib.fp_excl_fill(x.data_ptr(), B, N, thr2.data_ptr(), L, offsets.data_ptr(), entries.data_ptr(),
                                  entries.numel(), ws.data_ptr(), ws.numel(), stream)
    if status != 0:
        raise RuntimeError(lib.fp_status_string(status).decode())
    return offsets, entries


def run(state):
    case, x, k = state["case"], state["xyz"], state["case"]["k"]
    path = case["path"]
    if path == "upsample":
        return fp.knn(x, state["samples"], k)
    if path == "upsample_grid":
        return fp.knn_grid(x, state["samples"], k, state["radius"])
    if path == "lists":
        offsets, entries = _lists(state)
        L = state["thr2"].shape[1]
        return offsets, entries, fp.ball_query_lists(offsets, entries, case["B"], case["N"], L, L - 1, state["samples"], k)
    out = []
    for s, (N, n, r) in enumerate(state["stages"]):
        if path == "exact":
            idx = fp.fps_exact(x, n)
            out.append((idx, fp.ball_query(x, idx, r, k)))
        elif path == "pruned":
            idx = fp.fps_exact_pruned(x, n)
            out.append((idx, fp.ball_query_grid(x, idx, r, k)))
        else:
            sample = fp.mdps_sample_pruned if N >= PRUNED_FROM else fp.mdps_sample
            idx = sample(x, n, state["prm"][s], bq_cache=state["cache"][s], bq_radius=r)
            out.append((idx, fp.ball_query(x, idx, r, k, bq_cache=state["cache"][s])))
        if s + 1 < len(state["stages"]):
            x = fp.gather_xyz(x, idx)
            out.append(x)
    return out


def work(case):
    """Bytes: clouds and index lists read once, results written once.  Operations: a squared distance is eight.
    A point's nearest sample changes about ln n times over a run of farthest point sampling, so those
    distances have to be formed, and so has the distance of every neighbour that is returned."""
    B, N, n, k = case["B"], case["N"], case["n"], case["k"]
    if case["path"].startswith("upsample"):
        return {"bytes": B * (12.0 * N + 4.0 * n + 8.0 * N * k), "flops": 8.0 * B * N * k}
    if case["path"] == "lists":
        members = float(ROOM_LIST_MEMBERS) * B * N
        return {"bytes": 12.0 * B * N + 4.0 * members + 8.0 * 7 * B * N + 4.0 * B * n * (k + 2), "flops": 8.0 * members / 2}
    byts = flops = 0.0
    for s, (N, n, _) in enumerate(_stages(case)):
        byts += B * (12.0 * N + 4.0 * n + 4.0 * n * (k + 1) + (12.0 * n if s + 1 < case["stages"] else 0.0))
        flops += B * (8.0 * N * math.log(n + 1.0) + 8.0 * n * k)
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    """Indices, counts and offsets are whole numbers; the distances of the k-NN are defined operation by
    operation in binary32 and gathered coordinates are copies, so those come out bit for bit as well."""
    return "exact"
