"""The framework's workloads as measurable cases.

Each case is one pass through the package's public entry points (``ops`` for a
single call, ``nets`` for a network) on sizes of the networks in ``synth`` or
of the same kind.  The kinds:

  net           a whole network forward: eager calls, or the captured graph
                that a server replays
  fps           farthest-point sampling of one level
  ball_query    one level's neighbor table
  edgeconv      one DGCNN layer: kNN in feature space, the folded product on
                every point, the aggregation
  mlp           one shared MLP on [xyz | features] rows, fp32 or bf16,
                optionally max-pooled over groups of rows (group-all)
  conventional  one module in the original order: gather, MLP on every
                (centroid, neighbor) row, max
  aggregate     one delayed aggregation from an fp32 or bf16 feature table
  propagate     one feature-propagation level: 3-NN search, interpolation,
                MLP on [interpolated | skip] rows

Inputs come from the generators of ``synth``, seeded.  ``exact`` evaluates the
same function in 64 bits with plain torch; searches follow the documented
fp32 distance (so that they select the same points) and have no 64-bit value
of their own.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2008_06967_amd import nets, ops, synth
from paper_2008_06967_amd._lib import BF16, F32

DEV = "cuda"


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # one small module on one cloud: the latency of a single call chain
        dict(name="module_1cloud", kind="net", net="sa_module", B=1, N=1024, dtype="f32", graph=False),
        # the segmentation network as served: one captured batch of rooms
        dict(name="seg_net", kind="net", net="pointnet2_seg", B=16, N=4096, dtype="f32", graph=True),
        # the LiDAR backbone, bf16, called eagerly
        dict(name="lidar_net_bf16", kind="net", net="lidar", B=4, N=16384, dtype="bf16", graph=False),
        # the classifier's first sampling, a batch of objects
        dict(name="fps_objects", kind="fps", gen="mesh_surfaces", B=32, N=1024, M=512),
        # a sampling whose sizes fit no tile
        dict(name="fps_ragged", kind="fps", gen="indoor_room", B=3, N=5003, M=1251),
        # first-level neighbor tables of a batch of rooms
        dict(name="ball_query_rooms", kind="ball_query", gen="indoor_room", B=16, N=4096, M=1024, K=32, radius=0.1),
        # DGCNN's third layer
        dict(name="edgeconv_64_128", kind="edgeconv", B=16, N=1024, C=64, Cout=128, K=20),
        # the classifier's second module's MLP on its points
        dict(name="mlp_sa2", kind="mlp", B=32, N=512, cf=128, widths="128,128,256", dtype="f32", pool=False),
        # the classifier's group-all module
        dict(name="mlp_group_all", kind="mlp", B=32, N=128, cf=256, widths="256,512,1024", dtype="f32", pool=True),
        # the bf16 segmentation network's second module's MLP, on all points
        dict(name="mlp_bf16", kind="mlp", B=16, N=4096, cf=128, widths="128,128,256", dtype="bf16", pool=False),
        # the classifier's first module in the original order
        dict(name="conventional_sa1", kind="conventional", B=32, N=1024, M=512, K=32, radius=0.2, cf=0,
             widths="64,64,128"),
        # the finest feature-propagation level of the segmentation network
        dict(name="propagate_rooms", kind="propagate", B=16, N=4096, M=1024, C=128, cf=3, widths="128,128,128"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["net", "fps", "fps", "ball_query", "edgeconv", "mlp", "mlp", "conventional", "aggregate",
                       "propagate"])
    if kind == "net":
        net = rng.choice(["sa_module", "pointnet2_cls", "pointnet2_seg", "lidar"])
        B, N = {"sa_module": (_log(rng, 1, 8), _log(rng, 600, 2500)),
                "pointnet2_cls": (_log(rng, 1, 32), _log(rng, 600, 2500)),
                "pointnet2_seg": (_log(rng, 1, 16), _log(rng, 1500, 4096)),
                "lidar": (rng.randint(1, 4), _log(rng, 8192, 16384))}[net]
        return dict(kind=kind, net=net, B=B, N=N, dtype="bf16" if net == "lidar" else rng.choice(["f32", "bf16"]),
                    graph=rng.random() < 0.5)
    if kind == "fps":
        gen, N = rng.choice([("uniform_cube", _log(rng, 100, 30000)), ("mesh_surfaces", _log(rng, 500, 4096)),
                             ("indoor_room", _log(rng, 1000, 12000)), ("lidar_scene", _log(rng, 6000, 16384))])
        return dict(kind=kind, gen=gen, B=_log(rng, 1, 4 if N > 8192 else 32), N=N,
                    M=max(1, int(N * rng.choice([0.125, 0.25, 0.5]) * rng.uniform(0.8, 1.0))))
    if kind == "ball_query":
        N = _log(rng, 500, 16384)
        return dict(kind=kind, gen=rng.choice(["mesh_surfaces", "indoor_room"]), B=_log(rng, 1, 16), N=N,
                    M=max(1, N // rng.choice([2, 4])), K=rng.choice([16, 32, 64]), radius=rng.choice([0.1, 0.2, 0.4]))
    if kind == "edgeconv":
        C, Cout = rng.choice([(3, 64), (64, 64), (64, 128), (128, 256)])
        return dict(kind=kind, B=_log(rng, 1, 16), N=_log(rng, 256, 1024), C=C, Cout=Cout, K=rng.choice([10, 20, 40]))
    if kind == "mlp":
        pool = rng.random() < 0.25
        N = rng.choice([32, 64, 128]) if pool else _log(rng, 64, 4096)
        B = _log(rng, 1, 32) if pool else _log(rng, 1, max(1, min(32, 65536 // N)))
        widths = "256,512,1024" if pool else rng.choice(["32,32,64", "64,64,128", "128,128,256", "256,256,512",
                                                         "128,128,128"])
        return dict(kind=kind, B=B, N=N, cf=rng.choice([0, 3, 64, 128, 256]), widths=widths,
                    dtype=rng.choice(["f32", "bf16"]), pool=pool)
    if kind == "conventional":
        N = _log(rng, 256, 1024)
        return dict(kind=kind, B=_log(rng, 1, 16), N=N, M=N // rng.choice([2, 4]), K=rng.choice([16, 32]), radius=0.2,
                    cf=rng.choice([0, 64]), widths=rng.choice(["64,64,128", "128,128,256"]))
    if kind == "aggregate":
        N = _log(rng, 256, 16384)
        return dict(kind=kind, B=_log(rng, 1, max(1, min(32, 65536 // N))), N=N, M=N // rng.choice([2, 4]),
                    K=rng.choice([20, 32, 64]), C=rng.choice([64, 128, 256]), dtype=rng.choice(["f32", "bf16"]))
    N = _log(rng, 64, 4096)
    return dict(kind=kind, B=_log(rng, 1, 16), N=N, M=max(3, N // 4), C=rng.choice([128, 256]),
                cf=rng.choice([0, 3, 64, 128]), widths=rng.choice(["128,128,128", "256,128", "256,256"]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _np_rng(seed, stream):
    return np.random.default_rng(np.random.SeedSequence([int(seed), stream]))


def _cloud(gen, seed, B, N):
    g = _np_rng(seed, 0)
    if gen == "uniform_cube":
        x = synth.uniform_cube(g, B, N)
    elif gen == "mesh_surfaces":
        x = synth.mesh_surfaces(g, B, N)
    elif gen == "indoor_room":
        x = synth.indoor_room(g, B, N, n_feat=0)[0]
    else:
        x = synth.lidar_scene(g, B, N)
    return torch.from_numpy(x).to(DEV)


def _feat(seed, stream, *shape):
    """Features as they leave a ReLU layer: half of them zero."""
    t = torch.Generator(device=DEV).manual_seed(int(seed) * 16 + stream)
    return torch.randn(shape, generator=t, device=DEV).relu_()


def _layers(seed, dims):
    return synth.he_layers(_np_rng(seed, 2), _np_rng(seed, 3), dims)


def _widths(case):
    return [int(w) for w in case["widths"].split(",")]


def _spec(case):
    s = synth.workload(case["net"], B=case["B"], N=case["N"], dtype=case["dtype"])
    for m in s["sa"]:    # the levels keep their shares of the input points
        m["M"] = max(16, m["M"] * case["N"] // synth.WORKLOADS[case["net"]]["N"])
    return s


def _net_inputs(case, seed):
    spec = _spec(case)
    xyz = _cloud(spec["gen"], seed, case["B"], case["N"])
    feat = None
    if spec["n_feat"]:
        feat = torch.from_numpy(_np_rng(seed, 1).uniform(0.0, 1.0, (case["B"], case["N"], spec["n_feat"]))
                                .astype(np.float32)).to(DEV)
    return spec, xyz, feat, synth.make_weights(dict(spec, id=int(seed)))


def _table(seed, B, N, M, K):
    """A neighbor table with the locality of a search: centroid c and rows near it."""
    t = torch.Generator(device=DEV).manual_seed(int(seed) * 16 + 7)
    cidx = torch.argsort(torch.rand((B, N), generator=t, device=DEV), dim=1)[:, :M].to(torch.int32).contiguous()
    off = torch.randint(-2 * K, 2 * K + 1, (B, M, K), generator=t, device=DEV)
    return cidx, ((cidx[..., None] + off) % N).to(torch.int32).contiguous()


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case)
    if kind == "net":
        spec, xyz, feat, w = _net_inputs(case, seed)
        s.update(xyz=xyz, feat=feat, net=nets.build(spec, w, delayed=True, device=DEV), graph=None)
        if case["graph"]:
            s["graph"], s["out"] = s["net"].capture(xyz, feat)
        return s
    B, N = case["B"], case["N"]
    if kind == "fps":
        s["xyz"] = _cloud(case["gen"], seed, B, N)
        return s
    if kind == "ball_query":
        s["xyz"] = _cloud(case["gen"], seed, B, N)
        s["q"] = s["xyz"][:, : case["M"]].contiguous()
        return s
    if kind == "edgeconv":
        C, Cout = case["C"], case["Cout"]
        s["x"] = _cloud("mesh_surfaces", seed, B, N) if C == 3 else _feat(seed, 1, B, N, C)
        Ws, bs = _layers(seed, [2 * C, Cout])
        s["W"], s["b"] = torch.from_numpy(Ws[0]).to(DEV), torch.from_numpy(bs[0]).to(DEV)
        Wf, bf = ops.edgeconv_fold(s["W"], s["b"])
        s["p"] = ops.MLPParams([Wf], [bf], device=DEV)
        return s
    if kind == "aggregate":
        s["pft"] = _feat(seed, 1, B, N, case["C"])
        if case["dtype"] == "bf16":
            s["pft"] = s["pft"].to(torch.bfloat16)
        s["cidx"], s["nit"] = _table(seed, B, N, case["M"], case["K"])
        return s
    if kind == "mlp":
        s["xyz"] = _cloud("mesh_surfaces", seed, B, N)
        s["f"] = _feat(seed, 1, B, N, case["cf"]) if case["cf"] else None
        s["layers"] = _layers(seed, [3 + case["cf"]] + _widths(case))
        s["p"] = ops.MLPParams(*s["layers"], dtype=BF16 if case["dtype"] == "bf16" else F32, device=DEV)
        return s
    if kind == "conventional":
        s["xyz"] = _cloud("mesh_surfaces", seed, B, N)
        s["q"] = s["xyz"][:, : case["M"]].contiguous()
        s["f"] = _feat(seed, 1, B, N, case["cf"]) if case["cf"] else None
        s["nit"], _ = ops.ball_query(s["xyz"], s["q"], case["radius"], case["K"])
        s["layers"] = _layers(seed, [3 + case["cf"]] + _widths(case))
        s["p"] = ops.MLPParams(*s["layers"], device=DEV)
        return s
    s["xyz"] = _cloud("indoor_room", seed, B, N)                       # propagate
    s["src"] = s["xyz"][:, : case["M"]].contiguous()
    s["f"] = _feat(seed, 1, B, case["M"], case["C"])
    s["skip"] = _feat(seed, 4, B, N, case["cf"]) if case["cf"] else None
    s["layers"] = _layers(seed, [case["C"] + case["cf"]] + _widths(case))
    s["p"] = ops.MLPParams(*s["layers"], device=DEV)
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "net":
        if s["graph"] is not None:
            s["graph"].replay()
            out = s["out"]
        else:
            out = s["net"].forward(s["xyz"], s["feat"])
        return [out["out"], out["idx0"], out["nit0"]]
    if kind == "fps":
        return ops.fps(s["xyz"], case["M"])
    if kind == "ball_query":
        return ops.ball_query(s["xyz"], s["q"], case["radius"], case["K"])[0]
    if kind == "edgeconv":
        nit, _ = ops.knn(s["x"], s["x"], case["K"])
        P = ops.pointwise_mlp(s["x"], s["p"], relu_mask=0)
        c = case["Cout"]
        return [ops.aggregate_max(P[..., c:], nit, cfeat=P[..., :c], sign=+1, relu=True), nit]
    if kind == "aggregate":
        return ops.aggregate_max(s["pft"], s["nit"], cidx=s["cidx"])
    if kind == "mlp":
        return ops.pointwise_mlp(s["xyz"], s["p"], x1=s["f"], out_dtype=F32 if case["pool"] else s["p"].dtype,
                                 pool_group=case["N"] if case["pool"] else 0)
    if kind == "conventional":
        return ops.conventional_module(s["nit"], s["p"], xyz=s["xyz"], feat=s["f"], cxyz=s["q"])
    nit, dist = ops.three_nn(s["xyz"], s["src"])
    interp = ops.interpolate3_apply(nit, dist, s["f"])
    return [ops.pointwise_mlp(interp, s["p"], x1=s["skip"]), nit]


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _mlp_work(rows, dims, s):
    return (sum(a * b for a, b in zip(dims, dims[1:])) * s + rows * (dims[0] + dims[-1]) * s,
            2 * rows * sum(a * b for a, b in zip(dims, dims[1:])))


def _fps_work(B, N, M):
    return 12 * B * N + 16 * B * M, 8 * B * (N + M)


def _ball_work(B, N, M, K):
    return 12 * B * (N + M) + 4 * B * M * K, 8 * B * M * K


def work(case):
    kind = case["kind"]
    if kind == "net":
        spec = _spec(case)
        B, n, c, e = case["B"], case["N"], spec["n_feat"], 2 if case["dtype"] == "bf16" else 4
        # inputs and outputs once, weights once, the arithmetic of the MLPs
        by, fl = 12 * B * n + 4 * B * n * c, 0
        widths, sizes = [c], [n]
        for m in spec["sa"]:
            dims = [3 + c] + m["mlp"]
            fl += _mlp_work(B * n, dims, e)[1] + _fps_work(B, n, m["M"])[1] + B * m["M"] * m["K"] * m["mlp"][-1]
            by += sum(a * b for a, b in zip(dims, dims[1:])) * e
            n, c = m["M"], m["mlp"][-1]
            widths.append(c)
            sizes.append(n)
        by += 4 * B * spec["sa"][0]["M"] * (1 + spec["sa"][0]["K"])
        rest = []
        if spec.get("group_all"):
            rest.append((B * n, [3 + c] + spec["group_all"]))
            rest.append((B, spec["group_all"][-1:] + spec["fc"]))
        for i, d in enumerate(spec.get("fp", [])):
            rest.append((B * sizes[-2 - i], [c + widths[-2 - i]] + d))
            c = d[-1]
        if spec.get("head"):
            rest.append((B * sizes[0], [c] + spec["head"]))
        for rows, dims in rest:
            fl += _mlp_work(rows, dims, e)[1]
            by += sum(a * b for a, b in zip(dims, dims[1:])) * e
        out = rest[-1][0] * rest[-1][1][-1] if rest else B * n * c
        return {"bytes": by + 4 * out, "flops": fl}
    B, N = case["B"], case["N"]
    if kind == "fps":
        by, fl = _fps_work(B, N, case["M"])
    elif kind == "ball_query":
        by, fl = _ball_work(B, N, case["M"], case["K"])
    elif kind == "edgeconv":
        C, Co, K = case["C"], case["Cout"], case["K"]
        by = 4 * B * N * (C + Co + K) + 4 * 2 * C * Co
        fl = B * N * (2 * C * N + 4 * C * Co + K * Co)
    elif kind == "aggregate":
        C, M, K = case["C"], case["M"], case["K"]
        by = B * N * C * (2 if case["dtype"] == "bf16" else 4) + 4 * B * M * (K + 1 + C)
        fl = B * M * K * C
    elif kind == "mlp":
        dims, s = [3 + case["cf"]] + _widths(case), 2 if case["dtype"] == "bf16" else 4
        fl = _mlp_work(B * N, dims, s)[1]
        by = sum(a * b for a, b in zip(dims, dims[1:])) * s + 4 * B * N * dims[0]
        by += 4 * B * dims[-1] if case["pool"] else s * B * N * dims[-1]
    elif kind == "conventional":
        dims, M, K = [3 + case["cf"]] + _widths(case), case["M"], case["K"]
        by = 4 * B * (N * dims[0] + 3 * M + M * K + M * dims[-1]) + 4 * sum(a * b for a, b in zip(dims, dims[1:]))
        fl = _mlp_work(B * M * K, dims, 4)[1]
    else:
        C, M, dims = case["C"], case["M"], [case["C"] + case["cf"]] + _widths(case)
        by = 4 * B * (N * (3 + case["cf"] + 3 + dims[-1]) + M * (3 + C)) + 4 * sum(a * b for a, b in zip(dims, dims[1:]))
        fl = _mlp_work(B * N, dims, 4)[1] + 8 * B * N * 3 + 6 * B * N * C
    return {"bytes": by, "flops": fl}


def tolerance(case):
    kind = case["kind"]
    if kind in ("fps", "ball_query", "aggregate"):
        return "exact"     # selections, and a maximum followed by one fp32 subtraction
    if case.get("dtype") == "bf16":
        # every stored activation is rounded to 8 bits of mantissa: another
        # order of the fp32 sums flips some roundings (against fp64 sums with
        # the same roundings: one MLP 1e-4 / max 0.013, whole networks
        # 2e-3 to 6.5e-3 / max 0.07)
        return {"rel": 2.5e-2, "max": 0.3, "differ": 0.0} if kind == "net" else {"rel": 1e-3, "max": 0.06, "differ": 0.0}
    if kind == "net":
        return {"rel": 1e-5, "max": 2e-4, "differ": 0.0}
    return {"rel": 4e-6, "max": 1e-4, "differ": 0.0}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _d(t):
    return None if t is None else t.double()


def _dist(a, b):
    """The documented fp32 distance: t = a - b, d = fma(t, t, d) per channel.
    (A product of two fp32 values is exact in fp64.)"""
    d = None
    for c in range(a.shape[-1]):
        t = (a[..., c] - b[..., c]).double()
        d = (t * t if d is None else t * t + d.double()).float()
    return d


def _fps_ref(xyz, M):
    B, N, _ = xyz.shape
    dm = torch.full((B, N), math.inf, device=xyz.device)
    idx = torch.zeros((B, M), dtype=torch.int64, device=xyz.device)
    row = torch.arange(B, device=xyz.device)
    ids = torch.arange(N, device=xyz.device)
    cur = idx[:, 0]
    for m in range(1, M):
        dm = torch.minimum(dm, _dist(xyz, xyz[row, cur][:, None]))
        top = dm.max(1, keepdim=True).values
        cur = torch.where(dm == top, ids, N).min(1).values      # the lowest index of a tie
        idx[:, m] = cur
    return idx


def _rows(x, idx):
    """x [B, N, C], idx [B, ...] -> x's rows."""
    B = x.shape[0]
    flat = idx.reshape(B, -1).long()
    return torch.gather(x, 1, flat[..., None].expand(-1, -1, x.shape[-1])).reshape(tuple(idx.shape) + (x.shape[-1],))


def _ball_ref(xyz, q, r, K):
    B, N, _ = xyz.shape
    r2 = float(np.float32(r) * np.float32(r))
    ids = torch.arange(N, device=xyz.device, dtype=torch.int32)
    out = []
    step = max(1, (1 << 26) // (B * N))
    for m in range(0, q.shape[1], step):
        hit = _dist(q[:, m:m + step, None], xyz[:, None]) < r2
        key = torch.where(hit, ids, N)
        k = min(K, N)
        first = torch.topk(key, k, dim=-1, largest=False, sorted=True).values
        if k < K:
            first = torch.nn.functional.pad(first, (0, K - k), value=N)
        one = torch.where(first[..., :1] == N, 0, first[..., :1])
        out.append(torch.where(first == N, one, first))
    return torch.cat(out, 1)


def _nearest(ref, q, K):
    out = []
    step = max(1, (1 << 25) // (ref.shape[0] * ref.shape[1]))
    for m in range(0, q.shape[1], step):
        d = _dist(q[:, m:m + step, None], ref[:, None])
        v, i = torch.sort(d, dim=-1, stable=True)
        out.append((v[..., :K], i[..., :K]))
    return torch.cat([v for v, _ in out], 1), torch.cat([i for _, i in out], 1)


def _mlp64(x, Ws, bs, last_relu=True):
    x = x.double()
    for l, (W, b) in enumerate(zip(Ws, bs)):
        x = x @ torch.as_tensor(W).to(DEV).double().t() + torch.as_tensor(b).to(DEV).double()
        if last_relu or l + 1 < len(Ws):
            x = x.relu()
    return x


def _cat(*ts):
    return torch.cat([t.double() for t in ts if t is not None], -1)


def _aggregate64(pft, nit, cidx):
    out = torch.empty(nit.shape[:2] + pft.shape[-1:], dtype=torch.float64, device=pft.device)
    step = max(1, (1 << 27) // (pft.shape[0] * nit.shape[2] * pft.shape[-1]))
    for m in range(0, nit.shape[1], step):
        out[:, m:m + step] = _rows(pft, nit[:, m:m + step]).amax(2)
    return out - _rows(pft, cidx)


def _interp64(dst, src, f):
    v, i = _nearest(src, dst, 3)
    w = 1.0 / v.double().clamp_min(1e-10)
    w = w / w.sum(-1, keepdim=True)
    return (_rows(f, i) * w[..., None]).sum(2)


def _net64(case, seed):
    spec, xyz, feat, w = _net_inputs(case, seed)
    p, f = xyz, _d(feat)
    levels = [(p, f)]
    for m, (Ws, bs) in zip(spec["sa"], w["sa"]):
        idx = _fps_ref(p, m["M"])
        c = _rows(p, idx)
        nit = _ball_ref(p, c, m["radius"], m["K"])
        f = _aggregate64(_mlp64(_cat(p, f), Ws, bs), nit, idx)
        p = c
        levels.append((p, f))
    if spec.get("group_all"):
        f = _mlp64(_cat(p, f), *w["group_all"]).amax(1)
        f = _mlp64(f, *w["fc"], last_relu=False)
    for i, (Ws, bs) in enumerate(w.get("fp", [])):
        fine, skip = levels[len(levels) - 2 - i]
        f = _mlp64(_cat(_interp64(fine, p, f), skip), Ws, bs)
        p = fine
    if "head" in w:
        f = _mlp64(f, *w["head"], last_relu=False)
    return [f, None, None]


def exact(case, seed):
    kind = case["kind"]
    if kind == "net":
        return _net64(case, seed)
    if kind in ("fps", "ball_query"):
        return None
    s = prepare(case, seed)
    if kind == "edgeconv":
        _, nit = _nearest(s["x"], s["x"], case["K"])
        C = case["C"]
        W, x = s["W"].double(), s["x"].double()
        own = x @ (W[:, :C] - W[:, C:]).t() + s["b"].double()
        far = x @ W[:, C:].t()
        return [(own + _rows(far, nit).amax(2)).relu(), None]
    if kind == "aggregate":
        return _aggregate64(s["pft"].double(), s["nit"], s["cidx"])
    if kind == "mlp":
        y = _mlp64(_cat(s["xyz"], s["f"]), *s["layers"])
        return y.amax(1) if case["pool"] else y
    if kind == "conventional":
        out, step = [], max(1, (1 << 24) // (case["N"] * case["K"]))
        for b in range(0, case["B"], step):
            nit = s["nit"][b:b + step]
            rel = _rows(s["xyz"][b:b + step].double(), nit) - s["q"][b:b + step, :, None].double()
            f = None if s["f"] is None else _rows(s["f"][b:b + step].double(), nit)
            out.append(_mlp64(_cat(rel, f), *s["layers"]).amax(2))
        return torch.cat(out)
    y = _interp64(s["xyz"], s["src"], s["f"].double())
    return [_mlp64(_cat(y, s["skip"]), *s["layers"]), None]
