"""Performance cases of the framework: what a training or inference program on
the library does, through its public entry points.

A program samples nodes, gathers their rows, builds the radius graph, runs
edge-conditioned layers forward and backward (packing the weights each step,
since an optimiser has changed them), or whole hop-loop training steps, or
sub-domain inference.  Every case is one of those calls, at the sizes of the
repository's workloads and their neighbours: 2-D squares of about a thousand to
tens of thousands of nodes without a cap, a 2-D mesh crowded toward a wall with
a cap of 32, 3-D channels of about 1e5 to 2.6e5 nodes with a cap of 24 and halo
rows; float32 layers of width 32 and 64, bf16 layers of width 32, 64 and 128.

Inputs are drawn on the GPU from the seed alone.  Node order is what sampling
gives: ascending lattice index for the squares and channels (neighbours in
space are near in memory), no order for the mesh around a wall.
"""

import math

import numpy as np
import torch

import paper_2402_15106_amd as dm

# (d, h1, h2) of the layer shapes, by width; the types each is used in.
WIDTHS = {32: (32, 64, 64), 64: (64, 128, 128), 128: (128, 256, 256)}


def listed():
    return [
        # the smallest call: 1,024 of a 64 x 64 grid's nodes and their rows (latency)
        dict(name="sample-1k", kind="sample", M=4096, s=1024, dim=2, d=32, dtype="f32"),
        # one GPU's slab of a large 3-D channel: 262,144 of 764,077 candidates
        dict(name="sample-262k", kind="sample", M=764077, s=262144, dim=3, d=128, dtype="bf16"),
        # graph of a small 2-D square, every neighbour kept (latency)
        dict(name="graph-1k", kind="graph", geo="square", n=1024, halo=0, deg=20.6, cap=0, mode="knn"),
        # graph of an airfoil-like mesh: nodes crowded toward a wall, 32 nearest kept
        dict(name="graph-33k", kind="graph", geo="wall", n=32768, halo=0, deg=0.0, cap=32, mode="knn"),
        # graph of a channel slab with halo rows, 24 nearest kept of about 90
        dict(name="graph-286k", kind="graph", geo="channel", n=262144, halo=23420, length=2.74, deg=94.0, cap=24,
             mode="knn"),
        # one float32 layer of a small square, forward and backward
        dict(name="layer-f32-1k", kind="layer", geo="square", n=1024, halo=0, deg=20.6, cap=0, mode="knn", dtype="f32",
             d=32, act="identity", residual=True, attr="concat", backward=True),
        # one bf16 layer of a 2-D square at mean degree 40, forward and backward
        dict(name="layer-8k", kind="layer", geo="square", n=8192, halo=0, deg=41.2, cap=0, mode="knn", dtype="bf16",
             d=64, act="identity", residual=True, attr="concat", backward=True),
        # one bf16 layer on the airfoil-like mesh, forward only (evaluation), an odd node count
        dict(name="layer-fwd-30k", kind="layer", geo="wall", n=30011, halo=0, deg=0.0, cap=32, mode="knn", dtype="bf16",
             d=64, act="identity", residual=True, attr="concat", backward=False),
        # one bf16 layer of a long 3-D channel at mean degree about 11, forward and backward
        dict(name="layer-100k", kind="layer", geo="channel", n=100000, halo=0, length=9.5, deg=9.5, cap=24, mode="knn",
             dtype="bf16", d=64, act="identity", residual=True, attr="concat", backward=True),
        # the largest: one bf16 layer of width 128 on a channel slab with halo rows, forward and backward
        dict(name="layer-262k", kind="layer", geo="channel", n=262144, halo=23420, length=2.74, deg=94.0, cap=24,
             mode="knn", dtype="bf16", d=128, act="identity", residual=True, attr="concat", backward=True),
        # a whole hop-loop training step (encoder, four hops of layer and decoder, loss, backward)
        dict(name="hop-8k", kind="hop", geo="square", n=8192, halo=0, deg=41.2, cap=0, mode="knn", dtype="bf16", d=64,
             hid=64, hops=4),
        # sub-domain inference: four boxes with overlap, four layers each, outputs put back
        dict(name="infer-8k", kind="infer", geo="square", n=8192, halo=0, deg=41.2, cap=0, mode="knn", dtype="bf16",
             d=64, layers=4, cuts=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_geometry(rng, n, halo=True, wall=True):
    geo = rng.choice(["square", "wall", "channel"] if wall else ["square", "channel"])
    if geo == "wall":
        return dict(geo=geo, n=n, halo=0, deg=0.0, cap=rng.choice([16, 24, 32]), mode=rng.choice(["knn", "knn", "random"]))
    # about half keep every neighbour (a mean degree of 8 to 48), the others have a cap
    if rng.random() < 0.5:
        out = dict(geo=geo, n=n, deg=round(rng.uniform(10.0, 44.0), 1), cap=0, mode="knn")
    else:
        out = dict(geo=geo, n=n, deg=round(rng.uniform(20.0, 95.0), 1), cap=rng.choice([12, 16, 24, 32]),
                   mode=rng.choice(["knn", "knn", "random"]))
    if geo == "channel":
        out["length"] = round(rng.uniform(2.0, 10.0), 2)
    out["halo"] = int(n * rng.uniform(0.02, 0.15)) if halo and geo == "channel" and rng.random() < 0.5 else 0
    return out


def draw(rng):
    kind = rng.choice(["sample", "graph", "graph", "layer", "layer", "layer", "layer", "hop", "infer"])
    if kind == "sample":
        d, dtype = rng.choice([(32, "f32"), (64, "f32"), (64, "bf16"), (128, "bf16")])
        M = _log_int(rng, 3000, 764077)
        return dict(kind=kind, M=M, s=max(1, int(M * rng.uniform(0.08, 0.6))), dim=rng.choice([2, 3]), d=d, dtype=dtype)
    if kind == "graph":
        return dict(kind=kind, **_draw_geometry(rng, _log_int(rng, 700, 240000)))
    if kind == "layer":
        d, dtype, most = rng.choice([(32, "f32", 60000), (64, "f32", 16000), (32, "bf16", 100000), (64, "bf16", 100000),
                                     (64, "bf16", 100000), (128, "bf16", 130000)])
        # a ReLU after the layer in forward passes only: backward, the decisions near
        # its kink that either rounding may take move a bf16 gradient by 4 %
        backward = rng.random() < 0.75
        return dict(kind=kind, **_draw_geometry(rng, _log_int(rng, 700, most)), dtype=dtype, d=d,
                    act="identity" if backward else rng.choice(["identity", "relu"]), residual=rng.random() < 0.8,
                    attr=rng.choice(["concat", "concat", "diff"]), backward=backward)
    d, dtype = rng.choice([(32, "f32"), (64, "bf16"), (64, "bf16"), (128, "bf16")])
    if kind == "hop":
        # not around a wall: there the gradients of several bf16 hops cancel to where
        # their rounding is 6 % of them
        return dict(kind=kind, **_draw_geometry(rng, _log_int(rng, 900, 12000), halo=False, wall=False), dtype=dtype,
                    d=d, hid=rng.choice([32, 64, 64]), hops=rng.choice([1, 2, 3, 4]))
    g = _draw_geometry(rng, _log_int(rng, 2000, 20000), halo=False)
    g["mode"] = "knn"
    return dict(kind=kind, **g, dtype=dtype, d=d, layers=rng.choice([2, 4]), cuts=rng.choice([1, 2]))


# ---------------------------------------------------------------- inputs

_LIB = []


def _lib():
    """The program's one handle."""
    if not _LIB:
        _LIB.append(dm.Dsmp(0))
    return _LIB[0]


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 12345)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _dim(case):
    return 3 if case["geo"] == "channel" else 2


def _points(case, g):
    """(positions [n_src, dim], node scalar [n_src]) in float64, owned rows
    first, and the radius."""
    n, n_src = case["n"], case["n"] + case["halo"]
    if case["geo"] == "square":
        # a sampled m x m grid of the unit square holding eight times the nodes
        # (four for small ones), in lattice order
        m = int(math.ceil(math.sqrt((4 if n <= 2048 else 8) * n_src)))
        pick = torch.randperm(m * m, generator=g, device="cuda")[:n_src].sort().values
        P = torch.stack([pick // m, pick % m], 1).double() / (m - 1)
        k = _rand(g, 4, 2) * 12.0 - 6.0
        ph = _rand(g, 4) * 2 * math.pi
        s = torch.exp(torch.sin(P @ k.T + ph).sum(1) * 0.7)
        return P, s, math.sqrt(case["deg"] / (math.pi * n_src))
    if case["geo"] == "wall":
        # nodes around a thin unit body, no order: nearly half with density falling as
        # 1 / (0.01 + distance) on both sides of it, the others spread around it (the
        # neighbour counts of the airfoil mesh: mean 78, an eighth above 256, at most ~400)
        u, c, t = _rand(g, n_src), _rand(g, n_src), _rand(g, n_src) * 2 * math.pi
        w = 0.01 * (torch.pow(torch.full_like(u, 1.0 + 1.5 / 0.01), u) - 1.0)
        side = torch.sign(torch.sin(t))
        near = torch.stack([c + 0.3 * w * torch.cos(t), side * (0.12 * torch.sqrt(c * (1 - c)) + w)], 1)
        wf = 2.0 * _rand(g, n_src)
        far = torch.stack([0.5 + (0.5 + wf) * torch.cos(t), (0.1 + wf) * torch.sin(t)], 1)
        out = _rand(g, n_src) < 0.55
        return torch.where(out[:, None], far, near), torch.where(out, wf, w), 0.05 * math.sqrt(32768.0 / n_src)
    # channel: a lattice of length x 1 x 1 refined four times near its walls,
    # holding about three times the nodes, in lattice order
    length = case["length"]
    m = int(math.ceil((3.0 * n_src / (0.52 * length)) ** (1.0 / 3.0))) + 1
    nx = int(math.ceil(length * m))
    lat = torch.arange(nx * m * m, device="cuda")
    y, z = ((lat // m) % m).double() / (m - 1), (lat % m).double() / (m - 1)
    wd = torch.minimum(torch.minimum(y, 1 - y), torch.minimum(z, 1 - z))
    keep = (wd < 0.1) | (_rand(g, lat.numel()) < 0.25)
    lat = lat[keep]
    lat = lat[torch.randperm(lat.numel(), generator=g, device="cuda")[:n_src]].sort().values
    if case["halo"]:   # strips at both ends are halo rows, after the owned ones
        a = case["halo"] // 2
        lat = torch.cat([lat[a:a + n], lat[:a], lat[a + n:]])
    P = torch.stack([lat // (m * m), (lat // m) % m, lat % m], 1).double() / (m - 1)
    wd = torch.minimum(torch.minimum(P[:, 1], 1 - P[:, 1]), torch.minimum(P[:, 2], 1 - P[:, 2]))
    return P, wd, (case["deg"] * length / (n_src * 4.0 / 3.0 * math.pi)) ** (1.0 / 3.0)


def _mode(case):
    return dm.CAP_RANDOM if case["mode"] == "random" else dm.CAP_KNN


def _uniform(g, shape, fan_in):
    return ((2 * _rand(g, *shape) - 1) / math.sqrt(fan_in)).float()


def _layer_params(g, d, de, h1, h2, dtype):
    P = {"W1": _uniform(g, (h1, de), de), "b1": _uniform(g, (h1,), de),
         "W2": _uniform(g, (h2, h1), h1), "b2": _uniform(g, (h2,), h1),
         "W3": _uniform(g, (d * d, h2), h2), "b3": _uniform(g, (d * d,), h2),
         "Wr": _uniform(g, (d, d), d), "br": _uniform(g, (d,), d)}
    if dtype == "bf16":   # the operands a bf16 layer takes in bfloat16
        for k in ("W2", "W3", "b3", "Wr"):
            P[k] = P[k].bfloat16().float()
    return P


def _mlp_params(g, d_in, hid, d_out):
    return {"W1": _uniform(g, (hid, d_in), d_in), "b1": _uniform(g, (hid,), d_in),
            "W2": _uniform(g, (hid, hid), hid), "b2": _uniform(g, (hid,), hid),
            "W3": _uniform(g, (d_out, hid), hid), "b3": _uniform(g, (d_out,), hid)}


def _nodes(case, seed):
    """Everything a program holds about its nodes: positions, attribute rows,
    features (a linear lift of the attributes), the radius, the generator."""
    g = _gen(seed)
    P, s, r = _points(case, g)
    pos = P.float().contiguous()
    attr = torch.cat([pos, s.float()[:, None]], 1).contiguous()
    h = None
    if "d" in case:
        c = attr.shape[1]
        h = (attr @ _uniform(g, (c, case["d"]), c) + _uniform(g, (case["d"],), c))
        h = (h.bfloat16() if case["dtype"] == "bf16" else h).contiguous()
    return g, pos, attr, h, r


def _desc(case, attr_mode, act="identity", residual=True):
    d, h1, h2 = WIDTHS[case["d"]]
    return dm.layer_desc(_dim(case), d, h1, h2, dm.BF16 if case["dtype"] == "bf16" else dm.F32,
                         dm.ACT_RELU if act == "relu" else dm.ACT_IDENTITY, int(residual),
                         dm.ATTR_DIFF if attr_mode == "diff" else dm.ATTR_CONCAT)


def prepare(case, seed):
    lib = _lib()
    st = dict(case=case, lib=lib)
    kind = case["kind"]
    if kind == "sample":
        g = _gen(seed)
        M, s = case["M"], case["s"]
        tdt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        st["pos"] = torch.rand(M, case["dim"], generator=g, device="cuda")
        st["attr"] = torch.rand(M, case["dim"] + 1, generator=g, device="cuda")
        st["h"] = torch.randn(M, case["d"], generator=g, device="cuda").to(tdt)
        st["key"] = int(seed) * 1000003 + 4001
        st["idx"] = torch.empty(s, dtype=torch.int32, device="cuda")
        st["out"] = [torch.empty(s, *st[k].shape[1:], dtype=st[k].dtype, device="cuda") for k in ("pos", "attr", "h")]
        return st
    g, pos, attr, h, r = _nodes(case, seed)
    n = case["n"]
    st.update(pos=pos, attr=attr, h=h, r=r, gseed=int(seed) + 17)
    if kind == "graph":
        # buffers for the graph of every step's nodes, sized once with room to spare
        cap = n * case["cap"] if case["cap"] else 2 * _edges(case)
        i32 = dict(dtype=torch.int32, device="cuda")
        st["graph"] = dm.Graph(n, pos.shape[0], 0, torch.zeros(n + 1, **i32), torch.zeros(cap, **i32),
                               torch.zeros(cap, **i32), torch.zeros(pos.shape[0] + 1, **i32), torch.zeros(cap, **i32))
        return st
    if kind == "infer":
        d, h1, h2 = WIDTHS[case["d"]]
        desc = _desc(case, "concat")
        de = 2 * _dim(case) + 2
        st["params"] = [_layer_params(g, d, de, h1, h2, case["dtype"]) for _ in range(case["layers"])]
        packed = [lib.dsmp_nnconv_pack(desc, P) for P in st["params"]]
        st["boxes"] = _boxes(case, pos)
        st["net"] = dm.SubdomainInference(lib, desc, packed, r, case["cap"], _mode(case), st["gseed"])
        return st
    st["graph"] = lib.dsmp_radius_graph_build(pos, n, r, case["cap"], _mode(case), st["gseed"])
    d, h1, h2 = WIDTHS[case["d"]]
    dim = _dim(case)
    if kind == "hop":
        c = dim + 1
        st["enc"], st["dec"] = _mlp_params(g, c, case["hid"], d), _mlp_params(g, d, case["hid"], c)
        st["conv"] = _layer_params(g, d, c, h1, h2, case["dtype"])
        st["Y"] = torch.randn(n, c, generator=g, device="cuda")
        st["mask"] = (torch.rand(n, generator=g, device="cuda") < 0.9).to(torch.uint8)
        st["step"] = dm.HopStep(lib, st["graph"], dm.HopShapes(
            n=n, dim=dim, d=d, h1=h1, h2=h2, hid_enc=case["hid"], hid_dec=case["hid"],
            dtype=dm.BF16 if case["dtype"] == "bf16" else dm.F32, hops=case["hops"]))
        st["packed"] = lib.dsmp_nnconv_pack(st["step"].conv, st["conv"])
        return st
    desc = st["desc"] = _desc(case, case["attr"], case["act"], case["residual"])
    de = 2 * dim + 2 if case["attr"] == "concat" else dim + 1
    st["params"] = _layer_params(g, d, de, h1, h2, case["dtype"])
    st["packed"] = lib.dsmp_nnconv_pack(desc, st["params"])
    sb, _, _ = lib.dsmp_nnconv_workspace(desc, st["graph"])
    st["saved"] = torch.empty(max(sb, 256), dtype=torch.uint8, device="cuda")
    st["out"] = torch.empty(n, d, device="cuda")
    if case["backward"]:
        f32 = dict(dtype=torch.float32, device="cuda")
        st["G"] = torch.randn(n, d, generator=g, device="cuda")
        st["grad_h"] = torch.empty(pos.shape[0], d, **f32)
        st["grads"] = {"d" + k: torch.empty_like(v) for k, v in st["params"].items()}
    return st


def _boxes(case, pos):
    """Boxes that tile space: `cuts` cuts per axis (3-D: along the channel only)."""
    dim, cuts = pos.shape[1], case["cuts"]
    lo, hi = pos.min(0).values.tolist(), pos.max(0).values.tolist()
    edges = []
    for a in range(dim):
        k = cuts if dim == 2 or a == 0 else 0
        edges.append([-math.inf] + [float(np.float32(lo[a] + (hi[a] - lo[a]) * (i + 1 + 0.07 * (a + 1)) / (k + 1.2)))
                                    for i in range(k)] + [math.inf])
    return [([edges[a][c[a]] for a in range(dim)], [edges[a][c[a] + 1] for a in range(dim)])
            for c in np.ndindex(*[len(e) - 1 for e in edges])]


def run(st):
    case, lib = st["case"], st["lib"]
    kind = case["kind"]
    if kind == "sample":
        idx = lib.dsmp_sample_nodes(case["M"], case["s"], st["key"], out=st["idx"])
        return [idx] + [lib.dsmp_gather_rows(st[k], idx, out=o) for k, o in zip(("pos", "attr", "h"), st["out"])]
    if kind == "graph":
        g = st["graph"]
        lib.dsmp_radius_graph_build(st["pos"], case["n"], st["r"], case["cap"], _mode(case), st["gseed"],
                                    capacity=g.col.numel(), out=g)
        return [g.n_edges, g.row_ptr, g.col, g.dst, g.csc_ptr, g.csc_eid]
    if kind == "infer":
        return st["net"].run(st["pos"], st["attr"], st["h"], st["boxes"], st["r"])
    if kind == "hop":
        hs = st["step"]
        lib.dsmp_nnconv_pack(hs.conv, st["conv"], out=st["packed"])
        loss, grads = hs.step(st["enc"], st["packed"], st["dec"], st["attr"], st["Y"], st["mask"])
        return {"loss": loss, "v": hs.v[case["hops"] - 1], **{k: grads[k] for k in ("enc", "conv", "dec")}}
    lib.dsmp_nnconv_pack(st["desc"], st["params"], out=st["packed"])
    lib.dsmp_nnconv_forward(st["desc"], st["packed"], st["graph"], st["attr"], st["h"], h_out=st["out"],
                            saved=st["saved"])
    if not case["backward"]:
        return {"out": st["out"]}
    lib.dsmp_nnconv_backward(st["desc"], st["packed"], st["graph"], st["attr"], st["h"], st["saved"], st["G"],
                             grad_h=st["grad_h"], grads=st["grads"])
    return {"out": st["out"], "grad_h": st["grad_h"], **st["grads"]}


# ---------------------------------------------------------------- work and tolerance

def _edges(case):
    """About how many edges the case's graph has: the mean degree less what a
    boundary cuts off, under the cap."""
    if case["geo"] == "wall":
        return int(case["n"] * 0.7 * case["cap"])
    d = case["deg"] * (0.93 if case["geo"] == "square" else 1.0)
    return int(case["n"] * (min(d, case["cap"]) if case["cap"] else d))


def _layer_work(n, n_src, E, dim, d, h1, h2, de, esz, backward):
    """Flops of eq. (1) with the sum over a node's edges taken before the
    product with W3 (fewer than one product per edge), and its inputs and
    outputs moved once."""
    params = 4 * (h1 * de + h1 + h2 * h1 + h2 + d * d * (h2 + 1) + d * d + d)
    kt = (h2 + 1) * d
    by = params + n_src * (4 * (dim + 1) + d * esz) + 8 * E + 4 * n + 4 * n * d
    fl = 2 * E * (de * h1 + h1 * h2) + 2 * E * kt + 2 * n * kt * d + 2 * n * d * d
    if backward:
        by += params + 4 * n * d + 4 * n_src * d + 4 * E + 4 * n_src
        fl += 4 * n * kt * d + 4 * E * kt + 4 * E * h1 * h2 + 2 * E * de * h1 + 4 * n * d * d
    return by, fl


def work(case):
    kind = case["kind"]
    if kind == "sample":
        row = 4 * case["dim"] + 4 * (case["dim"] + 1) + case["d"] * (2 if case["dtype"] == "bf16" else 4)
        return {"bytes": case["s"] * (2 * row + 4), "flops": 0}
    n, n_src, E, dim = case["n"], case["n"] + case["halo"], _edges(case), _dim(case)
    if kind == "graph":
        return {"bytes": 4 * dim * n_src + 12 * E + 4 * (n + 1) + 4 * (n_src + 1), "flops": 0}
    d, h1, h2 = WIDTHS[case["d"]]
    esz = 2 if case["dtype"] == "bf16" else 4
    if kind == "layer":
        de = 2 * dim + 2 if case["attr"] == "concat" else dim + 1
        by, fl = _layer_work(n, n_src, E, dim, d, h1, h2, de, esz, case["backward"])
    elif kind == "hop":
        c, hid, hops = dim + 1, case["hid"], case["hops"]
        by, fl = _layer_work(n, n, E, dim, d, h1, h2, c, esz, True)
        mlp = 2 * n * (c * hid + hid * hid + hid * d)
        by, fl = by * hops + 3 * 4 * n * c, fl * hops + 3 * mlp * (hops + 1)
    else:
        by, fl = _layer_work(n, n, E, dim, d, h1, h2, 2 * dim + 2, esz, False)
        by, fl = by * case["layers"] + 4 * n * (2 * dim + 1), fl * case["layers"]
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # sampling, gathers and graphs are whole numbers and copied rows
    if case["kind"] in ("sample", "graph"):
        return "exact"
    # bf16: about four times what the per-edge form of the layer (the same sums
    # in another order, other intermediates rounded) differs by from the aggregate
    # form: 2e-3 to 4e-3 of a gradient, single values 5e-2 to 1e-1 where a ReLU
    # decision near its kink goes the other way; either is up to 3e-2 from 64 bits
    if case["dtype"] == "bf16":
        return {"rel": 0.02, "max": 0.4}
    # float32: 4e-7 for the sums; a decision near a kink moves a gradient by up
    # to 3e-4 over a hop loop (against 64 bits), less in one layer
    if case["kind"] == "hop":
        return {"rel": 1e-3, "max": 1e-2}
    return {"rel": 1e-4, "max": 4e-3} if case.get("backward") else {"rel": 2e-6, "max": 2e-5}


# ---------------------------------------------------------------- 64-bit reference

def _edge_features(vi, vj, dim, mode):
    if mode == "diff":
        return vi - vj
    return torch.cat([vi[..., :dim], vj[..., :dim], vi[..., dim:], vj[..., dim:]], -1)


def _mm(a, b):
    """Product of a batch with one matrix as a plain two-dimensional product."""
    return (a.reshape(-1, a.shape[-1]) @ b).reshape(*a.shape[:-1], b.shape[-1])


def _layer64(P, attr, h, col, valid, i0, i1, dim, mode, act, residual):
    """Rows i0..i1 of the layer in float64: col [rows, slots] sources of each
    row's edges, valid [rows, slots]."""
    d = h.shape[1]
    x = _edge_features(attr[i0:i1, None, :].expand(-1, col.shape[1], -1), attr[col], dim, mode)
    z1 = torch.relu(_mm(x, P["W1"].T) + P["b1"])
    z = torch.relu(_mm(z1, P["W2"].T) + P["b2"])
    z = torch.cat([z, torch.ones_like(z[..., :1])], -1) * valid[..., None]
    S = torch.bmm(z.transpose(1, 2).contiguous(), h[col])             # [rows, h2+1, d]
    W = torch.cat([P["W3"], P["b3"][:, None]], 1).reshape(d, d, -1)   # [p, q, k]
    deg = valid.sum(1).clamp(min=1.0)
    agg = S.reshape(S.shape[0], -1) @ W.permute(2, 0, 1).reshape(-1, d) / deg[:, None]
    y = agg + h[i0:i1] @ P["Wr"].T + P["br"]
    y = torch.relu(y) if act == "relu" else y
    return y + h[i0:i1] if residual else y


def _slots(row_ptr, col, i0, i1):
    rp = row_ptr[i0:i1 + 1].long()
    deg = rp[1:] - rp[:-1]
    k = torch.arange(max(1, int(deg.max())), device="cuda")
    valid = k[None, :] < deg[:, None]
    at = (rp[:-1, None] + k[None, :]).clamp(max=max(0, col.numel() - 1))
    c = col[at.reshape(-1)].long().reshape(at.shape) if col.numel() else at * 0
    return torch.where(valid, c, torch.zeros_like(c)), valid.double()


def _round_to(h, dtype):
    """h as the layer takes it (rounded to its type, the gradient passed through)."""
    return h + (h.bfloat16().double() - h).detach() if dtype == "bf16" else h


def _graph64(st):
    """row_ptr and col of the graph, an input of the layer."""
    g = st["graph"]
    return g.row_ptr, g.col[:g.n_edges]


def _neighbours(pos, r, cap):
    """(col, valid) of the radius graph by all pairs: the float32 distance test
    with every operation rounded, the cap's nearest by (distance, index)."""
    n, r2, cols, vals = pos.shape[0], np.float32(r) * np.float32(r), [], []
    for i in range(0, n, 1024):
        p = pos[i:i + 1024]
        d2 = None
        for a in range(pos.shape[1]):
            dx = pos[None, :, a] - p[:, None, a]
            d2 = dx * dx if d2 is None else d2 + dx * dx
        d2[torch.arange(p.shape[0]), torch.arange(i, i + p.shape[0])] = math.inf
        d2 = torch.where(d2 <= float(r2), d2, torch.full_like(d2, math.inf))
        most = max(1, int(torch.isfinite(d2).sum(1).max()))
        d2, c = torch.sort(d2, dim=1, stable=True)
        k = min(most, cap or most)
        cols.append(c[:, :k])
        vals.append(torch.isfinite(d2[:, :k]).double())
    k = max(c.shape[1] for c in cols)
    pad = lambda t: torch.nn.functional.pad(t, (0, k - t.shape[1]))   # noqa: E731
    return torch.cat([pad(c) for c in cols]), torch.cat([pad(v) for v in vals])


def exact(case, seed):
    if case["kind"] in ("sample", "graph"):
        return None
    st = prepare(case, seed)
    dim = _dim(case)
    D = lambda P: {k: v.double().requires_grad_(True) for k, v in P.items()}   # noqa: E731
    if case["kind"] == "layer":
        rp, col = _graph64(st)
        P, h, attr = D(st["params"]), st["h"].double().requires_grad_(True), st["attr"].double()
        n, outs = case["n"], []
        deg = max(1, int((rp[1:] - rp[:-1]).max()))
        rows = int(max(64, min(8192, 2.5e8 / ((P["W2"].shape[0] + 1) * max(case["d"], 4 * deg)))))
        for i0 in range(0, n, rows):
            i1 = min(n, i0 + rows)
            with torch.set_grad_enabled(case["backward"]):
                o = _layer64(P, attr, h, *_slots(rp, col, i0, i1), i0, i1, dim, case["attr"], case["act"],
                             case["residual"])
                if case["backward"]:
                    o.backward(st["G"][i0:i1].double())
            outs.append(o.detach())
        if not case["backward"]:
            return {"out": torch.cat(outs)}
        return {"out": torch.cat(outs), "grad_h": h.grad, **{"d" + k: v.grad for k, v in P.items()}}
    if case["kind"] == "hop":
        rp, col = _graph64(st)
        c, valid = _slots(rp, col, 0, case["n"])
        enc, conv, dec = D(st["enc"]), D(st["conv"]), D(st["dec"])

        def mlp(P, x):
            x = torch.relu(x @ P["W1"].T + P["b1"])
            return torch.relu(x @ P["W2"].T + P["b2"]) @ P["W3"].T + P["b3"]

        v, lat = st["attr"].double(), mlp(enc, st["attr"].double())
        for _ in range(case["hops"]):
            lat = _layer64(conv, v, _round_to(lat, case["dtype"]), c, valid, 0, case["n"], dim, "diff", "identity", True)
            v = mlp(dec, lat)
        m = st["mask"].bool()
        loss = ((v[m] - st["Y"][m].double()) ** 2).mean()
        loss.backward()
        G = lambda P: {"d" + k: t.grad for k, t in P.items()}   # noqa: E731
        return {"loss": loss.detach().reshape(1), "v": v.detach(), "enc": G(enc), "conv": G(conv), "dec": G(dec)}
    # infer: each box is a graph of its own
    out = torch.zeros(case["n"], case["d"], dtype=torch.float64, device="cuda")
    for lo, hi in st["boxes"]:
        l32 = np.float32(st["r"])
        own = torch.ones(case["n"], dtype=torch.bool, device="cuda")
        near = own.clone()
        for a in range(dim):
            p = st["pos"][:, a].double()
            own &= (p >= float(np.float32(lo[a]))) & (p < float(np.float32(hi[a])))
            near &= (p >= float(np.float32(lo[a]) - l32)) & (p < float(np.float32(hi[a]) + l32))
        idx = torch.cat([own.nonzero()[:, 0], (near & ~own).nonzero()[:, 0]])
        if idx.numel() == 0:
            continue
        c, valid = _neighbours(st["pos"][idx], float(st["r"]), case["cap"])
        attr, h = st["attr"][idx].double(), st["h"][idx].double()
        with torch.no_grad():
            for P in st["params"]:
                y = torch.cat([_layer64({k: t.double() for k, t in P.items()}, attr, h, c[i:i + 2048], valid[i:i + 2048],
                                        i, min(i + 2048, idx.numel()), dim, "concat", "identity", True)
                               for i in range(0, idx.numel(), 2048)])
                h = _round_to(y, case["dtype"])
        no = int(own.sum())
        out[idx[:no]] = y[:no]
    return out
