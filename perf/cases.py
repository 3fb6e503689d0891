"""Workloads of the library through its public entry points, for timing.

Every case is one whole solve as a program makes it: the tree is built from
points that are in device memory, the search or the clustering runs on it, and
the tree is released. Sizes, options and point sets are those of the tests, of
``bench.py`` and of its batched and served modes: clustered sets (Gaussian
clumps on a uniform background) of 2^10 to 2^24 points, uniform ones where the
separate query / source search uses them, k up to 64, linking lengths of 0.1
and 0.2 mean spacings.

A case holds ``kind`` and the fields that this kind uses:

  knn        build + kNN                            n, k, data
  fof        build + FoF                            n, alpha, data
  both       build + kNN and FoF in one call        n, k, alpha, coarsen
  periodic   the same in the periodic unit cube     n, k, alpha
  query      joint build + kNN of the query points  n, n_qry, k, data
  forest     many sets: one build, kNN, FoF         sets, log2_min, log2_max, k, alpha
  catalogue  build + group catalogue (velocities)   n, alpha, min_members
"""
import math

import numpy as np
import torch

from paper_2604_05885_amd import api, inputs


def listed():
    return [
        # one small call: latency, launches and host work
        {"name": "knn_1k", "kind": "knn", "n": 1000, "k": 8, "data": "clustered"},
        # the smoke run's size, clustering only
        {"name": "fof_4k", "kind": "fof", "n": 4096, "alpha": 0.2, "data": "clustered"},
        # an average set of the batched workload, solved by itself; odd size
        {"name": "both_50k", "kind": "both", "n": 50021, "k": 16, "alpha": 0.2, "coarsen": 8},
        # an ordinary served request with the largest k of one leaf pass
        {"name": "knn_300k_k32", "kind": "knn", "n": 300007, "k": 32, "data": "clustered"},
        # the method's usual comparison: uniform points
        {"name": "knn_uniform_1m", "kind": "knn", "n": 1000000, "k": 16, "data": "uniform"},
        # more neighbours than one leaf pass keeps
        {"name": "knn_1m_k64", "kind": "knn", "n": 1000003, "k": 64, "data": "clustered"},
        # separate query and source points (cross search, k = 30)
        {"name": "query_2m_2m", "kind": "query", "n": 2 ** 21, "n_qry": 2 ** 21, "k": 30,
         "data": "uniform"},
        # group catalogue of a simulation output with velocities
        {"name": "catalogue_4m", "kind": "catalogue", "n": 2 ** 22, "alpha": 0.2,
         "min_members": 20},
        # a periodic simulation box
        {"name": "periodic_4m", "kind": "periodic", "n": 2 ** 22, "k": 16, "alpha": 0.2},
        # repeated evaluations: many sets of ragged sizes in one forest
        {"name": "forest_256", "kind": "forest", "sets": 256, "log2_min": 10.0, "log2_max": 18.0,
         "k": 16, "alpha": 0.2},
        # clustering of the benchmark's set alone
        {"name": "fof_16m", "kind": "fof", "n": 2 ** 24, "alpha": 0.2, "data": "clustered"},
        # the benchmark step
        {"name": "both_16m", "kind": "both", "n": 2 ** 24, "k": 16, "alpha": 0.2, "coarsen": 16},
    ]


def draw(rng):
    """One more case: sizes spread over their logarithm, mostly odd, with n * k
    bounded so that none costs more than the benchmark step."""
    kind = rng.choice(["knn", "knn", "knn", "fof", "fof", "both", "both", "periodic", "query",
                       "forest", "catalogue"])
    k = rng.choice([2, 4, 8, 8, 10, 16, 16, 20, 30, 32, 32, 48, 64])
    alpha = rng.choice([0.1, 0.2, 0.2])

    def size(lo, hi):
        return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))

    if kind == "knn":
        return {"kind": kind, "n": size(1000, min(2 ** 23, 2 ** 27 // k)), "k": k,
                "data": rng.choice(["clustered", "uniform"])}
    if kind == "fof":
        return {"kind": kind, "n": size(1000, 2 ** 23), "alpha": alpha,
                "data": rng.choice(["clustered", "uniform"])}
    if kind == "both":
        return {"kind": kind, "n": size(1000, min(2 ** 23, 2 ** 26 // k)), "k": k, "alpha": alpha,
                "coarsen": rng.choice([8, 8, 16])}
    if kind == "periodic":
        return {"kind": kind, "n": size(1000, min(2 ** 22, 2 ** 26 // k)), "k": k, "alpha": alpha}
    if kind == "query":
        return {"kind": kind, "n": size(1000, min(2 ** 21, 2 ** 26 // k)),
                "n_qry": size(1000, min(2 ** 21, 2 ** 26 // k)), "k": k,
                "data": rng.choice(["clustered", "uniform"])}
    if kind == "forest":
        return {"kind": kind, "sets": size(2, 256), "log2_min": 8.0,
                "log2_max": rng.uniform(10.0, 16.0), "k": min(k, 32), "alpha": alpha}
    return {"kind": kind, "n": size(1000, 2 ** 22), "alpha": alpha,
            "min_members": rng.choice([2, 20])}


def _points(n, data, seed):
    """n points in device memory, float32 (n, 3), in [0, 1)^3."""
    if data == "uniform":
        return torch.from_numpy(inputs.uniform(n, seed)).cuda()
    n_cl, cen, sig, cnt = inputs.clump_params(n, max(1, round(4096 * n / 2 ** 24)), seed)
    return inputs.clustered_device(n, seed, n_cl, torch.from_numpy(cen).cuda(),
                                   torch.from_numpy(sig).cuda(), torch.from_numpy(cnt).cuda())


def _sets(case):
    """Offsets and linking lengths of a forest: the sizes belong to the case."""
    return inputs.batched_sets(case["sets"], 4, case["log2_min"], case["log2_max"],
                               alpha=case["alpha"], size_only=True)[1:]


def _inputs(case, seed):
    """The device arrays (and for a forest the host arrays) of a case."""
    kind = case["kind"]
    if kind == "forest":
        off, b = _sets(case)
        p = np.concatenate([inputs.clustered(int(m), max(1, round(4096 * m / 2 ** 24)), [seed, i])
                            for i, m in enumerate(np.diff(off))])
        return {"points": torch.from_numpy(p).cuda(), "offsets": off, "b": b}
    s = {"points": _points(case["n"], case.get("data", "clustered"), seed)}
    if kind == "query":
        s["queries"] = _points(case["n_qry"], case["data"], seed + 1000003)
    if kind == "catalogue":
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        s["vel"] = 300.0 * torch.randn((case["n"], 3), generator=g, device="cuda")
    if "alpha" in case:
        s["b"] = inputs.linking_length(case["n"], case["alpha"])
    return s


def prepare(case, seed):
    """Points, output buffers and build options, as a program keeps them."""
    s = dict(_inputs(case, seed), case=case)
    opts = {}
    if case.get("coarsen", 8) != 8:
        opts["coarsen"] = case["coarsen"]
    if case["kind"] == "periodic":
        opts["period"] = 1.0
    s["opts"] = api.default_opts(**opts) if opts else None
    rows = case["n_qry"] if case["kind"] == "query" else s["points"].shape[0]
    if "k" in case:
        s["idx"] = torch.empty((rows, case["k"]), dtype=torch.int32, device="cuda")
        s["dist2"] = torch.empty((rows, case["k"]), dtype=torch.float32, device="cuda")
    if case["kind"] == "catalogue":
        # the group table of the program, as long as the set can have groups
        m = case["n"] // case["min_members"] + 1
        s["table"] = {"label": np.zeros(m, np.int32), "count": np.zeros(m, np.int32),
                      "first": np.zeros(m, np.int64), "cm": np.zeros((m, 3)),
                      "vcm": np.zeros((m, 3)), "r_inertia": np.zeros(m)}
    elif "alpha" in case:
        s["label"] = torch.empty(rows, dtype=torch.int32, device="cuda")
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "query":
        with api.jz_build_joint(s["points"], s["queries"], s["opts"]) as t:
            idx, d2 = t.knn_query(case["k"], s["idx"], s["dist2"])
        return {"idx": idx, "dist2": d2}
    if kind == "forest":
        with api.jz_forest_build(s["points"], s["offsets"], s["opts"]) as t:
            idx, d2 = t.knn(case["k"], s["idx"], s["dist2"])
            label = t.fof(s["b"], s["label"])
        return {"idx": idx, "dist2": d2, "label": label}
    with api.jz_build(s["points"], s["opts"]) as t:
        if kind == "knn":
            idx, d2 = t.knn(case["k"], s["idx"], s["dist2"])
            return {"idx": idx, "dist2": d2}
        if kind == "fof":
            return {"label": t.fof(s["b"], s["label"])}
        if kind == "catalogue":
            c = t.catalogue(s["b"], case["min_members"], vel=s["vel"])
            for f, column in s["table"].items():
                column[:len(c["groups"])] = c["groups"][f]
            return {"label": c["label"], "order": c["order"], "table": s["table"]}
        idx, d2, label = t.knn_fof(case["k"], s["b"], s["idx"], s["dist2"], s["label"])
        return {"idx": idx, "dist2": d2, "label": label}


def work(case):
    """Every point read once, every output written once; per neighbour row k
    distances of 8 operations, per linked point one."""
    kind = case["kind"]
    if kind == "forest":
        n = int(_sets(case)[0][-1])
    else:
        n = case["n"]
    rows = case["n_qry"] if kind == "query" else n
    bytes_ = 12 * n + (12 * rows if kind == "query" else 0)
    flops = 0
    if "k" in case:
        bytes_ += 8 * rows * case["k"]
        flops += 8 * rows * case["k"]
    if "alpha" in case:
        bytes_ += 4 * n
        flops += 8 * n
    if kind == "catalogue":
        bytes_ += 12 * n + 4 * n
        flops += 20 * n
    return {"bytes": bytes_, "flops": flops}


def _dist2(q, p, period):
    d = q[:, None, :] - p[None, :, :]
    if period:
        d = d - period * torch.round(d / period)
    return (d * d).sum(-1)


def _knn_exact(p, q, k, period=0.0):
    p, q = p.double(), q.double()
    step = max(1, 2 ** 25 // p.shape[0])
    rows = [torch.topk(_dist2(q[i:i + step], p, period), min(k, p.shape[0]), dim=1, largest=False,
                       sorted=True)[0] for i in range(0, q.shape[0], step)]
    d2 = torch.cat(rows)
    if k > p.shape[0]:
        d2 = torch.nn.functional.pad(d2, (0, k - p.shape[0]), value=math.inf)
    return d2


def _catalogue_exact(p, vel, b, min_members):
    p, n = p.double(), p.shape[0]
    step = max(1, 2 ** 25 // n)
    src, dst = [], []
    for i in range(0, n, step):
        a, c = torch.nonzero(_dist2(p[i:i + step], p, 0.0) <= b * b, as_tuple=True)
        src.append(a + i)
        dst.append(c)
    src, dst = torch.cat(src), torch.cat(dst)
    label = torch.arange(n, device=p.device)
    while True:
        new = label.scatter_reduce(0, src, label[dst], "amin")
        new = new[new]
        if torch.equal(new, label):
            break
        label = new
    members = torch.bincount(label, minlength=n)
    groups = torch.nonzero(members >= min_members)[:, 0]
    c = members[groups].double()[:, None]

    def mean(x):
        return torch.zeros_like(x).index_add(0, label, x)[groups] / c

    cm = mean(p)
    full = torch.zeros_like(p)
    full[groups] = cm
    r2 = ((p - full[label]) ** 2).sum(-1, keepdim=True)
    table = {"cm": cm, "vcm": mean(vel.double()), "r_inertia": mean(r2)[:, 0].sqrt()}
    rows = n // min_members + 1
    return {"table": {f: torch.cat([x, x.new_zeros((rows - x.shape[0],) + x.shape[1:])])
                      for f, x in table.items()}}


def exact(case, seed):
    """Squared distances (and catalogue means) in binary64 by brute force, for
    sets small enough for it; indices and labels are whole numbers."""
    kind = case["kind"]
    if kind == "forest" or case["n"] > (2 ** 15 if kind == "catalogue" else 2 ** 17):
        return None
    if kind == "query" and case["n_qry"] > 2 ** 17:
        return None
    s = _inputs(case, seed)
    if kind == "catalogue":
        return _catalogue_exact(s["points"], s["vel"], s["b"], case["min_members"])
    if "k" not in case:
        return None
    return {"idx": None, "dist2": _knn_exact(s["points"], s.get("queries", s["points"]), case["k"],
                                             1.0 if kind == "periodic" else 0.0)}
