"""Performance cases: the calls a user of this library makes, over the range of
sizes it serves.

Kinds of case (``kind``) and what each stands for in real use:

  embed      one projection of n points on the landmarks (``Context.embed``),
             the call every frame of an interactive session makes;
  frame      a frame of semi-supervised work on a large sample: projection with
             the neighbour list, then a k-means step of the landmarks that
             reuses each point's nearest landmark;
  update     one landmark step on its own, which finds the nearest landmarks
             itself (batch SOM on the 2-D grid, or k-means);
  som        a sweep of online SOM training (mini-batches, falling sigma and
             learning rate), as when a user lets the map settle;
  embed3     projection onto 3-D landmark positions;
  graph      graph mode between two frames: the landmarks' neighbourhood graph
             and a few steps of the force layout;
  serve      an edit of 2-D landmarks sent to the serving runtime for a resident
             data set, from submission to the result in host memory.

Points are cytometry-like Gaussian mixtures with a uniform background
(``data = "mixture"``) or uniform on the unit cube (``"uniform"``, the paper's
benchmark data); landmarks are noisy points of the sample on a 2-D grid, as
``synth`` draws them for the tests and the benchmark, drawn here on the GPU.
"""
import math

import torch

from paper_2201_00701_amd import esom

DEVICE = "cuda"


def _embed(name, n, d, g, k, mode, data="mixture", adjust=1.0, boost=1.0, knn=False):
    return {"name": name, "kind": "embed", "n": n, "d": d, "g": g, "k": k, "mode": mode, "data": data,
            "adjust": adjust, "boost": boost, "knn": knn}


def listed():
    return [
        # the smallest requests of the serving mix: launches and latency
        _embed("embed_1k_16d", 1_000, 16, 100, 8, "bf16"),
        # the headline workload of the benchmark in both modes
        _embed("embed_1m_32d_bf16", 1_000_000, 32, 400, 16, "bf16"),
        _embed("embed_1m_32d_fp32", 1_000_000, 32, 400, 16, "fp32"),
        # more dimensions, a 32 x 32 grid and a larger neighbourhood
        _embed("embed_1m_48d_bf16", 1_000_000, 48, 1024, 20, "bf16"),
        # a sample the shape of the paper's bone-marrow data (841,644 cells,
        # 39 markers: ragged rows) with the neighbour list returned
        _embed("embed_842k_39d_fp32", 841_644, 39, 625, 24, "fp32", boost=1.5, knn=True),
        # wide data: more dimensions than the fused kernel takes in FP32 mode
        _embed("embed_50k_100d_fp32", 50_000, 100, 400, 16, "fp32"),
        # the largest: a frame of 10 million points
        {"name": "frame_10m_64d", "kind": "frame", "n": 10_000_000, "d": 64, "g": 1024, "k": 16,
         "mode": "bf16", "data": "mixture_lognormal", "alpha": 0.1},
        # a SOM step of the headline sample
        {"name": "som_step_1m_32d", "kind": "update", "update": "som", "n": 1_000_000, "d": 32, "g": 400,
         "alpha": 0.3, "sigma": 2.0, "data": "mixture"},
        # a training sweep
        {"name": "som_train_100k_32d", "kind": "som", "n": 100_000, "d": 32, "g": 400, "steps": 50,
         "batch": 1024, "data": "mixture"},
        # 3-D output
        _embed3("embed3_200k_32d", 200_000, 32, 400, 16, "bf16"),
        # graph mode on a 32 x 32 grid of landmarks
        {"name": "graph_1024", "kind": "graph", "g": 1024, "d": 48, "kg": 10, "steps": 10},
        # an interactive 2-D edit of a resident sample
        {"name": "serve_edit_100k_32d", "kind": "serve", "n": 100_000, "d": 32, "g": 400, "k": 16,
         "mode": "bf16", "data": "mixture"},
    ]


def _embed3(name, n, d, g, k, mode):
    return {"name": name, "kind": "embed3", "n": n, "d": d, "g": g, "k": k, "mode": mode, "data": "mixture"}


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges; point counts, landmark counts and steps
    are bounded so that none costs more than the largest listed ones."""
    kind = rng.choice(["embed"] * 6 + ["frame", "update", "update", "som", "embed3", "graph", "serve"])
    data = rng.choice(["mixture", "mixture", "mixture_lognormal", "uniform"])
    mode = rng.choice(["bf16", "fp32"])
    if kind == "embed":
        d = _log(rng, 4, 128)
        g = _log(rng, 49, 2048)
        k = min(g, rng.choice([3, 5, 8, 10, 16, 16, 20, 24, 30]))
        wide = d > (128 if mode == "bf16" else 64)
        n = max(2 * g, _log(rng, 500, 60_000 if wide else 2_000_000 if g <= 1024 else 500_000))
        return {"kind": "embed", "n": n, "d": d, "g": g, "k": k, "mode": mode, "data": data,
                "adjust": rng.choice([1.0, 1.0, 1.0, 0.5]), "boost": round(rng.uniform(0.7, 2.0), 2),
                "knn": rng.random() < 0.3}
    if kind == "frame":
        return {"kind": "frame", "n": _log(rng, 20_000, 2_000_000), "d": _log(rng, 4, 64),
                "g": _log(rng, 49, 1024), "k": rng.choice([8, 13, 16, 20]), "mode": mode, "data": data,
                "alpha": 0.1}
    if kind == "update":
        return {"kind": "update", "update": rng.choice(["som", "kmeans"]), "n": _log(rng, 5_000, 2_000_000),
                "d": _log(rng, 4, 64), "g": _log(rng, 49, 1024), "alpha": round(rng.uniform(0.05, 1.0), 3),
                "sigma": round(rng.uniform(0.4, 4.0), 2), "data": data}
    if kind == "som":
        return {"kind": "som", "n": _log(rng, 5_000, 300_000), "d": _log(rng, 4, 64), "g": _log(rng, 49, 1024),
                "steps": rng.randint(3, 20), "batch": _log(rng, 1, 2048), "data": data}
    if kind == "embed3":
        return {"kind": "embed3", "n": _log(rng, 2_100, 200_000), "d": _log(rng, 4, 64), "g": _log(rng, 49, 1024),
                "k": rng.choice([5, 8, 12, 16, 20]), "mode": mode, "data": data}
    if kind == "graph":
        return {"kind": "graph", "g": _log(rng, 49, 1024), "d": _log(rng, 4, 48), "kg": rng.randint(4, 10),
                "steps": rng.randint(1, 10)}
    return {"kind": "serve", "n": _log(rng, 5_000, 300_000), "d": _log(rng, 8, 48), "g": _log(rng, 49, 1024),
            "k": rng.choice([8, 16, 20]), "mode": mode, "data": data}


# ---------------------------------------------------------------- inputs

def _points(n, d, data, gen):
    if data == "uniform":
        return torch.rand((n, d), generator=gen, device=DEVICE)
    ncl = 50 if data == "mixture_lognormal" else 30
    means = torch.rand((ncl, d), generator=gen, device=DEVICE) * 10 - 5
    sds = torch.rand((ncl, d), generator=gen, device=DEVICE) * 1.7 + 0.3
    w = torch.ones(ncl, device=DEVICE)
    if data == "mixture_lognormal":
        w = torch.exp(torch.randn(ncl, generator=gen, device=DEVICE))
    X = torch.empty((n, d), device=DEVICE)
    for s in range(0, n, 1 << 20):
        m = min(1 << 20, n - s)
        lab = torch.multinomial(w, m, replacement=True, generator=gen)
        rows = torch.randn((m, d), generator=gen, device=DEVICE) * sds[lab] + means[lab]
        bg = torch.rand(m, generator=gen, device=DEVICE) < 0.05
        box = torch.rand((m, d), generator=gen, device=DEVICE) * 16 - 8
        X[s:s + m] = torch.where(bg[:, None], box, rows)
    return X


def _landmarks(X, g, data, gen):
    noise = 0.0 if data == "uniform" else 0.1
    n, d = X.shape
    at = torch.randint(0, n // g, (g,), generator=gen, device=DEVICE) + torch.arange(g, device=DEVICE) * (n // g)
    return (X[at] + noise * torch.randn((g, d), generator=gen, device=DEVICE)).contiguous()


def _grid(g):
    cols = math.ceil(math.sqrt(g))
    j = torch.arange(g, device=DEVICE)
    return torch.stack([j % cols, j // cols], 1).float().contiguous()


def _grid3(l, gen):
    z = 2.0 * torch.sin(l[:, 0] / 3.0) * torch.cos(l[:, 1] / 4.0)
    z = z + 0.2 * torch.randn(l.shape[0], generator=gen, device=DEVICE)
    return torch.cat([l, z[:, None]], 1).contiguous()


def _schedule(steps):
    t = [i / max(steps - 1, 1) for i in range(steps)]
    return [3.0 * (0.4 / 3.0) ** u for u in t], [0.5 * 0.1 ** u for u in t]


def _inputs(case, seed):
    """The case's input tensors, from the seed alone."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    c = case
    if c["kind"] == "graph":
        X = _points(4 * c["g"], c["d"], "mixture", gen)
        L = _landmarks(X, c["g"], "mixture", gen)
        l0 = (_grid(c["g"]) + 0.3 * torch.randn((c["g"], 2), generator=gen, device=DEVICE)).contiguous()
        return {"L": L, "l0": l0}
    X = _points(c["n"], c["d"], c["data"], gen)
    s = {"X": X, "L": _landmarks(X, c["g"], c["data"], gen), "l": _grid(c["g"])}
    if c["kind"] == "embed3":
        s["l3"] = _grid3(s["l"], gen)
    if c["kind"] == "som":
        s["rows"] = torch.randint(0, c["n"], (c["steps"], c["batch"]), generator=gen, device=DEVICE,
                                  dtype=torch.int32)
        s["sigma"], s["alpha"] = _schedule(c["steps"])
    if c["kind"] == "serve":
        moved = torch.randint(0, c["g"], (4,), generator=gen, device=DEVICE)
        s["l_edit"] = s["l"].clone()
        s["l_edit"][moved] += 0.5 * torch.randn((4, 2), generator=gen, device=DEVICE)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    kind = case["kind"]
    if kind == "serve":
        X, L, l = (s[q].cpu().numpy() for q in ("X", "L", "l"))
        s = {"case": case, "L": L, "l_edit": s["l_edit"].cpu().numpy(), "srv": esom.Server(0)}
        s["out"] = l[:1].repeat(case["n"], 0)
        s["id"] = s["srv"].put(X)
        # the session's first frame
        s["srv"].wait(s["srv"].submit(L, l, k=case["k"], mode=case["mode"], dataset=s["id"], out=s["out"]))
        return s
    s["ctx"] = esom.Context(0)
    if kind in ("embed", "frame"):
        s["out"] = torch.empty((case["n"], 2), device=DEVICE)
    if kind == "frame":
        s["idx"] = torch.empty((case["n"], case["k"]), dtype=torch.int32, device=DEVICE)
    if kind in ("frame", "update", "som"):
        # every pass starts from the same landmarks
        s["L0"] = s["L"].clone()
    if kind == "graph":
        s["l"] = s["l0"].clone()
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "embed":
        r = s["ctx"].embed(s["X"], s["L"], s["l"], k=c["k"], mode=c["mode"], boost=c["boost"],
                           adjust=c["adjust"], out=s["out"], knn=c["knn"])
        return {"out": r[0], "idx": r[1], "d2": r[2]} if c["knn"] else {"out": r}
    if kind == "frame":
        s["L"].copy_(s["L0"])
        st = torch.cuda.current_stream().cuda_stream
        rc = esom.esom_embed(s["ctx"].handle, s["X"].data_ptr(), c["n"], c["d"], c["d"], s["L"].data_ptr(),
                             s["l"].data_ptr(), c["g"], esom.esom_default_params(k=c["k"], mode=c["mode"]),
                             s["out"].data_ptr(), s["idx"].data_ptr(), 0, st)
        if rc != esom.ESOM_OK:
            raise esom.EsomError(rc, esom.esom_last_error())
        cnt = s["ctx"].landmark_update(s["X"], s["L"], s["l"], kind="kmeans", alpha=c["alpha"],
                                       nearest=s["idx"][:, 0], counts=True)
        return {"out": s["out"], "idx": s["idx"], "L": s["L"], "counts": cnt}
    if kind == "update":
        s["L"].copy_(s["L0"])
        cnt = s["ctx"].landmark_update(s["X"], s["L"], s["l"], kind=c["update"], alpha=c["alpha"],
                                       sigma=c["sigma"], counts=True)
        return {"L": s["L"], "counts": cnt}
    if kind == "som":
        s["L"].copy_(s["L0"])
        s["ctx"].som_train(s["X"], s["L"], s["l"], s["rows"], s["sigma"], s["alpha"])
        return {"L": s["L"]}
    if kind == "embed3":
        out, idx = s["ctx"].embed3(s["X"], s["L"], s["l3"], k=c["k"], mode=c["mode"], knn=True)
        return {"out": out, "idx": idx}
    if kind == "graph":
        s["l"].copy_(s["l0"])
        nbr, d2 = esom.landmark_graph(s["L"], c["kg"])
        s["ctx"].graph_layout(s["L"], nbr, s["l"], steps=c["steps"], scale=0.4)
        return {"nbr": nbr, "d2": d2, "l": s["l"]}
    srv = s["srv"]
    r = srv.wait(srv.submit(s["L"], s["l_edit"], k=c["k"], mode=c["mode"], dataset=s["id"], out=s["out"]))
    return {"out": r["out"]}


def work(case):
    """Each input read once and each output written once; the distance
    contraction (2 n g d), the pair terms of the active neighbours (about 20
    operations a pair in 2-D, 30 in 3-D), and the landmark sums."""
    c = case
    g, d = c["g"], c["d"]
    if c["kind"] == "graph":
        return {"bytes": 4 * g * d + 8 * g * c["kg"] + 16 * g,
                "flops": 2 * g * g * d + c["steps"] * 10 * g * g}
    n = c["n"]
    x = 4 * n * d + 4 * g * (d + 2)
    if c["kind"] == "som":
        rows = c["steps"] * c["batch"]
        return {"bytes": 4 * rows * (d + 1) + 8 * g * d,
                "flops": rows * (2 * g * d + d) + c["steps"] * 2 * g * g * d}
    if c["kind"] == "update":
        blend = 2 * g * g * d if c["update"] == "som" else 0
        return {"bytes": x + 4 * g * (d + 1), "flops": 2 * n * g * d + n * d + blend}
    k = c["k"]
    pairs = (k - 1) * (k - 2) / 2
    if c["kind"] == "serve":  # from the cached neighbours
        return {"bytes": 8 * n * k + 16 * n + 4 * g * (d + 2), "flops": n * 20 * pairs + g * g * d}
    if c["kind"] == "embed3":
        return {"bytes": x + 12 * n + 4 * n * k, "flops": n * (2 * g * d + 3 * k * d + 30 * pairs)}
    b = {"bytes": x + 8 * n, "flops": n * (2 * g * d + 3 * k * d + 20 * pairs)}
    if c["kind"] == "frame":
        b["bytes"] += 4 * n * k + 4 * g * (d + 1)
        b["flops"] += n * d
    elif c["knn"]:
        b["bytes"] += 8 * n * k
    return b


# ---------------------------------------------------------------- 64-bit values

def _nearest(x, L, k):
    """The k nearest of the landmarks L by (distance, index): squared distances
    (64 bits, from differences) and indices."""
    d2 = (x * x).sum(1, keepdim=True) + (L * L).sum(1)[None] - 2.0 * x @ L.T
    m = min(L.shape[0], k + 2)
    _, idx = torch.topk(d2, m, dim=1, largest=False)
    idx, _ = torch.sort(idx, dim=1)
    d2 = torch.stack([((x - L[idx[:, j]]) ** 2).sum(1) for j in range(m)], 1)
    d2, at = torch.sort(d2, dim=1, stable=True)
    return d2[:, :k].contiguous(), idx.gather(1, at)[:, :k].contiguous()


def _project(x, L, l, d2, idx, boost, adjust, cutoff=10.0, gravity=1e-5):
    """Scores, segment projections and the solve, in any number of output dimensions."""
    n, k = d2.shape
    g, m = l.shape
    dl = d2.sqrt()
    w = 1.0 / torch.arange(1, k + 1, device=x.device, dtype=x.dtype)
    mu = (dl * w).sum(1, keepdim=True) / w.sum()
    var = (w * (dl - mu) ** 2).sum(1, keepdim=True) / w.sum()
    flat = ~(var > 1e-30 * mu * mu)
    s = torch.where(flat, torch.ones_like(dl), torch.exp(boost * (mu - dl) / var.sqrt()))
    if k < g:
        s = s * (1.0 - torch.exp(cutoff * (dl / dl[:, -1:] - 1.0)))
    same = dl[:, :1] == dl[:, -1:]
    s = torch.where(same, torch.zeros_like(s), s)
    P = l[idx]
    M = torch.zeros((n, m, m), dtype=x.dtype, device=x.device)
    r = torch.zeros((n, m), dtype=x.dtype, device=x.device)
    LL = ((L[:, None] - L[None]) ** 2).sum(2) if g * g * L.shape[1] < 2e8 else torch.cdist(L, L) ** 2
    for a in range(k - 1):
        h = P[:, a + 1:] - P[:, a:a + 1]
        hh = (h * h).sum(2)
        HH = LL[idx[:, a:a + 1], idx[:, a + 1:]]
        D = 0.5 + (d2[:, a:a + 1] - d2[:, a + 1:]) / (2.0 * HH)
        ok = (HH > 0) & (hh > 0)
        q = torch.where(ok, s[:, a:a + 1] * s[:, a + 1:] * hh ** (-adjust), torch.zeros_like(hh))
        rhs = torch.where(ok, D + (h * P[:, a:a + 1]).sum(2) / hh, torch.zeros_like(hh))
        qh = torch.where(ok, q / hh, torch.zeros_like(hh))
        for i in range(m):
            r[:, i] += (q * h[:, :, i] * rhs).sum(1)
            for j in range(m):
                M[:, i, j] += (qh * h[:, :, i] * h[:, :, j]).sum(1)
    for i in range(m):
        M[:, i, i] += gravity * s.sum(1)
        r[:, i] += gravity * (s * P[:, :, i]).sum(1)
    det = torch.linalg.det(M)
    tr = M.diagonal(dim1=1, dim2=2).sum(1) / m
    bad = same[:, 0] | ~(s.sum(1) > 0) | ~(det > 1e-9 * tr ** m)
    eye = torch.eye(m, dtype=x.dtype, device=x.device).expand_as(M)
    p = torch.linalg.solve(torch.where(bad[:, None, None], eye, M), r[:, :, None])[:, :, 0]
    return torch.where(bad[:, None], P.mean(1), p)


def _exact_embed(X, L, l, k, boost, adjust):
    L, l = L.double(), l.double()
    out, ii, dd = [], [], []
    step = max(1024, min(65536, 1 << 26 >> (L.shape[0] - 1).bit_length()))
    for s in range(0, X.shape[0], step):
        x = X[s:s + step].double()
        d2, idx = _nearest(x, L, k)
        out.append(_project(x, L, l, d2, idx, boost, adjust))
        ii.append(idx.int())
        dd.append(d2)
    return torch.cat(out), torch.cat(ii), torch.cat(dd)


def _sums(X, near, g):
    S = torch.zeros((g, X.shape[1]), dtype=torch.float64, device=X.device)
    for s in range(0, X.shape[0], 1 << 20):
        S.index_add_(0, near[s:s + (1 << 20)].long(), X[s:s + (1 << 20)].double())
    return S, torch.bincount(near.long(), minlength=g).double()


def _argmin(X, L):
    L = L.double()
    return torch.cat([_nearest(X[s:s + 65536].double(), L, 1)[1][:, 0] for s in range(0, X.shape[0], 65536)])


def _topology(l, sigma):
    l = l.double()
    d2 = ((l[:, None] - l[None]) ** 2).sum(2)
    return torch.exp(-d2 / (2.0 * sigma * sigma))


def _f32(v):
    """The value a float argument of the C interface takes."""
    return float(torch.tensor(v, dtype=torch.float32))


def exact(case, seed):
    c = case
    s = _inputs(case, seed)
    kind = c["kind"]
    if kind in ("embed", "embed3", "serve"):
        l = s["l3"] if kind == "embed3" else s["l_edit"] if kind == "serve" else s["l"]
        out, idx, d2 = _exact_embed(s["X"], s["L"], l, c["k"], _f32(c.get("boost", 1.0)),
                                    _f32(c.get("adjust", 1.0)))
        if kind == "embed":
            return {"out": out, "idx": idx, "d2": d2} if c["knn"] else {"out": out}
        return {"out": out, "idx": idx} if kind == "embed3" else {"out": out.cpu().numpy()}
    L = s["L"].double()
    if kind == "frame":
        out, idx, _ = _exact_embed(s["X"], s["L"], s["l"], c["k"], 1.0, 1.0)
        S, cnt = _sums(s["X"], idx[:, 0], c["g"])
        mean = torch.where(cnt[:, None] > 0, S / cnt[:, None].clamp(min=1), L)
        return {"out": out, "idx": idx, "L": L + _f32(c["alpha"]) * (mean - L), "counts": cnt.int()}
    if kind == "update":
        S, cnt = _sums(s["X"], _argmin(s["X"], s["L"]), c["g"])
        counts = cnt.int()
        if c["update"] == "som":
            h = _topology(s["l"], _f32(c["sigma"]))
            S, cnt = h @ S, h @ cnt
        mean = torch.where(cnt[:, None] > 0, S / torch.where(cnt > 0, cnt, torch.ones_like(cnt))[:, None], L)
        return {"L": L + _f32(c["alpha"]) * (mean - L), "counts": counts}
    if kind == "som":
        L32 = s["L"].clone()
        for t in range(c["steps"]):
            xb = s["X"][s["rows"][t].long()]
            S, cnt = _sums(xb, _argmin(xb, L32), c["g"])
            h = _topology(s["l"], _f32(s["sigma"][t]))
            L = L32.double()
            L = L + _f32(s["alpha"][t]) / c["batch"] * (h @ S - (h @ cnt)[:, None] * L)
            L32 = L.float()
        return {"L": L}
    # graph
    g, kg = c["g"], c["kg"]
    d2 = torch.stack([((L - L[u]) ** 2).sum(1) for u in range(g)])
    hd = d2.sqrt()
    d2.fill_diagonal_(math.inf)
    dn, nbr = torch.sort(d2, dim=1, stable=True)
    dn, nbr = dn[:, :kg].contiguous(), nbr[:, :kg].contiguous()
    edge = torch.zeros((g, g), dtype=torch.bool, device=L.device)
    edge.scatter_(1, nbr, True)
    edge |= edge.clone().T
    l = s["l0"]
    scale, rep, soft, step, most = _f32(0.4), _f32(0.05), _f32(0.5), _f32(0.1), _f32(0.5)
    for _ in range(c["steps"]):
        p = l.double()
        df = p[None] - p[:, None]
        r2 = (df * df).sum(2)
        r = r2.sqrt()
        pull = torch.where(edge & (r > 0), (r - scale * hd) / r, torch.zeros_like(r))
        mv = step * ((pull - rep / (r2 + soft * soft))[:, :, None] * df).sum(1)
        length = mv.norm(dim=1, keepdim=True)
        mv = torch.where(length > most, mv * most / length, mv)
        p = p + mv
        l = p.float()
    return {"nbr": nbr.int(), "d2": dn, "l": p}
