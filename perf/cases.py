"""The measured cases: what a program that searches an IVF-PQ index asks of the library, from one
query to ten thousand, through the public entry points of `paper_2312_01712_amd.binding`.

A case is a dict of plain values:
  call     "search"   one `search` call (filtering, tables, scan, top-k), workspace and outputs kept
           "noalloc"  the same through `search_noalloc`
           "coarse"   the filtering stage alone, lists and distances
           "dynamic"  `coarse`, `query_radii`, `scan_topk`: per-query radii from a density map
  family   the data: "gauss", "sift", "deep" or "tti" mixtures of `workloads`, spread `sigma`,
           `centres` components; `shift` moves the queries' components
  N, D, nlist, M, Q, nprobe, k, mode (scoring), metric (0 squared L2, 1 inner product), keep (share
  of the codebook entries inside the radius; 1: infinite radii)

The index is trained here and not by `workloads.train_index`: that one adds floats with atomics, so
two runs differ in the last bits; here every mean is a sum of integers, and a seed gives the same
index in every run.
"""
import math

import numpy as np
import torch

from paper_2312_01712_amd import binding
from paper_2312_01712_amd import workloads as wl


def listed():
    sift = dict(call="search", family="sift", sigma=20.0, shift=0.0, N=1_000_000, D=128, nlist=1024, M=64, centres=1024,
                nprobe=32, k=100, mode=0, metric=0, keep=0.25)
    deep = dict(call="search", family="deep", sigma=0.1, shift=0.0, N=1_000_000, D=96, nlist=1024, M=48, centres=2048,
                nprobe=64, k=100, mode=0, metric=0, keep=0.25)
    tti = dict(call="search", family="tti", sigma=0.25, shift=0.3, N=1_000_000, D=200, nlist=1024, M=100, centres=1024,
               nprobe=64, k=100, mode=0, metric=0, keep=0.25)
    return [
        # one query against the one-million-point 128-d index: an interactive look-up, latency only
        dict(sift, name="single_query", Q=1),
        # a small serving batch on the smallest index, through the entry point that takes no workspace
        dict(name="serving_batch", call="noalloc", family="gauss", sigma=0.15, shift=0.0, N=100_000, D=64, nlist=256,
             M=16, centres=256, Q=32, nprobe=8, k=10, mode=0, metric=0, keep=0.25),
        # per-query radii looked up in a density map, a few hundred queries at a time
        dict(sift, name="dynamic_radii", call="dynamic", Q=300),
        # a code length and a dimension of no benchmark: 30 subspaces of 4, every size odd
        dict(name="other_shape", call="search", family="gauss", sigma=0.4, shift=0.0, N=500_000, D=120, nlist=701,
             M=30, centres=900, Q=999, nprobe=24, k=10, mode=0, metric=0, keep=0.5),
        # the headline batch: 10 000 queries, 128 dimensions, clustered data
        dict(sift, name="batch_128", Q=10_000),
        # the 96-d batch on data without cluster structure, 64 probes
        dict(deep, name="batch_96", Q=10_000),
        # the 200-d batch (100 subspaces)
        dict(tti, name="batch_200", Q=10_000),
        # lists of the length of the 100-million-point configuration (6 000 to 8 000 points), some of
        # them holding two components of the data
        dict(sift, name="long_lists", N=8_000_000, nlist=1024, centres=1088, Q=4096, nprobe=64),
        # the filtering stage of the 100-million-point configuration
        dict(sift, name="filter_16k", call="coarse", N=65_536, nlist=16_384, centres=16_384, Q=10_000, nprobe=64),
        # a thousand neighbours per query (the second quality figure, R100@1000)
        dict(sift, name="thousand_neighbours", Q=2000, k=1000),
        # maximum inner product search over the 200-d index
        dict(tti, name="inner_product", Q=4000, metric=1),
        # hit-count scoring on the 96-d index
        dict(deep, name="hit_counts", Q=5000, mode=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case over the same ranges: any size of batch, code lengths with and without a kernel of
    their own, both metrics, every scoring, k from 1 to 1000."""
    kind = rng.choice(["sift", "sift", "deep", "tti", "gauss", "gauss", "odd", "coarse"])
    c = dict(call="search", shift=0.0, mode=0, metric=0, keep=rng.choice([0.1, 0.25, 0.5, 1.0]))
    if kind == "sift":
        c.update(family="sift", sigma=20.0, D=128, M=64)
    elif kind == "deep":
        c.update(family="deep", sigma=0.1, D=96, M=48)
    elif kind == "tti":
        c.update(family="tti", sigma=0.25, shift=0.3, D=200, M=100)
    elif kind == "gauss":
        c.update(family="gauss", sigma=rng.choice([0.15, 0.4]), D=64, M=16)
    elif kind == "odd":
        dsub = rng.choice([1, 2, 3, 4, 6, 8])
        c.update(family="gauss", sigma=rng.choice([0.15, 0.4]), M=rng.randint(5, min(80, 240 // dsub)))
        c["D"] = c["M"] * dsub
    else:
        c.update(call="coarse", family="sift", sigma=20.0, D=rng.choice([96, 100, 128, 200]))
        c["M"] = c["D"] // 2
    if kind == "coarse":
        nlist = _log(rng, 3000, 16_384)
        c.update(N=65_536, nlist=nlist, centres=nlist, Q=_log(rng, 1, 10_000), nprobe=_log(rng, 8, 128), k=1)
        return c
    c["N"] = _log(rng, 50_000, 2_000_000)
    c["nlist"] = _log(rng, max(64, c["N"] // 6000), max(128, c["N"] // 600))
    c["centres"] = int(c["nlist"] * rng.choice([1.0, 1.07, 2.0]))
    c["Q"] = _log(rng, 1, 10_000)
    c["nprobe"] = min(_log(rng, 4, 64), c["nlist"] // 2)
    c["k"] = rng.choice([1, 10, 10, 33, 100, 100, 100, 129, 500, 1000])
    c["k"] = min(c["k"], 50 * c["nprobe"])
    roll = rng.random()
    if roll < 0.15:
        c["metric"] = 1
    elif roll < 0.3:
        c["mode"] = rng.choice([1, 2])
        c["keep"] = min(c["keep"], 0.5)
    elif roll < 0.4 and c["D"] == 2 * c["M"]:
        c["call"] = "dynamic"
    elif roll < 0.5 and c["Q"] <= 500:
        c["call"] = "noalloc"
    # no dearer than the largest listed case, also where nothing can be pruned
    dear = c["nprobe"] * (c["N"] / c["nlist"]) * c["M"] * max(1, c["k"] // 128)
    c["Q"] = max(1, min(c["Q"], int(3e10 / dear)))
    return c


# ---- the index ------------------------------------------------------------------------------

def _means(x, labels, k, old):
    """Mean of the rows of each label, summed as integers (in 2^-20) so that the order of the
    additions does not matter; a label without rows keeps its old value."""
    fixed = torch.round(x.double() * (1 << 20)).to(torch.int64)
    sums = torch.zeros((k, x.shape[1]), dtype=torch.int64, device=x.device).index_add_(0, labels, fixed)
    n = torch.bincount(labels, minlength=k)[:, None]
    return torch.where(n > 0, (sums.double() / n.clamp(min=1) / (1 << 20)).float(), old)


def _nearest(x, c):
    out = torch.empty(x.shape[0], dtype=torch.int64, device=x.device)
    cc = (c * c).sum(1)
    for s in range(0, x.shape[0], 1 << 16):
        out[s:s + (1 << 16)] = (cc[None, :] - 2.0 * (x[s:s + (1 << 16)] @ c.T)).argmin(1)
    return out


def _workload(case, seed):
    return wl.Workload("case", case["N"], case["D"], case["nlist"], case["M"], case["Q"], case["nprobe"], case["k"],
                       case["family"], case["centres"], case["sigma"], query_shift=case["shift"],
                       seed=int(seed) % 1_000_003)


def _index(case, seed):
    """Arrays of a trained index on the GPU: centroids (k-means started from the data's components,
    so components beyond nlist share lists), residual codebooks, points sorted by list."""
    w = _workload(case, seed)
    dev = "cuda"
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) % 1_000_003 + 17)
    comps = wl.mixture_centres(w, dev)
    n_train = min(w.N, max(16 * w.nlist, 65_536), wl.BASE_CHUNK)
    xt = wl.base_chunk(w, comps, 0, n_train)
    cent = comps[:w.nlist].clone()
    for _ in range(3):
        cent = _means(xt, _nearest(xt, cent), w.nlist, cent)
    n_pq = min(n_train, 32_768)
    res = (xt[:n_pq] - cent[_nearest(xt[:n_pq], cent)]).reshape(n_pq, w.M, w.dsub).transpose(0, 1).contiguous()
    cb = res[:, torch.randperm(n_pq, generator=g, device=dev)[:256], :].clone()         # [M][256][dsub]
    rows = torch.arange(w.M, device=dev)[:, None] * 256
    for _ in range(3):
        a = ((cb * cb).sum(2)[:, None, :] - 2.0 * torch.bmm(res, cb.transpose(1, 2).contiguous())).argmin(2)
        cb = _means(res.reshape(-1, w.dsub), (a + rows).reshape(-1), w.M * 256, cb.reshape(-1, w.dsub)).reshape(cb.shape)
    if case["call"] == "coarse":   # the filtering stage never looks at the codes
        labels = torch.randint(0, w.nlist, (w.N,), generator=g, device=dev)
        codes = torch.randint(0, 256, (w.N, w.M), generator=g, device=dev, dtype=torch.uint8)
    else:
        labels = torch.empty(w.N, dtype=torch.int64, device=dev)
        codes = torch.empty((w.N, w.M), dtype=torch.uint8, device=dev)
        for s in range(0, w.N, wl.BASE_CHUNK):
            n = min(wl.BASE_CHUNK, w.N - s)
            labels[s:s + n], codes[s:s + n] = wl.encode(wl.base_chunk(w, comps, s, n), cent, cb)
    order = torch.argsort(labels, stable=True)
    offs = torch.zeros(w.nlist + 1, dtype=torch.int64, device=dev)
    offs[1:] = torch.cumsum(torch.bincount(labels, minlength=w.nlist), 0)
    return w, comps, cent, cb.contiguous(), offs, codes[order].contiguous(), order


def _radii(case, cent, cb, cal):
    """Per-subspace radius that holds `keep` of the entries around the calibration queries'
    residuals (around the queries themselves, on the enlarged spheres, for inner products)."""
    M, _, dsub = cb.shape
    if case["keep"] >= 1.0:
        return np.full(M, np.inf, dtype=np.float32)
    if case["metric"] == 1:
        p = cal
    else:
        d = (cent * cent).sum(1)[None, :] - 2.0 * (cal @ cent.T)
        near = d.topk(min(case["nprobe"], 16), dim=1, largest=False).indices
        p = (cal[:, None, :] - cent[near]).reshape(-1, cal.shape[1])
    p = p.reshape(-1, M, dsub)
    out = np.empty(M, dtype=np.float32)
    for m in range(M):
        d2 = ((p[:, m, None, :] - cb[m][None, :, :]) ** 2).sum(2)
        if case["metric"] == 1:
            d2 = d2 - (cb[m] * cb[m]).sum(1)[None, :]
        d2 = d2.reshape(-1).sort().values
        out[m] = math.sqrt(max(float(d2[int(case["keep"] * d2.numel())]), 0.0))
    return out


def _density_model(case, w, comps, cent, cb):
    """A radius model as `binding.RadiusModel` takes it: 100 x 100 maps of log(1 + density) of
    residual projections, and a straight line from it to the radius that holds `keep` of the
    entries around a residual (the denser the place, the smaller the radius)."""
    G, M = 100, w.M
    x = wl.base_chunk(w, comps, 0, min(w.N, 100_000))
    p = (x - cent[_nearest(x, cent)]).reshape(-1, M, 2)
    lo = p.amin(0)
    per_unit = float(G) / (p.amax(0) - lo).clamp(min=1e-12)
    cell = ((p - lo) * per_unit).floor().clamp(0, G - 1).to(torch.int64)
    flat = (torch.arange(M, device=p.device)[None, :] * G * G + cell[..., 0] * G + cell[..., 1]).reshape(-1)
    count = torch.bincount(flat, minlength=M * G * G).reshape(M, G * G)
    fmap = torch.log1p(count.float() * (per_unit[:, 0] * per_unit[:, 1])[:, None])
    radius = _radii(dict(case, keep=min(case["keep"], 0.5)), cent, cb, wl.queries(w, comps, 64, sub=3))
    top = fmap.amax(1).clamp(min=1e-6).cpu().numpy()
    coef = np.stack([1.5 * radius, -radius / top], 1).astype(np.float32)
    return [lo.cpu().numpy(), per_unit.cpu().numpy(), fmap.reshape(M, G, G).cpu().numpy(), coef, radius]


def _inputs(case, seed):
    w, comps, cent, cb, offs, codes, ids = _index(case, seed)
    q = wl.queries(w, comps)
    radii = _radii(case, cent, cb, wl.queries(w, comps, 64, sub=3))
    model = _density_model(case, w, comps, cent, cb) if case["call"] == "dynamic" else None
    return w, cent, cb, offs, codes, ids, q, radii, model


# ---- one pass -------------------------------------------------------------------------------

def prepare(case, seed):
    w, cent, cb, offs, codes, ids, q, radii, model = _inputs(case, seed)
    index = binding.IvfPqIndex(cent.cpu().numpy(), cb.cpu().numpy(), offs.cpu().numpy(), codes, ids,
                               metric=case["metric"])
    st = dict(case=case, index=index, queries=q, radii=radii)
    Q, k, nprobe = case["Q"], case["k"], case["nprobe"]
    if case["call"] != "noalloc":
        st["workspace"] = index.workspace(Q, nprobe, k)
    st["out"] = (torch.empty((Q, k), dtype=torch.int64, device="cuda"), torch.empty((Q, k), dtype=torch.float32, device="cuda"))
    if case["call"] in ("coarse", "dynamic"):
        st["probes"] = torch.empty((Q, nprobe), dtype=torch.int32, device="cuda")
    if model is not None:
        st["model"] = binding.RadiusModel(index, *model)
        st["query_radii"] = torch.empty((Q, w.M), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    return st


def run(st):
    c, ix, q = st["case"], st["index"], st["queries"]
    if c["call"] == "coarse":
        return ix.coarse(q, c["nprobe"], workspace=st["workspace"], out=st["probes"])
    if c["call"] == "noalloc":
        return ix.search_noalloc(q, c["nprobe"], c["k"], st["radii"], st["out"])
    if c["call"] == "dynamic":
        ix.coarse(q, c["nprobe"], workspace=st["workspace"], out=st["probes"], with_distances=False)
        ix.query_radii(st["model"], q, st["probes"], 1.0, out=st["query_radii"])
        ids, dist = ix.scan_topk(q, st["probes"], c["k"], None, workspace=st["workspace"], mode=c["mode"],
                                 query_radii=st["query_radii"], out=st["out"])
        return st["probes"], st["query_radii"], ids, dist
    return ix.search(q, c["nprobe"], c["k"], st["radii"], workspace=st["workspace"], out=st["out"], mode=c["mode"])


def work(case):
    """What no implementation avoids.  Bytes: queries, centroids, codebooks and results once, and
    the codes of one list per query (each list once: the nearest list has to be ranked; whether
    the other lists have to be read depends on the data).  Operations: the products of every
    query with every centroid, one table per query and one sum over a mean list's codes."""
    Q, D, M, nlist = case["Q"], case["D"], case["M"], case["nlist"]
    mean = case["N"] / nlist
    nbytes = 4.0 * Q * D + 4.0 * nlist * D
    flops = 2.0 * Q * nlist * D
    if case["call"] == "coarse":
        return {"bytes": nbytes + 8.0 * Q * case["nprobe"], "flops": flops}
    nbytes += 4.0 * 256 * D + min(Q, nlist) * mean * M + 12.0 * Q * case["k"]
    flops += Q * (3.0 * 256 * D + mean * M)
    if case["call"] == "dynamic":
        nbytes += 4.0 * Q * (M + case["nprobe"])
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Lists, ids and the 32-bit sums in their stated order are a definition here: every path
    through the library returns the same bits."""
    return "exact"


# ---- the same results in 64 bits ------------------------------------------------------------

def exact(case, seed):
    Q, M, nprobe, k = case["Q"], case["M"], case["nprobe"], case["k"]
    if case["call"] != "coarse" and Q * nprobe * (case["N"] / case["nlist"]) * M > 8e10:
        return None   # over 20 seconds
    w, cent, cb, offs, codes, ids, q, radii, model = _inputs(case, seed)
    ip = case["metric"] == 1
    q, cent, cb = q.double(), cent.double(), cb.double()
    prods = q @ cent.T
    coarse = -prods if ip else (q * q).sum(1)[:, None] - 2.0 * prods + (cent * cent).sum(1)[None, :]
    near = coarse.topk(nprobe, dim=1, largest=False)
    if case["call"] == "coarse":
        return None, near.values
    r2 = torch.from_numpy(radii).to(q.device).double() ** 2
    r2 = r2[None, :].expand(Q, M)
    if model is not None:
        lo, per_unit, fmap, coef, fallback = [torch.from_numpy(np.ascontiguousarray(a)).to(q.device).double() for a in model]
        G = fmap.shape[1]
        x = (q - cent[near.indices[:, 0]]).reshape(Q, M, 2)
        cell = ((x - lo) * per_unit).floor().clamp(0, G - 1).to(torch.int64)
        f = torch.gather(fmap.reshape(M, G * G), 1, (cell[..., 0] * G + cell[..., 1]).T).T
        r = coef[:, 0] + coef[:, 1] * f
        radius = torch.where((r > 0) & torch.isfinite(r), r, fallback[None, :])
        r2 = radius ** 2
    flat = near.indices.reshape(-1)
    by_list = torch.argsort(flat, stable=True)
    ends = torch.cumsum(torch.bincount(flat, minlength=w.nlist), 0).tolist()
    offs_h = offs.tolist()
    best = torch.full((Q, k), float("inf"), dtype=torch.float64, device=q.device)
    for c in range(w.nlist):
        who = by_list[(ends[c - 1] if c else 0):ends[c]] // nprobe
        pts = codes[offs_h[c]:offs_h[c + 1]].long()
        if who.numel() == 0 or pts.shape[0] == 0:
            continue
        x = (q[who] if ip else q[who] - cent[c]).reshape(-1, M, w.dsub)
        total = torch.zeros((who.numel(), pts.shape[0]), dtype=torch.float64, device=q.device)
        if ip and case["mode"] == 0:
            total -= prods[who, c][:, None]
        for m in range(M):
            rm2 = r2[who, m][:, None]
            if ip:
                val = x[:, m] @ cb[m].T
                norm = (x[:, m] ** 2).sum(1)[:, None]
                out, inn = val < 0.5 * (norm - rm2), val < 0.5 * (norm - 0.25 * rm2)
                kept = -torch.maximum(val, 0.5 * (norm - rm2))
            else:
                val = ((x[:, m, None, :] - cb[m][None, :, :]) ** 2).sum(2)
                out, inn = val > rm2, val > 0.25 * rm2
                kept = torch.minimum(val, rm2)
            if case["mode"] == 1:
                kept = out.double()
            elif case["mode"] == 2:
                kept = out.double() + inn.double()
            total += kept[:, pts[:, m]]
        merged = torch.cat([best[who], total], 1)
        best[who] = merged.topk(k, dim=1, largest=False).values
    best = best.sort(1).values
    return (None, radius, None, best) if case["call"] == "dynamic" else (None, best)
