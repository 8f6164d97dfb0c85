"""The workloads this library is timed on, through the entry points of its Python binding.

Every case is one of five kinds of call, each as a program that clusters vectors makes it:

  lloyd   fk_lloyd_iter: a fit of `iters` iterations from given starting centroids
  assign  fk_assign: new points against finished centroids (with the distances, where asked for)
  update  fk_update: new centroids from a given assignment
  ooc     fk_lloyd_ooc: a fit whose points stay in pinned host memory

The sizes are the configurations of paper_2603_09229_amd/workloads.py, the shapes of the tests
(widths and counts that are no multiple of anything) and generic ones between them.  Workspaces
and result buffers are kept from call to call, as a program that calls more than once keeps them.

Points are drawn from Gaussian mixtures with as many components as centroids.  A fit starts from
one row of each component, which is what a seeding such as k-means++ gives: no point then lies
within rounding of the border of two clusters, and correct implementations agree on every
assignment after several iterations too.  `assign` cases take further points of the mixture as
centroids, some components with several and some with none, so that many points have several
centroids at nearly equal distances.
"""
import math

import torch

from paper_2603_09229_amd import binding as fk

_TYPES = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}
# spread of the mixture's centres and of the points around them, as the workloads have them
_SPREAD = {"fp32": (10.0, 1.0), "fp16": (4.0, 1.0), "bf16": (1.0, 0.5)}


def _case(name, kind, dtype, B, N, d, K, iters=1, zipf=0.0, min_dist=False, chunk=0):
    return {"name": name, "kind": kind, "dtype": dtype, "B": B, "N": N, "d": d, "K": K, "iters": iters, "zipf": zipf,
            "min_dist": min_dist, "chunk": chunk}


def listed():
    return [
        # the small fp32 configuration: a fit that is over in a fraction of a millisecond
        _case("fit_f32_tiny", "lloyd", "fp32", 1, 16384, 64, 64, iters=10),
        # the headline configuration: a million descriptors, a thousand clusters
        _case("fit_f16_mid", "lloyd", "fp16", 1, 1 << 20, 128, 1024, iters=4),
        # token clustering: many independent problems in one call
        _case("fit_bf16_batched", "lloyd", "bf16", 32, 32768, 128, 256, iters=10),
        # very many points, few clusters of very unequal sizes
        _case("fit_f16_skewed", "lloyd", "fp16", 1, 1 << 24, 64, 16, iters=4, zipf=1.2),
        # full-precision features, medium size
        _case("fit_f32_mid", "lloyd", "fp32", 1, 300000, 96, 400, iters=3),
        # nothing is a multiple of anything: rows of 100 features, several instances
        _case("fit_bf16_ragged", "lloyd", "bf16", 3, 70001, 100, 333, iters=5),
        # serving: a request's vectors against a codebook
        _case("assign_bf16_small", "assign", "bf16", 1, 1000, 128, 1024),
        # labelling a collection with a large codebook, distances wanted (residual quantisation)
        _case("assign_f16_large", "assign", "fp16", 1, 1 << 20, 128, 8192, min_dist=True),
        # wide embeddings
        _case("assign_f16_wide", "assign", "fp16", 1, 131072, 512, 4096),
        # wide embeddings in full precision
        _case("assign_f32_wide", "assign", "fp32", 1, 65536, 256, 512, min_dist=True),
        # new centroids of a large collection from an assignment in hand
        _case("update_f16_large", "update", "fp16", 1, 1 << 23, 128, 4096),
        # points beyond the device memory granted: chunks streamed from the host
        _case("ooc_f16", "ooc", "fp16", 1, 1 << 21, 128, 1024, iters=2, chunk=1 << 18),
    ]


def _between(rng, lo, hi):
    """A whole number between lo and hi, even over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    while True:
        kind = rng.choice(["lloyd", "lloyd", "lloyd", "assign", "assign", "update", "ooc"])
        dtype = rng.choice(["fp32", "fp16", "bf16"])
        B = rng.choice([1, 1, 1, 2, 5, 32]) if kind != "ooc" else 1
        N = _between(rng, 1000, 1 << 24)
        # widths: a round one, or any
        d = rng.choice([32, 64, 128, 256, 512]) if rng.random() < 0.5 else _between(rng, 16, 512)
        K = _between(rng, 8, 8192)
        iters = rng.choice([1, 2, 4, 10]) if kind == "lloyd" else rng.choice([1, 2]) if kind == "ooc" else 1
        zipf = rng.choice([0.0, 0.0, 1.2]) if kind != "assign" else 0.0
        min_dist = kind == "assign" and rng.random() < 0.5
        chunk = -(-N // rng.choice([2, 3, 5, 8])) if kind == "ooc" else 0
        size = 4 if dtype == "fp32" else 2
        points = B * N
        terms = points * K * d * iters
        if points * d * size > 1 << 31 or points * d * size * iters > 6 << 30 or (K * 2 > N and kind != "assign") or points > 1 << 24:
            continue
        if terms > (2e10 if dtype == "fp32" else 4e11):
            continue
        if kind == "ooc" and points * d * size * iters > 1 << 30:
            continue
        return {"kind": kind, "dtype": dtype, "B": B, "N": N, "d": d, "K": K, "iters": iters, "zipf": zipf, "min_dist": min_dist, "chunk": chunk}


def _draw_points(case, seed):
    """On the GPU: X [B,N,d] of the stored type, the component of every point [B,N] int32, and K more
    points of each instance [B,K,d], the centroids of `assign` cases."""
    B, N, d, K = case["B"], case["N"], case["d"], case["K"]
    t = _TYPES[case["dtype"]]
    between, around = _SPREAD[case["dtype"]]
    between *= max(1.0, 48 / d)       # narrow rows: components as well apart as in wide ones
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    weight = torch.arange(1, K + 1, dtype=torch.float64).pow(-case["zipf"])
    upto = (weight / weight.sum()).cumsum(0).float().cuda()
    X = torch.empty((B, N, d), dtype=t, device="cuda")
    label = torch.empty((B, N), dtype=torch.int32, device="cuda")
    book = torch.empty((B, K, d), dtype=t, device="cuda")
    step = max(1, (1 << 28) // d)
    for b in range(B):
        centre = torch.randn((K, d), generator=g, device="cuda") * between
        of = torch.searchsorted(upto, torch.rand((N,), generator=g, device="cuda"), right=True).clamp_(max=K - 1)
        if N >= K:
            of[:K] = torch.randperm(K, generator=g, device="cuda")  # the first K points: one of each component
        for r in range(0, N, step):
            part = of[r : r + step]
            X[b, r : r + step] = (torch.randn((part.numel(), d), generator=g, device="cuda") * around + centre[part]).to(t)
        label[b] = of.int()
        of = torch.randint(0, K, (K,), generator=g, device="cuda")
        book[b] = (torch.randn((K, d), generator=g, device="cuda") * around + centre[of]).to(t)
    return X, label, book


def prepare(case, seed):
    B, N, d, K, kind = case["B"], case["N"], case["d"], case["K"], case["kind"]
    X, label, book = _draw_points(case, seed)
    t = X.dtype
    s = {"case": case}
    if kind == "assign":
        s["X"], s["C"] = X, book
        s["out"] = torch.empty((B, N), dtype=torch.int32, device="cuda")
        s["ws"] = fk.make_workspace(B, N, d, K, t, X.device)
        return s
    s["C0"] = X[:, :K].float().contiguous()
    s["C"] = torch.empty_like(s["C0"])
    if kind == "lloyd":
        s["X"] = X
        s["lp"] = torch.empty((B, K, d), dtype=t, device="cuda")
        s["out"] = torch.empty((B, N), dtype=torch.int32, device="cuda")
        s["counts"] = torch.empty((B, K), dtype=torch.int32, device="cuda")
        s["ws"] = fk.make_workspace(B, N, d, K, t, X.device)
    elif kind == "update":
        s["X"], s["label"] = X, label
        s["ws"] = fk.make_workspace(B, N, d, K, t, X.device)
    else:
        host = torch.empty((N, d), dtype=t, pin_memory=True)
        host.copy_(X[0])
        s["X"], s["C0"], s["C"] = host, s["C0"][0].contiguous(), s["C"][0].contiguous()
        s["ws"] = torch.empty(fk.fk_ooc_workspace_bytes(case["chunk"], d, K, t), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "assign":
        got = fk.fk_assign(s["X"], s["C"], min_dist=case["min_dist"], ws=s["ws"], out=s["out"])
        return list(got) if case["min_dist"] else [got]
    if kind == "update":
        return list(fk.fk_update(s["X"], s["label"], s["C0"], ws=s["ws"]))
    s["C"].copy_(s["C0"])
    if kind == "lloyd":
        out, counts, lp = fk.fk_lloyd_iter(s["X"], s["C"], case["iters"], ws=s["ws"], C_lp=s["lp"], assign=s["out"], counts=s["counts"])
        return [s["C"], lp, counts, out]
    out, counts = fk.fk_lloyd_ooc(s["X"], s["C"], case["iters"], dev_ws=s["ws"], chunk_rows=case["chunk"])
    return [s["C"], counts, out]


def work(case):
    B, N, d, K, kind, iters = case["B"], case["N"], case["d"], case["K"], case["kind"], case["iters"]
    size = 4 if case["dtype"] == "fp32" else 2
    points, centroids = B * N * d * size, B * K * d * size
    if kind == "assign":
        return {"bytes": points + centroids + B * N * (8 if case["min_dist"] else 4), "flops": 2 * B * N * K * d}
    if kind == "update":
        return {"bytes": points + B * N * 4 + B * K * (d * (8 + size) + 4), "flops": B * N * d}
    # every iteration has to see every point; centroids, counts and assignment leave once
    return {"bytes": iters * points + B * K * (d * 8 + 4) + (centroids if kind == "lloyd" else 0) + B * N * 4,
            "flops": iters * (2 * B * N * K * d + B * N * d)}


def tolerance(case):
    """About four times what the path is off from `exact` on the listed cases and forty drawn ones."""
    kind, dtype = case["kind"], case["dtype"]
    if dtype == "fp32":
        # sums and distances in 32 bits: up to 2.5e-7 off, 1.1e-6 in a single element
        return {"rel": 1e-6, "max": 5e-6, "differ": 1e-5}
    if kind == "assign":
        # scores are compared to 2^-19: up to 5e-6 of the rows go to the other of two centroids at
        # equal distance, the distances are 1.3e-6 off, 5.6e-6 in a single element
        return {"rel": 5e-6, "max": 2.5e-5, "differ": 2e-5}
    # the 32-bit centroids are 1.3e-7 off; sums in another order move the rounded copy by one place
    # in the few elements that lie on the edge of it
    return {"rel": 1e-4, "max": 1.6e-2 if dtype == "bf16" else 2e-3, "differ": 1e-5}


def _nearest(x, c):
    """(index of the nearest row of c, squared distance to it) for every row of x, in 64 bits."""
    c = c.double()
    half = (c * c).sum(1) * 0.5
    step = max(1, (1 << 28) // c.shape[0])
    at, dist = [], []
    for r in range(0, x.shape[0], step):
        part = x[r : r + step].double()
        best, k = (part @ c.t() - half).max(1)
        at.append(k)
        dist.append((part * part).sum(1) - 2 * best)
    return torch.cat(at), torch.cat(dist).clamp_(min=0)


def _means(x, at, before):
    """(means of the rows of x by cluster, rows of `before` where there are none; counts), in 64 bits."""
    K, d = before.shape
    total = torch.zeros((K, d), dtype=torch.float64, device="cuda")
    step = max(1, (1 << 27) // max(K, d))
    for r in range(0, x.shape[0], step):
        member = torch.zeros((K, min(step, x.shape[0] - r)), dtype=torch.float64, device="cuda")
        member.scatter_(0, at[None, r : r + step], 1.0)
        total += member @ x[r : r + step].double()
    n = torch.bincount(at, minlength=K)
    return torch.where((n > 0)[:, None], total / n.clamp(min=1)[:, None], before), n


def exact(case, seed):
    K, kind = case["K"], case["kind"]
    X, label, book = _draw_points(case, seed)
    t = X.dtype
    if kind == "assign":
        got = [_nearest(X[b], book[b]) for b in range(case["B"])]
        at = torch.stack([a for a, _ in got]).int()
        return [at, torch.stack([m for _, m in got])] if case["min_dist"] else [at]
    C, n, at = [], [], []
    for b in range(case["B"]):
        c = X[b, :K].double()
        if kind == "update":
            c, m = _means(X[b], label[b].long(), c)
            C, n = C + [c], n + [m]
            continue
        for _ in range(case["iters"]):
            a, _ = _nearest(X[b], c.float().to(t))
            c, m = _means(X[b], a, c)
        C, n, at = C + [c], n + [m], at + [a]
    C, n = torch.stack(C), torch.stack(n).int()
    if kind == "update":
        return [C, None, n]
    at = torch.stack(at).int()
    return [C, None, n, at] if kind == "lloyd" else [C[0], n[0], at[0]]
