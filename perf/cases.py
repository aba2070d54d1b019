"""The calls that a user of this library makes, as cases that can be timed and checked.

A case names one public entry point and the shape of the scene it is called on.  Scenes are
drawn on the GPU from a seed with the recipe of this repository's synthetic scenes: objects
that recur across the frames of an indoor video, positions scattered around the objects' centres
with depth noise along the camera ray, a few per cent of outliers, unit-norm features.  Sizes are
those of the repository's own workloads (scenes.CONFIGS and bench.py), of its tests, or
products of ordinary frame counts and patch grids.

Kinds of case:
  prune     cp.prune: cost and incremental greedy of one scene, the main path (one call per request)
  select    cp.sgs_select over a cost that is already there (dense, incremental or compact form)
  batch     cp.sgs_select_batch: several requests' greedies in one launch
  local     cp.knn, then cp.sgs_local_select over the neighbour tables
  capacity  cp.fst_capacity: target capacities from each token's nearest neighbours
  lite      cp.lite_select: the alternative without an N x N cost
  literal   cp.sgs_literal_select: the greedy with each step's transport solved
"""
import math

import torch

import paper_2608_13226_amd as cp

DEVICE = "cuda"
WEIGHTS = (1.0, 1.0, 1.0)
C0 = 3.0                     # sum of the weights, the default cost of an uncovered target
KAPPA = cp.DEFAULT_KAPPA
BYTES = {"f32": 4, "bf16": 2}


def listed():
    return [
        # The smallest workload: eight frames of an encoder with narrow float32 features.  Launches
        # and waits between compute units are all there is.
        dict(name="prune_1024x256_f32", kind="prune", n=1024, per_frame=128, d=256, dtype="f32", k=102,
             objects=12, capacity="density"),
        # Sixteen frames of 16 x 16 patches at a vision tower's width.
        dict(name="prune_4096x1152", kind="prune", n=4096, per_frame=256, d=1152, dtype="bf16", k=410,
             objects=40, capacity="density"),
        # Thirty frames of 13 x 13 patches: a token count that no tile divides.
        dict(name="prune_5070x1152", kind="prune", n=5070, per_frame=169, d=1152, dtype="bf16", k=761,
             objects=60, capacity="uniform"),
        # The paper's own efficiency shape: 32 frames of 14 x 14 patches at a language model's width.
        dict(name="prune_6272x3584", kind="prune", n=6272, per_frame=196, d=3584, dtype="bf16", k=628,
             objects=80, capacity="uniform"),
        # The largest full-path workload: 64 frames, a 1 GiB cost.
        dict(name="prune_16384x3584", kind="prune", n=16384, per_frame=256, d=3584, dtype="bf16", k=1638,
             objects=160, capacity="density"),
        # The greedy alone in its default, dense form on a cost that the caller has.
        dict(name="select_dense_4096", kind="select", form="dense", n=4096, per_frame=256, d=1152, dtype="bf16",
             k=410, objects=40, capacity="density"),
        # Four requests of different lengths served together.
        dict(name="batch_4_scenes", kind="batch", count=4, n=6272, n_min=2304, per_frame=196, d=512, dtype="bf16",
             keep=0.1, objects=60, capacity="uniform"),
        # The spatially local greedy with its neighbour tables, 64 neighbours.
        dict(name="local_8192_g64", kind="local", n=8192, per_frame=256, d=512, dtype="bf16", k=819, g=64,
             objects=80, capacity="uniform"),
        # Capacities of the largest full-path workload from 16 neighbours.
        dict(name="capacity_16384x3584", kind="capacity", n=16384, per_frame=256, d=3584, dtype="bf16", nn=16,
             objects=160),
        # The alternative method on the paper's shape and on its own largest workload, whose capacities
        # are those of the 16 nearest neighbours.
        dict(name="lite_6272x3584", kind="lite", n=6272, per_frame=196, d=3584, dtype="bf16", k=628, voxel=0.25,
             objects=80, capacity="uniform"),
        dict(name="lite_32768x3584", kind="lite", n=32768, per_frame=256, d=3584, dtype="bf16", k=3277, voxel=0.25,
             objects=300, capacity="fst"),
        # The greedy with the transport of every step solved: 50 scaling rounds a step.
        dict(name="literal_2048", kind="literal", n=2048, per_frame=256, d=512, dtype="bf16", k=205, rounds=50,
             eps=0.05, objects=30, capacity="uniform"),
    ]


def _log_size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["prune", "select", "batch", "local", "capacity", "lite", "literal"],
                       [8, 2, 2, 2, 2, 4, 1])[0]
    # Token counts: whole frames half of the time, else any number (tokens already dropped upstream).
    hi = {"prune": 16384, "select": 8192, "batch": 6272, "local": 8192, "capacity": 16384, "lite": 32768,
          "literal": 2048}[kind]
    n = _log_size(rng, 1024 if kind == "batch" else 256, hi)
    per = rng.choice([64, 100, 128, 144, 169, 196, 256])
    if rng.random() < 0.5:
        n = min(hi, max(1, round(n / per)) * per)
    dtype = "bf16" if rng.random() < 0.8 or n > 6000 else "f32"
    d = rng.choice([256, 512, 768, 1000, 1024, 1152, 1536, 2048, 3584])
    c = dict(kind=kind, n=n, per_frame=per, d=d, dtype=dtype, objects=max(8, n // 100))
    if kind in ("select", "batch", "local", "literal"):
        c["d"] = 512          # the features only make the cost that these calls are given
    if kind != "capacity":
        c["capacity"] = rng.choice(["uniform", "density"] + (["fst"] if kind == "lite" else []))
    keep = rng.uniform(0.05, 0.2)
    k = max(1, int(round(n * keep)))
    if kind == "prune":
        c["k"] = min(k, 1638)
    elif kind == "select":
        c["form"] = rng.choice(["dense", "incremental", "compact"])
        # A dense step reads the whole cost, so large scenes keep fewer tokens here.
        c["k"] = min(k, max(16, int(6.9e9 / n ** 2))) if c["form"] == "dense" else k
    elif kind == "batch":
        c.update(count=rng.randint(2, 8), n_min=max(256, n // rng.randint(1, 4)), keep=round(min(keep, 0.1), 3))
        c["n"] = min(n, 6272 if c["count"] <= 4 else 4096)
        c["n_min"] = min(c["n_min"], c["n"])
    elif kind == "local":
        c.update(g=rng.choice([16, 32, 50, 64]), k=min(k, 819))
    elif kind == "capacity":
        c["nn"] = rng.choice([8, 12, 16])
    elif kind == "lite":
        c.update(k=k, voxel=rng.choice([0.1, 0.25, 0.5]))
    else:
        c.update(k=min(k, 205), rounds=rng.choice([20, 50]), eps=rng.choice([0.05, 0.1]))
    return c


# ---------------------------------------------------------------------------
# Scenes.

def _scene(case, seed, n=None):
    """Features, positions (metres), frame indices and capacities of a scene, on the GPU."""
    n = case["n"] if n is None else n
    d, per, obj = case["d"], case["per_frame"], case["objects"]
    g = torch.Generator(device=DEVICE).manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, device=DEVICE, generator=g)

    def uniform(*shape):
        return torch.rand(*shape, device=DEVICE, generator=g)

    frames = (n + per - 1) // per
    side = 4.0 + 6.0 * min(1.0, obj / 160.0)
    box = torch.tensor([side, side, 3.0], device=DEVICE)
    low = torch.tensor([-side / 2, -side / 2, 0.0], device=DEVICE)
    protos = normal(obj, d)
    centres = low + box * uniform(obj, 3)
    weight = torch.arange(1, obj + 1, device=DEVICE, dtype=torch.float32) ** -1.2
    # Each object is seen in some of the frames; a frame that sees none sees all.
    seen = (uniform(frames, obj) < min(1.0, 8.0 / frames)).float()
    seen = torch.where(seen.sum(1, keepdim=True) > 0, seen, torch.ones_like(seen))
    frame = (torch.arange(n, device=DEVICE) // per).to(torch.int32)
    which = torch.multinomial(seen * weight, per, replacement=True, generator=g).reshape(-1)[:n]
    outlier = uniform(n) < 0.05
    # Feature: the object's prototype, its look in this frame, and the token's own noise.
    look = 0.2 * normal(frames, min(obj, 32), d)
    feats = protos[which] + look[frame.long(), which % look.shape[1]] + 0.3 * normal(n, d)
    feats = torch.where(outlier[:, None], normal(n, d), feats)
    feats = feats / feats.norm(dim=1, keepdim=True)
    # Position: around the object's centre, moved along the ray from a camera on a 3 m orbit.
    angle = 2 * math.pi * uniform(frames)
    cam = torch.stack([3 * torch.cos(angle), 3 * torch.sin(angle), torch.full_like(angle, 1.5)], 1)[frame.long()]
    pos = centres[which] + 0.25 * normal(n, 3)
    ray = pos - cam
    dist = ray.norm(dim=1, keepdim=True).clamp_min(1e-3)
    pos = cam + ray * (1 + 0.05 * normal(n, 1) / dist)
    pos = torch.where(outlier[:, None], low + box * uniform(n, 3), pos).contiguous()

    feats = feats.to(torch.bfloat16 if case["dtype"] == "bf16" else torch.float32).contiguous()
    out = dict(feats=feats, pos=pos, frame=frame)
    how = case.get("capacity")
    if how == "uniform":
        out["capacity"] = torch.full((n,), 1.0 / n, device=DEVICE)
    elif how == "density":
        count = torch.bincount(which[~outlier], minlength=obj).double()
        v = torch.where(outlier, torch.ones((), device=DEVICE, dtype=torch.float64), count[which].clamp_min(1.0))
        out["capacity"] = (v / v.sum()).float()
    elif how == "fst":
        out["capacity"] = _capacity64(out, min(16, n - 1))[0].float()
    return out


def _gram64(feats, rows=slice(None)):
    f = feats.double()
    f = f / f.norm(dim=1, keepdim=True).clamp_min(1e-300)
    return f[rows] @ f.t()


def _phi(z):
    return torch.log1p(KAPPA * z) / math.log1p(KAPPA)


def _over(x, m):
    return x / m if float(m) > 0 else torch.zeros_like(x)


def _sq_dist64(pos, rows=slice(None)):
    p = pos.double()
    q = p[rows]
    out = (q[:, None, 0] - p[None, :, 0]) ** 2
    out += (q[:, None, 1] - p[None, :, 1]) ** 2
    out += (q[:, None, 2] - p[None, :, 2]) ** 2
    return out


def _cost64(s):
    """Target-major cost of Eq. 8 in 64 bits, and the three maxima."""
    df = (1 - _gram64(s["feats"])).clamp_(0, 2)
    df.fill_diagonal_(0)
    m_f = df.max()
    dx = _sq_dist64(s["pos"]).sqrt_()
    m_x = dx.max()
    t = s["frame"].double()
    m_t = t.max() - t.min()
    c = _over(df, m_f)
    del df
    c += _phi(_over(dx, m_x))
    del dx
    c += _over((t[None, :] - t[:, None]).clamp_min_(0), m_t)     # source (column) later than target (row)
    return c, torch.stack([m_f, m_x, m_t])


def _neighbours(pos, g, drop_self):
    """The g nearest tokens of every token by (distance, index), with or without the token itself."""
    n, out = pos.shape[0], []
    for lo in range(0, n, 2048):
        rows = torch.arange(lo, min(n, lo + 2048), device=DEVICE)
        d2 = _sq_dist64(pos, rows)
        if drop_self:
            d2[torch.arange(len(rows), device=DEVICE), rows] = math.inf
        far = d2.topk(g, dim=1, largest=False).values[:, -1:]
        # Every token up to the g-th distance, the first g of them by (distance, index).
        some = (d2 <= far).sum(1).max()
        idx = (d2 <= far).int().topk(int(some), dim=1).indices.sort(1).values
        key = d2.gather(1, idx)
        out.append(idx.gather(1, key.sort(dim=1, stable=True).indices[:, :g]))
    return torch.cat(out)


def _capacity64(s, nn):
    nb = _neighbours(s["pos"], nn, True)
    n = nb.shape[0]
    d_f = torch.empty(n, nn, device=DEVICE, dtype=torch.float64)
    for lo in range(0, n, 1024):
        f = s["feats"][lo:lo + 1024].double()
        h = s["feats"][nb[lo:lo + 1024]].double()
        dot = (h @ f[:, :, None])[..., 0]
        d_f[lo:lo + 1024] = (1 - dot / (h.norm(dim=2) * f.norm(dim=1, keepdim=True))).clamp_(0, 2)
    p, t = s["pos"].double(), s["frame"].double()
    d_x = (p[:, None] - p[nb]).square().sum(2).sqrt()
    d_t = (t[:, None] - t[nb]).clamp_min(0)
    r = (_over(d_f, d_f.max()) + _over(d_x, d_x.max()) + _over(d_t, d_t.max())).mean(1)
    return (r / r.sum() if float(r.sum()) > 0 else torch.full_like(r, 1.0 / n)), r


# ---------------------------------------------------------------------------
# What a program holds before the call, and the call.

def _batch_sizes(case):
    m, lo, hi = case["count"], case["n_min"], case["n"]
    return [hi - (hi - lo) * i // max(1, m - 1) for i in range(m)]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        sizes = _batch_sizes(case)
        scenes = [_scene(case, seed * 16 + i, n) for i, n in enumerate(sizes)]
        return dict(case=case, costs=[_cost64(s)[0].float() for s in scenes],
                    capacities=[s["capacity"] for s in scenes],
                    ks=[max(1, int(n * case["keep"])) for n in sizes])
    s = _scene(case, seed)
    if kind in ("select", "local", "literal"):
        s["cost"] = _cost64(s)[0].float()
        del s["feats"]
    return dict(case=case, **s)


def _sgs(r):
    return dict(selected=r.selected, gain=r.gain, objective=r.objective, assign=r.assign)


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "prune":
        cost, maxima, r = cp.prune(s["feats"], s["pos"], s["frame"], s["capacity"], c["k"])
        return dict(cost=cost, maxima=maxima, **_sgs(r))
    if kind == "select":
        return _sgs(cp.sgs_select(s["cost"], s["capacity"], c["k"], incremental=c["form"] != "dense",
                                  compact=c["form"] == "compact"))
    if kind == "batch":
        return [_sgs(r) for r in cp.sgs_select_batch(s["costs"], s["capacities"], s["ks"])]
    if kind == "local":
        nb = cp.knn(s["pos"], c["g"])
        return dict(neighbours=nb, **_sgs(cp.sgs_local_select(s["cost"], s["capacity"], nb, c["k"])))
    if kind == "capacity":
        v, r = cp.fst_capacity(s["feats"], s["pos"], s["frame"], c["nn"])
        return dict(capacity=v, score=r)
    if kind == "lite":
        r = cp.lite_select(s["feats"], s["pos"], s["frame"], s["capacity"], c["k"], voxel_size=c["voxel"],
                           token_cost=True)
        return dict(selected=r.selected, group=r.group, objective=r.objective, token_cost=r.token_cost)
    r = cp.sgs_literal_select(s["cost"], s["capacity"], c["k"], epsilon=c["eps"], rounds=c["rounds"])
    return dict(selected=r.selected, score=r.score, residual=r.residual, objective=r.objective)


def work(case):
    """Inputs read once, outputs written once, and the arithmetic of the definition's cheapest form:
    the Gram of unique pairs, one pass of the greedy's terms over the cost (later steps only touch
    the targets whose best cost falls, a share of it)."""
    kind, n, d = case["kind"], case["n"], case["d"]
    feats = n * d * BYTES[case["dtype"]] + n * 16 + n * 4
    k = case.get("k", 0)
    picks = 20 * k + 4 * n
    if kind == "prune":
        return dict(bytes=feats + 4 * n * n + picks, flops=n * (n + 1) * d + 3 * n * n)
    if kind == "select":
        return dict(bytes=4 * n * n + 4 * n + picks, flops=3 * n * n)
    if kind == "batch":
        sizes = _batch_sizes(case)
        return dict(bytes=sum(4 * m * m + 8 * m + 20 * int(m * case["keep"]) for m in sizes),
                    flops=sum(3 * m * m for m in sizes))
    if kind == "local":
        # The winners' costs to every target and the neighbours' costs; gains over the neighbours.
        return dict(bytes=4 * n * k + 8 * n * case["g"] + 16 * n + picks,
                    flops=8 * n * n // 2 + 3 * n * case["g"])
    if kind == "capacity":
        return dict(bytes=feats + 12 * n, flops=8 * n * n // 2 + 4 * n * case["nn"] * d)
    if kind == "lite":
        # Groups of n / k tokens on average, unique pairs.
        return dict(bytes=feats + 4 * k + 12 * n, flops=n * (n / k) * d)
    l2 = k * (k + 1) / 2
    return dict(bytes=4 * n * n + 4 * n + 20 * k, flops=4.0 * n * l2 * case["rounds"] + 2.0 * n * n)


def tolerance(case):
    """Several times what exact() and the library were seen to differ by, per kind.  Picks whose gains
    agree to rounding may change places, and every later place can shift with them."""
    kind = case["kind"]
    if kind == "prune":       # float32 cost and sums over its entries: 4e-7 seen, more for small scenes
        return dict(rel=4e-6, max=1e-4, differ=0.01)
    if kind in ("select", "batch"):     # float32 differences, sums in float64 or finer: 2e-9 seen
        return dict(rel=2e-8, max=1e-7, differ=0.01)
    if kind == "local":       # float64 terms in exact sums: no difference seen
        return dict(rel=1e-12, max=1e-11, differ=0.001)
    if kind == "capacity":    # float64 scores, one rounding to float32: 3e-8 seen
        return dict(rel=1e-7, max=5e-7)
    if kind == "lite":        # float32 dot products: 7e-7 seen; prototypes of nearly equal cost
        return dict(rel=3e-6, max=1e-5, differ=0.005)
    return dict(rel=1e-12, max=1e-11, differ=0.01)      # float64 throughout: 2e-16 seen


# ---------------------------------------------------------------------------
# The same in 64 bits, in plain torch.

def _first_max(x):
    return (x == x.max()).nonzero()[0, 0]


def _greedy64(c, v, k, neighbours=None):
    """Greedy coverage over the target-major cost c."""
    n = c.shape[0]
    c, v = c.double(), v.double()
    b = torch.full((n,), C0, device=DEVICE, dtype=torch.float64)
    assign = torch.full((n,), -1, device=DEVICE, dtype=torch.int32)
    if neighbours is not None:
        nb = neighbours.long()
        cn, vn = c[nb, torch.arange(n, device=DEVICE)[:, None]], v[nb]

        def gains():
            return (vn * (b[nb] - cn).clamp_min(0)).sum(1)
    full = torch.zeros(n, device=DEVICE, dtype=torch.float64)
    for lo in range(0, n, 2048):
        full += v[lo:lo + 2048] @ (C0 - c[lo:lo + 2048]).clamp_min_(0)
    gain = gains() if neighbours is not None else full
    out = torch.zeros(n, device=DEVICE, dtype=torch.bool)
    picks, won, left = [], [], []
    for _ in range(k):
        s = _first_max(gain.masked_fill(out, -1.0))
        picks.append(s)
        won.append(gain[s].clone())
        out[s] = True
        col = c[:, s]
        hit = (col < b).nonzero()[:, 0]
        if neighbours is None:
            for h in hit.split(2048):
                rows, old, new = c[h], b[h][:, None], col[h][:, None]
                gain -= v[h] @ ((old - rows).clamp_min(0) - (new - rows).clamp_min_(0))
        b[hit] = col[hit]
        assign[hit] = s.int()
        left.append(v @ b)
        if neighbours is not None:
            gain = gains()
    return dict(selected=torch.stack(picks).int(), gain=torch.stack(won), objective=torch.stack(left), assign=assign)


def _lite64(case, s):
    n, k = case["n"], case["k"]
    p = s["pos"].double()
    scale = 256.0 / float(torch.tensor(case["voxel"], dtype=torch.float32))
    q = ((p - p.min(0).values) * scale).floor().clamp_(0, 2 ** 21 - 1).long()
    key = torch.zeros(n, device=DEVICE, dtype=torch.long)
    for i in range(21):
        for a in range(3):
            key |= ((q[:, a] >> i) & 1) << (3 * i + a)
    order = key.sort(stable=True).indices
    units = (s["capacity"].double() * 2.0 ** 40).floor().long()[order].tolist()
    total, before, at, groups = sum(units), 0, 0, [0] * n
    for i in range(1, n):
        before += units[i - 1]
        if at < k - 1 and (k * before >= (at + 1) * total or n - i == k - 1 - at):
            at += 1
        groups[i] = at
    groups = torch.tensor(groups, device=DEVICE)
    size = torch.bincount(groups, minlength=k)
    start = size.cumsum(0) - size
    group = torch.empty_like(groups)
    group[order] = groups
    vox, t, v = q >> 8, s["frame"].double(), s["capacity"].double()
    # Blocks of groups, each padded to its largest; first the maxima, then the costs.
    most, blocks, maxima, lo = 6e8, [], torch.zeros(3, device=DEVICE, dtype=torch.float64), 0
    sizes = size.tolist()
    while lo < k:
        hi, m = lo, 0
        while hi < k and (hi - lo + 1) * max(m, sizes[hi]) * (case["d"] + max(m, sizes[hi])) <= most:
            m = max(m, sizes[hi])
            hi += 1
        hi = max(hi, lo + 1)
        m = max(sizes[lo:hi])
        col = torch.arange(m, device=DEVICE)[None, :]
        there = col < size[lo:hi, None]
        idx = order[(start[lo:hi, None] + col).clamp_max(n - 1)]
        f = s["feats"][idx].double()
        f = f / f.norm(dim=2, keepdim=True).clamp_min(1e-300)
        d_f = (1 - torch.bmm(f, f.transpose(1, 2).contiguous())).clamp_(0, 2)
        d_f.diagonal(dim1=1, dim2=2).zero_()
        d_x = (p[idx][:, :, None] - p[idx][:, None]).square().sum(3).sqrt()
        d_t = (t[idx][:, :, None] - t[idx][:, None]).clamp_min(0)
        pair = there[:, :, None] & there[:, None]
        near = pair & ((vox[idx][:, :, None] - vox[idx][:, None]).abs() <= 1).all(3)
        maxima = torch.maximum(maxima, torch.stack([x[near].max() for x in (d_f, d_x, d_t)]))
        blocks.append((idx, there, pair, near, d_f, d_x, d_t))
        lo = hi
    token = torch.zeros(n, device=DEVICE, dtype=torch.float64)
    selected, objective = [], torch.zeros((), device=DEVICE, dtype=torch.float64)
    for idx, there, pair, near, d_f, d_x, d_t in blocks:
        c = _over(d_f, maxima[0]) + _phi(_over(d_x, maxima[1])) + _over(d_t, maxima[2])
        c = torch.where(near, c, torch.full_like(c, C0)) * pair
        cost = (c * v[idx][:, None, :]).sum(2)
        token[idx[there]] = cost[there]
        cost = cost.masked_fill(~there, math.inf)
        best = cost.min(1, keepdim=True).values
        selected.append(torch.where(cost == best, idx, n).min(1).values)
        objective += best.sum()
    return dict(selected=torch.cat(selected).int(), group=group.int(), objective=objective[None], token_cost=token)


def _literal64(case, s):
    n, k, rounds = case["n"], case["k"], case["rounds"]
    eps = float(torch.tensor(case["eps"], dtype=torch.float32))
    c, v = s["cost"].t().double().contiguous(), s["capacity"].double()      # source-major
    e = torch.exp(-c / eps)
    u = 1.0 / k
    picks, score, mass = [], [], []
    out = torch.zeros(n, device=DEVICE, dtype=torch.bool)

    def solve(rows):
        b = torch.ones(n, device=DEVICE, dtype=torch.float64)
        for _ in range(rounds):
            a = u / (rows @ b)
            t = a @ rows
            b = torch.where(t > 0, (v / t).clamp_max(1.0), 1.0)
        return a, b, t

    for step in range(k):
        r = v
        if step:
            _, b, t = solve(e[torch.stack(picks)])
            r = (v - b * t).clamp_min(0)
        x = (c @ r).masked_fill(out, math.inf)
        pick = (x == x.min()).nonzero()[0, 0]
        picks.append(pick)
        score.append(x[pick])
        mass.append(r.sum())
        out[pick] = True
    at = torch.stack(picks)
    a, b, _ = solve(e[at])
    cost = (a[:, None] * e[at] * b * c[at]).sum()
    return dict(selected=at.int(), score=torch.stack(score), residual=torch.stack(mass), objective=cost[None])


def exact(case, seed):
    kind = case["kind"]
    s = prepare(case, seed)
    if kind == "prune":
        c, maxima = _cost64(s)
        return dict(cost=c, maxima=maxima, **_greedy64(c, s["capacity"], case["k"]))
    if kind == "select":
        return _greedy64(s["cost"], s["capacity"], case["k"])
    if kind == "batch":
        return [_greedy64(c, v, k) for c, v, k in zip(s["costs"], s["capacities"], s["ks"])]
    if kind == "local":
        nb = _neighbours(s["pos"], case["g"], False)
        return dict(neighbours=nb.int(), **_greedy64(s["cost"], s["capacity"], case["k"], nb))
    if kind == "capacity":
        v, r = _capacity64(s, case["nn"])
        return dict(capacity=v, score=r)
    return _lite64(case, s) if kind == "lite" else _literal64(case, s)
