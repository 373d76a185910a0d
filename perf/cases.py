"""The work that users of the tree force have it do, as cases that can be timed and checked.

A case is a dict of plain values.  Its "path" says which calls of the package one pass makes:

  short  treepm_build, treepm_walk, treepm_force_short on one box (FP32 or FP64 kernel, fixed
         or distance-dependent opening angle, monopole or quadrupole cells)
  long   treepm_force_long on a built box (the particle mesh)
  step   a whole time step: build, walk, short-range force, long-range force accumulated onto
         it, the shared step of eq. (7), kick and drift
  batch  treepm_build of several boxes, then one treepm_force_short_batch over them
  serve  requests on several boxes submitted to an ensemble server from host memory, and
         polled until all results are back on the host

Boxes are the unit cube, uniform or clustered (half of the particles in NFW halos of
concentration 10), in random input order, with mesh = 1/round(N^(1/3)) unless the case gives
the mesh, r_cut = 3 mesh and eps = mesh/20.
"""
import math
import time

import torch

import paper_0910_0121_amd as tp

K_PP = 38  # flops of one pair interaction (FMA = 2; add, mul, rsqrt, sqrt = 1)
_EXACT_MOST = 2_200_000  # particles up to which exact() of a tree force stays within seconds


def listed():
    short = dict(path="short", kind="nfw", masses="equal", n_leaf=10, theta=0.5, precision="fp32",
                 opening="fixed", quadrupole=False)
    return [
        # The smallest calls: a box of a few thousand particles, where launches and the host's
        # waits for small results are all there is.
        dict(short, name="short_3k", n=3000, kind="uniform", n_crit=64),
        # The plain-method box: 32^3 uniform particles.
        dict(short, name="short_32k", n=32768, kind="uniform", n_crit=64),
        # A mid-sized clustered box of an odd size, as an ensemble of boxes holds.
        dict(short, name="short_700k", n=700001, n_crit=256),
        # The headline workload: the 256^3 clustered box at theta = 0.5.
        dict(short, name="short_256c", n=256 ** 3, n_crit=256),
        # The FP64 kernel on the 128^3 clustered box: reference forces and accuracy studies.
        dict(short, name="fp64_128c", n=128 ** 3, n_crit=128, precision="fp64"),
        # Quadrupole cells, which buy accuracy at a larger opening angle; masses over three
        # decades.
        dict(short, name="quad_1m", n=1000003, n_crit=256, theta=0.7, quadrupole=True,
             masses="mixed"),
        # The distance-dependent opening angle of eq. (12), theta_0 = 0.3 capped at 0.5.
        dict(short, name="theta_r_500k", n=500009, n_crit=192, theta=0.3, opening="distance"),
        # The long-range half of the force on the headline box: once per step.
        dict(path="long", name="long_256c", kind="nfw", masses="equal", n=256 ** 3, n_crit=256,
             mesh_n=256),
        # A whole time step of a smaller simulation.
        dict(path="step", name="step_250k", kind="nfw", masses="equal", n=250007, n_crit=256,
             theta=0.5, mesh_n=64),
        # Several boxes at once through shared launches.
        dict(path="batch", name="batch_8", kind="nfw", boxes=8, n_min=20000, n_max=120000,
             n_crit=256, theta=0.5),
        # The ensemble server: requests on boxes of mixed sizes from host memory.
        dict(path="serve", name="serve_12", kind="nfw", boxes=12, n_min=32768, n_max=400000,
             n_crit=256, theta=0.5),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["short"] * 4 + ["fp64", "quad", "long", "step", "batch", "serve"])
    kind = rng.choice(["nfw", "nfw", "uniform"])
    masses = rng.choice(["equal", "equal", "mixed"])
    n_crit = rng.choice([64, 128, 192, 256, 300])
    theta = rng.choice([0.4, 0.5, 0.6, 0.7])
    if path in ("short", "fp64", "quad"):
        top = {"short": 12_000_000, "fp64": 1_500_000, "quad": 1_500_000}[path]
        distance = path == "short" and rng.random() < 0.25
        return dict(path="short", kind=kind, masses=masses, n=_log_uniform(rng, 2500, top),
                    n_crit=n_crit, n_leaf=rng.choice([8, 10, 16]),
                    theta=0.3 if distance else theta,
                    precision="fp64" if path == "fp64" else "fp32",
                    opening="distance" if distance else "fixed", quadrupole=path == "quad")
    if path == "long":
        return dict(path="long", kind=kind, masses=masses, n=_log_uniform(rng, 2500, 12_000_000),
                    n_crit=n_crit, mesh_n=rng.choice([16, 32, 64, 128, 256]))
    if path == "step":
        mesh_n = rng.choice([32, 64, 128])
        n = int(mesh_n ** 3 * rng.uniform(0.5, 1.5)) | 1
        return dict(path="step", kind=kind, masses=masses, n=n, n_crit=n_crit, theta=theta,
                    mesh_n=mesh_n)
    lo = _log_uniform(rng, 5000, 50000)
    hi = lo + _log_uniform(rng, 10000, 300000)
    return dict(path=path, kind=kind, boxes=rng.randint(3, 12), n_min=lo, n_max=hi,
                n_crit=n_crit, theta=theta)


# ------------------------------------------------------------------------------- inputs


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _wrap(v):
    v = v - torch.floor(v)
    v[v >= 1.0] = 0.0
    return v


def _positions(n, kind, g):
    """(3, n) positions in [0, 1): uniform, or half in NFW halos (one per 8,400 particles, halo
    masses from dN/dM ~ M^-1.9 over two decades, truncated at r_200)."""
    def u(*size):
        return torch.rand(*size, generator=g, device="cuda", dtype=torch.float64)

    if kind == "uniform":
        return u(3, n)
    nh = max(1, round(n / 8400))
    mh = (1.0 - u(nh) * (1.0 - 100.0 ** -0.9)) ** (-1.0 / 0.9)
    count = torch.floor(mh / mh.sum() * (0.5 * n)).to(torch.int64)
    inside = int(count.sum())
    r200 = (3.0 * (count.double() / n) / (800.0 * math.pi)) ** (1.0 / 3.0)
    halo = torch.repeat_interleave(torch.arange(nh, device="cuda"), count)
    # radius from the enclosed mass mu(x) / mu(10), mu(x) = ln(1 + x) - x / (1 + x)
    xs = torch.logspace(-4, 1, 8192, device="cuda", dtype=torch.float64)
    mu = torch.log1p(xs) - xs / (1.0 + xs)
    mu = mu / mu[-1].clone()
    t = u(inside)
    k = torch.searchsorted(mu, t).clamp(1, xs.numel() - 1)
    f = ((t - mu[k - 1]) / (mu[k] - mu[k - 1])).clamp(0.0, 1.0)
    r = (xs[k - 1] + f * (xs[k] - xs[k - 1])) * 0.1 * r200[halo]
    ct = 2.0 * u(inside) - 1.0
    ph = 2.0 * math.pi * u(inside)
    st = torch.sqrt(1.0 - ct * ct)
    centre = u(3, nh)
    p = centre[:, halo] + r * torch.stack([st * torch.cos(ph), st * torch.sin(ph), ct])
    p = _wrap(torch.cat([p, u(3, n - inside)], dim=1))
    return p[:, torch.randperm(n, generator=g, device="cuda")].contiguous()


def _box(n, kind, masses, seed):
    """Positions (3, n) and masses (n) of one box: total mass 1, masses equal or spread over
    three decades."""
    g = _generator(seed)
    p = _positions(n, kind, g)
    if masses == "equal":
        m = torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
    else:
        m = 10.0 ** (3.0 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64))
        m = m / m.sum()
    return p, m


def _params(case, n):
    mesh = 1.0 / case.get("mesh_n", round(n ** (1.0 / 3.0)))
    return tp.make_params(
        L=1.0, mesh=mesh, r_cut=3.0 * mesh, eps=mesh / 20.0, theta=case.get("theta", 0.5),
        n_leaf=case.get("n_leaf", 10), n_crit=case["n_crit"],
        precision=tp.TREEPM_FP64 if case.get("precision") == "fp64" else tp.TREEPM_FP32,
        opening=(tp.TREEPM_OPEN_DISTANCE if case.get("opening") == "distance"
                 else tp.TREEPM_OPEN_FIXED),
        theta_max=0.5 if case.get("opening") == "distance" else 0.0,
        quadrupole=1 if case.get("quadrupole") else 0)


def _sizes(case, seed):
    g = torch.Generator()
    g.manual_seed(int(seed))
    lo, hi = math.log(case["n_min"]), math.log(case["n_max"])
    u = torch.rand(case["boxes"], generator=g, dtype=torch.float64).tolist()
    return [int(round(math.exp(lo + v * (hi - lo)))) for v in u]


def _boxes(case, seed):
    """(n, positions, masses) of every box of a case."""
    if case["path"] in ("batch", "serve"):
        # the sizes of an ensemble's boxes are the case's; their particles come from the seed
        sizes = _sizes(case, 999)
    else:
        sizes = [case["n"]]
    return [(n,) + _box(n, case["kind"], case.get("masses", "equal"), 1000 * seed + b)
            for b, n in enumerate(sizes)]


class _Box:
    """One box and its context, with the output arrays a program keeps for it."""

    def __init__(self, case, n, p, m):
        self.n, self.p, self.m = n, p, m
        self.params = _params(case, n)
        self.ctx = tp.treepm_create(self.params, 0)
        dtype = torch.float64 if case.get("precision") == "fp64" else torch.float32
        self.acc = torch.empty(3, n, dtype=dtype, device="cuda")

    def build(self):
        tp.treepm_build(self.ctx, self.p[0], self.p[1], self.p[2], self.m)

    def __del__(self):
        if getattr(self, "ctx", None):
            tp.treepm_destroy(self.ctx)


class _Server:
    def __init__(self, case, boxes):
        self.boxes = []
        for n, p, m in boxes:
            host = [a.cpu().numpy() for a in (p[0], p[1], p[2], m)]
            out = [torch.empty(n, dtype=torch.float32).numpy() for _ in range(3)]
            self.boxes.append((_params(case, n), host, out))
        self.ens = tp.treepm_ens_create(0, 16 << 30, 8)

    def __del__(self):
        if getattr(self, "ens", None):
            tp.treepm_ens_destroy(self.ens)


def prepare(case, seed):
    boxes = _boxes(case, seed)
    if case["path"] == "serve":
        return case, _Server(case, boxes)
    state = [_Box(case, *b) for b in boxes]
    if case["path"] == "long":
        state[0].build()
    if case["path"] == "step":
        b = state[0]
        b.p0 = b.p
        b.p = b.p0.clone()
        b.v0 = _velocities(b.n, seed)
        b.v = b.v0.clone()
    torch.cuda.synchronize()
    return case, state


def _velocities(n, seed):
    return 2.0 * torch.randn(3, n, generator=_generator(7777 + seed), device="cuda",
                             dtype=torch.float64)


# --------------------------------------------------------------------------------- a pass


def run(state):
    case, s = state
    path = case["path"]
    if path == "short":
        b = s[0]
        b.build()
        st = tp.treepm_walk(b.ctx)
        tp.treepm_force_short(b.ctx, b.acc[0], b.acc[1], b.acc[2])
        return {"acc": b.acc, "counts": [st.n_nodes, st.n_groups, st.interactions]}
    if path == "long":
        b = s[0]
        tp.treepm_force_long(b.ctx, b.acc[0], b.acc[1], b.acc[2])
        return {"acc": b.acc}
    if path == "step":
        b = s[0]
        # every pass steps the same snapshot
        b.p.copy_(b.p0)
        b.v.copy_(b.v0)
        b.build()
        tp.treepm_walk(b.ctx)
        a = (b.acc[0], b.acc[1], b.acc[2])
        v = (b.v[0], b.v[1], b.v[2])
        tp.treepm_force_short(b.ctx, *a)
        tp.treepm_force_long(b.ctx, *a, accumulate=True)
        dt = tp.treepm_timestep(b.ctx, *v, *a, b.params.eps, 1.0)
        tp.treepm_kick_drift(b.ctx, b.p[0], b.p[1], b.p[2], *v, *a, dt, dt)
        return {"acc": b.acc, "x": b.p, "v": b.v, "dt": dt}
    if path == "batch":
        for b in s:
            b.build()
        tp.treepm_force_short_batch([b.ctx for b in s],
                                    [(b.acc[0], b.acc[1], b.acc[2]) for b in s])
        return {"acc": [b.acc for b in s]}
    pending = {tp.treepm_ensemble_submit(s.ens, i, b[0], *b[1]): b
               for i, b in enumerate(s.boxes)}
    while pending:
        for t in list(pending):
            rc, _ = tp.treepm_ensemble_poll(s.ens, t, *pending[t][2])
            if rc == tp.TREEPM_OK:
                del pending[t]
        if pending:
            time.sleep(0.0001)
    return {"acc": [b[2] for b in s.boxes]}


# ----------------------------------------------------------------------------------- work


def work(case):
    """Bytes: positions and masses read once (32 B a particle), accelerations written once.
    Flops: 38 per interaction of the lists that the case's opening angle defines (an estimate
    from the box's mean density and clustering), and the transforms of the mesh."""
    sizes = _sizes(case, 999) if case["path"] in ("batch", "serve") else [case["n"]]
    out = 24 if case.get("precision") == "fp64" else 12
    nbytes = sum(n * (32 + out) for n in sizes)
    flops = 0.0
    if case["path"] != "long":
        theta = 0.45 if case.get("opening") == "distance" else case["theta"]
        per = 1500.0 * (0.5 / theta) ** 1.5 * (case["n_crit"] / 256.0) ** 0.25
        flops += K_PP * per * sum(sizes)
    if case["path"] in ("long", "step"):
        pts = case["mesh_n"] ** 3
        nbytes += 8 * pts
        flops += 2 * 5.0 * pts * math.log2(pts) + 27 * 10.0 * sum(sizes)
    if case["path"] == "step":
        nbytes += 96 * sum(sizes)
    return {"bytes": float(nbytes), "flops": flops}


# ---------------------------------------------------------------------- values in 64 bits
# The method itself in plain torch: Morton keys, octree, group walk, pair sum, and the
# particle mesh, all in double precision.


def _image(d):
    return torch.where(d >= 0.5, d - 1.0, torch.where(d < -0.5, d + 1.0, d))


def _g(R):
    """The cutoff function of eq. (2)."""
    a = 1.0 + R ** 3 * (-1.6 + R * R * (1.6 + R * (-0.5 + R * (-12.0 / 35.0 + 0.15 * R))))
    b = (2.0 - R).clamp(min=0.0) ** 5 * (((7.0 * R + 22.0) * R + 10.0) * R + 4.0) / 140.0
    return torch.where(R < 1.0, a, b)


def _g_derivatives(R):
    R2 = R * R
    a1 = R2 * (-4.8 + R2 * (8.0 + R * (-3.0 + R * (-2.4 + 1.2 * R))))
    a2 = R * (-9.6 + R2 * (32.0 + R * (-15.0 + R * (-14.4 + 8.4 * R))))
    b1 = R * (448 + R * (-2688 + R * (3360 + R * (-1120 + R * (-420 + R * (336 - 56 * R)))))) / 140
    b2 = (448 + R * (-5376 + R * (10080 + R * (-4480 + R * (-2100 + R * (2016 - 392 * R)))))) / 140
    one, out = R < 1.0, R >= 2.0
    return (torch.where(out, 0.0, torch.where(one, a1, b1)),
            torch.where(out, 0.0, torch.where(one, a2, b2)))


class _Tree:
    def __init__(self, p, m, n_leaf, n_crit):
        n, dev = m.numel(), m.device
        q = torch.floor(p * 2.0 ** 21).to(torch.int64).clamp(0, 2 ** 21 - 1)
        key = torch.zeros(n, dtype=torch.int64, device=dev)
        for b in range(21):
            for a in range(3):
                key |= ((q[a] >> b) & 1) << (3 * b + 2 - a)
        key, self.idx = torch.sort(key, stable=True)
        self.x, self.m = p[:, self.idx].contiguous(), m[self.idx]
        # nodes, level by level
        first, count = [torch.zeros(1, dtype=torch.int64, device=dev)], [
            torch.full((1,), n, dtype=torch.int64, device=dev)]
        parents, base, off = [torch.full((1,), -1, dtype=torch.int64, device=dev)], 0, [0, 1]
        leaf_of = torch.zeros(n, dtype=torch.int64, device=dev)
        for lev in range(21):
            sub = torch.nonzero(count[lev] >= n_leaf).flatten()
            if not sub.numel():
                break
            f, c = first[lev][sub], count[lev][sub]
            mark = torch.zeros(n + 1, dtype=torch.int64, device=dev)
            mark[f] += 1
            mark[f + c] -= 1
            active = torch.cumsum(mark, 0)[:n] > 0
            pre = key >> (3 * (20 - lev))
            start = torch.ones(n, dtype=torch.bool, device=dev)
            start[1:] = pre[1:] != pre[:-1]
            start[f] = True
            pos = torch.nonzero(start).flatten()
            end = torch.cat([pos[1:], torch.tensor([n], device=dev)])
            keep = active[pos]
            first.append(pos[keep])
            count.append((end - pos)[keep])
            parents.append(sub[torch.searchsorted(f, pos[keep], right=True) - 1] + base)
            base = off[-1]
            off.append(base + first[-1].numel())
            node = torch.repeat_interleave(torch.arange(first[-1].numel(), device=dev) + base,
                                           count[-1])
            leaf_of[active] = node
        self.first, self.count, self.parent = map(torch.cat, (first, count, parents))
        self.level = torch.cat([torch.full_like(f, k) for k, f in enumerate(first)])
        nn = self.first.numel()
        self.nchild = torch.zeros(nn, dtype=torch.int64, device=dev)
        self.nchild.index_add_(0, self.parent[1:], torch.ones_like(self.parent[1:]))
        self.child = torch.full((nn,), nn, dtype=torch.int64, device=dev)
        self.child.scatter_reduce_(0, self.parent[1:], torch.arange(1, nn, device=dev), "amin")
        mom = torch.zeros(4, nn, dtype=torch.float64, device=dev)
        mom.index_add_(1, leaf_of, torch.cat([self.x * self.m, self.m[None]]))
        for lev in range(len(first) - 1, 0, -1):
            s = slice(off[lev], off[lev + 1])
            mom.index_add_(1, self.parent[s], mom[:, s].clone())
        self.mass, self.com = mom[3], mom[:3] / mom[3]
        side = 0.5 ** self.level.double()
        self.side = side
        cell = torch.zeros(3, nn, dtype=torch.int64, device=dev)
        k0 = key[self.first]
        for b in range(21):
            for a in range(3):
                cell[a] |= ((k0 >> (3 * b + 2 - a)) & 1) << b
        cell >>= (21 - self.level)
        self.centre = (cell.double() + 0.5) * side
        # groups: the first node on each path that is a leaf or holds at most n_crit
        can = (self.nchild == 0) | (self.count <= n_crit)
        under = torch.zeros(nn, dtype=torch.bool, device=dev)
        for lev in range(1, len(first)):
            s = slice(off[lev], off[lev + 1])
            under[s] = can[self.parent[s]] | under[self.parent[s]]
        g = torch.nonzero(can & ~under).flatten()
        self.group = g[torch.argsort(self.first[g])]
        ng = self.group.numel()
        self.gcount, self.gfirst = self.count[self.group], self.first[self.group]
        of = torch.repeat_interleave(torch.arange(ng, device=dev), self.gcount)
        lo = torch.full((3, ng), 2.0, dtype=torch.float64, device=dev)
        lo.scatter_reduce_(1, of.expand(3, n), self.x, "amin")
        hi = torch.full((3, ng), -1.0, dtype=torch.float64, device=dev)
        hi.scatter_reduce_(1, of.expand(3, n), self.x, "amax")
        self.gc, self.gh = (lo + hi) * 0.5, (hi - lo) * 0.5
        self.leaf_of, self.off = leaf_of, off

    def second_moments(self):
        """Q about each node's centre of mass: xx, yy, zz, xy, xz, yz."""
        pair = ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))
        Q = torch.zeros(6, self.mass.numel(), dtype=torch.float64, device=self.m.device)
        d = self.x - self.com[:, self.leaf_of]
        Q.index_add_(1, self.leaf_of, torch.stack([self.m * d[a] * d[b] for a, b in pair]))
        for lev in range(len(self.off) - 2, 0, -1):
            s = slice(self.off[lev], self.off[lev + 1])
            up = self.parent[s]
            d = self.com[:, s] - self.com[:, up]
            Q.index_add_(1, up, Q[:, s] + torch.stack([self.mass[s] * d[a] * d[b]
                                                       for a, b in pair]))
        return Q

    def walk(self, g0, g1, r_cut, theta, theta_max):
        """Lists of groups g0..g1: (group, entry) pairs sorted by group, cells as node indices,
        particles as -1 - position in key order."""
        dev = self.m.device
        grp = torch.arange(g0, g1, device=dev)
        node = torch.zeros_like(grp)
        cells, leaves = [], []
        while grp.numel():
            gc, gh = self.gc[:, grp], self.gh[:, grp]
            side = self.side[node]
            gap = (_image(self.centre[:, node] - gc).abs() - (0.5 * side + gh)).clamp(min=0.0)
            gap = gap[0] * gap[0] + gap[1] * gap[1] + gap[2] * gap[2]
            near = gap < r_cut * r_cut
            grp, node, gap, side, gc, gh = (grp[near], node[near], gap[near], side[near],
                                            gc[:, near], gh[:, near])
            d = (_image(self.com[:, node] - gc).abs() - gh).clamp(min=0.0)
            d2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
            if theta_max is None:
                th2 = theta * theta
            else:
                R = torch.sqrt(d2) / (0.5 * r_cut)
                w = R * _g(R)
                th = torch.where(w > 0.0, theta / torch.sqrt(w.clamp(min=1e-300)), theta_max)
                th2 = th.clamp(max=theta_max) ** 2
            take = (side * side < th2 * d2) & (gap > 0.0)
            cells.append((grp[take], node[take]))
            leaf = ~take & (self.nchild[node] == 0)
            leaves.append((grp[leaf], node[leaf]))
            more = ~take & ~leaf
            grp, node = grp[more], node[more]
            c = self.nchild[node]
            run0 = torch.cumsum(c, 0) - c
            k = torch.arange(int(c.sum()), device=dev) - torch.repeat_interleave(run0, c)
            grp = torch.repeat_interleave(grp, c)
            node = torch.repeat_interleave(self.child[node], c) + k
        lg = torch.cat([a for a, _ in leaves])
        ln = torch.cat([b for _, b in leaves])
        c = self.count[ln]
        run0 = torch.cumsum(c, 0) - c
        k = torch.arange(int(c.sum()), device=dev) - torch.repeat_interleave(run0, c)
        part = torch.repeat_interleave(self.first[ln], c) + k
        grp = torch.cat([a for a, _ in cells] + [torch.repeat_interleave(lg, c)])
        ent = torch.cat([b for _, b in cells] + [-1 - part])
        order = torch.argsort(grp, stable=True)
        return grp[order], ent[order]


def _tree_force(p, m, prm, quadrupole):
    """Short-range accelerations (3, n) in input order, and the counts of the lists."""
    t = _Tree(p, m, prm.n_leaf, prm.n_crit)
    dev, n = m.device, m.numel()
    theta_max = prm.theta_max if prm.opening == tp.TREEPM_OPEN_DISTANCE else None
    Q = t.second_moments() if quadrupole else None
    acc = torch.zeros(3, n, dtype=torch.float64, device=dev)
    ng, total, eta, e2 = t.group.numel(), 0, 0.5 * prm.r_cut, prm.eps ** 2
    for g0 in range(0, ng, 8192):
        g1 = min(ng, g0 + 8192)
        grp, ent = t.walk(g0, g1, prm.r_cut, prm.theta, theta_max)
        length = torch.bincount(grp - g0, minlength=g1 - g0)
        start = torch.cumsum(length, 0) - length
        pairs = length * t.gcount[g0:g1]
        total += int(pairs.sum())
        cum = torch.cumsum(pairs, 0).cpu()
        a = 0
        while a < g1 - g0:
            done = int(cum[a - 1]) if a else 0
            b = max(a + 1, int(torch.searchsorted(cum, done + (1 << 24), right=True)))
            b = min(b, g1 - g0)
            i0 = int(t.gfirst[g0 + a])
            cnt = t.gcount[g0 + a:g0 + b]
            per = torch.repeat_interleave(length[a:b], cnt)      # list length per particle
            beg = torch.repeat_interleave(start[a:b], cnt)
            off = torch.cumsum(per, 0) - per
            tot = int(per.sum())
            i = torch.repeat_interleave(torch.arange(per.numel(), device=dev), per)
            e = ent[torch.arange(tot, device=dev) - off[i] + beg[i]]
            cell = e >= 0
            node, part = e.clamp(min=0), (-1 - e).clamp(min=0)
            d = torch.where(cell, t.com[:, node], t.x[:, part]) - t.x[:, i + i0]
            d = _image(d)
            mass = torch.where(cell, t.mass[node], t.m[part])
            r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
            R = torch.sqrt(r2) / eta
            s2 = r2 + e2
            f = torch.where(r2 > 0.0, mass * _g(R) / (s2 * torch.sqrt(s2)), 0.0)
            v = f * d
            if quadrupole:
                v = v + torch.where(cell & (r2 > 0.0), _quad_term(d, r2, R, s2, Q[:, node], eta),
                                    0.0)
            acc[:, i0:i0 + per.numel()].index_add_(1, i, v)
            a = b
    out = torch.empty_like(acc)
    out[:, t.idx] = acc
    return out, [t.first.numel(), ng, total]


def _quad_term(d, r2, R, s2, Q, eta):
    r2 = torch.where(r2 > 0.0, r2, 1.0)
    r = torch.sqrt(r2)
    g, (g1, g2) = _g(R), _g_derivatives(R)
    q = 1.0 / (s2 * torch.sqrt(s2))
    p = q / s2
    u = g1 * q / (eta * r) - 3.0 * g * p
    w = (g2 * q / (eta * eta * r2) - g1 * q / (eta * r2 * r) - 6.0 * g1 * p / (eta * r)
         + 15.0 * g * p / s2)
    out = R >= 2.0
    u, w = torch.where(out, 0.0, u), torch.where(out, 0.0, w)
    qd = torch.stack([Q[0] * d[0] + Q[3] * d[1] + Q[4] * d[2],
                      Q[3] * d[0] + Q[1] * d[1] + Q[5] * d[2],
                      Q[4] * d[0] + Q[5] * d[1] + Q[2] * d[2]])
    tr = Q[0] + Q[1] + Q[2]
    dqd = d[0] * qd[0] + d[1] * qd[1] + d[2] * qd[2]
    return qd * u + 0.5 * tr * d * u + 0.5 * dqd * d * w


def _mesh_force(p, m, mesh_n, r_cut):
    """Long-range accelerations: TSC assignment, transforms, fourth-order differences, TSC
    interpolation."""
    dev, n = m.device, mesh_n
    x = p * n
    near = torch.floor(x + 0.5)
    d = x - near
    w = torch.stack([0.5 * (0.5 - d) ** 2, 0.75 - d * d, 0.5 * (0.5 + d) ** 2])
    near = near.to(torch.int64)
    clouds = []
    for a in range(3):
        for b in range(3):
            for c in range(3):
                at = (((near[0] + a - 1) % n) * n + (near[1] + b - 1) % n) * n + (near[2] + c - 1) % n
                clouds.append((at, w[a, 0] * w[b, 1] * w[c, 2]))
    rho = torch.zeros(n ** 3, dtype=torch.float64, device=dev)
    for at, wt in clouds:
        rho.index_add_(0, at, wt * m)
    k = 2.0 * math.pi * torch.fft.fftfreq(n, 1.0 / n, device=dev, dtype=torch.float64)
    k2 = k[:, None, None] ** 2 + k[None, :, None] ** 2 + k[None, None, :] ** 2
    y = torch.sqrt(k2) * (0.5 * r_cut)
    y[0, 0, 0] = 1.0
    # transform of the S2 cloud of radius eta, with its series where the closed form cancels
    series = 1.0 - y ** 2 / 15.0 + y ** 4 / 560.0 - y ** 6 / 37800.0
    y_ = y.clamp(min=1e-2)
    shape = torch.where(y < 0.1, series,
                        12.0 * (2.0 - 2.0 * torch.cos(y_) - y_ * torch.sin(y_)) / y_ ** 4)
    s = torch.sinc(k / (2.0 * math.pi * n)) ** 3
    win = s[:, None, None] * s[None, :, None] * s[None, None, :]
    k2[0, 0, 0] = 1.0
    green = -4.0 * math.pi * shape ** 2 / (k2 * win ** 2)
    green[0, 0, 0] = 0.0
    phi = torch.fft.ifftn(torch.fft.fftn(rho.reshape(n, n, n)) * green).real * n ** 3
    out = torch.zeros_like(p)
    for axis in range(3):
        f = -((2.0 / 3.0) * (torch.roll(phi, -1, axis) - torch.roll(phi, 1, axis))
              - (torch.roll(phi, -2, axis) - torch.roll(phi, 2, axis)) / 12.0) * n
        f = f.reshape(-1)
        for at, wt in clouds:
            out[axis] += wt * f[at]
    return out


def exact(case, seed):
    boxes = _boxes(case, seed)
    if case["path"] == "long":
        n, p, m = boxes[0]
        return {"acc": _mesh_force(p, m, case["mesh_n"], 3.0 / case["mesh_n"])}
    if max(b[0] for b in boxes) > _EXACT_MOST:
        return None
    got = []
    for n, p, m in boxes:
        a, counts = _tree_force(p, m, _params(case, n), bool(case.get("quadrupole")))
        got.append(a)
    if case["path"] == "short":
        return {"acc": got[0], "counts": counts}
    if case["path"] == "step":
        n, p, m = boxes[0]
        a = got[0] + _mesh_force(p, m, case["mesh_n"], 3.0 / case["mesh_n"])
        v, eps = _velocities(n, seed), _params(case, n).eps
        dt = float(torch.minimum(torch.sqrt(eps / a.norm(dim=0)), eps / v.norm(dim=0)).min())
        v = v + a * dt
        return {"acc": a, "x": _wrap(p + v * dt), "v": v, "dt": dt}
    if case["path"] == "batch":
        return {"acc": got}
    return {"acc": [[a[0].cpu(), a[1].cpu(), a[2].cpu()] for a in got]}
