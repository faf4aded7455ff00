"""The work that users of this library have it do, as cases of a few plain values.

Every case is one pass of a program's inner loop through the public calls:

- ``step``     one fused step of Alg. 1 (cells, k-NN lists, Eq. 2, Eq. 1) of one system
- ``lists``    cells and k-NN lists with squared distances (a neighbour query alone)
- ``metric``   one step with the metric rule: cells, CSR rows, alignment and move;
               with ``two_call`` the count / allocate / fill protocol and the polar
               order parameter read back, without it preallocated rows and no wait
- ``fov``      cells and field-of-view lists
- ``forces``   cells, Voronoi rows and the Voronoi model's energy and forces
- ``reuse``    one Vicsek step with Voronoi neighbours: last step's rows brought up to
               date at the new positions, then alignment and move
- ``batch``    one step of many independent systems of uneven size
- ``served``   a burst of jobs with host inputs through the request loop, results back

The box is 2^20 units, particles move 64 units a step at noise 0.2 and the noise seed
is 0, as in the benchmark; positions are uniform or drawn from 256 Gaussian clusters
of width 0.01 of the box (the states a flock starts from and contracts to).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2103_10239_amd as nm

BOX = 1 << 20
V0 = 64
ETA = 0.2
STEP = 3          # step index of the noise stream
DEV = "cuda"
SUB = 0x100       # sub-strip kernel flag of the grid's block choice

ANGULAR, NEW_HEADING = 1, 2


def _case(name, path, n, k=0, **kw):
    c = {"name": name, "path": path, "n": n, "k": k, "points": "uniform", "per_cell": 2.0, "block": 0}
    c.update(kw)
    return c


def listed():
    return [
        # A small system stepped by itself: launches and latency are all there is.
        _case("step_1k", "step", 1000, 7, variant=0, self=1),
        # An ordinary single system of odd size with longer lists.
        _case("step_50k_k12", "step", 50021, 12, variant=0, self=1),
        # The headline workload, on the grid that the tuner picks for it.
        _case("step_1m", "step", 1 << 20, 7, per_cell=1.0, block=6, variant=0, self=1),
        # The largest system: strongly clustered, long lists, sub-strip kernel.
        _case("step_4m_clustered", "step", 1 << 22, 20, points="clustered", per_cell=4.0, block=SUB,
              variant=0, self=1),
        # A neighbour query alone on a clustered state, distances too.
        _case("lists_200k_k31", "lists", 200003, 31, points="clustered"),
        # The metric rule's step at the mean degree of the benchmark, rows preallocated.
        _case("metric_1m", "metric", 1 << 20, mean=7.0, per_cell=1.0, two_call=False),
        # The metric rule on a clustered mid-size system: uneven rows, sizes read back.
        _case("metric_60k_clustered", "metric", 60013, mean=4.0, points="clustered", per_cell=1.0,
              two_call=True),
        # Vision-limited neighbours: half plane ahead, the benchmark's grid.
        _case("fov_300k", "fov", 300007, 7, cos_q=0, per_cell=4.0),
        # The Voronoi model of a dense tissue: rows, energy, forces.
        _case("forces_250k", "forces", 250007, per_cell=1.0),
        # Vicsek dynamics with Voronoi neighbours: rows reused between steps.
        _case("reuse_1m", "reuse", 1 << 20, per_cell=1.0),
        # The many-systems form at the benchmark's mix of sizes.
        _case("batch_512", "batch", 512, 7, lo=256, hi=65536),
        # The served form: a burst of requests with host data.
        _case("served_16", "served", 16, 7, lo=1024, hi=1 << 17, steps=20),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    path = rng.choice(["step", "step", "step", "lists", "metric", "fov", "forces", "reuse", "batch", "served"])
    points = rng.choice(["uniform", "clustered"])
    per_cell = rng.choice([1.0, 2.0, 4.0])
    if path == "step":
        block = rng.choice([0, 6]) if points == "uniform" else rng.choice([0, SUB])
        return _case("", path, _log(rng, 1000, 1 << 20), rng.choice([1, 4, 6, 7, 12, 20]), points=points,
                     per_cell=per_cell, block=block, variant=rng.choice([0, 0, 1, 2, 3]),
                     self=rng.choice([1, 1, 0]))
    if path == "lists":
        return _case("", path, _log(rng, 1000, 400000), rng.randint(1, 32), points=points, per_cell=per_cell)
    if path == "metric":
        n = _log(rng, 1000, 1 << 20) if points == "uniform" else _log(rng, 1000, 1 << 17)
        mean = rng.uniform(3.0, 15.0) if points == "uniform" else rng.uniform(1.0, 4.0)
        return _case("", path, n, mean=mean, points=points, per_cell=per_cell,
                     two_call=rng.choice([True, False]))
    if path == "fov":
        return _case("", path, _log(rng, 4096, 1 << 20), rng.randint(3, 8),
                     cos_q=rng.choice([-4096, -2048, 0, 2048]), per_cell=4.0)
    if path == "forces":
        return _case("", path, _log(rng, 4096, 1 << 20), per_cell=rng.choice([1.0, 2.0]))
    if path == "reuse":
        return _case("", path, _log(rng, 4096, 1 << 20), per_cell=rng.choice([1.0, 2.0]))
    if path == "batch":
        return _case("", path, _log(rng, 8, 512), rng.choice([6, 7, 12]), lo=256, hi=_log(rng, 4096, 65536))
    return _case("", path, rng.randint(4, 16), rng.choice([7, 12]), lo=1024, hi=_log(rng, 8192, 1 << 17),
                 steps=rng.randint(4, 20))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _points(kind, n, rng):
    """int32 coordinates in the box (uniform, or 256 Gaussian clusters) and fp32 headings."""
    if kind == "clustered":
        centre = rng.uniform(0.0, BOX, size=(256, 2))
        p = centre[rng.integers(0, 256, size=n)]
        p = np.floor(p + 0.01 * BOX * rng.standard_normal((n, 2), dtype=np.float32)).astype(np.int64) % BOX
        x, y = p[:, 0].astype(np.int32), p[:, 1].astype(np.int32)
    else:
        x = rng.integers(0, BOX, size=n, dtype=np.int32)
        y = rng.integers(0, BOX, size=n, dtype=np.int32)
    th = rng.uniform(-np.pi, np.pi, size=n).astype(np.float32)
    return x, y, th


def _distinct(x, y, rng):
    """Move particles that share a position (the Voronoi model gives each its own cell)."""
    while True:
        code = x.astype(np.int64) * BOX + y
        _, first = np.unique(code, return_index=True)
        if len(first) == len(code):
            return x, y
        again = np.ones(len(code), bool)
        again[first] = False
        x[again] = rng.integers(0, BOX, size=int(again.sum()), dtype=np.int32)
        y[again] = rng.integers(0, BOX, size=int(again.sum()), dtype=np.int32)


def _state(case, seed):
    rng = np.random.default_rng(seed)
    x, y, th = _points(case["points"], case["n"], rng)
    if case["path"] in ("forces", "reuse"):
        x, y = _distinct(x, y, rng)
    return x, y, th


def _sizes(case, seed):
    """Log-uniform sizes; those of the benchmark's mix for every seed, so that a case's work is one number."""
    rng = np.random.default_rng(4)
    return np.rint(np.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]), size=case["n"]))).astype(np.int64)


def _systems(case, seed):
    """Systems of the batch or the jobs: every second one clustered."""
    rng = np.random.default_rng(seed)
    return [_points("clustered" if s % 2 else "uniform", int(m), rng) for s, m in enumerate(_sizes(case, seed))]


def _rc2(case):
    return int(round(case["mean"] * BOX * BOX / (math.pi * (case["n"] - 1))))


def _tissue(n):
    """Moduli and targets of Eq. 3 for unit mean area in units of the box."""
    a0 = BOX * BOX / n
    return dict(ka=1.0 / a0, kp=1.0, a0=a0, p0=3.8 * math.sqrt(a0))


def _params(case):
    return nm.make_params(BOX, v0=V0, eta=ETA, include_self=case.get("self", 1), seed=0,
                          variant=case.get("variant", 0))


def _like(n, k=None):
    i32 = dict(dtype=torch.int32, device=DEV)
    out = {"x": torch.empty(n, **i32), "y": torch.empty(n, **i32),
           "theta": torch.empty(n, dtype=torch.float32, device=DEV)}
    if k:
        out["nbr"] = torch.empty((n, k), **i32)
    return out


def prepare(case, seed):
    path, n, k = case["path"], case["n"], case["k"]
    p = _params(case)
    st = {"case": case, "p": p}
    if path == "batch":
        sys = _systems(case, seed)
        cat = [np.concatenate([s[q] for s in sys]) for q in range(3)]
        st["batch"] = nm.Batch([len(s[0]) for s in sys], *cat, k, p, sys_ids=list(range(n)), step0=STEP)
        st["batch"].tune(2)
        return st
    if path == "served":
        st["jobs"] = _systems(case, seed)
        st["server"] = nm.Server(4 << 30)
        return st
    x, y, th = _state(case, seed)
    dev = lambda a: torch.from_numpy(a).to(DEV)
    st.update(x=dev(x), y=dev(y), theta=dev(th))
    w = nm.suggest_cell_w(n, BOX, case["per_cell"])
    st["ws"] = nm.Workspace(n, BOX, w, DEV, block=case["block"])
    if path == "step":
        st["out"] = _like(n, k)
    elif path == "lists":
        st["nbr"] = torch.empty((n, k), dtype=torch.int32, device=DEV)
        st["d2"] = torch.empty((n, k), dtype=torch.int64, device=DEV)
    elif path == "metric":
        st["rc2"] = _rc2(case)
        st["out"] = _like(n)
        # room for the mean degree, about 4 times that where particles cluster
        room = int(n * case["mean"] * (1.25 if case["points"] == "uniform" else 8.0)) + 1024
        st["idx"] = torch.zeros(room, dtype=torch.int32, device=DEV)
        st["offsets"] = torch.empty(n + 1, dtype=torch.int32, device=DEV)
    elif path == "fov":
        st["nbr"] = torch.empty((n, k), dtype=torch.int32, device=DEV)
    elif path == "reuse":
        # the step before: rows at the positions that the last move came from
        st["out"] = _like(n)
        bx = (st["x"] - torch.round(V0 * torch.cos(st["theta"])).int()) & (BOX - 1)
        by = (st["y"] - torch.round(V0 * torch.sin(st["theta"])).int()) & (BOX - 1)
        nm.build_cells(st["ws"], bx, by)
        st["ring_was"], st["deg_was"] = nm.voronoi(st["ws"])
        st["ring"], st["deg"] = torch.empty_like(st["ring_was"]), torch.empty_like(st["deg_was"])
    return st


def run(st):
    case, p, path = st["case"], st["p"], st["case"]["path"]
    if path == "step":
        o = st["out"]
        nm.step(st["ws"], st["x"], st["y"], st["theta"], case["k"], p, STEP, o["nbr"], o["x"], o["y"], o["theta"])
        return o
    if path == "batch":
        b = st["batch"]
        b.step(1)
        x, y, th = b.current()
        return {"x": x, "y": y, "theta": th, "nbr": b.nbr}
    if path == "served":
        srv = st["server"]
        ids = [srv.submit(x, y, th, case["k"], 1 + (7 * s) % case["steps"],
                          nm.make_params(BOX, v0=V0, eta=ETA, seed=0, sys_id=s))
               for s, (x, y, th) in enumerate(st["jobs"])]
        got = [srv.wait(j) for j in ids]
        return [[g["x"], g["y"], g["theta"]] for g in got]
    ws, x, y, th = st["ws"], st["x"], st["y"], st["theta"]
    nm.build_cells(ws, x, y)
    if path == "lists":
        nm.knn(ws, case["k"], st["nbr"], st["d2"])
        return {"nbr": st["nbr"], "d2": st["d2"]}
    if path == "fov":
        return {"nbr": nm.knn_fov(ws, case["k"], th, case["cos_q"], st["nbr"])}
    if path == "metric":
        o = st["out"]
        out = (o["x"], o["y"], o["theta"])
        if case["two_call"]:
            offsets, idx = nm.metric_list(ws, st["rc2"])
            nm.align_step(x, y, th, p, STEP, offsets=offsets, idx=idx, out=out, ws=ws)
            st["idx"][:idx.numel()].copy_(idx)  # the rows are kept in the program's own buffer
            return {**o, "offsets": offsets, "idx": st["idx"], "order": nm.polar_order(o["theta"])}
        nm.metric_list(ws, st["rc2"], st["offsets"], st["idx"])
        nm.align_step(x, y, th, p, STEP, offsets=st["offsets"], idx=st["idx"], out=out, ws=ws)
        return {**o, "offsets": st["offsets"], "idx": st["idx"]}
    if path == "forces":
        ring, deg = nm.voronoi(ws)
        f = nm.voronoi_forces(x, y, BOX, ring, deg, **_tissue(case["n"]), ws=ws)
        return {"ring": ring, "deg": deg, **{q: f[q] for q in ("area", "perim", "fx", "fy", "energy")}}
    # reuse: last step's rows stay with the program, this step's are made from them
    st["ring"].copy_(st["ring_was"])
    st["deg"].copy_(st["deg_was"])
    nm.voronoi_update(ws, x, y, st["ring"], st["deg"])
    o = st["out"]
    nm.align_step(x, y, th, p, STEP, nbr=st["ring"], out=(o["x"], o["y"], o["theta"]), ws=ws)
    return {**o, "ring": st["ring"], "deg": st["deg"]}


def work(case):
    """Compulsory traffic: state read and written once, rows written once."""
    path, n, k = case["path"], case["n"], case["k"]
    step_b, step_f = 24 + 4 * k, 60 + 2 * (k + 1) + 5 * k  # Eq. 2 and Eq. 1; a distance per neighbour
    if path == "step":
        return {"bytes": step_b * n, "flops": step_f * n}
    if path == "lists":
        return {"bytes": (8 + 12 * k) * n, "flops": 5 * k * n}
    if path == "metric":
        # a clustered system of density contrast c has about c times the mean degree
        deg = case["mean"] if case["points"] == "uniform" else case["mean"] * 4.0
        return {"bytes": (24 + 4 + 4 * deg) * n, "flops": (60 + 7 * deg) * n}
    if path == "fov":
        return {"bytes": (12 + 4 * k) * n, "flops": 10 * k * n}
    if path == "forces":  # rows of 16 entries, area, perimeter, force
        return {"bytes": (8 + 68 + 32) * n, "flops": 600 * n}
    if path == "reuse":   # rows of 16 entries read and written, one step
        return {"bytes": (24 + 2 * 68) * n, "flops": 250 * n}
    if path == "batch":
        tot = int(_sizes(case, 0).sum())
        return {"bytes": step_b * tot, "flops": step_f * tot}
    sizes = _sizes(case, 0)
    tot = int(sum(int(m) * (1 + (7 * s) % case["steps"]) for s, m in enumerate(sizes)))
    return {"bytes": step_b * tot, "flops": step_f * tot}


# ---------------------------------------------------------------------------
# exact values, in plain torch and numpy
# ---------------------------------------------------------------------------
def _philox(n, step, sys_id, seed=0):
    """Word i mod 4 of Philox4x32-10 at counter (i / 4, step, 0, sys_id), for i < n."""
    m = (n + 3) // 4
    u64, low = np.uint64, np.uint64(0xFFFFFFFF)
    c = [np.arange(m, dtype=u64), np.full(m, step, u64), np.zeros(m, u64), np.full(m, sys_id, u64)]
    ka, kb = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        a, b = c[0] * u64(0xD2511F53), c[2] * u64(0xCD9E8D57)
        c = [(b >> u64(32)) ^ c[1] ^ u64(ka), b & low, (a >> u64(32)) ^ c[3] ^ u64(kb), a & low]
        ka, kb = (ka + 0x9E3779B9) & 0xFFFFFFFF, (kb + 0xBB67AE85) & 0xFFFFFFFF
    return np.stack(c, 1).reshape(-1)[:n]


def _near(d):
    return ((d + BOX // 2) & (BOX - 1)) - BOX // 2


class _Cells:
    """Particles sorted by cell of width w; the candidates of a query are its 3 x 3 cells."""

    def __init__(self, x, y, w):
        self.g = BOX // w
        self.w = w
        cell = (y // w) * self.g + x // w
        self.order = torch.argsort(cell)
        self.start = torch.searchsorted(cell[self.order], torch.arange(self.g * self.g + 1, device=x.device))
        self.x, self.y = x, y

    def chunks(self, q, most=1 << 24):
        """(queries, candidates [q, m], valid, d2, clear distance) in pieces of at most `most` entries."""
        cx, cy = self.x[q] // self.w, self.y[q] // self.w
        step = torch.arange(-1, 2, device=q.device)
        c = ((cy[:, None, None] + step[None, :, None]) % self.g) * self.g + \
            (cx[:, None, None] + step[None, None, :]) % self.g
        c = c.reshape(-1, 9)
        beg, cnt = self.start[c], self.start[c + 1] - self.start[c]
        total = cnt.sum(1)
        by = torch.argsort(total)
        q, beg, cnt, total = q[by], beg[by], cnt[by], total[by]
        sizes = total.cpu().numpy()
        ox, oy = self.x[q] % self.w, self.y[q] % self.w
        clear = self.w + torch.minimum(torch.minimum(ox, self.w - 1 - ox), torch.minimum(oy, self.w - 1 - oy)) + 1
        a = 0
        while a < len(sizes):
            e = min(len(sizes), a + max(1, most // max(1, int(sizes[min(len(sizes) - 1, a + 4096)]))))
            while e > a + 1 and (e - a) * int(sizes[e - 1]) > 2 * most:
                e = a + (e - a + 1) // 2
            m = max(1, int(sizes[e - 1]))
            t = torch.arange(m, device=q.device)
            end = cnt[a:e].cumsum(1)
            part = torch.searchsorted(end, t.expand(e - a, m).contiguous(), right=True).clamp(max=8)
            at = t + (beg[a:e] - (end - cnt[a:e])).gather(1, part)
            ok = t < total[a:e, None]
            j = self.order[at.clamp(0, len(self.order) - 1)]
            dx, dy = _near(self.x[j] - self.x[q[a:e], None]), _near(self.y[j] - self.y[q[a:e], None])
            yield q[a:e], j, ok & (j != q[a:e, None]), dx * dx + dy * dy, clear[a:e]
            a = e


def _nearest(x, y, k, left=None):
    """The k nearest of every particle (of the particles `left`) by (d^2, index): exact integers."""
    n = len(x)
    out = torch.empty((n, k), dtype=torch.int64, device=x.device)
    asked = left
    left = torch.arange(n, device=x.device) if left is None else left
    w = 1 << max(6, int(math.log2(BOX / math.sqrt(n) * math.sqrt(k / 9.0))) - 1)
    while len(left) and w * 4 <= BOX:
        cells, again = _Cells(x, y, w), []
        for q, j, ok, d2, clear in cells.chunks(left):
            if j.shape[1] < k + 1:
                again.append(q)
                continue
            key = torch.where(ok, (d2 << 23) | j, 1 << 62)
            key = key.topk(k, dim=1, largest=False, sorted=True).values
            sure = (key[:, -1] >> 23) < clear * clear
            out[q[sure]] = key[sure] & ((1 << 23) - 1)
            again.append(q[~sure])
        left = torch.cat(again) if again else left[:0]
        w *= 2
    everyone = torch.arange(n, device=x.device)
    for a in range(0, len(left), max(1, (1 << 24) // n)):
        q = left[a:a + max(1, (1 << 24) // n)]
        dx, dy = _near(x[None] - x[q, None]), _near(y[None] - y[q, None])
        key = torch.where(everyone[None] != q[:, None], ((dx * dx + dy * dy) << 23) | everyone, 1 << 62)
        out[q] = key.topk(k, dim=1, largest=False, sorted=True).values & ((1 << 23) - 1)
    return out if asked is None else out[asked]


def _turn(sx, sy, m, th, p_variant, include_self, sys_id, step=STEP):
    """Eq. 2 in 64 bits from the sums of the neighbours' unit vectors."""
    n = len(th)
    if include_self:
        sx, sy, m = sx + torch.cos(th), sy + torch.sin(th), m + 1
    phi = torch.from_numpy(_philox(n, step, sys_id).astype(np.float64)).to(th.device) * 2.0 ** -32 * (2 * math.pi) - math.pi
    ax, ay = sx / m.clamp(min=1), sy / m.clamp(min=1)
    eta = float(np.float32(ETA))
    if p_variant & ANGULAR:
        base = torch.where((ax == 0) & (ay == 0), th, torch.atan2(ay, ax))
        t = base + eta * phi
        return t - 2 * math.pi * torch.floor((t + math.pi) / (2 * math.pi))
    vx, vy = ax + eta * torch.cos(phi), ay + eta * torch.sin(phi)
    return torch.where((vx == 0) & (vy == 0), th, torch.atan2(vy, vx))


def _heading_fixed(x, y, th, k, variant, include_self, sys_id):
    c, s = torch.cos(th), torch.sin(th)
    nbr = _nearest(x, y, k)
    sx, sy = torch.zeros_like(th), torch.zeros_like(th)
    for t in range(k):
        sx += c[nbr[:, t]]
        sy += s[nbr[:, t]]
    return _turn(sx, sy, torch.full_like(th, k), th, variant, include_self, sys_id)


def _long(x, y, th):
    dev = lambda a, t: torch.from_numpy(a).to(DEV).to(t)
    return dev(x, torch.int64), dev(y, torch.int64), dev(th, torch.float64)


def _delaunay(x, y):
    """Voronoi neighbours of every particle counter-clockwise, [n, 24] with a mask of those there are.

    They are looked for among the m nearest; a cell whose farthest vertex lies farther out than
    half the m-th distance is done again with more.
    """
    n, width = len(x), 24
    nbr = torch.zeros((n, width), dtype=torch.int64, device=x.device)
    ok = torch.zeros((n, width), dtype=torch.bool, device=x.device)
    left = torch.arange(n, device=x.device)
    for m in (32, 64, 160, 400):
        m = min(m, n - 1)
        near, again = _nearest(x, y, m, left), []
        for a in range(0, len(left), max(1, (1 << 25) // (m * m))):
            q = left[a:a + max(1, (1 << 25) // (m * m))]
            j = near[a:a + len(q)]
            ox, oy = _near(x[j] - x[q, None]).double(), _near(y[j] - y[q, None]).double()
            d2 = ox * ox + oy * oy
            # on the bisector of j: o/2 + t perp(o); particle c is farther while t 2 (o x c) <= c.c - o.c
            num = d2[:, None, :] - (ox[:, :, None] * ox[:, None, :] + oy[:, :, None] * oy[:, None, :])
            den = 2 * (ox[:, :, None] * oy[:, None, :] - oy[:, :, None] * ox[:, None, :])
            t = num / den
            hi = torch.where(den > 0, t, math.inf).amin(2)
            lo = torch.where(den < 0, t, -math.inf).amax(2)
            behind = ((den == 0) & (num < 0)).any(2)
            far = (0.25 + torch.maximum(hi * hi, lo * lo)) * d2  # squared distance of the edge's ends
            keep = (lo < hi) & ~behind & (d2 > 0)
            sure = torch.where(keep, far, 0.0).amax(1) * 4.0001 < d2[:, -1]
            keep |= d2 == 0
            ang = torch.atan2(oy, ox)
            by = torch.argsort(torch.where(keep, torch.where(ang < 0, ang + 2 * math.pi, ang), 100.0), dim=1)[:, :width]
            nbr[q], ok[q] = j.gather(1, by), keep.gather(1, by)
            again.append(q[~sure])
        left = torch.cat(again)
        if not len(left):
            break
    return nbr, ok


def _exact_forces(case, seed):
    x, y, _ = _long(*_state(case, seed))
    n, t = len(x), _tissue(case["n"])
    nbr, ok = _delaunay(x, y)
    cnt = ok.sum(1)
    nxt = torch.arange(nbr.shape[1], device=x.device)[None] + 1
    nxt = torch.where(nxt < cnt[:, None], nxt, torch.zeros_like(nxt))
    third = nbr.gather(1, nxt)
    rx, ry = x.double().requires_grad_(), y.double().requires_grad_()

    def offset(r, i, j, whole):
        return r[j] - r[i] + (_near(whole[j] - whole[i]) - (whole[j] - whole[i])).double()

    me = torch.arange(n, device=x.device)[:, None].expand_as(nbr)
    ax, ay = offset(rx, me, nbr, x), offset(ry, me, nbr, y)
    bx, by = offset(rx, me, third, x), offset(ry, me, third, y)
    cr = torch.where(ok, 2 * (ax * by - ay * bx), torch.ones_like(ax))
    na, nb = ax * ax + ay * ay, bx * bx + by * by
    hx, hy = (by * na - ay * nb) / cr, (ax * nb - bx * na) / cr
    gx, gy = hx.gather(1, nxt), hy.gather(1, nxt)
    area = torch.where(ok, hx * gy - hy * gx, torch.zeros_like(hx)).sum(1) / 2
    length = torch.where(ok, (gx - hx) ** 2 + (gy - hy) ** 2, torch.ones_like(hx)).sqrt()
    perim = torch.where(ok, length, torch.zeros_like(hx)).sum(1)
    e = (t["ka"] * (area - t["a0"]) ** 2 + t["kp"] * (perim - t["p0"]) ** 2).sum()
    fx, fy = torch.autograd.grad(e, (rx, ry))
    return {"ring": None, "deg": None, "area": area.detach(), "perim": perim.detach(), "fx": -fx, "fy": -fy,
            "energy": e.detach().reshape(1)}


def exact(case, seed):
    path = case["path"]
    if path in ("lists", "fov", "served"):
        # whole numbers alone; a served job's many steps round positions and headings at each
        return None
    if path == "forces":
        return _exact_forces(case, seed) if case["n"] <= 400000 else None
    if path == "batch":
        if case["n"] * case["hi"] > 1 << 25:
            return None
        got = [_heading_fixed(*_long(*s), case["k"], 0, 1, i) for i, s in enumerate(_systems(case, seed))]
        return {"x": None, "y": None, "theta": torch.cat(got), "nbr": None}
    x, y, th = _long(*_state(case, seed))
    if path == "step":
        got = _heading_fixed(x, y, th, case["k"], case["variant"], case["self"], 0)
        return {"x": None, "y": None, "theta": got, "nbr": None}
    c, s = torch.cos(th), torch.sin(th)
    sx, sy, m = torch.zeros_like(th), torch.zeros_like(th), torch.zeros_like(th)
    if path == "reuse":
        nbr, ok = _delaunay(x, y)
        sx, sy, m = (ok * c[nbr]).sum(1), (ok * s[nbr]).sum(1), ok.sum(1).double()
        return {"x": None, "y": None, "theta": _turn(sx, sy, m, th, 0, 1, 0), "ring": None, "deg": None}
    rc2 = _rc2(case)
    w = 1 << max(6, math.isqrt(rc2).bit_length())
    for q, j, ok, d2, _ in _Cells(x, y, w).chunks(torch.arange(len(x), device=x.device)):
        ok = ok & (d2 <= rc2)
        sx[q], sy[q], m[q] = (ok * c[j]).sum(1), (ok * s[j]).sum(1), ok.sum(1).double()
    got = {"x": None, "y": None, "theta": _turn(sx, sy, m, th, 0, 1, 0), "offsets": None,
           "idx": None}
    if case["two_call"]:
        t = got["theta"]
        got |= {"order": float(torch.hypot(torch.cos(t).sum(), torch.sin(t).sum()) / len(t))}
    return got
