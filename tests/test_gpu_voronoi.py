"""Parity of the Voronoi (Delaunay) neighbour lists on the GPU with the
brute-force oracle (Sec. III, Sec. IV): rows bit-exact (same neighbours, same
counter-clockwise order from the +x axis); the "do I need to recompute?"
test flags every row that changed; the update gives the oracle's rows for the
new positions; the alignment step over the rows matches the oracle.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2103_10239_amd as nm
from paper_2103_10239_amd import workloads

pytestmark = pytest.mark.gpu
TOL = 1e-5


def _dev(a, dtype):
    return torch.as_tensor(np.ascontiguousarray(a)).to(dtype).to("cuda")


def _gpu_rows(x, y, box, w, dmax=16):
    ws = nm.Workspace(len(x), box, w)
    nm.build_cells(ws, _dev(x, torch.int32), _dev(y, torch.int32))
    ring, deg = nm.voronoi(ws, dmax)
    st = nm.check(ws)
    return ring.cpu().numpy(), deg.cpu().numpy(), st, ws


def _rows_of(ring, deg):
    return [ring[i, :deg[i]].tolist() for i in range(len(deg))]


def _oracle_rows(x, y, box, rows=None, rho0=None):
    off, idx = oracle.voronoi(x, y, box, rows=rows, rho0=rho0)
    return [idx[off[r]:off[r + 1]].tolist() for r in range(len(off) - 1)]


def _clustered(n, box, ncl, sf, seed=3):
    return workloads.clustered(n, box=box, n_clusters=ncl, sigma_frac=sf, seed=seed)


# (kind, n, box, cell width): narrow cells (offsets < 2^14) in boxes up to
# 2^17, cells handed to the 64-bit kernel in sparse boxes, and a mix
CASES = [("uniform", 4097, 1 << 16, 1024), ("uniform", 4097, 1 << 16, 2048), ("uniform", 4097, 1 << 16, 512),
         ("uniform", 20013, 1 << 17, 1024), ("uniform", 3001, 1 << 20, 16384), ("uniform", 3, 64, 16),
         ("clustered", 8191, 1 << 20, 4096), ("clustered", 20013, 1 << 20, 2048),
         ("clustered", 6000, 1 << 17, 512)]


def _gen(kind, n, box):
    if kind == "uniform":
        return workloads.uniform(n, box=box, seed_pos=n + box)
    return _clustered(n, box, 128, 0.02)


@pytest.mark.parametrize("kind,n,box,w", CASES)
def test_voronoi_matches_oracle(kind, n, box, w):
    x, y, _ = _gen(kind, n, box)
    try:
        ref = _oracle_rows(x, y, box)
    except oracle.OracleError as e:
        assert e.status == oracle.E_RANGE
        _, _, st, _ = _gpu_rows(x, y, box, w)
        assert st == nm.NM_E_RANGE
        return
    ring, deg, st, _ = _gpu_rows(x, y, box, w)
    assert st == 0
    assert _rows_of(ring, deg) == ref
    assert (ring[np.arange(ring.shape[1])[None, :] >= deg[:, None]] == -1).all()


def _ring_of(m, box):
    """One particle with m neighbours almost on a circle, in a sparser uniform background."""
    x, y, _ = workloads.uniform(2000, box=box, seed_pos=77)
    c, r = box // 2, box // 16
    d2 = (x.astype(np.int64) - c) ** 2 + (y.astype(np.int64) - c) ** 2
    x, y = x[d2 > (2 * r) ** 2], y[d2 > (2 * r) ** 2]
    a = np.arange(m) * (2 * np.pi / m) + 0.01
    return (np.concatenate([x, [c], c + np.rint(r * np.cos(a)).astype(np.int32)]).astype(np.int32),
            np.concatenate([y, [c], c + np.rint(r * np.sin(a)).astype(np.int32)]).astype(np.int32))


def _clump(n, dense, box, w):
    """A uniform system with `dense` more particles inside two cells of width w, some of them coincident."""
    x, y, _ = workloads.uniform(n, box=box, seed_pos=78)
    cx, cy, _ = workloads.uniform(dense, box=w, seed_pos=79)
    return (np.concatenate([x, 5 * w + 2 * cx]).astype(np.int32), np.concatenate([y, 7 * w + cy]).astype(np.int32))


# Rows built from staged strips, by a wavefront each, or by the general
# kernels: grids on both sides of what strips take (blocks of 3 to 15 cells,
# 16-bit and 32-bit offsets, a halo as wide as the box), strips whose halo
# overflows, rows of more than 16 entries, coincident particles in both.
STRIP_CASES = [("uniform", 513, 1 << 12, 1 << 9), ("uniform", 513, 1 << 12, 1 << 8), ("uniform", 513, 1 << 20, 1 << 15),
               ("uniform", 4099, 1 << 15, 1 << 7), ("uniform", 4099, 1 << 18, 1 << 12), ("uniform", 4099, 1 << 17, 1 << 12),
               ("uniform", 4099, 1 << 20, 1 << 13), ("uniform", 9001, 1 << 14, 1 << 10), ("uniform", 65, 1 << 10, 1 << 7),
               ("ring15", 0, 1 << 14, 1 << 9), ("ring17", 0, 1 << 14, 1 << 9), ("ring60", 0, 1 << 14, 1 << 8),
               ("ring60", 0, 1 << 20, 1 << 15), ("clump", 4000, 1 << 14, 1 << 8), ("clump", 4000, 1 << 20, 1 << 14)]


@pytest.mark.parametrize("kind,n,box,w", STRIP_CASES)
def test_voronoi_strip_wave_and_general_rows_match_oracle(kind, n, box, w):
    if kind.startswith("ring"):
        x, y = _ring_of(int(kind[4:]), box)
    elif kind == "clump":
        x, y = _clump(n, 3000, box, w)
    else:
        x, y, _ = workloads.uniform(n, box=box, seed_pos=n + w)
    try:
        ref = _oracle_rows(x, y, box)
    except oracle.OracleError as e:
        assert e.status == oracle.E_RANGE
        assert _gpu_rows(x, y, box, w, dmax=64)[2] == nm.NM_E_RANGE
        return
    for dmax in (64, max(len(r) for r in ref)):
        ring, deg, st, _ = _gpu_rows(x, y, box, w, dmax=dmax)
        assert st == 0
        assert _rows_of(ring, deg) == ref
        assert (ring[np.arange(dmax)[None, :] >= deg[:, None]] == -1).all()


@pytest.mark.parametrize("m,box,wdiv", [(32, 1 << 20, 1), (32, 1 << 20, 2), (64, 1 << 16, 1), (64, 1 << 16, 4)])
def test_voronoi_square_lattice_degenerate(m, box, wdiv):
    # four co-circular particles at every lattice square: only the axis neighbours
    x, y, a = workloads.lattice(m, box=box)
    ring, deg, st, _ = _gpu_rows(x, y, box, a // wdiv)
    assert st == 0
    assert _rows_of(ring, deg) == _oracle_rows(x, y, box)
    assert (deg == 4).all()


def test_voronoi_perturbed_lattice_worked_example():
    x, y, a = workloads.lattice(8)
    x, y = x.copy(), y.copy()
    x[0], y[0] = 1, 1
    ring, deg, st, _ = _gpu_rows(x, y, workloads.BOX, a)
    assert st == 0
    rows = _rows_of(ring, deg)
    assert rows == _oracle_rows(x, y, workloads.BOX)
    assert rows[0] == [9, 8, 7, 56, 1] and rows[7] == [0, 8, 15, 6, 63, 56]


def test_voronoi_centred_lattice_and_small_box():
    m, box = 16, 1 << 20
    a = box // m
    idx = np.arange(m * m)
    r, c = idx // m, idx % m
    x = (c * a + (r % 2) * (a // 2)).astype(np.int32)
    y = (r * a).astype(np.int32)
    ring, deg, st, _ = _gpu_rows(x, y, box, a)
    assert st == 0 and (deg == 6).all()
    assert _rows_of(ring, deg) == _oracle_rows(x, y, box)
    # the same lattice scaled into a 2^12 box (narrow cells, tiny offsets)
    s = box // (1 << 12)
    ring, deg, st, _ = _gpu_rows(x // s, y // s, 1 << 12, a // s)
    assert st == 0 and _rows_of(ring, deg) == _oracle_rows(x // s, y // s, 1 << 12)


@pytest.mark.parametrize("case", ["pairs", "lattice_sites"])
def test_voronoi_coincident_particles_share_a_site(case):
    if case == "pairs":  # a few coincident pairs and a triple in a uniform set
        n, box, w = 4097, 1 << 16, 1024
        x, y, _ = workloads.uniform(n, box=box, seed_pos=31)
        for a, b in ((9, 5), (40, 5), (100, 3000), (7, 8)):
            x[a], y[a] = x[b], y[b]
    else:  # 4097 particles on the sites of a 32 x 32 lattice (degenerate too)
        n, box, w = 4097, 1 << 16, 2048
        x, y, _ = workloads.uniform(n, box=box, seed_pos=32)
        x, y = (x // 2048) * 2048, (y // 2048) * 2048
    ring, deg, st, _ = _gpu_rows(x, y, box, w, dmax=64)
    assert st == 0
    assert _rows_of(ring, deg) == _oracle_rows(x, y, box)


def test_voronoi_errors():
    x, y, _ = workloads.uniform(6)  # cells beyond L/8
    _, _, st, _ = _gpu_rows(x, y, workloads.BOX, 1 << 17)
    assert st == nm.NM_E_RANGE
    x, y, _ = workloads.uniform(4097, box=1 << 16)
    _, deg, st, _ = _gpu_rows(x, y, 1 << 16, 1024, dmax=5)  # rows of 6+ entries
    assert st == nm.NM_E_CAPACITY and deg.max() == 5
    with pytest.raises(nm.NMError):
        ws = nm.Workspace(4097, 1 << 16, 1024)
        nm.voronoi(ws, 65)


def test_voronoi_full_size_sampled_and_invariants():
    n, box = 1 << 20, workloads.BOX
    x, y, _ = workloads.uniform(n)
    ring_t, deg_t = None, None
    for w in (1024, 2048):
        ring, deg, st, _ = _gpu_rows(x, y, box, w)
        assert st == 0
        if ring_t is None:
            ring_t, deg_t = ring, deg
        else:  # the lists do not depend on the cell width
            assert np.array_equal(ring, ring_t) and np.array_equal(deg, deg_t)
    assert int(deg_t.sum()) == 6 * n  # Euler on the torus (general position)
    # reciprocity of every row
    ii = np.repeat(np.arange(n), deg_t)
    jj = ring_t[ring_t >= 0]
    a = np.sort(ii.astype(np.int64) * n + jj)
    b = np.sort(jj.astype(np.int64) * n + ii)
    assert np.array_equal(a, b)
    rows = np.unique(np.random.default_rng(5).integers(0, n, 400)).astype(np.int32)
    ref = _oracle_rows(x, y, box, rows=rows, rho0=4096)
    assert [ring_t[r, :deg_t[r]].tolist() for r in rows] == ref


def _moved(x, y, box, step, seed):
    rng = np.random.default_rng(seed)
    return ((x + rng.integers(-step, step + 1, len(x))) % box).astype(np.int32), \
           ((y + rng.integers(-step, step + 1, len(y))) % box).astype(np.int32)


@pytest.mark.parametrize("step,coincide", [(0, None), (8, None), (64, None), (400, None), (0, "stay"),
                                           (8, "stay"), (0, "change"), (8, "change")])
def test_reuse_test_and_update(step, coincide):
    n, box, w = 8191, 1 << 16, 1024
    x0, y0, _ = workloads.uniform(n, box=box, seed_pos=71)
    x1, y1 = _moved(x0, y0, box, step, 72)
    if coincide:  # coincident pairs (and a triple) that stay together
        for a, b in ((5, 6), (70, 71), (72, 71)):
            x0[a], y0[a] = x0[b], y0[b]
            x1[a], y1[a] = x1[b], y1[b]
    if coincide == "change":  # pairs that form, a pair that parts
        for a, b in ((300, 301), (4000, 17)):
            x1[a], y1[a] = x1[b], y1[b]
        x0[900], y0[900] = x0[901], y0[901]
    ring0, deg0, st, _ = _gpu_rows(x0, y0, box, w)
    assert st == 0
    ref1 = _oracle_rows(x1, y1, box)
    ws1 = nm.Workspace(n, box, w)
    X1, Y1 = _dev(x1, torch.int32), _dev(y1, torch.int32)
    nm.build_cells(ws1, X1, Y1)
    ring, deg = _dev(ring0, torch.int32), _dev(deg0, torch.int32)
    stale, nfail = nm.voronoi_check(ws1, X1, Y1, ring, deg)
    assert nm.check(ws1) == 0
    stale = stale.cpu().numpy().astype(bool)
    old = _rows_of(ring0, deg0)
    changed = np.array([set(old[i]) != set(ref1[i]) for i in range(n)])
    if step == 0 and coincide != "change":  # nothing moved: the rows are certified as they are
        assert int(nfail.item()) == 0 and not stale.any()
    if int(nfail.item()) == 0:  # the certificate: no failure, no change
        assert not changed.any() and not stale.any()
    if changed.any():
        assert int(nfail.item()) > 0 and stale.any()
    nf = nm.voronoi_update(ws1, X1, Y1, ring, deg)
    assert nm.check(ws1) == 0
    assert int(nf.item()) == int(nfail.item())
    assert _rows_of(ring.cpu().numpy(), deg.cpu().numpy()) == ref1


# Rows held in registers (up to 12 entries, rows of 12 or more) and rows walked
# by index; no row failing, a few, and most of them; both in the cells' order
# (the update) and in the caller's (the check alone).
@pytest.mark.parametrize("kind,dmax,move", [("lattice", 11, 0), ("lattice", 12, 0), ("lattice", 11, 40), ("lattice", 12, 40),
                                            ("lattice", 64, 400), ("ring", 64, 0), ("ring", 64, 20), ("pairs", 16, 30)])
def test_update_short_long_and_shared_rows(kind, dmax, move):
    box, w = 1 << 16, 1 << 11
    rng = np.random.default_rng(dmax + move)
    if kind == "ring":
        x, y = _ring_of(40, box)
    else:
        m, a = 32, box // 32
        i = np.arange(m * m)
        x = (i % m) * a + (i // m % 2) * (a // 2) + rng.integers(-60, 61, m * m)
        y = (i // m) * a + rng.integers(-60, 61, m * m)
        if kind == "pairs":
            x[[5, 300, 301]], y[[5, 300, 301]] = x[[700, 900, 900]], y[[700, 900, 900]]
    n = len(x)
    x, y = x.astype(np.int64) % box, y.astype(np.int64) % box
    # a turn of every row's start comes with the common shift, failures with the rest
    x1 = ((x + 3 + rng.integers(-move, move + 1, n)) % box).astype(np.int32)
    y1 = ((y - 2 + rng.integers(-move, move + 1, n)) % box).astype(np.int32)
    if kind == "pairs":  # they move together
        x1[[5, 300, 301]], y1[[5, 300, 301]] = x1[[700, 900, 900]], y1[[700, 900, 900]]
    x, y = x.astype(np.int32), y.astype(np.int32)
    ring, deg, st, ws = _gpu_rows(x, y, box, w, dmax=dmax)
    assert st == 0
    R, D, X1, Y1 = _dev(ring, torch.int32), _dev(deg, torch.int32), _dev(x1, torch.int32), _dev(y1, torch.int32)
    alone = int(nm.voronoi_check(ws, X1, Y1, R, D)[1].item())
    nm.build_cells(ws, X1, Y1)
    nfail = int(nm.voronoi_update(ws, X1, Y1, R, D).item())
    assert nm.check(ws) == 0 and nfail == alone
    assert move > 0 or nfail == 0
    assert _rows_of(R.cpu().numpy(), D.cpu().numpy()) == _oracle_rows(x1, y1, box)


# Rounds of stale rows (few failures) and all rows at once (more than one in
# 512), on strips and on a grid too coarse for them.
@pytest.mark.parametrize("moved", [1, 3, 4, 5, 40, 4096])
@pytest.mark.parametrize("w", [1024, 1 << 14])
def test_update_rebuilds_stale_rows_or_all(moved, w):
    n, box = 4096, 1 << 16
    x, y, _ = workloads.uniform(n, box=box, seed_pos=91)
    ring, deg, st, ws = _gpu_rows(x, y, box, w)
    assert st == 0
    rng = np.random.default_rng(moved)
    x1, y1 = x.copy(), y.copy()
    who = rng.choice(n, moved, replace=False)
    x1[who] = (x1[who] + rng.integers(300, 900, moved)) % box
    R, D, X1, Y1 = _dev(ring, torch.int32), _dev(deg, torch.int32), _dev(x1, torch.int32), _dev(y1, torch.int32)
    nm.build_cells(ws, X1, Y1)
    want = _oracle_rows(x1, y1, box)
    for _ in range(2):  # the second update finds nothing to do
        nfail = nm.voronoi_update(ws, X1, Y1, R, D)
        assert nm.check(ws) == 0
        assert _rows_of(R.cpu().numpy(), D.cpu().numpy()) == want
    assert int(nfail.item()) == 0


def test_update_all_rows_keeps_a_passing_row_beyond_the_domain():
    # A void whose rim particles' cells reach past L/8: such rows are outside the
    # lists' domain for nm_voronoi, but rows that pass the reuse test are kept by
    # the update, also where so many others fail that every row is built again.
    # (rows by the oracle's definition on the periodic images: scipy's Qhull)
    from scipy.spatial import Delaunay
    box, w = 1 << 14, 1 << 10
    rng = np.random.default_rng(12)
    x, y, _ = workloads.uniform(3000, box=box, seed_pos=92)
    far = (x.astype(np.int64) - box // 2) ** 2 + (y.astype(np.int64) - box // 2) ** 2 > (box / 7.6) ** 2
    x, y = x[far], y[far]
    n = len(x)

    def rows(px, py):
        off = np.array([(a, b) for a in (0, -1, 1) for b in (0, -1, 1)]) * box
        pts = np.concatenate([np.stack([px, py], 1) + o for o in off])
        t = Delaunay(pts)
        start, nb = t.vertex_neighbor_vertices
        out = []
        for i in range(n):
            j = nb[start[i]:start[i + 1]]
            d = pts[j] - pts[i]
            a = np.arctan2(d[:, 1], d[:, 0]) % (2 * np.pi)
            out.append((j[np.argsort(a)] % n).astype(np.int32))
        return out

    near_rim = (x.astype(np.int64) - box // 2) ** 2 + (y.astype(np.int64) - box // 2) ** 2 < (box // 4) ** 2
    was = rows(x.astype(np.int64), y.astype(np.int64))
    dmax = max(len(r) for r in was) + 4
    ring = np.full((n, dmax), -1, np.int32)
    for i, r in enumerate(was):
        ring[i, :len(r)] = r
    deg = np.array([len(r) for r in was], np.int32)
    # particles away from the void move; those around it stay
    x1, y1 = x.copy(), y.copy()
    mv = np.flatnonzero(~near_rim)
    mv = mv[(np.abs(x[mv] - box // 2) > box // 3) | (np.abs(y[mv] - box // 2) > box // 3)]
    x1[mv] = (x1[mv] + rng.integers(-60, 61, len(mv))) % box
    y1[mv] = (y1[mv] + rng.integers(-60, 61, len(mv))) % box
    ws = nm.Workspace(n, box, w)
    X1, Y1 = _dev(x1, torch.int32), _dev(y1, torch.int32)
    nm.build_cells(ws, X1, Y1)
    nm.voronoi(ws, dmax)
    assert nm.check(ws) == nm.NM_E_RANGE  # the domain, for every row built anew
    ws = nm.Workspace(n, box, w)
    nm.build_cells(ws, X1, Y1)
    R, D = _dev(ring, torch.int32), _dev(deg, torch.int32)
    nfail = int(nm.voronoi_update(ws, X1, Y1, R, D).item())
    assert nm.check(ws) == 0
    assert nfail * 512 > n
    got = _rows_of(R.cpu().numpy(), D.cpu().numpy())
    assert got == [r.tolist() for r in rows(x1.astype(np.int64), y1.astype(np.int64))]


def test_update_from_unrelated_rows():
    n, box, w = 4097, 1 << 16, 1024
    xa, ya, _ = workloads.uniform(n, box=box, seed_pos=81)
    xb, yb, _ = workloads.uniform(n, box=box, seed_pos=82)
    ring0, deg0, st, _ = _gpu_rows(xa, ya, box, w)
    ws = nm.Workspace(n, box, w)
    X, Y = _dev(xb, torch.int32), _dev(yb, torch.int32)
    nm.build_cells(ws, X, Y)
    ring, deg = _dev(ring0, torch.int32), _dev(deg0, torch.int32)
    nf = nm.voronoi_update(ws, X, Y, ring, deg)
    assert nm.check(ws) == 0 and int(nf.item()) > 0
    assert _rows_of(ring.cpu().numpy(), deg.cpu().numpy()) == _oracle_rows(xb, yb, box)
    # garbage rows (out-of-range indices, bad degrees) are flagged, never read through
    ring.fill_(-7)
    deg.fill_(99)
    nm.voronoi_update(ws, X, Y, ring, deg)
    assert nm.check(ws) == 0
    assert _rows_of(ring.cpu().numpy(), deg.cpu().numpy()) == _oracle_rows(xb, yb, box)


@pytest.mark.parametrize("include_self,variant", [(1, 0), (0, nm.NM_NOISE_SCALAR | nm.NM_MOVE_NEW_HEADING)])
def test_voronoi_vicsek_step_matches_oracle(include_self, variant):
    # the Vicsek model with Voronoi neighbours (Sec. IV): Eq. (2) over the rows
    n, box = 8191, 1 << 16
    x, y, th = workloads.uniform(n, box=box, seed_pos=91)
    ring, deg, st, _ = _gpu_rows(x, y, box, 1024)
    assert st == 0
    off, idx = oracle.voronoi(x, y, box)
    p = nm.make_params(box, v0=64, eta=0.3, include_self=include_self, seed=4, sys_id=1, variant=variant)
    xo, yo, to = nm.align_step(_dev(x, torch.int32), _dev(y, torch.int32), _dev(th, torch.float32), p, 3,
                               nbr=_dev(ring, torch.int32))
    torch.cuda.synchronize()
    rx, ry, rt = oracle.align_step(x, y, th, box, offsets=off, idx=idx, v0=64, eta=0.3, seed=4, sys_id=1,
                                   include_self=include_self, step=3, variant=variant)
    assert np.array_equal(xo.cpu().numpy(), rx) and np.array_equal(yo.cpu().numpy(), ry)
    d = np.abs(np.remainder(to.cpu().numpy().astype(np.float64) - rt + np.pi, 2 * np.pi) - np.pi)
    assert d.max() <= TOL
    # the oracle reads padded rows the same way
    rx2, ry2, rt2 = oracle.align_step(x, y, th, box, nbr=ring, v0=64, eta=0.3, seed=4, sys_id=1,
                                      include_self=include_self, step=3, variant=variant)
    assert np.array_equal(rx2, rx) and np.array_equal(ry2, ry) and np.array_equal(rt2, rt)


def _vm_args(n, box):
    a_mean = box * box / n
    return dict(ka=1.0 / a_mean, kp=1.0, a0=0.9 * a_mean, p0=3.7 * np.sqrt(a_mean))


def _force_scale(a):
    return 2 * a["ka"] * a["a0"] * np.sqrt(a["a0"]) + 2 * a["kp"] * a["p0"]


@pytest.mark.parametrize("kind,n,box,w", [("uniform", 4097, 1 << 16, 1024), ("uniform", 3001, 1 << 20, 16384),
                                          ("clustered", 8191, 1 << 20, 4096)])
def test_voronoi_forces_match_oracle(kind, n, box, w):
    # Sec. V: areas, perimeters, Eq. (3), vertex forces (Eqs. 5-8), particle
    # forces (Eqs. 9-19); the oracle works from its own rows
    x, y, _ = _gen(kind, n, box)
    ring, deg, st, ws = _gpu_rows(x, y, box, w)
    assert st == 0
    off, idx = oracle.voronoi(x, y, box)
    a = _vm_args(n, box)
    ref = oracle.voronoi_forces(x, y, box, off, idx, vertices=True, **a)
    got = nm.voronoi_forces(_dev(x, torch.int32), _dev(y, torch.int32), box, _dev(ring, torch.int32),
                            _dev(deg, torch.int32), vertices=True, ws=ws, **a)
    assert nm.check(ws) == 0
    g = {k: v.cpu().numpy() for k, v in got.items()}
    scale = _force_scale(a)
    assert np.allclose(g["area"], ref["area"], rtol=1e-12, atol=0)
    assert np.allclose(g["perim"], ref["perim"], rtol=1e-12, atol=0)
    assert abs(g["energy"][0] - ref["energy"]) <= 1e-12 * abs(ref["energy"])
    assert np.abs(g["fx"] - ref["fx"]).max() <= 1e-9 * scale
    assert np.abs(g["fy"] - ref["fy"]).max() <= 1e-9 * scale
    v = g["vertex"]
    sel = np.arange(ring.shape[1])[None, :] < deg[:, None]
    for c, key in enumerate(("hx", "hy", "vfx", "vfy")):
        tol = 1e-9 * (box if c < 2 else scale)
        assert np.abs(v[..., c][sel] - ref[key]).max() <= tol


# Rows on both sides of the eight lanes that share a particle and of the rows
# read whole, and rows too narrow for that; the same bits in every order.
@pytest.mark.parametrize("m,dmax", [(6, 7), (7, 16), (8, 16), (9, 16), (15, 16), (17, 64), (40, 64)])
def test_voronoi_forces_rows_around_the_lane_group(m, dmax):
    box, w = 1 << 14, 1 << 9
    if dmax < 8:  # the centred lattice, a little out of place: six neighbours each
        i = np.arange(32 * 32)
        rng = np.random.default_rng(3)
        x = ((i % 32) * 512 + (i // 32 % 2) * 256 + rng.integers(-20, 21, len(i))) % box
        y = ((i // 32) * 512 + rng.integers(-20, 21, len(i))) % box
        x, y = x.astype(np.int32), y.astype(np.int32)
    else:
        x, y = _ring_of(m, box)
    n = len(x)
    ring, deg, st, ws = _gpu_rows(x, y, box, w, dmax=dmax)
    assert st == 0 and m in deg
    off, idx = oracle.voronoi(x, y, box)
    a = _vm_args(n, box)
    ref = oracle.voronoi_forces(x, y, box, off, idx, **a)
    args = (_dev(x, torch.int32), _dev(y, torch.int32), box, _dev(ring, torch.int32), _dev(deg, torch.int32))
    other = nm.Workspace(n + 1, box, w)
    got = [nm.voronoi_forces(*args, ws=q, **a) for q in (ws, None, other)]
    assert nm.check(ws) == 0 and nm.check(other) == 0
    for k in ("area", "perim", "fx", "fy", "energy"):
        assert torch.equal(got[0][k], got[1][k]) and torch.equal(got[0][k], got[2][k])
    scale = _force_scale(a)
    assert np.allclose(got[0]["area"].cpu().numpy(), ref["area"], rtol=1e-12, atol=0)
    assert np.allclose(got[0]["perim"].cpu().numpy(), ref["perim"], rtol=1e-12, atol=0)
    assert np.abs(got[0]["fx"].cpu().numpy() - ref["fx"]).max() <= 1e-9 * scale
    assert np.abs(got[0]["fy"].cpu().numpy() - ref["fy"]).max() <= 1e-9 * scale


def test_voronoi_forces_vanish_on_the_centred_lattice():
    m, box = 16, 1 << 20
    a = box // m
    idx = np.arange(m * m)
    r, c = idx // m, idx % m
    x = (c * a + (r % 2) * (a // 2)).astype(np.int32)
    y = (r * a).astype(np.int32)
    ring, deg, st, ws = _gpu_rows(x, y, box, a)
    assert st == 0
    args = dict(ka=1.0, kp=1.0, a0=0.9 * a * a, p0=3.0 * a)
    got = nm.voronoi_forces(_dev(x, torch.int32), _dev(y, torch.int32), box, _dev(ring, torch.int32),
                            _dev(deg, torch.int32), ws=ws, **args)
    assert np.allclose(got["area"].cpu().numpy(), a * a, rtol=1e-13)
    assert np.allclose(got["perim"].cpu().numpy(), a * (np.sqrt(5.0) + 1.5), rtol=1e-13)
    scale = 2 * (0.1 * a * a) * a + 2 * abs(a * (np.sqrt(5.0) + 1.5) - 3.0 * a)
    assert got["fx"].abs().max().item() <= 1e-9 * scale and got["fy"].abs().max().item() <= 1e-9 * scale


def test_voronoi_forces_full_size_sampled():
    n, box = 1 << 20, workloads.BOX
    x, y, _ = workloads.uniform(n)
    ring, deg, st, ws = _gpu_rows(x, y, box, 1024)
    assert st == 0
    a = _vm_args(n, box)
    got = nm.voronoi_forces(_dev(x, torch.int32), _dev(y, torch.int32), box, _dev(ring, torch.int32),
                            _dev(deg, torch.int32), ws=ws, **a)
    assert nm.check(ws) == 0
    area = got["area"].cpu().numpy()
    assert abs(area.sum() - float(box) ** 2) <= 1e-9 * float(box) ** 2  # the cells tile the torus
    rows = np.unique(np.random.default_rng(8).integers(0, n, 200)).astype(np.int32)
    # the oracle's own rows for the sampled particles and their neighbours
    o1, i1 = oracle.voronoi(x, y, box, rows=rows, rho0=4096)
    nb = np.unique(np.concatenate([rows, i1])).astype(np.int32)
    o2, i2 = oracle.voronoi(x, y, box, rows=nb, rho0=4096)
    keep = [np.zeros(0, np.int32)] * n
    for r, p in enumerate(nb):
        keep[p] = i2[o2[r]:o2[r + 1]]
    off = np.zeros(n + 1, np.int64)
    np.cumsum([len(k) for k in keep], out=off[1:])
    ref = oracle.voronoi_forces(x, y, box, off, np.concatenate(keep), rows=rows, **a)
    scale = _force_scale(a)
    assert np.abs(got["fx"].cpu().numpy()[rows] - ref["fx"]).max() <= 1e-9 * scale
    assert np.abs(got["fy"].cpu().numpy()[rows] - ref["fy"]).max() <= 1e-9 * scale
    assert np.allclose(area[nb], ref["area"][nb], rtol=1e-12, atol=0)


def test_voronoi_forces_reject_coincident_particles():
    n, box = 4097, 1 << 16
    x, y, _ = workloads.uniform(n, box=box, seed_pos=6)
    x[11], y[11] = x[12], y[12]
    ring, deg, st, ws = _gpu_rows(x, y, box, 1024)
    assert st == 0
    nm.voronoi_forces(_dev(x, torch.int32), _dev(y, torch.int32), box, _dev(ring, torch.int32),
                      _dev(deg, torch.int32), ws=ws, **_vm_args(n, box))
    assert nm.check(ws) == nm.NM_E_RANGE


def test_voronoi_forces_reject_inconsistent_rows():
    n, box = 4097, 1 << 16
    x, y, _ = workloads.uniform(n, box=box, seed_pos=6)
    assert len(np.unique(x.astype(np.int64) * box + y)) == n  # no coincident particles
    ring, deg, st, ws = _gpu_rows(x, y, box, 1024)
    ring[10, :2] = ring[10, 1::-1]  # swap two neighbours: not a triangulation any more
    nm.voronoi_forces(_dev(x, torch.int32), _dev(y, torch.int32), box, _dev(ring, torch.int32),
                      _dev(deg, torch.int32), ws=ws, **_vm_args(n, box))
    assert nm.check(ws) == nm.NM_E_INVAL


# A workspace without cells may hold anything: a call reports it and follows no
# list that its header seems to count (header words 5: built, 10: cells for the
# 64-bit kernel, 12: rows for the wave and general kernels).
def test_rows_without_cells_are_refused_whatever_the_lists_hold():
    n, box, w = 1000, 1 << 16, 1 << 11
    x, y, _ = workloads.uniform(n, box=box)
    X, Y = _dev(x, torch.int32), _dev(y, torch.int32)
    ws = nm.Workspace(n, box, w)
    nm.build_cells(ws, X, Y)
    ring, deg = nm.voronoi(ws, 16)
    assert nm.check(ws) == 0
    h = ws.buf[:256].view(torch.int32)
    for word in (10, 12):
        h[5], h[word] = 0, 7
        R, D = torch.full_like(ring, -7), torch.full_like(deg, -7)
        nm.voronoi(ws, 16, R, D)
        assert nm.check(ws) == nm.NM_E_INVAL
        assert (R == -7).all() and (D == -7).all()
        h[word] = 0


# The reuse test uses a workspace for its counters only: one of another grid, or
# one never prepared, does, and nothing beyond the 256 bytes of its header is
# written.  The update needs cells, refuses a workspace without, and leaves it alone.
@pytest.mark.parametrize("of", ["this grid", "another grid", "nothing"])
@pytest.mark.parametrize("moved", [0, 40])
def test_check_needs_the_workspace_header_only(of, moved):
    n, box, w = 4096, 1 << 16, 1 << 11
    x, y, _ = workloads.uniform(n, box=box)
    ring, deg, st, good = _gpu_rows(x, y, box, w)
    assert st == 0
    x1 = ((x + np.random.default_rng(2).integers(-moved, moved + 1, n)) % box).astype(np.int32)
    R, D, X1, Y1 = _dev(ring, torch.int32), _dev(deg, torch.int32), _dev(x1, torch.int32), _dev(y, torch.int32)
    stale, nfail = nm.voronoi_check(good, X1, Y1, R, D)
    assert (int(nfail.item()) > 0) == (moved > 0)
    ws = nm.Workspace(300, box, w, nbytes=good.nbytes) if of == "another grid" else nm.Workspace(n, box, w)
    ws.grid = good.grid
    ws.buf[0 if of == "nothing" else 256:] = 0x5A
    ws.buf[4:8] = 0  # (the error word)
    s2, f2 = nm.voronoi_check(ws, X1, Y1, R, D)
    assert nm.check(ws) == 0
    assert torch.equal(stale, s2) and torch.equal(nfail, f2)
    assert (ws.buf[256:] == 0x5A).all()
    nm.voronoi_update(ws, X1, Y1, R, D)
    assert nm.check(ws) == nm.NM_E_INVAL
    assert (ws.buf[256:] == 0x5A).all()
    assert np.array_equal(R.cpu().numpy(), ring) and np.array_equal(D.cpu().numpy(), deg)


# Updates of states that the strips leave much of to the other kernels (dense
# clumps, coincident particles, offsets of more than 16 bits): every row built
# again where many fail, those left by the strips and passing the test kept.
@pytest.mark.parametrize("box,w", [(1 << 14, 1 << 8), (1 << 14, 1 << 11), (1 << 20, 1 << 14), (1 << 20, 1 << 17)])
@pytest.mark.parametrize("move", [1, 6])
def test_update_of_clumped_states_matches_oracle(box, w, move):
    x, y = _clump(900, 1100, box, min(w, 1 << 14))
    n = len(x)
    rng = np.random.default_rng(move)
    x1 = ((x + rng.integers(-move, move + 1, n)) % box).astype(np.int32)
    y1 = ((y + rng.integers(-move, move + 1, n)) % box).astype(np.int32)
    ring, deg, st, ws = _gpu_rows(x, y, box, w, dmax=64)
    assert st == 0
    R, D, X1, Y1 = _dev(ring, torch.int32), _dev(deg, torch.int32), _dev(x1, torch.int32), _dev(y1, torch.int32)
    nm.build_cells(ws, X1, Y1)
    nfail = int(nm.voronoi_update(ws, X1, Y1, R, D).item())
    assert nm.check(ws) == 0
    assert nfail * 512 > n
    assert _rows_of(R.cpu().numpy(), D.cpu().numpy()) == _oracle_rows(x1, y1, box)


# Equal and nearly equal circle parameters on strips: lattices whose particles
# are all co-circular in fours, or are up to a few units out of place, in
# wide and narrow strips, and rings of particles on one circle (up to 12 ties a step).
@pytest.mark.parametrize("jitter", [0, 1, 2])
@pytest.mark.parametrize("rings,box,w", [(True, 1 << 14, 1 << 8), (True, 1 << 20, 1 << 14), (False, 1 << 16, 1 << 9),
                                         (False, 1 << 20, 1 << 14)])
def test_voronoi_strips_near_ties(rings, box, w, jitter):
    x, y, a = workloads.lattice(64, box=box)
    x, y = x.astype(np.int64), y.astype(np.int64)
    if rings:  # nothing inside the circle through the twelve lattice points at distance 5 of some
        keep = np.ones(len(x), bool)
        for c in range(0, len(x), 650):
            d = (x // a - x[c] // a + 32) % 64 - 32, (y // a - y[c] // a + 32) % 64 - 32
            r2 = d[0] ** 2 + d[1] ** 2
            keep &= (r2 >= 25) | (r2 == 0)
        x, y = x[keep], y[keep]
    rng = np.random.default_rng(jitter)
    x = ((x + rng.integers(-jitter, jitter + 1, len(x))) % box).astype(np.int32)
    y = ((y + rng.integers(-jitter, jitter + 1, len(y))) % box).astype(np.int32)
    ring, deg, st, _ = _gpu_rows(x, y, box, w, dmax=32)
    assert st == 0
    some = np.arange(0, len(x), 8, dtype=np.int32)
    got = _rows_of(ring, deg)
    assert [got[i] for i in some] == _oracle_rows(x, y, box, rows=some)


# Coincident particles in rows from strips (16-bit and 32-bit offsets): sites of
# one to four particles in shuffled order, rows that just fit dmax and that don't.
@pytest.mark.parametrize("box,w", [(1 << 14, 1 << 9), (1 << 20, 1 << 15), (1 << 14, 1 << 7)])
@pytest.mark.parametrize("most", [2, 4])
def test_voronoi_strips_shared_sites(box, w, most):
    rng = np.random.default_rng(most)
    x, y, _ = workloads.uniform(700, box=box, seed_pos=most)
    times = rng.integers(1, most + 1, 700) if most > 2 else np.full(700, 2)
    x, y = np.repeat(x, times), np.repeat(y, times)
    o = rng.permutation(len(x))
    x, y = x[o], y[o]
    ref = _oracle_rows(x, y, box)
    longest = max(len(r) for r in ref)
    for dmax in (longest, longest - 1):
        ring, deg, st, _ = _gpu_rows(x, y, box, w, dmax=dmax)
        assert st == (0 if dmax == longest else nm.NM_E_CAPACITY)
        assert _rows_of(ring, deg) == [r[:dmax] for r in ref]
        assert (ring[np.arange(dmax)[None, :] >= deg[:, None]] == -1).all()


# Both ways an update goes on strips, each shown to be taken by the first test's
# count: rounds of stale rows while at most one row in 512 fails, every row at
# once beyond; the rows are those of a build from nothing.
@pytest.mark.parametrize("moved,rounds", [(1, True), (4, True), (8, True), (400, False), (1 << 16, False)])
@pytest.mark.parametrize("box,w", [(1 << 18, 1 << 10), (1 << 20, 1 << 13)])
def test_update_takes_rounds_or_all_rows(moved, rounds, box, w):
    n = 1 << 16
    x, y, _ = workloads.uniform(n, box=box, seed_pos=94)
    X, Y = _dev(x, torch.int32), _dev(y, torch.int32)
    ws = nm.Workspace(n, box, w)
    nm.build_cells(ws, X, Y)
    R, D = nm.voronoi(ws, 24)
    assert nm.check(ws) == 0
    rng = np.random.default_rng(moved)
    x1, y1 = x.copy(), y.copy()
    who = rng.choice(n, moved, replace=False)
    x1[who] = (x1[who] + rng.integers(1, box // 256, moved)) % box
    X1, Y1 = _dev(x1, torch.int32), _dev(y1, torch.int32)
    nm.build_cells(ws, X1, Y1)
    nfail = int(nm.voronoi_update(ws, X1, Y1, R, D).item())
    assert nm.check(ws) == 0
    assert 0 < nfail * 512 <= n if rounds else nfail * 512 > n
    R1, D1 = nm.voronoi(ws, 24)
    assert nm.check(ws) == 0
    assert torch.equal(R, R1) and torch.equal(D, D1)
