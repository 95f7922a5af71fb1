"""Performance cases of the tracker: the calls a user's program makes, over the range of sizes, fields and options.

The sizes and field recipes are those of the repository's benchmark workloads and tests (moving Gaussian blobs, blobs
with noise, a blob field rounded to integer levels, moving sources and vortices, random cosine waves, Delaunay
meshes), here evaluated on the GPU as products of separable terms.

listed() and draw() give cases; prepare() makes what a program holds before the call; run() is one pass; work() the
bytes and operations a pass cannot do without; exact() the floating outputs in 64 bits, in plain torch.
"""
import itertools
import math

import numpy as np
import torch

import paper_2011_08697_amd as F
from paper_2011_08697_amd import synth

OUT_ALL = F.OUT_ALL


def listed():
    return [
        # The smallest call: a 64 x 64 x 10 scalar field, a few hundred hits.  Interactive use; launches and host
        # work are all of it.
        dict(name="scalar_64", path="track2d", recipe="blobs", nx=64, ny=64, nt=10, blobs=8, amp=1.0, precision=0,
             outputs=0),
        # A serving loop that may not allocate, on image-like integer data (16 levels: the perturbation decides most
        # zeros), 64-bit evaluation and every output asked for; odd sizes.
        dict(name="into_levels_509", path="into2d", recipe="levels", nx=509, ny=383, nt=24, blobs=48, amp=1.0,
             precision=1, outputs=OUT_ALL),
        # The headline workload: noisy measurements, dense hits (1.7 per vertex).
        dict(name="noise_1024", path="track2d", recipe="noise", nx=1024, ny=1024, nt=100, blobs=256, amp=1.0,
             precision=0, outputs=0),
        # A large simulation's velocity field, sparse hits.
        dict(name="vector_4096", path="track2d", recipe="vector", nx=4096, ny=4096, nt=50, blobs=1024, amp=1.0,
             precision=0, outputs=0),
        # A velocity field in physical units (components of a few tens: beyond the narrow integer range); odd sizes.
        dict(name="vector_wide_1021", path="track2d", recipe="vector", nx=1021, ny=769, nt=40, blobs=96, amp=800.0,
             precision=0, outputs=0),
        # Many independent series of uneven sizes in one call (an ensemble).
        dict(name="batch_12", path="batch2d", recipe="blobs", series=12, shape_seed=3, lo=128, hi=2048, nt_lo=8,
             nt_hi=64, amp=1.0),
        # In-situ use: one step pushed at a time while a simulation runs; ragged width.
        dict(name="stream_500", path="stream", recipe="blobs", nx=500, ny=384, nz=0, nt=24, blobs=32, amp=1.0),
        # Critical points of a 3D scalar series.
        dict(name="blobs3d_256", path="track3d", recipe="blobs3d", nx=256, ny=256, nz=256, nt=16, blobs=512, amp=1.0),
        # Level set of the same series.
        dict(name="iso3d_256", path="iso3d", recipe="blobs3d", nx=256, ny=256, nz=256, nt=16, blobs=512, amp=1.0,
             isovalue=0.5),
        # Vortex surfaces of a complex series at the superconductivity grid's shape.
        dict(name="vortex3d_512", path="vortex3d", recipe="waves", nx=512, ny=128, nz=64, nt=8, waves=8),
        # Critical points on an unstructured mesh, topology kept in a handle.
        dict(name="mesh_200k", path="mesh2d", recipe="mesh", points=200000, nt=40, terms=16),
        # Post-processing of a dense result: table, order, smoothing, simplification, loop filter, one slice.
        dict(name="post_noise_1024", path="post2d", recipe="noise", nx=1024, ny=1024, nt=24, blobs=256, amp=1.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: sizes spread over their logarithm, odd ones among them."""
    path = rng.choice(["track2d", "track2d", "track2d", "into2d", "batch2d", "stream", "track3d", "iso3d", "vortex3d",
                       "mesh2d", "post2d"])
    if path in ("track2d", "into2d", "post2d"):
        big = {"track2d": 3.0e7, "into2d": 3.0e6, "post2d": 1.2e7}[path]
        nx, ny, nt = _log_int(rng, 48, 2200), _log_int(rng, 48, 2200), _log_int(rng, 4, 64)
        nt = max(3, min(nt, int(big / (nx * ny))))
        ny = max(16, min(ny, int(big / (nx * nt))))
        recipe = rng.choice(["blobs", "noise", "levels", "vector"]) if path != "post2d" else rng.choice(["blobs", "noise"])
        c = dict(path=path, recipe=recipe, nx=nx, ny=ny, nt=nt, blobs=max(8, min(1024, nx * ny // 8192)),
                 amp=rng.choice([1.0, 1.0, 800.0]) if recipe == "vector" else 1.0)
        if path != "post2d":
            c["precision"] = rng.choice([0, 0, 0, 1])
            c["outputs"] = rng.choice([0, 0, OUT_ALL])
        return c
    if path == "batch2d":
        return dict(path=path, recipe="blobs", series=rng.randint(2, 12), shape_seed=rng.randint(100, 10 ** 6), lo=64,
                    hi=rng.choice([256, 512, 1024]), nt_lo=4, nt_hi=40, amp=1.0)
    if path == "stream":
        if rng.random() < 0.3:
            n = [_log_int(rng, 24, 100) for _ in range(3)]
            return dict(path=path, recipe="blobs3d", nx=n[0], ny=n[1], nz=n[2], nt=rng.randint(4, 12),
                        blobs=max(8, n[0] * n[1] * n[2] // 32768), amp=1.0)
        nx, ny = _log_int(rng, 64, 1400), _log_int(rng, 64, 1400)
        return dict(path=path, recipe=rng.choice(["blobs", "vector", "noise"]), nx=nx, ny=ny, nz=0,
                    nt=rng.randint(4, 32), blobs=max(8, nx * ny // 8192), amp=1.0)
    if path in ("track3d", "iso3d"):
        n = [_log_int(rng, 20, 200) for _ in range(3)]
        c = dict(path=path, recipe="blobs3d", nx=n[0], ny=n[1], nz=n[2], nt=rng.randint(3, 14),
                 blobs=max(8, n[0] * n[1] * n[2] // 32768), amp=1.0)
        if path == "iso3d":
            c["isovalue"] = rng.choice([0.25, 0.5, 0.75])
        return c
    if path == "vortex3d":
        return dict(path=path, recipe="waves", nx=_log_int(rng, 16, 300), ny=_log_int(rng, 16, 128),
                    nz=_log_int(rng, 12, 64), nt=rng.randint(3, 8), waves=rng.choice([4, 8]))
    return dict(path="mesh2d", recipe="mesh", points=_log_int(rng, 500, 150000), nt=rng.randint(4, 48),
                terms=rng.choice([8, 16]))


# ---------------------------------------------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------------------------------------------
def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _blob_terms(rng, K, dims, sigma, vmax):
    sign = np.where(rng.random(K) < 0.5, -1.0, 1.0) * rng.uniform(0.5, 1.5, K)
    sig = rng.uniform(sigma[0], sigma[1], K)
    centre = np.stack([rng.uniform(0.0, float(n), K) for n in dims], axis=1)
    vel = np.stack([rng.uniform(-vmax, vmax, K) for _ in dims], axis=1)
    put = lambda a: torch.from_numpy(a).to(_dev())  # noqa: E731
    return put(sign), put(sig), put(centre), put(vel)


def _axis(n, centre, sig):
    """Per blob: offsets from the centre along one axis and the Gaussian factor, [K][n] in 64 bits."""
    d = torch.arange(n, dtype=torch.float64, device=_dev())[None, :] - centre[:, None]
    return d, torch.exp(-(d * d) / (2.0 * sig * sig)[:, None])


def _blobs2d(nx, ny, nt, K, seed, amp, noise):
    rng = np.random.Generator(np.random.PCG64(seed))
    a, sig, c, v = _blob_terms(rng, K, (nx, ny), (4.0, 10.0), 1.0)
    gen = torch.Generator(device=_dev())
    gen.manual_seed(seed)
    out = torch.empty((nt, ny, nx), dtype=torch.float32, device=_dev())
    for t in range(nt):
        _, ex = _axis(nx, c[:, 0] + v[:, 0] * t, sig)
        _, ey = _axis(ny, c[:, 1] + v[:, 1] * t, sig)
        f = (ey * (amp * a)[:, None]).t().contiguous() @ ex
        if noise:
            f += noise * torch.randn(f.shape, generator=gen, dtype=torch.float64, device=_dev())
        out[t] = f
    return out


def _vector2d(nx, ny, nt, K, seed, amp):
    """Half the blobs contribute grad G (sources, sinks), half the rotated gradient (vortices)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    a, sig, c, v = _blob_terms(rng, K, (nx, ny), (16.0, 48.0), 2.0)
    vort = torch.from_numpy(rng.random(K) < 0.5).to(_dev())
    w = -(amp * a) / (sig * sig)
    out = torch.empty((nt, 2, ny, nx), dtype=torch.float32, device=_dev())
    for t in range(nt):
        dx, ex = _axis(nx, c[:, 0] + v[:, 0] * t, sig)
        dy, ey = _axis(ny, c[:, 1] + v[:, 1] * t, sig)
        gxx, gyy = ex * dx, ey * dy * w[:, None]
        exw, eyw = ex, ey * w[:, None]
        s, r = (~vort)[:, None], vort[:, None]
        # gx = (w ey) (dx ex), gy = (w dy ey) ex; sources (gx, gy), vortices (-gy, gx)
        yu = torch.where(s, eyw, -gyy).t().contiguous()
        yv = torch.where(s, gyy, eyw).t().contiguous()
        out[t, 0] = yu @ torch.where(s, gxx, exw)
        out[t, 1] = yv @ torch.where(r, gxx, exw)
    return out


def _blobs3d(nx, ny, nz, nt, K, seed, amp):
    rng = np.random.Generator(np.random.PCG64(seed))
    a, sig, c, v = _blob_terms(rng, K, (nx, ny, nz), (6.0, 16.0), 1.0)
    out = torch.empty((nt, nz, ny, nx), dtype=torch.float32, device=_dev())
    for t in range(nt):
        e = [_axis(n, c[:, i] + v[:, i] * t, sig)[1] for i, n in enumerate((nx, ny, nz))]
        yx = (e[1][:, :, None] * e[0][:, None, :]).reshape(K, ny * nx)
        out[t] = ((e[2] * (amp * a)[:, None]).t().contiguous() @ yx).view(nz, ny, nx)
    return out


def _waves3d(nx, ny, nz, nt, K, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    X, Y, Z = (torch.arange(n, dtype=torch.float64, device=_dev()) for n in (nx, ny, nz))
    out = torch.empty((nt, 2, nz, ny, nx), dtype=torch.float32, device=_dev())
    for part in range(2):
        d = rng.normal(size=(K, 3))
        d /= np.linalg.norm(d, axis=1, keepdims=True)
        kv = d * (2 * np.pi / rng.uniform(6.0, 16.0, size=K))[:, None]
        w = 2 * np.pi / rng.uniform(6.0, 20.0, size=K)
        a = rng.uniform(0.5, 1.5, size=K)
        phi = rng.uniform(0, 2 * np.pi, size=K)
        for t in range(nt):
            acc = torch.zeros((nz, ny, nx), dtype=torch.float64, device=_dev())
            for k in range(K):
                acc += a[k] * torch.cos((kv[k, 2] * Z)[:, None, None] + (kv[k, 1] * Y)[None, :, None]
                                        + (kv[k, 0] * X + (phi[k] - w[k] * t))[None, None, :])
            out[t, part] = acc
    return out


def _mesh(c, seed):
    xy, tri = synth.delaunay_mesh(c["points"], extent=100.0, seed=seed)
    xy, tri = torch.from_numpy(xy).to(_dev()), torch.from_numpy(np.ascontiguousarray(tri, np.int32)).to(_dev())
    rng = np.random.Generator(np.random.PCG64(seed))
    P = xy.double() / 10.0
    f = torch.zeros((c["nt"], 2, xy.shape[0]), dtype=torch.float64, device=_dev())
    T = torch.arange(c["nt"], dtype=torch.float64, device=_dev())
    for _ in range(c["terms"]):
        p, v, rot = rng.uniform(1, 9, 2), rng.uniform(-0.1, 0.1, 2), rng.uniform(0, np.pi)
        dx = P[None, :, 0] - (p[0] + v[0] * T)[:, None]
        dy = P[None, :, 1] - (p[1] + v[1] * T)[:, None]
        w = torch.exp(-(dx * dx + dy * dy) / 2.0)
        f[:, 0] += w * (math.cos(rot) * dx - math.sin(rot) * dy)
        f[:, 1] += w * (math.sin(rot) * dx + math.cos(rot) * dy)
    return xy, tri, f.float()


def _field(c, seed):
    r = c["recipe"]
    if r == "vector":
        return _vector2d(c["nx"], c["ny"], c["nt"], c["blobs"], seed, c["amp"])
    if r == "blobs3d":
        return _blobs3d(c["nx"], c["ny"], c["nz"], c["nt"], c["blobs"], seed, c["amp"])
    if r == "waves":
        return _waves3d(c["nx"], c["ny"], c["nz"], c["nt"], c["waves"], seed)
    f = _blobs2d(c["nx"], c["ny"], c["nt"], c["blobs"], seed, c["amp"], 0.0 if r == "blobs" else 1e-3)
    if r == "levels":
        lo, hi = f.min().double(), f.max().double()
        f = torch.round((f.double() - lo) / (hi - lo) * 15.0).float()
    return f


def _shapes(c):
    """Sizes of a batch's series (nx, ny, nt, blobs), the recipe of the benchmark's uneven batch."""
    out = []
    for i in range(c["series"]):
        rng = np.random.Generator(np.random.PCG64(c["shape_seed"] + i))
        lo, hi = math.log(c["lo"]), math.log(c["hi"])
        nx, ny = int(round(math.exp(rng.uniform(lo, hi)))), int(round(math.exp(rng.uniform(lo, hi))))
        nt = int(rng.integers(c["nt_lo"], c["nt_hi"] + 1))
        out.append((nx, ny, nt, int(np.clip(round(512 * nx * ny / 2048.0 ** 2), 16, 512))))
    return out


def _batch_fields(c, seed):
    return [_blobs2d(nx, ny, nt, K, seed * 1009 + i, c["amp"], 0.0) for i, (nx, ny, nt, K) in enumerate(_shapes(c))]


def _kind(c):
    return F.VECTOR if c["recipe"] == "vector" else F.SCALAR


def _capacity(c):
    """Room for the hits of a call into caller-owned arrays: the library's fixed scratch region allows 20 bytes a hit
    besides 2 bytes a vertex and 12 a row segment."""
    V = c["nx"] * c["ny"] * c["nt"]
    seg = (c["nx"] + 63) // 64 * c["ny"] * c["nt"]
    return min(4 * V + 64, (F.STATIC_SCRATCH_BYTES - 2 * V - 13 * seg - 65536) // 20)


# ---------------------------------------------------------------------------------------------------------------
# The calls
# ---------------------------------------------------------------------------------------------------------------
def prepare(case, seed):
    c, p = case, case["path"]
    s = dict(case=c)
    if p == "batch2d":
        s["fields"] = _batch_fields(c, seed)
        return s
    if p == "mesh2d":
        xy, tri, s["field"] = _mesh(c, seed)
        s["mesh"] = F.Mesh(xy, tri)
        return s
    s["field"] = _field(c, seed)
    if p == "into2d":
        n = _capacity(c)
        d = _dev()
        s["out"] = dict(face_id=torch.empty(n, dtype=torch.int64, device=d), pos=torch.empty((n, 3), device=d),
                        type=torch.empty(n, dtype=torch.uint8, device=d),
                        flags=torch.empty(n, dtype=torch.uint8, device=d),
                        label=torch.empty(n, dtype=torch.int64, device=d))
        if c["outputs"] == OUT_ALL:
            s["out"]["mu"] = torch.empty((n, 3), device=d)
    if p == "post2d":
        s["dims"] = (c["nx"], c["ny"], c["nt"])
        s["res"] = F.track_cp2d(s["field"], kind=_kind(c))
        del s["field"]
    return s


# Entries that a result of the recipes may have per vertex, with a wide margin (iso: crossed edges, tetrahedra).
_ROOM = {"noise": 3.0, "levels": 3.0, "blobs": 0.05, "vector": 0.05, "blobs3d": 0.01, "waves": 2.0, "mesh": 0.05}


def _room(c, key, V):
    """Rows of an output array once padded (see Outputs)."""
    if c["path"] == "iso3d":
        return int((2.0 if key == "tets" else 0.35) * V if V > 3e7 else (8.0 if key == "tets" else 1.5) * V) + 4096
    return int(_ROOM[c["recipe"]] * V) + 4096 + (1000 * c["nt"] if c["path"] == "mesh2d" else 0)


def _pad(t, rows):
    if t.shape[0] > rows:
        raise ValueError("a result of %d entries is larger than its room of %d" % (t.shape[0], rows))
    out = torch.zeros((rows,) + tuple(t.shape[1:]), dtype=t.dtype, device=t.device)
    out[: t.shape[0]] = t
    return out


class Outputs(dict):
    """What a call returned, as it returned it.  The arrays have one entry per hit, and inputs of another seed have
    other numbers of hits: whoever reads an array here to compare it gets it filled up with zeros to a number of
    rows that the case alone fixes.  A pass itself only hands over the library's own arrays."""

    def __init__(self, items, c, V):
        super().__init__(items)
        self.c, self.V = c, V

    def __getitem__(self, k):
        v = super().__getitem__(k)
        return _pad(v, _room(self.c, k, self.V)) if torch.is_tensor(v) else v


def _outputs(r, c, V=None):
    return Outputs({k: v for k, v in r.items() if k not in ("stats", "n") and v is not None}, c,
                   _vertices(c) if V is None else V)


def _vertices(c):
    if c["path"] == "mesh2d":
        return c["points"] * c["nt"]
    return c["nx"] * c["ny"] * (c.get("nz") or 1) * c["nt"]


def run(state):
    c, p = state["case"], state["case"]["path"]
    if p == "track2d":
        return _outputs(F.track_cp2d(state["field"], kind=_kind(c), precision=c["precision"], outputs=c["outputs"]), c)
    if p == "into2d":
        return _outputs(F.track_cp2d_into(state["field"], kind=_kind(c), out=state["out"], precision=c["precision"],
                                          outputs=c["outputs"]), c)
    if p == "batch2d":
        res = F.track_cp2d_batched(state["fields"])
        return [_outputs({k: r[k] for k in ("face_id", "pos", "type", "flags", "label")}, c, f.numel())
                for r, f in zip(res, state["fields"])]
    if p == "stream":
        f = state["field"]
        dims = (c["nx"], c["ny"], c["nz"]) if c["nz"] else (c["nx"], c["ny"])
        tr = F.Tracker(len(dims), dims, kind=_kind(c))
        for t in range(f.shape[0]):
            tr.push(f[t])
        r = tr.finish()
        tr.close()
        return _outputs(r, c)
    if p == "track3d":
        return _outputs(F.track_cp3d(state["field"]), c)
    if p == "iso3d":
        return _outputs(F.track_iso3d(state["field"], c["isovalue"]), c)
    if p == "vortex3d":
        return _outputs(F.track_vortex3d(state["field"]), c)
    if p == "mesh2d":
        r = state["mesh"].track(state["field"])
        # the numbers of edges and faces a step are the mesh's own
        return _outputs({k: r[k] for k in ("n_hits", "n_trajectories", "face_id", "pos", "label")}, c)
    res, dims = state["res"], state["dims"]
    tab = F.trajectory_table(res, dims)
    order, off = F.trajectory_order(res, dims, tab)
    got = dict(slice=F.slice_at(res, dims, dims[-1] // 2), keep=F.filter_loops(res, tab, 1.0), order=order, offsets=off,
               smooth=F.smooth_types(res, tab, order, off, 2), simple=F.simplify_types(res, tab, order, off, 1.0))
    return _outputs(dict(tab, **got), c)


# Hits per vertex of the recipes (iso: crossed edges), as the workloads give them; used for the bytes written only.
_DENSITY = {"noise": 1.75, "levels": 0.3, "blobs": 0.004, "vector": 0.0008, "blobs3d": 0.0004, "waves": 0.7}


def work(case):
    c, p = case, case["path"]
    if p == "batch2d":
        V = sum(nx * ny * nt for nx, ny, nt, _ in _shapes(c))
    else:
        V = _vertices(c)
    if p == "mesh2d":  # field and mesh in; about 11 faces a vertex and step, three products each
        return dict(bytes=8.0 * V + 32.0 * c["points"], flops=11.0 * 9 * V)
    hits = _DENSITY[c["recipe"]] * V
    if p == "iso3d":  # field in; id, point and label of a crossing; four indices of a tetrahedron
        return dict(bytes=4.0 * V + 0.19 * V * 32 + 1.1 * V * 16, flops=15.0 * V)
    if p == "vortex3d":  # 15 edge determinants a vertex; id, point and label of a triangle
        return dict(bytes=8.0 * V + 32.0 * hits, flops=45.0 * V + 20.0 * hits)
    if p == "post2d":  # ids, positions, labels and types in; order, keep and two type arrays out
        return dict(bytes=hits * (8 + 12 + 8 + 1 + 8 + 1 + 1 + 1), flops=hits)
    comps = 2 if c["recipe"] == "vector" else 1
    rec = 30 if c.get("outputs", 0) != OUT_ALL else 42
    if c.get("nz"):  # 50 triangle determinants a vertex
        return dict(bytes=4.0 * V + 34.0 * hits, flops=50.0 * 14 * V)
    return dict(bytes=4.0 * comps * V + rec * hits, flops=29.0 * V + 60.0 * hits)


# ---------------------------------------------------------------------------------------------------------------
# The floating outputs in 64 bits, in plain torch
# ---------------------------------------------------------------------------------------------------------------
def _types(axes, k):
    """Ordered k-tuples of nonempty disjoint axis masks in lexicographic order: the simplex types."""
    return [m for m in itertools.product(range(1, 1 << axes), repeat=k)
            if all(not (a & b) for a, b in itertools.combinations(m, 2))]


def _perturbed_terms(n):
    """Terms of the determinant of an n x n matrix whose entry (row j, column k) carries eps^(2^(k n + j)), by
    increasing exponent: each a list of (sign, the (row, column) entries multiplied)."""
    by = {}
    for perm in itertools.permutations(range(n)):  # column k takes row perm[k]
        sign = 1
        for i in range(n):
            for j in range(i):
                if perm[j] > perm[i]:
                    sign = -sign
        for pick in itertools.product((0, 1), repeat=n):  # columns whose perturbation is taken
            e = sum(1 << (k * n + perm[k]) for k in range(n) if pick[k])
            by.setdefault(e, []).append((sign, [(perm[k], k) for k in range(n) if not pick[k]]))
    return [by[e] for e in sorted(by)]


_TERMS = {2: _perturbed_terms(2), 3: _perturbed_terms(3)}


def _term(cols, term):
    total = 0
    for sign, entries in term:
        v = sign
        for j, k in entries:
            v = v * cols[k][:, j]
        total = total + v
    return total


def _inside(q):
    """Simplices q (list of n + 1 int64 tensors [m][n], vertices in global order): whether the perturbed simplex holds
    the origin, and its barycentric coordinates."""
    n = len(q) - 1
    C, S = [], []
    for i in range(n + 1):
        cols = [q[k] for k in range(n + 1) if k != i]
        d = _term(cols, _TERMS[n][0])
        sg = torch.sign(d)
        for term in _TERMS[n][1:]:
            left = sg == 0
            if not bool(left.any()):
                break
            w = [x[left] for x in cols]
            v = _term(w, term)
            sg[left] = torch.sign(v) if torch.is_tensor(v) else torch.full_like(sg[left], 1 if v > 0 else -1)
        flip = -1 if i & 1 else 1
        C.append(flip * d)
        S.append(flip * sg)
    hit = torch.ones_like(S[0], dtype=torch.bool)
    for s in S[1:]:
        hit &= s == S[0]
    C = torch.stack([x[hit] for x in C], dim=1).double()
    D = C.sum(dim=1, keepdim=True)
    return hit, torch.where(D == 0, torch.full_like(C, 1.0 / (n + 1)), C / torch.where(D == 0, torch.ones_like(D), D))


def _grid_points(q_of, dims, k):
    """Points (x, y, [z], t) and coordinates of the punctured k-simplices of the grid dims = (nx, ny, [nz,] nt), in
    id order.  q_of(t): integer vectors of step t, [..., y, x, k]."""
    axes = len(dims)
    types = _types(axes, k)
    space = list(dims[:-1])
    stride = [1]
    for n in space[:-1]:
        stride.append(stride[-1] * n)
    all_pos, all_mu = [], []
    nxt = q_of(0)
    for t in range(dims[-1]):
        cur, nxt = nxt, (q_of(t + 1) if t + 1 < dims[-1] else None)
        ids, pos, mus = [], [], []
        for ty, masks in enumerate(types):
            used = sum(masks)
            if (used >> (axes - 1)) & 1 and nxt is None:
                continue
            corner, vs = 0, [0]
            for m in masks:
                corner |= m
                vs.append(corner)
            views = []
            for v in vs:
                sl = tuple(slice((v >> a) & 1, space[a] - ((used >> a) & 1) + ((v >> a) & 1))
                           for a in reversed(range(axes - 1)))
                views.append((nxt if (v >> (axes - 1)) & 1 else cur)[sl])
            # a component of one strict sign at every vertex, or all vectors zero: never punctured
            may = None
            zero = None
            for j in range(k):
                lo, hi = views[0][..., j], views[0][..., j]
                for w in views[1:]:
                    lo, hi = torch.minimum(lo, w[..., j]), torch.maximum(hi, w[..., j])
                m1, z1 = (lo <= 0) & (hi >= 0), (lo == 0) & (hi == 0)
                may, zero = (m1, z1) if may is None else (may & m1, zero & z1)
            at = (may & ~zero).nonzero()
            if not at.numel():
                continue
            idx = tuple(at[:, a] for a in range(axes - 1))
            hit, mu = _inside([w[idx].long() for w in views])
            at = at[hit].flip(1)  # x, y, [z]
            g = sum(at[:, a] * stride[a] for a in range(axes - 1))
            p = []
            for a in range(axes):
                base = at[:, a].double() if a < axes - 1 else torch.full((at.shape[0],), float(t), dtype=torch.float64,
                                                                         device=at.device)
                p.append(sum(mu[:, i] * (base + ((v >> a) & 1)) for i, v in enumerate(vs)))
            ids.append(g * len(types) + ty)
            pos.append(torch.stack(p, dim=1))
            mus.append(mu)
        if ids:
            o = torch.argsort(torch.cat(ids))
            all_pos.append(torch.cat(pos)[o])
            all_mu.append(torch.cat(mus)[o])
    if not all_pos:
        z = torch.zeros((0, axes), dtype=torch.float64, device=_dev())
        return z, torch.zeros((0, k + 1), dtype=torch.float64, device=_dev())
    return torch.cat(all_pos), torch.cat(all_mu)


def _gradient(f):
    """Binary32 differences along the last axes (x, y, [z]): central inside, one-sided at the ends."""
    out = []
    for d in range(f.dim() - 1, -1, -1):
        n = f.shape[d]
        g = torch.empty_like(f)
        g.narrow(d, 1, n - 2).copy_((f.narrow(d, 2, n - 2) - f.narrow(d, 0, n - 2)) * 0.5)
        g.narrow(d, 0, 1).copy_(f.narrow(d, 1, 1) - f.narrow(d, 0, 1))
        g.narrow(d, n - 1, 1).copy_(f.narrow(d, n - 1, 1) - f.narrow(d, n - 2, 1))
        out.append(g)
    return out


def _quantised(comps):
    return torch.stack([torch.round(c * 1048576.0) for c in comps], dim=-1).to(torch.int32)


def _track_exact(field, vector):
    if vector:
        q_of, dims = (lambda t: _quantised([field[t, 0], field[t, 1]])), (field.shape[3], field.shape[2], field.shape[0])
    else:
        q_of, dims = (lambda t: _quantised(_gradient(field[t]))), tuple(reversed(field.shape[1:])) + (field.shape[0],)
    return _grid_points(q_of, dims, len(dims) - 1)


def _iso_exact(f, c):
    nt, nz, ny, nx = f.shape
    out = []
    for t in range(nt):
        ids, pos = [], []
        for M in range(1, 16):
            d = [(M >> a) & 1 for a in range(4)]
            if d[3] and t + 1 >= nt:
                continue
            p = f[t][: nz - d[2], : ny - d[1], : nx - d[0]]
            q = f[t + d[3]][d[2]:, d[1]:, d[0]:]
            at = ((p >= c) != (q >= c)).nonzero()
            z, y, x = at[:, 0], at[:, 1], at[:, 2]
            f0, f1 = p[z, y, x].double(), q[z, y, x].double()
            mu = (c - f0) / (f1 - f0)
            ids.append(((z * ny + y) * nx + x) * 15 + (M - 1))
            pos.append(torch.stack([x + mu * d[0], y + mu * d[1], z + mu * d[2], t + mu * d[3]], dim=1))
        out.append(torch.cat(pos)[torch.argsort(torch.cat(ids))])
    return torch.cat(out)


def _mesh_exact(xy, tri, field):
    tri = torch.sort(tri.long(), dim=1).values
    nv = xy.shape[0]
    e = torch.cat([tri[:, [0, 1]], tri[:, [1, 2]], tri[:, [0, 2]]])
    e = torch.unique(e[:, 0] * nv + e[:, 1])
    a, b = e // nv, e % nv
    both = lambda p, q: torch.stack([p, q], dim=1).reshape(-1)  # noqa: E731
    # faces of a step: mesh triangles, edge faces (a, b, b') and (a, a', b'), interior faces (v0, v1, v2'), (v0, v1', v2')
    v = [torch.cat([tri[:, 0], both(a, a), both(tri[:, 0], tri[:, 0])]),
         torch.cat([tri[:, 1], both(b, a), both(tri[:, 1], tri[:, 1])]),
         torch.cat([tri[:, 2], both(b, b), both(tri[:, 2], tri[:, 2])])]
    z, o = torch.zeros_like(tri[:, 0]), torch.ones_like(tri[:, 0])
    ze, oe = torch.zeros_like(a), torch.ones_like(a)
    dt = [torch.cat([z, both(ze, ze), both(z, z)]), torch.cat([z, both(ze, oe), both(z, o)]),
          torch.cat([z, both(oe, oe), both(o, o)])]
    out = []
    for t in range(field.shape[0]):
        n = v[0].shape[0] if t + 1 < field.shape[0] else tri.shape[0]
        two = field[t:t + 2]
        q2 = torch.round(two * 1048576.0).long().permute(0, 2, 1)
        hit, mu = _inside([q2[dt[i][:n], v[i][:n]] for i in range(3)])
        at = hit.nonzero()[:, 0]
        p = sum(mu[:, i:i + 1] * torch.cat([xy[v[i][at]].double(), (dt[i][at] + t).double()[:, None]], dim=1)
                for i in range(3))
        out.append(p)
    return torch.cat(out)


def _filled(items, c, V=None):
    o = _outputs(items, c, V)
    return {k: o[k] for k in o}


def exact(case, seed):
    c, p = case, case["path"]
    if p == "post2d":
        return None  # whole numbers, and extrema of given values
    if p == "batch2d":
        return [_filled(dict(pos=_track_exact(f, False)[0]), c, f.numel()) for f in _batch_fields(c, seed)]
    if p == "mesh2d":
        return _filled(dict(pos=_mesh_exact(*_mesh(c, seed))), c)
    f = _field(c, seed)
    if p == "iso3d":
        return _filled(dict(pos=_iso_exact(f, c["isovalue"])), c)
    if p == "vortex3d":
        q_of = lambda t: _quantised([f[t, 0], f[t, 1]])  # noqa: E731
        return _filled(dict(pos=_grid_points(q_of, (f.shape[4], f.shape[3], f.shape[2], f.shape[0]), 2)[0]), c)
    pos, mu = _track_exact(f, c["recipe"] == "vector")
    return _filled(dict(pos=pos, mu=mu) if c.get("outputs", 0) == OUT_ALL else dict(pos=pos), c)
