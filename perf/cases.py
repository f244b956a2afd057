"""The work that programs have this library do, as a list of cases to measure.

A case is one pass of a user's program through the public entry points of
``paper_2209_11606_amd.vorohip``: positions that are already in device memory
(or on their way out to the host, where the call returns host arrays) are
binned and every Voronoi cell is computed with its statistics.  ``prepare``
holds what such a program keeps between passes (the container or batch, the
result and its device arrays); ``run`` is the pass.

Four kinds of call:

* ``step``: one container kept over the steps of a simulation or an analysis,
  ``vc_container_rebin`` with the step's positions, ``vc_compute``, and the
  result's fields as device arrays.  The neighbour lists, whose length the
  library gives, are taken over into the program's own arrays.
* ``batch``: several independent tessellations (or one) as a ``vc_batch``,
  ``vc_batch_rebin`` and a ``vc_batch_compute`` replayed from its graph.
* ``noalloc``: ``vc_tessellate_noalloc`` into the caller's own arrays.
* ``tessellate``: the one-shot call, device positions to host arrays (the
  per-cell statistics).

The outputs are the cells: volumes, centroids, counts, face orders, neighbour
lists, and where asked the perimeters or the Weinberg codes.  Two fields are
not among them, because they tell how a cell was computed and not what it is:
the run counters, and the status, whose value "spilled" names the pass that
finished a cell (a cell that failed has a NaN volume and no faces).
"""
import math

import numpy as np
import torch

from paper_2209_11606_amd import vorohip as v
from paper_2209_11606_amd import workloads

FIELDS = v.VC_VOLUME | v.VC_CENTROID | v.VC_COUNTS | v.VC_FACE_ORDERS | v.VC_NEIGHBORS


def listed():
    return [
        # one small walled set with every option at its default: the latency
        # of a step, most of it launches (the library's smallest set of 1,000)
        dict(name="walled_1k", call="step", set="uniform", dim=3, n=1000, periodic=False),
        # a serving loop that must not allocate
        dict(name="noalloc_5k", call="noalloc", set="uniform", dim=3, n=5003, periodic=True),
        # the one-shot call of the README, host arrays back
        dict(name="tessellate_100k", call="tessellate", set="uniform", dim=3, n=100_000, periodic=True,
             cells_per_wave=2),
        # the benchmark's periodic set of 10^6 at density 1, as a container
        # with default options
        dict(name="periodic_1m", call="step", set="uniform", dim=3, n=1_000_000, periodic=True),
        # the same set in the benchmark's batched form (two cells per wave,
        # graph replay)
        dict(name="periodic_1m_batched", call="batch", set="uniform", dim=3, n=1_000_000, periodic=True,
             cells_per_wave=2),
        # the FP32-filtered side tests on an odd count
        dict(name="f32_filter_300k", call="step", set="uniform", dim=3, n=300_007, periodic=True,
             cells_per_wave=2, precision=v.VC_F32_FILTER),
        # a crystal: the perturbed FCC lattice of the benchmark, 50^3 unit
        # cells, where vertices of degree above three nearly coincide
        dict(name="fcc_500k", call="batch", set="fcc", dim=3, n=500_000, periodic=True, cells_per_wave=2),
        # many small problems in one launch: periodic and walled, uniform and
        # perturbed BCC, 100 to 10,000 particles each
        dict(name="batch_256", call="batch", set="mixed", dim=3, n=256, cells_per_wave=2),
        # the planar form with the perimeter
        dict(name="periodic_2d_1m", call="step", set="uniform", dim=2, n=1_000_000, periodic=True),
        # a polydisperse packing: radical cells
        dict(name="polydisperse_200k", call="step", set="polydisperse", dim=3, n=200_000, periodic=True,
             cells_per_wave=2),
        # structure analysis: every cell with its Weinberg code
        dict(name="vorotop_200k", call="step", set="uniform", dim=3, n=200_000, periodic=True, cells_per_wave=2,
             weinberg=True),
        # an imbalanced set: a dense cube in a mostly empty walled box, whose
        # surface cells reach far (about 10^5 cells)
        dict(name="localized_100k", call="step", set="localized", dim=3, n=1_000_000, periodic=False),
    ]


def _size(rng, lo, hi):
    """A size spread over the logarithm of [lo, hi], odd more often than not."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, n | 1 if rng.random() < 0.7 else n))


def draw(rng):
    kind = rng.choice(["step", "step", "wave2", "wave2", "batch", "mixed", "noalloc", "tessellate", "fcc", "planar",
                       "planar", "polydisperse", "vorotop", "localized"])
    periodic = rng.random() < 0.7
    if kind == "step":
        return dict(call="step", set="uniform", dim=3, n=_size(rng, 500, 500_000), periodic=periodic,
                    precision=rng.choice([v.VC_FP64, v.VC_FP64, v.VC_F32_FILTER]))
    if kind == "wave2":
        return dict(call="step", set="uniform", dim=3, n=_size(rng, 2000, 1_000_000), periodic=periodic,
                    cells_per_wave=2, precision=rng.choice([v.VC_FP64, v.VC_F32_FILTER]))
    if kind == "batch":
        return dict(call="batch", set="uniform", dim=3, n=_size(rng, 10_000, 1_000_000), periodic=periodic,
                    cells_per_wave=2)
    if kind == "mixed":
        return dict(call="batch", set="mixed", dim=3, n=_size(rng, 8, 400), cells_per_wave=2)
    if kind == "noalloc":
        return dict(call="noalloc", set="uniform", dim=rng.choice([2, 3, 3]), n=_size(rng, 500, 65_536),
                    periodic=periodic, cells_per_wave=rng.choice([0, 0, 2]))
    if kind == "tessellate":
        return dict(call="tessellate", set="uniform", dim=3, n=_size(rng, 1000, 200_000), periodic=periodic,
                    cells_per_wave=rng.choice([0, 2]))
    if kind == "fcc":
        m = _size(rng, 8, 56)
        return dict(call=rng.choice(["step", "batch"]), set="fcc", dim=3, n=4 * m ** 3, periodic=True,
                    cells_per_wave=2)
    if kind == "planar":
        return dict(call="step", set=rng.choice(["uniform", "uniform", "polydisperse"]), dim=2,
                    n=_size(rng, 1000, 1_500_000), periodic=periodic)
    if kind == "polydisperse":
        return dict(call="step", set="polydisperse", dim=3, n=_size(rng, 2000, 400_000), periodic=periodic,
                    cells_per_wave=rng.choice([0, 2]))
    if kind == "vorotop":
        return dict(call="step", set="uniform", dim=3, n=_size(rng, 1000, 300_000), periodic=True,
                    cells_per_wave=rng.choice([0, 2]), weinberg=True)
    return dict(call="step", set="localized", dim=3, n=_size(rng, 50_000, 1_500_000), periodic=False,
                cells_per_wave=rng.choice([0, 2]))


# ---------------------------------------------------------------------------
# Inputs: each made on the GPU from the seed alone, density 1 where periodic.
# ---------------------------------------------------------------------------

def _rand(seed, *shape):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    return torch.rand(*shape, dtype=torch.float64, device="cuda", generator=g)


def _randn(seed, *shape):
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 77)
    return torch.randn(*shape, dtype=torch.float64, device="cuda", generator=g)


def _wrap(x, hi):
    x = torch.remainder(x, hi)
    return torch.where(x >= hi, torch.zeros_like(x), x).contiguous()


def _inside(x, hi):
    """A product can round up to the box side itself: keep the box half open."""
    return torch.clamp(x, max=float(np.nextafter(hi, 0.0)))


def _members(case, seed):
    """The sets of a case: dicts of positions, box side(s), periodicity, grid, radii."""
    n, dim = case["n"], case["dim"]
    kind = case["set"]
    if kind == "mixed":
        out = []
        sizes = workloads.batch_sizes(n, 100, 10_000)
        for t, nt in enumerate(sizes.tolist()):
            periodic = t % 2 == 0
            s = int(seed) * 1009 + t
            if (t // 2) % 2:
                m = max(2, round((nt / 2) ** (1 / 3)))
                a = 2.0 ** (1 / 3)
                basis = torch.tensor([[.25, .25, .25], [.75, .75, .75]], dtype=torch.float64, device="cuda")
                g = torch.cartesian_prod(*[torch.arange(m, dtype=torch.float64, device="cuda")] * 3)
                x = ((g[:, None, :] + basis[None]) * a).reshape(-1, 3)
                hi = m * a
                x = x + 0.05 * a * _randn(s, *x.shape)
                x = _wrap(x, hi) if periodic else torch.clamp(x, 0.0, float(np.nextafter(hi, 0.0)))
            else:
                hi = float(nt) ** (1 / 3)
                x = _inside(_rand(s, nt, 3) * hi, hi)
            out.append(dict(xyz=x.contiguous(), hi=[hi] * 3, periodic=[int(periodic)] * 3))
        return out
    per = [int(bool(case["periodic"]))] * dim
    if kind == "fcc":
        m = round((n / 4) ** (1 / 3))
        basis = torch.tensor([[0, 0, 0], [0, .5, .5], [.5, 0, .5], [.5, .5, 0]], dtype=torch.float64, device="cuda")
        g = torch.cartesian_prod(*[torch.arange(m, dtype=torch.float64, device="cuda")] * 3)
        x = (g[:, None, :] + basis[None] + 0.25).reshape(-1, 3)
        return [dict(xyz=_wrap(x + 1e-3 * _randn(seed, *x.shape), float(m)), hi=[float(m)] * 3, periodic=per)]
    if kind == "localized":
        # the points of a uniform set of n that fall into the central cube of
        # volume 0.1, and the grid of the whole set
        x = 0.5 + (_rand(seed, n // 10, 3) - 0.5) * 0.1 ** (1 / 3)
        g = int((n / 49.0) ** (1 / 3))
        return [dict(xyz=x, hi=[1.0] * 3, periodic=per, grid=[g] * 3)]
    side = float(n) ** (1.0 / dim) if case["periodic"] else 1.0
    x = _inside(_rand(seed, n, dim) * side, side)
    w = dict(xyz=x, hi=[side] * dim, periodic=per)
    if kind == "polydisperse":
        w["radii"] = _rand(int(seed) + 1, n) * (0.6 * side * n ** (-1.0 / dim))
    return [w]


# ---------------------------------------------------------------------------
# The state of a user's program and one pass.
# ---------------------------------------------------------------------------

class _Owner:
    """A container or batch with its result: freed when neither the state nor
    one of the arrays that point into it is left."""

    def __init__(self, destroy):
        self.destroy, self.handle, self.result = destroy, None, None

    def __del__(self):
        if self.handle is None:
            return
        torch.cuda.synchronize()
        if self.result is not None:
            v.vc_result_destroy(self.result)
        self.destroy(self.handle)


class _View:
    """A device array of the library as a tensor (no copy); the tensor keeps
    this object, and so the array's owner."""

    def __init__(self, owner, ptr, count, dtype):
        self.owner = owner
        self.__cuda_array_interface__ = dict(shape=(count,), typestr=dtype, data=(ptr, False), version=2, strides=None)


def _view(owner, field):
    ptr, count = v.vc_result_get(owner.result, field)
    return torch.as_tensor(_View(owner, ptr, count, np.dtype(v._FIELD_DTYPE[field]).str), device="cuda")


class _State:
    def __init__(self, case, members):
        self.call = case["call"]
        self.dim = case["dim"]
        self.mask = FIELDS
        if self.dim == 2:
            self.mask = (FIELDS & ~v.VC_FACE_ORDERS) | v.VC_PERIMETER
        if case.get("weinberg"):
            self.mask |= v.VC_WEINBERG
        if self.call == "tessellate":
            self.mask &= ~v.VC_NEIGHBORS
        form = {k: case[k] for k in ("cells_per_wave", "precision") if case.get(k)}
        self.opts = [v.vc_options_init(self.dim, [0.0] * self.dim, m["hi"], m["periodic"],
                                       **(dict(form, grid=m["grid"]) if "grid" in m else form)) for m in members]
        self.form, self.member = form, members[0]
        self.xyz = members[0]["xyz"] if len(members) == 1 else torch.cat([m["xyz"] for m in members])
        n = self.xyz.shape[0]
        torch.cuda.synchronize()
        if self.call == "noalloc":
            z = dict(device="cuda")
            self.out = dict(vol=torch.empty(n, dtype=torch.float64, **z), cen=torch.empty(3 * n, dtype=torch.float64, **z),
                            nv=torch.empty(n, dtype=torch.int32, **z), ne=torch.empty(n, dtype=torch.int32, **z),
                            nf=torch.empty(n, dtype=torch.int32, **z), fo=torch.empty(32 * n, dtype=torch.uint8, **z))
            if self.dim == 2:
                del self.out["fo"]
            self.args = dict(self.out, status=torch.empty(n, dtype=torch.uint8, **z))
            return
        if self.call == "tessellate":
            return
        self.stream = torch.cuda.Stream() if self.call == "batch" else torch.cuda.current_stream()
        own = self.own = _Owner(v.vc_batch_destroy if self.call == "batch" else v.vc_container_destroy)
        if self.call == "batch":
            off = np.cumsum([0] + [m["xyz"].shape[0] for m in members])
            own.handle = v.vc_batch_create(self.xyz, off, self.opts, self.stream)
            own.result = v.vc_batch_result_create(own.handle, self.mask)
        else:
            own.handle = v.vc_container_create(self.xyz, self.opts[0], self.stream)
            if "radii" in self.member:
                v.vc_container_set_radii(own.handle, self.member["radii"], self.stream)
            own.result = v.vc_result_create(own.handle, self.mask)
        fields = dict(vol=v.VC_F_VOLUME, cen=v.VC_F_CENTROID, nv=v.VC_F_NV, ne=v.VC_F_NE, nf=v.VC_F_NF,
                      nbr_off=v.VC_F_NBR_OFFSETS)
        if self.dim == 2:
            fields["perim"] = v.VC_F_PERIMETER
        else:
            fields["fo"] = v.VC_F_FACE_ORDERS
        if case.get("weinberg"):
            fields.update(wb_off=v.VC_F_WB_OFFSETS, wb_sym=v.VC_F_WB_SYM, wb_chiral=v.VC_F_WB_CHIRAL)
        self.fixed = {k: _view(own, f) for k, f in fields.items()}
        # the program's arrays for the lists, with room for more than any
        # mean number of faces (6 in the plane, under 17 in space)
        self.listed = dict(nbr_ids=v.VC_F_NBR_IDS, nbr_sh=v.VC_F_NBR_SHIFTS)
        self.kept = dict(nbr_ids=torch.zeros(20 * n, dtype=torch.int32, device="cuda"),
                         nbr_sh=torch.zeros(20 * n, dtype=torch.uint8, device="cuda"))
        if case.get("weinberg"):
            self.listed["wb_codes"] = v.VC_F_WB_CODES
            self.kept["wb_codes"] = torch.zeros(100 * n, dtype=torch.uint8, device="cuda")
        self.fixed.update(self.kept)


def prepare(case, seed):
    return _State(case, _members(case, seed))


def run(state):
    s = state
    if s.call == "noalloc":
        v.vc_tessellate_noalloc(s.xyz, s.opts[0], s.args)
        return s.out
    if s.call == "tessellate":
        m = s.member
        got = v.tessellate(s.xyz, [0.0] * s.dim, m["hi"], m["periodic"], s.mask, radii=m.get("radii"), **s.form)
        return {k: x for k, x in got.items() if k not in ("diag", "status")}
    if s.call == "batch":
        v.vc_batch_rebin(s.own.handle, s.xyz, s.stream)
        v.vc_batch_compute(s.own.handle, s.own.result, True, s.stream)
    else:
        v.vc_container_rebin(s.own.handle, s.xyz, s.stream)
        v.vc_compute(s.own.handle, s.own.result, s.stream)
    for k, f in s.listed.items():
        got = _view(s.own, f)  # at the length that the library gives
        s.kept[k][:got.shape[0]].copy_(got)
    return s.fixed


def work(case):
    """Bytes: positions (and radii) once, the outputs once, neighbour labels
    of 5 bytes for the mean face count of the set.  Flops: candidates in
    reach, side tests, new vertices and fan pieces that an FP64 cell takes
    with neighbours in order of distance (a count per cell: in 3D about 43
    candidates, 900 vertex tests, 75 new vertices, 50 fan tetrahedra)."""
    n, dim = case["n"], case["dim"]
    if case["set"] == "mixed":
        n = int(n * 9900 / math.log(100))  # mean of the log-uniform sizes
    elif case["set"] == "localized":
        n = n // 10
    faces = 6.0 if dim == 2 else (14.0 if case["set"] == "fcc" else 15.5)
    per = 8 * dim + 8 + 24 + 4 + (8 if case["set"] == "polydisperse" else 0)
    if case["call"] == "noalloc":
        per += 8 + (32 if dim == 3 else 0)
    else:
        per += 8 + 8 + 5 * faces + (8 if dim == 2 else 32)
    if case.get("weinberg"):
        per += 8 + 5 + 6 * (faces - 2)
    return dict(bytes=n * per, flops=n * (700.0 if dim == 2 else 8150.0))


# ---------------------------------------------------------------------------
# The cells in plain FP64 torch: each face is a polygon in its bisector plane,
# clipped by every other bisector of its cell (no shared code or structure
# with the library).  Volumes and centroids only.
# ---------------------------------------------------------------------------

def _clip(P, cnt, n, h):
    """Convex polygons P[m, V, d] of cnt[m] vertices cut to n.x <= h."""
    m, V, d = P.shape
    ar = torch.arange(V, device=P.device)
    on = ar[None] < cnt[:, None]
    s = (P * n[:, None, :]).sum(-1) - h[:, None]
    nxt = torch.where(ar[None] + 1 < cnt[:, None], ar[None] + 1, torch.zeros_like(ar)[None])
    sn = torch.gather(s, 1, nxt)
    inside = (s <= 0) & on
    cross = on & ((s <= 0) != (sn <= 0))
    k = inside.long() + cross.long()
    at = torch.cumsum(k, 1) - k
    Q = torch.zeros(m, V + 2, d, dtype=P.dtype, device=P.device)
    Pn = torch.gather(P, 1, nxt[..., None].expand(-1, -1, d))
    t = torch.where(cross, s / torch.where(cross, s - sn, torch.ones_like(s)), torch.zeros_like(s))
    X = P + t[..., None] * (Pn - P)
    last = torch.full_like(at, V + 1)
    Q.scatter_(1, torch.where(inside, at, last)[..., None].expand(-1, -1, d), P)
    Q[:, V + 1] = 0
    Q.scatter_(1, torch.where(cross, at + inside.long(), last)[..., None].expand(-1, -1, d), X)
    return Q[:, :V], torch.clamp(k.sum(1), max=V)


def _near(x, lo_hi, periodic, rows, K):
    """For the particles `rows`: relative positions, input index and distance
    of the K nearest others (periodic images included)."""
    hi, n = lo_hi, x.shape[0]
    pts, ids = [x], [torch.arange(n, device=x.device)]
    reach = math.inf
    if any(periodic):
        d = x.shape[1]
        reach = min(hi[0], 4.0 * hi[0] * (max(K, 64) / max(n, 1)) ** (1.0 / d)) if n > 2 * K else hi[0]
        L = torch.tensor(hi, dtype=x.dtype, device=x.device)
        for s in torch.cartesian_prod(*[torch.tensor([-1.0, 0.0, 1.0], dtype=x.dtype, device=x.device)] * d):
            if not s.any():
                continue
            y = x + s * L
            keep = ((y >= -reach) & (y <= L + reach)).all(1)
            pts.append(y[keep])
            ids.append(ids[0][keep])
    pts, ids = torch.cat(pts), torch.cat(ids)
    K = min(K, pts.shape[0] - 1)
    q, nb, dist = [], [], []
    step = max(1, int(1.5e8 // pts.shape[0]))
    for a in range(0, len(rows), step):
        r = rows[a:a + step]
        d2 = torch.zeros(len(r), pts.shape[0], dtype=x.dtype, device=x.device)
        for k in range(x.shape[1]):
            d2 += (pts[None, :, k] - x[r, k, None]) ** 2
        d2[torch.arange(len(r), device=x.device), r] = math.inf
        dd, j = torch.topk(d2, K, largest=False, sorted=True)
        q.append(pts[j] - x[r][:, None, :])
        nb.append(ids[j])
        dist.append(dd.sqrt())
    return torch.cat(q), torch.cat(nb), torch.cat(dist), reach


def _near_grid(x, hi, periodic, rows, K):
    """The same from a grid, for evenly spread sets of many particles: all
    particles of the 5^d cells around a particle's own."""
    n, d = x.shape
    side = (1.75 if d == 3 else 2.2) * (math.prod(hi) / n) ** (1.0 / d)
    g = [max(1, int(h / side)) for h in hi]
    w = torch.tensor([h / k for h, k in zip(hi, g)], dtype=x.dtype, device=x.device)
    gt = torch.tensor(g, device=x.device)
    at = torch.minimum((x / w).long(), gt - 1)
    mul = torch.tensor([1, g[0], g[0] * g[1]][:d], device=x.device)
    order = torch.argsort((at * mul).sum(1))
    count = torch.bincount((at * mul).sum(1), minlength=math.prod(g))
    start = torch.cumsum(count, 0) - count
    most = int(count.max())
    off = torch.cartesian_prod(*[torch.arange(-2, 3, device=x.device)] * d)
    L = torch.tensor(hi, dtype=x.dtype, device=x.device)
    per = torch.tensor(periodic, device=x.device).bool()
    q, nb, dist = [], [], []
    step = max(1, int(6e7 // (len(off) * most)))
    slot = torch.arange(most, device=x.device)
    for a in range(0, len(rows), step):
        r = rows[a:a + step]
        c = at[r][:, None, :] + off[None]
        shift = torch.div(c, gt, rounding_mode="floor")
        ok = (per | (shift == 0)).all(-1)
        b = ((c - shift * gt) * mul).sum(-1)
        b = torch.where(ok, b, torch.zeros_like(b))
        k = torch.where(ok, count[b], torch.zeros_like(b))
        j = order[torch.clamp(start[b][..., None] + slot, max=n - 1)]
        have = slot < k[..., None]
        y = x[j] + (shift * L)[:, :, None, :] - x[r][:, None, None, :]
        d2 = torch.where(have, (y * y).sum(-1), torch.full_like(y[..., 0], math.inf))
        d2 = torch.where(d2 == 0, torch.full_like(d2, math.inf), d2).reshape(len(r), -1)
        dd, t = torch.topk(d2, min(K, d2.shape[1]), largest=False, sorted=True)
        y = torch.gather(y.reshape(len(r), -1, d), 1, t[..., None].expand(-1, -1, d))
        none = dd == math.inf  # fewer than K: a plane far out that cuts nothing
        y = torch.where(none[..., None], L.expand_as(y) * 4, y)
        q.append(y)
        nb.append(torch.where(none, r[:, None].expand_as(t), torch.gather(j.reshape(len(r), -1), 1, t)))
        dist.append(dd.sqrt())
    return torch.cat(q), torch.cat(nb), torch.cat(dist), 2.0 * float(w.min())


def _planes(w, rows, K):
    """Planes n.y <= h of the cells `rows` (bisectors, nearest first, then the
    walls) relative to each particle, and the distance they are complete to."""
    x, hi, per = w["xyz"], w["hi"], w["periodic"]
    d = x.shape[1]
    near = _near_grid if len(rows) > 10_000 and K < 100 else _near
    q, nb, dist, reach = near(x, hi, per, rows, K)
    h = 0.5 * (q * q).sum(-1)
    if "radii" in w:
        r2 = w["radii"] ** 2
        h = h + 0.5 * (r2[rows][:, None] - r2[nb])
    full = q.shape[1] >= x.shape[0] - 1 and not any(per)
    done = torch.full((len(rows),), math.inf, dtype=x.dtype, device=x.device) if full else torch.clamp(dist[:, -1], max=reach)
    ns, hs = [q], [h]
    for k in range(d):
        for side in (0, 1):
            e = torch.zeros(len(rows), 1, d, dtype=x.dtype, device=x.device)
            if per[k]:
                e[..., k] = hi[k] if side else -hi[k]
                hs.append(torch.full((len(rows), 1), 0.5 * hi[k] ** 2, dtype=x.dtype, device=x.device))
            else:
                e[..., k] = 1.0 if side else -1.0
                hs.append((hi[k] - x[rows, k] if side else x[rows, k])[:, None])
            ns.append(e)
    return torch.cat(ns, 1), torch.cat(hs, 1), done


def _moments(N, H, size):
    """Volume, first moment and largest vertex distance of {y: N y <= H}."""
    m, K, d = N.shape
    dev, V = N.device, 28
    vol = torch.zeros(m, dtype=N.dtype, device=dev)
    mom = torch.zeros(m, d, dtype=N.dtype, device=dev)
    far = torch.zeros(m, dtype=N.dtype, device=dev)
    if d == 2:
        P = torch.zeros(m, V, 2, dtype=N.dtype, device=dev)
        P[:, :4] = torch.tensor([[-1, -1], [1, -1], [1, 1], [-1, 1]], dtype=N.dtype, device=dev) * size[:, None, None]
        cnt = torch.full((m,), 4, dtype=torch.long, device=dev)
        for k in range(K):
            P, cnt = _clip(P, cnt, N[:, k], H[:, k])
        on = torch.arange(V, device=dev)[None] < cnt[:, None]
        nxt = torch.where(torch.arange(V, device=dev)[None] + 1 < cnt[:, None], torch.arange(V, device=dev)[None] + 1, 0)
        W = torch.gather(P, 1, nxt[..., None].expand(-1, -1, 2))
        P0 = P[:, :1]
        a, b = P - P0, W - P0
        cr = torch.where(on, a[..., 0] * b[..., 1] - a[..., 1] * b[..., 0], torch.zeros_like(a[..., 0]))
        vol = 0.5 * cr.sum(1)
        mom = (cr[..., None] * (a + b)).sum(1) / 6 + vol[:, None] * P0[:, 0]
        far = torch.where(on, (P * P).sum(-1), torch.zeros_like(cr)).amax(1).sqrt()
        return vol, mom, far, cnt
    face, pl = torch.meshgrid(torch.arange(m, device=dev), torch.arange(K, device=dev), indexing="ij")
    face, pl = face.reshape(-1), pl.reshape(-1)
    nn = N[face, pl]
    n2 = (nn * nn).sum(-1)
    c = nn * (H[face, pl] / n2)[:, None]
    u = nn / n2.sqrt()[:, None]
    e = torch.zeros_like(u)
    e.scatter_(1, u.abs().argmin(1)[:, None], 1.0)
    a = torch.linalg.cross(u, e)
    a = a / a.norm(dim=1, keepdim=True)
    b = torch.linalg.cross(u, a)
    s = (size[face] + c.norm(dim=1))[:, None]
    P = torch.zeros(len(face), V, 3, dtype=N.dtype, device=dev)
    for k, (i, j) in enumerate(((-1, -1), (1, -1), (1, 1), (-1, 1))):
        P[:, k] = c + s * (i * a + j * b)
    cnt = torch.full((len(face),), 4, dtype=torch.long, device=dev)
    for k in range(K):
        n, h = N[face, k], H[face, k]
        own = pl == k
        n = torch.where(own[:, None], torch.zeros_like(n), n)
        h = torch.where(own, torch.ones_like(h), h)
        P, cnt = _clip(P, cnt, n, h)
        if k % 4 == 3 or k == K - 1:
            keep = cnt >= 3
            face, pl, P, cnt, u, c = face[keep], pl[keep], P[keep], cnt[keep], u[keep], c[keep]
    ar = torch.arange(V, device=dev)
    on = ar[None] < cnt[:, None]
    nxt = torch.where(ar[None] + 1 < cnt[:, None], ar[None] + 1, 0)
    W = torch.gather(P, 1, nxt[..., None].expand(-1, -1, 3))
    P0 = P[:, :1]
    tri = torch.where(on, (torch.linalg.cross(P - P0, W - P0) * u[:, None, :]).sum(-1), torch.zeros_like(P[..., 0]))
    dist = (c * u).sum(-1)
    piece = tri * dist[:, None] / 6
    vol.index_add_(0, face, piece.sum(1))
    mom.index_add_(0, face, (piece[..., None] * (P0 + P + W)).sum(1) / 4)
    far.scatter_reduce_(0, face, torch.where(on, (P * P).sum(-1), torch.zeros_like(tri)).amax(1).sqrt(), "amax")
    nf = torch.zeros(m, dtype=torch.long, device=dev)
    nf.index_add_(0, face, torch.ones_like(face))
    return vol, mom, far, nf


def exact(case, seed):
    members = _members(case, seed)
    n = sum(m["xyz"].shape[0] for m in members)
    if case["set"] == "localized" or n > (1_100_000 if case["dim"] == 2 else 350_000) or len(members) > 40:
        return None  # over about 20 seconds in this form
    vols, cens = [], []
    for w in members:
        x = w["xyz"]
        n, d = x.shape
        vol = torch.zeros(n, dtype=x.dtype, device=x.device)
        cen = torch.zeros(n, 3, dtype=x.dtype, device=x.device)
        left = torch.arange(n, device=x.device)
        rm2 = float(w["radii"].max()) ** 2 if "radii" in w else 0.0
        K = 24 if d == 2 else 56
        while len(left):
            again = []
            step = 200_000 if d == 2 else max(16, 1_500_000 // K)
            for a in range(0, len(left), step):
                rows = left[a:a + step]
                N, H, done = _planes(w, rows, K)
                size = torch.full((len(rows),), 2.0 * math.sqrt(d) * max(w["hi"]), dtype=x.dtype, device=x.device)
                vv, mm, far, cnt = _moments(N, H, size)
                ri2 = w["radii"][rows] ** 2 if "radii" in w else 0.0
                ok = far + torch.sqrt(torch.clamp(far * far + (rm2 - ri2), min=0.0)) < done
                empty = cnt < (3 if d == 2 else 4)
                ok = ok | empty
                vol[rows[ok]] = torch.where(empty, torch.zeros_like(vv), vv)[ok]
                cc = torch.where(empty[:, None], torch.zeros_like(mm), mm / torch.where(empty, torch.ones_like(vv), vv)[:, None])
                cen[rows[ok], :d] = cc[ok]
                again.append(rows[~ok])
            left = torch.cat(again)
            K *= 3
            if K > 4 * n + 60:
                return None
        vols.append(vol)
        cens.append(cen)
    vol, cen = torch.cat(vols), torch.cat(cens)
    if case["call"] == "tessellate":
        return dict(vol=vol, cen=cen[:, :case["dim"]])
    return dict(vol=vol, cen=cen.reshape(-1))
