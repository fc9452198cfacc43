"""The work that a user of this library has it do, as cases that can be timed.

Each case is one call (or one batch, or one round of served requests) through the
public Python binding, on synthetic clouds of the protocol the workloads of
`bench.py` use: a reference sampled on a union of boxes and ellipsoids in the unit
sphere, a partial, noisy source with outliers, and a list of candidate rotations.
The sizes span those workloads, from 64 x 256 points and a few hundred rotations
to 4,096 x 16,384 points and the 36,864-rotation grid.
"""
import atexit
import functools
import math

import numpy as np
import torch

from paper_2502_00115_amd import dses, synth

LARGEST = 4096 * 16384 * 36864          # point pairs of the largest case
SERVED_REFERENCES = (2048, 3000, 5003, 8192)


# --------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------
def _register(name, n, m, k, eps, **more):
    """One dses_register call.  host: host arrays instead of device tensors;
    records: the per-rotation records too; top_k, q: those options."""
    return {"name": name, "kind": "register", "n": n, "m": m, "k": k, "eps": eps, "sigma": 0.01,
            "outliers": 0.1, "metric": "trunc_l2", "host": False, "records": False, "top_k": 0,
            "q": 0.0, **more}


def _resident(name, n, m, k, **more):
    """One dses_register_resident call against a reference and a rotation list that
    stay on the device, scored with the exact grid or the distance field."""
    return {"name": name, "kind": "resident", "n": n, "m": m, "k": k, "eps": 0.03, "sigma": 0.01,
            "outliers": 0.2, "metric": "trunc_l2", "field": True, "lookup": "nearest",
            "records": True, **more}


def listed():
    return [
        # the smallest registration in use: launches and latency
        _register("small", 64, 256, 577, 0.05, sigma=0.005, outliers=0.0, records=True),
        # one object against the uniform rotation grid: the ordinary call
        _register("object", 717, 1024, 36864, 0.03, records=True),
        # the same from host memory, odd sizes, squared metric, the best candidates too
        _register("object_host", 501, 1531, 9973, 0.03, metric="tls", host=True, records=True,
                  top_k=8),
        # pruned scoring (only candidates near the best vote count are scored)
        _register("pruned", 1203, 3001, 4608, 0.03, metric="trunc_l1", q=0.9, records=True),
        # a whole scene against the uniform grid: the largest call
        _register("scene", 4096, 16384, 36864, 0.02, sigma=0.005, outliers=0.2, records=True),
        # pose correction around an initial guess: Euler grid, small translation box
        {"name": "local", "kind": "local", "n": 1434, "m": 2048, "steps": 10, "records": True},
        # resident references as a service keeps them
        _resident("resident_field", 1001, 4096, 36864),
        _resident("resident_exact", 3777, 8192, 4608, field=False, metric="inliers",
                  records=False),
        # a reference seen for the first time: upload, distance field, first registration
        {"name": "new_reference", "kind": "new_reference", "n": 300, "m": 8192, "k": 576,
         "eps": 0.03},
        # many registrations of uneven sizes in one call
        {"name": "batch", "kind": "batch", "count": 16, "m_max": 4096, "k_max": 36864,
         "eps": 0.03},
        # a round of requests through the server, all outstanding at once
        {"name": "served", "kind": "served", "count": 16, "n_max": 4096, "k": 4608, "eps": 0.03},
        # the exhaustive baseline (every rotation with every lattice translation)
        {"name": "exhaustive", "kind": "exhaustive", "n": 64, "m": 256, "k": 577, "eps": 0.05,
         "box": 0.5},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["register", "register", "register", "register", "local", "resident",
                       "resident", "new_reference", "batch", "served", "exhaustive"])
    if kind == "register":
        n, m = _log(rng, 40, 4096), _log(rng, 128, 16384)
        k = min(_log(rng, 200, 36864), LARGEST // (n * m))
        pruned = rng.random() < 0.2
        c = _register("", n, m, k, rng.choice([0.02, 0.03, 0.04, 0.05]),
                      outliers=rng.choice([0.0, 0.1, 0.2, 0.3]),
                      metric=rng.choice(["trunc_l2", "trunc_l2", "tls", "trunc_l1", "inliers"]),
                      host=rng.random() < 0.3, records=rng.random() < 0.7,
                      top_k=rng.choice([0, 0, 5, 16]), q=rng.choice([0.5, 0.9]) if pruned else 0.0)
    elif kind == "local":
        c = {"kind": kind, "n": _log(rng, 100, 2000), "m": _log(rng, 300, 4000),
             "steps": rng.randint(4, 12), "records": rng.random() < 0.5}
    elif kind == "resident":
        field = rng.random() < 0.6
        c = _resident("", _log(rng, 256, 4096), _log(rng, 2048, 8192), _log(rng, 2000, 36864),
                      field=field, records=rng.random() < 0.5,
                      lookup=rng.choice(["nearest", "trilinear"]),
                      metric=rng.choice(["trunc_l2", "tls", "inliers"]))
    elif kind == "new_reference":
        c = {"kind": kind, "n": _log(rng, 64, 1000), "m": _log(rng, 1000, 16384),
             "k": _log(rng, 100, 2000), "eps": rng.choice([0.02, 0.03, 0.05])}
    elif kind == "batch":
        c = {"kind": kind, "count": rng.randint(3, 24), "m_max": _log(rng, 1024, 4096),
             "k_max": _log(rng, 4608, 36864), "eps": 0.03}
    elif kind == "served":
        c = {"kind": kind, "count": rng.randint(4, 24), "n_max": _log(rng, 512, 4096),
             "k": _log(rng, 1000, 4608), "eps": 0.03}
    else:
        c = {"kind": kind, "n": _log(rng, 32, 128), "m": _log(rng, 100, 512),
             "k": _log(rng, 64, 577), "eps": rng.choice([0.05, 0.06]),
             "box": rng.choice([0.3, 0.4, 0.5])}
    c.pop("name", None)
    return c


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _sizes(case):
    """(n, m, k) of each registration of the case; uneven sizes depend on the case alone."""
    kind = case["kind"]
    if kind == "local":
        return [(case["n"], case["m"], (2 * case["steps"] + 1) ** 3)]
    if kind == "batch":
        rng = np.random.default_rng([case["count"], case["m_max"], case["k_max"]])
        out = []
        for _ in range(case["count"]):
            m = _log(rng, 512, case["m_max"])
            out.append((int(m * rng.uniform(0.3, 0.8)), m,
                        _log(rng, case["k_max"] / 8, case["k_max"])))
        return out
    if kind == "served":
        rng = np.random.default_rng([case["count"], case["n_max"], case["k"]])
        return [(_log(rng, 256, case["n_max"]), SERVED_REFERENCES[int(rng.integers(0, 4))],
                 case["k"]) for _ in range(case["count"])]
    return [(case["n"], case["m"], case["k"])]


def _f32(a):
    return np.ascontiguousarray(np.asarray(a, np.float32))


@functools.lru_cache(maxsize=None)
def _grid(level):
    return synth.hopf_grid(level).reshape(-1, 9)


def _rotations(rng, k):
    """k candidates: the uniform grid of that size, or a random part of the next one."""
    level = next(v for v in range(5) if 72 * 8 ** v >= k)
    grid = _grid(level)
    return _f32(grid if len(grid) == k else grid[rng.permutation(len(grid))[:k]])


def _source(rng, shape, n, sigma, outliers, scale=1.0, clip=0.05, keep=0.7):
    """n points of a partial view: half-space cut, clipped jitter, uniform outliers."""
    pts = scale * synth.sample_surface(rng, shape, int(math.ceil(n / keep)) + 2)
    pts = pts[synth.halfspace_keep(rng, pts, keep)][:n]
    pts = synth.jitter(rng, pts, sigma, clip=clip)
    return synth.add_outliers(rng, pts, outliers, pts.min(axis=0), pts.max(axis=0))


def _clouds(rng, n, m, sigma=0.01, outliers=0.1):
    shape = synth.multi_primitive_shape(rng)
    tgt = synth.sample_surface(rng, shape, m)
    R, t = synth.random_transform(rng)
    return _f32(_source(rng, shape, n, sigma, outliers) @ R.T + t), _f32(tgt)


def _inputs(case, seed):
    """The case's clouds and rotations as host arrays (one set, or a list of sets)."""
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind in ("register", "resident"):
        src, tgt = _clouds(rng, case["n"], case["m"], case["sigma"], case["outliers"])
        return src, tgt, _rotations(rng, case["k"])
    if kind in ("new_reference", "exhaustive"):
        src, tgt = _clouds(rng, case["n"], case["m"])
        return src, tgt, _rotations(rng, case["k"])
    if kind == "local":
        # an object of 0.1 m radius, off by up to 4 degrees per Euler angle and 1.2 cm
        shape = synth.multi_primitive_shape(rng)
        tgt = 0.1 * synth.sample_surface(rng, shape, case["m"])
        src = _source(rng, shape, case["n"], 0.001, 0.1, scale=0.1, clip=0.005)
        a, b, c = rng.uniform(-4.0, 4.0, size=3)
        R = synth.euler_grid(1, 0.0)[0]
        for axis, deg in ((2, a), (1, b), (0, c)):
            R = R @ _axis_rotation(axis, math.radians(deg))
        src = src @ R.T + rng.uniform(-0.012, 0.012, size=3)
        return _f32(src), _f32(tgt), _f32(
            synth.euler_grid(case["steps"], math.radians(0.5)).reshape(-1, 9))
    if kind == "batch":
        return [_clouds(rng, n, m, 0.01, rng.uniform(0.0, 0.3)) + (_rotations(rng, k),)
                for n, m, k in _sizes(case)]
    # served: four resident references, sources cut from them
    shapes = [synth.multi_primitive_shape(rng) for _ in range(4)]
    tgts = [_f32(synth.sample_surface(rng, s, m)) for s, m in zip(shapes, SERVED_REFERENCES)]
    reqs = []
    for n, m, _ in _sizes(case):
        which = SERVED_REFERENCES.index(m)
        R, t = synth.random_transform(rng)
        reqs.append((which, _f32(_source(rng, shapes[which], n, 0.01, 0.2) @ R.T + t)))
    return tgts, reqs, _rotations(rng, case["k"])


def _axis_rotation(axis, angle):
    c, s = math.cos(angle), math.sin(angle)
    R = np.eye(3)
    i, j = [(1, 2), (2, 0), (0, 1)][axis]
    R[i, i] = R[j, j] = c
    R[i, j], R[j, i] = -s, s
    return R


def _dev(*arrays):
    return tuple(torch.from_numpy(a).cuda() for a in arrays)


_server = None


def _the_server():
    """The program's one server (it holds streams and a memory pool)."""
    global _server
    if _server is None:
        _server = dses.Server()
        atexit.register(_server.close)
    return _server


def prepare(case, seed):
    kind = case["kind"]
    data = _inputs(case, seed)
    s = {"case": dict(case)}
    if kind == "batch":
        s["problems"] = [dict(zip(("src", "tgt", "rotations"), _dev(*d)), eps=case["eps"])
                         for d in data]
    elif kind == "served":
        tgts, s["requests"], rots = data
        s["targets"] = [dses.Target(t, df_trunc=case["eps"]) for t in tgts]
        s["rotset"] = dses.RotationSet(rots)
        s["server"] = _the_server()
    elif kind == "register" and case["host"]:
        s["src"], s["tgt"], s["rot"] = data
    elif kind == "resident":
        src, tgt, rots = data
        s["src"], = _dev(src)
        s["target"] = dses.Target(tgt, df_trunc=case["eps"] if case["field"] else 0.0)
        s["rotset"] = dses.RotationSet(rots)
    elif kind == "new_reference":
        src, tgt, rots = data
        s["src"], s["tgt"] = _dev(src, tgt)
        s["rotset"] = dses.RotationSet(rots)
    else:
        s["src"], s["tgt"], s["rot"] = _dev(*data)
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def _answer(r):
    """A registration's whole answer as numbers and arrays."""
    out = {"R": r.R, "t": r.t, "rot_index": r.rot_index, "inliers": r.inliers, "error": r.error,
           "votes": r.votes, "n_valid": r.n_valid}
    if r.records is not None:
        out["records"] = {f: r.records[f] for f in ("bin", "votes", "inliers", "error")}
    if r.top is not None:
        out["top"] = {f: r.top[f] for f in ("rot_index", "inliers", "error", "votes", "t")}
    return out


def _answers(rs):
    """The answers of several registrations, field by field."""
    out = {"R": np.stack([r.R for r in rs]), "t": np.stack([r.t for r in rs])}
    for f, kind in (("rot_index", np.int64), ("inliers", np.int64), ("error", np.float32),
                    ("votes", np.int64), ("n_valid", np.int64)):
        out[f] = np.array([getattr(r, f) for r in rs], kind)
    return out


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "register":
        return _answer(dses.register(s["src"], s["tgt"], s["rot"], c["eps"], c["metric"],
                                     records=c["records"], top_k=c["top_k"], q=c["q"]))
    if kind == "local":
        return _answer(dses.register(s["src"], s["tgt"], s["rot"], 0.002, t_min=-0.016,
                                     t_max=0.016, records=c["records"]))
    if kind == "resident":
        return _answer(dses.register_resident(s["target"], s["rotset"], s["src"], c["eps"],
                                              c["metric"], records=c["records"],
                                              df_lookup=c["lookup"]))
    if kind == "new_reference":
        target = dses.Target(s["tgt"], df_trunc=c["eps"])
        r = dses.register_resident(target, s["rotset"], s["src"], c["eps"], records=True,
                                   df_lookup="trilinear")
        target.close()
        return _answer(r)
    if kind == "batch":
        rs, _ = dses.register_batch(s["problems"], records=True)
        out = _answers(rs)
        recs = np.concatenate([r.records for r in rs])
        out["records"] = {f: recs[f] for f in ("bin", "votes", "inliers", "error")}
        return out
    if kind == "served":
        ids = [s["server"].submit(s["targets"][w], s["rotset"], src, c["eps"])
               for w, src in s["requests"]]
        return _answers([s["server"].wait(i) for i in ids])
    return _answer(dses.register_exhaustive(s["src"], s["tgt"], s["rot"], c["eps"],
                                            t_min=-c["box"], t_max=c["box"], records=True))


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def work(case):
    """Clouds and rotations in, a 24-byte record per rotation out; three subtractions per
    point pair of a candidate, one rotation (18) and one distance (8) per source point.
    The exhaustive search instead takes one distance per source point, rotation and
    lattice translation; a new reference also writes its 128^3 field."""
    byts = flops = 0.0
    for n, m, k in _sizes(case):
        byts += 12 * n + 12 * m + (36 + 24) * k
        if case["kind"] == "exhaustive":
            bins = (2 * math.floor(case["box"] / case["eps"] + 1e-4) + 1) ** 3
            flops += k * n * (18 + 8.0 * bins)
        else:
            flops += k * n * (3.0 * m + 26)
    if case["kind"] == "new_reference":
        byts += 4 * 128 ** 3
        flops += 8 * 128 ** 3
    return {"bytes": float(byts), "flops": float(flops)}


# --------------------------------------------------------------------------
# the same in 64 bits, by the definitions in include/dses.h
# --------------------------------------------------------------------------
def _rho(metric, d, l1, eps, tau):
    if metric == "tls":
        return torch.clamp(d, max=tau) ** 2
    if metric == "trunc_l1":
        return torch.clamp(l1, max=tau)
    if metric == "inliers":
        return (d >= eps).double()
    return torch.clamp(d, max=tau)


def _nearest(q, y, want_l1):
    """Distance of each point of q (..., 3) to its nearest point of y, and the L1 one."""
    flat = q.reshape(-1, 3)
    step = max(1, (1 << 25) // len(y))
    d2, l1 = [], []
    for i in range(0, len(flat), step):
        d = (flat[i:i + step, None, :] - y[None]).abs_()
        d2.append((d * d).sum(-1).amin(1))
        l1.append(d.sum(-1).amin(1) if want_l1 else d2[-1])
    shape = q.shape[:-1]
    return torch.cat(d2).sqrt_().reshape(shape), torch.cat(l1).reshape(shape)


def _trilinear(y, eps, res=128):
    """The reference's distance field and a function that interpolates it."""
    lo = y.amin(0) - eps
    h = (y.amax(0) + eps - lo) / res
    ax = [lo[a] + (torch.arange(res, device=y.device, dtype=torch.float64) + 0.5) * h[a]
          for a in range(3)]
    field = torch.full((res + 2,) * 3, eps, dtype=torch.float64, device=y.device)
    # each reference point lowers the voxels within eps of it
    flat = field.view(-1)
    cell = ((y - lo) / h).long()
    reach = [int(math.ceil(eps / float(h[a]))) + 1 for a in range(3)]
    for dx in range(-reach[0], reach[0] + 1):
        for dy in range(-reach[1], reach[1] + 1):
            for dz in range(-reach[2], reach[2] + 1):
                v = cell + torch.tensor([dx, dy, dz], device=y.device)
                ok = ((v >= 0) & (v < res)).all(1)
                v = v[ok]
                c = torch.stack([ax[a][v[:, a]] for a in range(3)], 1)
                d = (c - y[ok]).norm(dim=1).clamp_(max=eps)
                at = ((v[:, 0] + 1) * (res + 2) + v[:, 1] + 1) * (res + 2) + v[:, 2] + 1
                flat.scatter_reduce_(0, at, d, "amin")

    def at(q):
        u = (q - lo) / h - 0.5
        inside = ((u >= -1) & (u < res)).all(-1)
        f = u.floor()
        w = u - f
        i = f.long().clamp_(-1, res - 1) + 1
        val = 0.0
        for a in range(2):
            for b in range(2):
                for c in range(2):
                    wt = ((w[..., 0] if a else 1 - w[..., 0]) * (w[..., 1] if b else 1 - w[..., 1])
                          * (w[..., 2] if c else 1 - w[..., 2]))
                    val = val + wt * field[i[..., 0] + a, i[..., 1] + b, i[..., 2] + c]
        return torch.where(inside, val, torch.full_like(val, eps))

    return at


def _box(lo, hi, delta):
    k0 = math.ceil(lo / delta - 1e-4)
    return k0, math.floor(hi / delta + 1e-4) - k0 + 1


def _modes(x, y, R, delta, k0, size):
    """Mode bin and count of every rotation's pair translations, by the definition."""
    nb = size ** 3
    step = max(1, min(len(R), (1 << 25) // (len(x) * len(y)), (1 << 27) // nb))
    bins, counts = [], []
    for i in range(0, len(R), step):
        p = torch.matmul(x[None], R[i:i + step].transpose(1, 2).contiguous())
        r = len(p)
        lin = torch.arange(r, device=x.device).view(r, 1, 1)
        ok = None
        for a in range(3):
            b = ((y[:, a].view(1, 1, -1) - p[:, :, a].unsqueeze(2)) / delta + 0.5).floor_()
            b = b.sub_(k0)
            good = (b >= 0) & (b < size)
            ok = good if ok is None else ok & good
            lin = lin * size + b.long()
        h = torch.bincount(lin[ok], minlength=r * nb).view(r, nb)
        top = h.amax(1)
        first = torch.where(h == top[:, None], torch.arange(nb, device=x.device), nb).amin(1)
        bins.append(first)
        counts.append(top)
    b = torch.cat(bins)
    c = torch.stack([b // (size * size), b // size % size, b % size], 1) + k0
    return c, torch.cat(counts)


def _scored(case, src, tgt, rots, eps, metric, box, q, field=False):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    x, y = (torch.from_numpy(a).double().to(dev) for a in (src, tgt))
    R = torch.from_numpy(rots).double().to(dev).view(-1, 3, 3)
    eps = float(np.float32(eps))
    k0, size = _box(-box, box, eps)
    n_valid = len(R)
    read = _trilinear(y, eps) if field else None
    if case["kind"] == "exhaustive":
        b = torch.arange(size, device=dev) + k0
        ts = torch.stack(torch.meshgrid(b, b, b, indexing="ij"), -1).view(-1, 3).double() * eps
        errors, best_t = [], []
        for r in R:
            d, l1 = _nearest((x @ r.T)[None] + ts[:, None], y, False)
            e = _rho(metric, d, l1, eps, eps).sum(1)
            errors.append(e.min())
            best_t.append(ts[e.argmin()])
        errors, t = torch.stack(errors), torch.stack(best_t)
    else:
        bins, votes = _modes(x, y, R, eps, k0, size)
        t = bins.double() * eps
        errors = []
        step = max(1, (1 << 22) // len(x))
        for i in range(0, len(R), step):
            p = torch.matmul(x[None], R[i:i + step].transpose(1, 2).contiguous())
            p = p + t[i:i + step, None]
            d, l1 = (read(p),) * 2 if field else _nearest(p, y, metric == "trunc_l1")
            errors.append(_rho(metric, d, l1, eps, eps).sum(1))
        errors = torch.cat(errors)
        off = (votes == 0) | (votes.double() < float(np.float32(q)) * votes.max().double())
        errors = torch.where(off, torch.full_like(errors, math.inf), errors)
        n_valid = int((votes > 0).sum())
    return R, t, errors, n_valid


def exact(case, seed):
    kind = case["kind"]
    if kind in ("resident", "batch", "served"):
        return None                     # large, and a nearest-voxel lookup has steps
    (n, m, k), = _sizes(case)
    if n * m * k > 3.2e10:
        return None
    src, tgt, rots = _inputs(case, seed)
    if kind == "local":
        R, t, e, _ = _scored(case, src, tgt, rots, 0.002, "trunc_l2", float(np.float32(0.016)), 0.0)
    else:
        box = float(np.float32(case["box"])) if kind == "exhaustive" else 1.0
        R, t, e, _ = _scored(case, src, tgt, rots, case["eps"], case.get("metric", "trunc_l2"),
                             box, case.get("q", 0.0), field=kind == "new_reference")
    k = int(e.argmin())
    out = {"R": R[k].cpu().numpy(), "t": t[k].cpu().numpy(), "rot_index": None, "inliers": None,
           "error": float(e[k]), "votes": None, "n_valid": None}
    if case.get("records", True):
        out["records"] = {"bin": None, "votes": None, "inliers": None, "error": e.cpu().numpy()}
    if case.get("top_k", 0):
        at = torch.sort(e, stable=True).indices[:case["top_k"]]
        out["top"] = {"rot_index": None, "inliers": None, "error": e[at].cpu().numpy(),
                      "votes": None, "t": t[at].cpu().numpy()}
    return out
