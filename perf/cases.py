"""What users of the framework have it do, as cases for a timing program.

A grasp-synthesis program builds a hand's contact field once, then runs batches
of palm poses through domain query -> contact-set search -> realisation, alone,
as one pass of a ``Pipeline`` or through the server; a program with the learned
proposer also trains it and runs its encoder.  The listed cases take each of
those through the public entry points, from the smallest workload (latency and
launches) to the full one; ``draw`` spreads the same kinds over their sizes.

Hands are the three capsule hands the repository's workloads use (9, 16 and 22
joints), with link lengths from the seed; objects are spheres, superquadrics and
tool-like unions, their points in Morton order; poses put the object 8 to 12 cm
from the palm under a uniform rotation.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2511_07418_amd import lg
from paper_2511_07418_amd.pipeline import Pipeline

GOLDEN = math.pi * (3.0 - math.sqrt(5.0))
FINGERS = {9: 3, 16: 4, 22: 5}
FULL = 65536


# ---- cases -------------------------------------------------------------------
def listed():
    return [
        # a new hand: its field at the full sample count, with the witness table
        # that realisation reads, and the table saved to the host
        dict(name="build_full", kind="build", dof=22, samples=262144, grid=64, bins=64, witness=True),
        # the domain query of the full workload: every point of a large object
        # against every pose (bounded by the chunk spheres, as the pipeline runs it)
        dict(name="query_full", kind="query", dof=22, shape="tool", n=FULL, p=FULL, bounds=True, cone_deg=0.0,
             lattice=True),
        # the plain query on ragged sizes, no bounds, windows along each finger's
        # own axes (a hand whose windows share no lattice)
        dict(name="query_plain_odd", kind="query", dof=16, shape="superquadric", n=5003, p=2999, bounds=False,
             cone_deg=0.0, lattice=False),
        # the angular-tolerance query of a user who asks for a wider hit cone
        dict(name="query_cone", kind="query", dof=22, shape="tool", n=30011, p=8191, bounds=True, cone_deg=12.0,
             lattice=True),
        # draws, verdicts and compaction of the full workload on given domains
        # (also what every further pass over cached domains costs)
        dict(name="search_full", kind="search", dof=22, shape="tool", n=FULL, p=FULL, d=64, k=5, rounds=0),
        # the search with one round of contact-point optimisation
        dict(name="search_optimised", kind="search", dof=22, shape="tool", n=FULL, p=8192, d=64, k=5, rounds=1),
        # inverse kinematics and penetration of the full workload's accepted sets
        dict(name="realize_full", kind="realize", dof=22, shape="tool", n=FULL, p=FULL, d=64, k=5),
        # the smallest whole pass: a planar-fingered hand and a sphere (launch-bound)
        dict(name="step_small", kind="step", dof=9, shape="sphere", n=2048, p=256, d=16, k=3),
        # an ordinary whole pass: the four-fingered hand on a superquadric
        dict(name="step_mid", kind="step", dof=16, shape="superquadric", n=16384, p=16384, d=32, k=4),
        # a burst of requests of mixed sizes and hands through the batched server
        dict(name="serve_burst", kind="serve", requests=12, n_lo=2048, n_hi=FULL, p_lo=1024, p_hi=32768, d=32),
        # proposer inference over a large batch of objects
        dict(name="propose_batch", kind="propose", b=512, np=2048),
        # one training step of the proposer at the training batch size
        dict(name="train_step", kind="train", b=32, np=2048, targets=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["build", "query", "query", "search", "search", "realize", "step", "step", "serve", "propose",
                       "train"])
    dof = rng.choice([9, 16, 22])
    shape = rng.choice(["sphere", "superquadric", "tool"])
    n, p = _log_int(rng, 2048, FULL), _log_int(rng, 256, FULL)
    d, k = rng.choice([16, 32, 64]), FINGERS[dof] - rng.choice([0, 0, 1])
    if kind == "build":
        bins, grid = rng.choice([(32, 32), (64, 64)])
        return dict(kind=kind, dof=dof, samples=_log_int(rng, 8192, 262144), grid=grid, bins=bins,
                    witness=rng.choice([True, False]))
    if kind == "query":
        cone = rng.choice([0.0, 0.0, 10.0, 15.0])
        return dict(kind=kind, dof=dof, shape=shape, n=n, p=min(p, 16384) if cone else p,
                    bounds=rng.choice([True, True, False]), cone_deg=cone, lattice=rng.choice([True, True, False]))
    if kind == "search":
        rounds = rng.choice([0, 0, 1])
        return dict(kind=kind, dof=dof, shape=shape, n=n, p=min(p, 8192) if rounds else p, d=d, k=k, rounds=rounds)
    if kind in ("realize", "step"):
        return dict(kind=kind, dof=dof, shape=shape, n=n, p=p, d=d, k=k)
    if kind == "serve":
        return dict(kind=kind, requests=rng.randint(1, 12), n_lo=2048, n_hi=_log_int(rng, 4096, FULL), p_lo=1024,
                    p_hi=_log_int(rng, 2048, 32768), d=rng.choice([16, 32]))
    if kind == "propose":
        return dict(kind=kind, b=_log_int(rng, 1, 512), np=_log_int(rng, 257, 2048))
    return dict(kind=kind, b=_log_int(rng, 4, 64), np=_log_int(rng, 257, 2048), targets=_log_int(rng, 8, 64))


# ---- hands -------------------------------------------------------------------
def _capsule_samples(length, radius, n):
    """n area-uniform (point, normal) samples of a capsule along +z."""
    cyl, cap = 2.0 * math.pi * radius * length, 2.0 * math.pi * radius * radius
    n_cyl = int(round(n * cyl / (cyl + 2.0 * cap)))
    n_top = (n - n_cyl + 1) // 2
    i = np.arange(n_cyl)
    c, s = np.cos(i * GOLDEN), np.sin(i * GOLDEN)
    out = [np.stack([radius * c, radius * s, (i + 0.5) / max(1, n_cyl) * length, c, s, 0.0 * c], axis=1)]
    for count, z0, sign in ((n_top, length, 1.0), (n - n_cyl - n_top, 0.0, -1.0)):
        i = np.arange(count)
        cz = 1.0 - (i + 0.5) / max(1, count)
        sz = np.sqrt(1.0 - cz * cz)
        m = np.stack([sz * np.cos(i * GOLDEN), sz * np.sin(i * GOLDEN), sign * cz], axis=1)
        out.append(np.concatenate([radius * m + np.array([0.0, 0.0, z0]), m], axis=1))
    return np.concatenate(out)


def _hand(dof, seed, splay=0.9, n_surf=256):
    """Serial capsule fingers on a palm circle, splayed outward; flexion about x
    curls them towards the palm's centre."""
    rng = np.random.default_rng([seed, 1])
    X, Y, Z = (1.0, 0.0, 0.0), (0.0, 1.0, 0.0), (0.0, 0.0, 1.0)
    flex = (-0.3, 1.7)
    if dof == 9:
        spec = [(a, 0.030, [(X, 0.0, 1.6)] * 3) for a in (0.0, 120.0, 240.0)]
    elif dof == 16:
        spec = [(a, 0.030, [(Y, *flex)] + [(X, *flex)] * 3) for a in (0.0, 90.0, 180.0, 270.0)]
    else:
        spec = [(180.0, 0.035, [(Y, -0.5, 0.5), (Z, -0.8, 0.8)] + [(X, *flex)] * 3)]
        spec += [(a, 0.040, [(Y, -0.4, 0.4)] + [(X, *flex)] * 3) for a in (60.0, 20.0, -20.0)]
        spec += [(-60.0, 0.040, [(X, 0.0, 0.8), (Y, -0.4, 0.4)] + [(X, *flex)] * 3)]
    finger, parent, origin, axis, capsule, limits, surf, bases = [], [], [], [], [], [], [], []
    for f, (deg, rad, joints) in enumerate(spec):
        a = math.radians(deg)
        c, s = math.cos(splay), math.sin(splay)
        R = np.array([[math.sin(a), math.cos(a), 0.0], [-math.cos(a), math.sin(a), 0.0], [0.0, 0.0, 1.0]])
        R = R @ np.array([[1.0, 0.0, 0.0], [0.0, c, s], [0.0, -s, c]])
        base = np.concatenate([R, np.array([[rad * math.cos(a)], [rad * math.sin(a)], [0.0]])], axis=1)
        bases.append(base)
        radius = 0.008 if dof == 9 else 0.009
        lengths = np.array([0.045, 0.030, 0.025]) if dof == 9 else rng.uniform(0.020, 0.050, size=len(joints))
        for t, (ax, lo, hi) in enumerate(joints):
            finger.append(f)
            parent.append(-1 if t == 0 else len(parent) - 1)
            step = np.eye(3, 4)
            step[2, 3] = lengths[t - 1]
            origin.append((base if t == 0 else step).reshape(12))
            axis.append(ax)
            capsule.append([0.0, 0.0, 0.0, 0.0, 0.0, lengths[t], radius])
            limits.append([lo, hi])
            surf.append(_capsule_samples(lengths[t], radius, n_surf))
    f32 = lambda v: np.asarray(v, np.float64).astype(np.float32)  # noqa: E731
    return SimpleNamespace(n_fingers=len(spec), n_joints=len(finger), joint_finger=np.asarray(finger, np.int32),
                           joint_parent=np.asarray(parent, np.int32), joint_origin=f32(origin), joint_axis=f32(axis),
                           capsule=f32(capsule), limits=f32(limits), surf=f32(surf), bases=bases)


def _field_params(hand, samples, grid, bins, seed, lattice=True):
    """Windows near the fingers' reach: on one lattice of 4-voxel bricks along
    the palm's axes, or along each finger's base."""
    h = 0.003 if grid == 64 else 0.004
    frames = []
    for f, base in enumerate(hand.bases):
        own = hand.joint_finger == f
        reach = float(hand.capsule[own, 5].sum() + hand.capsule[own, 6][0])
        R, t = base[:, :3], base[:, 3]
        if lattice:
            shift = np.array([0.37, 0.29, 0.41]) * h
            o = t + R @ (np.array([0.0, -0.30, 0.22]) * reach) - 0.5 * grid * h
            o, R = np.round((o - shift) / (4 * h)) * (4 * h) + shift, np.eye(3)
        else:
            o = t + R @ (np.array([0.0, -0.30, 0.22]) * reach + np.array([0.37 * h, 0.0, 0.0]) - 0.5 * grid * h)
        frames.append(np.concatenate([R, o[:, None]], axis=1).reshape(12))
    return SimpleNamespace(samples=samples, seed=seed, grid=grid, h=h, bins=bins,
                           grid_frame=np.asarray(frames).astype(np.float32))


def _field(dof, seed, witness, lattice=True):
    hand = _hand(dof, seed)
    grid, bins, samples = (32, 32, 8192) if dof == 9 else (64, 64, 262144)
    return lg.lg_build_field(hand, _field_params(hand, samples, grid, bins, seed, lattice), keep_witness=witness)


# ---- objects and poses -------------------------------------------------------
def _rotations(rng, n):
    u = rng.uniform(size=(n, 3))
    a, b = np.sqrt(1.0 - u[:, 0]), np.sqrt(u[:, 0])
    x, y = a * np.sin(2 * math.pi * u[:, 1]), a * np.cos(2 * math.pi * u[:, 1])
    z, w = b * np.sin(2 * math.pi * u[:, 2]), b * np.cos(2 * math.pi * u[:, 2])
    return np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                     2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                     2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], axis=1).reshape(n, 3, 3)


def _poses(n, seed):
    rng = np.random.default_rng([seed, 2])
    cz, ph, dist = rng.uniform(size=n), rng.uniform(0.0, 2.0 * math.pi, size=n), rng.uniform(0.08, 0.12, size=n)
    sz = np.sqrt(1.0 - cz * cz)
    t = dist[:, None] * np.stack([sz * np.cos(ph), sz * np.sin(ph), cz], axis=1)
    return np.concatenate([_rotations(rng, n), t[:, :, None]], axis=2).reshape(n, 12).astype(np.float32)


def _morton(p):
    q = ((p - p.min(axis=0)) / np.ptp(p, axis=0).max() * 1023.0).astype(np.int64)
    code = np.zeros(len(p), np.int64)
    for b in range(10):
        for a in range(3):
            code |= ((q[:, a] >> b) & 1) << (3 * b + a)
    return np.argsort(code, kind="stable")


def _pow(x, e):
    return np.sign(x) * np.abs(x) ** e


class _Part:
    """A capsule of axis a..b whose radius goes from ra to rb (a ball swept along it)."""

    def __init__(self, a, b, ra, rb):
        self.a, self.b, self.ra, self.rb = np.asarray(a), np.asarray(b), ra, rb

    def distance(self, x):
        ab = self.b - self.a
        t = np.clip((x - self.a) @ ab / (ab @ ab), 0.0, 1.0)
        return np.linalg.norm(x - self.a - t[:, None] * ab, axis=1) - (self.ra + t * (self.rb - self.ra))

    def surface(self, rng, m):
        ab = self.b - self.a
        t = rng.uniform(size=m)
        v = rng.normal(size=(m, 3))
        v /= np.linalg.norm(v, axis=1, keepdims=True)
        side = rng.uniform(size=m) < 0.7
        axis = ab / np.linalg.norm(ab)
        w = v - (v @ axis)[:, None] * axis
        w /= np.linalg.norm(w, axis=1, keepdims=True)
        v = np.where(side[:, None], w, v)
        t = np.where(side, t, ((v @ axis) > 0).astype(float))
        return self.a + t[:, None] * ab + (self.ra + t * (self.rb - self.ra))[:, None] * v, v


def _object(shape, n, seed):
    """(points [n, 3], normals, distance function) of a seeded object; the
    distance is exact outside the sphere and the tool, radial for the superquadric."""
    rng = np.random.default_rng([seed, 3])
    if shape == "sphere":
        i = np.arange(n)
        z = 1.0 - (2.0 * i + 1.0) / n
        s = np.sqrt(1.0 - z * z)
        ph = i * GOLDEN + rng.uniform(0.0, 2.0 * math.pi)
        nrm = np.stack([s * np.cos(ph), s * np.sin(ph), z], axis=1)
        pts = 0.04 * nrm
        dist = lambda x: np.linalg.norm(x, axis=1) - 0.04  # noqa: E731
    elif shape == "superquadric":
        ax, (e1, e2) = rng.uniform(0.030, 0.080, size=3), rng.uniform(0.3, 2.0, size=2)
        eta, om = rng.uniform(-0.5 * math.pi, 0.5 * math.pi, size=8 * n), rng.uniform(-math.pi, math.pi, size=8 * n)

        def at(eta, om):
            ce = _pow(np.cos(eta), e1)
            return ax * np.stack([ce * _pow(np.cos(om), e2), ce * _pow(np.sin(om), e2), _pow(np.sin(eta), e1)], axis=1)

        area = np.linalg.norm(np.cross(at(eta + 1e-6, om) - at(eta - 1e-6, om),
                                       at(eta, om + 1e-6) - at(eta, om - 1e-6)), axis=1)
        cum = np.cumsum(np.nan_to_num(area, nan=0.0, posinf=0.0))
        pick = np.searchsorted(cum, rng.uniform(size=n) * cum[-1])
        eta, om = eta[pick], om[pick]
        pts = at(eta, om)
        ce = _pow(np.cos(eta), 2 - e1)
        nrm = np.stack([ce * _pow(np.cos(om), 2 - e2), ce * _pow(np.sin(om), 2 - e2), _pow(np.sin(eta), 2 - e1)],
                       axis=1) / ax
        bad = np.linalg.norm(nrm, axis=1) < 1e-9
        nrm[bad] = pts[bad]

        def dist(x):
            y = np.abs(x) / ax
            f = (y[:, 0] ** (2 / e2) + y[:, 1] ** (2 / e2)) ** (e2 / e1) + y[:, 2] ** (2 / e1)
            return np.linalg.norm(x, axis=1) * (1.0 - np.maximum(f, 1e-12) ** (-0.5 * e1))
    else:
        length = rng.uniform(0.080, 0.160)
        handle = rng.uniform(0.008, 0.015)
        parts = [_Part([-length / 2, 0, 0], [length / 2, 0, 0], handle, handle)]
        head = rng.uniform(0.015, 0.030, size=2)
        parts.append(_Part([length / 2, 0, -0.4 * head[0]], [length / 2 + 0.01, 0, 0.4 * head[1]], *head))
        for _ in range(int(rng.integers(0, 4))):
            a = np.array([rng.uniform(-length / 2, length / 2), 0.0, 0.0])
            v = rng.normal(size=3)
            parts.append(_Part(a, a + rng.uniform(0.02, 0.05) * v / np.linalg.norm(v), rng.uniform(0.006, 0.014),
                               rng.uniform(0.005, 0.010)))
        dist = lambda x: np.min([q.distance(x) for q in parts], axis=0)  # noqa: E731
        pts, nrm = np.zeros((0, 3)), np.zeros((0, 3))
        while len(pts) < n:
            for i, q in enumerate(parts):
                x, v = q.surface(rng, n)
                ok = np.all([o.distance(x) > 0.0 for j, o in enumerate(parts) if j != i], axis=0)
                pts, nrm = np.concatenate([pts, x[ok]]), np.concatenate([nrm, v[ok]])
        pick = rng.permutation(len(pts))[:n]
        pts, nrm = pts[pick], nrm[pick]
    nrm = nrm / np.linalg.norm(nrm, axis=1, keepdims=True)
    order = _morton(pts)
    return pts[order].astype(np.float32), nrm[order].astype(np.float32), dist


def _sdf(pts, dist, dims=64):
    lo, hi = pts.min(axis=0).astype(np.float64), pts.max(axis=0).astype(np.float64)
    h = max(0.002, (float((hi - lo).max()) + 0.022) / (dims - 1))
    origin = (0.5 * (lo + hi) - 0.5 * h * (dims - 1)).astype(np.float32)
    ax = np.arange(dims) * h
    z, y, x = np.meshgrid(ax, ax, ax, indexing="ij")
    v = dist(np.stack([x.ravel(), y.ravel(), z.ravel()], axis=1) + origin)
    return SimpleNamespace(origin=origin, h=float(np.float32(h)), dims=dims,
                           values=v.reshape(dims, dims, dims).astype(np.float32))


def _search(pts, d, k, seed, rounds=0):
    return SimpleNamespace(draws=d, k=k, mu=0.5, m_edges=8, eps=1e-3, seed=seed, request_id=0, pose_offset=0,
                           moment_scale=float(np.linalg.norm(pts.astype(np.float64), axis=1).max()), opt_outer=rounds,
                           opt_inner=8, opt_sigma=0.004)


IK = SimpleNamespace(iters=10, phase1=5, lam=1e-2, beta=0.01, tol_pos=0.002, tol_ang=0.35, margin=0.002,
                     self_collision=0)


def _pipeline(case, seed, realize):
    pts, nrm, dist = _object(case["shape"], case["n"], seed)
    kw = dict(ik=IK, sdf=_sdf(pts, dist)) if realize else {}
    pipe = Pipeline(_field(case["dof"], seed, realize), pts, nrm, _poses(case["p"], seed),
                    _search(pts, case["d"], case["k"], seed, case.get("rounds", 0)), **kw)
    # the lists and the realised rows beyond the accepted count keep these values
    pipe.sbuf.acc_list.fill_(-1)
    if realize:
        for t in (pipe.rbuf.q, pipe.rbuf.contact_err, pipe.rbuf.contact_ang, pipe.rbuf.depth, pipe.rbuf.valid):
            t.zero_()
    return pipe


# ---- the proposer ------------------------------------------------------------
LAYERS = ((6, 128), (128, 256), (256, 256), (256, 256), (256, 152))


def _weights(seed):
    """Flat parameters: per layer W [in][out] (He-uniform, the last one small), then b."""
    rng = np.random.default_rng([seed, 4])
    flat = []
    for i, (a, b) in enumerate(LAYERS):
        w = rng.uniform(-1.0, 1.0, size=a * b) * math.sqrt(6.0 / a) * (0.1 if i == 4 else 1.0)
        flat += [w, 0.05 * rng.normal(size=b)]
    return np.concatenate(flat).astype(np.float32)


def _clouds(case, seed):
    """[b][np][6]: points (m) and unit normals of ellipsoids, one per object."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    b, n = case["b"], case["np"]
    v = torch.nn.functional.normalize(torch.randn((b, n, 3), generator=g, device="cuda"), dim=2)
    ax = 0.03 + 0.05 * torch.rand((b, 1, 3), generator=g, device="cuda")
    return torch.cat([ax * v, torch.nn.functional.normalize(v / ax, dim=2)], dim=2).contiguous()


def _targets(case, seed):
    """Targets [T][9] (two rotation columns, translation / 0.1 m) and offsets [b + 1]."""
    t = case["b"] * case["targets"]
    p = _poses(t, seed).reshape(t, 3, 4)
    y = np.concatenate([p[:, :, 0], p[:, :, 1], p[:, :, 3] / 0.1], axis=1).astype(np.float32)
    off = np.arange(case["b"] + 1, dtype=np.int32) * case["targets"]
    return torch.from_numpy(y).cuda(), torch.from_numpy(off).cuda()


# ---- states and passes -------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    if kind == "build":
        hand = _hand(case["dof"], seed)
        return dict(kind=kind, hand=hand, witness=case["witness"],
                    fp=_field_params(hand, case["samples"], case["grid"], case["bins"], seed))
    if kind == "query":
        pts, nrm, _ = _object(case["shape"], case["n"], seed)
        field = _field(case["dof"], seed, False, case["lattice"])
        dev = [torch.from_numpy(np.ascontiguousarray(a.T)).cuda() for a in (pts, nrm)]
        dom = (torch.empty((case["p"], field.n_fingers, (case["n"] + 31) // 32), dtype=torch.int32, device="cuda"),
               torch.empty((case["p"], field.n_fingers), dtype=torch.int32, device="cuda"))
        return dict(kind=kind, field=field, pts=dev[0], nrm=dev[1], poses=torch.from_numpy(_poses(case["p"], seed)).cuda(),
                    bounds=lg.lg_chunk_bounds(dev[0]) if case["bounds"] else None, dom=dom,
                    cos=math.cos(math.radians(case["cone_deg"])) if case["cone_deg"] else None)
    if kind == "search":
        pipe = _pipeline(case, seed, False)
        pipe.query()
        return dict(kind=kind, pipe=pipe)
    if kind == "realize":
        pipe = _pipeline(case, seed, True)
        pipe.query()
        pipe.search()
        return dict(kind=kind, pipe=pipe)
    if kind == "step":
        return dict(kind=kind, pipe=_pipeline(case, seed, True))
    if kind == "serve":
        rng = np.random.default_rng([seed, 5])
        fields = {dof: _field(dof, seed, True) for dof in (16, 22)}
        objects = []
        for i, shape in enumerate(("sphere", "superquadric")):
            pts, nrm, dist = _object(shape, case["n_hi"], seed + i)
            objects.append((pts, nrm, _sdf(pts, dist)))
        # room for every request's inputs and two chunks of working buffers
        server = lg.Server(budget_bytes=12 << 30)
        requests = []
        for r in range(case["requests"]):
            u = (r + rng.uniform()) / case["requests"]
            v = rng.uniform()
            n = int(case["n_lo"] * (case["n_hi"] / case["n_lo"]) ** v)
            p = int(case["p_lo"] * (case["p_hi"] / case["p_lo"]) ** u)
            pts, nrm, sdf = objects[int(rng.integers(0, 2))]
            sel = np.sort(rng.choice(len(pts), size=n, replace=False))
            field = fields[(16, 22)[int(rng.integers(0, 2))]]
            requests.append(server.make_request(field, pts[sel], nrm[sel], _poses(p, seed + r),
                                                _search(pts, case["d"], field.n_fingers, seed), 1 + r, ik=IK, sdf=sdf))
        return dict(kind=kind, server=server, requests=requests, fields=fields)
    prop = lg.Proposer(max_batch=case["b"], max_points=case["np"], max_targets=case["b"] * case.get("targets", 1),
                       seed=seed)
    prop.set_params(_weights(seed))
    state = dict(kind=kind, prop=prop, x=_clouds(case, seed))
    if kind == "train":
        state["y"], state["off"] = _targets(case, seed)
    return state


def run(state):
    kind = state["kind"]
    if kind == "build":
        field = lg.lg_build_field(state["hand"], state["fp"], keep_witness=state["witness"])
        bits, _ = field.export()
        info = field.info()
        field.release()
        return dict(bits=bits.view(np.int32), set=info["bits_set"], vectors=info["vectors"], dropped=info["dropped"])
    if kind == "query":
        s = state
        args = (s["field"], s["pts"], s["nrm"], s["poses"])
        if s["cos"] is not None:
            lg.lg_query_domains_cone(*args, s["cos"], *s["dom"], bounds=s["bounds"])
        elif s["bounds"] is not None:
            lg.lg_query_domains_bounded(*args, s["bounds"], *s["dom"])
        else:
            lg.lg_query_domains(*args, *s["dom"])
        return dict(bits=s["dom"][0], count=s["dom"][1])
    if kind in ("search", "realize", "step"):
        pipe = state["pipe"]
        out = {}
        if kind == "step":
            pipe.step()
            out.update(bits=pipe.dom_bits, count=pipe.dom_count)
        elif kind == "search":
            pipe.search()
        if kind != "realize":
            b = pipe.sbuf
            out.update(set_pt=b.set_pt, set_link=b.set_link, verdict=b.verdict, tstar=b.tstar, acc=b.acc_list,
                       n_acc=b.n_acc)
        if kind == "realize":
            pipe.realize()
        if kind != "search":
            r = pipe.rbuf
            out.update(q=r.q, err=r.contact_err, ang=r.contact_ang, depth=r.depth, valid=r.valid)
        return out
    if kind == "serve":
        server = state["server"]
        tickets = [server.submit(req) for req, _ in state["requests"]]
        results = [server.wait(t) for t in tickets]
        return dict(state=np.array([r["state"] for r in results]), n_acc=np.array([r["n_acc"] for r in results]),
                    n_valid=np.array([r["n_valid"] for r in results]),
                    hash=np.array([r["acc_hash"] for r in results], np.uint64).view(np.int64))
    if kind == "propose":
        return state["prop"].forward(state["x"])
    loss, grad = state["prop"].backward(state["x"], state["y"], state["off"])
    state["prop"].adam(1e-3)
    return dict(loss=loss, grad=grad)


# ---- what a pass cannot do without -------------------------------------------
def _encoder_flops(case):
    return 2.0 * case["b"] * case["np"] * (6 * 128 + 128 * 256)


def work(case):
    kind = case["kind"]
    if kind == "build":
        # per joint sample and link: the frame, then each surface vector's window map and normal; every table written once
        j, cells = case["dof"], case["grid"] ** 3 * case["bins"]
        vectors = float(case["samples"]) * j * 256
        return dict(bytes=j * cells * (0.25 + (4.0 if case["witness"] else 0.0)), flops=vectors * 38.0)
    if kind == "propose":
        return dict(bytes=case["b"] * (case["np"] * 24.0 + 4 * (152 + 512)), flops=_encoder_flops(case))
    if kind == "train":
        n = sum(a * b + b for a, b in LAYERS)
        return dict(bytes=case["b"] * case["np"] * 24.0 + 7 * 4.0 * n, flops=_encoder_flops(case))
    if kind == "serve":
        # requests at the middle of their ranges
        n, p = math.sqrt(case["n_lo"] * case["n_hi"]), math.sqrt(case["p_lo"] * case["p_hi"])
        one = work(dict(kind="step", dof=22, n=n, p=p, d=case["d"], k=5))
        return {key: v * case["requests"] for key, v in one.items()}
    f, n, p = FINGERS[case["dof"]], case["n"], case["p"]
    grid = 32 if case["dof"] == 9 else 64
    total = dict(bytes=0.0, flops=0.0)
    if kind in ("query", "step"):
        # object, poses and merged tables in, domain bits and counts out; the points' map into the hand frame
        total["bytes"] += 24.0 * n + 48.0 * p + f * grid ** 3 * (4 if grid == 32 else 8) + p * f * (n / 8.0 + 4)
        total["flops"] += 18.0 * n * p
    if kind in ("search", "step"):
        # every domain word counted once; a set's points, links, verdict, t* and list entry; for a quarter of the
        # sets the criterion's simplex (about ten 7 x 7 pivots), with rounds 8 k warm-started ones of a pivot or two
        sets = float(p) * case["d"]
        total["bytes"] += p * f * (n / 8.0 + 4) + sets * (5 * case["k"] + 9 + 4)
        total["flops"] += 0.25 * sets * (4000.0 + (8 * case["k"] * 1000.0 if case.get("rounds") else 0.0))
    if kind in ("realize", "step"):
        # a tenth of the sets accepted: ten damped steps of every finger, then a sample per mm of every link
        acc = 0.1 * p * case["d"]
        total["bytes"] += acc * (4 + 5 * case["k"] + 4 * case["dof"] + 8 * case["k"] + 5) + 4.0 * 64 ** 3
        total["flops"] += acc * case["dof"] * (20.0 * 85 + 63 * 36)
    return total


# ---- 64-bit results ----------------------------------------------------------
def _split(flat):
    w, at = [], 0
    for a, b in LAYERS:
        w.append((flat[at:at + a * b].reshape(a, b), flat[at + a * b:at + a * b + b]))
        at += a * b + b
    return w


def _pooled(x, w):
    """Max over the points of the encoder's second layer, object by object."""
    scale = torch.tensor([10.0] * 3 + [1.0] * 3, dtype=torch.float64, device=x.device)
    rows = [(torch.relu((o.double() * scale) @ w[0][0] + w[0][1]) @ w[1][0] + w[1][1]).amax(dim=0) for o in x]
    return torch.relu(torch.stack(rows))


def _head(feat, w):
    return torch.relu(torch.relu(feat @ w[2][0] + w[2][1]) @ w[3][0] + w[3][1]) @ w[4][0] + w[4][1]


def exact(case, seed):
    """The proposer's results in 64 bits.  The other kinds return whole numbers,
    or values of sets that the library draws itself (their criterion is computed
    in 64 bits, their realisation depends on those draws)."""
    if case["kind"] not in ("propose", "train"):
        return None
    flat = torch.from_numpy(_weights(seed)).cuda().double().requires_grad_(case["kind"] == "train")
    x, w = _clouds(case, seed), _split(flat)
    feat = _pooled(x, w)
    out = _head(feat, w)
    if case["kind"] == "propose":
        return dict(out=out, feat=feat, arg=None)
    y, off = _targets(case, seed)
    o = out.repeat_interleave(case["targets"], dim=0)
    mean, ls = o[:, 8:80].reshape(-1, 8, 9), o[:, 80:].reshape(-1, 8, 9).clamp(-5.0, 2.0)
    z = (y.double()[:, None] - mean) * torch.exp(-ls)
    comp = torch.log_softmax(o[:, :8], dim=1) + (-0.5 * z * z - ls - 0.5 * math.log(2.0 * math.pi)).sum(dim=2)
    loss = -torch.logsumexp(comp, dim=1).mean()
    (grad,) = torch.autograd.grad(loss, flat)
    return dict(loss=loss.detach().reshape(1), grad=grad)
