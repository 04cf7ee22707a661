"""The work a program has this library do, as cases to measure.

A case is one pass of a program through the public entry points of
paper_1904_13073_amd.swgn: a frame solved and its warp field read back, a
batch of frames of uneven streams, a burst of frames through the serving
loop, a new model installed and solved, or a whole tracking step with the
geometry update. Scenes are synthesised here on the GPU from a seed: analytic
spheres and a bumpy wall seen by a pinhole depth camera, surfels at pixel
centres, nodes by Poisson-disk sampling, the live frame as the surface moved
by a smooth random field, with sensor noise and dropout.

`exact` solves the same frames in 64 bits with plain torch: every decision
that yields an integer (nearest nodes, pixel, index-map winner, gates) is
taken in 32 bits as the library defines it, all arithmetic in 64.
"""
import math
import random

import numpy as np
import torch

from paper_1904_13073_amd import swgn

F64 = torch.float64
I64 = torch.int64

# The values a case has where it does not give its own.
DEFAULTS = dict(width=640, height=480, surfels=250000, nodes=1800, gn=10, pcg=10, lam=5.0, spacing=0.025, deg=8.0,
                trans=0.02, noise=0.0015, dropout=0.05, wall=True, ball=0.0, jac=0, rigid=0, splat=False,
                host=False, streams=1, mix=0)


def listed():
    return [
        # the smallest call: a preview-sized image and a handful of nodes, where launches and latency are everything
        dict(name="frame_80x60", kind="frame", width=80, height=60, surfels=3200, nodes=40, spacing=0.05, gn=4,
             deg=3.0, trans=0.005, noise=0.001, dropout=0.0, ball=0.5),
        # a quarter-VGA-and-below sensor on one object: the repository's 160x120 workload
        dict(name="frame_160x120", kind="frame", width=160, height=120, surfels=17800, nodes=200, gn=5, lam=2.3,
             deg=3.0, trans=0.005, noise=0.001, dropout=0.0, ball=1.0),
        # an odd crop, few surfels per node (a sparse model), frames handed over from host memory as a driver does
        dict(name="frame_333x251_sparse", kind="frame", width=333, height=251, surfels=10700, nodes=1983, host=True),
        # the headline: a full 640x480 depth frame against a quarter of a million surfels
        dict(name="frame_640x480", kind="frame", surfels=248000, nodes=1788),
        # the largest single model of the range: 300k surfels and 4,000 nodes, a longer linear solve
        dict(name="frame_640x480_4k_nodes", kind="frame", surfels=300000, nodes=4000, pcg=20),
        # tracking with the rigid pre-alignment and a Jacobian kept in bf16
        dict(name="frame_320x240_rigid_bf16", kind="frame", width=320, height=240, surfels=53000, nodes=760, rigid=5,
             jac=1),
        # surfels rendered as opaque discs
        dict(name="splat_640x480", kind="frame", surfels=248000, nodes=1788, gn=5, splat=True),
        # a host that reconstructs many cameras on one GPU: 16 uneven streams per call
        dict(name="batch_16_uneven", kind="batch", streams=16, mix=400),
        # the serving loop: one frame from each of 24 attached streams arrives at once
        dict(name="serve_24_burst", kind="serve", streams=24, mix=500),
        # a new model (first frame, or a reinitialisation): surfels, node graph, then its first frame
        dict(name="model_640x480", kind="model", surfels=248000, nodes=1788, gn=3),
        # a tracking step of the whole method: solve, fuse the frame, update the geometry, read the model back
        dict(name="track_320x240", kind="track", width=320, height=240, surfels=40000, nodes=500, gn=5),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any entry point, any image, model and iteration count of the listed ranges."""
    kind = rng.choices(["frame", "batch", "serve", "model", "track"], [6, 2, 2, 1, 1])[0]
    if kind in ("batch", "serve"):
        return dict(kind=kind, streams=rng.randint(2, 14), mix=rng.randrange(1 << 20))
    w = _log_uniform(rng, 80, 640)
    h = max(60, int(w * rng.uniform(0.7, 0.8)))
    c = dict(kind=kind, width=w, height=h, surfels=_log_uniform(rng, min(3000, w * h // 3), int(0.9 * w * h)),
             gn=rng.randint(2, 10), pcg=rng.choice([5, 8, 10, 10, 15]), lam=round(rng.uniform(2.0, 6.0), 2))
    c["nodes"] = _log_uniform(rng, 30, max(60, min(4000, c["surfels"] // 5)))
    if kind == "frame":
        c["rigid"] = rng.choice([0, 0, 0, 3])
        c["jac"] = rng.choice([0, 0, 0, 0, 1, 2])
        c["splat"] = rng.random() < 0.15
        c["host"] = rng.random() < 0.3
    return c


# ----------------------------------------------------------------------------
# Scenes
# ----------------------------------------------------------------------------

def _full(case):
    return {**DEFAULTS, **case}


def _members(case):
    """The streams of a case: itself, or the uneven mix of a batch."""
    c = _full(case)
    if c["streams"] == 1:
        return [c]
    rng = random.Random(c["mix"])
    out = []
    for _ in range(c["streams"]):
        w, h = rng.choice([(320, 240), (640, 480)])
        wall = rng.random() < 0.5
        nodes = rng.randint(300, 4000)
        surfels = rng.randint(4000, int(min(300000, 0.95 * w * h)) if wall else w * h // 8)
        out.append({**c, "width": w, "height": h, "wall": wall, "surfels": max(surfels, 5 * nodes), "nodes": nodes})
    return out


def _focal(c):
    return (0.9375 if c["ball"] else 0.890625) * c["width"]


class _Scene:
    """A reference model and the live frame to solve it against."""


def _uniform(g, *shape):
    return torch.rand(shape, generator=g, dtype=F64)


def _scene(c, seed):
    dev = torch.device("cuda")
    g = torch.Generator().manual_seed(seed)
    w, h, f = c["width"], c["height"], _focal(c)
    cx, cy = w / 2.0, h / 2.0
    if c["ball"]:
        balls = [(0.02 * (float(_uniform(g)) - 0.5), 0.02 * (float(_uniform(g)) - 0.5),
                  0.4 + 1.6 * c["ball"], c["ball"])]
        wall = False
    else:
        balls = []
        for _ in range(3):
            r = 0.10 + 0.15 * float(_uniform(g))
            near = 0.8 + 0.5 * float(_uniform(g))
            xy = (2.0 * _uniform(g, 2) - 1.0) * 0.30 * (near + r)
            balls.append((float(xy[0]), 0.75 * float(xy[1]), near + r, r))
        wall = c["wall"]
    phase = 2.0 * math.pi * _uniform(g, 2)

    def depths(u, v):
        """Depth of every primitive along the rays of pixel coordinates (u, v)."""
        x, y = (u - cx) / f, (v - cy) / f
        a = x * x + y * y + 1.0
        out = []
        for bx, by, bz, r in balls:
            b = x * bx + y * by + bz
            disc = b * b - a * (bx * bx + by * by + bz * bz - r * r)
            out.append(torch.where(disc > 0, (b - torch.sqrt(disc.clamp_min(0.0))) / a, torch.inf))
        if wall:
            k = 2.0 * math.pi / 0.25
            out.append(1.45 + 0.03 * torch.sin(k * 1.45 * x + float(phase[0])) * torch.cos(k * 1.45 * y + float(phase[1])))
        return torch.stack(out)

    v, u = torch.meshgrid(torch.arange(h, dtype=F64, device=dev), torch.arange(w, dtype=F64, device=dev), indexing="ij")
    t, prim = depths(u, v).min(0)
    hit = torch.isfinite(t)
    label = torch.where(hit, prim, -1).float()[None, None]
    pool = torch.nn.functional.max_pool2d
    same = hit & (pool(label, 3, 1, 1) == label)[0, 0] & (pool(-label, 3, 1, 1) == -label)[0, 0]
    same[0] = same[-1] = False
    same[:, 0] = same[:, -1] = False

    def point(du, dv):
        z = depths(u + du, v + dv).gather(0, prim[None])[0]
        return torch.stack([(u + du - cx) / f * z, (v + dv - cy) / f * z, z], -1)

    e = 1e-3
    n = torch.linalg.cross(point(e, 0) - point(-e, 0), point(0, e) - point(0, -e))
    p = point(0, 0)
    n = n * -torch.sign((n * p).sum(-1, keepdim=True))
    n = n / n.norm(dim=-1, keepdim=True)
    facing = -(n * p).sum(-1) / p.norm(dim=-1)
    keep = (same & (facing > 0.15)).reshape(-1).nonzero()[:, 0]
    if keep.numel() > c["surfels"]:
        keep = keep[torch.randperm(keep.numel(), generator=g)[:c["surfels"]].sort().values.to(dev)]
    pos, nrm = p.reshape(-1, 3)[keep], n.reshape(-1, 3)[keep]
    area = float(((t / f) ** 2 / facing.clamp_min(0.15))[same & (facing > 0.15)].sum())

    # the live surface: pixel-space shifts and a depth offset, smooth over a few decimetres
    def field(amp, wave_px):
        out = torch.zeros_like(u)
        for _ in range(3):
            th, ph = 2.0 * math.pi * _uniform(g, 2)
            out += torch.sin((u * math.cos(th) + v * math.sin(th)) * (2.0 * math.pi / wave_px) + float(ph)) * (amp / 3)
        return out

    wave = 0.35 * f / 1.2
    shift = c["trans"] * f / 1.2
    bend = min(c["trans"], math.radians(c["deg"]) * 0.35 / (2 * math.pi))
    uu, vv = u + field(shift, 1.7 * wave), v + field(shift, 1.7 * wave)
    live = depths(uu, vv).min(0).values + field(bend, wave)
    live = live + c["noise"] * torch.randn(h, w, generator=g, dtype=F64).to(dev)
    gone = (_uniform(g, h, w) < c["dropout"]).to(dev) | ~torch.isfinite(live)

    s = _Scene()
    s.pos, s.nrm = pos.float().contiguous(), nrm.float().contiguous()
    s.depth = torch.where(gone, 0.0, live).float().contiguous()
    s.spacing = min(c["spacing"], math.sqrt(0.5 * area / c["nodes"]))
    nodes = _poisson(s.pos, s.spacing, c["nodes"], g)
    while nodes.numel() < c["nodes"]:                        # (a sparse or ragged model: nodes nearer together)
        s.spacing *= 0.85
        nodes = _poisson(s.pos, s.spacing, c["nodes"], g)
    s.node_pos = s.pos[nodes].contiguous()
    s.radius = (0.7 * 1.4142 * s.pos[:, 2] / f).contiguous()
    s.f, s.cx, s.cy = f, cx, cy
    return s


def _poisson(pos, spacing, target, g):
    """Poisson-disk sample of the surfels: random order, nobody nearer than `spacing` to one taken before."""
    alive = torch.randperm(pos.shape[0], generator=g).to(pos.device)
    taken, count = [], 0
    while alive.numel() and count < target:
        cand = pos[alive[:256]]
        near = torch.zeros(cand.shape[0], cand.shape[0], device=pos.device)
        for k in range(3):
            near += (cand[:, None, k] - cand[None, :, k]).square()
        got = ~torch.tril(near < spacing * spacing, -1).any(1)      # nobody before it in the batch is near
        taken.append(alive[:256][got])
        count += int(got.sum())
        chosen, rest = cand[got], pos[alive]
        far = torch.ones(rest.shape[0], dtype=torch.bool, device=pos.device)
        for part in chosen.split(64):
            d = torch.zeros(part.shape[0], rest.shape[0], device=pos.device)
            for k in range(3):
                d += (part[:, None, k] - rest[None, :, k]).square()
            far &= (d >= spacing * spacing).all(0)
        alive = alive[far]
    return torch.cat(taken)[:target]


# ----------------------------------------------------------------------------
# The cases through the library
# ----------------------------------------------------------------------------

def _config(c, s):
    return swgn.sw_config_default(width=c["width"], height=c["height"], fx=s.f, fy=s.f, cx=s.cx, cy=s.cy,
                                  gn_iters=c["gn"], pcg_iters=c["pcg"], lambda_reg=c["lam"], node_sigma=s.spacing,
                                  jac_dtype=c["jac"], rigid_iters=c["rigid"], splat=int(c["splat"]))


def _install(st, c, s):
    st.set_reference_surfels(s.pos, s.nrm)
    if c["splat"] or c["kind"] == "track":
        st.set_surfel_attributes(radius=s.radius)
    st.set_node_graph(s.node_pos)


class _State:
    """What a program keeps between frames: its streams, and the frames at hand."""


def prepare(case, seed):
    z = _State()
    z.kind = case["kind"]
    z.members = _members(case)
    z.scenes = [_scene(c, 1000 * seed + i) for i, c in enumerate(z.members)]
    torch.cuda.synchronize()
    z.streams = []
    for c, s in zip(z.members, z.scenes):
        st = swgn.Stream(_config(c, s))
        _install(st, c, s)
        z.streams.append(st)
    z.frames = [s.depth.cpu().numpy() if c["host"] else s.depth for c, s in zip(z.members, z.scenes)]
    z.t_now = 1
    if z.kind == "track":                                    # where the program keeps the model it reads back
        z.room = z.members[0]["surfels"] + 2 * z.members[0]["width"] * z.members[0]["height"]
        z.model = {k: np.zeros((z.room,) + d, t) for k, d, t in (
            ("pos", (3,), np.float32), ("nrm", (3,), np.float32), ("radius", (), np.float32),
            ("confidence", (), np.float32), ("t_observed", (), np.int32))}
    if z.kind == "batch":
        z.batch = swgn.Batch()
    if z.kind == "serve":
        z.server = swgn.Server()
        for st in z.streams:
            z.server.attach(st)
    return z


def _result(stats, se3):
    """A frame's outputs: the node transforms and the statistics of its iterations."""
    f = lambda k: np.concatenate([np.asarray(s[k], np.float32) for s in stats])     # noqa: E731
    return {"se3": np.concatenate(se3), "e_data": f("e_data"), "e_reg": f("e_reg"), "pcg_resid": f("pcg_resid"),
            "n_corr": np.concatenate([np.asarray(s["n_corr"], np.int32) for s in stats])}


def run(state):
    z = state
    if z.kind == "batch":
        stats, _ = z.batch.solve(z.streams, z.frames)
        return _result(stats, [st.node_se3() for st in z.streams])
    if z.kind == "serve":
        tickets = [z.server.submit(st, d) for st, d in zip(z.streams, z.frames)]
        stats = [z.server.poll(t)[0] for t in tickets]
        return _result(stats, [st.node_se3() for st in z.streams])
    st, c, s, depth = z.streams[0], z.members[0], z.scenes[0], z.frames[0]
    if z.kind == "model":
        _install(st, c, s)
    out = _result([st.solve_frame(depth)], [st.node_se3()])
    if z.kind == "track":
        st.fuse_frame(depth, z.t_now)
        z.t_now += 1
        st.update_geometry()
        for k, v in zip(z.model, st.reference_surfels() + st.surfel_attributes()):
            n = min(len(v), z.room)
            z.model[k][:n] = v[:n]
            z.model[k][n:] = 0
        out.update(z.model)
    return out


def work(case):
    """Each surfel, its skinning and each pixel read once per frame, the node transforms written once; the
    arithmetic of the iterations (warp, Jacobian and its products with itself, the linear solve's products)."""
    total = {"bytes": 0.0, "flops": 0.0}
    for c in _members(case):
        px, ns, nn = c["width"] * c["height"], c["surfels"], c["nodes"]
        total["bytes"] += 4.0 * px + 56.0 * ns + 48.0 * nn
        total["flops"] += (c["gn"] + c["rigid"]) * 400.0 * ns + c["gn"] * (1250.0 * ns + c["pcg"] * 72.0 * 15 * nn)
        if c["kind"] == "model":
            total["bytes"] += 24.0 * ns
            total["flops"] += 8.0 * ns * 64
        if c["kind"] == "track":
            total["bytes"] += 2.0 * 36.0 * ns + 36.0 * px
            total["flops"] += 300.0 * ns + 1500.0 * px
    return total


# ----------------------------------------------------------------------------
# The same frames in 64 bits
# ----------------------------------------------------------------------------

def _nearest(p, q, k):
    """The k nearest of q to every p by the 32-bit squared distance, ties to the lower index."""
    out = []
    ids = torch.arange(q.shape[0], device=q.device, dtype=I64)
    for part in p.split(8192):
        d = [part[:, None, a] - q[None, :, a] for a in range(3)]
        key = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]
        out.append(torch.topk((key.view(torch.int32).to(I64) << 32) | ids, k, largest=False).values & 0xFFFFFFFF)
    return torch.cat(out)


def _qmul(a, b):
    aw, av, bw, bv = a[..., :1], a[..., 1:], b[..., :1], b[..., 1:]
    return torch.cat([aw * bw - (av * bv).sum(-1, keepdim=True), aw * bv + bw * av + torch.linalg.cross(av, bv)], -1)


def _qconj(a):
    return torch.cat([a[..., :1], -a[..., 1:]], -1)


def _pure(v):
    return torch.cat([torch.zeros_like(v[..., :1]), v], -1)


def _rotate(q, v):
    return _qmul(_qmul(q, _pure(v)), _qconj(q))[..., 1:]


def _blend(q, t, a, v):
    """Warped points: q [n,4,4], t [n,4,3] node transforms, a [n,4] signed weights, v [n,3]."""
    r = (a[..., None] * q).sum(1)
    d = (a[..., None] * 0.5 * _qmul(_pure(t), q)).sum(1)
    norm = r.norm(dim=-1, keepdim=True)
    r, d = r / norm, d / norm
    return _rotate(r, v) + 2.0 * _qmul(d, _qconj(r))[..., 1:], r


def _normals(depth, s, gate):
    """Normal map by central differences (validity in 32 bits), zero where there is none."""
    h, w = depth.shape
    ok = (depth > 0) & torch.isfinite(depth)
    c = depth[1:-1, 1:-1]
    nb = [depth[:-2, 1:-1], depth[2:, 1:-1], depth[1:-1, :-2], depth[1:-1, 2:]]
    good = ok[1:-1, 1:-1] & ok[:-2, 1:-1] & ok[2:, 1:-1] & ok[1:-1, :-2] & ok[1:-1, 2:]
    for x in nb:
        good &= (x - c).abs() <= gate
    v, u = torch.meshgrid(torch.arange(h, dtype=F64, device=depth.device),
                          torch.arange(w, dtype=F64, device=depth.device), indexing="ij")
    P = torch.stack([(u - s.cx) / s.f * depth, (v - s.cy) / s.f * depth, depth.double()], -1)
    n = torch.linalg.cross(P[2:, 1:-1] - P[:-2, 1:-1], P[1:-1, 2:] - P[1:-1, :-2])
    length = n.norm(dim=-1, keepdim=True)
    good &= length[..., 0] > 0
    n = n / length.clamp_min(1e-300)
    n = n * torch.where((n * P[1:-1, 1:-1]).sum(-1, keepdim=True) > 0, -1.0, 1.0)
    N = torch.zeros(h, w, 3, dtype=F64, device=depth.device)
    N[1:-1, 1:-1] = torch.where(good[..., None], n, 0.0)
    return N.reshape(-1, 3), P.reshape(-1, 3), (N.abs().sum(-1) > 0).reshape(-1)


def _pairs(c, s, v, n, radius, N, valid, depth):
    """Matched (surfel, pixel) pairs of warped points v with normals n: index map, then the gates, in 32 bits."""
    w, h = c["width"], c["height"]
    v, n = v.float(), n.float()
    x, y, z = v.unbind(1)
    hx, hy = (s.f * (x / z) + s.cx) + 0.5, (s.f * (y / z) + s.cy) + 0.5
    inside = (z > 0) & (hx >= 0) & (hx < w) & (hy >= 0) & (hy < h)
    ux, uy = torch.where(inside, hx, 0).floor().to(I64), torch.where(inside, hy, 0).floor().to(I64)
    ids = torch.arange(v.shape[0], device=v.device, dtype=I64)
    zmap = torch.full((w * h,), torch.iinfo(I64).max, device=v.device)

    def render(mask, px, py, zz):
        key = (zz[mask].contiguous().view(torch.int32).to(I64) << 32) | ids[mask]
        zmap.scatter_reduce_(0, (py * w + px)[mask], key, "amin")

    if c["splat"]:
        half = torch.ceil((s.f * radius) / z).clamp_max(4.0)
        nv, r2 = (n[:, 0] * x + n[:, 1] * y) + n[:, 2] * z, radius * radius
        render(inside & ~(radius > 0), ux, uy, z)
        for oy in range(-4, 5):
            for ox in range(-4, 5):
                px, py = ux + ox, uy + oy
                m = inside & (radius > 0) & (max(abs(ox), abs(oy)) <= half) & (px >= 0) & (px < w) & (py >= 0) & (py < h)
                dx, dy = (px.float() - s.cx) / s.f, (py.float() - s.cy) / s.f
                nd = (n[:, 0] * dx + n[:, 1] * dy) + n[:, 2]
                t = nv / nd
                ex, ey, ez = t * dx - x, t * dy - y, t - z
                m &= (nd != 0) & (t > 0) & (((ex * ex + ey * ey) + ez * ez) <= r2)
                render(m, px, py, t)
    else:
        render(inside, ux, uy, z)
    pix = ((zmap != torch.iinfo(I64).max) & valid).nonzero()[:, 0]
    sf = zmap[pix] & 0xFFFFFFFF
    d = depth.reshape(-1)[pix]
    e = v[sf] - torch.stack([((pix % w).float() - s.cx) / s.f * d, ((pix // w).float() - s.cy) / s.f * d, d], 1)
    Nf = N[pix].float()
    dist = (e[:, 0] * e[:, 0] + e[:, 1] * e[:, 1]) + e[:, 2] * e[:, 2]
    cos = (n[sf, 0] * Nf[:, 0] + n[sf, 1] * Nf[:, 1]) + n[sf, 2] * Nf[:, 2]
    gate = float(np.float32(0.05) * np.float32(0.05))
    ok = (dist < gate) & (cos > 0.5)
    return sf[ok], pix[ok]


def _cg(apply, minv, b, steps):
    x, r = torch.zeros_like(b), b.clone()
    z = torch.einsum("kij,kj->ki", minv, r)
    p, rho = z.clone(), (r * z).sum()
    for _ in range(steps):
        if float(rho) == 0.0:
            break
        q = apply(p)
        a = rho / (p * q).sum()
        x, r = x + a * p, r - a * q
        z = torch.einsum("kij,kj->ki", minv, r)
        new = (r * z).sum()
        p, rho = z + (new / rho) * p, new
    return x, r


def _expmap(w):
    th = w.norm(dim=-1, keepdim=True)
    s = torch.where(th < 1e-12, 0.5, torch.sin(0.5 * th) / th.clamp_min(1e-300))
    return torch.cat([torch.cos(0.5 * th), s * w], -1)


def _solve(c, s):
    """The frame's Gauss-Newton solve: node transforms [nn, 12] and the statistics of its iterations."""
    dev = s.pos.device
    p, n, g = s.pos.double(), s.nrm.double(), s.node_pos.double()
    nn = g.shape[0]
    sigma = float(np.float32(s.spacing))
    idx = _nearest(s.pos, s.node_pos, 4)
    wt = torch.exp(-(p[:, None] - g[idx]).square().sum(-1) / (2.0 * sigma * sigma))
    wt = wt / wt.sum(1, keepdim=True)
    self_first = _nearest(s.node_pos, s.node_pos, 9)
    own = torch.arange(nn, device=dev)[:, None]
    me = self_first == own
    me[:, 8] |= ~me.any(1)
    nbr = self_first[~me].reshape(nn, 8)
    ej, em = own.expand(nn, 8).reshape(-1), nbr.reshape(-1)
    q = torch.zeros(nn, 4, dtype=F64, device=dev)
    q[:, 0] = 1.0
    t = torch.zeros(nn, 3, dtype=F64, device=dev)
    lam, mu = float(np.float32(c["lam"])), float(np.float32(1e-4))
    N, P, valid = _normals(s.depth, s, float(np.float32(0.03)))
    eye = torch.eye(3, dtype=F64, device=dev)

    def warped():
        sign = torch.where((q[idx] * q[idx[:, :1]]).sum(-1) >= 0, 1.0, -1.0)
        y, r = _blend(q[idx], t[idx], wt * sign, p)
        return y, _rotate(r, n), sign

    if c["rigid"]:
        R, tc = eye.clone(), torch.zeros(3, dtype=F64, device=dev)
        y0, n0, _ = warped()
        for _ in range(c["rigid"]):
            y = y0 @ R.T + tc
            sf, pix = _pairs({**c, "splat": False}, s, y, n0 @ R.T, None, N, valid, s.depth)
            J = torch.cat([torch.linalg.cross(y[sf], N[pix]), N[pix]], 1)
            res = (N[pix] * (y[sf] - P[pix])).sum(1)
            xi = -torch.linalg.solve(J.T @ J + mu * torch.eye(6, dtype=F64, device=dev), J.T @ res)
            e = _expmap(xi[None, :3])[0]
            E = torch.stack([_rotate(e, eye[k]) for k in range(3)], 1)
            R, tc = E @ R, E @ tc + xi[3:]
        qr = torch.empty(4, dtype=F64, device=dev)           # (the rotations of a rigid step are small)
        qr[0] = 0.5 * torch.sqrt(1.0 + R.trace())
        qr[1:] = torch.stack([R[2, 1] - R[1, 2], R[0, 2] - R[2, 0], R[1, 0] - R[0, 1]]) / (4.0 * qr[0])
        q, t = _qmul(qr.expand(nn, 4), q), t @ R.T + tc
    stats = dict(e_data=[], e_reg=[], pcg_resid=[], n_corr=[])
    for _ in range(c["gn"]):
        y, ny, sign = warped()
        sf, pix = _pairs(c, s, y, ny, s.radius, N, valid, s.depth)
        cl = _rotate(q, g) + t
        # each pair's residual as a function of the four twists of its surfel, differentiated at zero
        xi = torch.zeros(sf.numel(), 4, 6, dtype=F64, device=dev, requires_grad=True)
        k = idx[sf]
        turn = torch.cat([torch.ones_like(xi[..., :1]), 0.5 * xi[..., :3]], -1)
        arm = t[k] - cl[k]
        moved = arm + torch.linalg.cross(xi[..., :3], arm) + cl[k] + xi[..., 3:]
        yy, _ = _blend(_qmul(turn, q[k]), moved, (wt * sign)[sf], p[sf])
        res = (N[pix] * (yy - P[pix])).sum(1)
        J, = torch.autograd.grad(res.sum(), xi)
        res = res.detach()
        arm = _rotate(q[em], g[ej] - g[em])
        er = cl[ej] - cl[em] - arm
        Jm = torch.zeros(ej.numel(), 3, 6, dtype=F64, device=dev)
        Jm[:, 0, 1], Jm[:, 0, 2], Jm[:, 1, 2] = -arm[:, 2], arm[:, 1], -arm[:, 0]
        Jm[:, 1, 0], Jm[:, 2, 0], Jm[:, 2, 1] = arm[:, 2], -arm[:, 1], arm[:, 0]
        Jm[:, :, 3:] = -eye

        def scatter(data, edge_j, edge_m):
            out = torch.zeros((nn,) + data.shape[2:], dtype=F64, device=dev)
            out.index_add_(0, k.reshape(-1), data.reshape((-1,) + data.shape[2:]))
            out.index_add_(0, em, lam * edge_m)
            out[(slice(None),) + (slice(3, None),) * (data.dim() - 2)].index_add_(0, ej, lam * edge_j)
            return out

        def apply(x):
            a = torch.einsum("nki,nki->n", J, x[k])
            e = x[ej, 3:] + torch.einsum("eri,ei->er", Jm, x[em])
            return scatter(J * a[:, None, None], e, torch.einsum("eri,er->ei", Jm, e)) + mu * x

        diag = scatter(J[..., :, None] * J[..., None, :], eye.expand(ej.numel(), 3, 3),
                       torch.einsum("eri,erj->eij", Jm, Jm)) + mu * torch.eye(6, dtype=F64, device=dev)
        grad = scatter(J * res[:, None, None], er, torch.einsum("eri,er->ei", Jm, er))
        x, r = _cg(apply, torch.linalg.inv(diag), -grad, c["pcg"])
        stats["e_data"].append(float(res.square().sum()))
        stats["e_reg"].append(float(er.square().sum()))
        stats["pcg_resid"].append(float(r.norm()))
        stats["n_corr"].append(None)
        turn = _expmap(x[:, :3])
        t = _rotate(turn, t - cl) + cl + x[:, 3:]
        q = _qmul(turn, q)
        q = q / q.norm(dim=-1, keepdim=True)
    R = torch.stack([_rotate(q, e.expand(nn, 3)) for e in eye], -1)
    return torch.cat([R, t[..., None]], -1).reshape(nn, 12).cpu().numpy(), stats


def exact(case, seed):
    # (a tracking step's model has as many rows as 32-bit decisions let in: only its frame's solve has a 64-bit value)
    frames = [_solve(c, _scene(c, 1000 * seed + i)) for i, c in enumerate(_members(case))]
    out = {"se3": np.concatenate([f[0] for f in frames]), "n_corr": None}
    for k in ("e_data", "e_reg", "pcg_resid"):
        out[k] = np.concatenate([np.asarray(f[1][k]) for f in frames])
    return out
