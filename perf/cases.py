"""Workloads that the performance of this library is followed on.

Each case is one pass of work as a program does it: a sensor frame through the
whole path, the separate calls, a batch of frames of several sensors, a mesh
alone, and the calls on meshes and normals (twins of a user's mesh, plane
groups with the Gaussian accumulator, the vertex update).  Sizes follow the
organized clouds the library is built for: depth cameras from 120 x 160 to
720 x 1280, spinning LiDARs from 64 x 1024 to 128 x 2048, structured-light
scanners up to 1200 x 1944, and the odd sizes cropping leaves.

Inputs are synthetic range images made on the GPU from a seed: a floor, two
walls and boxes with depth noise and clustered holes (8 %), or a road with
curbs and boxes, range noise and dropouts (10 %).
"""
import math

import numpy as np
import torch

import paper_2007_12065_amd as pl

DEV = "cuda"

# What each listed case stands for:
CASES = [
    # the smallest frame: a time-of-flight or down-sampled depth camera, where launches count
    dict(name="frame_120x160", kind="frame", scene="room", M=120, N=160, klap=3, nlap=3, kbil=3, nbil=2, f16=False),
    # the ordinary depth camera (VGA), float32 normals, the settings of the benchmark
    dict(name="frame_480x640", kind="frame", scene="room", M=480, N=640, klap=3, nlap=4, kbil=3, nbil=2, f16=False),
    # a cropped VGA frame with float16 normals: no dimension a multiple of a tile
    dict(name="frame_437x613_f16", kind="frame", scene="room", M=437, N=613, klap=3, nlap=4, kbil=3, nbil=2, f16=True),
    # the largest depth-camera frame (1280 x 720)
    dict(name="frame_720x1280", kind="frame", scene="room", M=720, N=1280, klap=3, nlap=4, kbil=3, nbil=2, f16=False),
    # a spinning LiDAR of 64 beams: 5 x 5 windows, three bilateral sweeps
    dict(name="lidar_64x1024", kind="frame", scene="road", M=64, N=1024, klap=5, nlap=4, kbil=5, nbil=3, f16=False),
    # a dense spinning LiDAR of 128 beams
    dict(name="lidar_128x2048", kind="frame", scene="road", M=128, N=2048, klap=5, nlap=4, kbil=5, nbil=3, f16=False),
    # the four separate calls on the ordinary frame: programs that need the unfiltered normals too
    dict(name="calls_480x640", kind="calls", scene="room", M=480, N=640, klap=3, nlap=4, kbil=3, nbil=2, f16=False),
    # one step of a server: frames of all four sensors in one batch, float16 normals, replayed from its graph
    dict(name="batch_mix_7", kind="batch", sizes="120x160,480x640,480x640,64x1024,128x2048,64x1024,480x640", f16=True),
    # the mesh alone, unsmoothed, of a structured-light scanner
    dict(name="mesh_1200x1944", kind="mesh", scene="room", M=1200, N=1944),
    # twins of a mesh that the caller brings (here about 0.5 M triangles, as a reader of a mesh file has them)
    dict(name="twins_480x640", kind="twins", scene="room", M=480, N=640, shuffled=True),
    # the start of the plane search on a frame: accumulator over a sample of the normals, then groups
    dict(name="planes_480x640", kind="planes", scene="room", M=480, N=640, stride=8, level=4, f16=False),
    # vertices moved by filtered normals, five sweeps
    dict(name="vertices_480x640", kind="vertices", scene="room", M=480, N=640, sweeps=5, f16=False),
]

SENSORS = {"120x160": ("room", 3, 3, 3, 2), "480x640": ("room", 3, 4, 3, 2),
           "64x1024": ("road", 5, 4, 5, 3), "128x2048": ("road", 5, 4, 5, 3)}
SIGMA = 0.1                        # sigma_length and sigma_angle
LAMBDA = 1.0


def listed():
    return [dict(c) for c in CASES]


def _size(rng, scene):
    """Rows and columns over the sensors' range, spread over the logarithm."""
    if scene == "road":
        return rng.choice([16, 32, 40, 64, 100, 128]), int(round(math.exp(rng.uniform(math.log(512), math.log(2048)))))
    m = math.exp(rng.uniform(math.log(97), math.log(720)))
    return int(m), int(min(1280, m * rng.uniform(1.2, 1.8)))


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "calls", "batch", "mesh", "twins", "planes", "vertices"])
    if kind == "batch":
        n = rng.randint(2, 7)
        sizes = [rng.choice(["120x160", "480x640", "64x1024", "128x2048"]) for _ in range(n)]
        return dict(kind=kind, sizes=",".join(sizes), f16=rng.random() < 0.6)
    scene = "road" if kind in ("frame", "calls") and rng.random() < 0.4 else "room"
    M, N = _size(rng, scene)
    c = dict(kind=kind, scene=scene, M=M, N=N)
    if kind in ("frame", "calls"):
        k = rng.choice([3, 5, 5, 7]) if scene == "road" else rng.choice([3, 3, 3, 5])
        if scene == "room" and k == 5 and M > 400:          # wide windows on the smaller frames
            c.update(M=M // 2, N=N // 2)
        return dict(c, klap=min(k, 5), nlap=rng.randint(1, 5), kbil=k, nbil=rng.randint(1, 3), f16=rng.random() < 0.4)
    if kind == "mesh":
        s = math.exp(rng.uniform(0.0, math.log(1.6)))
        return dict(c, M=int(M * s), N=int(N * s))
    if kind == "twins":
        return dict(c, shuffled=rng.random() < 0.5)
    if kind == "planes":
        return dict(c, stride=rng.choice([1, 4, 8]), level=rng.choice([3, 4]), f16=rng.random() < 0.3)
    return dict(c, sweeps=rng.randint(1, 6), f16=rng.random() < 0.3)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _boxes(d, o, centers, yaws, halves):
    """First hit of rays d [P, 3] from o with upright boxes turned by yaw."""
    t = torch.full(d.shape[:1], math.inf, dtype=d.dtype, device=d.device)
    for c, yaw, h in zip(centers, yaws, halves):
        cs, sn = math.cos(yaw), math.sin(yaw)
        rot = torch.tensor([[cs, -sn, 0.0], [sn, cs, 0.0], [0.0, 0.0, 1.0]], dtype=d.dtype, device=d.device)
        q, ol = d @ rot, (torch.tensor(o, dtype=d.dtype, device=d.device) - torch.tensor(c, dtype=d.dtype, device=d.device)) @ rot
        hv = torch.tensor(h, dtype=d.dtype, device=d.device)
        q = torch.where(q == 0, torch.full_like(q, 1e-30), q)
        a, b = (-hv - ol) / q, (hv - ol) / q
        lo, hi = torch.minimum(a, b).amax(1), torch.maximum(a, b).amin(1)
        t = torch.where((hi >= lo) & (lo > 1e-6), torch.minimum(t, lo), t)
    return t


def _room(M, N, seed):
    """A pinhole camera 1.2 m above the floor, pitched 20 degrees down toward a
    room corner, with six boxes; noise 0.0012 z^2, clustered holes 8 %."""
    r = np.random.default_rng(seed)
    g = torch.Generator(device=DEV).manual_seed(seed)
    f = 525.0 * N / 640.0
    row, col = torch.meshgrid(torch.arange(M, dtype=torch.float64, device=DEV),
                              torch.arange(N, dtype=torch.float64, device=DEV), indexing="ij")
    cam = torch.stack([(col - (N - 1) / 2) / f, (row - (M - 1) / 2) / f, torch.ones_like(row)], -1).reshape(-1, 3)
    wx, wy = (float(v) for v in r.uniform(2.2, 3.8, 2))
    yaw, pitch = math.atan2(wy, wx) + float(r.uniform(-0.08, 0.08)), math.radians(20.0)
    fw = np.array([math.cos(pitch) * math.cos(yaw), math.cos(pitch) * math.sin(yaw), -math.sin(pitch)])
    rt = np.array([math.sin(yaw), -math.cos(yaw), 0.0])
    axes = torch.tensor(np.stack([rt, np.cross(fw, rt), fw]), device=DEV)
    d = cam @ axes
    inf = torch.full(d.shape[:1], math.inf, dtype=d.dtype, device=DEV)
    t = torch.where(d[:, 2] < 0, -1.2 / d[:, 2], inf)
    t = torch.minimum(t, torch.where(d[:, 0] > 0, wx / d[:, 0], inf))
    t = torch.minimum(t, torch.where(d[:, 1] > 0, wy / d[:, 1], inf))
    centers, yaws, halves = [], [], []
    for _ in range(6):
        side = r.uniform(0.1, 0.5, 3)
        rho, phi = float(r.uniform(1.2, 2.2)), yaw + float(r.uniform(-0.4, 0.4))
        centers.append([rho * math.cos(phi), rho * math.sin(phi), side[2] / 2])
        yaws.append(float(r.uniform(0, math.pi)))
        halves.append((side / 2).tolist())
    t = torch.minimum(t, _boxes(d, [0.0, 0.0, 1.2], centers, yaws, halves))
    z = t + torch.randn(t.shape, generator=g, device=DEV, dtype=torch.float64) * 0.0012 * t * t
    pts = (cam * z[:, None]).reshape(M, N, 3).float()
    blob = torch.nn.functional.avg_pool2d(torch.rand((1, 1, M, N), generator=g, device=DEV), 3, 1, 1).reshape(-1)
    pts.view(-1, 3)[torch.topk(blob, int(0.08 * M * N)).indices] = math.nan
    return pts


def _road(M, N, seed):
    """A spinning LiDAR 1.73 m above a road with curbs and ten car-sized boxes;
    range noise 2 cm, no return past 120 m, 10 % dropouts."""
    r = np.random.default_rng(seed)
    g = torch.Generator(device=DEV).manual_seed(seed)
    e = torch.deg2rad(3.0 - 28.0 * torch.arange(M, dtype=torch.float64, device=DEV) / max(M - 1, 1))
    a = 2 * math.pi * torch.arange(N, dtype=torch.float64, device=DEV) / N
    E, A = torch.meshgrid(e, a, indexing="ij")
    d = torch.stack([torch.cos(E) * torch.cos(A), torch.cos(E) * torch.sin(A), torch.sin(E)], -1).reshape(-1, 3)
    inf = torch.full(d.shape[:1], math.inf, dtype=d.dtype, device=DEV)
    road = torch.where(d[:, 2] < 0, -1.73 / d[:, 2], inf)
    walk = torch.where(d[:, 2] < 0, -1.58 / d[:, 2], inf)
    curb = torch.where(d[:, 1] != 0, 4.0 / d[:, 1].abs(), inf)
    road = torch.where((road * d[:, 1]).abs() <= 4.0, road, inf)
    walk = torch.where((walk * d[:, 1]).abs() >= 4.0, walk, inf)
    zc = curb * d[:, 2]
    curb = torch.where((zc >= -1.73) & (zc <= -1.58), curb, inf)
    t = torch.minimum(torch.minimum(road, walk), curb)
    rad, th = 6.0 + 34.0 * np.sqrt(r.uniform(size=10)), r.uniform(0, 2 * math.pi, 10)
    centers = [[float(p * math.cos(q)), float(p * math.sin(q)), -0.98] for p, q in zip(rad, th)]
    t = torch.minimum(t, _boxes(d, [0.0, 0.0, 0.0], centers, [float(v) for v in r.uniform(0, math.pi, 10)],
                                [[2.25, 0.9, 0.75]] * 10))
    far = t > 120.0
    t = torch.where(far, torch.zeros_like(t), t) + 0.02 * torch.randn(t.shape, generator=g, device=DEV, dtype=torch.float64)
    pts = (d * t[:, None]).float()
    pts[far | (torch.rand(t.shape, generator=g, device=DEV) < 0.1)] = math.nan
    return pts.reshape(M, N, 3)


def _points(scene, M, N, seed):
    return (_room if scene == "room" else _road)(M, N, seed)


# ---------------------------------------------------------------------------
# The same quantities in plain torch: geometry and T for the cases that start
# from them, and the 64-bit values
# ---------------------------------------------------------------------------

def _triangles_ok(p):
    """[M-1, N-1, 2]: which triangles of the full mesh have three valid corners."""
    ok = ~p.isnan().any(-1)
    p1, p2, p3, p4 = ok[:-1, :-1], ok[:-1, 1:], ok[1:, 1:], ok[1:, :-1]
    return torch.stack([p1 & p2 & p3, p1 & p3 & p4], -1)


def _geometry(p):
    """Unit normals and centroids [M-1, N-1, 2, 3], NaN where a corner is missing."""
    p1, p2, p3, p4 = p[:-1, :-1], p[:-1, 1:], p[1:, 1:], p[1:, :-1]
    a, b, c = torch.stack([p3, p1], 2), torch.stack([p2, p4], 2), torch.stack([p1, p3], 2)
    n = torch.linalg.cross(b - a, c - a)
    return n / n.norm(dim=-1, keepdim=True), (a + b + c) / 3


def _laplacian(p, kernel, sweeps):
    R = kernel // 2
    M, N = p.shape[:2]
    if M <= 2 * R or N <= 2 * R:
        return p
    p = p.clone()
    for _ in range(sweeps):
        c = p[R:M - R, R:N - R]
        ws, s = torch.zeros_like(c[..., :1]), torch.zeros_like(c)
        for dy in range(-R, R + 1):
            for dx in range(-R, R + 1):
                e = p[R + dy:M - R + dy, R + dx:N - R + dx] - c
                d = e.norm(dim=-1, keepdim=True)
                use = d > 0                       # false for NaN, for distance 0 and for the point itself
                w = torch.where(use, 1 / d, torch.zeros_like(d))
                ws += w
                s += torch.where(use, w * e, torch.zeros_like(e))
        move = torch.where(ws > 0, LAMBDA * s / ws, torch.zeros_like(s))
        p[R:M - R, R:N - R] = c + torch.where(c.isnan().any(-1, keepdim=True), torch.zeros_like(c), move)
    return p


def _bilateral(n, c, kernel, sweeps):
    R = kernel // 2
    Mq, Nq = n.shape[:2]
    k = 1 / (2 * SIGMA * SIGMA)
    for _ in range(sweeps):
        ok = ~(n.isnan().any(-1) | c.isnan().any(-1))
        pad = lambda t, v: torch.nn.functional.pad(t.movedim((0, 1), (-2, -1)), (R, R, R, R), value=v).movedim((-2, -1), (0, 1))
        nn = pad(torch.where(ok[..., None], n, torch.zeros_like(n)), 0.0)
        cc = pad(torch.where(ok[..., None], c, torch.zeros_like(c)), 0.0)
        oo = pad(ok.to(n.dtype), 0.0) > 0

        def terms():
            for dy in range(2 * R + 1):
                for dx in range(2 * R + 1):
                    if dy == R and dx == R:
                        continue
                    at = (slice(dy, dy + Mq), slice(dx, dx + Nq))
                    for j in (0, 1):
                        nj, cj = nn[at][:, :, j:j + 1], cc[at][:, :, j:j + 1]
                        e = k * ((c - cj).square().sum(-1) + (n - nj).square().sum(-1))
                        yield torch.where(oo[at][:, :, j:j + 1], e, torch.full_like(e, math.inf)), nj

        low = torch.full_like(n[..., 0], math.inf)
        for e, _nj in terms():
            low = torch.fmin(low, e)
        low = torch.where(low.isfinite(), low, torch.zeros_like(low))
        s = torch.zeros_like(n)
        for e, nj in terms():
            s += torch.exp(low - e)[..., None].nan_to_num(0.0) * nj
        l2 = s.norm(dim=-1, keepdim=True)
        n = torch.where(ok[..., None] & (l2 > 0), s / l2, n)
    return n


def _frame64(p, klap, nlap, kbil, nbil):
    """points, raw normals, centroids, filtered normals and these on T, in 64 bits."""
    t = _triangles_ok(p).reshape(-1)
    q = _laplacian(p.double(), klap, nlap)
    n, c = _geometry(q)
    f = _bilateral(n, c, kbil, nbil)
    on_t = torch.zeros((t.numel(), 3), dtype=torch.float64, device=p.device)
    rows = f.reshape(-1, 3)[t]
    on_t[:len(rows)] = rows
    return q, n, c, f, on_t


def _mesh(p):
    """T of the full mesh in GID order, int32 [|T|, 3]."""
    M, N = p.shape[:2]
    i = torch.arange(M * N, dtype=torch.int32, device=p.device).reshape(M, N)
    p1, p2, p3, p4 = i[:-1, :-1], i[:-1, 1:], i[1:, 1:], i[1:, :-1]
    t = torch.stack([torch.stack([p3, p2, p1], -1), torch.stack([p1, p4, p3], -1)], 2)
    return t[_triangles_ok(p)].contiguous()


def _padded(t, rows):
    """`t` in a buffer of `rows` rows, as a program sized for every triangle holds it."""
    out = torch.zeros((rows,) + tuple(t.shape[1:]), dtype=t.dtype, device=t.device)
    out[:len(t)] = t
    return out


def _count(t):
    return torch.tensor([len(t)], dtype=torch.int32, device=DEV)


def _clear(v):
    """Rows past |T| are left as they are: give them a value."""
    for x in v:
        if x is not None:
            x.zero_()


# ---------------------------------------------------------------------------
# The work
# ---------------------------------------------------------------------------

def _batch_frames(case, seed):
    out = []
    for k, s in enumerate(case["sizes"].split(",")):
        M, N = (int(v) for v in s.split("x"))
        scene, klap, nlap, kbil, nbil = SENSORS[s]
        out.append(dict(pts=_points(scene, M, N, 64 * seed + k), kernel_lap=klap, lam=LAMBDA, iters_lap=nlap,
                        kernel_bil=kbil, sigma_length=SIGMA, sigma_angle=SIGMA, iters_bil=nbil))
    return out


def prepare(case, seed):
    kind = case["kind"]
    dt = torch.float16 if case.get("f16") else torch.float32
    if kind == "batch":
        b = pl.Batch(_batch_frames(case, seed), dt)
        for o in b.outputs:
            _clear(o.values())
        b.capture()
        return dict(kind=kind, batch=b)
    M, N = case["M"], case["N"]
    p = _points(case["scene"], M, N, seed)
    if kind in ("frame", "calls"):
        plan = pl.FramePlan(M, N, case["klap"], LAMBDA, case["nlap"], case["kbil"], SIGMA, SIGMA, case["nbil"], dt)
        _clear((plan.triangles, plan.halfedges, plan.normals_T))
        return dict(kind=kind, pts=p, plan=plan)
    if kind == "mesh":
        T = 2 * (M - 1) * (N - 1)
        i32 = lambda *s: torch.zeros(s, dtype=torch.int32, device=DEV)
        out = dict(tri_valid=torch.zeros(T, dtype=torch.uint8, device=DEV), tri_map=i32(T), triangles=i32(T, 3),
                   halfedges=i32(3 * T), n_tri=i32(1))
        return dict(kind=kind, pts=p, out=out)
    if kind == "twins":
        t = _mesh(p)
        if case["shuffled"]:
            g = torch.Generator(device=DEV).manual_seed(seed)
            t = torch.randperm(M * N, generator=g, device=DEV).int()[t.long()]
            t = t[torch.randperm(len(t), generator=g, device=DEV)]
        T = 2 * (M - 1) * (N - 1)
        return dict(kind=kind, triangles=_padded(t, T), n=_count(t), out=torch.zeros(3 * T, dtype=torch.int32, device=DEV))
    p = _laplacian(p, 3, 2)
    n = _geometry(p)[0]
    if kind == "planes":
        tri = _mesh(p)
        rows = n[_triangles_ok(p)].to(dt)
        T = 2 * (M - 1) * (N - 1)
        dom = torch.nn.functional.normalize(rows[:: max(1, len(rows) // 7)][:6].float(), dim=-1).nan_to_num(0.5).contiguous()
        return dict(kind=kind, pts=p.contiguous(), triangles=_padded(tri, T), normals=_padded(rows, T), n=_count(tri),
                    dominant=dom, stride=case["stride"], ga=pl.GaussianAccumulator(case["level"]),
                    groups=torch.zeros(T, dtype=torch.uint8, device=DEV))
    return dict(kind=kind, pts=p.contiguous(), normals=n.to(dt).contiguous(), sweeps=case["sweeps"])


def run(s):
    kind = s["kind"]
    if kind == "batch":
        s["batch"].replay()
        return s["batch"].outputs
    if kind in ("frame", "calls"):
        plan = s["plan"]
        out = dict(points=plan.points, tri_valid=plan.tri_valid, tri_map=plan.tri_map, triangles=plan.triangles,
                   halfedges=plan.halfedges, n_tri=plan.n_tri, centroids=plan.centroids, normals=plan.filtered,
                   normals_T=plan.normals_T)
        if kind == "frame":
            plan.run_fused(s["pts"])
        else:
            plan.run(s["pts"])
            out["raw"] = plan.normals
        return out
    if kind == "mesh":
        return pl.pl_mesh_opc_static(s["pts"], out=s["out"])
    if kind == "twins":
        return pl.pl_user_halfedges(s["triangles"], s["n"], out=s["out"])
    if kind == "planes":
        counts, _ = s["ga"].integrate(s["normals"], n=s["n"], stride=s["stride"])
        groups = pl.pl_group_assign(s["pts"], s["triangles"], s["normals"], s["n"], s["dominant"], 0.05, 0.96,
                                    out=s["groups"])
        return dict(counts=counts, groups=groups)
    return pl.pl_vertex_update(s["pts"], s["normals"], s["sweeps"])


def _frame_work(M, N, klap, nlap, kbil, nbil, f16, raw=False):
    P, T = M * N, 2.0 * (M - 1) * (N - 1)
    nt, h = 0.85 * T, 6 if f16 else 12
    nbytes = 24 * P + 5 * T + 24 * nt + (12 + h) * T + h * nt + (h * T if raw else 0)
    return nbytes, nlap * 0.9 * P * ((klap * klap - 1) * 15 + 8) + nt * 31 + nbil * nt * (2 * (kbil * kbil - 1) * 21 + 10)


def work(case):
    """Bytes of inputs and outputs, and the operations of the formulas (for the
    filters, per neighbour), of one pass."""
    kind = case["kind"]
    if kind == "batch":
        w = [_frame_work(*(int(v) for v in s.split("x")), *SENSORS[s][1:], case["f16"]) for s in case["sizes"].split(",")]
        return {"bytes": sum(x[0] for x in w), "flops": sum(x[1] for x in w)}
    M, N = case["M"], case["N"]
    P, T = M * N, 2.0 * (M - 1) * (N - 1)
    nt, h = 0.85 * T, 6 if case.get("f16") else 12
    if kind in ("frame", "calls"):
        b, f = _frame_work(M, N, case["klap"], case["nlap"], case["kbil"], case["nbil"], case["f16"], kind == "calls")
        return {"bytes": b, "flops": f}
    if kind == "mesh":
        return {"bytes": 12 * P + 5 * T + 24 * nt, "flops": 6.0 * T}
    if kind == "twins":
        return {"bytes": 24 * nt, "flops": 10.0 * nt}
    if kind == "planes":
        return {"bytes": 12 * P + (12 + h + 1) * nt + h * nt / case["stride"], "flops": nt * (15 + 36) + 40 * nt / case["stride"]}
    return {"bytes": 24 * P + h * T, "flops": case["sweeps"] * 6.0 * 18 * P}


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = []
        for f in _batch_frames(case, seed):
            q, _n, c, fn, on_t = _frame64(f["pts"], f["kernel_lap"], f["iters_lap"], f["kernel_bil"], f["iters_bil"])
            out.append(dict(points=q, centroids=c, normals=fn, normals_T=on_t, tri_valid=None, tri_map=None,
                            triangles=None, halfedges=None, n_tri=None))
        return out
    if kind not in ("frame", "calls", "vertices"):
        return None                  # integers, compared as they are
    p = _points(case["scene"], case["M"], case["N"], seed)
    if kind == "vertices":
        q = _laplacian(p, 3, 2)
        n = _geometry(q)[0].to(torch.float16 if case["f16"] else torch.float32).double()
        return _update64(q.double(), n, case["sweeps"])
    q, n, c, f, on_t = _frame64(p, case["klap"], case["nlap"], case["kbil"], case["nbil"])
    out = dict(points=q, centroids=c, normals=f, normals_T=on_t, tri_valid=None, tri_map=None, triangles=None,
               halfedges=None, n_tri=None)
    if kind == "calls":
        out["raw"] = n
    return out


def _update64(p, n, sweeps):
    M, N = p.shape[:2]
    use = _triangles_ok(p) & ~n.isnan().any(-1)
    n = torch.where(use[..., None], n, torch.zeros_like(n))
    corners = (((1, 1), (0, 1), (0, 0)), ((0, 0), (1, 0), (1, 1)))
    for _ in range(sweeps):
        c = _geometry(p)[1]
        s, cnt = torch.zeros_like(p), torch.zeros_like(p[..., :1])
        for k in (0, 1):
            for dy, dx in corners[k]:
                at = (slice(dy, dy + M - 1), slice(dx, dx + N - 1))
                off = torch.where(use[:, :, k, None], c[:, :, k] - p[at], torch.zeros_like(n[:, :, k]))
                s[at] += n[:, :, k] * (n[:, :, k] * off).sum(-1, keepdim=True)
                cnt[at] += use[:, :, k, None]
        p = torch.where((cnt > 0) & ~p.isnan().any(-1, keepdim=True), p + s / cnt.clamp(min=1), p)
    return p
