"""The tracker's work as its users have it done, as cases that can be timed and compared.

A case is one context tracking depth frames (track_frame and its relatives,
then the state read back) or one server tracking many streams.  Inputs are the
synthetic body-shaped workloads of `synth`: a posed, folded template rendered
before a wall, with measurement noise and missing pixels, along a smooth
trajectory that is walked forward and back, so that a pass can follow a pass
for as long as a program runs.  The template of a size is the same for every
seed; the trajectory, the folds, the noise and the starting pose are the
seed's.

Poses are returned in float32: everything before the pose solve (the surface,
the residuals, the Gram matrix's products) is float32 in every form, so that
is what a pose is good to, and how a renderer takes it.
"""
import functools
import math

import numpy as np
import torch

import synth
from paper_1711_07999_amd import metrics
from paper_1711_07999_amd import track as T

# What a single stream's case may say; a listed or drawn case names the rest.
#   verts, width, height  template and camera ("arm": the 2,000-vertex tube)
#   schedule, iters       a mode of `metrics`, or "full" with `iters` iterations
#   frames                depth frames tracked per pass, then the state is read
#   source                depth image on the GPU or the host, or a point cloud on the GPU
#   surface               whether the skinned vertices are read back too
SINGLE = dict(kind="single", shape="body", gram=0, fp64=False, linear=False, lambda_t=0.0, source="device",
              surface=True)
MAX_VERTEX_ITERS = 32 * 4 * 5 * 50000   # of a pass: the batch of 32 copies below


def listed():
    return [
        # The smallest call: one frame of the short tube arm (8 joints), ten
        # iterations, launches and latency alone.
        dict(SINGLE, name="arm-2k-160x120", shape="arm", verts=2000, width=160, height=120, schedule="full",
             iters=10, frames=1),
        # A coarse body on a small odd image, as a preview gives: every size
        # is ragged.
        dict(SINGLE, name="body-7001-211x157", verts=7001, width=211, height=157, schedule="full", iters=5, frames=2),
        # The smallest serving size tracked alone, surface not asked for (an
        # avatar is driven by pose and offsets).
        dict(SINGLE, name="body-10k-320x240", verts=10000, width=320, height=240, schedule="full", iters=5,
             frames=4, surface=False),
        # The headline workload: a recorded clip's frames one after another.
        dict(SINGLE, name="body-50k-640x480", verts=50000, width=640, height=480, schedule="full", iters=5, frames=8),
        # The same with the bfloat16 hi/lo Gram matrix and float64 solves.
        dict(SINGLE, name="body-50k-640x480-bf16x3", verts=50000, width=640, height=480, schedule="full", iters=5,
             frames=8, gram=1, fp64=True),
        # One iteration per frame, as a fast camera is followed: the whole
        # frame is a single pose step and a single offset step.
        dict(SINGLE, name="body-50k-640x480-1it", verts=50000, width=640, height=480, schedule="full", iters=1,
             frames=1),
        # Pose only (smooth bind), the depth image in host memory as a camera
        # driver leaves it.
        dict(SINGLE, name="bind-50k-640x480-host", verts=50000, width=640, height=480, schedule="smooth-bind",
             iters=5, frames=4, source="host"),
        # The paper's twelve pose and two offset iterations with the linear
        # blend, on an odd template and an odd image.
        dict(SINGLE, name="paper-23457-333x251-linear", verts=23457, width=333, height=251,
             schedule="paper-schedule-linear", iters=14, frames=2, linear=True),
        # An organised point cloud instead of a depth image.
        dict(SINGLE, name="cloud-31113-424x320", verts=31113, width=424, height=320, schedule="full", iters=5,
             frames=4, source="cloud"),
        # The high-resolution configuration: temporal weight, float64 pose solve.
        dict(SINGLE, name="highres-200k-512x424", verts=200000, width=512, height=424, schedule="full", iters=5,
             frames=4, fp64=True, lambda_t=0.5),
        # The serving mix at saturation: two streams of each of its six sizes.
        dict(kind="mix", name="serve-mix-12", streams=12, iters=5, frames=3),
        # The largest: 32 streams of the headline size in one server.
        dict(kind="copies", name="serve-32x50k-640x480", streams=32, verts=50000, width=640, height=480, iters=5,
             frames=4),
    ]


def draw(rng):
    def spread(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    kind = rng.choice(["single", "single", "single", "copies"])
    width = spread(200, 640)
    height = int(width * rng.uniform(0.70, 0.83))
    if kind == "copies":
        case = dict(kind="copies", streams=spread(2, 32), verts=spread(7000, 60000), width=width, height=height,
                    iters=rng.choice([1, 3, 5]), frames=rng.randint(1, 4))
        while case["streams"] * case["frames"] * case["iters"] * case["verts"] > MAX_VERTEX_ITERS:
            case["streams"] -= 1
        return case
    schedule, iters = rng.choice([("full", 1), ("full", 3), ("full", 5), ("full", 10), ("smooth-bind", 5),
                                  ("smooth-bind", 12), ("paper-schedule", 14), ("paper-schedule-linear", 14)])
    gram = rng.choice([0, 0, 0, 1, 2])
    return dict(SINGLE, verts=spread(7000, 200000), width=width, height=height, schedule=schedule, iters=iters,
                frames=rng.randint(1, 6), gram=gram, fp64=gram != 0 or rng.random() < 0.25,
                linear=schedule.endswith("linear"), lambda_t=rng.choice([0.0, 0.0, 0.5]),
                source=rng.choice(["device", "device", "host", "cloud"]), surface=rng.random() < 0.5)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
@functools.lru_cache(maxsize=None)
def _body(shape, verts, width, height):
    """The template of a size: the same whatever the seed."""
    if shape == "arm":
        return synth.make_arm()
    focal = 0.8203125 * width   # 525 at 640 pixels, 262.5 at 320
    cam = dict(width=width, height=height, fx=focal, fy=focal, cx=(width - 1) / 2.0, cy=(height - 1) / 2.0)
    return synth.make_body(verts, cam, 2.6)


def _views(body, rng, n):
    """A trajectory of n poses, the depth image of each, and a starting pose
    a few degrees off the first."""
    P = len(body.model["joint_parent"])
    if body.model["rest_xyz"].shape[0] == 2000 and P == 8:
        poses = np.where(body.angular, rng.uniform(-math.radians(10), math.radians(10), P),
                         rng.uniform(-0.01, 0.01, P))[None].repeat(n, 0)
        phi, zeros, start = None, 0.30, np.zeros(P)
    else:
        phi = synth.fold_offsets(body, rng, 0.005)
        base = np.where(body.angular, rng.uniform(-math.radians(5), math.radians(5), P), 0.0)
        poses = synth.smooth_trajectory(body, rng, n, base, math.radians(3), 0.005)
        zeros = 0.25
        start = poses[0] + np.where(body.angular, rng.uniform(-math.radians(2), math.radians(2), P),
                                    rng.uniform(-0.01, 0.01, P))
    images = [synth.render_frame(body.model, body.camera, synth.pose_surface(body.model, p, phi), rng, zeros, 0.002)
              for p in poses]
    return poses, images, start


def _params(case, P):
    arm = case.get("shape") == "arm"
    prm = synth.default_params(P, case["iters"], 0.10 if arm else 0.05, lambda_t=case.get("lambda_t", 0.0),
                               lambda_k=0.01 if arm else 0.1)
    prm["do_pose"], prm["do_shape"] = metrics.mode_schedule(case.get("schedule", "full"), 0, case["iters"])
    prm["gram_mode"] = case.get("gram", 0)
    prm["pose_solve_fp64"] = int(case.get("fp64", False))
    prm["shape_solve_fp64"] = int(case.get("fp64", False) and case.get("gram", 0) != 0)
    prm["active"] = None
    return prm


def _cloud(depth, cam):
    """Organised point cloud of a depth image, in the tracker's float32 order."""
    v, u = np.mgrid[0:cam["height"], 0:cam["width"]].astype(np.float32)
    x = ((u - np.float32(cam["cx"])) * depth) / np.float32(cam["fx"])
    y = ((v - np.float32(cam["cy"])) * depth) / np.float32(cam["fy"])
    return np.stack([x, y, depth], -1).astype(np.float32)


def _model(case, body):
    return dict(body.model, blend=T.TRACK_BLEND_LINEAR) if case.get("linear") else body.model


class _Tracker(T.Tracker):
    """A context and the place in the walk of what it tracks."""

    at = 0


class _Server:
    """A server and its streams; closed with the last reference to it."""

    at = 0

    def __init__(self, params, max_streams):
        self.sv = T.track_server_create(params, 1 << 38, max_streams)
        self.ids, self.sizes, self.views, self.first = [], [], [], []

    def __del__(self):
        try:
            T.track_server_destroy(self.sv)
        except TypeError:
            pass   # at the interpreter's end the binding may be gone already


def _device(image):
    return torch.from_numpy(np.ascontiguousarray(image)).to("cuda")


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    if case["kind"] == "single":
        body = _body(case["shape"], case["verts"], case["width"], case["height"])
        _, images, start = _views(body, rng, min(case["frames"], 4) + 1)
        if case["source"] == "device":
            views = [_device(d) for d in images]
        elif case["source"] == "cloud":
            views = [_device(_cloud(d, body.camera)) for d in images]
        else:
            views = images
        params = _params(case, len(start))
        return dict(case=case, views=views, start=start,
                    tracker=_Tracker(_model(case, body), body.camera, params, start))
    sizes = [(case["verts"], case["width"], case["height"])] if case["kind"] == "copies" else \
        [(v, w, h) for v in (10000, 50000, 200000) for w, h in ((320, 240), (640, 480))]
    server = _Server(_params(case, 1), case["streams"])
    sets = []
    for v, w, h in sizes:
        body = _body("body", v, w, h)
        poses, images, start = _views(body, rng, 5)
        sets.append((body, poses, [_device(d) for d in images], start - poses[0]))
    for s in range(case["streams"]):
        body, poses, views, off = sets[s % len(sets)]
        first = (s // len(sets)) % len(poses)
        theta0 = poses[first] + off + np.where(body.angular, rng.uniform(-0.005, 0.005, len(off)), 0.0)
        server.ids.append(T.track_server_open(server.sv, body.model, body.camera, theta0))
        server.sizes.append((len(off), body.model["rest_xyz"].shape[0]))
        server.views.append(views)
        server.first.append(first)
    return dict(case=case, server=server)


def _walk(k, n):
    """Frame k of an endless forward-backward walk over n frames."""
    q = k % (2 * n - 2)
    return q if q < n else 2 * n - 2 - q


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(state):
    case = state["case"]
    if case["kind"] != "single":
        return _run_server(case, state["server"])
    trk, views = state["tracker"], state["views"]
    track = trk.frame_xyz if case["source"] == "cloud" else trk.frame
    failed = 0
    for _ in range(case["frames"]):
        if track(views[_walk(trk.at, len(views))]) != T.TRACK_OK:
            failed += 1
            trk.reset(state["start"])   # lost: back to the start, as a program would
        trk.at += 1
    theta, phi, verts, stats = trk.state(want_verts=case["surface"])
    return dict(theta=theta.astype(np.float32), phi=phi, verts=verts,
                counts=np.array([failed] + [stats[k] for k in ("n_valid_px", "n_assoc_px", "n_obs_verts")]),
                energy=np.array([stats["energy_first"], stats["energy_last"]], np.float32))


def _run_server(case, server):
    for _ in range(case["frames"]):
        for sid, views, first in zip(server.ids, server.views, server.first):
            T.track_server_submit(server.sv, sid, views[_walk(first + server.at, len(views))], tag=server.at)
        server.at += 1
    due = case["frames"] * case["streams"]
    while due:
        due -= T.track_server_step(server.sv)
    done = T.track_server_poll(server.sv, case["frames"] * case["streams"])
    done.sort(key=lambda c: (c["stream"], c["tag"]))
    states = [T.track_server_state(server.sv, sid, P, V) for sid, (P, V) in zip(server.ids, server.sizes)]
    return dict(theta=np.stack([th for th, _ in states]).astype(np.float32), phi=[ph for _, ph in states],
                counts=np.array([[c[k] for k in ("status", "n_valid_px", "n_assoc_px", "n_obs_verts")] for c in done]))


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    """Per iteration the image, the template (points, weights, links,
    triangles, neighbours) and the offsets are read and the offsets written
    where they move; the Gram matrix of the vertices in view (about a quarter
    of them), the skinning and one distance per vertex-sized step of the rest."""
    total = dict(bytes=0.0, flops=0.0)
    if case["kind"] == "mix":
        sizes = [(v, w, h) for v in (10000, 50000, 200000) for w, h in ((320, 240), (640, 480))]
        parts = [sizes[s % 6] for s in range(case["streams"])]
    else:
        parts = [(case["verts"], case["width"], case["height"])] * case.get("streams", 1)
    dp, ds = metrics.mode_schedule(case.get("schedule", "full"), 0, case["iters"])
    px = 12 if case.get("source") == "cloud" else 4
    for v, w, h in parts:
        P = 8 if case.get("shape") == "arm" else 75
        per = px * w * h + v * (12 + 16 + 4 + 12 + 24)
        shape = v * (16 + 12 + (12 if case.get("lambda_t", 0.0) > 0 else 0))
        total["bytes"] += case["frames"] * (len(dp) * per + int(np.sum(ds)) * shape)
        total["flops"] += case["frames"] * (len(dp) * 300 * v + int(np.sum(dp)) * (P + 1) * (P + 2) * v / 4)
    return total


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
def exact(case, seed):
    """One iteration of Gauss-Newton in float64.  A pass of several iterations
    has no such value: a pixel between two vertices goes to either within
    rounding, and a weakly seen joint carries that through the iterations
    that follow (1e-6 rad in the starting pose come out as 5e-3), so None."""
    if case["kind"] != "single" or case["frames"] * case["iters"] != 1 or case["schedule"] != "full":
        return None
    rng = np.random.default_rng(seed)
    body = _body(case["shape"], case["verts"], case["width"], case["height"])
    _, images, start = _views(body, rng, min(case["frames"], 4) + 1)
    return _gauss_newton(_model(case, body), body.camera, _params(case, len(start)), start, images[0],
                         case["surface"])


def _qmul(a, b):
    aw, ax, ay, az = a.unbind(-1)
    bw, bx, by, bz = b.unbind(-1)
    return torch.stack([aw * bw - ax * bx - ay * by - az * bz, aw * bx + ax * bw + ay * bz - az * by,
                        aw * by - ax * bz + ay * bw + az * bx, aw * bz + ax * by - ay * bx + az * bw], -1)


def _dqmul(a, b):
    return torch.cat([_qmul(a[..., :4], b[..., :4]),
                      _qmul(a[..., :4], b[..., 4:]) + _qmul(a[..., 4:], b[..., :4])], -1)


def _frames_of(model, theta):
    """Joint frames H_{0,j} as dual quaternions [P, 8]."""
    t64 = dict(dtype=torch.float64, device=theta.device)
    off, axis = torch.tensor(model["joint_offset"], **t64), torch.tensor(model["joint_axis"], **t64)
    q = off[:, :4] / off[:, :4].norm(dim=1, keepdim=True)
    o = torch.cat([q, _qmul(torch.cat([torch.zeros_like(off[:, :1]), 0.5 * off[:, 4:]], 1), q)], 1)
    hinge = torch.tensor(model["joint_type"] == synth.HINGE, device=theta.device)[:, None]
    h = 0.5 * theta[:, None]
    one, none = torch.ones_like(h), torch.zeros_like(axis)
    local = torch.where(hinge, torch.cat([torch.cos(h), torch.sin(h) * axis, 0 * one, none], 1),
                        torch.cat([one, none, 0 * one, h * axis], 1))
    local = _dqmul(o, local)
    out = []
    for j, p in enumerate(model["joint_parent"]):
        out.append(local[j] if p < 0 else _dqmul(out[p], local[j]))
    return torch.stack(out)


def _skin(model, theta, x):
    """Skinned points of the template points x [V, 3] at the pose theta."""
    dev = theta.device
    conj = torch.tensor([1, -1, -1, -1, 1, -1, -1, -1], dtype=torch.float64, device=dev)
    links = torch.tensor(model["link_joint"], device=dev).long()
    rel = _dqmul(_frames_of(model, theta)[links], _frames_of(model, torch.zeros_like(theta))[links] * conj)
    sl = torch.tensor(model["skin_link"], device=dev).long()
    w = torch.tensor(model["skin_w"], dtype=torch.float64, device=dev) * (sl >= 0)
    d = rel[sl.clamp(min=0)]   # [V, K, 8]

    def move(dq, p):
        r, t = dq[..., :4], dq[..., 4:]
        rc = r * conj[:4]
        q = _qmul(_qmul(r, torch.cat([torch.zeros_like(p[..., :1]), p], -1)), rc) + 2 * _qmul(t, rc)
        return q[..., 1:] / (r * r).sum(-1, keepdim=True)

    if model.get("blend", 0) == T.TRACK_BLEND_LINEAR:
        return (w[..., None] * move(d, x[:, None].expand(-1, d.shape[1], -1))).sum(1)
    # signs: the hemisphere of the heaviest influence (of equal ones, the lower link)
    heaviest = w == w.max(1, keepdim=True).values
    pivot = torch.where(heaviest & (sl >= 0), sl, sl.max() + 1).argmin(1)
    ref = d[torch.arange(len(d), device=dev), pivot][:, None, :4]
    sign = torch.where((d[..., :4] * ref).sum(-1) < 0, -1.0, 1.0)
    return move((w * sign)[..., None].mul(d).sum(1), x)


def _normals(v, faces):
    a, b, c = (v[faces[:, k]] for k in range(3))
    n = torch.zeros_like(v)
    cross = torch.linalg.cross(b - a, c - a)
    for k in range(3):
        n.index_add_(0, faces[:, k], cross)
    size = n.norm(dim=1, keepdim=True)
    return torch.where(size > 0, n / size, 0.0)


def _nearest(cam, tau, v, depth):
    """(point, vertex) pairs: each valid pixel's point and its nearest vertex
    in the image, closer than tau."""
    u = torch.floor(cam["fx"] * v[:, 0] / v[:, 2] + cam["cx"] + 0.5)
    w = torch.floor(cam["fy"] * v[:, 1] / v[:, 2] + cam["cy"] + 0.5)
    seen = torch.nonzero((v[:, 2] > 1e-3) & (u >= 0) & (u < cam["width"]) & (w >= 0) & (w < cam["height"]))[:, 0]
    pv, pu = torch.meshgrid(torch.arange(cam["height"], device=v.device), torch.arange(cam["width"], device=v.device),
                            indexing="ij")
    ok = torch.isfinite(depth) & (depth > 0)
    p = torch.stack([(pu - cam["cx"]) * depth / cam["fx"], (pv - cam["cy"]) * depth / cam["fy"], depth], -1)[ok]
    lo, hi = v[seen].min(0).values - tau, v[seen].max(0).values + tau
    n_valid, p = len(p), p[((p >= lo) & (p <= hi)).all(1)]
    best = torch.empty(len(p), dtype=torch.long, device=v.device)
    dist = torch.empty(len(p), dtype=torch.float64, device=v.device)
    for k in range(0, len(p), 2048):
        d2 = sum((p[k:k + 2048, None, c] - v[seen][None, :, c]) ** 2 for c in range(3))
        dist[k:k + 2048], best[k:k + 2048] = d2.min(1)
    keep = dist < tau * tau
    return p[keep], seen[best[keep]], n_valid


def _gauss_newton(model, cam, prm, start, depth, surface):
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    f64 = dict(dtype=torch.float64, device=dev)
    theta = torch.tensor(start, **f64)
    rest = torch.tensor(model["rest_xyz"], **f64)
    faces = torch.tensor(model["faces"], device=dev).long()
    depth = torch.tensor(depth, **f64)
    V, P = len(rest), len(theta)
    v = _skin(model, theta, rest)
    n = _normals(v, faces)
    p, at, n_valid = _nearest({k: float(np.float32(c)) if k[0] in "fc" else c for k, c in cam.items()},
                              float(np.float32(prm["tau"])), v, depth)
    count = torch.zeros(V, **f64).index_add_(0, at, torch.ones(len(at), **f64))
    delta = torch.zeros(V, 3, **f64).index_add_(0, at, p - v[at]) / count.clamp(min=1)[:, None]
    use = (count > 0) & (n.norm(dim=1) > 0)
    r = (n * delta).sum(1) * use
    # the pose step: r falls by n . dv along each joint (central differences in float64)
    J = torch.empty(V, P, **f64)
    for k in range(P):
        h = torch.zeros(P, **f64)
        h[k] = 1e-5
        J[:, k] = -(n * (_skin(model, theta + h, rest) - _skin(model, theta - h, rest))).sum(1) / 2e-5
    J = J * use[:, None]
    A = J.T @ J
    b = J.T @ r
    live = torch.diagonal(A) > 0
    M = A + float(np.float32(prm["lambda_k"])) * torch.diag(torch.diagonal(A))
    M = torch.where(live[:, None] & live[None, :], M, torch.eye(P, **f64))
    theta = theta - torch.linalg.solve(M, torch.where(live, b, 0.0))
    # the offset step at the new pose, from zero offsets (so the neighbour and
    # temporal terms only add to the diagonal)
    vn = _skin(model, theta, rest)
    nn = _normals(vn, faces)
    lam = {k: float(np.float32(prm[k])) for k in ("lambda_phi", "lambda_nbr", "lambda_t", "lambda_w")}
    use = (count > 0) & (nn.norm(dim=1) > 0)
    r = (nn * (delta + v - vn)).sum(1) * use
    U = torch.empty(V, 3, **f64)
    for k in range(3):   # dv/dx is exact: skinning is affine in the template point
        e = torch.zeros(3, **f64)
        e[k] = 1.0
        U[:, k] = -(nn * (_skin(model, theta, rest + e) - vn)).sum(1) * use
    nbr = torch.tensor((np.asarray(model["neighbors"]) >= 0).sum(1), **f64)
    alpha = lam["lambda_phi"] + lam["lambda_t"] + lam["lambda_nbr"] * nbr
    S = U[:, :, None] * U[:, None, :] + alpha[:, None, None] * torch.eye(3, **f64)
    S = S + lam["lambda_w"] * torch.diag_embed(torch.diagonal(S, dim1=1, dim2=2))
    phi = -torch.linalg.solve(S, U * r[:, None])
    energy = float(((n * delta).sum(1) * ((count > 0) & (n.norm(dim=1) > 0))).square().sum())
    return dict(theta=theta.cpu().numpy(), phi=phi.cpu().numpy(),
                verts=_skin(model, theta, rest + phi).cpu().numpy() if surface else None,
                counts=np.array([0, n_valid, len(at), int((count > 0).sum())]),
                energy=np.array([energy, energy]))
