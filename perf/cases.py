"""Performance cases: the work a program has this library do, one pass each.

Every case goes through a public entry point of the package with inputs made
from a seed: a serial arm (capsule and box links), smooth joint-space paths,
and obstacle clouds (a voxelised person and table, a uniform cube, or points
packed against the arm).  ``listed()`` names the cases, ``draw()`` gives more
of the same ranges, ``exact()`` the outputs in double precision.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2309_12543_amd import learned, lsdf

DEV = "cuda"
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
PAD = 0.05          # metres a link's grid box extends beyond its mesh
FAR = 1.0           # metres a network's domain extends beyond the grid box
MARGIN = 0.05       # learned estimates below this take the grid's value
HIDDEN = 128
FRNN_HIDDEN = 32


def listed():
    return [
        # one control tick on a small cloud, the arguments marshalled once:
        # latency and launches are what it costs
        {"name": "tick", "kind": "tick", "C": 50, "M": 2000, "n": 32, "joints": 6, "dtype": "f32", "cloud": "cube"},
        # a planned path of 500 waypoints against one depth-camera cloud (2 cm
        # voxels), kinematics included: the headline workload
        {"name": "path", "kind": "step", "C": 500, "M": 20000, "n": 64, "joints": 6, "dtype": "f32", "cloud": "scene"},
        # a fine map: 1 cm voxels, 128^3 grids in 16-bit storage, every link's
        # minimum returned
        {"name": "fine_map", "kind": "query", "C": 500, "M": 100000, "n": 128, "joints": 6, "dtype": "bf16",
         "cloud": "scene"},
        # an obstacle pressed against the arm, at ragged sizes: every point
        # lies in some link's box along the path
        {"name": "contact", "kind": "step", "C": 333, "M": 12345, "n": 64, "joints": 6, "dtype": "f32",
         "cloud": "contact"},
        # 64 re-planned paths, each with its own cloud, ragged, in one call
        {"name": "replan_batch", "kind": "batch", "K": 64, "Cmin": 50, "Cmax": 1000, "Mmin": 5000, "Mmax": 200000,
         "n": 64, "joints": 6, "dtype": "f32", "cloud": "scene"},
        # the learned distance beyond the grids' reach, on the fine cloud
        {"name": "learned_path", "kind": "learned", "C": 500, "M": 100000, "n": 64, "joints": 6, "dtype": "f32",
         "cloud": "scene"},
        # one optimiser step of every link's network at the recipe's batch
        {"name": "train_step", "kind": "train", "B": 8192, "N": 131072, "joints": 6},
        # training labels of every link's samples
        {"name": "labels", "kind": "labels", "N": 262144, "n": 64, "joints": 6, "nseg": 16, "dtype": "f32"},
        # a new robot: every link's distance grid from its mesh
        {"name": "link_grids", "kind": "grids", "n": 64, "joints": 6, "nseg": 16, "dtype": "f32"},
        # the aligned pipeline: whole-environment grids of a path prepared,
        # then a cloud looked up in them
        {"name": "robot_sdf", "kind": "robot_sdf", "C": 200, "M": 20000, "n": 64, "env": 128, "voxel": 0.03125,
         "joints": 6, "dtype": "f32", "cloud": "scene"},
        # one optimiser step of the grid-transformation network (44^3 voxels)
        {"name": "transform_train", "kind": "frnn_train", "m": 22, "B": 64},
        # the same preparation through the grid-transformation network
        {"name": "transform_build", "kind": "frnn_build", "C": 40, "n": 64, "env": 128, "voxel": 0.03125, "joints": 6,
         "dtype": "f32"},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["tick", "step", "query", "batch", "learned", "train", "labels", "grids", "robot_sdf",
                       "frnn_train", "frnn_build"])
    robot = {"kind": kind, "joints": rng.choice([4, 5, 6, 6, 7])}
    dtype = rng.choice(["f32", "f32", "bf16", "f16"])
    cloud = rng.choice(["scene", "scene", "cube", "contact"])
    if kind == "tick":
        return {**robot, "C": log_int(1, 200), "M": log_int(100, 8000), "n": rng.randint(16, 64), "dtype": dtype,
                "cloud": cloud}
    if kind in ("step", "query"):
        return {**robot, "C": log_int(100, 1000), "M": log_int(3000, 100000) if cloud != "contact" else
                log_int(1000, 20000), "n": rng.randint(32, 128), "dtype": dtype, "cloud": cloud}
    if kind == "batch":
        return {**robot, "K": log_int(2, 48), "Cmin": 50, "Cmax": log_int(100, 1000), "Mmin": 1000,
                "Mmax": log_int(5000, 150000), "n": rng.randint(32, 64), "dtype": dtype, "cloud": "scene"}
    if kind == "learned":
        return {**robot, "C": log_int(20, 400), "M": log_int(3000, 80000), "n": rng.randint(32, 64), "dtype": "f32",
                "cloud": rng.choice(["scene", "cube"])}
    if kind == "train":
        return {**robot, "B": 512 * log_int(2, 16), "N": log_int(20000, 131072)}
    if kind == "labels":
        return {**robot, "N": log_int(5000, 200000), "n": rng.randint(32, 64), "nseg": rng.choice([8, 12, 16, 20]),
                "dtype": "f32"}
    if kind == "grids":
        return {**robot, "n": rng.randint(24, 64), "nseg": rng.choice([8, 12, 16, 20]), "dtype": dtype}
    if kind == "robot_sdf":
        return {**robot, "C": log_int(20, 160), "M": log_int(2000, 60000), "n": rng.randint(32, 64),
                "env": rng.randint(60, 128), "voxel": 0.03125, "dtype": dtype, "cloud": "scene"}
    if kind == "frnn_train":
        return {"kind": kind, "m": rng.randint(6, 22), "B": rng.choice([1, 7, 16, 33, 64, 64])}
    return {**robot, "C": log_int(4, 32), "n": rng.randint(32, 64), "env": rng.randint(60, 128),
            "voxel": rng.choice([0.03125, 0.04, 0.05]), "dtype": dtype}


# ---------------------------------------------------------------------------
# the arm
# ---------------------------------------------------------------------------

class Mesh:
    def __init__(self, verts, tris, comp_first):
        self.verts, self.tris, self.comp_first = verts, tris, comp_first


def dh_table(joints):
    """Standard DH rows (a, alpha, d, theta_offset) of an arm with 4 to 7 joints."""
    alpha = [math.pi / 2, 0.0, math.pi / 2, -math.pi / 2, math.pi / 2, 0.0, -math.pi / 2]
    a = [0.0, 0.35, 0.27, 0.0, 0.0, 0.0, 0.0]
    d = [0.33, 0.0, 0.0, 0.31, 0.0, 0.17, 0.12]
    return np.array([[a[k], alpha[k], d[k], 0.0] for k in range(joints)], dtype=np.float32).astype(np.float64)


def link_parts(joints):
    """Per link, its parts: ("capsule", p0, p1, r) or ("box", centre, half)."""
    links = [[("box", (0.0, 0.0, -0.05), (0.15, 0.15, 0.05)), ("capsule", (0.0, 0.0, 0.0), (0.0, 0.0, 0.12), 0.09)]]
    for k, (a, alpha, d, _) in enumerate(dh_table(joints)):
        r = 0.05 + 0.01 * (k % 3)
        prev = np.array([-a, -d * math.sin(alpha), -d * math.cos(alpha)])
        if np.linalg.norm(prev) > 1e-6:
            parts = [("capsule", tuple(prev), (0.0, 0.0, 0.0), r)]
        else:
            parts = [("capsule", (-1.2 * r, 0.0, 0.0), (1.2 * r, 0.0, 0.0), r)]
        parts.append(("capsule", (0.0, 0.0, -1.2 * r), (0.0, 0.0, 1.2 * r), 1.15 * r))
        if k % 2 == 1:
            parts.append(("box", tuple(prev), (0.9 * r,) * 3))
        links.append(parts)
    return links


def _outward(verts, tris):
    a, b, c = (verts[tris[:, k]] for k in range(3))
    return tris if np.einsum("ij,ij->", a - verts.mean(0), np.cross(b - a, c - a)) > 0 else tris[:, [0, 2, 1]]


def capsule_mesh(p0, p1, r, nseg):
    """Closed latitude-longitude mesh of a capsule: nseg meridians, nseg / 4 rings a cap."""
    p0, p1 = np.asarray(p0, float), np.asarray(p1, float)
    w = (p1 - p0) / np.linalg.norm(p1 - p0)
    u = np.cross(w, [1.0, 0.0, 0.0] if abs(w[0]) < 0.9 else [0.0, 1.0, 0.0])
    u /= np.linalg.norm(u)
    v = np.cross(w, u)
    nring = max(2, nseg // 4)
    th = 2 * math.pi * np.arange(nseg) / nseg
    round_ = np.cos(th)[:, None] * u + np.sin(th)[:, None] * v
    lat = [(p0, -math.pi / 2 * (1 - k / nring)) for k in range(1, nring + 1)]
    lat += [(p1, math.pi / 2 * k / nring) for k in range(nring)]
    rings = [c + r * (math.cos(phi) * round_ + math.sin(phi) * w) for c, phi in lat]
    verts = np.concatenate([[p0 - r * w], *rings, [p1 + r * w]])
    tris, s = [], np.arange(nseg)
    s1 = (s + 1) % nseg
    tris.append(np.stack([0 * s, 1 + s1, 1 + s], 1))
    for j in range(len(rings) - 1):
        lo, hi = 1 + j * nseg, 1 + (j + 1) * nseg
        tris += [np.stack([lo + s, lo + s1, hi + s1], 1), np.stack([lo + s, hi + s1, hi + s], 1)]
    top = 1 + (len(rings) - 1) * nseg
    tris.append(np.stack([0 * s + len(verts) - 1, top + s, top + s1], 1))
    tris = np.concatenate(tris)
    return verts, _outward(verts, tris)


def box_mesh(c, h):
    verts = np.array([[c[0] + x * h[0], c[1] + y * h[1], c[2] + z * h[2]]
                      for z in (-1, 1) for y in (-1, 1) for x in (-1, 1)])
    quads = [(0, 2, 3, 1), (4, 5, 7, 6), (0, 1, 5, 4), (2, 6, 7, 3), (0, 4, 6, 2), (1, 3, 7, 5)]
    tris = np.array([t for a, b, cc, d in quads for t in ((a, b, cc), (a, cc, d))])
    return verts, _outward(verts, tris)


def link_meshes(joints, nseg=16):
    meshes = []
    for parts in link_parts(joints):
        verts, tris, first, n = [], [], [0], 0
        for p in parts:
            v, t = capsule_mesh(p[1], p[2], p[3], nseg) if p[0] == "capsule" else box_mesh(p[1], p[2])
            verts.append(v)
            tris.append(t + n)
            n += len(v)
            first.append(first[-1] + len(t))
        meshes.append(Mesh(np.concatenate(verts).astype(np.float32).astype(np.float64),
                           np.concatenate(tris).astype(np.int32), np.array(first, dtype=np.int32)))
    return meshes


def link_boxes(joints):
    """Grid boxes (lo, hi), float32 [L][3]: the meshes' bounding boxes grown by PAD."""
    ms = link_meshes(joints)
    return (np.array([m.verts.min(0) - PAD for m in ms], dtype=np.float32),
            np.array([m.verts.max(0) + PAD for m in ms], dtype=np.float32))


def parts_distance(parts, p):
    """Signed distance (float64) of points p [...][3] to a union of parts."""
    best = None
    for part in parts:
        if part[0] == "capsule":
            a, b = (torch.tensor(x, dtype=torch.float64, device=p.device) for x in part[1:3])
            t = (((p - a) * (b - a)).sum(-1) / ((b - a) ** 2).sum()).clamp(0.0, 1.0)
            d = (p - (a + t[..., None] * (b - a))).norm(dim=-1) - part[3]
        else:
            c, h = (torch.tensor(x, dtype=torch.float64, device=p.device) for x in part[1:3])
            q = (p - c).abs() - h
            d = q.clamp(min=0.0).norm(dim=-1) + q.amax(-1).clamp(max=0.0)
        best = d if best is None else torch.minimum(best, d)
    return best


def node_positions(lo, hi, n):
    """Nodes [n^3][3] (x fastest) of a grid, float64."""
    ax = [torch.linspace(float(lo[a]), float(hi[a]), n, dtype=torch.float64, device=DEV) for a in range(3)]
    z, y, x = torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    return torch.stack([x, y, z], -1).reshape(-1, 3)


def link_grids(joints, n, dtype):
    """The links' distance grids from the parts' closed forms (as loaded from a file)."""
    lo, hi = link_boxes(joints)
    gs = lsdf.GridSet(lo, hi, np.full((joints + 1, 3), n), device=DEV, dtype=DTYPES[dtype])
    for i, parts in enumerate(link_parts(joints)):
        d = parts_distance(parts, node_positions(lo[i], hi[i], n)).float()
        gs.grid(i).copy_(d.view(n, n, n).to(DTYPES[dtype]))
    return gs


def path(rng, C, joints):
    """Joint angles float32 [C][joints]: smooth through four random configurations."""
    knots = rng.uniform(-2.96, 2.96, size=(4, joints))
    t = np.linspace(0.0, 3.0, C) if C > 1 else np.zeros(1)
    k = np.minimum(t.astype(int), 2)
    s = 0.5 - 0.5 * np.cos(math.pi * (t - k))
    q = knots[k] * (1 - s)[:, None] + knots[k + 1] * s[:, None]
    return torch.as_tensor(q.astype(np.float32), device=DEV)


def poses(joints, q):
    """Link poses float64 [C][joints + 1][3][4] of float joint angles."""
    q = q.double()
    T = torch.eye(4, dtype=torch.float64, device=q.device).repeat(q.shape[0], 1, 1)
    out = [T[:, :3]]
    for k, (a, alpha, d, off) in enumerate(dh_table(joints)):
        ct, st = torch.cos(q[:, k] + off), torch.sin(q[:, k] + off)
        ca, sa = math.cos(alpha), math.sin(alpha)
        A = torch.zeros((q.shape[0], 4, 4), dtype=torch.float64, device=q.device)
        A[:, 0, 0], A[:, 0, 1], A[:, 0, 2], A[:, 0, 3] = ct, -st * ca, st * sa, a * ct
        A[:, 1, 0], A[:, 1, 1], A[:, 1, 2], A[:, 1, 3] = st, ct * ca, -ct * sa, a * st
        A[:, 2, 1], A[:, 2, 2], A[:, 2, 3], A[:, 3, 3] = sa, ca, d, 1.0
        T = (T[:, :, :, None] * A[:, None, :, :]).sum(2)
        out.append(T[:, :3])
    return torch.stack(out, 1).contiguous()


# ---------------------------------------------------------------------------
# clouds
# ---------------------------------------------------------------------------

def scene_cloud(rng, M):
    """M points of a voxelised person beside the arm and a table, in raster
    order: voxel centres, subsampled, or topped up with jittered repeats."""
    az, dist = rng.uniform(-math.pi, math.pi), rng.uniform(0.3, 1.5)
    t = np.array([dist * math.cos(az), dist * math.sin(az), -0.75])
    yaw = rng.uniform(-math.pi, math.pi)
    side = np.array([-math.sin(yaw), math.cos(yaw), 0.0])
    body = [((0, 0, 1.58), (0.09, 0.10, 0.12)), ((0, 0, 1.18), (0.14, 0.16, 0.28))]
    for s in (-1, 1):
        lean = rng.normal(0.0, 0.05, size=2)
        body += [(s * 0.25 * side + [lean[0], 0, 1.25], (0.05, 0.05, 0.16)),
                 (s * 0.27 * side + [lean[0] + 0.05, lean[1], 0.98], (0.04, 0.04, 0.14)),
                 (s * 0.09 * side + [0, lean[1], 0.68], (0.08, 0.08, 0.22)),
                 (s * 0.09 * side + [lean[1], 0, 0.25], (0.06, 0.06, 0.21))]
    taz = rng.uniform(-math.pi, math.pi)
    c, s = math.cos(taz), math.sin(taz)
    lo = np.minimum(t - [0.6, 0.6, 0.0], [0.6 * c - 0.75, 0.6 * s - 0.75, -0.75])
    hi = np.maximum(t + [0.6, 0.6, 1.75], [0.6 * c + 0.75, 0.6 * s + 0.75, 0.0])
    for voxel in (0.04, 0.02, 0.01):
        ax = [(torch.arange(math.floor(lo[a] / voxel), math.ceil(hi[a] / voxel), device=DEV) + 0.5) * voxel
              for a in range(3)]
        z, y, x = torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
        occ = torch.zeros_like(x, dtype=torch.bool)
        for centre, semi in body:
            e = np.asarray(centre, float) + t
            occ |= ((x - e[0]) / semi[0]) ** 2 + ((y - e[1]) / semi[1]) ** 2 + ((z - e[2]) / semi[2]) ** 2 <= 1.0
        u, v = (x - 0.6 * c) * c + (y - 0.6 * s) * s, -(x - 0.6 * c) * s + (y - 0.6 * s) * c
        occ |= (u.abs() <= 0.4) & (v.abs() <= 0.6) & (z > -max(voxel, 0.02)) & (z < 0.0)
        at = occ.reshape(-1).nonzero()[:, 0]
        if len(at) >= M:
            break
    V = len(at)
    if V >= M:
        keep = torch.as_tensor(np.sort(rng.choice(V, size=M, replace=False)), device=DEV)
        jitter = 0.0
    else:
        extra = np.sort(np.concatenate([np.arange(V), rng.integers(0, V, size=M - V)]))
        jitter = rng.uniform(-0.5, 0.5, size=(M, 3)) * np.concatenate([[False], extra[1:] == extra[:-1]])[:, None]
        keep, jitter = torch.as_tensor(extra, device=DEV), torch.as_tensor(jitter * voxel, device=DEV)
    pts = torch.stack([a.reshape(-1)[at[keep]] for a in (x, y, z)], 1).double() + jitter
    return pts.float().contiguous()


def contact_cloud(rng, M, joints, q):
    """M points, each uniform in a random link's box at a random waypoint."""
    lo, hi = link_boxes(joints)
    T = poses(joints, q).cpu().numpy()
    c, i = rng.integers(0, len(T), M), rng.integers(0, joints + 1, M)
    local = rng.uniform(lo[i], hi[i])
    pts = (T[c, i, :, :3] * local[:, None, :]).sum(-1) + T[c, i, :, 3]
    return torch.as_tensor(pts.astype(np.float32), device=DEV)


def cloud(rng, case, M, q):
    if case["cloud"] == "cube":
        return torch.as_tensor(rng.uniform(-1.0, 1.0, size=(M, 3)).astype(np.float32), device=DEV)
    return contact_cloud(rng, M, case["joints"], q) if case["cloud"] == "contact" else scene_cloud(rng, M)


# ---------------------------------------------------------------------------
# the networks' inputs
# ---------------------------------------------------------------------------

def mlp_domains(joints):
    """(centre, half, core_half) float32 [L][3] of the links' networks."""
    lo, hi = (b.astype(np.float64) for b in link_boxes(joints))
    return (((lo + hi) / 2).astype(np.float32), ((hi - lo) / 2 + FAR).astype(np.float32),
            ((hi - lo) / 2 - PAD).astype(np.float32))


def mlp_init(rng, L):
    parts = [rng.uniform(-1, 1, size=(L, o * i + o)) / math.sqrt(i) for i, o in ((3, HIDDEN), (HIDDEN, HIDDEN),
                                                                                   (HIDDEN, HIDDEN), (HIDDEN, 1))]
    return torch.as_tensor(np.concatenate(parts, 1).astype(np.float32), device=DEV)


def mlp_split(p):
    """W1, b1, W2, b2, W3, b3, w4, b4 of one link's parameters."""
    out, k = [], 0
    for shape in ((HIDDEN, 3), (HIDDEN,), (HIDDEN, HIDDEN), (HIDDEN,), (HIDDEN, HIDDEN), (HIDDEN,), (HIDDEN,), (1,)):
        n = math.prod(shape)
        out.append(p[k:k + n].view(shape))
        k += n
    return out


def _rounded(x):
    """x rounded to bfloat16, as the networks' weights and activations are used; gradients pass."""
    return x + (x.detach().float().bfloat16().to(x.dtype) - x.detach())


def mlp_hidden(p, xh):
    W1, b1, W2, b2, W3, b3, _, _ = mlp_split(p)
    h = _rounded(torch.nn.functional.silu(xh @ _rounded(W1).T + b1))
    h = _rounded(torch.nn.functional.silu(h @ _rounded(W2).T + b2))
    return _rounded(torch.nn.functional.silu(h @ _rounded(W3).T + b3))


def core_distance(u, core):
    return (u.abs() - torch.as_tensor(core, device=u.device).double()).clamp(min=0.0).norm(dim=-1)


def link_samples(rng, i, joints, N):
    """Link-frame training positions: most in the shell around the link, the rest over the domain."""
    cen, half, core = (a[i].astype(np.float64) for a in mlp_domains(joints))
    near = cen + rng.uniform(-1, 1, size=(N, 3)) * (core + rng.choice([0.03, 0.15, 0.5], size=(N, 1)))
    wide = cen + rng.uniform(-1, 1, size=(N, 3)) * half
    return torch.as_tensor(np.where(rng.uniform(size=(N, 1)) < 0.85, near, wide).astype(np.float32), device=DEV)


def fitted_networks(rng, joints):
    """Networks whose output layer is fitted to the links' remainders over
    the core boxes, and their remainder bounds (whole centimetres)."""
    params, bound = mlp_init(rng, joints + 1), []
    cen, half, core = mlp_domains(joints)
    for i, parts in enumerate(link_parts(joints)):
        x = link_samples(rng, i, joints, 16384).double()
        u = x - torch.as_tensor(cen[i], device=DEV).double()
        rest = parts_distance(parts, x) - core_distance(u, core[i])
        h = mlp_hidden(params[i].double(), u / torch.as_tensor(half[i], device=DEV).double())
        h = torch.cat([h, torch.ones_like(h[:, :1])], 1)
        A = h.T @ h + 1e-2 * torch.eye(HIDDEN + 1, dtype=torch.float64, device=DEV)
        params[i, -(HIDDEN + 1):] = torch.linalg.solve(A, h.T @ rest).float()
        bound.append(math.ceil(125.0 * float(rest.abs().max())) / 100.0)
    return params, np.array(bound, dtype=np.float32)


def frnn_split(p):
    H = FRNN_HIDDEN
    O = (len(p) - 10 * H) // (H + 1)
    return p[:9 * H].view(H, 9), p[9 * H:10 * H], p[10 * H:10 * H + O * H].view(O, H), p[10 * H + O * H:]


def block_centres(m, dtype=torch.float64):
    """Normalised voxel centres [(2m)^3][3] of a block, x fastest."""
    a = (torch.arange(2 * m, dtype=dtype, device=DEV) + 0.5) / m - 1.0
    z, y, x = torch.meshgrid(a, a, a, indexing="ij")
    return torch.stack([x, y, z], -1).reshape(-1, 3)


def frnn_params(rng, m, noise):
    """A network near R^T P: +-R on 18 hidden units, the outputs that combine them, plus noise."""
    p = torch.zeros(lsdf.frnn_nparam(m), device=DEV)
    W1, _, W2, _ = frnn_split(p)
    P = block_centres(m).float()
    for e in range(9):
        W1[2 * e, e], W1[2 * e + 1, e] = 1.0, -1.0
        W2.view(-1, 3, FRNN_HIDDEN)[:, e % 3, 2 * e] = P[:, e // 3]
        W2.view(-1, 3, FRNN_HIDDEN)[:, e % 3, 2 * e + 1] = -P[:, e // 3]
    gen = torch.Generator(device=DEV).manual_seed(int(rng.integers(1 << 31)))
    return p + noise * torch.randn(len(p), generator=gen, device=DEV)


def rotations(rng, B):
    w = rng.normal(size=(B, 4))
    a, b, c, d = (w / np.linalg.norm(w, axis=1, keepdims=True)).T
    R = np.stack([1 - 2 * (c * c + d * d), 2 * (b * c - a * d), 2 * (b * d + a * c), 2 * (b * c + a * d),
                  1 - 2 * (b * b + d * d), 2 * (c * d - a * b), 2 * (b * d - a * c), 2 * (c * d + a * b),
                  1 - 2 * (b * b + c * c)], 1)
    return torch.as_tensor(R.astype(np.float32), device=DEV)


def moments(rng, like, scale):
    """Adam moments of a run under way: gradients of about `scale` so far."""
    gen = torch.Generator(device=DEV).manual_seed(int(rng.integers(1 << 31)))
    m = scale * torch.randn(like.shape, generator=gen, device=DEV)
    v = scale ** 2 * (0.5 + torch.rand(like.shape, generator=gen, device=DEV))
    return m, v


def block_half_width(case):
    """Smallest block half-width (voxels) that holds every link's box."""
    lo, hi = (b.astype(np.float64) for b in link_boxes(case["joints"]))
    far = np.sqrt((np.maximum(np.abs(lo), np.abs(hi)) ** 2).sum(1)).max()
    return int(math.ceil(far / float(np.float32(case["voxel"])))) + 2


def environment(case):
    return lsdf.make_env([-0.5 * case["env"] * case["voxel"]] * 3, case["voxel"], [case["env"]] * 3)


# ---------------------------------------------------------------------------
# the interface
# ---------------------------------------------------------------------------

def prepare(case, seed):
    rng = np.random.default_rng(seed)
    kind, s = case["kind"], {"case": case}
    joints = case.get("joints", 6)
    if kind in ("tick", "step", "query", "learned", "robot_sdf"):
        s["grids"] = link_grids(joints, case["n"], case["dtype"])
        s["q"] = path(rng, case["C"], joints)
        s["points"] = cloud(rng, case, case["M"], s["q"])
        s["dh"] = dh_table(joints)
        if kind == "tick":
            s["call"] = lsdf.PreparedQueryFromJoints(s["dh"], s["q"], s["grids"], s["points"])
        elif kind != "step":
            s["T"] = poses(joints, s["q"]).float().contiguous()
        if kind == "learned":
            s["params"], bound = fitted_networks(rng, joints)
            s["bound"], s["domains"] = bound, lsdf.make_domains(*mlp_domains(joints), bound)
        if kind == "robot_sdf":
            s["env"] = environment(case)
            s["out"] = torch.empty([case["C"]] + [case["env"]] * 3, device=DEV)
    elif kind == "batch":
        s["grids"] = link_grids(joints, case["n"], case["dtype"])
        sizes = np.random.default_rng(case["K"])   # the case's, whatever the seed
        Cs = sizes.integers(case["Cmin"], case["Cmax"] + 1, size=case["K"])
        Ms = sizes.integers(case["Mmin"], case["Mmax"] + 1, size=case["K"])
        s["q"] = torch.cat([path(rng, int(C), joints) for C in Cs])
        s["T"] = poses(joints, s["q"]).float().contiguous()
        s["points"] = torch.cat([scene_cloud(rng, int(M)) for M in Ms])
        s["c_off"] = torch.as_tensor(np.concatenate([[0], np.cumsum(Cs)]).astype(np.int32), device=DEV)
        s["m_off"] = torch.as_tensor(np.concatenate([[0], np.cumsum(Ms)]).astype(np.int64), device=DEV)
    elif kind == "train":
        L = joints + 1
        s["domains"] = lsdf.make_domains(*mlp_domains(joints), 0.15)
        s["params"] = mlp_init(rng, L)
        s["m"], s["v"] = moments(rng, s["params"], 1e-3)
        s["samples"] = torch.stack([link_samples(rng, i, joints, case["N"]) for i in range(L)])
        s["labels"] = torch.stack([parts_distance(parts, s["samples"][i].double()).float()
                                   for i, parts in enumerate(link_parts(joints))])
        s["index"] = torch.as_tensor(rng.integers(0, case["N"], size=(L, case["B"])).astype(np.int32), device=DEV)
        s["ws"] = torch.empty(lsdf.mlp_train_workspace_size(L, case["B"]), dtype=torch.uint8, device=DEV)
        s["loss"], s["grad"] = torch.empty(L, device=DEV), torch.empty_like(s["params"])
    elif kind == "labels":
        s["grids"] = link_grids(joints, case["n"], case["dtype"])
        s["meshes"] = link_meshes(joints, case["nseg"])
        s["samples"] = torch.stack([link_samples(rng, i, joints, case["N"]) for i in range(joints + 1)])
    elif kind == "grids":
        # another seed is another robot: its meshes scaled a little
        s["meshes"] = link_meshes(joints, case["nseg"])
        for m in s["meshes"]:
            m.verts = (m.verts * rng.uniform(0.9, 1.1, size=3)).astype(np.float32).astype(np.float64)
        s["lo"] = np.array([m.verts.min(0) - PAD for m in s["meshes"]], dtype=np.float32)
        s["hi"] = np.array([m.verts.max(0) + PAD for m in s["meshes"]], dtype=np.float32)
    elif kind == "frnn_train":
        s["params"] = frnn_params(rng, case["m"], 0.01)
        s["R"] = rotations(rng, case["B"])
        s["m"], s["v"] = moments(rng, s["params"], 0.25 / (math.sqrt(case["B"]) * 24 * case["m"] ** 3))
        s["loss"], s["grad"] = torch.empty(1, device=DEV), torch.empty_like(s["params"])
    elif kind == "frnn_build":
        s["grids"] = link_grids(joints, case["n"], case["dtype"])
        s["T"] = poses(joints, path(rng, case["C"], joints)).float().contiguous()
        s["env"], s["half"] = environment(case), block_half_width(case)
        s["params"] = frnn_params(rng, s["half"], 2e-5)
        s["out"] = torch.empty([case["C"]] + [case["env"]] * 3, device=DEV)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "tick":
        s["call"]()
        return s["call"].dist, s["call"].link
    if kind == "step":
        return lsdf.query_from_joints(s["dh"], s["q"], s["grids"], s["points"])
    if kind == "query":
        return lsdf.query_min_distance(s["T"], s["grids"], s["points"], link_dist=True)
    if kind == "batch":
        return lsdf.query_min_distance_batched(s["T"], s["grids"], s["points"], s["c_off"], s["m_off"])
    if kind == "learned":
        return lsdf.query_min_distance_mlp(s["T"], s["grids"], s["params"], s["domains"], s["points"], margin=MARGIN,
                                           link_dist=True)
    if kind == "train":
        lsdf.mlp_train_step(s["params"], s["m"], s["v"], 1000, 1e-3, s["domains"], s["samples"], s["labels"],
                            case["B"], s["index"], loss=s["loss"], grad=s["grad"], workspace=s["ws"])
        return s["params"], s["m"], s["v"], s["loss"], s["grad"]
    if kind == "labels":
        return learned.labels_for_samples(s["meshes"], s["grids"], s["samples"])
    if kind == "grids":
        return lsdf.build_robot_grids(s["meshes"], s["lo"], s["hi"], np.full((len(s["meshes"]), 3), case["n"]),
                                      device=DEV, dtype=DTYPES[case["dtype"]]).buf
    if kind == "robot_sdf":
        lsdf.robot_sdf_build(s["T"], s["grids"], s["env"], out=s["out"])
        return s["out"], lsdf.robot_sdf_query(s["out"], s["env"], s["points"])
    if kind == "frnn_train":
        lsdf.frnn_train_step(s["params"], case["m"], s["R"], adam=(s["m"], s["v"]), t=1000, lr=1e-4, grad=s["grad"],
                             loss=s["loss"])
        return s["params"], s["m"], s["v"], s["loss"], s["grad"]
    return lsdf.robot_sdf_build_frnn(s["T"], s["grids"], s["env"], s["params"], s["half"], out=s["out"])


def work(case):
    """What one pass cannot do without: inputs read and outputs written once;
    the arithmetic of the method where it is fixed, and for a clearance one
    bound test (24 operations) per link, waypoint and run of 32 points."""
    kind, L = case["kind"], case.get("joints", 6) + 1
    cell = 4 if case.get("dtype", "f32") == "f32" else 2
    grid = L * case.get("n", 0) ** 3 * cell
    if kind in ("tick", "step", "query"):
        C, M = case["C"], case["M"]
        return {"bytes": grid + 12 * M + C * (48 * L + 8), "flops": 24.0 * C * L * M / 32}
    if kind == "batch":
        C, M = 0.5 * (case["Cmin"] + case["Cmax"]), 0.5 * (case["Mmin"] + case["Mmax"])
        return {"bytes": grid + case["K"] * (12 * M + C * (48 * L + 8)), "flops": 24.0 * case["K"] * C * L * M / 32}
    if kind == "learned":
        # the network on the pairs of about 1 in 30 tiles
        C, M = case["C"], case["M"]
        return {"bytes": grid + 12 * M + C * L * 52 + L * 134660, "flops": C * L * M * (24 / 32 + 2 * 33000 / 30)}
    if kind == "train":
        return {"bytes": L * (134660 * 7 + case["B"] * 20), "flops": 6.0 * 33300 * L * case["B"]}
    if kind == "labels":
        # a mesh has about 2.1 nseg^2 triangles; the nearest one and the sign take at least one test of 40 a point
        return {"bytes": grid + L * case["N"] * 16, "flops": 40.0 * L * case["N"]}
    if kind == "grids":
        return {"bytes": grid, "flops": 40.0 * L * case["n"] ** 3}
    if kind == "robot_sdf":
        return {"bytes": grid + case["C"] * (4 * case["env"] ** 3 + 48 * L) + 12 * case["M"],
                "flops": 6.0 * case["C"] * case["env"] ** 3}
    O = 24 * (case["m"] if kind == "frnn_train" else block_half_width(case)) ** 3
    if kind == "frnn_train":
        # parameters, moments read and written, the gradient written
        return {"bytes": 4.0 * 33 * O * 7, "flops": 6.0 * 32 * O * case["B"]}
    return {"bytes": grid + 4.0 * 33 * O + case["C"] * (4 * case["env"] ** 3 + 48 * L),
            "flops": 2.0 * 32 * O * case["C"] * L}


# ---------------------------------------------------------------------------
# the outputs in double precision
# ---------------------------------------------------------------------------

def interpolate(gs, i, local):
    """Trilinear values (float64) of link i's grid at link-frame points in its box."""
    g, n = gs.grid(i).double(), gs.n[i]
    lo, hi = (torch.as_tensor(b[i].astype(np.float64), device=DEV) for b in (gs.lo, gs.hi))
    size = torch.as_tensor(n.astype(np.float64), device=DEV)
    u = (local - lo) / (hi - lo) * (size - 1)
    k = torch.minimum(u.floor().clamp(min=0), size - 2).long()
    f = u - k
    v = 0.0
    for dz in (0, 1):
        for dy in (0, 1):
            for dx in (0, 1):
                w = 1.0
                for a, d in enumerate((dx, dy, dz)):
                    w = w * (f[:, a] if d else 1 - f[:, a])
                v = v + w * g[k[:, 2] + dz, k[:, 1] + dy, k[:, 0] + dx]
    return v


def local_points(T, x):
    """Points x [M][3] in the frames of poses T [C][3][4]: [C][M][3]."""
    return torch.matmul(x - T[:, None, :, 3], T[:, :, :3])


def link_minima(gs, T, x):
    """Per-link minima float64 [C][L] over points x; +inf where no point lies in the box."""
    C, L = T.shape[:2]
    out = torch.full((C, L), math.inf, dtype=torch.float64, device=DEV)
    step = max(1, 12_000_000 // max(1, len(x)))
    for i in range(L):
        lo, hi = (torch.as_tensor(b[i].astype(np.float64), device=DEV) for b in (gs.lo, gs.hi))
        for c0 in range(0, C, step):
            l = local_points(T[c0:c0 + step, i], x)
            at = ((l >= lo) & (l <= hi)).all(-1).nonzero()
            if len(at):
                out[:, i].scatter_reduce_(0, at[:, 0] + c0, interpolate(gs, i, l[at[:, 0], at[:, 1]]), "amin")
    return out


def learned_minima(s):
    """Per-link minima of the learned clearance, the pairs that cannot hold one left out."""
    joints = s["case"]["joints"]
    T, x, gs = s["T"].double(), s["points"].double(), s["grids"]
    cen, half, core = mlp_domains(joints)
    out = torch.full((len(T), joints + 1), math.inf, dtype=torch.float64, device=DEV)
    step = max(1, 4_000_000 // len(x))
    for i in range(joints + 1):
        p, B = s["params"][i].double(), float(s["bound"][i])
        w4, b4 = _rounded(mlp_split(p)[6]), mlp_split(p)[7]
        ce, ha = (torch.as_tensor(a[i], device=DEV).double() for a in (cen, half))
        lo, hi = (torch.as_tensor(b[i].astype(np.float64), device=DEV) for b in (gs.lo, gs.hi))
        for c0 in range(0, len(T), step):
            l = local_points(T[c0:c0 + step, i], x)
            xh = (l - ce) / ha
            E = torch.where(xh.abs().amax(-1) <= 1.0, core_distance(l - ce, core[i]), math.inf)
            U = torch.where(E - B >= MARGIN, E + B, math.inf).amin(1).clamp(min=MARGIN)
            at = ((E - B <= U[:, None] + 1e-3) & (E < math.inf)).nonzero()
            for part in at.split(1 << 20):
                pl = l[part[:, 0], part[:, 1]]
                m = mlp_hidden(p, xh[part[:, 0], part[:, 1]]) @ w4 + b4
                v = E[part[:, 0], part[:, 1]] + B * torch.tanh(m / B)
                near = ((v < MARGIN) & ((pl >= lo) & (pl <= hi)).all(-1)).nonzero()[:, 0]
                if len(near):
                    v[near] = interpolate(gs, i, pl[near])
                out[:, i].scatter_reduce_(0, part[:, 0] + c0, v, "amin")
    return out


def mesh_distance(mesh, x):
    """Signed distance float64 of points x [N][3] to a mesh of closed parts:
    the minimum over parts, negative where a part's winding number exceeds 1/2."""
    verts = torch.as_tensor(mesh.verts.astype(np.float32).astype(np.float64), device=DEV)
    tris = torch.as_tensor(mesh.tris, device=DEV).long()
    out = []
    for p in x.split(max(1, 6_000_000 // len(tris))):
        best = torch.full((len(p),), math.inf, dtype=torch.float64, device=DEV)
        for k in range(len(mesh.comp_first) - 1):
            A, B, C = (verts[tris[mesh.comp_first[k]:mesh.comp_first[k + 1], j]][None] - p[:, None] for j in range(3))
            d2 = torch.full(A.shape[:2], math.inf, dtype=torch.float64, device=DEV)
            for P, Q in ((A, B), (B, C), (C, A)):
                e = Q - P
                t = (-(P * e).sum(-1) / (e * e).sum(-1)).clamp(0.0, 1.0)
                d2 = torch.minimum(d2, ((P + t[..., None] * e) ** 2).sum(-1))
            n = torch.linalg.cross(B - A, C - A)
            nn = (n * n).sum(-1)
            # inside the triangle's prism: the plane's distance
            w = [(torch.linalg.cross(Q - P, -P) * n).sum(-1) for P, Q in ((A, B), (B, C), (C, A))]
            face = (w[0] >= 0) & (w[1] >= 0) & (w[2] >= 0)
            d2 = torch.where(face, torch.minimum(d2, (A * n).sum(-1) ** 2 / nn), d2)
            la, lb, lc = (V.norm(dim=-1) for V in (A, B, C))
            det = (A * torch.linalg.cross(B, C)).sum(-1)
            den = la * lb * lc + (A * B).sum(-1) * lc + (A * C).sum(-1) * lb + (B * C).sum(-1) * la
            inside = torch.atan2(det, den).sum(1) > math.pi
            d = d2.amin(1).sqrt()
            best = torch.minimum(best, torch.where(inside, -d, d))
        out.append(best)
    return torch.cat(out)


def environment_grids(s, sample):
    """Robot SDFs float64 [C][V]: per configuration, `sample(c, i, lo, hi)` gives
    the flat voxels in link i's box and their values."""
    case, gs = s["case"], s["grids"]
    out = torch.full((case["C"], case["env"] ** 3), math.inf, dtype=torch.float64, device=DEV)
    for i in range(case["joints"] + 1):
        lo, hi = (torch.as_tensor(b[i].astype(np.float64), device=DEV) for b in (gs.lo, gs.hi))
        for c in range(case["C"]):
            at, v = sample(c, i, lo, hi)
            out[c].scatter_reduce_(0, at, v, "amin")
    return out


def voxel_centres(case):
    a = -0.5 * case["env"] * case["voxel"] + (torch.arange(case["env"], device=DEV).double() + 0.5) * case["voxel"]
    a = a.float().double()
    z, y, x = torch.meshgrid(a, a, a, indexing="ij")
    return torch.stack([x, y, z], -1).reshape(-1, 3)


def adam(p, m, v, g, lr):
    m2, v2 = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
    c1, c2 = 1 - 0.9 ** 1000, 1 - 0.999 ** 1000
    return p - lr * (m2 / c1) / ((v2 / c2).sqrt() + 1e-8), m2, v2


def exact(case, seed):
    kind = case["kind"]
    if kind == "frnn_build" and case["C"] * case["env"] ** 3 > 1.2e8:
        return None
    s = prepare(case, seed)
    if kind in ("tick", "step"):
        return link_minima(s["grids"], poses(case["joints"], s["q"]), s["points"].double()).amin(1), None
    if kind == "query":
        ld = link_minima(s["grids"], s["T"].double(), s["points"].double())
        return ld.amin(1), None, ld
    if kind == "batch":
        c, m = s["c_off"].tolist(), s["m_off"].tolist()
        return torch.cat([link_minima(s["grids"], s["T"][c[k]:c[k + 1]].double(),
                                      s["points"][m[k]:m[k + 1]].double()).amin(1) for k in range(case["K"])]), None
    if kind == "learned":
        ld = learned_minima(s)
        return ld.amin(1), None, ld
    if kind == "train":
        cen, half, core = mlp_domains(case["joints"])
        P, loss = s["params"].double().requires_grad_(), []
        for i in range(case["joints"] + 1):
            at = s["index"][i].long()
            u = s["samples"][i][at].double() - torch.as_tensor(cen[i], device=DEV).double()
            h = mlp_hidden(P[i], u / torch.as_tensor(half[i], device=DEV).double())
            share = h @ _rounded(mlp_split(P[i])[6]) + mlp_split(P[i])[7]
            B = float(np.float32(0.15))
            est = B * torch.tanh(share / B) + core_distance(u, core[i])
            loss.append((est - s["labels"][i][at].double()).abs().mean())
        loss = torch.stack(loss)
        g, = torch.autograd.grad(loss.sum(), P)
        return (*adam(P.detach(), s["m"].double(), s["v"].double(), g, 1e-3), loss.detach(), g)
    if kind == "labels":
        out = []
        for i, mesh in enumerate(s["meshes"]):
            x = s["samples"][i].double()
            lo, hi = (torch.as_tensor(b[i].astype(np.float64), device=DEV) for b in (s["grids"].lo, s["grids"].hi))
            inside = ((x >= lo) & (x <= hi)).all(-1)
            v = torch.empty(len(x), dtype=torch.float64, device=DEV)
            v[inside] = interpolate(s["grids"], i, x[inside])
            v[~inside] = mesh_distance(mesh, x[~inside])
            out.append(v)
        return torch.stack(out)
    if kind == "grids":
        return torch.cat([mesh_distance(m, node_positions(s["lo"][i], s["hi"][i], case["n"]))
                          for i, m in enumerate(s["meshes"])])
    if kind == "robot_sdf":
        x, T = voxel_centres(case), s["T"].double()

        def sample(c, i, lo, hi):
            l = local_points(T[c:c + 1, i], x)[0]
            at = ((l >= lo) & (l <= hi)).all(-1).nonzero()[:, 0]
            return at, interpolate(s["grids"], i, l[at])
        rs = environment_grids(s, sample)
        v = (s["points"].double() / case["voxel"] + 0.5 * case["env"]).floor().long()
        v = v[((v >= 0) & (v < case["env"])).all(-1)]
        flat = torch.unique((v[:, 2] * case["env"] + v[:, 1]) * case["env"] + v[:, 0])
        return rs.view(case["C"], *[case["env"]] * 3), rs[:, flat].amin(1)
    if kind == "frnn_train":
        P = s["params"].double().requires_grad_()
        W1, b1, W2, b2 = frnn_split(P)
        R = s["R"].double()
        f = torch.relu(R @ W1.T + b1) @ W2.T + b2
        target = torch.matmul(block_centres(case["m"]), R.view(-1, 3, 3)).reshape(case["B"], -1)
        loss = (f - target).abs().mean()
        g, = torch.autograd.grad(loss, P)
        return (*adam(P.detach(), s["m"].double(), s["v"].double(), g, 1e-4), loss.detach().view(1), g)
    # frnn_build: each link's block of voxels at the points the network gives
    m, T, E, r = s["half"], s["T"].double(), case["env"], float(np.float32(case["voxel"]))
    W1, b1, W2, b2 = (a.double() for a in frnn_split(s["params"]))
    lo_env = float(np.float32(-0.5 * E * case["voxel"]))
    j = torch.arange(2 * m, device=DEV)

    def sample(c, i, lo, hi):
        R, t_o = T[c, i, :, :3], T[c, i, :, 3] - lo_env
        k = (t_o / r).round().long() - m
        dt = t_o - (k + m) * r
        f = (torch.relu(W1 @ R.reshape(9) + b1) @ W2.T + b2).view(-1, 3)
        l = m * r * f - dt @ R
        vz, vy, vx = torch.meshgrid(j + k[2], j + k[1], j + k[0], indexing="ij")
        v = torch.stack([vx, vy, vz], -1).reshape(-1, 3)
        at = (((l >= lo) & (l <= hi)).all(-1) & ((v >= 0) & (v < E)).all(-1)).nonzero()[:, 0]
        return (v[at, 2] * E + v[at, 1]) * E + v[at, 0], interpolate(s["grids"], i, l[at])
    return environment_grids(s, sample).view(case["C"], E, E, E)
