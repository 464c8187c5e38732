"""The calls a program makes through this package's public entry points, with
the inputs it makes them on and what plain FP64 torch gives for them.

A case is one pass of such a program: a tactile sensor pad stepped alone, a
batch of hands stepped in a rollout, the same with gradients for calibration
or policy search, the contact pass alone, scenes with triangle-mesh objects,
the articulated hand with its contact reward, and the real-sensor regressor.
Inputs are drawn from the seed on the GPU; plans and output buffers are kept
between passes, as a simulation loop keeps them.
"""
import math

import numpy as np
import torch

from paper_2604_20295_amd import _native, autograd

FULL, DECAY, RESIDUAL = _native.ETAC_FULL, _native.ETAC_DECAY_ONLY, _native.ETAC_RESIDUAL_ONLY
SPHERE, BOX, CAPSULE, MESH = 0, 1, 2, 3


def listed():
    return [
        # one sensor pad in a control loop: latency of a single step
        dict(name="pad_step", kind="step", mesh="pad", envs=1, mode=FULL, back=False),
        # calibration of alpha and the network on a handful of pad indentations (autograd)
        dict(name="pad_fit", kind="fit", mesh="pad", envs=8, mode=FULL, back=True),
        # the rollout of a trained policy on very many hands: forward only
        dict(name="hand_rollout", kind="step", mesh="hand", envs=16384, mode=FULL, back=False),
        # the benchmark's step: forward with the pooling record, then the adjoint
        dict(name="hand_train", kind="step", mesh="hand", envs=4096, mode=FULL, back=True),
        # a mid-size batch of hands whose patches have odd node counts
        dict(name="ragged_train", kind="step", mesh="ragged", envs=301, mode=FULL, back=True),
        # Eq. 1 alone with gradients: fitting the decay rates
        dict(name="decay_train", kind="step", mesh="hand", envs=509, mode=DECAY, back=True),
        # contact masks and displacements only (a reward, or a user's own propagation)
        dict(name="hand_contact", kind="contact", mesh="hand", envs=4096, mode=FULL, back=False),
        # high-resolution pads for rendering tactile images: forward only
        dict(name="hires_step", kind="step", mesh="hires", envs=48, mode=FULL, back=False),
        # high-resolution pads with gradients
        dict(name="hires_train", kind="step", mesh="hires", envs=9, mode=FULL, back=True),
        # scenes with triangle-mesh objects, forward and adjoint (autograd)
        dict(name="object_train", kind="object", mesh="hand", envs=256, mode=FULL, back=True),
        # articulated hand with self-contact and the contact reward, forward and adjoint
        dict(name="grasp_train", kind="grasp", mesh="fingers", envs=1024, mode=FULL, back=True),
        # taxel outputs of a step's displacement field
        dict(name="taxels", kind="taxels", mesh="hand", envs=1024, mode=FULL, back=False),
    ]


# envs per case kind and mesh: the smallest and the largest a drawn case takes
RANGES = {("step", "pad"): (1, 64), ("fit", "pad"): (1, 32), ("step", "hand"): (8, 4096), ("step", "ragged"): (8, 1024),
          ("contact", "hand"): (8, 8192), ("step", "hires"): (1, 24), ("object", "hand"): (8, 256),
          ("grasp", "fingers"): (8, 1024), ("taxels", "hand"): (8, 1024), ("taxels", "ragged"): (8, 512)}


def draw(rng):
    kind, mesh = rng.choice(sorted(RANGES))
    lo, hi = RANGES[kind, mesh]
    envs = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    back = kind in ("fit", "object", "grasp") or (kind == "step" and rng.random() < 0.5)
    if mesh == "hires" and back:
        envs = min(envs, 12)
    mode = rng.choice((FULL, FULL, DECAY, RESIDUAL)) if kind in ("step", "fit") else FULL
    # `turn` moves the fixed draws of the surface (its patch sizes where they are ragged)
    return dict(kind=kind, mesh=mesh, envs=envs, mode=mode, back=back, turn=rng.randrange(1 << 16))


# ---------------------------------------------------------------------------
# elastomer surfaces (host arrays, as the plan takes them)
# ---------------------------------------------------------------------------
def _grid(nx, ny, pitch, centre, radius):
    u = (np.arange(nx) - (nx - 1) / 2.0) * pitch
    v = (np.arange(ny) - (ny - 1) / 2.0) * pitch
    U, V = (a.ravel() for a in np.meshgrid(u, v))
    th = V / radius if radius > 0 else np.zeros_like(V)
    y, z = (radius * np.sin(th), radius * (np.cos(th) - 1.0)) if radius > 0 else (V, np.zeros_like(V))
    pos = np.stack([U + centre[0], y + centre[1], z + centre[2]])
    return pos, np.stack([np.zeros_like(U), np.sin(th), np.cos(th)])


class Surface:
    """Patches of an elastomer surface and, for the articulated hand, its links."""

    def __init__(self, patches, origins, pitches, grids, hand=None):
        self.offset = np.cumsum([0] + [p.shape[1] for p, _ in patches]).astype(np.int32)
        self.pos = np.concatenate([p for p, _ in patches], 1).astype(np.float32)
        self.nrm = np.concatenate([n for _, n in patches], 1).astype(np.float32)
        self.origin = np.asarray(origins, np.float32)
        self.pitch = np.asarray(pitches, np.float64)
        self.grids = grids              # (nx, ny, curvature radius or 0) per patch
        self.hand = hand
        self.K, self.N = len(patches), int(self.offset[-1])

    def sizes(self):
        return np.diff(self.offset)


def _surface(case):
    name = case["mesh"]
    if name == "pad":       # 32 x 32 nodes, 0.5 mm apart
        grids, pitch, centres = [(32, 32, 0.0)], [0.5], [(0.0, 0.0, 0.0)]
    elif name == "hires":   # four pads of 128 x 128 nodes, 0.125 mm apart
        grids, pitch = [(128, 128, 0.0)] * 4, [0.125] * 4
        centres = [((k % 2 - 0.5) * 24.0, (k // 2 - 0.5) * 24.0, 0.0) for k in range(4)]
    elif name in ("hand", "ragged"):
        rng = np.random.default_rng([0, 7])
        sizes = rng.choice((64, 128, 256, 512, 1024), size=16)
        curved = np.zeros(16, bool)
        curved[rng.permutation(16)[:8]] = True
        radii = rng.uniform(8.0, 15.0, size=16)
        shape = {64: (8, 8), 128: (16, 8), 256: (16, 16), 512: (32, 16), 1024: (32, 32)}
        wh = [shape[int(s)] for s in sizes]
        if name == "ragged":            # node counts between 35 and 1147, mostly odd
            r2 = np.random.default_rng([case.get("turn", 0), 13])
            wh = [(int(r2.integers(7, 38)), int(r2.integers(5, 32))) for _ in range(16)]
        grids = [(w, h, float(radii[k]) if curved[k] else 0.0) for k, (w, h) in enumerate(wh)]
        pitch = [1.0] * 16
        centres = [((k % 4 - 1.5) * 45.0, (k // 4 - 1.5) * 45.0, 0.0) for k in range(16)]
    else:
        return _fingers()
    patches = [_grid(nx, ny, p, c, r) for (nx, ny, r), p, c in zip(grids, pitch, centres)]
    return Surface(patches, centres, pitch, grids)


# the articulated hand: a palm and five fingers of three phalanges; link
# frames have y along the bone and z along the palmar normal
PALM = (42.0, 45.0, 12.0)
LENGTHS = ((40.0, 30.0, 24.0), (44.0, 26.0, 20.0), (46.0, 28.0, 22.0), (42.0, 26.0, 20.0), (34.0, 20.0, 18.0))
RADII = (10.0, 9.0, 9.5, 9.0, 8.0)
BASE_X = (None, -27.0, -9.0, 9.0, 27.0)


class Links:
    def __init__(self):
        L = self.n_links = 16
        self.parent = [-1] + [0 if s == 0 else 3 * f + s for f in range(5) for s in range(3)]
        self.patch_link = np.arange(L, dtype=np.int32)
        self.prim_type = np.full(L, CAPSULE, np.int32)
        self.prim_shape = np.zeros((L, 4), np.float32)
        self.prim_rot = np.tile(np.array([1, 0, 0, 0, 0, 1, 0, -1, 0], np.float32), (L, 1))
        self.prim_trans = np.zeros((L, 3), np.float32)
        self.joint = np.zeros((L, 3))
        self.base = np.tile(np.eye(3), (L, 1, 1))
        self.prim_type[0], self.prim_shape[0, :3], self.prim_rot[0] = BOX, PALM, np.eye(3).ravel()
        for f in range(5):
            for s in range(3):
                i = 1 + 3 * f + s
                half = LENGTHS[f][s] / 2.0
                self.prim_shape[i, :2] = RADII[f], half
                self.prim_trans[i] = 0.0, half, 0.0
                self.joint[i] = (0.0, LENGTHS[f][s - 1], 0.0) if s else \
                    ((BASE_X[f], PALM[1], 0.0) if f else (-PALM[0] + 6.0, -8.0, 2.0))
        a, b = math.radians(55.0), math.radians(-35.0)
        rz = np.array([[math.cos(a), -math.sin(a), 0], [math.sin(a), math.cos(a), 0], [0, 0, 1]])
        ry = np.array([[math.cos(b), 0, math.sin(b)], [0, 1, 0], [-math.sin(b), 0, math.cos(b)]])
        self.base[1] = rz @ ry
        # a link meets every other one but its joint neighbours
        near = [{i, self.parent[i]} | {j for j in range(L) if self.parent[j] == i} for i in range(L)]
        self.collide = np.array([sum(1 << j for j in range(L) if j not in near[i]) for i in range(L)], np.uint32)


def _fingers():
    h = Links()
    pos, nrm = _grid(32, 32, 2.5, (0.0, 0.0, PALM[2]), 0.0)
    patches, origins, pitches, grids = [(pos, nrm)], [(0.0, 0.0, PALM[2])], [2.5], [(32, 32, 0.0)]
    for f in range(5):
        for s, (na, nb, pitch) in enumerate(((32, 16, 1.25), (16, 16, 1.25), (16, 8, 1.0))):
            half, r = LENGTHS[f][s] / 2.0, RADII[f]
            u = (np.arange(na) - (na - 1) / 2.0) * pitch + half
            th = (np.arange(nb) - (nb - 1) / 2.0) * pitch / r
            Y, T = (a.ravel() for a in np.meshgrid(u, th))
            patches.append((np.stack([r * np.sin(T), Y, r * np.cos(T)]),
                            np.stack([np.sin(T), np.zeros_like(T), np.cos(T)])))
            origins.append((0.0, half, r))
            pitches.append(pitch)
            grids.append((na, nb, r))
    return Surface(patches, origins, pitches, grids, h)


# ---------------------------------------------------------------------------
# scenes (FP64 on the GPU, handed over in FP32)
# ---------------------------------------------------------------------------
class Draw:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.dev = torch.device("cuda", torch.cuda.current_device())
        self.g = torch.Generator(device=self.dev).manual_seed(int(seed))

    def uniform(self, lo, hi, shape):
        return lo + (hi - lo) * torch.rand(shape, generator=self.g, device=self.dev, dtype=torch.float64)

    def normal(self, shape, dtype=torch.float64):
        return torch.randn(shape, generator=self.g, device=self.dev, dtype=dtype)

    def integers(self, lo, hi, shape):
        return torch.randint(lo, hi, shape, generator=self.g, device=self.dev)

    def rotations(self, shape):
        q = self.normal(tuple(shape) + (4,))
        w, x, y, z = (q / q.norm(dim=-1, keepdim=True)).unbind(-1)
        rows = [1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]
        return torch.stack(rows, -1).reshape(*shape, 3, 3)


def _rodrigues(w):
    th = w.norm(dim=-1, keepdim=True).clamp_min(1e-12)
    k = w / th
    z = torch.zeros_like(k[..., 0])
    Kx = torch.stack([z, -k[..., 2], k[..., 1], k[..., 2], z, -k[..., 0], -k[..., 1], k[..., 0], z], -1)
    Kx = Kx.reshape(*w.shape[:-1], 3, 3)
    eye = torch.eye(3, dtype=w.dtype, device=w.device)
    return eye + torch.sin(th)[..., None] * Kx + (1 - torch.cos(th))[..., None] * (Kx @ Kx)


def _extent(ty, shape, R, u):
    """Extent of a primitive from its centre along the unit direction u."""
    box = (shape[..., :3] * (R.transpose(-1, -2) @ u[..., None])[..., 0].abs()).sum(-1)
    cap = shape[..., 0] + shape[..., 1] * (R[..., :, 2] * u).sum(-1).abs()
    return torch.where(ty == SPHERE, shape[..., 0], torch.where(ty == BOX, box, cap))


def _primitives(d, shape, scale=1.0):
    """Spheres r 10..40 mm, boxes with sides 20..60 mm, capsules r 8..20 mm, length 30..80 mm."""
    ty = d.integers(0, 3, shape)
    sh = torch.zeros(tuple(shape) + (4,), dtype=torch.float64, device=d.dev)
    r, sides = d.uniform(10, 40, shape), d.uniform(10, 30, tuple(shape) + (3,))
    cr, cl = d.uniform(8, 20, shape), d.uniform(15, 40, shape)
    sh[..., :3] = torch.where((ty == BOX)[..., None], sides, 0.0)
    sh[..., 0] = torch.where(ty == SPHERE, r, torch.where(ty == CAPSULE, cr, sh[..., 0]))
    sh[..., 1] = torch.where(ty == CAPSULE, cl, sh[..., 1])
    R = torch.where((ty == SPHERE)[..., None, None], torch.eye(3, dtype=torch.float64, device=d.dev), d.rotations(shape))
    return ty, sh * scale, R


def _footprint_scene(d, M, E, O=3):
    """1-3 primitives a hand that together press 8-24 % of its nodes, each on a patch of its own."""
    t64 = lambda a: torch.as_tensor(np.asarray(a), dtype=torch.float64, device=d.dev)  # noqa: E731
    sizes, K = t64(M.sizes()), M.K
    cnt = d.integers(1, O + 1, (E,))
    share = d.uniform(0.08, 0.24, (E,)) * M.N / cnt
    w = torch.where(0.85 * sizes >= share[:, None], sizes, 1e-5 * sizes)
    k = torch.multinomial(w, O, replacement=False, generator=d.g)              # [E][O] patches
    nodes = torch.minimum(share[:, None], 0.85 * sizes[k])
    g = t64([(a, b, r) for a, b, r in M.grids])
    nx, ny, rc = (g[:, c][k] for c in range(3))
    area = nodes * t64(M.pitch)[k] ** 2 * torch.where(rc > 0, 1.6, 1.0)
    i = torch.round(d.uniform(0.35, 0.65, (E, O)) * (nx - 1))
    j = torch.round(d.uniform(0.35, 0.65, (E, O)) * (ny - 1))
    node = torch.as_tensor(M.offset[:-1].astype(np.int64), device=d.dev)[k] + (j * nx + i).long()
    p, n = (t64(a).T[node] for a in (M.pos, M.nrm))
    n = n / n.norm(dim=-1, keepdim=True)
    ty = d.integers(0, 3, (E, O))
    a = torch.where(n[..., :1].abs() < 0.9, t64([1.0, 0, 0]), t64([0, 1.0, 0]))
    t1 = torch.linalg.cross(n, a)
    t1 = t1 / t1.norm(dim=-1, keepdim=True)
    t2 = torch.linalg.cross(n, t1)
    ph = d.uniform(0, 2 * math.pi, (E, O))[..., None]
    t1, t2 = torch.cos(ph) * t1 + torch.sin(ph) * t2, -torch.sin(ph) * t1 + torch.cos(ph) * t2
    # sphere: a disc of the area; capsule along the surface: a stadium; box: its face
    rs = torch.maximum(d.uniform(10, 40, (E, O)), torch.sqrt(area / (0.8 * math.pi)))
    ds = rs - torch.sqrt((rs * rs - area / math.pi).clamp_min(0))
    rcap, lcap = d.uniform(8, 20, (E, O)), d.uniform(15, 40, (E, O))
    le = torch.minimum(lcap, 0.5 * torch.minimum(nx, ny) * t64(M.pitch)[k])
    wc = (-4 * le + torch.sqrt(16 * le * le + 4 * math.pi * area)) / (2 * math.pi)
    wc = torch.minimum(wc, 0.95 * rcap)
    dc = rcap - torch.sqrt(rcap * rcap - wc * wc)
    sa = torch.sqrt(area) * torch.exp(d.uniform(-0.3, 0.3, (E, O)))
    hb, db = d.uniform(10, 30, (E, O)), d.uniform(1, 3, (E, O))
    sh = torch.zeros((E, O, 4), dtype=torch.float64, device=d.dev)
    sh[..., 0] = torch.where(ty == SPHERE, rs, torch.where(ty == BOX, sa / 2, rcap))
    sh[..., 1] = torch.where(ty == BOX, area / sa / 2, torch.where(ty == CAPSULE, lcap, 0.0))
    sh[..., 2] = torch.where(ty == BOX, hb, 0.0)
    R = torch.where((ty == BOX)[..., None, None], torch.stack([t1, t2, n], -1), torch.stack([t2, n, t1], -1))
    tilt = _rodrigues(t1 * torch.deg2rad(d.uniform(-2, 2, (E, O)))[..., None])
    R = torch.where((ty == SPHERE)[..., None, None], torch.eye(3, dtype=torch.float64, device=d.dev), tilt @ R)
    depth = torch.where(ty == SPHERE, ds, torch.where(ty == BOX, db, dc))
    ext = torch.where(ty == SPHERE, rs, torch.where(ty == BOX, hb, rcap))
    return cnt, ty, sh, R, p + (ext - depth)[..., None] * n


def _scene(d, case, M, tri=None):
    """(n_obj, type, shape, R, t) of the case's envs, FP32 / int32 on the GPU."""
    E, name = case["envs"], case["mesh"]
    up = torch.tensor([0.0, 0.0, 1.0], dtype=torch.float64, device=d.dev)
    if case["kind"] == "object":        # 1-3 objects of the mesh set, pressed 2-10 mm at a node
        O = 3
        cnt, m, R = d.integers(1, O + 1, (E,)), d.integers(0, len(tri.parts), (E, O)), d.rotations((E, O))
        p = torch.as_tensor(M.pos.T.astype(np.float64), device=d.dev)[d.integers(0, M.N, (E, O))]
        ext = torch.stack([((R.transpose(-1, -2) @ -up) @ torch.as_tensor(v.T.copy(), device=d.dev)).amax(-1)
                           for v, _ in tri.parts], -1).gather(-1, m[..., None])[..., 0]
        ty, sh = torch.full_like(m, MESH), torch.zeros((E, O, 4), dtype=torch.float64, device=d.dev)
        sh[..., 0] = m
        t = p + (ext - d.uniform(2, 10, (E, O)))[..., None] * up
    elif name == "pad":                 # one sphere of 5 mm pressed 0.2-1.5 mm
        cnt, ty = torch.ones(E, device=d.dev), torch.zeros((E, 1), device=d.dev)
        sh = torch.zeros((E, 1, 4), dtype=torch.float64, device=d.dev)
        sh[..., 0] = 5.0
        R = torch.eye(3, dtype=torch.float64, device=d.dev).expand(E, 1, 3, 3)
        t = torch.cat([d.uniform(-7.75, 7.75, (E, 1, 2)), 5.0 - d.uniform(0.2, 1.5, (E, 1, 1))], -1)
    elif name == "hires":               # a sphere or a turned box on every pad, pressed 0.1-2 mm
        K = M.K
        cnt, ty = torch.full((E,), K, device=d.dev), d.integers(0, 2, (E, K))
        sh = torch.zeros((E, K, 4), dtype=torch.float64, device=d.dev)
        sh[..., :3] = torch.where((ty == BOX)[..., None], d.uniform(2, 6, (E, K, 3)), 0.0)
        sh[..., 0] = torch.where(ty == SPHERE, d.uniform(3, 8, (E, K)), sh[..., 0])
        R = torch.where((ty == SPHERE)[..., None, None], torch.eye(3, dtype=torch.float64, device=d.dev),
                        d.rotations((E, K)))
        lift = _extent(ty, sh, R, up) - d.uniform(0.1, 2.0, (E, K))
        half = 127 * 0.125 / 2 - 2.0
        c = torch.as_tensor(M.origin.astype(np.float64), device=d.dev)
        t = c + torch.cat([d.uniform(-half, half, (E, K, 2)), lift[..., None]], -1)
    else:
        cnt, ty, sh, R, t = _footprint_scene(d, M, E)
    return _handed(cnt, ty, sh, R, t)


def _handed(cnt, ty, sh, R, t):
    E, O = ty.shape
    return (cnt.to(torch.int32).contiguous(), ty.to(torch.int32).contiguous(), sh.float().contiguous(),
            R.reshape(E, O, 9).float().contiguous(), t.float().contiguous())


def _grasp(d, M, E, O=2):
    """Objects pressed 1-4 mm into the palm, fingers curled around them: (scene, link rot, link trans)."""
    h = M.hand
    t64 = lambda a: torch.as_tensor(np.asarray(a), dtype=torch.float64, device=d.dev)  # noqa: E731
    R0, t0 = d.rotations((E,)), d.uniform(-50, 50, (E, 3))
    cnt = d.integers(1, O + 1, (E,))
    ty, sh, Ro = _primitives(d, (E, O), 0.8)
    ext = _extent(ty, sh, Ro, R0[:, None, :, 2].expand(E, O, 3))
    at = torch.stack([d.uniform(-18, 18, (E, O)), d.uniform(0, 30, (E, O)), torch.full_like(ext, PALM[2])], -1)
    t = (R0[:, None] @ at[..., None])[..., 0] + t0[:, None] + (ext - d.uniform(1, 4, (E, O)))[..., None] * R0[:, None, :, 2]
    R, tr = [R0], [t0]
    for f in range(5):
        lim = torch.deg2rad(t64((60.0, 70.0, 70.0) if f == 0 else (85.0, 100.0, 75.0)))
        flex = d.uniform(0.2, 0.9, (E, 1)) * d.uniform(0.7, 1.0, (E, 3)) * lim
        side = torch.deg2rad(d.uniform(-12, 12, (E,)))
        z = torch.zeros_like(side)
        for s in range(3):
            i = 1 + 3 * f + s
            turn = _rodrigues(torch.stack([flex[:, s], z, z], -1))
            if s == 0:
                turn = _rodrigues(torch.stack([z, z, side], -1)) @ turn
            P, tp = R[h.parent[i]], tr[h.parent[i]]
            R.append(P @ t64(h.base[i]) @ turn)
            tr.append((P @ t64(h.joint[i])) + tp)
    rot = torch.stack(R, 1).reshape(E, 16, 9).float().contiguous()
    return _handed(cnt, ty, sh, Ro, t), rot, torch.stack(tr, 1).float().contiguous()


# ---------------------------------------------------------------------------
# triangle-mesh objects
# ---------------------------------------------------------------------------
def _icosphere(levels):
    g = (1.0 + 5.0 ** 0.5) / 2.0
    v = [[-1, g, 0], [1, g, 0], [-1, -g, 0], [1, -g, 0], [0, -1, g], [0, 1, g], [0, -1, -g], [0, 1, -g],
         [g, 0, -1], [g, 0, 1], [-g, 0, -1], [-g, 0, 1]]
    v = [np.asarray(x) / np.linalg.norm(x) for x in v]
    f = [(0, 11, 5), (0, 5, 1), (0, 1, 7), (0, 7, 10), (0, 10, 11), (1, 5, 9), (5, 11, 4), (11, 10, 2), (10, 7, 6),
         (7, 1, 8), (3, 9, 4), (3, 4, 2), (3, 2, 6), (3, 6, 8), (3, 8, 9), (4, 9, 5), (2, 4, 11), (6, 2, 10),
         (8, 6, 7), (9, 8, 1)]
    for _ in range(levels):
        mid, nf = {}, []

        def half(a, b):
            key = (min(a, b), max(a, b))
            if key not in mid:
                m = v[a] + v[b]
                mid[key] = len(v)
                v.append(m / np.linalg.norm(m))
            return mid[key]
        for a, b, c in f:
            ab, bc, ca = half(a, b), half(b, c), half(c, a)
            nf += [(a, ab, ca), (b, bc, ab), (c, ca, bc), (ab, bc, ca)]
        f = nf
    return np.asarray(v), np.asarray(f)


class Objects:
    """An egg, a rock with bumps and dents, and a pebble: 1280, 1280 and 320 triangles."""

    def __init__(self):
        v, f = _icosphere(3)
        v1, f1 = _icosphere(2)
        rng = np.random.default_rng(31)
        c = rng.standard_normal((12, 3))
        c /= np.linalg.norm(c, axis=1, keepdims=True)
        bump = (rng.uniform(-0.3, 0.3, 12) * np.exp(-((v[:, None] - c) ** 2).sum(-1) / rng.uniform(0.35, 0.7, 12) ** 2))
        egg = v * np.stack([20 * (1 - 0.15 * v[:, 2].clip(0)), 20 * (1 - 0.15 * v[:, 2].clip(0)), 0 * v[:, 2] + 28], 1)
        parts = [(egg, f), (v * 20.0 * (1 + bump.sum(1))[:, None], f), (v1 * np.array([14.0, 11.0, 9.0]), f1)]
        self.parts = [(a.astype(np.float32).astype(np.float64), b) for a, b in parts]
        base = np.cumsum([0] + [len(a) for a, _ in self.parts])
        self.verts = np.concatenate([a for a, _ in self.parts]).astype(np.float32)
        self.tris = np.concatenate([b + o for (_, b), o in zip(self.parts, base)]).astype(np.int32)
        self.offset = np.cumsum([0] + [len(b) for _, b in self.parts]).astype(np.int32)


# ---------------------------------------------------------------------------
# models
# ---------------------------------------------------------------------------
LAYERS = (("W1", 64, 9), ("W2", 64, 64), ("W3", 64, 64), ("W4", 64, 128), ("W5", 3, 64))
HEAD = (("E1", 64, 6), ("E2", 64, 64), ("E3", 256, 64), ("A1", 128, 256), ("a2", 1, 128), ("D1", 128, 256),
        ("D2", 8, 128))


def _model(d, M):
    """alpha 1.5..3 per pitch; weights and biases U(+-1/sqrt(fan in)), the last layer scaled by 0.02."""
    alpha = (d.uniform(1.5, 3.0, (M.K,)) / torch.as_tensor(M.pitch, device=d.dev)).float()
    parts = []
    for name, o, i in LAYERS:
        s = (0.02 if name == "W5" else 1.0) / math.sqrt(i)
        parts += [d.uniform(-s, s, (o * i,)), d.uniform(-s, s, (o,))]
    return alpha, torch.cat(parts).float()


def _head(d):
    parts = []
    for name, o, i in HEAD:
        s = 1.0 / math.sqrt(i)
        parts.append(d.uniform(-s, s, (o * i,)))
        parts.append(torch.zeros(4, dtype=torch.float64, device=d.dev) if name == "a2" else d.uniform(-s, s, (o,)))
    return torch.cat(parts).float()


def _pull(d, M, E):
    """dL/dU of a loss on the displacement field: one direction for the whole batch, as a target of
    more or less deformation gives, varied between envs and over the surface."""
    pos = torch.as_tensor(M.pos, device=d.dev)
    w = d.uniform(0.5, 1.5, (3, 1)) * (2 * d.integers(0, 2, (3, 1)) - 1)
    w = (w * (1.0 + 0.3 * d.normal((3, E)))).float()
    k, ph = d.uniform(-0.4, 0.4, (3, 3)).float(), d.uniform(0, 2 * math.pi, (3, E)).float()
    return torch.stack([0.3 * torch.sin((k[c] @ pos) + ph[c][:, None]) + w[c][:, None] for c in range(3)]).contiguous()


# ---------------------------------------------------------------------------
# the passes
# ---------------------------------------------------------------------------
class State:
    pass


def _inputs(case, seed):
    """Everything drawn from the seed, the same for run() and exact()."""
    s, d = State(), Draw(seed)
    s.M = _surface(case)
    s.tri = Objects() if case["kind"] == "object" else None
    if case["kind"] == "grasp":
        s.scene, s.lrot, s.ltrans = _grasp(d, s.M, case["envs"])
    else:
        s.scene = _scene(d, case, s.M, s.tri)
    s.alpha, s.phi = _model(d, s.M)
    s.gu = _pull(d, s.M, case["envs"]) if case["back"] else None
    s.reg = _head(d) if case["kind"] == "taxels" else None
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s.case, M, dev = case, s.M, s.alpha.device
    E, O, N, K = case["envs"], s.scene[1].shape[1], M.N, M.K
    s.plan = p = _native.Plan(M.offset, M.pos, M.nrm, M.origin, E, O, backward=case["back"])
    new = lambda shape, dt=torch.float32: torch.empty(shape, dtype=dt, device=dev)  # noqa: E731
    if case["kind"] == "fit":
        s.leaves = [x.requires_grad_(True) for x in (*s.scene[3:], s.alpha, s.phi)]
        return s
    if case["kind"] == "object":
        s.ms = _native.MeshSet(s.tri.verts, s.tri.tris, s.tri.offset)
        s.leaves = [x.requires_grad_(True) for x in (*s.scene[3:], s.alpha, s.phi)]
        return s
    s.sc, s.md = p.scene_struct(*s.scene), p.model_struct(case["mode"], s.alpha, s.phi)
    s.u, s.cobj, s.na = new((3, E, N)), new((E, N), torch.int8), new((E, K), torch.int32)
    s.saved = _native.saved_buffer(p, E) if case["back"] and case["mode"] != DECAY else None
    s.grads = [new((E, O, 9)), new((E, O, 3)), new((K,)), new((_native.ETAC_PHI_SIZE,))] if case["back"] else []
    if case["kind"] == "grasp":
        p.set_hand(M.hand)
        s.lk = p.links_struct(s.lrot, s.ltrans)
        s.r = new((E,))
        s.rw = p.reward_struct(E, 1.0, r_contact=s.r)
        s.grads[2:2] = [new((E, 16, 9)), new((E, 16, 3))]
    if case["kind"] == "taxels":
        _native.etac_step(p, s.sc, s.md, s.u, s.cobj, s.na)
        s.y = new((E, K, _native.ETAC_TAXELS))
    return s


NAMES = ("grad_rot", "grad_trans", "grad_alpha", "grad_phi")
GRASP_NAMES = ("grad_rot", "grad_trans", "grad_link_rot", "grad_link_trans", "grad_alpha", "grad_phi")


def run(s):
    c, p, kind = s.case, s.plan, s.case["kind"]
    if kind == "contact":
        _native.etac_contact(p, s.sc, s.cobj, s.u, s.na)
        return dict(cobj=s.cobj, na=s.na, u=s.u)
    if kind == "taxels":
        _native.etac_regress(p, s.reg, s.u, s.na, s.y)
        return dict(taxels=s.y)
    if kind == "fit":
        u, cobj, na = autograd.etac_step(p, *s.scene[:3], *s.leaves, c["mode"])
        return dict(zip(NAMES, torch.autograd.grad(u, s.leaves, s.gu)), u=u.detach(), cobj=cobj, na=na)
    if kind == "object":
        u, cobj, na = autograd.etac_mesh_step(p, s.ms, *s.scene[:3], *s.leaves, c["mode"])
        return dict(zip(NAMES, torch.autograd.grad(u, s.leaves, s.gu)), u=u.detach(), cobj=cobj, na=na)
    out = dict(u=s.u, cobj=s.cobj, na=s.na)
    if kind == "grasp":
        _native.etac_hand_step(p, s.sc, s.lk, s.md, s.u, s.cobj, s.na, s.rw, saved=s.saved)
        _native.etac_hand_step_backward(p, s.sc, s.lk, s.md, s.gu, *s.grads, saved=s.saved)
        return dict(out, r=s.r, **dict(zip(GRASP_NAMES, s.grads)))
    _native.etac_step(p, s.sc, s.md, s.u, s.cobj, s.na, saved=s.saved)
    if c["back"]:
        _native.etac_step_backward(p, s.sc, s.md, s.gu, *s.grads, saved=s.saved)
        out.update(zip(NAMES, s.grads))
    return out


# nodes on patches in contact and nodes in contact, as shares of an env's nodes
SHARES = {"pad": (1.0, 0.11), "hand": (0.30, 0.13), "ragged": (0.32, 0.13), "hires": (1.0, 0.08),
          "fingers": (0.5, 0.03)}


def work(case):
    M = _surface(case)
    E, N, K, kind, mode = case["envs"], M.N, M.K, case["kind"], case["mode"]
    touched, active = SHARES[M.hand and "fingers" or case["mesh"]]
    touched, active = touched * E * N, active * E * N
    if kind == "taxels":
        return dict(bytes=12.0 * touched + 4.0 * E * K + 32.0 * E * K, flops=2.0 * 53632 * touched)
    out = 13.0 * E * N + 4.0 * E * K + 72.0 * E * 3      # displacements and winners, counts, poses
    if kind == "contact":
        return dict(bytes=out, flops=40.0 * touched)
    # Eq. 1: every active node against the passive nodes of its patch within reach (a weight of
    # 2^-50, at most some 800 nodes away); the encoder sees the active nodes, the output layer
    # every passive node of a patch in contact
    pairs = active * min(N / K * (1.0 - active / touched), 800.0)
    flops = (6.0 * pairs if mode != RESIDUAL else 0.0) + \
        (2.0 * 4672 * active + 2.0 * 256 * (touched - active) if mode != DECAY else 0.0)
    if case["back"]:
        return dict(bytes=out + 12.0 * touched + 48.0 * E * 3 + 70e3, flops=3.0 * flops)
    return dict(bytes=out, flops=flops)


# ---------------------------------------------------------------------------
# the same in plain FP64 torch
# ---------------------------------------------------------------------------
def _inside(ty, sh, R, t, pos, nrm):
    """One object of every row against the nodes of one patch: pos [n][3], R [B][3][3] ->
    inside [B][n], depth [B][n], displacement [B][n][3] (differentiable in R and t)."""
    d = pos - t[:, None]
    q = d @ R
    ty = ty[:, None]
    h = sh[:, None, :3]
    slack = h - q.abs()
    best, face = slack.min(-1)
    qf = q.gather(-1, face[..., None])[..., 0]
    hf = h.expand_as(q).gather(-1, face[..., None])[..., 0]
    sg = torch.where(qf >= 0, 1.0, -1.0).double()
    col = R.transpose(-1, -2).gather(1, face[..., None].expand(*face.shape, 3))
    ubox = (sg * hf - qf)[..., None] * col
    # sphere and capsule: towards the axis segment (of length 0 for a sphere)
    L = torch.where(ty == CAPSULE, sh[:, None, 1], 0.0)
    z = torch.maximum(torch.minimum(q[..., 2], L), -L)
    v = torch.where((ty == CAPSULE)[..., None], torch.cat([q[..., :2], (q[..., 2] - z)[..., None]], -1), d)
    r = sh[:, None, 0]
    s2 = (v * v).sum(-1)
    ln = torch.sqrt(torch.where(s2 > 0, s2, 1.0))
    vr = (r / ln - 1.0)[..., None] * v
    uround = torch.where((ty == CAPSULE)[..., None], vr @ R.transpose(-1, -2), vr)
    uround = torch.where((s2 > 0)[..., None], uround, -r[..., None] * nrm)
    box = ty == BOX
    inside = torch.where(box, (slack > 0).all(-1), s2 < r * r)
    depth = torch.where(box, best, r - torch.where(s2 > 0, ln, 0.0))
    return inside, depth.detach(), torch.where(box[..., None], ubox, uround)


def _closest(a, b, c, q):
    """Closest points of triangles (a, b, c) to q, differentiable (broadcast)."""
    def seg(p0, p1):
        e = p1 - p0
        w = ((q - p0) * e).sum(-1, keepdim=True) / (e * e).sum(-1, keepdim=True)
        return p0 + w.clamp(0, 1) * e
    n = torch.linalg.cross(b - a, c - a, dim=-1)
    nn = (n * n).sum(-1, keepdim=True)
    x = q - ((q - a) * n).sum(-1, keepdim=True) / nn * n
    within = torch.ones_like(nn, dtype=torch.bool)
    for p0, p1 in ((a, b), (b, c), (c, a)):
        within = within & ((torch.linalg.cross((p1 - p0).expand_as(x), x - p0, dim=-1) * n).sum(-1, keepdim=True) >= 0)
    far = lambda y: ((q - y) ** 2).sum(-1, keepdim=True)  # noqa: E731
    e = seg(a, b)
    for y in (seg(b, c), seg(c, a)):
        e = torch.where(far(y) < far(e), y, e)
    return torch.where(within, x, e)


def _inside_mesh(part, R, t, pos):
    """As _inside for one triangle mesh (a list of rows of their own): inside by the solid angle."""
    v, f = part
    v = torch.as_tensor(v, device=pos.device)
    A, B, C = (v[torch.as_tensor(f[:, i], device=pos.device)] for i in range(3))
    q = (pos - t[:, None]) @ R
    rad = v.norm(dim=-1).max()
    near = (q.detach().norm(dim=-1) < rad).nonzero()
    inside = torch.zeros(q.shape[:2], dtype=torch.bool, device=pos.device)
    depth = torch.zeros(q.shape[:2], dtype=torch.float64, device=pos.device)
    u = torch.zeros_like(q)
    got = []
    with torch.no_grad():
        for at in near.split(4096):
            x = q.detach()[at[:, 0], at[:, 1]][:, None]
            a, b, c = A - x, B - x, C - x
            la, lb, lc = a.norm(dim=-1), b.norm(dim=-1), c.norm(dim=-1)
            num = (a * torch.linalg.cross(b, c, dim=-1)).sum(-1)
            den = la * lb * lc + (a * b).sum(-1) * lc + (b * c).sum(-1) * la + (c * a).sum(-1) * lb
            ins = torch.atan2(num, den).sum(-1) > math.pi
            d2 = ((x - _closest(A, B, C, x)) ** 2).sum(-1)
            got.append((at[ins], d2[ins].argmin(-1)))
    if not got:
        return inside, depth, u
    at, tri = (torch.cat(g) for g in zip(*got))
    x = q[at[:, 0], at[:, 1]]
    w = _closest(A[tri], B[tri], C[tri], x) - x
    inside[at[:, 0], at[:, 1]] = True
    depth[at[:, 0], at[:, 1]] = w.detach().norm(dim=-1)
    u = u.index_put((at[:, 0], at[:, 1]), (R[at[:, 0]] @ w[..., None])[..., 0])
    return inside, depth, u


def _round32(x):
    """The value in FP32, with the gradient passed through."""
    return x + (x.detach().float().double() - x.detach())


def _unpack(phi, layers):
    at, out = 0, []
    for name, o, i in layers:
        w, b = phi[at:at + o * i].view(o, i), phi[at + o * i:at + o * i + (4 if name == "a2" else o)]
        at += w.numel() + b.numel()
        out.append((w, b))
    return out


def _candidates(s, k, env, leaves):
    """Objects that may touch patch k in the given envs: lists of (type, shape, R, t) over rows."""
    n_obj, ty, sh = s.scene[:3]
    rot, tr = leaves[0][env].view(len(env), -1, 3, 3), leaves[1][env]
    out = []
    if s.M.hand is None:
        for o in range(ty.shape[1]):
            t = torch.where(n_obj[env] > o, ty[env, o], -1)
            out.append((t, sh[env, o].double(), rot[:, o], tr[:, o], o))
        return out
    h = s.M.hand
    lr, lt = leaves[2][env].view(len(env), -1, 3, 3), leaves[3][env]
    link = int(h.patch_link[k])
    Rl, tl = lr[:, link].transpose(-1, -2), lt[:, link]
    rel = lambda R, t: (_round32(Rl @ R), _round32((Rl @ (t - tl)[..., None])[..., 0]))  # noqa: E731
    for o in range(ty.shape[1]):
        t = torch.where(n_obj[env] > o, ty[env, o], -1)
        out.append((t, sh[env, o].double(), *rel(rot[:, o], tr[:, o]), o))
    d64 = lambda a: torch.as_tensor(a, device=ty.device).double()  # noqa: E731
    for j in range(h.n_links):
        if (int(h.collide[link]) >> j) & 1:
            R = lr[:, j] @ d64(h.prim_rot[j]).view(3, 3)
            t = (lr[:, j] @ d64(h.prim_trans[j])[:, None])[..., 0] + lt[:, j]
            kind = torch.full((len(env),), int(h.prim_type[j]), device=ty.device)
            out.append((kind, d64(h.prim_shape[j]).expand(len(env), 4), *rel(R, t), ty.shape[1] + j))
    return out


def _contact(s, k, env, leaves, pos, nrm):
    """active [B][n], u_hat [B][n][3], winner's id [B][n] of patch k in the given envs."""
    B, n = len(env), pos.shape[0]
    best = torch.full((B, n), -1.0, dtype=torch.float64, device=pos.device)
    win = torch.full((B, n), -1, device=pos.device)
    u = torch.zeros((B, n, 3), dtype=torch.float64, device=pos.device)
    c = (pos.amax(0) + pos.amin(0)) / 2
    reach = (pos - c).norm(dim=-1).max()
    radii = torch.tensor([np.linalg.norm(v, axis=1).max() for v, _ in s.tri.parts], device=pos.device) if s.tri else None
    for ty, sh, R, t, ident in _candidates(s, k, env, leaves):
        rad = torch.where(ty == SPHERE, sh[:, 0], torch.where(ty == BOX, sh[:, :3].norm(dim=-1), sh[:, 0] + sh[:, 1]))
        if s.tri:
            rad = torch.where(ty == MESH, radii[sh[:, 0].long()], rad)
        may = (ty >= 0) & ((t.detach() - c).norm(dim=-1) < reach + rad + 1e-3)
        for m in range(len(s.tri.parts) if s.tri else 1):
            rows = (may & (sh[:, 0] == m) if s.tri else may).nonzero()[:, 0]
            if not len(rows):
                continue
            ins, dep, v = _inside_mesh(s.tri.parts[m], R[rows], t[rows], pos) if s.tri else \
                _inside(ty[rows], sh[rows], R[rows], t[rows], pos, nrm)
            take = ins & (dep > best[rows])
            best = best.index_put((rows,), torch.where(take, dep, best[rows]))
            win = win.index_put((rows,), torch.where(take, ident, win[rows]))
            u = u.index_put((rows,), torch.where(take[..., None], v, u[rows]))
    return win >= 0, u, win


def _field(s, k, act, uh, leaves, mode, D):
    """Eqs. 1-2 on patch k: U [B][n][3] from the active nodes' u_hat."""
    M = s.M
    sl = slice(int(M.offset[k]), int(M.offset[k + 1]))
    dev = act.device
    pos = torch.as_tensor(M.pos[:, sl].T.astype(np.float64), device=dev)
    uh = torch.where(act[..., None], uh, 0.0)
    out = torch.zeros_like(uh)
    if mode != RESIDUAL:
        W = torch.exp(-leaves[-2][k] * D)
        B, n = act.shape
        out = out + (W @ uh.transpose(0, 1).reshape(n, 3 * B)).view(n, B, 3).transpose(0, 1)
    if mode != DECAY:
        (W1, b1), (W2, b2), (W3, b3), (W4, b4), (W5, b5) = _unpack(leaves[-1], LAYERS)
        geo = torch.cat([pos - torch.as_tensor(M.origin[k].astype(np.float64), device=dev),
                         torch.as_tensor(M.nrm[:, sl].T.astype(np.float64), device=dev)], -1)
        x = torch.cat([geo.expand(len(act), *geo.shape), uh], -1)
        f = torch.relu(torch.relu(x @ W1.T + b1) @ W2.T + b2)
        g = torch.relu(f.max(1).values @ W3.T + b3)
        h = torch.relu(f @ W4[:, :64].T + (g @ W4[:, 64:].T + b4)[:, None])
        out = out + h @ W5.T + b5
    return torch.where(act[..., None], uh, out)


def exact(case, seed):
    s = _inputs(case, seed)
    M, E, kind, back = s.M, case["envs"], case["kind"], case["back"]
    dev = s.alpha.device
    src = [s.scene[3], s.scene[4]] + ([s.lrot, s.ltrans] if M.hand else []) + [s.alpha, s.phi]
    leaves = [x.detach().double().requires_grad_(back) for x in src]
    u = torch.zeros((3, E, M.N), dtype=torch.float64, device=dev)
    touch = torch.zeros((E, M.K), dtype=torch.int64, device=dev)
    taxels = torch.zeros((E, M.K, 8), dtype=torch.float64, device=dev)
    for k in range(M.K):
        sl = slice(int(M.offset[k]), int(M.offset[k + 1]))
        pos, nrm = (torch.as_tensor(a[:, sl].T.astype(np.float64), device=dev) for a in (M.pos, M.nrm))
        n = pos.shape[0]
        D = sum((c[:, None] - c) ** 2 for c in pos.T).sqrt_() if kind != "contact" else None
        for env in torch.arange(E, device=dev).split(max(1, (1 << 19) // n)):
            with torch.no_grad():   # rows without contact stay zero
                act = _contact(s, k, env, leaves, pos, nrm)[0]
            live = env[act.any(1)]
            if kind == "taxels":
                taxels[env, k] = _taxels(s, k, torch.zeros((1, n, 3), dtype=torch.float64, device=dev), pos)
            for part in live.split(max(1, (1 << 18) // n)) if len(live) else ():
                act, uh, win = _contact(s, k, part, leaves, pos, nrm)
                if kind == "contact":
                    U = torch.where(act[..., None], uh, 0.0)
                else:
                    U = _field(s, k, act, uh, leaves, case["mode"], D)
                if back:
                    g = s.gu[:, part, sl].permute(1, 2, 0).double()
                    (U * g).sum().backward()
                u[:, part, sl] = U.detach().permute(2, 0, 1)
                touch[part, k] = (act & (win < s.scene[1].shape[1])).sum(1)
                if kind == "taxels":
                    taxels[part, k] = _taxels(s, k, U, pos)
    if kind == "taxels":
        return dict(taxels=taxels)
    out = dict(u=u, cobj=None, na=None)
    if back:
        grads = [torch.zeros_like(x) if x.grad is None else x.grad for x in leaves]
        out.update(zip(GRASP_NAMES if M.hand else NAMES, grads))
    if M.hand:
        na = touch.sum(1).double()
        r = torch.where(na > 0, na / M.N, -0.1)
        out["r"] = (touch > 0).sum(1).double() / M.hand.n_links + r
    return out


def _taxels(s, k, U, pos):
    (E1, e1), (E2, e2), (E3, e3), (A1, a1), (a2, _), (D1, d1), (D2, d2) = _unpack(s.reg.double(), HEAD)
    geo = pos - torch.as_tensor(s.M.origin[k].astype(np.float64), device=pos.device)
    out = []
    for v in U.split(max(1, (1 << 17) // pos.shape[0])):
        x = torch.cat([geo.expand(len(v), *geo.shape), v], -1)
        h = torch.relu(x @ E1.T + e1)
        h = torch.relu(h @ E2.T + e2) + h
        f = torch.relu(h @ E3.T + e3)
        w = torch.softmax(torch.tanh(f @ A1.T + a1) @ a2[0], -1)
        g = (w[..., None] * f).sum(1)
        out.append(torch.relu(g @ D1.T + d1) @ D2.T + d2)
    return torch.cat(out)
